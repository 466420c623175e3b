// Which layer-steps stream their experts by whole rows (stream_gemm.hip), and how a row is laid over lanes (host code without HIP,
// so that the lines can be checked on the CPU).
#pragma once

#include <cstdint>

namespace wisp {

// A row of 16-byte chunks: lpr lanes, nl chunks per lane, kw waves (long rows).
struct StreamLanes { int lpr, nl, kw; };

// The lanes, chunks per lane and waves with the least padding (whole lines of a row per load), or false if they would read
// more than a quarter for nothing.
constexpr StreamLanes kStreamLanes[] = {{64, 1, 1}, {64, 2, 1}, {64, 3, 1}, {64, 4, 1}, {64, 5, 1}, {64, 6, 1}, {64, 7, 1},
                                        {64, 8, 1}, {32, 1, 1}, {32, 3, 1}, {32, 5, 1}, {16, 1, 1}, {16, 3, 1}, {64, 3, 4},
                                        {64, 4, 4}, {64, 5, 4}, {64, 6, 4}, {64, 7, 4}, {64, 8, 4}};
inline bool stream_lanes(int chunks, StreamLanes* o) {
  int best = 0;
  for (const StreamLanes& s : kStreamLanes) {
    const int pad = s.lpr * s.nl * s.kw;
    if (pad >= chunks && (s.kw == 1 || chunks > 512) && (!best || pad < best)) {
      best = pad;
      *o = s;
    }
  }
  return best > 0 && 4 * best <= 5 * chunks;
}
// (d and I: the widths; elem: bytes of a weight)
inline bool stream_widths(int d, int I, int elem) {
  StreamLanes s{};
  return stream_lanes(d * elem / 16, &s) && stream_lanes(I * elem / 16, &s);
}

constexpr int kStreamMaxTokens = 15;

// Up to 15 tokens (the alternative is the per-item kernels): fp8 weights, and bf16 from two tokens (one token has the
// single-token kernels), in layers whose experts are large.  A wave goes through its token rows one after the other, each a
// round trip for its inputs and a sum over the lanes: the weight stream has to be long against that.  Rows of one chunk
// per lane never are (a sum over the lanes for every chunk), rows of two need 1.5 M weights a matrix, longer ones 1 M; 1.2 M
// and 0.45 M where the per-item kernels read a row with eight lanes only (an odd number of 128 bytes).
// us per launch pair, gate/up + down, streamed against per item.  Stream: fp8, one token (9 experts, d 7168, I 2048) 66.8
// against 94.1; bf16, d 2048, I 768, seven tokens of 50 experts 71.6 against 92, two tokens of 8 19.4 against 18.8; 16 experts
// by two rows: d 1024, I 1536 30.0 against 33.8; d 1536, I 768 22.2 against 25.2; d 1472, I 704 20.9 against 22.7; fp8, d 2048,
// I 768 25.7 against 30.1.  Per item: d 1024, I 1024 25.7 against 27.6 there, but 30.7 against 20.8 with four experts by eight
// rows; d 512, I 512 20.3 against 13.9 and 44 against 14; fp8, d 1024, I 512 22.1 against 19.8 and 51 against 16.
inline bool stream_few_tokens(int d, int I, int elem, int T) {
  StreamLanes up{};
  if (T < (elem == 1 ? 1 : 2) || T > kStreamMaxTokens || !stream_widths(d, I, elem) || !stream_lanes(d * elem / 16, &up)) return false;
  const int64_t n = static_cast<int64_t>(d) * I;
  const bool eight_lanes = d * elem / 16 % 16 != 0;
  if (up.nl == 1) return false;
  return n >= (up.nl == 2 ? (eight_lanes ? 1200000 : 1500000) : (eight_lanes ? 450000 : 1000000));
}

// Token batches of bf16 layers (the alternative is a grouped GEMM, whose time hardly depends on the rows while they fit its
// tiles): rows, over all experts of the layer-step that have any (used of them; a shared expert counts), at most c of them per
// expert.  A row costs a sum over the lanes beside its products: the shorter the weight rows the sooner it outweighs the faster
// stream; rows of more than five chunks per lane or of four waves run fewer waves at once.  tiles: the column tiles of
// the grouped launch, kStreamChip of which run at a time (0: a form whose last round does not show); a last round that is not
// full counts for the stream.  An expert of more than kStreamRows rows is read again for the next ones, which costs about as much
// as four rows (64 experts of eight rows 138 us, of ten 195).  us per launch pair, streamed against grouped, in the order of c: d 512, I 512, 128 experts
// by one / two rows 42 / 56 against 46 / 47; d 1024, I 1024, 128 by 3 / 4 137 / 157 against 146; d 1024, I 2816, 64 by 4 / 5
// 207 / 232 against 204, 16 by 4 / 5 / 8 59 / 66 / 88 against 84; d 3072, I 1024, 64 by 3 / 4 196 / 222 against 212; d 5120, I 8192, 16
// by 4 / 5 711 / 797 against 738; d 4096, I 14336, 8 by 4 / 5 490 / 537 against 556, 16 by 4 / 5 982 / 1081 against 958; d 2048,
// I 768, 128 by 4 / 5 193 / 214 against 223, 64 by 6 / 8 122 / 138 against 133, 32 by 4 / 5 56 / 61 against 57, 16 by 32 119 against 53;
// d 768, I 768, 128 by 5 86 against 96; d 1472, I 704 with a shared expert, 60 by 4 / 5 79 / 86 against 79.  fp8 rows cost the
// conversion of every code each: 597 against 560 at two rows already (64 experts, d 7168).
constexpr int kStreamChip = 256;
constexpr int kStreamRows = 8;   // token rows of an expert that a launch takes with one read of its weights (an item)
inline bool stream_batch(int d, int I, int elem, int64_t rows, int64_t used, int64_t items, int64_t tiles) {
  StreamLanes up{}, dn{};
  if (elem != 2 || !stream_lanes(d * elem / 16, &up) || !stream_lanes(I * elem / 16, &dn)) return false;
  const int c2 = up.nl == 1 ? 0 : up.kw > 1 ? 8 : up.nl == 2 ? (dn.nl <= 2 ? 6 : 8) : up.nl <= 5 ? 11 : up.nl <= 7 ? 8 : 10;   // 2 c
  rows += 4 * (items - used);
  if (tiles <= kStreamChip) return 2 * rows <= c2 * used;
  const int64_t rounds = (tiles + kStreamChip - 1) / kStreamChip;
  return 2 * rows * tiles <= c2 * used * rounds * kStreamChip;
}

}  // namespace wisp
