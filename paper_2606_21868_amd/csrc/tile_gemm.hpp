// Grouped GEMMs of a token batch for fp8 or bf16 weights of any supported width, with or without a shared
// expert: per expert, H = silu(X W1^T) * (X W3^T) (gate/up) and O = H W2^T (down), on
// v_mfma_f32_16x16x32_bf16 with the token rows as the A operand.
//
// What bounds it: HBM, at the 20 to 130 rows an expert has in a prompt (38 rows per fp8 expert: 60 FLOP per
// byte against a ridge near 250).  So every weight byte is read once per row block, straight into the registers of
// the one wave that uses it, and everything else is arranged around that stream:
//  - A wave owns 16 h columns (16 rows of W1 and the same 16 of W3, so SwiGLU is applied in registers) or
//    32 output columns (W2 rows; its two blocks are the even and the odd columns, so a lane's two results
//    are neighbours) for all token rows of the row block: fp8 codes are converted (exactly) once, and the
//    work of the waves is equal however many rows the block has.
//  - A stage is 128 bytes of every weight row.  Its token rows go through an LDS ring shared by the waves
//    (buffer-to-LDS loads, chunk-swizzled rows), both kTB - 1 stages ahead; one barrier per stage.
//  - Persistent workgroups walk tiles as one sequence of stages; the next tile's loads are in flight while
//    the current one ends.
//  - fp8: a stage is one 128-column scale block, so its products are summed from zero and multiplied by the
//    block's scale in fp32 into the accumulator, as scale * sum(code * x) requires.
// Every output is one fixed chain over K, whatever tile, row block or launch holds its row, so paged and
// resident runs give the same bits.
//
// Measured (64 fp8 experts + shared, d 7168, I 2048, 301 tokens): gate/up 461 us, down 254 us, against 5.30
// and 3.26 ms of the per-item kernels.  With work taken out (scratch copies of an earlier 510 / 252 us build): no
// MFMAs and LDS reads 447 / 233 us, no token rows 464 / 237, the weight stream alone 396 / 219 (4.8 TB/s;
// 369 us of gate/up's 475 once the last round of tiles was dealt over the XCDs).  Strided rows stream
// at 5.1-5.7 TB/s here, a plain read at 7.0.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "kernels.hpp"

namespace wisp {
namespace tile {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));   // a plain vector: stays in registers
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr uint32_t kOutOfRange = 0x80000000u;   // a byte offset past every resource below 2 GiB
constexpr int MODE_UP = 0, MODE_DN = 1;
constexpr int kTB = 4;                          // ring slots; loads run kTB - 1 stages ahead
constexpr int kTD = kTB - 1;

__device__ __forceinline__ uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// s_waitcnt immediates (gfx9 encoding): vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8
constexpr int vmcnt_only(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8); }
constexpr int vmcnt_lgkm0(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4); }

// chunk swizzle of row r of a 128-byte-row LDS tile: rows r .. r + 7 take distinct positions for one
// chunk, and so do the pairs (r & 1, position) of rows r .. r + 15
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// One int32 per lane, by inline asm like the weights (waited for by count, then pinned).
__device__ __forceinline__ int32_t load_i32(const int32_t* p) {
  int32_t v;
  asm volatile("global_load_dword %0, %1, off" : "=&v"(v) : "v"(p) : "memory");
  return v;
}
__device__ __forceinline__ void pin_i32(int32_t& v) { asm volatile("; pin %0" : "+v"(v)); }
__device__ __forceinline__ void lds_write_i32(uint32_t addr, int32_t v) {
  asm volatile("ds_write_b32 %0, %1" : : "v"(addr), "v"(v) : "memory");
}
__device__ __forceinline__ u32x4_t lds_read_4(uint32_t addr) {
  u32x4_t v;
  asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)\n\t; pin %0" : "=&v"(v) : "v"(addr) : "memory");
  return v;
}
// Four fragments of a batch of slabs: a0, a1 and the same DELTA bytes further, read by inline ds_reads (the compiler
// would make plain LDS reads wait for every buffer-to-LDS load in flight).  A batch's reads go out before the
// batch ahead of it is used: read_next issues them and waits for the batch before (LDS reads return in order),
// whose registers the compiler reads only after that; read_last waits for the last.  One wait per batch for its
// own reads took 733 us per fp8 layer pass where this takes 720 (301 tokens, the shape above), 1828 against 1670 (1100).
template <int DELTA>
__device__ __forceinline__ void read_first(u32x4_t (&f)[4], uint32_t a0, uint32_t a1) {
  asm volatile(
      "ds_read_b128 %0, %4\n\t"
      "ds_read_b128 %1, %5\n\t"
      "ds_read_b128 %2, %4 offset:%6\n\t"
      "ds_read_b128 %3, %5 offset:%6"
      : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3])
      : "v"(a0), "v"(a1), "i"(DELTA)
      : "memory");
}
template <int DELTA>
__device__ __forceinline__ void read_next(u32x4_t (&f)[4], u32x4_t (&n)[4], uint32_t a0, uint32_t a1) {
  asm volatile(
      "ds_read_b128 %4, %8\n\t"
      "ds_read_b128 %5, %9\n\t"
      "ds_read_b128 %6, %8 offset:%10\n\t"
      "ds_read_b128 %7, %9 offset:%10\n\t"
      "s_waitcnt lgkmcnt(4)\n\t"
      "; pin %0 %1 %2 %3"
      : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "=&v"(n[0]), "=&v"(n[1]), "=&v"(n[2]), "=&v"(n[3])
      : "v"(a0), "v"(a1), "i"(DELTA)
      : "memory");
}
__device__ __forceinline__ void read_last(u32x4_t (&f)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)\n\t; pin %0 %1 %2 %3" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]) : : "memory");
}
// 16 E4M3 codes to bf16 (exact): the first and the last eight
__device__ __forceinline__ void fp8_to_bf16(u32x4_t v, bf16x8_t& lo, bf16x8_t& hi) {
  bf16x2_t p[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[2 * i] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[i], 1.0f, false);
    p[2 * i + 1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(v[i], 1.0f, true);
  }
  lo = bf16x8_t{p[0][0], p[0][1], p[1][0], p[1][1], p[2][0], p[2][1], p[3][0], p[3][1]};
  hi = bf16x8_t{p[4][0], p[4][1], p[5][0], p[5][1], p[6][0], p[6][1], p[7][0], p[7][1]};
}
// One stage's weights of a wave: 128 bytes of its 16 rows of each block (two 16-byte loads per lane and
// block), by inline asm that the compiler neither counts nor waits for: the caller waits by count and then
// passes the registers through pin_w, after which the compiler reads them.
__device__ __forceinline__ void load_w(u32x4_t (&w)[2][2], u32x4_t rs, uint32_t v0, uint32_t v1, uint32_t soff) {
  asm volatile(
      "buffer_load_dwordx4 %0, %4, %6, %7 offen\n\t"
      "buffer_load_dwordx4 %1, %4, %6, %7 offen offset:64\n\t"
      "buffer_load_dwordx4 %2, %5, %6, %7 offen\n\t"
      "buffer_load_dwordx4 %3, %5, %6, %7 offen offset:64"
      : "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(w[1][0]), "=&v"(w[1][1])
      : "v"(v0), "v"(v1), "s"(rs), "s"(soff)
      : "memory");
}
// ... and the two blocks' scales of the stage's 128 columns (fp8)
__device__ __forceinline__ void load_s(uint32_t (&s)[2], u32x4_t rs, uint32_t v0, uint32_t v1, uint32_t soff) {
  asm volatile(
      "buffer_load_ushort %0, %2, %4, %5 offen\n\t"
      "buffer_load_ushort %1, %3, %4, %5 offen"
      : "=&v"(s[0]), "=&v"(s[1])
      : "v"(v0), "v"(v1), "s"(rs), "s"(soff)
      : "memory");
}
__device__ __forceinline__ void pin_w(u32x4_t (&w)[2][2]) {
  asm volatile("; pin %0 %1 %2 %3" : "+v"(w[0][0]), "+v"(w[0][1]), "+v"(w[1][0]), "+v"(w[1][1]));
}
__device__ __forceinline__ void pin_s(uint32_t (&s)[2]) { asm volatile("; pin %0 %1" : "+v"(s[0]), "+v"(s[1])); }
// raw buffer resource words (stride 0) over [p, p + bytes), as uniform values
__device__ __forceinline__ u32x4_t rsrc_words(const void* p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  u32x4_t r;
  r.x = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
  r.y = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32) & 0xFFFFu);
  r.z = __builtin_amdgcn_readfirstlane(bytes);
  r.w = 0x00020000u;
  return r;
}
// WT weights, NW waves, RB token rows per row block.
template <int WT, int MODE, int NW, int RB>
__device__ __forceinline__ void tile_body(const GroupedBatch& gb, const uint16_t* __restrict__ a_src, uint32_t a_bytes,
                                          const int32_t* __restrict__ perm, int k, int d, int I, uint32_t off0,
                                          uint32_t off1, uint32_t soff0, uint32_t soff1, uint32_t w_bytes,
                                          void* __restrict__ out) {
  constexpr int WB = WT == DT_BF16 ? 2 : 1;       // bytes per weight
  constexpr int KS = 128 / WB;                    // K per stage: 128 bytes of every weight row
  constexpr int SUB = KS / 64;                    // 64-column halves of a stage's token rows
  constexpr int ASLOT = RB * KS * 2;              // bytes of the token rows of a stage
  constexpr int AI = ASLOT / 1024 / NW;           // buffer-to-LDS loads per wave per stage
  constexpr int LD = WT == DT_BF16 ? 4 : 6;       // weight (and scale) loads per wave per stage
  constexpr int NSL = RB / 16;                    // 16-row slabs of the row block
  constexpr int SB = WT == DT_BF16 ? 2 : 1;       // slabs per batch of fragment reads
  constexpr int CW = MODE == MODE_UP ? 16 : 32;   // output columns per wave
  constexpr int CT = NW * CW;
  constexpr int RW = RB / NW;                     // token rows a wave stages
  static_assert(ASLOT % (1024 * NW) == 0 && NSL % SB == 0 && RW <= 64 && RW % 8 == 0, "");
  __shared__ __attribute__((aligned(1024))) uint8_t ring[kTB * ASLOT];
  __shared__ int32_t otab[MODE == MODE_DN ? 8 * RB : 1];   // output rows of the tiles in flight
  const int K = MODE == MODE_UP ? d : I;
  const int cols = MODE == MODE_UP ? I : d;
  const int spt = K / KS;
  const int n_ct = (cols + CT - 1) / CT;
  const int n_tiles = gb.tile_end[gb.n_groups - 1] * n_ct;
  const int G = static_cast<int>(gridDim.x);
  const int xcd = static_cast<int>(blockIdx.x) % 8, jx = static_cast<int>(blockIdx.x) / 8;
  // XCD-aware: workgroups are dealt to the 8 XCDs round-robin; in a full round the workgroups of one XCD take
  // consecutive tiles (the column tiles of a few experts, whose token rows then stay in that XCD's L2).  The
  // last, partial round is dealt round-robin instead: the tiles left over would all fall to the first XCDs and wait
  // for their share of the memory system (510 -> 475 us for 2208 tiles over 512
  // workgroups, 66 -> 55 for 704).
  const int L = xcd * (G / 8) + min(xcd, G % 8) + jx;
  const int full = n_tiles / G;
  const int my_tiles = full + (static_cast<int>(blockIdx.x) < n_tiles - full * G ? 1 : 0);
  auto tile_no = [&](int i) __attribute__((always_inline)) { return i * G + (i < full ? L : static_cast<int>(blockIdx.x)); };
  const int nq = my_tiles * spt;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int c = lane & 15, g = lane >> 4;
  const uint32_t wrow = static_cast<uint32_t>(K) * WB, arow = static_cast<uint32_t>(K) * 2;

  struct T { const uint8_t* w; int rows, base, m0, c0, shared; };
  auto decode = [&](int t) __attribute__((always_inline)) -> T {
    const int rb_all = t / n_ct;
    int lo = 0, hi = gb.n_groups - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (rb_all >= gb.tile_end[mid]) lo = mid + 1;
      else hi = mid;
    }
    const int b0 = lo > 0 ? gb.tile_end[lo - 1] : 0, nrb = gb.tile_end[lo] - b0;
    const int local = t - b0 * n_ct, ct = local / nrb, rb = local - ct * nrb;
    return T{gb.w[lo], gb.rows[lo], gb.row_off[lo], rb * RB, ct * CT, lo == gb.shared};
  };

  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr_t)ring));
  const uint32_t otab0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr_t)otab));
  uint32_t fo[2];   // fragment reads: the two 16-byte chunks of a lane in a 64-column half
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int ch = WT == DT_BF16 ? 4 * s + g : 2 * g + s;
    fo[s] = lds0 + c * 128 + ((ch ^ swz(c)) << 4);
  }
  // staging load j of a wave: 8 rows (j % (RW / 8)) of half j / (RW / 8); lane l holds chunk (l & 7) ^ swz(row)
  const int arl = lane >> 3;
  constexpr int AR = RW / 8;

  const __amdgpu_buffer_rsrc_t a_rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a_src), 0, static_cast<int>(a_bytes), 0x00020000);
  u32x4_t w_rs = rsrc_words(a_src, 0);
  uint32_t wvo[2] = {kOutOfRange, kOutOfRange}, svo[2] = {0, 0}, avo[AR];
  // a lane's rows are read through the pair order, loaded a whole tile ahead and waited for by count (all at
  // once where a tile has fewer stages than the count covers)
  const bool short_k = spt < kTD + 2;
  int32_t pn = 0;
  auto pair_of = [&](const T& t) __attribute__((always_inline)) -> int32_t {
    return load_i32(perm + (t.shared ? 0 : t.base) + min(t.m0 + wave * RW + lane % RW, t.rows - 1));
  };
  int is_tile = 0, is_s = 0;
  auto enter_tile = [&](int i) __attribute__((always_inline)) {
    if (i >= my_tiles) {   // past the last tile: loads that touch no memory keep the counts
      w_rs = rsrc_words(a_src, 0);
#pragma unroll
      for (int j = 0; j < AR; ++j) avo[j] = kOutOfRange;
      return;
    }
    const T t = decode(tile_no(i));
    w_rs = rsrc_words(t.w + off0, w_bytes);
    const bool on = t.c0 + wave * CW < cols;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t r = MODE == MODE_UP ? t.c0 + wave * 16 + c : t.c0 + wave * 32 + 2 * c + b;
      const uint32_t o = r * wrow + g * 16 + (MODE == MODE_UP && b ? off1 - off0 : 0u);
      wvo[b] = on ? o : kOutOfRange;
      if constexpr (WT == DT_FP8)
        svo[b] = on ? (b ? soff1 : soff0) - off0 + (t.c0 + wave * CW) / 128 * (K / 128) * 2 : kOutOfRange;
    }
    const int myrow = t.m0 + wave * RW + lane % RW;
    if (short_k) __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
    pin_i32(pn);
    const int tt = t.shared ? myrow : pn / k;   // the token of the lane's row
    int ro = tt;
    if constexpr (MODE == MODE_DN) {
      const int j = t.shared ? k : pn - tt * k;
      lds_write_i32(otab0 + ((i & 7) * RB + wave * RW + lane % RW) * 4, tt * (k + 1) + j);
      ro = t.base + myrow;
    }
#pragma unroll
    for (int j = 0; j < AR; ++j) {
      const int rl = j * 8 + arl;
      const int rr = __shfl(ro, rl, 64);
      avo[j] = t.m0 + wave * RW + rl < t.rows
                   ? static_cast<uint32_t>(rr) * arow + (((lane & 7) ^ swz((wave * RW + rl) & 15)) << 4)
                   : kOutOfRange;
    }
    if (i + 1 < my_tiles) pn = pair_of(decode(tile_no(i + 1)));
  };
  u32x4_t W[kTB][2][2];
  uint32_t S[kTB][2];
  auto issue = [&](int slot, u32x4_t (&w)[2][2], uint32_t (&sc)[2]) __attribute__((always_inline)) {
    if (is_s == 0) enter_tile(is_tile);
    const int sw = __builtin_amdgcn_readfirstlane(is_s * 128), sa = __builtin_amdgcn_readfirstlane(is_s * KS * 2);
    load_w(w, w_rs, wvo[0], wvo[1], sw);
    if constexpr (WT == DT_FP8) load_s(sc, w_rs, svo[0], svo[1], __builtin_amdgcn_readfirstlane(is_s * 2));
#pragma unroll
    for (int h = 0; h < SUB; ++h)
#pragma unroll
      for (int j = 0; j < AR; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            a_rs, (lds_ptr_t)(ring + slot * ASLOT + h * RB * 128 + (wave * AR + j) * 1024), 16, avo[j] + h * 128, sa, 0, 0);
    asm volatile("" ::: "memory");   // the waits count stages: no load moves into another stage
    if (++is_s == spt) {
      is_s = 0;
      ++is_tile;
    }
  };

  f32x4_t acc[2][NSL] = {};
  int cs_tile = 0, cs_s = 0;
  T ct = decode(tile_no(0));
  pn = pair_of(ct);
  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
  auto epilogue = [&]() __attribute__((always_inline)) {
    const int n_rows = min(ct.rows - ct.m0, RB);
    if (ct.c0 + wave * CW >= cols) return;
    if constexpr (MODE == MODE_UP) {
      uint32_t* hs = static_cast<uint32_t*>(out);
      const int colp = (ct.c0 + wave * 16 + (c & ~1)) / 2;
#pragma unroll
      for (int s = 0; s < NSL; ++s) {
        if (s * 16 < n_rows) {
          uint32_t hv[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float a = acc[0][s][i];
            hv[i] = bf16_rne(a / (1.0f + __expf(-a)) * acc[1][s][i]);
          }
          // even lanes take rows i = 0, 2 and odd lanes rows 1, 3, two columns each
#pragma unroll
          for (int i = 0; i < 4; i += 2) {
            const uint32_t o0 = __builtin_amdgcn_mov_dpp(hv[i], 0xB1, 0xF, 0xF, true);
            const uint32_t o1 = __builtin_amdgcn_mov_dpp(hv[i + 1], 0xB1, 0xF, 0xF, true);
            const uint32_t v = (c & 1) ? (o1 | (hv[i + 1] << 16)) : (hv[i] | (o0 << 16));
            const int row = s * 16 + g * 4 + i + (c & 1);
            if (row < n_rows) hs[static_cast<size_t>(ct.base + ct.m0 + row) * (I / 2) + colp] = v;
          }
        }
      }
    } else {
      const int col = ct.c0 + wave * 32 + 2 * c;
#pragma unroll
      for (int s = 0; s < NSL; ++s) {
        if (s * 16 < n_rows) {
          const u32x4_t orow = lds_read_4(otab0 + ((cs_tile & 7) * RB + s * 16 + g * 4) * 4);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (s * 16 + g * 4 + i < n_rows) {
              const size_t o = static_cast<size_t>(orow[i]) * d + col;
              *reinterpret_cast<float2*>(static_cast<float*>(out) + o) = make_float2(acc[0][s][i], acc[1][s][i]);
            }
          }
        }
      }
    }
  };

#pragma unroll
  for (int u = 0; u < kTD; ++u) issue(u, W[u], S[u]);

  auto step = [&](auto U_) __attribute__((always_inline)) {
    constexpr int U = decltype(U_)::value;
    // this stage's own loads have landed: what was issued after them is the loads of the kTD - 1 stages
    // behind it, plus, after a tile's end, its stores (the count then waits a little longer than it must)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "i"((kTD - 1) * (LD + AI)) : "memory");
    __builtin_amdgcn_s_barrier();   // every wave's share landed; every wave is done with the stage before
    asm volatile("" ::: "memory");
    pin_w(W[U]);
    if constexpr (WT == DT_FP8) pin_s(S[U]);
    constexpr int V = (U + kTD) % kTB;
    issue(V, W[V], S[V]);
    const int ns = (min(ct.rows - ct.m0, RB) + 15) >> 4;
    if (ct.c0 + wave * CW < cols) {
      bf16x8_t wf[2][2 * SUB];   // [block][32-column step]
      float sc[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        if constexpr (WT == DT_BF16) {
          wf[b][0] = __builtin_bit_cast(bf16x8_t, W[U][b][0]);
          wf[b][1] = __builtin_bit_cast(bf16x8_t, W[U][b][1]);
        } else {
          fp8_to_bf16(W[U][b][0], wf[b][0], wf[b][1]);
          fp8_to_bf16(W[U][b][1], wf[b][2 * SUB - 2], wf[b][2 * SUB - 1]);
          sc[b] = __uint_as_float(S[U][b] << 16);
        }
      }
      // bf16: steps 0, 1 of slabs sl, sl + 1; fp8: steps 0 .. 3 of slab sl
      constexpr int DELTA = WT == DT_BF16 ? 2048 : RB * 128;
      u32x4_t fr[2][4];
      read_first<DELTA>(fr[0], fo[0] + U * ASLOT, fo[1] + U * ASLOT);
#pragma unroll
      for (int sl = 0; sl < NSL; sl += SB) {
        // read also for slabs past the last row (within the slot, and not used): a branch around the reads
        // would make the compiler copy registers that are still in flight
        u32x4_t(&f)[4] = fr[(sl / SB) & 1];
        if (sl + SB < NSL)
          read_next<DELTA>(f, fr[(sl / SB + 1) & 1], fo[0] + U * ASLOT + (sl + SB) * 2048, fo[1] + U * ASLOT + (sl + SB) * 2048);
        else
          read_last(f);
        if (sl < ns) {
          if constexpr (WT == DT_BF16) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
              for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                  acc[b][sl + x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f[2 * x + s]),
                                                                          wf[b][s], acc[b][sl + x], 0, 0, 0);
          } else {
            f32x4_t P[2] = {};
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int b = 0; b < 2; ++b)
                P[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f[s]), wf[b][s], P[b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[b][sl][i] = fmaf(sc[b], P[b][i], acc[b][sl][i]);
          }
        }
      }
    }
    if (++cs_s == spt) {
      epilogue();
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int s = 0; s < NSL; ++s) acc[b][s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      cs_s = 0;
      if (++cs_tile < my_tiles) ct = decode(tile_no(cs_tile));
    }
  };
  // the loop is unrolled over the ring, so that slots and register sets have fixed indices.  Each way out
  // ends the program there: an exit that met the loop's end again would make the compiler's own waits
  // strict (it would count the loads of steps that did not run).
  static_assert(kTB == 4, "one step per ring slot below");
  auto end_if = [&](bool done) __attribute__((always_inline)) {
    if (done) {
      __builtin_amdgcn_s_waitcnt(vmcnt_only(0));   // the last staging loads write LDS: none may outlive the workgroup
      __builtin_amdgcn_endpgm();
    }
  };
  for (int q = 0;; q += kTB) {
    end_if(q >= nq);
    step(std::integral_constant<int, 0>{});
    end_if(q + 1 >= nq);
    step(std::integral_constant<int, 1>{});
    end_if(q + 2 >= nq);
    step(std::integral_constant<int, 2>{});
    end_if(q + 3 >= nq);
    step(std::integral_constant<int, 3>{});
  }
}
}  // namespace tile
}  // namespace wisp
