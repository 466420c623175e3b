// Expert FFN of a few tokens per expert (a decode batch, a short prompt): every expert's weights are
// streamed once for all the token rows that use it (gfx950).
//
// What bounds it: HBM.  With one to a few rows per expert the work is the weight stream of a GEMV, and how fast
// that stream runs depends on how it is read.  At 50 experts of 2 x 768 rows of 4 KB (315 MB): in the matrix
// cores' operand layout (16 rows x 64 bytes per load) 54 us, 61 with non-temporal loads (the second half of a
// line is fetched again); one contiguous kilobyte of a row per load 46 us, 6.8 TB/s.  So a wave reads whole
// rows: LPR lanes per row, lane l the 16-byte chunks l, l + LPR, ...; it takes RP rows of W1 and the same of
// W3 (gate/up) or RP rows of W2 (down) at once, about 16 loads in flight per lane, issued before anything
// else, and holds them in registers while it goes through the expert's token rows.  A token costs 4
// v_dot2_f32_bf16 per chunk (8 with fp8: codes converted exactly to bf16, pairs summed in fp32, times
// the chunk's block scale in fp32) and a butterfly over the lanes that halves the values as it goes.  No LDS and no
// barrier, except where four waves share a row: their sums of a token meet in LDS.  A launch takes up to 224 items.
// Token rows go one after the other, each a round trip for its inputs: which layers and batches stream is stream_rules.hpp's.  A row's chain depends on the shape alone, so a result has the same bits
// whichever launch holds its expert.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "blob_copy.hpp"
#include "stream_rules.hpp"
#include "tile_gemm.hpp"

namespace wisp {
namespace {

using tile::bf16x2_t;
using tile::u32x4_t;
using tile::MODE_DN;
using tile::MODE_UP;

__device__ __forceinline__ float dot2(uint32_t w, uint32_t x, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w), __builtin_bit_cast(bf16x2_t, x), acc, false);
}

// one 16-byte weight chunk times the matching inputs (8 bf16, or 16 for 16 fp8 codes of one scale block)
template <int WT>
__device__ __forceinline__ float chunk_dot(u32x4_t w, const u32x4_t* x, float scale, float acc) {
  if constexpr (WT == DT_BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = dot2(w[i], x[0][i], acc);
    return acc;
  } else {
    float p = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p = dot2(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[i], 1.0f, false)), x[i / 2][2 * (i % 2)], p);
      p = dot2(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[i], 1.0f, true)), x[i / 2][2 * (i % 2) + 1], p);
    }
    return fmaf(scale, p, acc);
  }
}

// Where an item's token rows come from: the launch's argument (pairs packed in it, pairs of the device's sorted
// order, or tokens of the shared expert) or a plan in HBM.
struct ArgRows {
  const StreamBatch& b;
  const int32_t* perm;
  int item, k;
  __device__ int n() const { return b.rows[item]; }
  __device__ void row(int i, int* tok, int* orow) const {
    const uint64_t at = b.at[item];
    if (!perm) {
      *tok = static_cast<int>(at >> (4 * i)) & 15;
      *orow = *tok * (k + 1) + (static_cast<int>(at >> (32 + 4 * i)) & 15);
    } else if (at & kStreamShared) {
      *tok = static_cast<int>(at & 0xFFFFFFFFu) + i;
      *orow = *tok * (k + 1) + k;
    } else {
      const int pr = __builtin_amdgcn_readfirstlane(perm[static_cast<int>(at) + i]);
      *tok = pr / k;
      *orow = pr + *tok;   // t (k + 1) + j
    }
  }
};
struct PlanRows {
  const FfnItem& it;
  __device__ int n() const { return it.ntok; }
  __device__ void row(int i, int* tok, int* orow) const {
    *tok = it.tok[i];
    *orow = it.out[i];
  }
};

// One wave's rows of an item: LPR lanes per row, NL chunks per lane, RP row slots (a slot is the 64 / LPR rows of
// one load), KW waves of the workgroup sharing a row's K (1, or 4 for rows too long for one wave's
// registers).  row0: the lane's row in slot 0.  Weights and scales are read from the blob at w; if wr is not
// null every chunk is also stored at the same place there (a faulted expert streamed from its host master into
// its slot while being used).
template <int WT, int MODE, int LPR, int NL, int RP, int KW, bool FILL, typename Rows>
__device__ __forceinline__ void stream_rows(const uint8_t* w, uint8_t* wr, const Rows& R, int row0, int sl, int wave,
                                            const uint8_t* __restrict__ vin, int d, int I, uint32_t off0, uint32_t off1,
                                            uint32_t soff0, uint32_t soff1, int bf16_out, void* __restrict__ out) {
  constexpr int G = 64 / LPR;
  constexpr int NM = MODE == MODE_UP ? 2 : 1;     // matrices
  constexpr int V = NM * RP;                      // sums per lane and token
  constexpr int XS = WT == DT_BF16 ? 1 : 2;       // 16-byte input chunks per weight chunk
  constexpr int WB = WT == DT_BF16 ? 2 : 1;       // bytes per weight
  constexpr bool FP8 = WT == DT_FP8;
  static_assert((V & (V - 1)) == 0 && V <= LPR, "the butterfly halves the sums");
  __shared__ float part[2][4][KW > 1 ? V : 1];    // KW > 1: the waves' sums of one token
  const int K = MODE == MODE_UP ? d : I;
  const int chunks = K * WB / 16;
  // a chunk past the row's end (where the lanes do not divide the row) repeats the row's last chunk; its inputs and its
  // weights (fp8, whose codes are finite: its scale) are then replaced by zeros, both, as an infinite weight times a zero
  // input is no number
  const int c0 = (wave % KW) * (NL * LPR) + sl;
  int ci[NL];
#pragma unroll
  for (int m = 0; m < NL; ++m) ci[m] = min(c0 + m * LPR, chunks - 1);
  u32x4_t wv[NM][RP][NL];
  uint32_t sv[NM][FP8 ? RP : 1];
#pragma unroll
  for (int p = 0; p < RP; ++p)
#pragma unroll
    for (int q = 0; q < NM; ++q) {
      const u32x4_t* row = reinterpret_cast<const u32x4_t*>(w + (q ? off1 : off0) + static_cast<size_t>(row0 + p * G) * K * WB);
#pragma unroll
      for (int m = 0; m < NL; ++m) wv[q][p][m] = __builtin_nontemporal_load(row + ci[m]);
    }
  if constexpr (FP8) {   // lane sl holds scale sl of the row's part (at most 8 NL LPR / 64 blocks), shuffled out per chunk
#pragma unroll
    for (int p = 0; p < RP; ++p)
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const uint16_t* sc = reinterpret_cast<const uint16_t*>(w + (q ? soff1 : soff0)) + static_cast<size_t>((row0 + p * G) / 128) * (K / 128);
        sv[q][p] = sc[min((wave % KW) * (NL * LPR / 8) + sl, K / 128 - 1)];
      }
  }
  const int rows = R.n();
  for (int i = 0; i < rows; ++i) {
    int tok, orow;
    R.row(i, &tok, &orow);
    const u32x4_t* xp = reinterpret_cast<const u32x4_t*>(vin + static_cast<size_t>(MODE == MODE_UP ? tok : orow) * K * 2);
    float v[V];
#pragma unroll
    for (int j = 0; j < V; ++j) v[j] = 0.f;
    u32x4_t x[NL][XS];
#pragma unroll
    for (int m = 0; m < NL; ++m)
#pragma unroll
      for (int s = 0; s < XS; ++s) x[m][s] = xp[ci[m] * XS + s];
    if constexpr (FILL) {
      if (i == 0) {
#pragma unroll
        for (int p = 0; p < RP; ++p)
#pragma unroll
          for (int q = 0; q < NM; ++q) {
            u32x4_t* dst = reinterpret_cast<u32x4_t*>(wr + (q ? off1 : off0) + static_cast<size_t>(row0 + p * G) * K * WB);
#pragma unroll
            for (int m = 0; m < NL; ++m) dst[ci[m]] = wv[q][p][m];
          }
      }
    }
    if (chunks != KW * NL * LPR) {
      if (!FP8 && i == 0) {   // once, with the first row's inputs on their way too
#pragma unroll
        for (int m = KW > 1 ? 0 : NL - 1; m < NL; ++m)
#pragma unroll
          for (int q = 0; q < NM; ++q)
#pragma unroll
            for (int p = 0; p < RP; ++p)
              if (c0 + m * LPR >= chunks) wv[q][p][m] = u32x4_t{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int m = KW > 1 ? 0 : NL - 1; m < NL; ++m)
#pragma unroll
        for (int s = 0; s < XS; ++s)
          if (c0 + m * LPR >= chunks) x[m][s] = u32x4_t{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int m = 0; m < NL; ++m)
#pragma unroll
      for (int q = 0; q < NM; ++q)
#pragma unroll
        for (int p = 0; p < RP; ++p) {
          float s = 1.f;
          if constexpr (FP8) {
            // the codes are converted anew for every token: converted once, ahead of the loop (as the compiler
            // would), they take twice the registers and a wave per SIMD (57 us a launch instead of 43)
            asm volatile("" : "+v"(wv[q][p][m]));
            s = __uint_as_float(static_cast<uint32_t>(__shfl(static_cast<int>(sv[q][p]), m * (LPR / 8) + sl / 8, LPR)) << 16);
            if ((KW > 1 || m == NL - 1) && c0 + m * LPR >= chunks) s = 0.f;
          }
          v[q * RP + p] = chunk_dot<WT>(wv[q][p][m], x[m], s, v[q * RP + p]);
        }
    // sum over the row's LPR lanes: each step adds across half the lanes and leaves every lane half the sums
    int off = LPR / 2;
#pragma unroll
    for (int n = V; n > 1; n >>= 1, off >>= 1) {
      const bool hi = sl & off;
#pragma unroll
      for (int j = 0; j < n / 2; ++j) {
        const float keep = hi ? v[j + n / 2] : v[j], send = hi ? v[j] : v[j + n / 2];
        v[j] = keep + __shfl_xor(send, off, 64);
      }
    }
#pragma unroll
    for (; off > 0; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
    // the lane holds sum number sl / (LPR / V): the matrix in its top bit, then the slot
    const int q = sl / (LPR / V), p = q % RP;
    if constexpr (KW > 1) {   // the waves' sums in wave order
      if (sl % (LPR / V) == 0) part[i & 1][wave][q] = v[0];
      __syncthreads();
      float a = part[i & 1][0][q];
#pragma unroll
      for (int z = 1; z < KW; ++z) a += part[i & 1][z][q];
      v[0] = a;
      if (wave != 0) continue;
    }
    const size_t o = static_cast<size_t>(orow) * (MODE == MODE_UP ? I : d) + row0 + p * G;
    if constexpr (MODE == MODE_UP) {
      const float u = __shfl_xor(v[0], LPR / 2, 64);
      if (q < RP && sl % (LPR / V) == 0)
        static_cast<uint16_t*>(out)[o] = tile::bf16_rne(v[0] / (1.0f + __expf(-v[0])) * u);
    } else if (sl % (LPR / V) == 0) {
      if (bf16_out) static_cast<uint16_t*>(out)[o] = tile::bf16_rne(v[0]);
      else static_cast<float*>(out)[o] = v[0];
    }
  }
}

// Host-planned: grid (row blocks, items).
template <int WT, int MODE, int LPR, int NL, int RP, int KW>
__global__ void __launch_bounds__(256) stream_kernel(const StreamBatch B, const uint8_t* __restrict__ vin,
                                                     const int32_t* __restrict__ perm, int k, int d, int I,
                                                     uint32_t off0, uint32_t off1, uint32_t soff0, uint32_t soff1,
                                                     int bf16_out, void* __restrict__ out) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, sub = lane / LPR, sl = lane - sub * LPR;
  const int item = blockIdx.y;
  const int row0 = (static_cast<int>(blockIdx.x) * (4 / KW) + wave / KW) * (64 / LPR * RP) + sub;
  stream_rows<WT, MODE, LPR, NL, RP, KW, false>(B.w[item], nullptr, ArgRows{B, perm, item, k}, row0, sl, wave, vin, d,
                                                I, off0, off1, soff0, soff1, bf16_out, out);
}

// Device-planned gate/up (the plan the device pager of this layer wrote to HBM): grid (workgroups, item slots).  A
// resident expert takes a workgroup per row block; a faulted one fault_wgs that stream its W1 / W3 rows from
// the host master (computing and filling the slot) and copy_wgs that copy the rest of its blob.
template <int WT, int LPR, int NL, int RP>
__global__ void __launch_bounds__(256) stream_gateup_dev(const FfnBatch* __restrict__ P, const uint8_t* __restrict__ vin,
                                                         int d, int I, int fault_wgs, int copy_wgs, uint32_t off0,
                                                         uint32_t off1, uint32_t soff0, uint32_t soff1,
                                                         uint32_t copy_off, uint32_t copy_bytes,
                                                         uint16_t* __restrict__ h) {
  const int j = blockIdx.x;
  if (static_cast<int>(blockIdx.y) >= P->n_items) return;
  const FfnItem& it = P->items[blockIdx.y];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, sub = lane / LPR, sl = lane - sub * LPR;
  constexpr int R = 4 * (64 / LPR) * RP;   // rows of a workgroup's pass
  const int blocks = I / R;
  const int r = wave * (64 / LPR * RP) + sub;
  if (!it.fault) {
    if (j < blocks)
      stream_rows<WT, MODE_UP, LPR, NL, RP, 1, false>(it.w, nullptr, PlanRows{it}, j * R + r, sl, wave, vin, d, I, off0,
                                                      off1, soff0, soff1, 0, h);
  } else if (j < fault_wgs) {
    const int per = (blocks + fault_wgs - 1) / fault_wgs;
    for (int b = j * per; b < min(blocks, (j + 1) * per); ++b)
      stream_rows<WT, MODE_UP, LPR, NL, RP, 1, true>(it.src, const_cast<uint8_t*>(it.w), PlanRows{it}, b * R + r, sl,
                                                     wave, vin, d, I, off0, off1, soff0, soff1, 0, h);
  } else if (j < fault_wgs + copy_wgs) {
    copy_share(it.src, const_cast<uint8_t*>(it.w), copy_off, copy_bytes, j - fault_wgs, copy_wgs);
  }
}

// Device-planned down: every expert of the step is resident by now.
template <int WT, int LPR, int NL, int RP>
__global__ void __launch_bounds__(256) stream_down_dev(const FfnBatch* __restrict__ P, const uint8_t* __restrict__ h,
                                                       int d, int I, uint32_t off0, uint32_t soff0,
                                                       float* __restrict__ buf) {
  if (static_cast<int>(blockIdx.y) >= P->n_items) return;
  const FfnItem& it = P->items[blockIdx.y];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, sub = lane / LPR, sl = lane - sub * LPR;
  const int row0 = (static_cast<int>(blockIdx.x) * 4 + wave) * (64 / LPR * RP) + sub;
  stream_rows<WT, MODE_DN, LPR, NL, RP, 1, false>(it.w, nullptr, PlanRows{it}, row0, sl, wave, h, d, I, off0, off0, soff0,
                                                  soff0, 0, buf);
}

using Shape = StreamLanes;

using Kern = void (*)(const StreamBatch, const uint8_t*, const int32_t*, int, int, int, uint32_t, uint32_t, uint32_t,
                      uint32_t, int, void*);

// about 16 loads in flight per lane, and a workgroup's rows a divisor of 64
template <int MODE, int LPR, int NL, int KW>
constexpr int row_slots() {
  int rp = 16 / (NL * (MODE == MODE_UP ? 2 : 1));
  rp = rp >= 8 ? 8 : rp >= 4 ? 4 : rp >= 2 ? 2 : 1;
  while (4 / KW * (64 / LPR) * rp > 64) rp /= 2;
  return rp;
}

using DevUp = void (*)(const FfnBatch*, const uint8_t*, int, int, int, int, uint32_t, uint32_t, uint32_t, uint32_t,
                       uint32_t, uint32_t, uint16_t*);
using DevDn = void (*)(const FfnBatch*, const uint8_t*, int, int, uint32_t, uint32_t, float*);

// the shapes of the device pager (ffn_dev_supported) that stream (stream_few_tokens)
template <int WT>
DevUp dev_up_of(const Shape& s, int* rows_per_wg) {
#define WISP_U(L, N)                                                                 \
  if (s.lpr == L && s.nl == N && s.kw == 1) {                                        \
    *rows_per_wg = 4 * (64 / L) * row_slots<MODE_UP, L, N, 1>();                     \
    return &stream_gateup_dev<WT, L, N, row_slots<MODE_UP, L, N, 1>()>;              \
  }
  if constexpr (WT == DT_BF16) {
    WISP_U(64, 4)                  // d = 2048
  } else {
    WISP_U(64, 7)                  // d = 7168
  }
#undef WISP_U
  return nullptr;
}
template <int WT>
DevDn dev_dn_of(const Shape& s, int* rows_per_wg) {
#define WISP_D(L, N)                                                                 \
  if (s.lpr == L && s.nl == N && s.kw == 1) {                                        \
    *rows_per_wg = 4 * (64 / L) * row_slots<MODE_DN, L, N, 1>();                     \
    return &stream_down_dev<WT, L, N, row_slots<MODE_DN, L, N, 1>()>;                \
  }
  if constexpr (WT == DT_BF16) {
    WISP_D(32, 3)                  // I = 768
  } else {
    WISP_D(64, 2) WISP_D(16, 1)    // I = 2048, 256
  }
#undef WISP_D
  return nullptr;
}

template <int WT, int MODE>
Kern kernel_of(const Shape& s, int* rows_per_wg) {
#define WISP_S(L, N, W)                                     \
  if (s.lpr == L && s.nl == N && s.kw == W) {               \
    constexpr int rp = row_slots<MODE, L, N, W>();          \
    *rows_per_wg = 4 / W * (64 / L) * rp;                   \
    return &stream_kernel<WT, MODE, L, N, rp, W>;           \
  }
  if constexpr (MODE == MODE_DN) {   // (one chunk per lane of a gate/up row: such layers do not stream)
    WISP_S(64, 1, 1) WISP_S(32, 1, 1) WISP_S(16, 1, 1)
  }
  WISP_S(64, 2, 1) WISP_S(64, 3, 1) WISP_S(64, 4, 1) WISP_S(64, 5, 1) WISP_S(64, 6, 1) WISP_S(64, 7, 1)
  WISP_S(64, 8, 1) WISP_S(32, 3, 1) WISP_S(32, 5, 1) WISP_S(16, 3, 1) WISP_S(64, 3, 4) WISP_S(64, 4, 4)
  WISP_S(64, 5, 4) WISP_S(64, 6, 4) WISP_S(64, 7, 4) WISP_S(64, 8, 4)
#undef WISP_S
  return nullptr;
}

template <int MODE>
hipError_t launch(const StreamBatch& b, const FfnShape& s, const void* vin, const int32_t* perm, int k, void* out,
                  bool bf16_out, hipStream_t st, const LaunchTiming& tm) {
  if (b.n_items <= 0) return hipSuccess;
  if (b.n_items > kMaxStreamItems || !stream_supported(s)) return hipErrorInvalidValue;
  constexpr bool up = MODE == MODE_UP;
  const BlobLayout& B = s.blob;
  Shape sh{};
  if (!stream_lanes((up ? B.d : B.I) * static_cast<int>(B.elem) / 16, &sh)) return hipErrorInvalidValue;
  int rpw = 0;
  Kern kern = B.w_dtype == DT_FP8 ? kernel_of<DT_FP8, MODE>(sh, &rpw) : kernel_of<DT_BF16, MODE>(sh, &rpw);
  if (!kern) return hipErrorInvalidValue;
  const uint32_t off0 = static_cast<uint32_t>(up ? B.off_w1 : B.off_w2), off1 = static_cast<uint32_t>(up ? B.off_w3 : B.off_w2);
  const uint32_t s0 = static_cast<uint32_t>(up ? B.off_s1 : B.off_s2), s1 = static_cast<uint32_t>(up ? B.off_s3 : B.off_s2);
  hipExtLaunchKernelGGL(kern, dim3((up ? B.I : B.d) / rpw, b.n_items), dim3(256), 0, st, tm.start, tm.stop, 0, b,
                        static_cast<const uint8_t*>(vin), perm, k, B.d, B.I, off0, off1, s0, s1, bf16_out ? 1 : 0, out);
  return hipGetLastError();
}

Shape shape_of(const BlobLayout& B, bool up) {
  Shape sh{};
  (void)stream_lanes((up ? B.d : B.I) * static_cast<int>(B.elem) / 16, &sh);
  return sh;
}

}  // namespace

hipError_t launch_stream_dev(const FfnBatch* plan, int max_items, const FfnShape& s, const void* x, void* h, float* buf,
                             hipStream_t st, const LaunchTiming& tm_gateup, const LaunchTiming& tm_down) {
  if (!stream_supported(s)) return hipErrorNotSupported;
  const BlobLayout& L = s.blob;
  const Shape su = shape_of(L, true), sd = shape_of(L, false);
  int ru = 0, rd = 0;
  const bool fp8 = L.w_dtype == DT_FP8;
  DevUp ku = fp8 ? dev_up_of<DT_FP8>(su, &ru) : dev_up_of<DT_BF16>(su, &ru);
  DevDn kd = fp8 ? dev_dn_of<DT_FP8>(sd, &rd) : dev_dn_of<DT_BF16>(sd, &rd);
  if (!ku || !kd) return hipErrorNotSupported;
  const int fault_wgs = 32, copy_wgs = 16;   // the host link needs no more (expert_ffn.hip's device-planned launch)
  int blocks = L.I / ru;
  if (blocks < fault_wgs + copy_wgs) blocks = fault_wgs + copy_wgs;
  hipExtLaunchKernelGGL(ku, dim3(blocks, max_items), dim3(256), 0, st, tm_gateup.start, tm_gateup.stop, 0, plan,
                        static_cast<const uint8_t*>(x), L.d, L.I, fault_wgs, copy_wgs, static_cast<uint32_t>(L.off_w1),
                        static_cast<uint32_t>(L.off_w3), static_cast<uint32_t>(L.off_s1),
                        static_cast<uint32_t>(L.off_s3), static_cast<uint32_t>(L.off_w2),
                        static_cast<uint32_t>(L.bytes - L.off_w2), static_cast<uint16_t*>(h));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipExtLaunchKernelGGL(kd, dim3(L.d / rd, max_items), dim3(256), 0, st, tm_down.start, tm_down.stop, 0, plan,
                        static_cast<const uint8_t*>(h), L.d, L.I, static_cast<uint32_t>(L.off_w2),
                        static_cast<uint32_t>(L.off_s2), buf);
  return hipGetLastError();
}

bool stream_supported(const FfnShape& s) {
  return s.x_dtype == DT_BF16 && s.h_dtype == DT_BF16 && s.blob.bytes < (1ull << 32) &&
         stream_widths(s.blob.d, s.blob.I, static_cast<int>(s.blob.elem));
}

hipError_t launch_stream_gateup(const StreamBatch& b, const FfnShape& s, const void* x, const int32_t* perm, int k,
                                void* h, hipStream_t st, const LaunchTiming& tm) {
  return launch<MODE_UP>(b, s, x, perm, k, h, false, st, tm);
}

hipError_t launch_stream_down(const StreamBatch& b, const FfnShape& s, const void* h, const int32_t* perm, int k,
                              void* buf, bool bf16_out, hipStream_t st, const LaunchTiming& tm) {
  return launch<MODE_DN>(b, s, h, perm, k, buf, bf16_out, st, tm);
}

}  // namespace wisp
