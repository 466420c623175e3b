// Router scoring and top-k for gfx950 (the routing that decides R at each layer, WiSP Sec. 3.1).
//
// router_logits: z[t, e] = W_r[e] . x[t] in fp32.  Decode sizes (T <= 8): one workgroup per
//   expert row, so the fp32 router matrix is read by N workgroups at once (one HBM round trip);
//   token batches: fp32 matrix cores (a block of tokens against a group of router rows over a slice of
//   the columns per workgroup, slices summed by the selection).
// router_select: top-k selection and gates (select.hpp), optionally publishing the ids to the
//   host pager through host-coherent memory.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>

#include "kernels.hpp"
#include "router_row.hpp"
#include "router_rules.hpp"
#include "select.hpp"

namespace wisp {
namespace {

// Decode-sized logits: one workgroup per expert row (router_row in router_row.hpp), up to four
// tokens per pass.
template <int XT, int NT>
__global__ void __launch_bounds__(256) router_logits_wide_kernel(const float* __restrict__ wr,
                                                                 const void* __restrict__ x, int T, int N, int d,
                                                                 float* __restrict__ logits) {
  __shared__ float part[4][4];
  const int e = blockIdx.x;
  for (int t0 = 0; t0 < T; t0 += 4) {
    const int ntok = min(4, T - t0);
    const float z = router_row<XT, NT>(wr, x, t0, ntok, d, e, part);
    if (threadIdx.x < ntok) logits[static_cast<size_t>(t0 + threadIdx.x) * N + e] = z;
    __syncthreads();
  }
}

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Token-batch logits on the fp32 matrix cores (v_mfma_f32_16x16x4_f32): a workgroup computes 16 TB tokens
// against a group of 64 RB router rows over one slice of the columns (grid: token blocks x slices x row groups).
// Wave w takes the 16-row blocks w, w + 4, ... of the group and all TB 16-token blocks; per 16-column step
// lane l (r = l % 16, g = l / 16) holds columns 4g .. 4g + 3 of token r of each token block and of row r of
// each row block, PF steps ahead of the matrix-core work.  The slice's sums go to
// partial[slice][token][row]; the selection adds the slices in order.  Rows past N repeat the last one and
// are not stored.  A logit is the same chain whatever TB, RB and the grouping: only the slices order its sum.
template <int XT, int RB, int TB, int PF>
__global__ void __launch_bounds__(256) router_logits_split_kernel(const float* __restrict__ wr,
                                                                  const void* __restrict__ x, int T, int N, int d,
                                                                  int slice_steps, float* __restrict__ partial) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int t0 = blockIdx.x * 16 * TB, q = blockIdx.y, kbeg = q * slice_steps * 16;
  const int steps = min(slice_steps, d / 16 - q * slice_steps);   // >= 1 for every slice of the grid
  const int blk0 = blockIdx.z * 4 * RB + wave;
  const float* wrow[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b)
    wrow[b] = wr + static_cast<size_t>(min(16 * (blk0 + 4 * b) + r, N - 1)) * d + kbeg + 4 * g;
  size_t xoff[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const int t = t0 + 16 * tb + r;
    xoff[tb] = static_cast<size_t>(t < T ? t : 0) * d + kbeg + 4 * g;
  }
  f32x4_t acc[TB][RB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb)
#pragma unroll
    for (int b = 0; b < RB; ++b) acc[tb][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // operands of PF 16-column steps in flight: the loads of a step are issued PF steps before its
  // matrix-core work; step j lives in ring slot j % PF.  The loads are unconditional (a token past T reads
  // token 0's row, never stored; a step past the slice reads its last columns again, never used) and the
  // inputs stay raw until used, so no load waits for another.
  constexpr int XW = XT == DT_F32 ? 4 : 2;   // 32-bit words of four inputs
  float4 w[PF][RB];
  uint32_t v[PF][TB][XW];
  auto load = [&](int slot, int step) {
    const int k0 = 16 * min(step, steps - 1);
#pragma unroll
    for (int b = 0; b < RB; ++b) w[slot][b] = *reinterpret_cast<const float4*>(wrow[b] + k0);
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      if constexpr (XT == DT_F32) {
        const uint4 q4 = *reinterpret_cast<const uint4*>(static_cast<const float*>(x) + xoff[tb] + k0);
        v[slot][tb][0] = q4.x; v[slot][tb][1] = q4.y; v[slot][tb][2] = q4.z; v[slot][tb][3] = q4.w;
      } else {
        const uint2 q2 = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(x) + xoff[tb] + k0);
        v[slot][tb][0] = q2.x; v[slot][tb][1] = q2.y;
      }
    }
  };
  // input c (0..3) of token block tb in slot `slot`, widened exactly to fp32
  auto xin = [&](int slot, int tb, int c) -> float {
    if constexpr (XT == DT_F32) return __uint_as_float(v[slot][tb][c]);
    const uint32_t q = v[slot][tb][c >> 1];
    return __uint_as_float((c & 1) ? (q & 0xFFFF0000u) : (q << 16));
  };
  // one column of the quad at a time over all TB x RB accumulators, so that consecutive matrix-core
  // instructions rarely wait on each other's result (each accumulator still takes its columns in order)
  auto mma = [&](int slot) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int b = 0; b < RB; ++b) {
          const float wc = c == 0 ? w[slot][b].x : c == 1 ? w[slot][b].y : c == 2 ? w[slot][b].z : w[slot][b].w;
          acc[tb][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xin(slot, tb, c), wc, acc[tb][b], 0, 0, 0);
        }
  };
#pragma unroll
  for (int j = 0; j < PF; ++j) load(j, j);
  // every step but the last PF loads the step PF ahead, with no branch around the loads (a load
  // behind a branch makes the compiler wait for every load in flight before the next step's work)
  int j0 = 0;
  for (; j0 + PF < steps; j0 += PF) {
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      mma(j);
      load(j, j0 + j + PF);
      __builtin_amdgcn_sched_barrier(0);   // keeps the scheduler from moving later steps above the loads
    }
  }
#pragma unroll
  for (int j = 0; j < PF; ++j)
    if (j0 + j < steps) mma(j);
  float* out = partial + static_cast<size_t>(q) * T * N;
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int row = 16 * (blk0 + 4 * b) + r;
    if (row >= N) continue;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = t0 + 16 * tb + 4 * g + i;
        if (t < T) out[static_cast<size_t>(t) * N + row] = acc[tb][b][i];
      }
  }
}

// Selection (select.hpp) of the workgroup's tokens (tpw <= 4); wave w, lane j < k writes rank j of
// token blockIdx.x * tpw + w.  The indices can also be published to host-coherent memory as 64-bit
// (seq << 32 | id) words: the host knows an entry is current from its tag alone, so it needs no
// copy, event or fence to read them.
__global__ void __launch_bounds__(256) router_select_kernel(const float* __restrict__ logits, int n_split, int T,
                                                            int N, int k, int route, int n_groups, int topk_groups,
                                                            int32_t* __restrict__ idx, float* __restrict__ w,
                                                            uint64_t* __restrict__ idx_host, uint32_t seq, int tpw) {
  __shared__ SelectShared sh;
  const int t0 = blockIdx.x * tpw, t1 = min(T, t0 + tpw);
  select_tokens(logits, 0, t0, t1, N, k, route, n_groups, topk_groups, sh, n_split, static_cast<size_t>(T) * N);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = t0 + wave;
  if (t < t1 && lane < k) {
    const int e = sh.sel[wave][lane];
    idx[t * k + lane] = e;
    w[t * k + lane] = sh.gate[wave][lane];
    if (idx_host)
      __hip_atomic_store(idx_host + t * k + lane, (static_cast<uint64_t>(seq) << 32) | static_cast<uint32_t>(e),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Router logits and the selection of up to eight tokens in one launch (decode).  Workgroup e computes
// logit row e (router_row: the arithmetic of router_logits_wide_kernel) and publishes it as tagged words
// (tag_logit, one atomic store each); workgroup q < ceil(T / tpw), after its own row, selects for the tokens
// q tpw .. q tpw + tpw - 1 on the complete logits, reading each word until it carries this launch's tag, and writes idx, w
// and, if asked, the tagged ids for the host.  The other workgroups wait for nothing, and a selecting one
// has published its row before it waits; the tags (atomic accesses to one location are coherent) make it
// read this launch's logits with no ordering between locations.  (Seven tokens, 128 experts, d 2048:
// 8.2 us against 6.1 + 6.9 us in two launches; four tokens, 8 experts, d 4096: 11.3 -> 5.6 us with the tokens' rows
// loaded together and a selecting workgroup per token.)
template <int XT, int NT>
__global__ void __launch_bounds__(256) route_select_kernel(const float* __restrict__ wr, const void* __restrict__ x,
                                                           int d, uint64_t* __restrict__ logits, uint32_t tag, int T,
                                                           int N, int k, int route, int n_groups, int topk_groups,
                                                           int32_t* __restrict__ idx, float* __restrict__ w,
                                                           uint64_t* __restrict__ idx_host, uint32_t seq, int tpw) {
  __shared__ SelectShared sh;
  __shared__ float part[4][4];
  const int e = blockIdx.x;
  auto publish = [&](int t0, int nt) {
    const float z = router_row<XT, NT>(wr, x, t0, nt, d, e, part);
    if (static_cast<int>(threadIdx.x) < nt)
      __hip_atomic_store(logits + static_cast<size_t>(t0 + threadIdx.x) * N + e, tag_logit(tag, z), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  };
  publish(0, min(NT, T));
  if (NT > 1 && T > 4) publish(4, T - 4);
  const int s0 = e * tpw, s1 = min(T, s0 + tpw);
  if (s0 >= T) return;
  select_tokens<true>(logits, tag, s0, s1, N, k, route, n_groups, topk_groups, sh);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = s0 + wave;
  if (t < s1 && lane < k) {
    const int s = sh.sel[wave][lane];
    idx[t * k + lane] = s;
    w[t * k + lane] = sh.gate[wave][lane];
    if (idx_host)
      __hip_atomic_store(idx_host + t * k + lane, (static_cast<uint64_t>(seq) << 32) | static_cast<uint32_t>(s),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace

hipError_t launch_route_select(const float* wr, const void* x, int x_dtype, int d, uint64_t* logits, uint32_t tag,
                               int T, int N, int k, int route, int n_groups, int topk_groups,
                               int32_t* idx, float* w, uint64_t* idx_host, uint32_t seq, hipStream_t st,
                               const LaunchTiming& tm) {
  // a workgroup per token ranks its keys in a quarter of the time that four tokens take; it is a router row's
  // workgroup, so with fewer rows than tokens one selects for four
  const int tpw = T <= N ? 1 : 4;
  if (T < 1 || T > kRouteSelectTokens || (T + tpw - 1) / tpw > N || N < 1 || N > 256 || k < 1 || k > 8 || d % 4 != 0 ||
      (route == R_SIGMOID_GROUP && (n_groups > 32 || N % n_groups != 0)))
    return hipErrorInvalidValue;
  auto kern = WISP_ROUTER_ROW_KERNEL(route_select_kernel, x_dtype == DT_F32, T);
  hipExtLaunchKernelGGL(kern, dim3(N), dim3(256), 0, st, tm.start, tm.stop, 0, wr, x, d, logits, tag, T, N, k, route,
                        n_groups, topk_groups, idx, w, idx_host, seq, tpw);
  return hipGetLastError();
}

hipError_t launch_router_logits(const float* wr, const void* x, int x_dtype, int T, int N, int d, float* logits,
                                int* n_split, hipStream_t st, const LaunchTiming& tm) {
  *n_split = 1;
  if (T <= 0) return hipSuccess;
  if (d % 4 != 0) return hipErrorInvalidValue;
  if (T <= 8) {
    auto kern = WISP_ROUTER_ROW_KERNEL(router_logits_wide_kernel, x_dtype == DT_F32, T);
    hipExtLaunchKernelGGL(kern, dim3(N), dim3(256), 0, st, tm.start, tm.stop, 0, wr, x, T, N, d, logits);
    return hipGetLastError();
  }
  if (N > 256 || d % 16 != 0) return hipErrorInvalidValue;
  // how the logits are cut (router_tiles); 37 tokens, 128 experts, d 2048: 12.9 -> 5.4 us; 301 tokens, 64 experts, d 7168:
  // 33 -> 14.4; 203 tokens, 60 experts, d 1472: 101 (LDS-tiled FMA kernel) -> 5.5
  const RouterTiles r = router_tiles(T, N, d);
  *n_split = r.slices;
  using K = void (*)(const float*, const void*, int, int, int, int, float*);
  K kern = nullptr;
  const bool f32 = x_dtype == DT_F32;
#define WISP_RK(R, TB, PF) \
  kern = f32 ? &router_logits_split_kernel<DT_F32, R, TB, PF> : &router_logits_split_kernel<DT_BF16, R, TB, PF>
  if (r.tb == 4) {
    if (r.rb == 1) WISP_RK(1, 4, 4); else if (r.rb == 2) WISP_RK(2, 4, 4); else if (r.rb == 3) WISP_RK(3, 4, 4); else WISP_RK(4, 4, 4);
  } else if (r.tb == 2) {
    WISP_RK(1, 2, 8);
  } else {
    WISP_RK(1, 1, 8);
  }
#undef WISP_RK
  hipExtLaunchKernelGGL(kern, dim3((T + 16 * r.tb - 1) / (16 * r.tb), r.slices, r.groups), dim3(256), 0, st, tm.start,
                        tm.stop, 0, wr, x, T, N, d, r.steps, logits);
  return hipGetLastError();
}

hipError_t launch_router_select(const float* logits, int n_split, int T, int N, int k, int route, int n_groups,
                                int topk_groups, int32_t* idx, float* w, uint64_t* idx_host, uint32_t seq,
                                hipStream_t st, const LaunchTiming& tm) {
  if (T <= 0) return hipSuccess;
  if (N > 256 || k > 8 || k < 1 || (route == R_SIGMOID_GROUP && (n_groups > 32 || N % n_groups != 0)))
    return hipErrorInvalidValue;
  // four tokens per workgroup share its passes over the keys; while the chip is not full, a workgroup per
  // token ranks its keys in a quarter of the time (37 tokens: 9.7 -> 4.7 us; 301 tokens of 64
  // experts: 10.0 -> 6.0)
  const int tpw = T <= 1024 ? 1 : 4;
  dim3 grid((T + tpw - 1) / tpw), block(256);
  if (n_split < 1 || n_split > kRouterMaxSplit) return hipErrorInvalidValue;
  hipExtLaunchKernelGGL(router_select_kernel, grid, block, 0, st, tm.start, tm.stop, 0, logits, n_split, T, N, k,
                        route, n_groups, topk_groups, idx, w, idx_host, seq, tpw);
  return hipGetLastError();
}

}  // namespace wisp
