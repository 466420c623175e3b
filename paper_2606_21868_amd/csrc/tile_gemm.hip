// Launches of the fp8 / any-width grouped GEMMs (tile_gemm.hpp).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tile_gemm.hpp"

namespace wisp {
namespace {

template <int WT, int MODE, int NW, int RB>
__global__ void __launch_bounds__(NW * 64, 2) tile_kernel(GroupedBatch gb, const uint16_t* __restrict__ a_src,
                                                          uint32_t a_bytes, const int32_t* __restrict__ perm, int k,
                                                          int d, int I, uint32_t off0, uint32_t off1, uint32_t soff0,
                                                          uint32_t soff1, uint32_t w_bytes, void* __restrict__ out) {
  tile::tile_body<WT, MODE, NW, RB>(gb, a_src, a_bytes, perm, k, d, I, off0, off1, soff0, soff1, w_bytes, out);
}

template <int WT, int MODE, int NW, int RB>
hipError_t launch(GroupedBatch b, const FfnShape& s, const void* a, uint32_t a_bytes, const int32_t* perm, int k,
                  void* out, hipStream_t st, const LaunchTiming& tm) {
  constexpr bool up = MODE == tile::MODE_UP;
  const BlobLayout& B = s.blob;
  int nb = 0;
  for (int g = 0; g < b.n_groups; ++g) b.tile_end[g] = nb += (b.rows[g] + RB - 1) / RB;
  const int cols = up ? B.I : B.d, ct = NW * (up ? 16 : 32);
  const int tiles = nb * ((cols + ct - 1) / ct);
  const uint32_t off0 = static_cast<uint32_t>(up ? B.off_w1 : B.off_w2);
  const uint32_t off1 = static_cast<uint32_t>(up ? B.off_w3 : B.off_w2);
  const uint32_t s0 = static_cast<uint32_t>(up ? B.off_s1 : B.off_s2);
  const uint32_t s1 = static_cast<uint32_t>(up ? B.off_s3 : B.off_s2);
  const uint32_t w_bytes = WT == DT_FP8 ? static_cast<uint32_t>(B.bytes) - off0
                                        : static_cast<uint32_t>(B.d) * B.I * 2 * (up ? 2 : 1);
  const int grid = std::min(tiles, compute_units() * (8 / NW));   // eight waves per CU
  hipExtLaunchKernelGGL((tile_kernel<WT, MODE, NW, RB>), dim3(grid), dim3(NW * 64), 0, st, tm.start, tm.stop, 0, b,
                        static_cast<const uint16_t*>(a), a_bytes, perm, k, B.d, B.I, off0, off1, s0, s1, w_bytes, out);
  return hipGetLastError();
}

// Row blocks of 64 in two four-wave workgroups per CU, with tiles of 64 h (128 output) columns, which split the
// launch finer; or row blocks of 128 in one eight-wave workgroup, which reads an expert's weights for more
// rows at once and its token rows half as often.  The second is the better one once it saves a quarter of the row
// blocks, that is when a part of the experts has more than 64 rows.  us per layer pass at mean rows 38 / 50 /
// 57 / 64 / 87 (64 fp8 experts, d 7168): 740 against 870, 817 against 920, 876 against 935, 1005 against 953,
// 1304 against 1009; at 20 / 52 / 62 / 80 / 150 (60 bf16 experts, d 1472): 254 against 290, 314 against 325, 336
// against 325, 392 against 339, 544 against 476.  The choice does not change a bit of any output.
bool wide_rows(const GroupedBatch& b) {
  int64_t n64 = 0, n128 = 0;
  for (int g = 0; g < b.n_groups; ++g) {
    n64 += (b.rows[g] + 63) / 64;
    n128 += (b.rows[g] + 127) / 128;
  }
  return 3 * n64 > 4 * n128;
}

template <int MODE>
hipError_t dispatch(const GroupedBatch& b, const FfnShape& s, const void* a, uint32_t a_bytes, const int32_t* perm,
                    int k, void* out, hipStream_t st, const LaunchTiming& tm) {
  const bool wide = wide_rows(b);
  if (s.blob.w_dtype == DT_FP8)
    return wide ? launch<DT_FP8, MODE, 8, 128>(b, s, a, a_bytes, perm, k, out, st, tm)
                : launch<DT_FP8, MODE, 4, 64>(b, s, a, a_bytes, perm, k, out, st, tm);
  return wide ? launch<DT_BF16, MODE, 8, 128>(b, s, a, a_bytes, perm, k, out, st, tm)
              : launch<DT_BF16, MODE, 4, 64>(b, s, a, a_bytes, perm, k, out, st, tm);
}
}  // namespace

hipError_t launch_tile_gateup(const GroupedBatch& b, const FfnShape& s, const void* x, uint32_t x_bytes,
                              const int32_t* perm, int k, void* hs, hipStream_t st, const LaunchTiming& tm) {
  return dispatch<tile::MODE_UP>(b, s, x, x_bytes, perm, k, hs, st, tm);
}

hipError_t launch_tile_down(const GroupedBatch& b, const FfnShape& s, const void* hs, uint32_t hs_bytes,
                            const int32_t* perm, int k, float* buf, hipStream_t st, const LaunchTiming& tm) {
  return dispatch<tile::MODE_DN>(b, s, hs, hs_bytes, perm, k, buf, st, tm);
}

}  // namespace wisp
