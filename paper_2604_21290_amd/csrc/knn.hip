// Standalone kNN graph kernel and its launcher (the tile itself is in knn_tile.h).
#include "knn_tile.h"

namespace gl {

size_t knn_smem_bytes(int C, int dt_bf16) {
  (void)C;
  (void)dt_bf16;
  return (size_t)kKnnRows * kKnnChunk * 4;
}

// Three waves per SIMD.  bf16 gets them by itself (148 VGPRs and 16 accumulation
// registers); fp32 took 156 to 162 and fell to two unless told (32 x 3136 rows, 196
// keys, us, two waves / three: C = 48 66 / 52, C = 96 105 / 88).
template <int DT, int R, bool SKIP_NAN>
__global__ __launch_bounds__(kKnnThreads) __attribute__((amdgpu_waves_per_eu(DT ? 1 : 3, 8))) void knn_kernel(KnnArgs a) {
  extern __shared__ __align__(16) char smem[];
  const int nt = (a.N + kKnnRows - 1) / kKnnRows;
  const int blk = xcd_remap(blockIdx.x, gridDim.x);
  const int b = blk / nt, tile = blk - b * nt;
  constexpr int ES = DT ? 2 : 4;
  knn_tile<DT, R, SKIP_NAN>(smem, static_cast<const char*>(a.x) + (size_t)b * a.N * a.C * ES,
                            static_cast<const char*>(a.keys) + (size_t)b * a.M * a.C * ES, a.N, a.C,
                            a.M, a.k, a.dil, a.KK, a.ib, a.qscale, a.qmax, tile * kKnnRows,
                            a.idx + (size_t)b * a.N * a.k);
}

template <int DT, bool SKIP_NAN>
const void* knn_fn(int R) {
  return R == 1 ? (const void*)&knn_kernel<DT, 1, SKIP_NAN>
         : R == 2 ? (const void*)&knn_kernel<DT, 2, SKIP_NAN> : (const void*)&knn_kernel<DT, 4, SKIP_NAN>;
}

KnnArgs make_knn_args(const void* x, const void* keys, int B, int N, int C, int M, int k, int dil,
                      int32_t* idx) {
  KnnArgs a;
  a.x = x;
  a.keys = keys;
  a.idx = idx;
  a.B = B;
  a.N = N;
  a.C = C;
  a.M = M;
  a.k = k;
  a.dil = dil;
  a.KK = k * dil;
  a.ib = 1;
  while ((1 << a.ib) < M) ++a.ib;
  a.qscale = (float)(1u << (30 - a.ib));
  a.qmax = (1u << (32 - a.ib)) - 2u;
  return a;
}

int knn_list_regs(int KK) { return KK <= 16 ? 1 : KK <= 32 ? 2 : 4; }

hipError_t launch_knn_tile(const KnnArgs& a, int dt_bf16, hipStream_t stream, hipEvent_t ev0,
                           hipEvent_t ev1) {
  const size_t smem = knn_smem_bytes(a.C, dt_bf16);
  const dim3 grid(a.B * ((a.N + kKnnRows - 1) / kKnnRows)), block(kKnnThreads);
  const int R = knn_list_regs(a.KK);
  // Key sets that larger grids stream: non-finite rows rank as they do there,
  // whatever the grid.
  const bool skip = knn_use_stream(a.M, a.C, dt_bf16);
  const void* fn = dt_bf16 ? (skip ? knn_fn<1, true>(R) : knn_fn<1, false>(R))
                           : (skip ? knn_fn<0, true>(R) : knn_fn<0, false>(R));
  return launch_with_smem(fn, grid, block, smem, stream, ev0, ev1, a);
}

hipError_t launch_knn(const void* x, const void* keys, int B, int N, int C, int M, int k,
                      int dil, int dt_bf16, int32_t* idx_out, hipStream_t stream,
                      hipEvent_t ev0, hipEvent_t ev1) {
  const KnnArgs a = make_knn_args(x, keys, B, N, C, M, k, dil, idx_out);
  // Large key sets on small grids take the in-register kernel, which ranks the
  // same packed keys.  A streamed workgroup lives for one wave's sweep of all
  // keys, whatever the grid; here four waves share the sweep of 16 rows, so
  // time grows with the workgroups instead.  us, streamed / in-register, k = 9,
  // d = 2: 3 x 513, C = 204, fp32 89 / 27 (99 workgroups); bf16 1 x 3136, C = 96
  // 106 / 41 (196), 12 x 1024, C = 200 69 / 48 (768), 32 x 513, C = 200 47.8 / 46.2
  // (1056), 12 x 2048, C = 200 126 / 176 (1536), 32 x 1024, C = 96 54 / 59 (2048).
  if (knn_use_stream(M, C, dt_bf16) && (long long)B * ((N + kKnnRows - 1) / kKnnRows) <= 1024)
    return launch_knn_tile(a, dt_bf16, stream, ev0, ev1);
  if (knn_use_stream(M, C, dt_bf16)) return launch_knn_stream(a, dt_bf16, stream, ev0, ev1);
  if (knn_use_resident(B, N, M, C, dt_bf16)) return launch_knn_resident(a, stream, ev0, ev1);
  if (knn_use_wide(M, C, dt_bf16)) return launch_knn_wide(a, stream, ev0, ev1);
  return launch_knn_tile(a, dt_bf16, stream, ev0, ev1);
}

}  // namespace gl
