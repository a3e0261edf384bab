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

// Tiles of 16 query rows up to which more than 256 keys are ranked by the
// in-register kernel, which packs the same keys, instead of the streamed one.
// A streamed workgroup lives for one wave's sweep of all keys, whatever the grid;
// here four waves share the sweep of 16 rows, so time grows with the workgroups, in
// steps of one per CU, and with the key rows that each reads from L2 (about 6.5 TB/s
// in all).  Rows of whole 128-byte lines are the slowest for their length.
// us, streamed / in-register, k = 9, d = 2:
//   bf16, M = 1024      512 tiles    768        1024      M = 4096, 1024 tiles
//   C = 96               55 / 19    55 / 24    56 / 32    140 / 108
//   C = 192              65 / 35    65 / 47    65 / 64    187 / 239
//   C = 256              76 / 47    76 / 65    76 / 88    243 / 340
//   C = 640             127 / 101  126 / 146  126 / 192   468 / 754
// and, streamed over in-register at 1024 tiles, M = 300 and 4096: bf16 C = 160 1.5,
// 1.2, 248 1.3, 1.1, 368 1.2, 1.3, 480 1.1, 1.3; 64 1.6, 0.97 (768: 2.1, 1.3); 304 1.1,
// 1.0 and 600 0.9, 0.9 (768: 1.3, 1.3 and 1.1, 1.2); fp32 C = 96 1.5, 1.3,
// 128 1.3, 1.2, 252 1.1, 1.2, 360 1.3, 1.4; 64 1.4, 1.02 and 160 0.9, 0.8 (768: 1.8, 1.4 and
// 1.1, 1.1).  From 12 contraction steps on streamed workgroups of 64 rows run one
// per CU: where they need a second round, in-register is 1.3 to 2.1 times as fast.
static bool knn_few_tiles(int B, int N, int C, int dt_bf16) {
  const long long tiles = (long long)B * ((N + kKnnRows - 1) / kKnnRows);
  if (tiles > 1024) return false;
  const int rowb = C * (dt_bf16 ? 2 : 4), steps = (rowb + 63) / 64;
  if (steps > 8 && (long long)B * ((N + 63) / 64) > 256) return true;
  int limit = 1024;
  if (rowb % 128 == 0) limit = dt_bf16 ? (rowb > 128 ? 512 : 768) : rowb == 256 || rowb > 512 ? 768 : 1024;
  else if (dt_bf16 && (steps == 10 || (steps > 16 && steps <= 20))) limit = 768;
  return tiles <= limit;
}

hipError_t launch_knn(const void* x, const void* keys, int B, int N, int C, int M, int k,
                      int dil, int dt_bf16, int32_t* idx_out, hipStream_t stream,
                      hipEvent_t ev0, hipEvent_t ev1) {
  const KnnArgs a = make_knn_args(x, keys, B, N, C, M, k, dil, idx_out);
  if (knn_use_stream(M, C, dt_bf16) && knn_few_tiles(B, N, C, dt_bf16))
    return launch_knn_tile(a, dt_bf16, stream, ev0, ev1);
  if (knn_use_stream(M, C, dt_bf16)) return launch_knn_stream(a, dt_bf16, stream, ev0, ev1);
  if (knn_use_resident(B, N, M, C, dt_bf16)) return launch_knn_resident(a, stream, ev0, ev1);
  if (knn_use_wide(M, C, dt_bf16)) return launch_knn_wide(a, stream, ev0, ev1);
  return launch_knn_tile(a, dt_bf16, stream, ev0, ev1);
}

}  // namespace gl
