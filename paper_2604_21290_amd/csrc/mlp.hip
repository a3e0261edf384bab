// The row-local tail of a full ViG block in one launch (the tile is in
// mlp_tile.h).
#include "mlp_tile.h"

namespace gl {

template <class M, bool FC1>
__global__ __launch_bounds__(64 * (M::kWaves)) void mlp_kernel(MlpArgs a) {
  extern __shared__ __align__(16) char smem[];
  M m(a, smem, xcd_remap(blockIdx.x, gridDim.x) * M::TM);
  m.stage();
  m.template run<FC1>();
}

template <int KP, int JK, int NW, int RT>
hipError_t launch_rt(const MlpArgs& a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1) {
  using M = Mlp<KP, JK, NW, RT>;
  static_assert(M::kSmem <= 160 * 1024, "LDS");
  const void* fn = a.u_next ? (const void*)&mlp_kernel<M, true> : (const void*)&mlp_kernel<M, false>;
  return launch_with_smem(fn, dim3((a.R + M::TM - 1) / M::TM), dim3(64 * NW), M::kSmem, stream, ev0, ev1, a);
}

template <int KP, int JK, int NW>
hipError_t launch_ks(const MlpArgs& a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1) {
  // 16 nodes per workgroup while those fit the chip in one round, else 32: the
  // weights are streamed once per workgroup, but a workgroup of 32 nodes lives
  // longer (196 x 192: 11.2 against 14.8 us, 3000 x 168 12.0 against 15.1; at
  // 6272 x 192 24.7 against 17.3; 64 nodes, where they fit LDS, gain nothing)
  if ((a.R + 15) / 16 <= 256) return launch_rt<KP, JK, NW, 1>(a, stream, ev0, ev1);
  return launch_rt<KP, JK, NW, 2>(a, stream, ev0, ev1);
}

// Up to 192 channels the tile's rows and the ring of W fit LDS, from 97 on with one
// workgroup of 32 nodes per CU.  The rule is by measurement: up to 128 channels one
// launch is faster at every size, past that the separate layers, whose tiles read W
// once per 128 nodes, are as fast from about 25 K nodes on (us, without and with FC1,
// layers / one launch: 6272 x 192 24.8, 29.4 / 15.3, 17.3; 12544 x 192 35.6, 42.3 /
// 29.0, 33.0; 25088 x 160 49.1, 58.0 / 49.8, 55.3; 50176 x 192 98.5, 110 / 99.4, 108;
// 25088 x 96 31.6, 37.6 / 21.7, 23.7; 100352 x 80 80, 92 / 63, 67;
// 100352 x 128 111, 117 / 108, 112; 196 x 192 14.5, 20.3 / 10.0, 11.2).
bool mlp_use_fused(int R, int C, int dt_bf16) {
  return dt_bf16 && (C <= 128 || (C <= 192 && R <= 16384));
}

hipError_t launch_mlp(const MlpArgs& a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1) {
  switch ((a.C + 31) / 32) {
    case 1: return launch_ks<1, 1, 2>(a, stream, ev0, ev1);
    case 2: return launch_ks<2, 2, 4>(a, stream, ev0, ev1);
    case 3: return launch_ks<3, 3, 6>(a, stream, ev0, ev1);
    case 4: return launch_ks<4, 4, 8>(a, stream, ev0, ev1);
    case 5: return launch_ks<6, 3, 10>(a, stream, ev0, ev1);
    case 6: return launch_ks<6, 3, 12>(a, stream, ev0, ev1);
  }
  return hipErrorInvalidValue;
}

}  // namespace gl
