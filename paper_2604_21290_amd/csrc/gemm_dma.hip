// bf16 tiled MFMA GEMM whose operands reach LDS by direct loads:
//   out[R, Cout] = act_out(A[R, K] W[Cout, K]^T + b) + residual
// The bf16 layers without a GELU on their input run here: FC1, FC2 + residual, the
// FFN, the GEMM pass of the two-pass MRConv and gl_linear (gemm.hip has fp32, the
// GELU on A and some layers of short rows).
//   - Staging: global_load_lds moves 16 bytes per lane from a row of A or W
//     straight into LDS, so a stage in flight holds no registers and is not
//     written by ds_write.  A wave's load fills 1024 consecutive bytes of LDS, so
//     rows cannot be padded; instead a row's 16-byte slots are permuted by its
//     number (slot ^ (row & 7)), which spreads the 16 rows an operand read
//     touches over all banks.  128 or 256 bytes of K per row and stage: 64-byte
//     rows load half cache lines and measured 25 % slower.  Two buffers, one
//     barrier per stage: a stage's loads are issued as the one before it starts to
//     be multiplied, and must arrive while it is.
//   - MFMA operands are swapped (W rows first), so a lane ends with four
//     consecutive output columns of one row.
//   - Epilogue: the tile passes through LDS in fp32, wave by wave, so that
//     every store (and residual load) covers whole rows of the wave's tile with
//     16 bytes per lane.  With 8-byte stores straight from the accumulators
//     the same kernel took 80 instead of 70 us on the first layer below, and
//     23.5 instead of 18 us on the last: partial lines bound the end of a layer,
//     where all workgroups store at once.  The residual is requested before
//     the contraction.
//   - What bounds it: 128 x 128 tiles read 642 MB through L2 for the third layer
//     below, about 21 us at the 30 TB/s that these loads reach from L2; launch,
//     ramp and the final stores take 8-9 us of every layer.
// Measured (us, cached operands, R = 12544 = 64 images of 196 nodes; before:
// register-staged tiles with 2-byte stores; outputs bit-identical):
//   640 -> 2560 GELU 97 -> 70, 1280 -> 640 35.6 -> 25.7,
//   2560 -> 640 + residual 71 -> 47, 640 -> 640 + residual 29.6 -> 18.0.
#include "gl_device.h"
#include "gl_kernels.h"

namespace gl {

// BM x BN output tile, STEP bytes of K per row and stage, WR x WC waves.
template <int BM_, int BN_, int STEP_, int WR_, int WC_>
struct DmaCfg {
  static constexpr int BM = BM_, BN = BN_, STEP = STEP_, WR = WR_, WC = WC_;
  static constexpr int kWaves = WR * WC, kThreads = 64 * kWaves;
  static constexpr int kStage = (BM + BN) * STEP;         // bytes of one stage buffer
  static constexpr int kLoads = kStage / 16 / kThreads;   // loads per lane and stage
  static constexpr int TM = BM / WR / 16, TN = BN / WC / 16;  // MFMA tiles per wave
  static constexpr size_t kSmem = (size_t)2 * kStage;
  // the epilogue's fp32 tile reuses the stage buffers
  static_assert((size_t)BM * BN * 4 <= kSmem, "epilogue tile exceeds the stage buffers");
  static_assert(kStage % (1024 * kWaves) == 0 && (STEP == 128 || STEP == 256), "whole loads per wave");
};

// HALVES: the contraction's halves come from a.A and a.A2 (no residual).
template <class G, int ACT_OUT, bool RES, bool HALVES = false>
__global__ __launch_bounds__(G::kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void gemm_dma_kernel(GemmArgs a) {
  extern __shared__ __align__(16) char smem[];
  constexpr int BM = G::BM, BN = G::BN, STEP = G::STEP, TM = G::TM, TN = G::TN, NL = G::kLoads;
  constexpr int SPR = STEP / 16, RPL = 64 / SPR;  // slots per row, rows per wave load
  const int R = a.R, Cout = a.Cout, rowb = a.K * 2;
  const int nstages = (rowb + STEP - 1) / STEP;
  const int ntn = (Cout + BN - 1) / BN;
  const int blk = xcd_remap(blockIdx.x, gridDim.x);
  const int mt = blk / ntn, nt = blk - mt * ntn;
  const int m0 = mt * BM, n0 = nt * BN;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, t = lane & 15;
  const int wm = w / G::WC, wn = w % G::WC;

  // -- staging: load i of wave w fills rows RPL (w + waves i) .. of the stage
  //    (BM rows of A, then BN rows of W); lane l's 16 bytes land at place l % SPR
  //    of row l / SPR and hold slot place ^ (row & (SPR - 1)).  Rows past R or Cout
  //    repeat the last one; slots past K read zeros.
  const uint32_t lds0 = lds_offset(smem);
  const char* src[NL];
  int slot[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int r = RPL * (w + G::kWaves * i) + lane / SPR;
    slot[i] = ((lane % SPR) ^ (r & (SPR - 1))) * 16;
    src[i] = (r < BM ? static_cast<const char*>(a.A) + (size_t)min(m0 + r, R - 1) * (HALVES ? rowb >> 1 : rowb)
                     : static_cast<const char*>(a.W) + (size_t)min(n0 + r - BM, Cout - 1) * rowb) +
             slot[i];
  }
  // from a row of A to the same place of the contraction in A2's row
  const ptrdiff_t half = HALVES ? static_cast<const char*>(a.A2) - static_cast<const char*>(a.A) - (rowb >> 1) : 0;
  auto stage = [&](int s) {
    const int off = s * STEP;
    const uint32_t d = lds0 + (s & 1) * G::kStage + w * 1024;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const char* p = src[i] + off;
      if (HALVES && RPL * (w + G::kWaves * i) < BM && off + slot[i] >= rowb >> 1) p += half;
      if (off + STEP > rowb)  // uniform: the last, partial stage
        p = off + slot[i] < rowb ? p : reinterpret_cast<const char*>(kZero16);
      lds_dma16(p, d + G::kWaves * i * 1024);
    }
  };
  stage(0);

  // -- the output place of this lane: 8 consecutive columns of every RPP-th row
  //    of the wave's tile; bias and residual are requested ahead of the product
  constexpr int WROWS = 16 * TM, WCOLS = 16 * TN;
  constexpr int LPR = WCOLS / 8, RPP = 64 / LPR, NP = WROWS / RPP;  // lanes per row, rows per pass
  constexpr int CSW = WCOLS / 4 < 16 ? WCOLS / 4 - 1 : 15;
  const int cq = lane % LPR, rq = lane / LPR;
  const int n = n0 + wn * WCOLS + cq * 8;
  const int row0 = m0 + wm * WROWS + rq;
  const uint16_t* bias = static_cast<const uint16_t*>(a.bias);
  const uint16_t* res = static_cast<const uint16_t*>(a.residual);
  uint16_t* out = static_cast<uint16_t*>(a.out);
  // out and the residual are accessed 16 bytes at a time whatever their rows'
  // alignment; only a row's last columns, fewer than eight, go one by one (before,
  // all did where rows were not whole vectors, us: 100352 x 160 -> 157 45.5 -> 24.5,
  // 25088 x 640 -> 637 47.0 -> 31.6; 2-byte stores of 16 neighbouring columns, register-staged
  // kernel, 26.1 and 38.2)
  const bool vec = n + 8 <= Cout;
  float bn[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) bn[v] = bias ? bf16_bits_to_f32(bias[min(n + v, Cout - 1)]) : 0.f;
  uint4 rv[NP];
  if (RES && vec) {
#pragma unroll
    for (int p = 0; p < NP; ++p)
      rv[p] = load16_any(res + (size_t)min(row0 + p * RPP, R - 1) * Cout + n);
  }

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < nstages; ++s) {
    // stage s has landed, and every wave is done reading stage s - 1's buffer
    dma_wait_barrier();
    if (s + 1 < nstages) stage(s + 1);
    const char* sa = smem + (s & 1) * G::kStage + (wm * WROWS + t) * STEP;
    const char* sb = smem + (s & 1) * G::kStage + (BM + wn * WCOLS + t) * STEP;
#pragma unroll
    for (int kk = 0; kk < STEP / 64; ++kk) {
      uint4 af[TM], bf[TN];
      const int co = ((kk * 4 + g) ^ (t & (SPR - 1))) * 16;
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const uint4*>(sa + i * 16 * STEP + co);
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[j] = *reinterpret_cast<const uint4*>(sb + j * 16 * STEP + co);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma_bf16(bf[j], af[i], acc[i][j]);
    }
  }

  // -- epilogue: lane (g, t) of MFMA tile (i, j) holds columns 4g .. 4g+3 of row t.
  //    The wave writes its tile to its own part of LDS as fp32 (16-byte chunks
  //    permuted by the row, as above) and reads it back in rows.
  __syncthreads();
  char* st = smem + w * (WROWS * WCOLS * 4);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      *reinterpret_cast<f32x4*>(st + (i * 16 + t) * (WCOLS * 4) + (((j * 4 + g) ^ (t & CSW)) * 16)) =
          acc[i][j];
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = p * RPP + rq, row = row0 + p * RPP;
    const char* sr = st + r * (WCOLS * 4);
    const f32x4 x0 = *reinterpret_cast<const f32x4*>(sr + ((2 * cq) ^ (r & CSW)) * 16);
    const f32x4 x1 = *reinterpret_cast<const f32x4*>(sr + ((2 * cq + 1) ^ (r & CSW)) * 16);
    float y[8];
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      y[v] = (v < 4 ? x0[v & 3] : x1[v & 3]) + bn[v];
      if (ACT_OUT) y[v] = gelu_f32(y[v]);
    }
    if (row >= R || n >= Cout) continue;
    const size_t o = (size_t)row * Cout + n;
    if (vec) {
      if (RES) {
        float f[8];
        unpack_bf16x8(rv[p], f);
#pragma unroll
        for (int v = 0; v < 8; ++v) y[v] += f[v];
      }
      store16_any(out + o, pack_bf16x8(y));
    } else {
#pragma unroll
      for (int v = 0; v < 8; ++v)
        if (n + v < Cout) {
          if (RES) y[v] += bf16_bits_to_f32(res[o + v]);
          out[o + v] = (uint16_t)f32_to_bf16_bits(y[v]);
        }
    }
  }
}

template <class G>
hipError_t launch_cfg(const GemmArgs& a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1) {
  if (a.A2 && a.residual) return hipErrorInvalidValue;
  const void* fn = a.A2 ? (a.act_out ? (const void*)&gemm_dma_kernel<G, 1, false, true>
                                     : (const void*)&gemm_dma_kernel<G, 0, false, true>)
                   : a.act_out ? (a.residual ? (const void*)&gemm_dma_kernel<G, 1, true>
                                           : (const void*)&gemm_dma_kernel<G, 1, false>)
                             : (a.residual ? (const void*)&gemm_dma_kernel<G, 0, true>
                                           : (const void*)&gemm_dma_kernel<G, 0, false>);
  const dim3 grid((unsigned)(((long)(a.R + G::BM - 1) / G::BM) * ((a.Cout + G::BN - 1) / G::BN)));
  return launch_with_smem(fn, grid, dim3(G::kThreads), G::kSmem, stream, ev0, ev1, a);
}

// The largest tile that still gives the chip enough workgroups: a larger tile
// reads less through L2, a fuller chip hides more latency.  us, measured:
//   tile (waves)    12544x640x640  6272x320x1280  6272x192x768  6272x640x320  196x768x192
//   128 x 128 (8)       17.9 *        14.2 *         10.9          11.1           9.8
//   128 x 64 (8)        23.8          16.4            9.8 *         8.5           7.5
//   64 x 64 (4)         24.6          16.6           10.9           8.0 *         7.0
//   32 x 64 (4)         32.6          21.1           11.6           8.9           5.4 *
// (* the tile the rule takes: 490, 490, 588, 490 and 21 of them).  128 x 128 tiles
// that just pass one round of two per CU (513 to 640) leave most of the second idle:
// 128 x 64 where a GELU or padded columns weigh (25088x80x320 GELU 16.0 -> 13.7,
// 25088x320x320 15.6 -> 14.8; 12544x192x768 13.0 -> 13.2).  64 x 64 tiles of 1 KB of K
// or more, up to two per CU: 8 waves and 256 bytes of K per stage, twice the bytes in
// flight, which operands that come from memory need (cached / not, K per stage 128 ->
// 256 bytes: 6272x1280x320 12.1, 20.0 -> 11.6, 15.5; 3136x2560x640 25.4, 34.4 -> 19.6,
// 24.2; 6272x768x192 8.3, 13.3 -> 8.3, 10.7; the register-staged kernel with three
// stages in flight 17.1, 18.8; 30.2, 31.1; 10.9, 12.1; 784x640x2560, 520 tiles, 9.4 ->
// 12.5).  The tiles of 32 rows take 256 bytes of K per stage: on a grid of a few
// workgroups each stage's round trip to memory shows.
hipError_t launch_gemm_dma(const GemmArgs& a, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1) {
  auto tiles = [&](int bm, int bn) { return (long)((a.R + bm - 1) / bm) * ((a.Cout + bn - 1) / bn); };
  const int pad64 = (a.Cout + 63) / 64, pad128 = 2 * ((a.Cout + 127) / 128);
  const long t128 = tiles(128, 128);
  const bool one_more = t128 > 512 && t128 <= 640 && (a.act_out || pad128 > pad64);
  if (t128 >= 384 && 4 * pad128 <= 5 * pad64 && !one_more)
    return launch_cfg<DmaCfg<128, 128, 128, 4, 2>>(a, stream, ev0, ev1);
  if (tiles(128, 64) >= 384) return launch_cfg<DmaCfg<128, 64, 128, 4, 2>>(a, stream, ev0, ev1);
  if (tiles(64, 64) >= 128 && tiles(64, 64) <= 512 && a.K >= 512)
    return launch_cfg<DmaCfg<64, 64, 256, 4, 2>>(a, stream, ev0, ev1);
  if (tiles(64, 64) >= 128) return launch_cfg<DmaCfg<64, 64, 128, 2, 2>>(a, stream, ev0, ev1);
  return launch_cfg<DmaCfg<32, 64, 256, 1, 4>>(a, stream, ev0, ev1);
}

}  // namespace gl
