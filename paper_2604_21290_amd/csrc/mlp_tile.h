// The row-local tail of a full ViG block (Sec. III Eq. 14-15, and FC1 of the next
// block, Eq. 11) for TM nodes whose sigma(U~) and X rows are in LDS:
//   Y  = S W_out^T + b_out + X
//   X' = GELU(Y W_1^T + b_1) W_2^T + b_2 + Y
//   U' = X' W_in'^T + b_in'                (when the next block's FC1 is given)
// The hidden rows, Y and X' stay in LDS, rounded to bf16 as the separate layers
// store them, with the same contraction order: the results are theirs bit for
// bit.
//
// What bounds it is the stream of weights, 10 C^2 of them per workgroup, from L2.
// Wave w owns the 16-column tile w of each layer (four of FFN1's) and streams its
// W rows through a ring of its own in LDS, by direct loads: a job is JK
// contraction steps of one tile, 16 rows x 64 JK bytes; two jobs fit the ring,
// so one is in flight while the other is multiplied, across the barriers between
// layers too, and no barrier orders the stream (a wave waits for its own
// loads).  Loading MFMA operands straight into registers, 16 rows x 64 bytes a
// load, took 25 us at 6272 x 192 however many were in flight.
#pragma once

#include "gl_device.h"
#include "gl_kernels.h"

namespace gl {

// KP: contraction steps of 32 channels, C padded up (a multiple of JK);
// NW: waves, at least ceil(C / 16); RT: row tiles of 16 nodes.
template <int KP, int JK, int NW, int RT>
struct Mlp {
  static constexpr int TM = 16 * RT, kWaves = NW;
  // LDS rows of C and 4C channels: whole steps, and 16 bytes that move
  // consecutive rows to other banks
  static constexpr int kRow = KP * 64 + 16, kHid = 4 * KP * 64 + 16;
  static constexpr int kJob = JK * 1024;                 // bytes of one job
  static constexpr int P = KP / JK;                      // jobs per tile of K = C
  static constexpr int J1 = P, J2 = 5 * P, J3 = 9 * P, J4 = 10 * P;  // FC2 | FFN1 | FFN2 | FC1
  static constexpr int kBias = 7 * KP * 32 * 2;          // b_out, b_1, b_2, b_in as stored
  static constexpr int kRows = TM * (2 * kRow + kHid);   // S / X', Y / U', hidden
  static constexpr size_t kSmem = (size_t)kRows + NW * 2 * kJob + kBias;

  const MlpArgs& a;
  char *sS, *sY, *sH, *ring;
  const uint16_t* sB;
  int row0, w, lane, g, t;
  uint32_t ring0;
  int lr[JK], lk[JK];   // W row and 16-byte slot that this lane's load i of a job brings

  // the slot of row r that lands at place p (spreads the 16 rows that an operand
  // read touches over the banks; rows are 4 JK slots apart)
  static __device__ __forceinline__ int swz(int r) {
    return JK % 4 == 0 ? r & 15 : JK % 4 == 2 ? (r >> 1) & 7 : (r >> 2) & 3;
  }

  __device__ __forceinline__ Mlp(const MlpArgs& a_, char* smem, int r0) : a(a_), row0(r0) {
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lane = threadIdx.x & 63;
    g = lane >> 4;
    t = lane & 15;
    sS = smem;
    sY = sS + TM * kRow;
    sH = sY + TM * kRow;
    ring = smem + kRows + w * 2 * kJob;
    ring0 = lds_offset(ring);
    sB = reinterpret_cast<const uint16_t*>(smem + kRows + NW * 2 * kJob);
#pragma unroll
    for (int i = 0; i < JK; ++i) {
      const int e = 64 * i + lane;
      lr[i] = e / (4 * JK);
      lk[i] = (e % (4 * JK)) ^ swz(lr[i]);
    }
  }

  // tile and part of job j (compile-time but for w)
  __device__ __forceinline__ int tile(int j) const {
    return j >= J1 && j < J2 ? w + NW * ((j - J1) / P) : w;
  }
  static __device__ __forceinline__ int part(int j) {
    return j < J1 ? j : j < J2 ? (j - J1) % P : j < J3 ? j - J2 : j - J3;
  }

  // Request job j: rows past the layer repeat its last one, slots past K are zero.
  __device__ __forceinline__ void issue(int j) {
    const bool two = j >= J2 && j < J3;
    const int K = two ? 4 * a.C : a.C, rows = j >= J1 && j < J2 ? 4 * a.C : a.C;
    const char* W = static_cast<const char*>(j < J1 ? a.W_out : j < J2 ? a.W_1 : j < J3 ? a.W_2 : a.W_in);
#pragma unroll
    for (int i = 0; i < JK; ++i) {
      const int k8 = part(j) * 4 * JK + lk[i];
      const char* p = W + ((size_t)min(16 * tile(j) + lr[i], rows - 1) * K + k8 * 8) * 2;
      lds_dma16(k8 * 8 < K ? p : reinterpret_cast<const char*>(kZero16), ring0 + (j & 1) * kJob + i * 1024);
    }
  }

  f32x4 acc[RT];

  __device__ __forceinline__ void mma(int j, const char* sA, int stride) {
    const char* rb = ring + (j & 1) * kJob + t * (64 * JK);
    uint4 bw[JK];
#pragma unroll
    for (int s = 0; s < JK; ++s) bw[s] = *reinterpret_cast<const uint4*>(rb + ((4 * s + g) ^ swz(t)) * 16);
#pragma unroll
    for (int s = 0; s < JK; ++s)
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const uint4 af = *reinterpret_cast<const uint4*>(sA + (r * 16 + t) * stride + (part(j) * JK + s) * 64 + g * 16);
        acc[r] = mfma_bf16(bw[s], af, acc[r]);
      }
  }

  // Lane (g, t) holds columns n .. n+3 of rows 16 r + t: + bias, [GELU,] [+ the
  // residual row in LDS,] rounded into dst.
  template <bool GELU, bool RES>
  __device__ __forceinline__ void put(int tl, int cols, const uint16_t* bias, const char* res, char* dst, int stride) {
    const int n = 16 * tl + 4 * g;
    const uint2 b2 = *reinterpret_cast<const uint2*>(bias + min(n, cols - 4));
    const float bn[4] = {__uint_as_float(b2.x << 16), __uint_as_float(b2.x & 0xffff0000u),
                         __uint_as_float(b2.y << 16), __uint_as_float(b2.y & 0xffff0000u)};
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      float y[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        y[v] = acc[r][v] + bn[v];
        if (GELU) y[v] = gelu_f32(y[v]);
      }
      if (RES) {
        const uint2 x = *reinterpret_cast<const uint2*>(res + (r * 16 + t) * kRow + min(n, cols - 4) * 2);
        y[0] += __uint_as_float(x.x << 16);
        y[1] += __uint_as_float(x.x & 0xffff0000u);
        y[2] += __uint_as_float(x.y << 16);
        y[3] += __uint_as_float(x.y & 0xffff0000u);
      }
      if (n < cols)
        *reinterpret_cast<uint2*>(dst + (r * 16 + t) * stride + n * 2) =
            make_uint2(f32x2_to_bf16x2_bits(y[0], y[1]), f32x2_to_bf16x2_bits(y[2], y[3]));
    }
  }

  // the tile's finished rows, contiguous in global memory, 16 bytes a lane
  __device__ __forceinline__ void store_rows(const char* src, void* dst) {
    const int vr = a.C >> 3;
    const int nv = min(TM, a.R - row0) * vr;
    char* d = static_cast<char*>(dst) + (size_t)row0 * a.C * 2;
    for (int e = threadIdx.x; e < nv; e += 64 * NW) {
      const int r = e / vr, v = e - r * vr;
      *reinterpret_cast<uint4*>(d + (size_t)e * 16) = *reinterpret_cast<const uint4*>(src + r * kRow + v * 16);
    }
  }

  // Stage the rows of S and X (rows past R repeat the last; channels past C are
  // zero), the biases (null: zeros) and zeros where the hidden rows' padding
  // meets zero weights, with the first two jobs of W in flight.
  __device__ __forceinline__ void stage() {
    constexpr int NT = 64 * NW, VR = 4 * KP, NV = (TM * VR + NT - 1) / NT;
    const int tid = threadIdx.x, C = a.C;
    uint4 vs[NV], vx[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int e = tid + NT * i, r = e / VR, v = e - r * VR;
      const size_t off = ((size_t)min(row0 + r, a.R - 1) * C + min(v * 8, C - 8)) * 2;
      vs[i] = *reinterpret_cast<const uint4*>(static_cast<const char*>(a.s) + off);
      vx[i] = *reinterpret_cast<const uint4*>(static_cast<const char*>(a.x) + off);
    }
    uint16_t* b = const_cast<uint16_t*>(sB);
    for (int e = tid; e < 7 * C; e += NT) {
      const int l = e / C;  // 0: b_out, 1..4: b_1, 5: b_2, 6: b_in
      const uint16_t* src = static_cast<const uint16_t*>(l == 0 ? a.b_out : l < 5 ? a.b_1 : l == 5 ? a.b_2 : a.b_in);
      b[e] = src ? src[l >= 1 && l < 5 ? e - C : e - l * C] : (uint16_t)0;
    }
    issue(0);
    issue(1);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int e = tid + NT * i, r = e / VR, v = e - r * VR;
      if (e >= TM * VR) continue;
      const bool in = v * 8 < C;
      *reinterpret_cast<uint4*>(sS + r * kRow + v * 16) = in ? vs[i] : make_uint4(0, 0, 0, 0);
      *reinterpret_cast<uint4*>(sY + r * kRow + v * 16) = in ? vx[i] : make_uint4(0, 0, 0, 0);
    }
    const int pv = 16 * KP - (C >> 1);  // 16-byte vectors of padding per hidden row
    for (int e = tid; e < TM * pv; e += NT) {
      const int r = e / pv;
      *reinterpret_cast<uint4*>(sH + r * kHid + 8 * C + (e - r * pv) * 16) = make_uint4(0, 0, 0, 0);
    }
  }

  // The layers, after stage().  Called by all threads.
  template <bool FC1>
  __device__ __forceinline__ void run() {
    constexpr int NJ = FC1 ? J4 : J3;
    const int C = a.C;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      // the layer before is complete (at j = 0: what stage() wrote)
      if (j == 0 || j == J1 || j == J2 || j == J3) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      // job j has landed (the next one may be in flight)
      if (j + 1 < NJ) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(JK) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (part(j) == 0) {
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      const bool h = j >= J2 && j < J3;
      mma(j, j < J1 ? sS : j < J2 ? sY : h ? sH : sS, h ? kHid : kRow);
      // its operands are read: its part of the ring takes the job after the next
      if (j + 2 < NJ) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(j + 2);
      }
      if (j < J1) {
        if (part(j) == P - 1) put<false, true>(tile(j), C, sB, sY, sY, kRow);
      } else if (j < J2) {
        if (part(j) == P - 1) put<true, false>(tile(j), 4 * C, sB + C, nullptr, sH, kHid);
      } else if (j < J3) {
        if (part(j) == 4 * P - 1) put<false, true>(tile(j), C, sB + 5 * C, sY, sS, kRow);
      } else {
        if (part(j) == P - 1) put<false, false>(tile(j), C, sB + 6 * C, nullptr, sY, kRow);
      }
    }
    __syncthreads();
    store_rows(sS, a.out);
    if (FC1) store_rows(sY, a.u_next);
  }
};

}  // namespace gl
