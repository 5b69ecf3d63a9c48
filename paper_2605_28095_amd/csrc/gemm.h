// What the projection kernels share: arguments, buffer loads, the epilogue.
#pragma once
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace sidp {

constexpr int kWaves = 4;          // waves per workgroup, one column group each
constexpr int kBK = 64;            // k per LDS stage
constexpr int kFragElems = 512;    // 64 lanes x 8 bf16

__host__ __device__ inline int round_up(int a, int b) { return (a + b - 1) / b * b; }

// Packed weights from here on do not stay cached from one reader to the next (k_gemm_deep.hip has the times).
constexpr size_t kNtBytes = (size_t)150 << 20;

struct GemmArgs {
  const uint16_t* x;   // [M, K] bf16, row stride K
  const uint16_t* w;   // packed
  int M, K, KP;        // KP = K rounded up to 64
  int NG;              // packed column groups (64 columns each)
  int tiles;           // ceil(NG / waves per workgroup)
  int splits;
  int N;               // valid output columns (SWIGLU: F)
  int mblocks;         // row blocks of BM rows
  void* out;
  const uint16_t* bias;  // EPI_BF16
  const float* resid;    // EPI_RESID
  float* ws;             // split-K partials [splits][M][NG*64]
};

__device__ __forceinline__ float silu_f(float g) { return g / (1.0f + __expf(-g)); }

constexpr uint32_t kRsrcWord3 = 0x00020000u;  // gfx9 raw buffer: 32-bit data, bounds-checked
constexpr uint32_t kOutOfRange = 0x80000000u;  // any offset past num_records reads as zero

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, (int)kRsrcWord3);
}

__device__ __forceinline__ u32x4_t buf_load16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

// 16 bytes per lane from r + voff + soff straight to LDS: lane l's land at dst + 16 l.
__device__ __forceinline__ void buf_load16_lds(__amdgpu_buffer_rsrc_t r, uint16_t* dst, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0, 0);
}

// s_waitcnt vmcnt(N) alone; also keeps the compiler from moving memory
// operations across it.
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Writes one wave's tile: rows row0 + [0, 32 MF), the 64 packed columns of
// group ng; acc[m][nf] holds the 32x32 block (m, nf) in the MFMA's layout
// (register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32).
template <int MF, int EPI, bool PARTIAL>
__device__ __forceinline__ void store_tile(const GemmArgs& a, const f32x16_t (&acc)[MF][2], int row0, int ng,
                                           int split, int lane) {
  const int NP = a.NG * 64;
#pragma unroll
  for (int m = 0; m < MF; m++) {
#pragma unroll
    for (int r = 0; r < 16; r++) {
      const int row = row0 + m * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
      if (row >= a.M) continue;
      if (PARTIAL) {
        float* dst = a.ws + ((int64_t)split * a.M + row) * NP + ng * 64 + (lane & 31);
        dst[0] = acc[m][0][r];
        dst[32] = acc[m][1][r];
      } else if (EPI == SIDP_EPI_SWIGLU) {
        const int f = ng * 32 + (lane & 31);
        if (f < a.N)
          ((uint16_t*)a.out)[(int64_t)row * a.N + f] = f2bf(silu_f(acc[m][0][r]) * acc[m][1][r]);
      } else {
#pragma unroll
        for (int nf = 0; nf < 2; nf++) {
          const int n = ng * 64 + nf * 32 + (lane & 31);
          if (n >= a.N) continue;
          const int64_t o = (int64_t)row * a.N + n;
          if (EPI == SIDP_EPI_BF16) {
            float v = acc[m][nf][r];
            if (a.bias) v += bf2f(a.bias[n]);
            ((uint16_t*)a.out)[o] = f2bf(v);
          } else {
            ((float*)a.out)[o] = a.resid ? a.resid[o] + acc[m][nf][r] : acc[m][nf][r];
          }
        }
      }
    }
  }
}

// The projection with the deep pipeline (k_gemm_deep.hip): `rows` per
// workgroup 32, 64 or 128, `waves` 4, 7 or 8. a.splits > 1 leaves partials in
// a.ws. Needs 16-byte aligned activations.
hipError_t launch_gemm_deep(GemmArgs a, int epilogue, int rows, int waves, hipStream_t s);

}  // namespace sidp
