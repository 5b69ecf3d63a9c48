// Per-head QK RMSNorm (Qwen3 family), rotary embedding, and the append of the
// new token's key and value to the paged KV cache (K3), plus the slot mapping
// slot = block_table[p / bs] * bs + p % bs (K9). A lane holds 8 consecutive dims
// of a head, D / 8 lanes a head, so a wave takes 4 heads (8 at D = 64) of one
// sequence and a workgroup 16 (32); the other half of a rotate-half pair sits
// D / 16 lanes away. Bound by latency, not bytes: 16-byte loads and stores and
// several heads to a wave keep a launch at one round of waves on the chip (256
// sequences of 80 heads with QK-norm 7.9 us; a wave per head, 2 bytes a lane and
// load, 9.6); beside slot fills a wave takes a head (k_rope_append_wave). The projection output is read either as bf16 or, when the QKV
// projection left split-K partials, reduced here: the partials are summed in
// split order, the bias added and the result rounded to bf16, which is the
// same value the projection's own reduction would have stored.
#include "common.h"
#include "internal.h"

namespace sidp {

// 8 bf16 values; ALIGNED: 16-byte aligned, one load.
template <bool ALIGNED>
__device__ __forceinline__ void load8(const uint16_t* p, float (&v)[8]) {
  if (ALIGNED) {
    const u32x4_t u = *(const u32x4_t*)p;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      v[2 * i] = bf2f((uint16_t)(u[i] & 0xffffu));
      v[2 * i + 1] = bf2f((uint16_t)(u[i] >> 16));
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = bf2f(p[i]);
  }
}

// The sum of a head's squares, on each of its D / 8 lanes: rotate-half pairs (i, i +
// D/2) first, then pairs of i that differ in their highest bit, and so on down, so
// that the roundings are those of one pair per lane and a butterfly over the lanes.
// Each of the first steps hands half of a lane's sums over and keeps the other half.
template <int D>
__device__ __forceinline__ float head_sum_sq(const float (&x)[8], int sub) {
  constexpr int kLanes = D / 8;
  const bool h4 = sub & (kLanes / 2), h2 = sub & (kLanes / 4), h1 = sub & (kLanes / 8);
  float t[4], u[2];
#pragma unroll
  for (int j = 0; j < 4; j++) {  // dims j of the lane's eight in its first half, 4 + j in its second
    const float own = h4 ? x[4 + j] : x[j];
    const float other = __shfl_xor(h4 ? x[j] : x[4 + j], kLanes / 2, 64);
    const float lo = h4 ? other : own, hi = h4 ? own : other;
    t[j] = fmaf(hi, hi, lo * lo);
  }
#pragma unroll
  for (int j = 0; j < 2; j++) u[j] = (h2 ? t[2 + j] : t[j]) + __shfl_xor(h2 ? t[j] : t[2 + j], kLanes / 4, 64);
  float v = (h1 ? u[1] : u[0]) + __shfl_xor(h1 ? u[0] : u[1], kLanes / 8, 64);
  if (D == 128) v += __shfl_xor(v, 1, 64);
#pragma unroll
  for (int o = kLanes / 2; o >= kLanes / 8; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <int D, bool ALIGNED>
__global__ void __launch_bounds__(256) k_rope_append(RopeCall c) {
  constexpr int kLanes = D / 8;         // lanes of a head
  constexpr int kHeads = 256 / kLanes;  // heads of a workgroup
  const int b = blockIdx.x;
  const int heads = c.hq + 2 * c.hkv;
  const int h = blockIdx.y * kHeads + threadIdx.x / kLanes;
  const int sub = threadIdx.x % kLanes, d0 = sub * 8;  // this lane's dims d0 .. d0 + 7
  const int pos = c.positions[b];
  const int lb = pos >= 0 ? pos / c.kv.bs : -1;
  const bool ok_pos = pos >= 0 && lb < c.max_blocks && pos < c.max_seq;
  const int blk = ok_pos ? c.block_tables[(int64_t)b * c.max_blocks + lb] : -1;
  const bool ok_blk = blk >= 0 && blk < c.kv.nblk;
  if (threadIdx.x == 0 && blockIdx.y == 0) {
    if (!ok_pos) atomicOr(c.err, SIDP_DEVERR_POSITION);
    else if (!ok_blk) atomicOr(c.err, SIDP_DEVERR_BLOCK);
  }
  if (h >= heads) return;  // whole heads at a time: the lanes of a shuffle stay together
  const int off = ok_pos ? pos % c.kv.bs : 0;
  const int rpos = ok_pos ? pos : 0;
  const int64_t region_base = (int64_t)c.region * c.kv.nblk;
  const bool is_q = h < c.hq, is_k = !is_q && h < c.hq + c.hkv;

  float x[8];  // the bf16 projection output
  if (c.ws) {
    // eight splits' partials in flight at a time, summed in split order
    f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
    const float* row = c.ws + (int64_t)b * c.ws_np + h * D + d0;
    const int64_t step = (int64_t)c.batch * c.ws_np;
    for (int sp0 = 0; sp0 < c.splits; sp0 += 8) {
      f32x4_t p0[8], p1[8];
#pragma unroll
      for (int j = 0; j < 8; j++)
        if (sp0 + j < c.splits) {
          p0[j] = *(const f32x4_t*)(row + (sp0 + j) * step);
          p1[j] = *(const f32x4_t*)(row + (sp0 + j) * step + 4);
        }
#pragma unroll
      for (int j = 0; j < 8; j++)
        if (sp0 + j < c.splits) {
          s0 += p0[j];
          s1 += p1[j];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
      x[i] = s0[i];
      x[4 + i] = s1[i];
    }
    if (c.bias) {
      float bias[8];
      load8<ALIGNED>(c.bias + h * D + d0, bias);
#pragma unroll
      for (int i = 0; i < 8; i++) x[i] += bias[i];
    }
#pragma unroll
    for (int i = 0; i < 8; i++) x[i] = bf2f(f2bf(x[i]));
  } else {
    load8<ALIGNED>(c.qkv + ((int64_t)b * heads + h) * D + d0, x);
  }
  if (!is_q && !is_k) {  // value head: store as is, transposed block layout [d][token]
    if (ok_blk) {
      const int vh = h - c.hq - c.hkv;
      uint16_t* vb = c.kv.v + ((region_base + blk) * c.kv.hkv + vh) * (int64_t)D * c.kv.bs;
#pragma unroll
      for (int i = 0; i < 8; i++) vb[(int64_t)(d0 + i) * c.kv.bs + off] = f2bf(x[i]);
    }
    return;
  }
  const uint16_t* gn = is_q ? c.g_q : c.g_k;
  if (gn) {
    float g[8];
    load8<ALIGNED>(gn + d0, g);
    const float r = 1.0f / sqrtf(head_sum_sq<D>(x, sub) / (float)D + c.qk_eps);
#pragma unroll
    for (int i = 0; i < 8; i++) x[i] = x[i] * r * g[i];
  }
  const int t0 = d0 % (D / 2);  // the pair's angle index
  const float* cs = c.rope_cos + (int64_t)rpos * (D / 2) + t0;
  const float* sn = c.rope_sin + (int64_t)rpos * (D / 2) + t0;
  const float sign = d0 < D / 2 ? -1.f : 1.f;
  uint32_t y[4];
#pragma unroll
  for (int i = 0; i < 8; i += 4) {
    const f32x4_t cv = *(const f32x4_t*)(cs + i), sv = *(const f32x4_t*)(sn + i) * sign;
    float o[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const float other = __shfl_xor(x[i + j], kLanes / 2, 64);
      o[j] = fmaf(x[i + j], cv[j], other * sv[j]);
    }
    y[i / 2] = pack_bf2(o[0], o[1]);
    y[i / 2 + 1] = pack_bf2(o[2], o[3]);
  }
  const u32x4_t out = {y[0], y[1], y[2], y[3]};
  if (is_q) {
    uint16_t* qo = c.q_out + ((int64_t)b * c.hq + h) * D + d0;
    if (ALIGNED) {
      *(u32x4_t*)qo = out;
    } else {
#pragma unroll
      for (int i = 0; i < 8; i++) qo[i] = (uint16_t)(out[i / 2] >> (16 * (i % 2)));
    }
  } else if (ok_blk) {
    // key blocks are [d / 8][token][d % 8]: the lane's 8 dims are one 16-byte piece
    const int kh = h - c.hq;
    uint16_t* kb = c.kv.k + ((region_base + blk) * c.kv.hkv + kh) * (int64_t)D * c.kv.bs;
    *(u32x4_t*)(kb + (sub * c.kv.bs + off) * 8) = out;
  }
}

// The same, bit for bit, with a wave per head and a rotate-half pair (i, i + D/2) per
// lane, four heads per workgroup, for streamed steps. Beside fill tile A it takes
// longer by itself (256 rows of the 70B heads 57 us, the kernel above 48), but the
// attention that follows is faster (0.734 against 0.782 ms a launch): 80 streamed
// layers at 256 rows run at 1905 tokens/s with it and 1891 with the other (means of
// four runs each, which differ by 0.1% and 0.3%). A smaller tile A makes it no better
// (24, 22, 20% with the other kernel: 1928, 1918, 1902 beside 1918 at 25%).
__global__ void __launch_bounds__(256) k_rope_append_wave(RopeCall c) {
  const int b = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int D = c.d, half = D >> 1;
  const int heads = c.hq + 2 * c.hkv;
  const int h = blockIdx.y * 4 + wave;
  if (h >= heads) return;
  const int pos = c.positions[b];
  const int lb = pos >= 0 ? pos / c.kv.bs : -1;
  const bool ok_pos = pos >= 0 && lb < c.max_blocks && pos < c.max_seq;
  const int blk = ok_pos ? c.block_tables[(int64_t)b * c.max_blocks + lb] : -1;
  const bool ok_blk = blk >= 0 && blk < c.kv.nblk;
  if (threadIdx.x == 0 && blockIdx.y == 0) {
    if (!ok_pos) atomicOr(c.err, SIDP_DEVERR_POSITION);
    else if (!ok_blk) atomicOr(c.err, SIDP_DEVERR_BLOCK);
  }
  const int off = ok_pos ? pos % c.kv.bs : 0;
  const int rpos = ok_pos ? pos : 0;
  const int64_t region_base = (int64_t)c.region * c.kv.nblk;

  const bool is_q = h < c.hq, is_k = !is_q && h < c.hq + c.hkv;
  const bool act = lane < half;
  const int col0 = h * D + lane, col1 = col0 + half;
  uint16_t v0 = 0, v1 = 0;  // the bf16 projection output of this lane's pair
  if (act) {
    if (c.ws) {
      // four splits' partials in flight at a time, summed in split order
      float s0 = 0.f, s1 = 0.f;
      for (int sp0 = 0; sp0 < c.splits; sp0 += 4) {
        float p0[4], p1[4];
#pragma unroll
        for (int j = 0; j < 4; j++)
          if (sp0 + j < c.splits) {
            const float* pr = c.ws + ((int64_t)(sp0 + j) * c.batch + b) * c.ws_np;
            p0[j] = pr[col0];
            p1[j] = pr[col1];
          }
#pragma unroll
        for (int j = 0; j < 4; j++)
          if (sp0 + j < c.splits) {
            s0 += p0[j];
            s1 += p1[j];
          }
      }
      if (c.bias) {
        s0 += bf2f(c.bias[col0]);
        s1 += bf2f(c.bias[col1]);
      }
      v0 = f2bf(s0);
      v1 = f2bf(s1);
    } else {
      const uint16_t* src = c.qkv + (int64_t)b * heads * D;
      v0 = src[col0];
      v1 = src[col1];
    }
  }
  if (!is_q && !is_k) {  // value head: store as is, transposed block layout [d][token]
    if (act && ok_blk) {
      const int vh = h - c.hq - c.hkv;
      uint16_t* vb = c.kv.v + ((region_base + blk) * c.kv.hkv + vh) * (int64_t)D * c.kv.bs;
      vb[(int64_t)lane * c.kv.bs + off] = v0;
      vb[(int64_t)(lane + half) * c.kv.bs + off] = v1;
    }
    return;
  }
  float x0 = bf2f(v0), x1 = bf2f(v1);
  const uint16_t* gn = is_q ? c.g_q : c.g_k;
  if (gn) {
    const float ss = wave_sum(fmaf(x1, x1, x0 * x0));
    const float r = 1.0f / sqrtf(ss / (float)D + c.qk_eps);
    if (act) {
      x0 = x0 * r * bf2f(gn[lane]);
      x1 = x1 * r * bf2f(gn[lane + half]);
    }
  }
  if (!act) return;
  const float cs = c.rope_cos[(int64_t)rpos * half + lane];
  const float sn = c.rope_sin[(int64_t)rpos * half + lane];
  const float y0 = fmaf(x0, cs, -(x1 * sn));
  const float y1 = fmaf(x1, cs, x0 * sn);
  if (is_q) {
    uint16_t* qo = c.q_out + ((int64_t)b * c.hq + h) * D;
    qo[lane] = f2bf(y0);
    qo[lane + half] = f2bf(y1);
  } else if (ok_blk) {
    // key blocks are [d / 8][token][d % 8]
    const int kh = h - c.hq;
    uint16_t* kb = c.kv.k + ((region_base + blk) * c.kv.hkv + kh) * (int64_t)D * c.kv.bs;
    const int d0 = lane, d1 = lane + half;
    kb[((d0 >> 3) * c.kv.bs + off) * 8 + (d0 & 7)] = f2bf(y0);
    kb[((d1 >> 3) * c.kv.bs + off) * 8 + (d1 & 7)] = f2bf(y1);
  }
}

template <int D>
static hipError_t launch_rope_d(const RopeCall& c, hipStream_t s) {
  const int per = 256 / (D / 8), heads = c.hq + 2 * c.hkv;
  const dim3 grid(c.batch, (heads + per - 1) / per);
  const uintptr_t ptrs = (uintptr_t)c.qkv | (uintptr_t)c.bias | (uintptr_t)c.g_q | (uintptr_t)c.g_k | (uintptr_t)c.q_out;
  if (ptrs % 16 == 0) k_rope_append<D, true><<<grid, 256, 0, s>>>(c);
  else k_rope_append<D, false><<<grid, 256, 0, s>>>(c);
  return hipGetLastError();
}

hipError_t launch_rope_append(const RopeCall& c, hipStream_t s) {
  if (c.batch <= 0) return hipSuccess;
  if (c.beside_fill) {
    k_rope_append_wave<<<dim3(c.batch, (c.hq + 2 * c.hkv + 3) / 4), 256, 0, s>>>(c);
    return hipGetLastError();
  }
  return c.d == 128 ? launch_rope_d<128>(c, s) : launch_rope_d<64>(c, s);
}

__global__ void k_slot_mapping(const int32_t* __restrict__ positions, const int32_t* __restrict__ bt, int max_blocks,
                               int batch, int bs, int nblk, int32_t* __restrict__ slots, uint32_t* err) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= batch) return;
  const int p = positions[b];
  int s = -1;
  if (p < 0 || p / bs >= max_blocks) {
    atomicOr(err, SIDP_DEVERR_POSITION);
  } else {
    const int blk = bt[(int64_t)b * max_blocks + p / bs];
    if (blk < 0 || blk >= nblk) atomicOr(err, SIDP_DEVERR_BLOCK);
    else s = blk * bs + p % bs;
  }
  slots[b] = s;
}

hipError_t launch_slot_mapping(const int32_t* positions, const int32_t* bt, int max_blocks, int batch, int bs,
                               int nblk, int32_t* slots, uint32_t* err, hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  k_slot_mapping<<<(batch + 255) / 256, 256, 0, s>>>(positions, bt, max_blocks, batch, bs, nblk, slots, err);
  return hipGetLastError();
}

}  // namespace sidp
