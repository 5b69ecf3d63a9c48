// Dense projections of the decoder layer on gfx950 MFMA (bf16 in, fp32 accumulate):
// QKV (+bias), O (+residual), gate/up (+SwiGLU), down (+residual).
//
// Shape of the problem: out[M, N] = X[M, K] * W[N, K]^T with M = decode batch
// (8..512) and N, K in the thousands, so the weights dominate the bytes and
// every weight byte must be read exactly once. Design:
//  * Weights are packed once (into the layer's pool blob) in MFMA B-fragment
//    order: for each 64-wide k-tile, for each group of 64 output columns, for
//    each 16-wide k step, two 32x16 fragments of 64 lanes x 8 bf16. A wave
//    that owns a column group streams its weights with 1 KB fully contiguous
//    loads straight into registers (no LDS traffic for W), and the waves of a
//    grid, which move through k together, read adjacent 8 KB pieces.
//  * Activations X are shared by the 4 waves of a workgroup: staged through
//    LDS (64-wide k tiles, double buffered). A row is 128 bytes; its 16-byte
//    chunk c is stored at slot c ^ ((row >> 1) & 7), so the 16 lanes that one
//    LDS cycle serves for a 128-bit fragment read (rows r..r+15, one chunk)
//    hit 16 distinct 16-byte bank groups of the 64 four-byte banks.
//  * A workgroup covers up to 128 rows x 256 columns with 4 waves; each wave
//    holds MF x 2 accumulators of 32x32 (up to 128 rows x 64 columns) and
//    issues v_mfma_f32_32x32x16_bf16; two workgroups fit on a CU.
//  * Loads go through raw buffer resources: addresses stay in scalar
//    registers, and an offset past the buffer reads zeros (row and K tails).
//  * When the column tiles alone cannot fill the 256 CUs (N = 8192 gives 32
//    tiles), K is split; each split writes fp32 partials, which are summed in
//    split order (deterministic, so streamed and resident runs are
//    bit-identical) with the epilogue applied, either by k_splitk_reduce here
//    or by the kernel that consumes the result (the RoPE/KV-append kernel for
//    QKV, the residual + RMSNorm reduction for O and down; LinearCall's
//    defer_reduce and norm_out select this).
//  * k_gemm runs beside slot fills, on unaligned activations and where its short
//    start pays (deep_pays); other projections with the chip to themselves run on
//    k_gemm_deep (k_gemm_deep.hip), the same tiles and sums with a deeper pipeline.
//  * k_gemm_lw is the same contraction with 256-row workgroups whose weight
//    tiles are staged once per CU in LDS (direct-to-LDS loads) and shared by
//    both 128-row halves. It halves the weight loads per flop but needs twice
//    the splits at a given batch; launch_linear takes it only where k_gemm
//    would leave a quarter of the CUs idle (use_lds_weights).
#include "gemm.h"

namespace sidp {

// ---------------------------------------------------------------- packing

// Packed order of one 16-byte chunk: [KP/64 k-tiles][NG column groups][4 k
// steps][2 column halves][64 lanes] of 8 bf16 each. A k-tile's 8 KB for every
// column group are adjacent, so the waves of a grid that all stand at the same
// k-tile read one contiguous stretch of the weights (spread over every HBM
// channel) rather than one 8 KB piece in each of NG regions a group apart.

// Rows of the matrix to pack, taken from up to three sources stacked in
// order (the QKV projection packs W_q, W_k, W_v as one matrix).
struct PackRows {
  const uint16_t* w[3];
  int n[3];  // rows from each source; the packed matrix has n[0] + n[1] + n[2]
};

// W (the stacked sources, [N, K]) -> packed as above, zero padded. With GATE_UP
// the sources are gate and up [N, K] and column group j takes {gate rows 32j ..
// 32j + 31, up rows 32j .. 32j + 31}. A workgroup turns one k-tile of one
// column group: 64 rows x 128 bytes in, one contiguous 8 KB piece out, so both
// sides move whole cache lines and the turn into fragment order happens in LDS.
// HBM-bound: a 5120-wide layer (0.98 GB) packs at 5.46 TB/s of read + write in
// 357 us, the rate of a plain copy; reading in fragment order (32-byte pieces
// of 32 rows per instruction) took 960 us. Two k-tiles per workgroup 362 us,
// four 692 us (too few workgroups in flight beside 32 KB of LDS each), cached
// instead of streaming stores 380 us.
// ALIGNED: K % 8 == 0 and 16-byte aligned sources, so that a chunk is one
// 16-byte load; else a chunk is gathered by elements.
template <bool GATE_UP, bool ALIGNED>
__global__ void __launch_bounds__(256) k_pack(PackRows src, int N, int K, int NG, uint16_t* __restrict__ out) {
  __shared__ u32x4_t lds[512];
  const int ng = blockIdx.x % NG, kt = blockIdx.x / NG;
  const int c = threadIdx.x % 8;  // chunk of the row: k step c / 2, k half c % 2
  const int64_t k0 = (int64_t)kt * kBK + c * 8;
  u32x4_t v[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int r = threadIdx.x / 8 + i * 32;  // row of the column group; i is its column half
    const uint16_t* w;
    int n;
    bool in;
    if (GATE_UP) {
      n = ng * 32 + r % 32;
      in = n < N;
      w = src.w[i];
    } else {
      n = ng * 64 + r;
      in = n < N;
      int seg = 0;
      while (seg < 2 && n >= src.n[seg]) n -= src.n[seg++];
      w = src.w[seg];
    }
    v[i] = u32x4_t{0, 0, 0, 0};
    if (in && k0 < K) {
      const uint16_t* p = w + (int64_t)n * K + k0;
      if (ALIGNED) {
        v[i] = __builtin_nontemporal_load((const u32x4_t*)p);
      } else {
        uint16_t e[8];
#pragma unroll
        for (int j = 0; j < 8; j++) e[j] = k0 + j < K ? p[j] : (uint16_t)0;
#pragma unroll
        for (int j = 0; j < 4; j++) v[i][j] = e[2 * j] | ((uint32_t)e[2 * j + 1] << 16);
      }
    }
  }
  // Chunk c of a half's 32 rows is one run of 32 slots; row r sits at slot
  // (r % 32) ^ c of it, so that a row's chunks fall on different bank groups.
#pragma unroll
  for (int i = 0; i < 2; i++) lds[(i * 8 + c) * 32 + ((threadIdx.x / 8) ^ c)] = v[i];
  __syncthreads();
  u32x4_t* dst = (u32x4_t*)out + ((int64_t)kt * NG + ng) * 512;
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int p = threadIdx.x + i * 256;  // packed chunk: k step p / 128, column half, k half, row
    const int nf = p / 64 % 2, cc = p / 128 * 2 + p / 32 % 2;
    __builtin_nontemporal_store(lds[(nf * 8 + cc) * 32 + (p % 32 ^ cc)], dst + p);
  }
}

// ---------------------------------------------------------------- GEMM

// One workgroup: W waves (4, or 8 for wide unsplit launches). Wave wn
// computes rows [row0, row0 + MF*32) x the 64 packed columns of group
// tile*W + wn; the activation tile staged in LDS serves all W waves.
template <int MF, int EPI, bool PARTIAL, int W = kWaves>
__global__ void __launch_bounds__(64 * W, W > 4 ? 1 : 2) k_gemm(GemmArgs a) {
  // Issue priority over waves of lower priority on the same SIMD: in the
  // streamed step the slot-fill waves (default, lowest priority) share the
  // CUs with the projections and then take the issue slots the projection's
  // waves leave idle (0.35% more tokens/s in the step, same session).
  __builtin_amdgcn_s_setprio(3);
  constexpr int NT = 64 * W;
  constexpr int BM = MF * 32;
  constexpr int CPT = (BM * 8 + NT - 1) / NT;  // 16-byte X chunks per thread per stage (the last may be idle)
  constexpr bool kXTail = BM * 8 % NT != 0;     // 7-wave workgroups: not every thread has a last chunk
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  uint16_t* lds0 = smem;
  uint16_t* lds1 = smem + BM * kBK;

  // Workgroup id -> (column tile, split, row block). The row blocks of one
  // (tile, split) sit 8 ids apart: dispatch deals ids round-robin to the 8
  // XCDs, so they run together on one XCD and share its L2 for the weights.
  int pair, mblk;
  {
    const int L = blockIdx.x;
    const int per_group = 8 * a.mblocks;
    const int r = L % per_group;
    pair = (L / per_group) * 8 + (r % 8);
    mblk = r / 8;
    if (pair >= a.tiles * a.splits) return;
  }
  const int split = pair % a.splits;
  const int tile = pair / a.splits;
  const int row0 = mblk * BM;
  // wave index made provably uniform so weight offsets live in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wn = wave;
  const int ng = tile * W + wn;
  const bool active = ng < a.NG;
  const int KT = a.KP / kBK;
  const int kt0 = (int)((int64_t)split * KT / a.splits);
  const int kt1 = (int)((int64_t)(split + 1) * KT / a.splits);

  const __amdgpu_buffer_rsrc_t xr_rsrc = make_rsrc(a.x, (uint32_t)((size_t)a.M * a.K * 2));
  const __amdgpu_buffer_rsrc_t wr_rsrc = make_rsrc(a.w, (uint32_t)((size_t)a.NG * a.KP * 64 * 2));
  // byte offset of this wave's 8 KB piece of k-tile kt: (kt * NG + ng) * 8 KB
  const uint32_t w_base = (uint32_t)(active ? ng : 0) * 8192u;
  const uint32_t w_tile = (uint32_t)a.NG * 8192u;
  const uint32_t w_lane = (uint32_t)lane * 16u;

  // X chunks this thread stages: row r, 16-byte column chunk cc of the 64-wide k tile
  int x_row[CPT], x_cc[CPT];
#pragma unroll
  for (int i = 0; i < CPT; i++) {
    const int ci = threadIdx.x + i * NT;
    x_row[i] = (!kXTail || ci < BM * 8) ? ci >> 3 : -1;  // -1: no chunk (out of range load, no store)
    x_cc[i] = ci & 7;
  }

  f32x16_t acc[MF][2];
#pragma unroll
  for (int m = 0; m < MF; m++)
#pragma unroll
    for (int n = 0; n < 2; n++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[m][n][r] = 0.f;

  const int arow = lane & 31;
  u32x4_t xs[CPT];
  // Weight fragments of a k-tile in two halves (k steps 0-1 and 2-3). The
  // next tile's low half is fetched at the top of an iteration, its high half
  // once the current low half is consumed, so 48 registers hold weights.
  u32x4_t wlo[4], whi[4], nlo[4], nhi[4];

  auto load_x = [&](int kt) {
#pragma unroll
    for (int i = 0; i < CPT; i++) {
      const int row = row0 + x_row[i];
      const int k = kt * kBK + x_cc[i] * 8;
      const bool in = (!kXTail || x_row[i] >= 0) && row < a.M && k < a.K;  // every thread issues the load
      const uint32_t off = in ? (uint32_t)(((size_t)row * a.K + k) * 2) : kOutOfRange;
      xs[i] = buf_load16(xr_rsrc, off, 0);
    }
  };
  auto store_x = [&](uint16_t* lds) {
#pragma unroll
    for (int i = 0; i < CPT; i++) {
      const int r = x_row[i];
      if (kXTail && r < 0) continue;
      *(u32x4_t*)(lds + r * kBK + ((x_cc[i] ^ ((r >> 1) & 7)) << 3)) = xs[i];
    }
  };
  // fragments (kb, nf) of tile kt live at 1 KB * (kb * 2 + nf) in the tile's 8 KB
  auto load_w_half = [&](int kt, int half, u32x4_t (&w)[4]) {
    const uint32_t soff = w_base + (uint32_t)kt * w_tile + (uint32_t)half * 4096u;
#pragma unroll
    for (int j = 0; j < 4; j++) w[j] = buf_load16(wr_rsrc, w_lane + j * 1024u, soff);
  };
  auto mma_half = [&](const uint16_t* cur, int half, const u32x4_t (&w)[4]) {
#pragma unroll
    for (int kh = 0; kh < 2; kh++) {
      const int kb = half * 2 + kh;
      const int cc = kb * 2 + (lane >> 5);
#pragma unroll
      for (int m = 0; m < MF; m++) {
        const int r = arow + m * 32;
        const bf16x8_t af = as_bf16x8(*(const u32x4_t*)(cur + r * kBK + ((cc ^ ((r >> 1) & 7)) << 3)));
        acc[m][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, as_bf16x8(w[kh * 2 + 0]), acc[m][0], 0, 0, 0);
        acc[m][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, as_bf16x8(w[kh * 2 + 1]), acc[m][1], 0, 0, 0);
      }
    }
    if constexpr (MF == 4) {
      // Scheduling hint (mask 0x100 = LDS reads, 0x008 = MFMAs): read each
      // activation fragment two MFMA pairs ahead of its use, so that an LDS
      // read's latency hides behind matrix work instead of stalling the pipe:
      // 3 reads, then (2 MFMAs, 1 read) x 5, then the last 6 MFMAs.
      __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
      for (int i = 0; i < 5; i++) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
    }
  };

  // Every load of the k loop is issued on every path (a wait count can only
  // be exact when all paths issue the same loads): the prefetch past the
  // split's last k-tile re-reads that tile (weights, an L2 hit) or reads past
  // K (activations, out of range, zeros), and is never consumed. The loop is
  // unrolled by two so the current and next weight registers swap roles
  // without copies.
  auto step = [&](int kt, const uint16_t* cur, uint16_t* nxt, u32x4_t (&clo)[4], u32x4_t (&chi)[4],
                  u32x4_t (&plo)[4], u32x4_t (&phi)[4]) {
    const int kn = min(kt + 1, kt1 - 1);
    load_x(kt + 1);
    load_w_half(kn, 0, plo);
    if (active) mma_half(cur, 0, clo);
    load_w_half(kn, 1, phi);
    if (active) mma_half(cur, 1, chi);
    store_x(nxt);
    __syncthreads();
  };
  load_x(kt0);
  load_w_half(kt0, 0, wlo);
  load_w_half(kt0, 1, whi);
  store_x(lds0);
  __syncthreads();
  // Pairs of k-tiles, then an odd last tile outside the loop: an exit from
  // the middle of the unrolled body would give the loop header a second
  // predecessor on which the first step's weight loads are still pending,
  // and the header would wait for them on every iteration.
  int kt = kt0;
  for (; kt + 1 < kt1; kt += 2) {
    step(kt, lds0, lds1, wlo, whi, nlo, nhi);
    step(kt + 1, lds1, lds0, nlo, nhi, wlo, whi);
  }
  if (kt < kt1) step(kt, lds0, lds1, wlo, whi, nlo, nhi);

  if (!active) return;
  store_tile<MF, EPI, PARTIAL>(a, acc, row0, ng, split, lane);
}

// LDS-staged weights. One 8-wave workgroup per CU covers 256 rows x 256
// columns: waves 0-3 take rows 0-127 and waves 4-7 rows 128-255 of the same
// four column groups. Each weight fragment of a stage is fetched once per
// workgroup, straight into LDS by direct-to-LDS buffer loads (no VGPR round
// trip), and read there by the two waves that use it; the 256-row activation
// tile is staged through LDS as in k_gemm. A stage is 32 k (two MFMA k steps);
// two stages (2 x 32 KB) are in LDS at once, which leaves room beside a CU's
// slot-fill workgroup. Each stage buffer is its own LDS array, so the compiler
// can tell that reading the current stage does not depend on the direct loads
// landing in the other one.
constexpr int kLwRows = 256;                 // rows per workgroup
constexpr int kLwBK = 32;                    // k per stage
constexpr int kLwA = kLwRows * kLwBK;        // bf16 elements of a stage's activations (16 KB)
constexpr int kLwW = 4 * 4 * kFragElems;     // 4 groups x 4 fragments (16 KB)

template <int EPI, bool PARTIAL>
__global__ void __launch_bounds__(512, 1) k_gemm_lw(GemmArgs a) {
  __builtin_amdgcn_s_setprio(3);  // as k_gemm: ahead of the slot-fill waves sharing the CU
  __shared__ __attribute__((aligned(1024))) uint16_t lw_a0[kLwA];
  __shared__ __attribute__((aligned(1024))) uint16_t lw_a1[kLwA];
  __shared__ __attribute__((aligned(1024))) uint16_t lw_w0[kLwW];
  __shared__ __attribute__((aligned(1024))) uint16_t lw_w1[kLwW];

  // workgroup id -> (column tile, split, row block), row blocks 8 ids apart (as k_gemm)
  int pair, mblk;
  {
    const int L = blockIdx.x;
    const int per_group = 8 * a.mblocks;
    const int r = L % per_group;
    pair = (L / per_group) * 8 + (r % 8);
    mblk = r / 8;
    if (pair >= a.tiles * a.splits) return;
  }
  const int split = pair % a.splits;
  const int tile = pair / a.splits;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int half = wave >> 2, g = wave & 3;
  const int ng = tile * 4 + g;
  const bool active = ng < a.NG;
  const int row0 = mblk * kLwRows + half * 128;  // this wave's rows
  // the split's k range in 64-wide k-tiles (as k_gemm), walked in 32-wide stages
  const int KT = a.KP / kBK;
  const int st0 = 2 * (int)((int64_t)split * KT / a.splits);
  const int st1 = 2 * (int)((int64_t)(split + 1) * KT / a.splits);

  const __amdgpu_buffer_rsrc_t xr_rsrc = make_rsrc(a.x, (uint32_t)((size_t)a.M * a.K * 2));
  const __amdgpu_buffer_rsrc_t wr_rsrc = make_rsrc(a.w, (uint32_t)((size_t)a.NG * a.KP * 64 * 2));

  // Activations: stage rows r = 0..255, 16-byte chunks c = 0..3 (8 k each);
  // thread t stages chunks t and t + 512. In LDS a row is 64 bytes and chunk
  // c sits at slot c ^ ((r >> 2) & 3): the 16 rows one LDS cycle serves for a
  // fragment read (one chunk each) then fall on 16 distinct 16-byte bank groups.
  int x_row[2], x_cc[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int ci = threadIdx.x + i * 512;
    x_row[i] = ci >> 2;
    x_cc[i] = ci & 3;
  }
  u32x4_t xs[2];
  auto load_x = [&](int st) {
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int row = mblk * kLwRows + x_row[i];
      const int k = st * kLwBK + x_cc[i] * 8;
      const bool in = row < a.M && k < a.K;
      const uint32_t off = in ? (uint32_t)(((size_t)row * a.K + k) * 2) : kOutOfRange;
      xs[i] = buf_load16(xr_rsrc, off, 0);
    }
  };
  auto store_x = [&](uint16_t* lds) {
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int r = x_row[i];
      *(u32x4_t*)(lds + r * kLwBK + ((x_cc[i] ^ ((r >> 2) & 3)) << 3)) = xs[i];
    }
  };
  // Weights of stage st: k-tile st / 2, k steps 2 (st % 2) and + 1, so bytes
  // [4 KB (st % 2), + 4 KB) of each group's 8 KB piece: fragments (k step,
  // column half) in packed order. Wave (half, g) fetches fragments 2 half and
  // 2 half + 1 of group g into LDS fragment slot 4 g + f (1 KB each; lane l's
  // 16 bytes land at 16 l). A group past NG re-reads group 0 (its waves skip
  // the MFMAs).
  const uint32_t w_lane = (uint32_t)lane * 16u;
  const uint32_t w_group = (uint32_t)(active ? ng : 0) * 8192u;
  auto load_w = [&](int st, uint16_t* lds) {
    const uint32_t soff = (uint32_t)(st >> 1) * (uint32_t)a.NG * 8192u + w_group + (uint32_t)(st & 1) * 4096u;
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int f = half * 2 + j;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          wr_rsrc, (__attribute__((address_space(3))) void*)(lds + (g * 4 + f) * kFragElems), 16, w_lane,
          soff + (uint32_t)f * 1024u, 0, 0);
    }
  };

  f32x16_t acc[4][2];
#pragma unroll
  for (int m = 0; m < 4; m++)
#pragma unroll
    for (int n = 0; n < 2; n++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[m][n][r] = 0.f;

  const int arow = lane & 31;
  auto mma_stage = [&](const uint16_t* xa, const uint16_t* wl) {
#pragma unroll
    for (int ks = 0; ks < 2; ks++) {
      const bf16x8_t b0 = as_bf16x8(*(const u32x4_t*)(wl + (g * 4 + ks * 2 + 0) * kFragElems + lane * 8));
      const bf16x8_t b1 = as_bf16x8(*(const u32x4_t*)(wl + (g * 4 + ks * 2 + 1) * kFragElems + lane * 8));
      const int cc = ks * 2 + (lane >> 5);
#pragma unroll
      for (int m = 0; m < 4; m++) {
        const int r = half * 128 + m * 32 + arow;
        const bf16x8_t af = as_bf16x8(*(const u32x4_t*)(xa + r * kLwBK + ((cc ^ ((r >> 2) & 3)) << 3)));
        acc[m][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, b0, acc[m][0], 0, 0, 0);
        acc[m][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, b1, acc[m][1], 0, 0, 0);
      }
    }
  };

  // Stage st computes from (xa, wl) while stage st + 1 is fetched into (xn,
  // wn); every path issues the same loads (the prefetch past the split's last
  // stage re-reads that stage).
  auto step = [&](int st, const uint16_t* xa, const uint16_t* wl, uint16_t* xn, uint16_t* wn) {
    const int sn = min(st + 1, st1 - 1);
    load_x(sn);
    load_w(sn, wn);
    if (active) mma_stage(xa, wl);
    store_x(xn);
    wait_vm<0>();  // this wave's direct-to-LDS loads have landed before the barrier
    __syncthreads();
  };
  load_x(st0);
  load_w(st0, lw_w0);
  store_x(lw_a0);
  wait_vm<0>();
  __syncthreads();
  int st = st0;
  for (; st + 1 < st1; st += 2) {
    step(st, lw_a0, lw_w0, lw_a1, lw_w1);
    step(st + 1, lw_a1, lw_w1, lw_a0, lw_w0);
  }
  if (st < st1) step(st, lw_a0, lw_w0, lw_a1, lw_w1);

  if (!active) return;
  store_tile<4, EPI, PARTIAL>(a, acc, row0, ng, split, lane);
}

// Sum split-K partials in split order and apply the epilogue. VEC columns per
// thread (4 with 16-byte loads, where the sizes and pointers allow; else 1), eight
// splits' loads in flight. Outputs are numbered through the rows: with a row per
// blockIdx.y the stores of rows of odd length began inside a cache line (466 rows
// of 7193 columns 17.2 us instead of 12.5). Bound by the partials' read:
// QKV at 256 rows (3 splits, 31 MB) takes 7.4 us; one column a thread, with a
// 64-bit division for its row, took 10.4.
template <int EPI, int VEC>
__global__ void __launch_bounds__(256) k_splitk_reduce(GemmArgs a) {
  typedef float vec_t __attribute__((ext_vector_type(VEC)));
  const int NP = a.NG * 64;
  const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * VEC;
  if (idx >= (int64_t)a.M * a.N) return;
  const int row = idx >> 32 ? (int)(idx / a.N) : (int)((uint32_t)idx / (uint32_t)a.N);
  const int c = (int)(idx - (int64_t)row * a.N);
  const int64_t step = (int64_t)a.M * NP;  // from one split's partials to the next's
  const float* p = a.ws + (int64_t)row * NP + (EPI == SIDP_EPI_SWIGLU ? (c / 32) * 64 + (c % 32) : c);
  vec_t v = 0.f, u = 0.f;  // SWIGLU: gate columns and, 32 on, their up columns
  for (int s0 = 0; s0 < a.splits; s0 += 8) {
    vec_t pv[8], pu[8];
#pragma unroll
    for (int j = 0; j < 8; j++)
      if (s0 + j < a.splits) {
        pv[j] = *(const vec_t*)(p + (s0 + j) * step);
        if (EPI == SIDP_EPI_SWIGLU) pu[j] = *(const vec_t*)(p + (s0 + j) * step + 32);
      }
#pragma unroll
    for (int j = 0; j < 8; j++)
      if (s0 + j < a.splits) {
        v += pv[j];
        if (EPI == SIDP_EPI_SWIGLU) u += pu[j];
      }
  }
  if (EPI == SIDP_EPI_SWIGLU) {
#pragma unroll
    for (int j = 0; j < VEC; j++) v[j] = silu_f(v[j]) * u[j];
  } else if (EPI == SIDP_EPI_BF16 && a.bias) {
#pragma unroll
    for (int j = 0; j < VEC; j++) v[j] += bf2f(a.bias[c + j]);
  }
  if (EPI == SIDP_EPI_RESID) {
    if (a.resid) v = *(const vec_t*)(a.resid + idx) + v;
    *(vec_t*)((float*)a.out + idx) = v;
  } else if constexpr (VEC == 4) {
    *(u32x2_t*)((uint16_t*)a.out + idx) = u32x2_t{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
  } else {
    ((uint16_t*)a.out)[idx] = f2bf(v[0]);
  }
}

// Four columns a thread only where that leaves more than a workgroup and a half a
// CU. Over 83 shapes, a call's time with four columns over its time with one: at
// 262144 outputs 1.02 (128 rows of 2048 columns, 16 splits 21.6 / 20.2 us, 64 of 4096
// 20.4 / 19.2; but 257 of 1024 20.1 / 26.7), up to 400000 1.00, up to 524288 0.98,
// from 2 million on 0.95.
constexpr int64_t kVecOutputs = 400 * 1024;

template <int EPI>
static hipError_t launch_splitk_reduce(const GemmArgs& a, hipStream_t s) {
  const size_t align = EPI == SIDP_EPI_RESID ? 16 : 8;
  const bool vec = a.N % 4 == 0 && (int64_t)a.M * a.N >= kVecOutputs && (uintptr_t)a.out % align == 0 && (uintptr_t)a.resid % 16 == 0;
  const int64_t outs = (int64_t)a.M * a.N, each = vec ? 1024 : 256;  // outputs per workgroup
  const unsigned grid = (unsigned)((outs + each - 1) / each);
  if (vec) k_splitk_reduce<EPI, 4><<<grid, 256, 0, s>>>(a);
  else k_splitk_reduce<EPI, 1><<<grid, 256, 0, s>>>(a);
  return hipGetLastError();
}

// ---------------------------------------------------------------- host side

size_t packed_bytes(int n, int k) { return (size_t)round_up(n, 64) * round_up(k, 64) * 2; }

// The kernels address the packed weights and the activations through 32-bit
// buffer offsets.
bool gemm_fits(int m, int n_cols_packed, int k) {
  // the activations stay below 2^31 bytes, so the out-of-range offset 2^31
  // that rows past M and k past K read through lies past them
  constexpr size_t kLimit = (size_t)1 << 32;
  return packed_bytes(n_cols_packed, k) < kLimit && (size_t)m * round_up(k, 64) * 2 < ((size_t)1 << 31);
}


static int splits_for(int tiles, int mblocks, int KT, int num_cus);

// Whether a projection runs on k_gemm_lw (256-row workgroups, weights staged in
// LDS) rather than kernel 0 (128-row blocks, weights into registers): where kernel
// 0 would run a single unsplit round on under three quarters of the CUs, as QKV
// does from 385 rows on (160 workgroups). Alone on the chip against k_gemm_deep
// (us a call, k_gemm_lw / k_gemm_deep, its reduction included): 10240 x 8192 at
// 400, 448, 512 rows 99.8 / 97.6, 101.5 / 104.4, 108.2 / 113.4; 10240 x 5120 70.0 /
// 66.3, 73.2 / 72.6, 79.5 / 77.5. Against k_gemm, which a streamed step would have
// in its place, QKV at 512 rows takes 95-97 plus a 16 us reduction against 128-132. At
// 256 rows it is slower than k_gemm on all four 70B projections (QKV 53 against 51
// us, O 46 against 40, down 143-148 against 129-136, gate/up 318-335 against 284-309).
static bool use_lds_weights(int M, int NG, int K, int num_cus) {
  if (M <= 128 || K % 64) return false;
  const int tiles = (NG + kWaves - 1) / kWaves, mblocks = (M + 127) / 128;
  return splits_for(tiles, mblocks, K / kBK, num_cus) == 1 && (int64_t)tiles * mblocks * 4 < 3 * (int64_t)num_cus;
}

int gemm_splits(int M, int n_cols_packed, int K, int num_cus) {
  const int NG = round_up(n_cols_packed, 64) / 64;
  const bool lw = use_lds_weights(M, NG, K, num_cus);
  const int tiles = (NG + kWaves - 1) / kWaves;
  const int mblocks = lw ? (M + kLwRows - 1) / kLwRows : (M + 127) / 128;
  const int KT = round_up(K, 64) / kBK;
  return splits_for(tiles, mblocks, KT, num_cus);
}

static int splits_for(int tiles, int mblocks, int KT, int num_cus) {
  const int base = tiles * mblocks;
  // As many splits as keep the grid at most one 4-wave workgroup per CU (two
  // fit): each split writes fp32 partials for all M x N outputs, and at decode
  // batches that traffic (O at B=256: 8 splits would write and re-read 67 MB
  // beside 134 MB of weights) costs more than the second workgroup's latency
  // hiding gains. Rounding down rather than to nearest keeps a few CUs from
  // running a second workgroup after the rest have finished (O and down at
  // M=384: 192 workgroups instead of 288, the step 2% faster). On k_gemm_deep two
  // workgroups a CU are slower too (us a call, one / two: QKV 10240 x 8192 at 64,
  // 256 rows 40.2 / 45.8, 57.6 / 72.8, O 37.8 / 43.0, 50.8 / 66.0, down 83.1 / 93.9,
  // 129 / 146) but where the rounding leaves CUs idle (down at 300, 400 rows 193 /
  // 177, 214 / 203).
  int s = num_cus / base;
  if (s < 1) s = 1;
  if (s > 16) s = 16;
  if (s > KT) s = KT;
  return s;
}

size_t gemm_ws_bytes(int M, int n_cols_packed, int K, int num_cus) {
  const int s = gemm_splits(M, n_cols_packed, K, num_cus);
  if (s <= 1) return 0;
  return (size_t)s * M * round_up(n_cols_packed, 64) * sizeof(float);
}

template <bool GATE_UP>
static hipError_t launch_pack(const PackRows& src, int n, int k, int NG, void* packed, hipStream_t s) {
  bool aligned = k % 8 == 0;
  for (const uint16_t* w : src.w) aligned = aligned && (uintptr_t)w % 16 == 0;
  const unsigned grid = (unsigned)NG * (round_up(k, 64) / kBK);
  if (aligned) k_pack<GATE_UP, true><<<grid, 256, 0, s>>>(src, n, k, NG, (uint16_t*)packed);
  else k_pack<GATE_UP, false><<<grid, 256, 0, s>>>(src, n, k, NG, (uint16_t*)packed);
  return hipGetLastError();
}

hipError_t launch_pack_linear(const void* w, int n, int k, void* packed, hipStream_t s) {
  PackRows src{{(const uint16_t*)w, nullptr, nullptr}, {n, 0, 0}};
  return launch_pack<false>(src, n, k, round_up(n, 64) / 64, packed, s);
}

hipError_t launch_pack_qkv(const void* wq, const void* wk, const void* wv, int nq, int nkv, int k, void* packed,
                           hipStream_t s) {
  PackRows src{{(const uint16_t*)wq, (const uint16_t*)wk, (const uint16_t*)wv}, {nq, nkv, nkv}};
  const int n = nq + 2 * nkv;
  return launch_pack<false>(src, n, k, round_up(n, 64) / 64, packed, s);
}

hipError_t launch_pack_gate_up(const void* wg, const void* wu, int f, int k, void* packed, hipStream_t s) {
  PackRows src{{(const uint16_t*)wg, (const uint16_t*)wu, nullptr}, {f, f, 0}};
  return launch_pack<true>(src, f, k, 2 * round_up(f, 32) / 64, packed, s);
}

template <int MF, int EPI, bool P, int W = kWaves>
static hipError_t launch_mf(GemmArgs a, hipStream_t s) {
  constexpr int BM = MF * 32;
  a.mblocks = (a.M + BM - 1) / BM;
  a.tiles = (a.NG + W - 1) / W;
  const size_t lds = (size_t)2 * BM * kBK * sizeof(uint16_t);
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e =
        hipFuncSetAttribute((const void*)k_gemm<MF, EPI, P, W>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int pairs = a.tiles * a.splits;
  const int grid = (pairs + 7) / 8 * 8 * a.mblocks;
  k_gemm<MF, EPI, P, W><<<grid, 64 * W, lds, s>>>(a);
  return hipGetLastError();
}

template <int EPI, bool P>
static hipError_t launch_lw(GemmArgs a, hipStream_t s) {
  a.mblocks = (a.M + kLwRows - 1) / kLwRows;
  a.tiles = (a.NG + 3) / 4;
  const int pairs = a.tiles * a.splits;
  const int grid = (pairs + 7) / 8 * 8 * a.mblocks;
  k_gemm_lw<EPI, P><<<grid, 512, 0, s>>>(a);
  return hipGetLastError();
}

template <int EPI, bool P>
static hipError_t launch_epi(const GemmArgs& a, hipStream_t s, int wide = 0) {
  if constexpr (!P) {
    if (wide == 7) return launch_mf<4, EPI, P, 7>(a, s);
    if (wide == 8) return launch_mf<4, EPI, P, 8>(a, s);
  }
  if (wide == -1) return launch_lw<EPI, P>(a, s);
  if (a.M <= 32) return launch_mf<1, EPI, P>(a, s);
  if (a.M <= 64) return launch_mf<2, EPI, P>(a, s);
  return launch_mf<4, EPI, P>(a, s);
}

// Without a split, past 64 rows, a 7- or 8-wave workgroup (128 rows x 448 or
// 512 columns) stages each activation tile once for all its column groups, so
// a wave issues fewer loads per k step (the projections pay per load
// instruction). The width is chosen by the waves a CU runs to finish the grid:
// 4-wave workgroups go two to a CU (rounds of 8 waves), 7- and 8-wave ones one
// (rounds of 7 or 8), and a wide width is a candidate only while it gives at
// least 0.8 workgroups per CU (fewer would leave CUs idle that the model
// counts as busy); ties go to the wider one. A 70B-shaped gate/up (896 column
// groups) gets 7 waves at 256 rows, exactly 256 workgroups; a 924-group one 8. On
// k_gemm_deep (us a call, chosen width / 4 waves) gate/up 28672 x 8192 takes at 200,
// 256, 384, 512 rows 219 / 237, 216 / 251, 358 / 374, 381 / 474; at 300, where 4 waves
// leave the last rows' workgroups short, 345 / 318.
// Returns 4, 7 or 8.
static int unsplit_width(int m, int NG, int num_cus) {
  int wide = 4;
  if (m > 64) {
    const int64_t mb = (m + 127) / 128, cus = std::max(1, num_cus);
    const int64_t n4 = (NG + 3) / 4 * mb, n7 = (NG + 6) / 7 * mb, n8 = (NG + 7) / 8 * mb;
    int64_t best = (n4 + 2 * cus - 1) / (2 * cus) * 8;
    if (n7 * 10 >= 8 * cus && (n7 + cus - 1) / cus * 7 <= best) best = (n7 + cus - 1) / cus * 7, wide = 7;
    if (n8 * 10 >= 8 * cus && (n8 + cus - 1) / cus * 8 <= best) best = (n8 + cus - 1) / cus * 8, wide = 8;
  }
  return wide;
}

GemmPlan plan_linear(int m, int n, int k, int epilogue, int num_cus) {
  const int ncols = epilogue == SIDP_EPI_SWIGLU ? 2 * round_up(n, 32) : n;
  const int NG = round_up(ncols, 64) / 64;
  GemmPlan p;
  p.splits = gemm_splits(m, ncols, k, num_cus);
  p.ws_bytes = gemm_ws_bytes(m, ncols, k, num_cus);
  if (use_lds_weights(m, NG, k, num_cus)) {
    p.kernel = 1;
    p.waves = 8;
    p.rows = kLwRows;
  } else {
    p.kernel = 0;
    p.waves = p.splits == 1 ? unsplit_width(m, NG, num_cus) : kWaves;
    p.rows = p.waves > kWaves ? 128 : m <= 32 ? 32 : m <= 64 ? 64 : 128;  // launch_epi's MF
  }
  const int cols_per_wg = p.kernel == 1 ? 4 : p.waves;  // column groups per workgroup
  const int tiles = (NG + cols_per_wg - 1) / cols_per_wg;
  const int mblocks = (m + p.rows - 1) / p.rows;
  p.workgroups = (tiles * p.splits + 7) / 8 * 8 * mblocks;
  return p;
}

// Whether k_gemm_deep is the faster form of kernel 0 alone on the chip. It is not
// (us a call, weights from HBM, k_gemm / deep; two figures: two cards)
//  * where a second row block of at most kThinRows rows shares weights too large to
//    stay cached over a long k range: 8192 x 28672 at 129, 144, 160 rows 128 / 143,
//    133 / 139, 134 / 131, 6144 x 28672 98 / 114, 103 / 110, 103 / 98; a shorter range
//    14336 x 8192 at 144 73 / 64, gate/up 28672 x 8192 227 / 211;
//  * where the row blocks of a full chip have few k-tiles each (the pipeline's start,
//    three stages and two weight tiles, is then most of it): 200 rows of 4096 x 2048
//    (4 k-tiles) 23.6 / 27.1, 23.1 / 25.0, of 4096 x 4096 (8) 25.3 / 28.3, 25.3 / 25.8;
//    512 rows of 5120 x 1024 (5) 26.6 / 30.6, 26.5 / 26.5; 256 rows of 10240 x 1024
//    (5) 25.8 / 28.7, 25.0 / 27.3. With 16 to 28 k-tiles and two row blocks the deep
//    one is 4% slower on one card and 3% faster on the other; on nine tenths of a
//    chip or less (12544 x 2048, 196 workgroups) it is 3-4% faster;
//  * where some CUs get two 4-wave workgroups and no row block is ragged, or the k
//    range is short: 384 rows of 24576 x 8192 213 / 235, of a 13824 x 5120 gate/up 142
//    / 157, 512 of 18304 x 4096 114 / 120, 300 of 24576 x 1024 39.4 / 40.4; but 300 of
//    24576 x 4096 111 / 107, of an 11008 x 4096 gate/up 96.9 / 85.1;
//  * where one row block of more than kAlignedRows rows has a workgroup on every CU
//    and splits of exactly 8 or 16 k-tiles: 8192 x 8192 at 48, 64, 128 rows 34.7 / 35.8,
//    35.8 / 37.2, 42.1 / 44.5, 8192 x 4096 at 64 25.3 / 26.2, 4096 x 8192 at 64 25.6 / 26.0;
//    two resident 70B layers at 128 rows 821 / 832. (16384 x 4096 at 64 the other way,
//    34.1 / 33.5; with one more k-tile, 8192 x 8256, they are level.)
constexpr size_t kThinBytes = (size_t)150 << 20;
constexpr int kThinRows = 24;
constexpr int kThinTiles = 224;       // k-tiles
constexpr int kAlignedRows = 32;
constexpr int kAlignedTiles = 16;     // k-tiles of a split
constexpr int kFewTiles = 32;         // k-tiles of a split times the row blocks
constexpr int kFewTilesUnsplit = 32;  // k-tiles

static bool deep_pays(const GemmArgs& a, const GemmPlan& p, int num_cus) {
  const int mblocks = (a.M + p.rows - 1) / p.rows, tiles = (a.NG + p.waves - 1) / p.waves, KT = a.KP / kBK;
  const int64_t grid = (int64_t)tiles * mblocks * p.splits;
  if (mblocks == 1) {
    const int each = KT / p.splits;
    return a.M <= kAlignedRows || grid != num_cus || KT % p.splits != 0 || each % 8 != 0 || each > kAlignedTiles;
  }
  if (a.M <= 128 + kThinRows && KT >= kThinTiles && (size_t)a.NG * 64 * a.KP * 2 >= kThinBytes) return false;
  if (p.splits > 1) return grid * 10 < 9 * (int64_t)num_cus || (int64_t)KT * mblocks > kFewTiles * (int64_t)p.splits;
  return p.waves > kWaves || grid <= num_cus || (a.M % p.rows != 0 && KT > kFewTilesUnsplit);
}

hipError_t launch_linear(const LinearCall& c, hipStream_t s) {
  GemmArgs a;
  a.x = (const uint16_t*)c.x;
  a.w = (const uint16_t*)c.packed;
  a.M = c.m;
  a.K = c.k;
  a.KP = round_up(c.k, 64);
  const int ncols = c.epilogue == SIDP_EPI_SWIGLU ? 2 * round_up(c.n, 32) : c.n;
  a.NG = round_up(ncols, 64) / 64;
  a.tiles = (a.NG + kWaves - 1) / kWaves;
  a.splits = gemm_splits(c.m, ncols, c.k, c.num_cus);
  a.N = c.n;
  a.out = c.out;
  a.bias = (const uint16_t*)c.bias;
  a.resid = c.residual;
  a.ws = c.ws;
  if (!gemm_fits(c.m, ncols, c.k)) return hipErrorInvalidValue;
  if (a.splits > 1 && (size_t)a.splits * a.M * a.NG * 64 * sizeof(float) > c.ws_bytes) return hipErrorInvalidValue;
  const bool fuse_norm = c.norm_out && c.epilogue == SIDP_EPI_RESID && c.residual == c.out;
  if (c.norm_out && !fuse_norm) return hipErrorInvalidValue;
  // the kernel and width plan_linear describes: -1 the LDS-staged kernel, 7 or
  // 8 a wide unsplit k_gemm, 0 the 4-wave k_gemm
  const GemmPlan plan = plan_linear(c.m, c.n, c.k, c.epilogue, c.num_cus);
  const int wide = plan.kernel == 1 ? -1 : plan.waves > kWaves ? plan.waves : 0;
  // Beside a slot fill the shallow kernel is the faster one (both sides' times in
  // k_gemm_deep.hip); the deep one's direct-to-LDS loads need 16-byte aligned activations.
  const bool deep = plan.kernel == 0 && !c.beside_fill && (uintptr_t)c.x % 16 == 0 && deep_pays(a, plan, c.num_cus);
  hipError_t e;
  if (a.splits == 1) {
    if (deep) e = launch_gemm_deep(a, c.epilogue, plan.rows, plan.waves, s);
    else if (c.epilogue == SIDP_EPI_BF16) e = launch_epi<SIDP_EPI_BF16, false>(a, s, wide);
    else if (c.epilogue == SIDP_EPI_RESID) e = launch_epi<SIDP_EPI_RESID, false>(a, s, wide);
    else e = launch_epi<SIDP_EPI_SWIGLU, false>(a, s, wide);
    if (e != hipSuccess || !fuse_norm) return e;
    return launch_rmsnorm((const float*)c.out, c.norm_gain, c.norm_eps, c.norm_out, a.M, a.N, s);
  }
  // partials only; epilogue in the reduction
  e = deep ? launch_gemm_deep(a, c.epilogue, plan.rows, plan.waves, s) : launch_epi<SIDP_EPI_BF16, true>(a, s, wide);
  if (e != hipSuccess || c.defer_reduce) return e;
  if (fuse_norm && reduce_resid_norm_fits(a.N))
    return launch_reduce_resid_norm(a.ws, a.splits, a.M, a.NG * 64, a.N, (float*)c.out, c.norm_gain, c.norm_eps,
                                    c.norm_out, s);
  if (c.epilogue == SIDP_EPI_BF16) e = launch_splitk_reduce<SIDP_EPI_BF16>(a, s);
  else if (c.epilogue == SIDP_EPI_RESID) e = launch_splitk_reduce<SIDP_EPI_RESID>(a, s);
  else e = launch_splitk_reduce<SIDP_EPI_SWIGLU>(a, s);
  if (e != hipSuccess || !fuse_norm) return e;
  return launch_rmsnorm((const float*)c.out, c.norm_gain, c.norm_eps, c.norm_out, a.M, a.N, s);
}

}  // namespace sidp
