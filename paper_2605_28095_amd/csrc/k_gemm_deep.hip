// The projection of k_gemm (same packed weights, row blocks, column tiles,
// splits and order of every sum, so the same bits) with a deeper pipeline, for
// projections that have the chip to themselves.
//
// What bounds it: at up to 128 rows the weight stream; in wide launches of many rows
// the matrix pipe at the clock that the card's power allows (512 rows of gate/up:
// MFMA busy 72% of the time at 1.67 GHz); split launches of 256 rows neither (QKV: 31%
// busy at 2.36 GHz, 202 MB in 50 us), with one wave a SIMD on 240 CUs over 43 k-tiles.
// What k_gemm leaves idle is its k loop: activations pass through registers
// into a double-buffered stage, so every 64-wide k-tile ends with their arrival,
// LDS writes, a barrier and the first fragment reads, with nothing to multiply
// meanwhile. Here
//  * activations go straight to LDS (direct loads), into a ring of four stages,
//    three tiles ahead; one barrier per tile, which only says that the next
//    tile has landed, and no wait for anything younger than two tiles;
//  * each activation fragment is read a whole k step (8 MFMAs at 128 rows)
//    before its use, across tile boundaries too;
//  * weights are loaded two tiles ahead into the registers that the MFMAs have
//    just freed;
//  * memory instructions are issued one at a time between MFMA pairs (in bursts
//    of four to twelve they fill the address unit's queue and hold up the
//    MFMAs behind them: 512 rows of a 70B gate/up 400 us in bursts, 385 spread).
// Alone, k_gemm -> this kernel (us): gate/up 57344 x 8192 at 16, 100, 256, 512
// rows 147 -> 134, 160 -> 146, 249 -> 228, 449 -> 395; down 8192 x 28672 82 ->
// 76, 96 -> 87, 150 -> 138, 262 -> 230. Without any load the loop runs at 96% of
// the MFMA rate; three or four weight tiles ahead are no faster.
// Beside a slot fill k_gemm stays: there the layer is bound by the bytes it
// shares with the fill, and four streamed 70B layers at 256 rows took 6.95 ms
// with k_gemm against 7.05 with this kernel.
#include <type_traits>

#include "gemm.h"

namespace sidp {

// Non-temporal weight loads pay from kNtBytes of packed weights on and while at
// most kNtRowBlocks row blocks read each weight. Weights from HBM (one call after
// another over different weights, us, cached / non-temporal): 168 MB at 1, 16, 48, 64,
// 128, 256 rows 33.9 / 32.5, 35.0 / 33.7, 38.4 / 38.5, 39.4 / 40.2, 46.0 / 45.5, 58.5 /
// 57.7; 262 MB at 16, 64, 128, 256 50.8 / 47.2, 56.2 / 53.3, 64.9 / 61.2, 86.9 / 82.7; 470
// MB at 100 95.8 / 87.3; 940 MB at 16, 512 152 / 137, 392 / 393; but 134 MB at 64 37.8 /
// 39.7. Between layers and their activations more is gained: QKV of 168 MB at 256
// rows 61.5 / 57.8, a 70B layer at 64 rows 350 / 345. A caller that repeats one
// projection of up to 250 MB loses: the 256 MB memory-side cache would hold it (168 MB
// again at 64, 256 rows 35.2 / 40.0, 48.5 / 57.6); no decode step does that.
// And only where no row block is ragged: the workgroups of a part-filled last
// block load fewer activations and run ahead of their pair, whose weights then
// come from HBM again (kernel alone, us, cached / non-temporal): 470 MB at 135 rows
// 209 / 228, at 300 346 / 353; 484 MB at 135 135 / 155; 206 MB at 200 62 / 67.
constexpr int kNtRowBlocks = 4;  // kNtBytes is in gemm.h

// One workgroup: W waves (4, or 7 or 8 for wide unsplit launches). Wave wn
// computes rows [row0, row0 + MF*32) x the 64 packed columns of group
// tile*W + wn; the activation tile staged in LDS serves all W waves. WNT: the
// weights are loaded non-temporally.
template <int MF, int EPI, bool PARTIAL, int W, bool WNT>
__global__ void __launch_bounds__(64 * W, W > 4 ? 1 : 2) k_gemm_deep(GemmArgs a) {
  __builtin_amdgcn_s_setprio(3);  // as k_gemm: ahead of whatever low-priority waves share the CU
  constexpr int BM = MF * 32;
  constexpr int kXBlocks = BM * 8 / 64;            // 1 KB pieces of a stage (64 chunks of 16 bytes)
  constexpr int XJ = (kXBlocks + W - 1) / W;       // pieces each wave fetches per stage
  constexpr int XMIN = kXBlocks / W;               // and at least
  constexpr int WD = 2;                            // weight k-tiles in registers
  // vector memory instructions a wave issues after the last piece of tile
  // j + 1 and before step j: the rest of step j - 2's weights, and step j - 1's
  // weights and pieces
  constexpr int kAfter = MF == 4 ? (3 - (XJ - 1) / 2) * 2 + XJ % 2 : (4 - XJ) * 2;
  constexpr int kYounger = kAfter + 8 + XMIN;
  static_assert(8 * WD - 2 >= kAfter, "tile 2's pieces are followed by as many before step 1");
  __shared__ __attribute__((aligned(1024))) uint16_t xs0[BM * kBK];
  __shared__ __attribute__((aligned(1024))) uint16_t xs1[BM * kBK];
  __shared__ __attribute__((aligned(1024))) uint16_t xs2[BM * kBK];
  __shared__ __attribute__((aligned(1024))) uint16_t xs3[BM * kBK];

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
  const int ng = tile * W + wave;
  const bool active = ng < a.NG;  // an idle wave computes group 0 again and stores nothing
  const int KT = a.KP / kBK;
  const int kt0 = (int)((int64_t)split * KT / a.splits);
  const int kt1 = (int)((int64_t)(split + 1) * KT / a.splits);

  const __amdgpu_buffer_rsrc_t xr_rsrc = make_rsrc(a.x, (uint32_t)((size_t)a.M * a.K * 2));
  const __amdgpu_buffer_rsrc_t wr_rsrc = make_rsrc(a.w, (uint32_t)((size_t)a.NG * a.KP * 64 * 2));
  // byte offset of this wave's 8 KB piece of k-tile kt: (kt * NG + ng) * 8 KB
  const uint32_t w_base = (uint32_t)(active ? ng : 0) * 8192u;
  const uint32_t w_tile = (uint32_t)a.NG * 8192u;
  const uint32_t w_lane = (uint32_t)lane * 16u;

  // Activation pieces this wave fetches: LDS chunk p (row p / 8, slot p % 8)
  // holds the row's chunk (p % 8) ^ ((row / 2) & 7). Rows past M lie past the
  // buffer, so nothing is fetched for them (their results are not stored). Fetching
  // the last row in their place filled the address units and the MFMAs with its
  // values: over 83 shapes of cold weights 100 and 129-176 rows took 3% longer.
  uint32_t x_off[XJ];
  int x_blk[XJ];
#pragma unroll
  for (int j = 0; j < XJ; j++) {
    x_blk[j] = min(wave + j * W, kXBlocks - 1);
    const int p = x_blk[j] * 64 + lane, r = p >> 3, c = (p & 7) ^ ((r >> 1) & 7);
    x_off[j] = row0 + r < a.M ? (uint32_t)(((size_t)(row0 + r) * a.K + c * 8) * 2) : kOutOfRange;
  }

  f32x16_t acc[MF][2];
#pragma unroll
  for (int m = 0; m < MF; m++)
#pragma unroll
    for (int n = 0; n < 2; n++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[m][n][r] = 0.f;

  const int arow = lane & 31;
  u32x4_t wr[WD][8];  // weight fragments, k-tile kt in wr[kt % WD]
  u32x4_t fr[MF];     // activation fragments of the next k step

  // Fetches piece j of the wave's share of k-tile kt.
  auto dma_x = [&](int kt, int j, uint16_t* dst) {
    if (j < XMIN || wave + j * W < kXBlocks)
      buf_load16_lds(xr_rsrc, dst + x_blk[j] * kFragElems, x_off[j], (uint32_t)kt * (kBK * 2));
  };
  // The last k-tile of a K that is no multiple of 64: its pieces run past the
  // rows' ends, so zeros replace what lies past K once they have landed.
  const bool ragged = kt1 == KT && a.K % kBK != 0;
  auto zero_past_k = [&](uint16_t* st) {
    for (int p = threadIdx.x; p < BM * 8; p += 64 * W)
      if (((p & 7) ^ ((p >> 4) & 7)) >= a.K % kBK / 8) *(u32x4_t*)(st + p * 8) = u32x4_t{0, 0, 0, 0};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // fragments (kb, nf) of tile kt live at 1 KB * (kb * 2 + nf) in the tile's 8 KB
  auto load_w = [&](int kt, int kb, int nf, u32x4_t (&w)[8]) {
    const uint32_t soff = w_base + (uint32_t)kt * w_tile + (uint32_t)kb * 2048u;
    w[kb * 2 + nf] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(wr_rsrc, w_lane + nf * 1024u, soff,
                                                                                         WNT ? 2 : 0));
  };
  // Byte offset in a stage of the lane's fragment of k step kb, rows 0-31; 32
  // rows on is 4 KB further.
  uint32_t f_off[4];
#pragma unroll
  for (int kb = 0; kb < 4; kb++) f_off[kb] = arow * (kBK * 2) + (((kb * 2 + (lane >> 5)) ^ ((arow >> 1) & 7)) << 4);
  auto frag = [&](const uint16_t* st, int kb, int m) {
    return *(const u32x4_t*)((const char*)st + f_off[kb] + m * (32 * kBK * 2));
  };
  auto mma = [&](int m, const u32x4_t& f, const u32x4_t& w0, const u32x4_t& w1) {
    acc[m][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f), as_bf16x8(w0), acc[m][0], 0, 0, 0);
    acc[m][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f), as_bf16x8(w1), acc[m][1], 0, 0, 0);
  };

  const int n = kt1 - kt0;  // at least 1: there are no more splits than k-tiles
  auto kt_of = [&](int j) { return kt0 + min(j, n - 1); };  // past the end: the last tile again, not consumed
  // One k-tile from stage `xs`: on entry its weights are in `w` (or in
  // flight) and the fragments of its first k step in fr (or in flight).
  // Between the MFMAs, one memory instruction at a time: the next k step's
  // activation fragments, tile j + WD's weights into the registers that the
  // k step before has freed (the last step's, of the tile before, in `wp`),
  // and the pieces of tile j + 3.
  //
  // left: the REST-th of the last n % 4 tiles, or -1 in the main loop. There
  // are no pieces left to fetch, and the compiler drops the weight loads that
  // nothing consumes, so the waits count only what the main loop (or the loads
  // before it) issued.
  auto step = [&](auto left, int j, const uint16_t* xs, uint16_t* xn, uint16_t* xd, u32x4_t (&wp)[8],
                  u32x4_t (&w)[8]) {
    constexpr int REST = decltype(left)::value;
    // This wave's pieces of tile j + 1 have landed (fetched two tiles ago),
    // and with the barrier everybody's; everybody has also read tile j - 1,
    // whose stage the pieces of tile j + 3 go to.
    if (REST < 2) {
      wait_vm<REST == 1 ? kAfter : kYounger>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (ragged && j + 2 == n) zero_past_k(xn);
    }
    const int kx = kt_of(j + 3), kp = kt_of(j + WD - 1), kn = kt_of(j + WD);
#pragma unroll
    for (int kb = 0; kb < 4; kb++) {
      auto load_half = [&](int nf) {
        if (kb == 0) load_w(kp, 3, nf, wp);
        else load_w(kn, kb - 1, nf, w);
      };
      // the stage's base goes into the read's offset field, not into a sum kept per stage
      asm volatile("" : "+v"(f_off[(kb + 1) & 3]));
#pragma unroll
      for (int m = 0; m < MF; m++) {
        mma(m, fr[m], w[kb * 2], w[kb * 2 + 1]);
        fr[m] = kb < 3 ? frag(xs, kb + 1, m) : frag(xn, 0, m);
        __builtin_amdgcn_sched_barrier(0);  // in this order: the read is a whole k step ahead of its use
        if (m % 2 == 0) load_half(m / 2);
        if (MF == 1 || (MF == 2 && m == 1)) load_half(1);
        const int piece = MF == 4 ? kb * 2 + m / 2 : kb;
        if (REST < 0 && (MF < 4 ? m == MF - 1 : m % 2 == 1) && piece < XJ) dma_x(kx, piece, xd);
        asm volatile("" ::: "memory");  // memory instructions stay in this order: kYounger counts on it
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
#pragma unroll
  for (int t = 0; t < 3; t++)
#pragma unroll
    for (int p = 0; p < XJ; p++) dma_x(kt_of(t), p, t == 0 ? xs0 : t == 1 ? xs1 : xs2);
  asm volatile("" ::: "memory");
#pragma unroll
  for (int t = 0; t < WD; t++)
#pragma unroll
    for (int kb = 0; kb < (t < WD - 1 ? 4 : 3); kb++) {
      load_w(kt_of(t), kb, 0, wr[t]);
      load_w(kt_of(t), kb, 1, wr[t]);
    }
  wait_vm<8 * WD - 2 + XMIN>();  // the pieces of tiles 0 and 1
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (ragged && n == 1) zero_past_k(xs0);
#pragma unroll
  for (int m = 0; m < MF; m++) fr[m] = frag(xs0, 0, m);
  int j = 0;
  constexpr std::integral_constant<int, -1> kMain;
  for (; j + 3 < n; j += 4) {
    step(kMain, j, xs0, xs1, xs3, wr[3 % WD], wr[0 % WD]);
    step(kMain, j + 1, xs1, xs2, xs0, wr[0 % WD], wr[1 % WD]);
    step(kMain, j + 2, xs2, xs3, xs1, wr[1 % WD], wr[2 % WD]);
    step(kMain, j + 3, xs3, xs0, xs2, wr[2 % WD], wr[3 % WD]);
  }
  if (j < n) step(std::integral_constant<int, 0>(), j, xs0, xs1, xs3, wr[3 % WD], wr[0 % WD]);
  if (j + 1 < n) step(std::integral_constant<int, 1>(), j + 1, xs1, xs2, xs0, wr[0 % WD], wr[1 % WD]);
  if (j + 2 < n) step(std::integral_constant<int, 2>(), j + 2, xs2, xs3, xs1, wr[1 % WD], wr[2 % WD]);

  if (!active) return;
  store_tile<MF, EPI, PARTIAL>(a, acc, row0, ng, split, lane);
}

template <int MF, int EPI, bool P, int W>
static hipError_t launch_w(GemmArgs a, hipStream_t s) {
  a.mblocks = (a.M + MF * 32 - 1) / (MF * 32);
  a.tiles = (a.NG + W - 1) / W;
  const int grid = (a.tiles * a.splits + 7) / 8 * 8 * a.mblocks;
  const bool nt = (size_t)a.NG * 64 * a.KP * 2 >= kNtBytes && (a.mblocks == 1 || (a.mblocks <= kNtRowBlocks && a.M % (MF * 32) == 0));
  if (nt) k_gemm_deep<MF, EPI, P, W, true><<<grid, 64 * W, 0, s>>>(a);
  else k_gemm_deep<MF, EPI, P, W, false><<<grid, 64 * W, 0, s>>>(a);
  return hipGetLastError();
}

template <int EPI, bool P>
static hipError_t launch_rows(const GemmArgs& a, int rows, int waves, hipStream_t s) {
  if constexpr (!P) {
    if (waves == 7) return launch_w<4, EPI, P, 7>(a, s);
    if (waves == 8) return launch_w<4, EPI, P, 8>(a, s);
  }
  if (rows == 32) return launch_w<1, EPI, P, 4>(a, s);
  if (rows == 64) return launch_w<2, EPI, P, 4>(a, s);
  return launch_w<4, EPI, P, 4>(a, s);
}

hipError_t launch_gemm_deep(GemmArgs a, int epilogue, int rows, int waves, hipStream_t s) {
  if (a.splits > 1) return launch_rows<SIDP_EPI_BF16, true>(a, rows, waves, s);
  if (epilogue == SIDP_EPI_BF16) return launch_rows<SIDP_EPI_BF16, false>(a, rows, waves, s);
  if (epilogue == SIDP_EPI_RESID) return launch_rows<SIDP_EPI_RESID, false>(a, rows, waves, s);
  return launch_rows<SIDP_EPI_SWIGLU, false>(a, rows, waves, s);
}

}  // namespace sidp
