// Paged grouped-query decode attention on gfx950 (K4).
//
// Work is a list of items (sequence b, partition p, KV head g). A planning
// kernel, run once per set of positions, chooses the partition length: whole
// sequences when the batch alone gives every workgroup several items or the block
// tables are short, else a length that follows the tokens these positions leave to
// each workgroup and the number of items that makes.
// It lists the full partitions first and then each sequence's shorter last
// partition by decreasing length; a persistent grid of 4-wave workgroups
// walks that list in snake order (workgroup w takes items w, 2G - 1 - w,
// 2G + w, ...), which keeps the workgroups' totals within about one short item
// of each other. Many short items go to single waves instead, in the same order.
// Within an item each wave owns a quarter of the tokens,
// processed in chunks of 32 tokens = two 16-token KV blocks, with the next
// chunk's K/V loads in flight while the current one computes. The query heads of a KV group (up to
// 16) ride in the MFMA's 16 columns, so every KV byte is read once for all of
// them:
//   S^T[token][head] = K[token][:] . Q^T[:][head]   (v_mfma_f32_16x16x32_bf16)
//   O^T[dim][head]  += V^T[dim][token] . P[token][head]
// V blocks are stored transposed ([d][token]) so V^T fragments are 8-byte row
// pieces; the MFMA's k order of tokens is permuted identically on P and V^T so
// that the softmax probabilities never leave the lanes that computed them. P
// is split into high and low bf16 parts (two MFMAs), keeping the product at
// fp32-like accuracy. Softmax is online in base-2 units; the four waves of an
// item are merged in LDS; a sequence spanning several partitions is merged
// by a log-sum-exp combine kernel. Every reduction has a fixed order.
#include <hip/hip_ext.h>
#include "common.h"
#include "internal.h"

namespace sidp {

constexpr float kLog2e = 1.4426950408889634f;

// A launch is left whole (no partial records and no combine) when batch x Hkv
// items already give each of the 2 x CUs persistent workgroups four of them:
// partials written for a later merge cost HBM writes beside the KV stream that
// slow it by more than their bytes, so whole sequences win as long as the
// workgroups stay balanced. And when no sequence can be longer than kWholeTokens,
// which one workgroup reads in about the time the combine's launch takes (16
// sequences of 256-512 tokens: 20.0 us whole, 21.6 split). Nor, up to
// kWholeTable tokens, from 3 items for 16 workgroups on while a table has at
// most kWholeShare tokens for each item that a workgroup would take: there the
// second launch costs more than shorter items save. Whole / split, us a call on
// the 70B heads: 12 sequences (96 items) of 900-1100 tokens 23.1 / 24.9, of
// 1024-1535 26.8 / 26.4; 16 of 900-1100 23.9 / 27.2, of 1024-2040 33.0 / 30.5; 20
// of 1800-2047 36.0 / 42.3; 24 of 1500 32.3 / 39.2, of 64-2047 31.6 / 30.2; 128
// of 1024-2040 136.8 / 138.8; but 8 of 512-1023 20.7 / 18.1, 10 of 1500 27.2 / 22.9.
// The host sees the table, not the lengths, so one long sequence among short ones
// pays for it: 128 of 16-64 tokens and one of 2000 41 / 23.
constexpr int kWholeTokens = 768;
constexpr int kWholeTable = 2048;
constexpr int kWholeShare = 6656;
static bool attn_whole(int batch, int hkv, int max_tokens, int num_cus) {
  const int64_t items = (int64_t)batch * hkv, G = 2 * (int64_t)std::max(num_cus, 1);
  return max_tokens <= kWholeTokens || items >= 4 * G ||
         (max_tokens <= kWholeTable && items * 16 >= 3 * G && max_tokens * G <= kWholeShare * items);
}
static bool attn_whole(const AttnCall& c) {
  return attn_whole(c.batch, c.hkv, c.max_blocks * c.kv.bs, c.num_cus);
}

// Partition length of a split launch whose positions leave `mean` tokens of one
// KV head to each of the persistent workgroups: the longest 2^k or 3 * 2^k of at
// least kMinLen tokens within kShare (kShareLong from kLongMean on) times the
// mean. A workgroup alone reads five times as fast as its share of HBM when all
// read, so uneven items level out by themselves and few long items cost less
// than the starts, merges and records of many short ones, until one item takes
// as long as the whole launch should. Measured on the 70B heads (us a call, at the
// length that the mean gives / at 2048 tokens): 1 sequence of
// 2000 (mean 31, 256 taken) 18.9 / 29.3, 1 of 8000 (125, 256) 24.8 / 35.5, 2 of
// 4-8K (190, 512) 25.2 / 36.2, 8 of 0.5-2K (160, 384) 26.4 / 33.9, 5 of 4-8K
// (480, 1024) 37.1 / 43.0, 16 of 1-8K (1150, 3072) 65.8 / 73.0; at 32 of 1-8K
// (2300) 2048 is the best (119; 3072 122, 6144 130), at 64 (4600) 4096 204
// against 216 for 2048 and 210 whole, at 128 (9200) 8192 393 against 421. Neither
// multiple is best on all of 1000-2000: there items decide that just fill the CUs
// or not (12 of 8190, mean 1535: 3072 tokens 71.6, 4096 73.0, 1536 83.8).
constexpr int kMinLen = 256;
constexpr float kShare = 2.7f, kShareLong = 1.3f, kLongMean = 1500.f;
constexpr int kMaxLen = 1 << 20;  // no sequence is longer

__host__ __device__ inline int split_len(float mean) {
  const int x = (int)fminf(mean * (mean < kLongMean ? kShare : kShareLong), (float)kMaxLen);
  if (x <= kMinLen) return kMinLen;
  const int p = 1 << (31 - __builtin_clz((unsigned)x));
  return p + p / 2 <= x ? p + p / 2 : p;
}

// Whether a list of `items` takes the next longer length: it is up to a fifth
// longer than one item a CU (G workgroups, two a CU). The few CUs that get two
// items then take almost twice as long as the rest, while with the next length no
// CU gets a second one. Length by the mean / next (tokens, items: us a call on the
// 70B heads): 11 sequences of 4095 1536, 264: 52.2 / 2048, 176: 41.6; 3 of 16000
// 1536, 264: 51.4 / 2048, 192: 42.7; 12 of 3000 1024, 288: 46.1 / 1536, 192: 35.9;
// 16 of 1-8K 3072, 280: 72.8 / 4096, 224: 67.3; 3 of 1-8K 512, 272: 30.8 / 768, 184:
// 25.9. From 1.2 to 1.5 items a CU the next length is as often the slower one, and
// just past two items a CU no neighbour is the better rule (72 of 8190, 576 items
// of 8192: 438, and 412 with 2048 tokens; the rule's largest loss, with 36 of 8190
// 233 / 215 and 128 of 256-512 beside eight of 4000 88 / 80).
__host__ __device__ inline bool split_crowded(int64_t items, int G) { return 2 * items > G && 10 * items <= 6 * (int64_t)G; }
__host__ __device__ inline int next_len(int p) { return p >= kMaxLen ? p : p & (p - 1) ? p / 3 * 4 : p + p / 2; }

// With more items than workgroups and at most this many tokens an item on
// average, a wave takes an item by itself: four waves on one would each read a
// few blocks (a wave's share is at least 64 tokens, so the fourth has nothing
// from 192 tokens down) and then merge. Shared / solo, us a call on the 70B
// heads: 512 sequences of 16-64 tokens 80 / 40, 256 of 64-128 49 / 35, 100 of
// 100-300 33 / 29, 512 of 64-1024 220 / 210, 300 of 400-600 124 / 121; but 256
// of 512-2048 226 / 242, and 16 of 256-512 (128 items) 19 / 26.
// And only while the longest item has at most kSoloLongest tokens for each item
// that a workgroup would take: a lone wave walks it serially, in about the time
// a workgroup needs for one short item per 256 tokens, and the launch ends with
// it. Shared / solo: 256 sequences of 16-64 tokens (4 items a workgroup) 41.7 /
// 22.1, one of them of 512 44.6 / 33.5, 1023 45.4 / 44.6, 1500 49.6 / 59.3, 8190
// 114 / 241; 512 of 64-512 (8 items a workgroup), one of them of 2000 147.5 /
// 144.2, 3000 155 / 171, 8190 209 / 311.
constexpr float kSoloTokens = 576.f;
constexpr int kSoloLongest = 256;
__host__ __device__ inline bool attn_solo(int64_t items, float mean_tokens, int longest, int G) {
  return items > G && mean_tokens <= kSoloTokens && (int64_t)longest * G <= kSoloLongest * items;
}

// Most items a split launch lists, and so the partial records it can need. A
// length is above 2/3 of its bound, so the full partitions number below 1.5 /
// kShareLong = 1.2 per workgroup; the sequences' last ones add fewer than 4.
static int attn_item_cap(int num_cus) { return 6 * 2 * std::max(num_cus, 1); }

// One partial record per item of a split launch: the group's outputs
// o[group][D], then a 128-byte line with (m, l) of each query head, zero
// padded. Records are whole cache lines (group * D is a multiple of 64), so
// every write of a record covers whole lines: HBM has no write mask, and a
// partly written line costs the memory controller a read-modify-write.
static __host__ __device__ inline int attn_rec_floats(int group, int d) { return group * d + 32; }

size_t attn_ws_bytes(int max_batch, int hq, int hkv, int d, int max_seq, int num_cus) {
  const int64_t finest = (int64_t)max_batch * hkv * ((max_seq + kMinLen - 1) / kMinLen);
  return (size_t)std::min<int64_t>(finest, attn_item_cap(num_cus)) * attn_rec_floats(hq / hkv, d) * sizeof(float);
}

// The plan: [0] entries listed, [1] partition length, [2] whether a wave takes
// an item by itself, then for each sequence
// the index of its first full partition and of its last, shorter one, then the
// entries, b | part << 16.
constexpr int kPlanHead = 3;
static int plan_entries(int batch) { return kPlanHead + 2 * batch; }

size_t attn_plan_bytes(int max_batch, int num_cus) {
  return (size_t)(plan_entries(max_batch) + std::max(max_batch, attn_item_cap(num_cus))) * sizeof(int32_t);
}

__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

// Writes the plan. Full partitions come first, in (b, part) order; then the
// last, shorter partition of every sequence that has one, by decreasing length
// and then increasing b. Positions outside a sequence's block table give no
// entries and set the position error bit.
//
// A latency chain on an otherwise idle chip, so short: every workgroup derives
// the totals from all positions for itself, and places only its own 64
// sequences, each one's rank among the short partitions counted by four threads
// (a bitonic sort by one workgroup took 10 us at 256 sequences; this 4).
constexpr int kPlanSeqs = 64;  // sequences placed per workgroup
__global__ void __launch_bounds__(256) k_attn_plan(const int32_t* __restrict__ positions, int batch, int max_tokens,
                                                   int hkv, int G, int whole, int32_t* __restrict__ plan,
                                                   uint32_t* __restrict__ err) {
  // [batch rounded up to 16] each: keys (length << 12 | 4095 - b) of the short partitions, tokens of the sequences
  extern __shared__ __attribute__((aligned(16))) uint32_t s_key[];
  __shared__ int s_sum[4];
  __shared__ int s_longest[4];
  __shared__ int s_items[4];
  __shared__ int s_scan[4];
  __shared__ int s_short[4];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int padded = (batch + 15) & ~15;
  int* s_seq = (int*)(s_key + padded);
  const int per = (batch + 255) / 256;  // thread t owns sequences [b0, b1)
  const int b0 = min(t * per, batch), b1 = min(b0 + per, batch);
  for (int b = b0; b < b1; b++) {
    const int n = positions[b] + 1;
    s_seq[b] = n >= 1 && n <= max_tokens ? n : 0;
  }
  int sum = 0, longest = 0;  // the sum in units of 16 tokens: at most 4096 sequences of 2^20 tokens
  for (int b = b0; b < b1; b++) {
    sum += (s_seq[b] + 15) / 16;
    longest = max(longest, s_seq[b]);
  }
  sum = wave_sum_i(sum);
  longest = wave_max_i(longest);
  if (lane == 0) {
    s_sum[wave] = sum;
    s_longest[wave] = longest;
  }
  __syncthreads();
  const float tokens = 16.f * (float)(s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]);
  int ptok = kMaxLen;
  if (!whole) {
    ptok = split_len(tokens * (float)hkv / (float)G);
    int items = 0;
    for (int b = b0; b < b1; b++) items += (s_seq[b] + ptok - 1) / ptok;
    items = wave_sum_i(items);
    if (lane == 0) s_items[wave] = items;
    __syncthreads();
    if (split_crowded((int64_t)(s_items[0] + s_items[1] + s_items[2] + s_items[3]) * hkv, G)) ptok = next_len(ptok);
  }
  // full partitions of each sequence, their exclusive prefix, and the keys of the short ones
  int local = 0, shorts = 0;
  for (int b = b0; b < b1; b++) {
    const int rem = s_seq[b] % ptok;
    local += s_seq[b] / ptok;
    shorts += rem > 0;
    s_key[b] = rem > 0 ? ((uint32_t)rem << 12 | (uint32_t)(4095 - b)) : 0u;
  }
  for (int b = batch + t; b < padded; b += 256) s_key[b] = 0u;
  int incl = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  shorts = wave_sum_i(shorts);
  if (lane == 63) s_scan[wave] = incl;
  if (lane == 0) s_short[wave] = shorts;
  __syncthreads();
  const int nfull = s_scan[0] + s_scan[1] + s_scan[2] + s_scan[3];
  int run = incl - local;
  for (int w = 0; w < wave; w++) run += s_scan[w];
  if (blockIdx.x == 0 && t == 0) {
    const int listed = nfull + s_short[0] + s_short[1] + s_short[2] + s_short[3];
    plan[0] = listed;
    plan[1] = ptok;
    longest = max(max(s_longest[0], s_longest[1]), max(s_longest[2], s_longest[3]));
    plan[2] = attn_solo((int64_t)listed * hkv, tokens / (float)max(listed, 1), min(longest, ptok), G);
  }
  int32_t* first = plan + kPlanHead;
  int32_t* last = first + batch;
  int32_t* entries = last + batch;
  const int lo = blockIdx.x * kPlanSeqs, hi = min(batch, lo + kPlanSeqs);
  for (int b = b0; b < b1; b++) {
    const int full = s_seq[b] / ptok;
    if (b >= lo && b < hi) {
      if (s_seq[b] == 0) atomicOr(err, SIDP_DEVERR_POSITION);
      first[b] = run;
      for (int p = 0; p < full; p++) entries[run + p] = b | (p << 16);
    }
    run += full;
  }
  // rank of this workgroup's short partitions: four threads a sequence, each over a quarter of the keys
  const int b = lo + (t >> 2);
  const uint32_t mine = b < hi ? s_key[b] : 0u;
  int rank = 0;
  const int q = padded / 4;
  const u32x4_t* keys = (const u32x4_t*)(s_key + (t & 3) * q);
  for (int i = 0; i < q / 4; i++) {
    const u32x4_t k = keys[i];
    rank += (k[0] > mine) + (k[1] > mine) + (k[2] > mine) + (k[3] > mine);
  }
  rank += __shfl_xor(rank, 1, 64);
  rank += __shfl_xor(rank, 2, 64);
  if ((t & 3) == 0 && mine) {
    last[b] = nfull + rank;
    entries[nfull + rank] = b | ((s_seq[b] / ptok) << 16);
  }
}

template <int D>
struct Chunk {
  u32x4_t k[2][D / 32];  // K fragments: token lane&15, dims (lane>>4)*8 + 32kk
  u32x2_t v[D / 16][2];  // V^T fragments: dim 16jd + lane&15, tokens (lane>>4)*4..+3
};

// Block tables and positions are read through the scalar cache: the reads are
// uniform per wave and nothing writes those arrays during the kernel, and
// scalar loads are counted apart from the vector loads of the KV stream. (A
// vector load of a block index would have to complete before the next
// chunk's addresses exist, and vector loads complete in order, so every such
// read would drain the chunk already in flight.)
typedef const __attribute__((address_space(4))) int32_t cint32_t;

// A chunk's source: one KV head of one sequence, tokens t0 .. t0 + 31.
struct ChunkSrc {
  cint32_t* bt;
  int seq, g, t0;
};

// Loads the 24 fragments of a chunk. Every call issues the same loads, so the
// compiler's wait before a chunk's compute counts exactly the other buffer's
// loads. A block's base address is uniform (scalar registers); each lane adds
// a fixed 32-bit byte offset, k_lane or v_lane, so no 64-bit per-lane address
// is rebuilt per chunk. An out-of-range block index is replaced by block 0
// and flagged.
template <int D>
__device__ __forceinline__ void load_chunk(const AttnCall& a, const ChunkSrc& src, int64_t region_blk,
                                           uint32_t k_lane, uint32_t v_lane, bool& bad, Chunk<D>& c) {
  constexpr int KK = D / 32, JD = D / 16;
  constexpr int64_t kBlockBytes = 16 * D * 2;  // one KV head of one 16-token block, K or V
  int blk[2];
  blk[0] = src.bt[src.t0 >> 4];
  blk[1] = (src.t0 + 16 < src.seq) ? src.bt[(src.t0 >> 4) + 1] : blk[0];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    if (blk[j] < 0 || blk[j] >= a.kv.nblk) {
      bad = true;
      blk[j] = 0;
    }
  }
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const int64_t off = ((region_blk + blk[j]) * a.kv.hkv + src.g) * kBlockBytes;
    const char* kb = (const char*)a.kv.k + off;
    const char* vb = (const char*)a.kv.v + off;
    // non-temporal: each KV byte is read once per layer, and streaming loads
    // that do not allocate in the caches read HBM about 10% faster
#pragma unroll
    for (int kk = 0; kk < KK; kk++) c.k[j][kk] = __builtin_nontemporal_load((const u32x4_t*)(kb + k_lane + kk * 1024));
#pragma unroll
    for (int jd = 0; jd < JD; jd++) c.v[jd][j] = __builtin_nontemporal_load((const u32x2_t*)(vb + v_lane + jd * 512));
  }
}

// Tokens from `te` on (the end of this wave's range) are masked; a chunk that
// starts at or past `te` changes nothing: every score is -inf, so P is 0 and
// alpha is 1 (or 0 while m_run is still -inf, when o and l_run are 0 anyway:
// the exponents are then taken against 0 instead of -inf).
template <int D>
__device__ __forceinline__ void compute_chunk(const Chunk<D>& c, const bf16x8_t (&qb)[D / 32], int t0, int te,
                                              int lane, float scale, float& m_run, float& l_run,
                                              f32x4_t (&o)[D / 16]) {
  constexpr int KK = D / 32, JD = D / 16;
  const int lg = lane >> 4;
  f32x4_t s[2];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    s[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
      s[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(c.k[j][kk]), qb[kk], s[j], 0, 0, 0);
  }
  const bool tail = t0 + 32 > te;
  float cmax = -INFINITY;
#pragma unroll
  for (int j = 0; j < 2; j++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      float v = s[j][r] * scale;
      if (tail && t0 + 16 * j + lg * 4 + r >= te) v = -INFINITY;
      s[j][r] = v;
      cmax = fmaxf(cmax, v);
    }
  cmax = fmaxf(cmax, __shfl_xor(cmax, 16, 64));
  cmax = fmaxf(cmax, __shfl_xor(cmax, 32, 64));
  const float m_new = fmaxf(m_run, cmax);
  const float m_ref = m_new == -INFINITY ? 0.f : m_new;
  const float alpha = exp2f(m_run - m_ref);
  m_run = m_new;
  float p[8];
  float psum = 0.f;
#pragma unroll
  for (int r = 0; r < 4; r++) {
    p[r] = exp2f(s[0][r] - m_ref);      // slots 0..3: block 0 tokens lg*4 + r
    p[4 + r] = exp2f(s[1][r] - m_ref);  // slots 4..7: block 1 tokens lg*4 + r
    psum += p[r] + p[4 + r];
  }
  l_run = l_run * alpha + psum;
  // P as high + low bf16 parts
  uint32_t hi[4], lo[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    hi[i] = pack_bf2(p[2 * i], p[2 * i + 1]);
    lo[i] = pack_bf2(p[2 * i] - bf2f((uint16_t)(hi[i] & 0xffffu)), p[2 * i + 1] - bf2f((uint16_t)(hi[i] >> 16)));
  }
  const bf16x8_t pb = as_bf16x8(u32x4_t{hi[0], hi[1], hi[2], hi[3]});
  const bf16x8_t pl = as_bf16x8(u32x4_t{lo[0], lo[1], lo[2], lo[3]});
#pragma unroll
  for (int jd = 0; jd < JD; jd++) {
    u32x2_t v0 = c.v[jd][0], v1 = c.v[jd][1];
    if (tail) {  // invalid tokens may hold anything (NaN); zero them so 0 * V stays 0
      const int tb = t0 + lg * 4;
      if (tb + 0 >= te) v0.x &= 0xffff0000u;
      if (tb + 1 >= te) v0.x &= 0x0000ffffu;
      if (tb + 2 >= te) v0.y &= 0xffff0000u;
      if (tb + 3 >= te) v0.y &= 0x0000ffffu;
      if (tb + 16 >= te) v1.x &= 0xffff0000u;
      if (tb + 17 >= te) v1.x &= 0x0000ffffu;
      if (tb + 18 >= te) v1.y &= 0xffff0000u;
      if (tb + 19 >= te) v1.y &= 0x0000ffffu;
    }
    const bf16x8_t va = as_bf16x8(u32x4_t{v0.x, v0.y, v1.x, v1.y});
    o[jd] = o[jd] * alpha;
    o[jd] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pb, o[jd], 0, 0, 0);
    o[jd] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pl, o[jd], 0, 0, 0);
  }
}

// Item i of the work list is (entry i / Hkv of the plan, KV head i % Hkv).
// Two 4-wave workgroups per CU; a wave holds 218 VGPRs (224 allocated), so
// two of them and a slot-fill wave (at most 48) fit in a SIMD's 512.
// SOLO: a wave takes a whole item by itself, so nothing is merged in LDS and the
// waves of a workgroup go their own ways (no barrier).
template <int D, bool SOLO>
__device__ __forceinline__ void run_items(const AttnCall& a, float* smem_f) {
  constexpr int KK = D / 32, JD = D / 16;
  float* s_m = smem_f;                             // [4][16]
  float* s_l = s_m + 64;                           // [4][16]
  float* s_o = s_l + 64;                           // [4][16][D + 1]

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int head = lane & 15, lg = lane >> 4;
  const int group = a.hq / a.hkv;

  cint32_t* plan = (cint32_t*)a.plan;
  const int total_items = plan[0] * a.hkv;
  const int part_tokens = plan[1];
  cint32_t* entries = plan + kPlanHead + 2 * a.batch;
  const float scale = kLog2e / sqrtf((float)D);
  const int64_t region_blk = (int64_t)a.region * a.kv.nblk;
  cint32_t* positions = (cint32_t*)a.positions;

  // An item's parameters; all uniform. This wave's tokens are [tb, te).
  struct Item {
    int b, part, nparts, seq, g, tb, te;
    cint32_t* bt;
  };
  auto get_item = [&](int item, Item& it) {
    const int e = entries[item / a.hkv];
    it.g = item % a.hkv;
    it.b = e & 0xffff;
    it.part = e >> 16;
    it.seq = positions[it.b] + 1;
    it.nparts = (it.seq + part_tokens - 1) / part_tokens;
    it.bt = (cint32_t*)(a.block_tables + (int64_t)it.b * a.max_blocks);
    // the partition's tokens split evenly over the four waves in whole pairs of
    // 32-token chunks (only the last wave's remainder can be an odd count, whose
    // masked extra chunk re-reads HBM: non-temporal loads leave nothing in L2),
    // so a sequence's shorter last partition keeps all four waves loading
    const int len = min(it.seq - it.part * part_tokens, part_tokens);
    const int share = SOLO ? len : ((len + 3) / 4 + 63) / 64 * 64;
    it.tb = it.part * part_tokens + (SOLO ? 0 : wave * share);
    it.te = min(it.tb + share, it.part * part_tokens + len);
  };
  // the r-th item of this worker (workgroup, or wave when solo) in snake order
  // over the sorted list; a workgroup's waves are a grid apart in the list, so
  // the longest items start on different CUs
  const int worker = SOLO ? wave * (int)gridDim.x + (int)blockIdx.x : (int)blockIdx.x;
  const int workers = SOLO ? 4 * (int)gridDim.x : (int)gridDim.x;
  auto item_of = [&](int r) { return (r & 1) ? (r + 1) * workers - 1 - worker : r * workers + worker; };
  // Query heads ride in the 16 MFMA columns; lanes past the group load a
  // duplicate of the group's first head (finite values whose columns are never
  // merged or written), so the loaded fragments feed the MFMA unmodified and
  // no wait is needed until the first chunk's compute.
  auto load_q = [&](const Item& it, bf16x8_t (&q)[KK]) {
    const int qh = it.g * group + (head < group ? head : 0);
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
      q[kk] = as_bf16x8(*(const u32x4_t*)(a.q + ((int64_t)it.b * a.hq + qh) * D + lg * 8 + kk * 32));
  };

  // K fragment: token lane & 15, dims (lane >> 4) * 8 + 32 kk; V^T fragment:
  // dim 16 jd + (lane & 15), tokens (lane >> 4) * 4 .. + 3 (byte offsets).
  // K blocks are stored [d / 8][token][d % 8], so the K fragment of MFMA kk is
  // the contiguous 1 KB run of 16-byte pieces 64 kk + lane: whole cache lines
  // per load instruction, which streaming (non-temporal) loads need.
  const uint32_t k_lane = (uint32_t)lane * 16u;
  const uint32_t v_lane = (uint32_t)(head * 16 + lg * 4) * 2u;
  bool bad = false;
  int round = 0;
  int item = item_of(0);
  if (item < total_items) {
    // The chunk stream of a wave runs across its items: the load slot after an
    // item's last chunk fetches the first chunk of the wave's part of the next
    // item (or, if there is none, re-reads the last chunk: an L2 hit that keeps
    // every iteration's loads identical), so that load is in flight while the
    // item's partial results are merged and written.
    Item cur;
    get_item(item, cur);
    bf16x8_t qb[KK];
    load_q(cur, qb);
    // Wait for the first queries here, once: later the merge reuses dead
    // query registers, and a load into them still pending on some path (a
    // wave without tokens in its first item never reads qb) would make that
    // reuse wait for every load in flight.
#pragma unroll
    for (int kk = 0; kk < KK; kk++) asm volatile("" ::"v"(qb[kk]));
    Chunk<D> ca, cb;
    // (a wave without tokens in its first item reads the item's first chunk: masked)
    load_chunk<D>(a, ChunkSrc{cur.bt, cur.seq, cur.g, cur.tb < cur.te ? cur.tb : cur.part * part_tokens}, region_blk,
                  k_lane, v_lane, bad, ca);
    for (;;) {
      const int nitem = item_of(round + 1);
      const bool has_next = nitem < total_items;
      Item nx = cur;
      if (has_next) get_item(nitem, nx);
      const bool pf = has_next && nx.tb < nx.te;
      const int n = cur.te > cur.tb ? (cur.te - cur.tb + 31) / 32 : 0;  // this wave's chunks in the item
      // Chunks are taken in pairs, at least one pair per item: an odd count
      // gets a masked extra chunk, a wave without tokens two, so that every
      // path through an item issues its loads in the same order, the prefetch
      // always lands in ca, and no wait the compiler places for a register
      // reuse or copy reaches a load still in flight.
      const int n2 = __builtin_amdgcn_readfirstlane(max(2, (n + 1) & ~1));
      // source of stream slot i of this item (slot n2 is the prefetch; the
      // extra chunk and a missing prefetch re-read the last chunk, or the
      // item's first chunk when this wave has none: L2 hits)
      auto src_of = [&](int i) -> ChunkSrc {
        if (i < n) return ChunkSrc{cur.bt, cur.seq, cur.g, cur.tb + 32 * i};
        if (i == n2 && pf) return ChunkSrc{nx.bt, nx.seq, nx.g, nx.tb};
        return ChunkSrc{cur.bt, cur.seq, cur.g, n > 0 ? cur.tb + 32 * (n - 1) : cur.part * part_tokens};
      };

      float m_run = -INFINITY, l_run = 0.f;
      f32x4_t o[JD];
#pragma unroll
      for (int j = 0; j < JD; j++) o[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      int ci = 0;
      do {
        load_chunk<D>(a, src_of(ci + 1), region_blk, k_lane, v_lane, bad, cb);
        compute_chunk<D>(ca, qb, cur.tb + 32 * ci, cur.te, lane, scale, m_run, l_run, o);
        load_chunk<D>(a, src_of(ci + 2), region_blk, k_lane, v_lane, bad, ca);
        compute_chunk<D>(cb, qb, cur.tb + 32 * (ci + 1), cur.te, lane, scale, m_run, l_run, o);
        ci += 2;
      } while (ci < n2);
      // qb is dead until the next item's first chunk: load the next item's
      // queries into it (this item's again when it is the last one, so that
      // every path issues the same loads)
      load_q(nx, qb);

      l_run += __shfl_xor(l_run, 16, 64);
      l_run += __shfl_xor(l_run, 32, 64);
      if (SOLO) {
        // the output rows of a one-partition sequence, else the item's partial
        // record, straight from the accumulators (four dims of a head each)
        const bool whole = cur.nparts == 1;
        const int64_t row0 = (int64_t)cur.b * a.hq + cur.g * group;
        float* rec = a.part + (whole ? 0 : (int64_t)item * attn_rec_floats(group, D));
#pragma unroll
        for (int jd = 0; jd < JD; jd++) {
          const int d = jd * 16 + lg * 4;
          if (head >= group) continue;
          if (whole)
            *(u32x2_t*)(a.out + (row0 + head) * D + d) =
                u32x2_t{pack_bf2(o[jd][0] / l_run, o[jd][1] / l_run), pack_bf2(o[jd][2] / l_run, o[jd][3] / l_run)};
          else
            *(f32x4_t*)(rec + head * D + d) = o[jd];
        }
        if (!whole && lg == 0) {
          rec[group * D + 2 * head] = head < group ? m_run : 0.f;
          rec[group * D + 2 * head + 1] = head < group ? l_run : 0.f;
        }
        if (!has_next) break;
        cur = nx;
        item = nitem;
        round++;
        continue;
      }
      if (lg == 0) {
        s_m[wave * 16 + head] = m_run;
        s_l[wave * 16 + head] = l_run;
      }
#pragma unroll
      for (int jd = 0; jd < JD; jd++)
#pragma unroll
        for (int r = 0; r < 4; r++) s_o[(wave * 16 + head) * (D + 1) + jd * 16 + lg * 4 + r] = o[jd][r];
      __syncthreads();
      // Merge the four waves' results: the output rows of a one-partition
      // sequence, else the item's partial record (each wave writes whole
      // lines of it, the first 32 threads its (m, l) line).
      {
        const int64_t row0 = (int64_t)cur.b * a.hq + cur.g * group;  // the group's first query head
        const int rf = attn_rec_floats(group, D);
        float* rec = a.part + (int64_t)item * rf;
        for (int i = threadIdx.x; i < group * D; i += 256) {
          const int hh = i / D, d = i % D;
          float M = -INFINITY;
#pragma unroll
          for (int w = 0; w < 4; w++) M = fmaxf(M, s_m[w * 16 + hh]);
          float L = 0.f, O = 0.f;
#pragma unroll
          for (int w = 0; w < 4; w++) {
            const float mw = s_m[w * 16 + hh];
            const float f = (mw == -INFINITY) ? 0.f : exp2f(mw - M);
            L += s_l[w * 16 + hh] * f;
            O += s_o[(w * 16 + hh) * (D + 1) + d] * f;
          }
          if (cur.nparts == 1) a.out[(row0 + hh) * D + d] = f2bf(O / L);
          else rec[i] = O;
        }
        if (cur.nparts > 1 && threadIdx.x < 32) {
          const int t = threadIdx.x, hh = t >> 1;
          float v = 0.f;
          if (hh < group) {
            float M = -INFINITY;
#pragma unroll
            for (int w = 0; w < 4; w++) M = fmaxf(M, s_m[w * 16 + hh]);
            float L = 0.f;
#pragma unroll
            for (int w = 0; w < 4; w++) {
              const float mw = s_m[w * 16 + hh];
              L += s_l[w * 16 + hh] * ((mw == -INFINITY) ? 0.f : exp2f(mw - M));
            }
            v = (t & 1) ? L : M;
          }
          rec[group * D + t] = v;
        }
      }
      __syncthreads();  // s_m, s_l and s_o are reused by the next item
      if (!has_next) break;
      cur = nx;
      item = nitem;
      round++;
    }
  }
  if (bad && lane == 0) atomicOr(a.err, SIDP_DEVERR_BLOCK);
}

template <int D>
__global__ void __launch_bounds__(256, 2) k_attn(AttnCall a) {
  extern __shared__ __attribute__((aligned(16))) float smem_f[];
  if (((cint32_t*)a.plan)[2]) run_items<D, true>(a, smem_f);
  else run_items<D, false>(a, smem_f);
}

// Log-sum-exp merge of a sequence's partitions: one workgroup per (KV head,
// sequence) covering the group's query heads, four dims per thread (16-byte
// loads from the partial records). Partitions are summed in index order. Bound
// by the latency of its loads, so none waits for another: the maxima come
// first, 16 partitions at a time, then every record's terms independently.
template <int D>
__global__ void __launch_bounds__(256) k_attn_combine(AttnCall a) {
  __shared__ float s_max[16][17];
  const int g = blockIdx.x, b = blockIdx.y;
  const int group = a.hq / a.hkv;
  cint32_t* plan = (cint32_t*)a.plan;
  const int part_tokens = plan[1];
  const int seq = a.positions[b] + 1;
  if (seq < 1 || seq > a.max_blocks * a.kv.bs) return;  // position outside its block table
  const int full = seq / part_tokens, nparts = full + (seq % part_tokens > 0);
  if (nparts <= 1) return;
  const int rf = attn_rec_floats(group, D);
  // records of partitions 0 .. full - 1 are hkv * rf floats apart; the short last one has its own place
  const float* recs = a.part + ((int64_t)plan[kPlanHead + b] * a.hkv + g) * rf;
  const float* tail = a.part + (nparts > full ? ((int64_t)plan[kPlanHead + a.batch + b] * a.hkv + g) * rf : 0);
  auto rec_of = [&](int j) { return j < full ? recs + (int64_t)j * a.hkv * rf : tail; };
  {
    const int hh = threadIdx.x & 15;  // (m, l) pairs past the group are zero padding
    float M = -INFINITY;
#pragma unroll 4
    for (int j = threadIdx.x >> 4; j < nparts; j += 16) M = fmaxf(M, rec_of(j)[group * D + 2 * hh]);
    s_max[threadIdx.x >> 4][hh] = M;
    __syncthreads();
  }
  for (int i = threadIdx.x; i < group * (D / 4); i += 256) {
    const int hh = i / (D / 4), d = (i % (D / 4)) * 4;
    const int ml = group * D + 2 * hh;  // (m, l) of head hh in a record
    float M = -INFINITY;
#pragma unroll
    for (int j = 0; j < 16; j++) M = fmaxf(M, s_max[j][hh]);
    float L = 0.f;
    f32x4_t O = {0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < nparts; j0 += 8) {
      float m[8], l[8];
      f32x4_t v[8];
#pragma unroll
      for (int j = 0; j < 8; j++) {
        const float* r = rec_of(min(j0 + j, nparts - 1));
        m[j] = r[ml];
        l[j] = r[ml + 1];
        v[j] = *(const f32x4_t*)(r + hh * D + d);
      }
#pragma unroll
      for (int j = 0; j < 8; j++) {
        if (j0 + j < nparts) {
          const float f = exp2f(m[j] - M);
          L += l[j] * f;
          O += v[j] * f;
        }
      }
    }
    uint16_t* o = a.out + ((int64_t)b * a.hq + g * group + hh) * D + d;
    *(uint32_t*)o = pack_bf2(O[0] / L, O[1] / L);
    *(uint32_t*)(o + 2) = pack_bf2(O[2] / L, O[3] / L);
  }
}

AttnPlan plan_attention(const int32_t* positions, int batch, int max_tokens, int hkv, int num_cus) {
  const int G = 2 * num_cus;
  auto tokens_of = [&](int b) {  // as k_attn_plan: none for a position outside its block table
    const int64_t n = (int64_t)positions[b] + 1;
    return n >= 1 && n <= max_tokens ? (int)n : 0;
  };
  int sum = 0, longest = 0;
  for (int b = 0; b < batch; b++) {
    sum += (tokens_of(b) + 15) / 16;
    longest = std::max(longest, tokens_of(b));
  }
  const float tokens = 16.f * (float)sum;
  AttnPlan p;
  p.combine = !attn_whole(batch, hkv, max_tokens, num_cus);
  p.part_tokens = p.combine ? split_len(tokens * (float)hkv / (float)G) : kMaxLen;
  auto count = [&] {
    int n = 0;
    for (int b = 0; b < batch; b++) n += (tokens_of(b) + p.part_tokens - 1) / p.part_tokens;
    return n;
  };
  int listed = count();
  if (p.combine && split_crowded((int64_t)listed * hkv, G)) {
    p.part_tokens = next_len(p.part_tokens);
    listed = count();
  }
  p.items = listed * hkv;
  p.wave_items = attn_solo(p.items, tokens / (float)std::max(listed, 1), std::min(longest, p.part_tokens), G);
  return p;
}

hipError_t launch_attn_plan(const AttnCall& c, hipStream_t s) {
  if (c.batch <= 0) return hipSuccess;
  if (c.batch > 4096) return hipErrorInvalidValue;
  const size_t lds = (size_t)((c.batch + 15) & ~15) * 2 * sizeof(uint32_t);
  k_attn_plan<<<(c.batch + kPlanSeqs - 1) / kPlanSeqs, 256, lds, s>>>(
      c.positions, c.batch, c.max_blocks * c.kv.bs, c.hkv, 2 * c.num_cus, attn_whole(c), c.plan,
      c.err);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_d(const AttnCall& c, int grid, bool split, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const size_t lds = (size_t)(128 + 4 * 16 * (D + 1)) * 4;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)k_attn<D>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if (!start && !stop) {
    k_attn<D><<<grid, 256, lds, s>>>(c);
    if (split) k_attn_combine<D><<<dim3(c.hkv, c.batch), 256, 0, s>>>(c);
    return hipGetLastError();
  }
  // timed: the events ride on the kernels' own dispatches
  AttnCall arg = c;
  void* args[] = {&arg};
  hipError_t e = hipExtLaunchKernel((const void*)k_attn<D>, dim3(grid), dim3(256), args, lds, s, start,
                                    split ? nullptr : stop, 0);
  if (e != hipSuccess || !split) return e;
  return hipExtLaunchKernel((const void*)k_attn_combine<D>, dim3(c.hkv, c.batch), dim3(256), args, 0, s, nullptr, stop,
                            0);
}

hipError_t launch_attention(const AttnCall& c, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  if (c.batch <= 0) return hipSuccess;
  if (c.hq / c.hkv > 16) return hipErrorInvalidValue;
  const bool split = !attn_whole(c);
  const int grid = 2 * c.num_cus;  // persistent: two 4-wave workgroups per CU
  if (c.d == 128) return launch_d<128>(c, grid, split, s, start, stop);
  if (c.d == 64) return launch_d<64>(c, grid, split, s, start, stop);
  return hipErrorInvalidValue;
}

}  // namespace sidp
