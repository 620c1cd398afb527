// Delimiter importance via attention dependency (Alg. 1 and the equation of Sec. 3) on one
// layer, for the sampled candidates, followed by the class-mean -> weight-in-tenths map.
//
// For a sampled candidate at position t the W queries that follow it, for the G query heads of
// one KV head, are W*G query rows; their logits against keys 0..t+W are a real dense contraction,
// so they run on the matrix cores: S^T tile [32 keys x 32 query rows] = K tile [32 x 128] .
// Q^T [128 x 32] as 8 MFMA 32x32x16 bf16 steps.  Keys are the MFMA "A" rows so that a lane ends up
// holding 16 keys of ONE query row: the softmax statistics (mass of all keys, of the retained region
// O_t, of the discarded region D_t) accumulate per lane with no cross-lane traffic until the very end.
//
// What bounds it: vector and matrix instructions next to each other, at the clock that the data leave.  Counted for 1024
// samples of eight sequences: per product of a key tile and a row tile 256 cycles of MFMA and 350 of vector issue (72
// instructions of a wavefront, the 16 exponentials taking two slots each), of 727 cycles that a SIMD spends, starts and
// waits included (matrix cores 35 % busy, vector ALU 48 %).  On zeros the same call takes the same cycles at 2.33 GHz, on
// random data at 1.97: 211 and 251 us.  Everything else is kept off that path:
//  - The samples of a sequence are ranked by position (latest first) and their rows packed back to back,
//    so that row tiles are full for any W*G and the samples of a workgroup end at about the same key.
//  - A workgroup (4 wavefronts x kImpNS row tiles, query operands in registers) shares every key tile
//    through LDS (two buffers of 64 rows, 16-byte chunks permuted by the row number so that the operand
//    reads touch all banks), loaded coalesced and once per kImpRows query rows.
//  - The work line -- for every KV head, every item (kImpRows rows of one sequence), every stage of 64
//    keys -- is cut into equal pieces, one per workgroup, wherever the cuts fall; a piece leaves its rows'
//    statistics in the workspace and the finishing kernel merges them.  (One workgroup per group of
//    samples left the chip idle half of the time: the latest sample has 2.5 times the mean's keys.)
//  - The exponentials are taken relative to a reference that is only moved when a tile's sum exceeds
//    kImpRescaleAt (at first, and seldom afterwards), so the usual tile has no maximum and no rescaling.
//  - The products of the next tile are issued in between the exponentials of the current one; with both
//    workgroups of a CU at work a product takes about 585 cycles of a SIMD inside the loop (440 when the other one
//    idles).  Holding the products of both row tiles at once spilled registers, leaving the MFMAs in front of the
//    branch on the kind of a tile serialised them (1.2 instead of 0.8 us per key tile).
//  - Tiles that cross a region's edge of some row (2.5 times the work) are left out of that loop and done by
//    each wavefront on its own, so that it does not hold up the others at a barrier.  A row tile of one sample has
//    two or three of them.  With fewer than 32 rows per sample a row tile holds several samples, and every tile
//    between their edges counts: 14 on average for 4 samples a row tile (128 samples of a long text), more
//    for samples far apart, which the flat kImpItemCost does not follow.
//  - Calls with few rows or short sequences run on a kernel of their own, importance_few_kernel below.
// Measured (stage IMPORTANCE, 32 query / 8 KV heads, W = 8): 128 samples of a 128K sequence 97.7 -> 57.9 us (58 to 66
// over the GPUs seen), 1024 samples of eight sequences of 24K to 64K tokens 370 -> 243 us, against one workgroup per
// 3 or 4 consecutive samples with the key tiles fetched by each wavefront; then 58.5 -> 55.0 and 235 -> 222 (both on one
// GPU) from key addresses without vector multiplies and the order of the two workgroups of a CU.  (A kImpItemCost of 6 did
// as well in these two, but took up to 8 % longer with 32 heads without groups.)  Keys straight to LDS three stages ahead
// (four buffers): 55.9 / 241 against 54.8 / 233 at that stage, latency is not what is missing; two masked tiles' keys on
// their way instead of one: no change.
#include <type_traits>

#include "dsk_common.hpp"
#include "dsk_internal.hpp"

namespace dsk {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr float kImpLog2e = 1.4426950408889634f;

struct RowStat {       // online-softmax statistics of one query row over a subset of keys
  float m;             // reference the sums are relative to (log2 units), -inf: no key seen
  float zt, zo, zd;    // sum of 2^(z-m): all causal keys, retained region, discarded region
};

__device__ __forceinline__ void stat_merge(RowStat& a, const RowStat& b) {
  const float m = fmaxf(a.m, b.m);
  const float fa = a.m == -__builtin_inff() ? 0.0f : exp2f(a.m - m);
  const float fb = b.m == -__builtin_inff() ? 0.0f : exp2f(b.m - m);
  a.zt = a.zt * fa + b.zt * fb;
  a.zo = a.zo * fa + b.zo * fb;
  a.zd = a.zd * fa + b.zd * fb;
  a.m = m;
}

constexpr int kImpThreads = 256;
constexpr int kImpWaves = kImpThreads / DSK_WAVE;
constexpr int kImpNS = kImpRows / 32 / kImpWaves;     // row tiles per wavefront
constexpr int kImpStage = 64;                         // keys per LDS buffer
constexpr int kImpMinStages = 4;                      // a piece shorter than this does not pay for its start
constexpr int kImpItemCost = 5;                       // start of an item and its tiles at the regions' edges, in stages
constexpr float kImpRescaleAt = 64.0f;
constexpr float kImpHeadroom = 4.0f;                  // log2 units a new reference lies above the largest logit seen
static_assert(kImpNS == 2, "the row tiles of a wavefront are written out below");

// low position bits left out of a sample's sort key (19 bits of it are in)
__device__ __forceinline__ int imp_slack(int L) { return L > (1 << 19) ? 13 - __clz(L - 1) : 0; }

// Lengths and cuts of the work line.  Piece w covers [seg_lo(w), seg_lo(w + 1)).
struct ImpLine {
  uint32_t per, extra;   // the first `extra` pieces have per + 1 stages, the others per
  __device__ __forceinline__ uint64_t lo(uint32_t w) const { return (uint64_t)w * per + (w < extra ? w : extra); }
  __device__ __forceinline__ uint32_t piece_of(uint64_t x) const {
    const uint64_t head = (uint64_t)extra * (per + 1);
    if (x < head) return (uint32_t)((x >> 32) ? x / (per + 1) : (uint32_t)x / (per + 1));
    const uint64_t y = x - head;
    return extra + (uint32_t)((y >> 32) ? y / per : (uint32_t)y / per);
  }
};

// exclusive prefix sum over the workgroup (one value per thread); *total = sum of all
__device__ __forceinline__ int block_excl_scan(int v, int* sm_wave, int* total) {
  const int lane = threadIdx.x & (DSK_WAVE - 1), wave = threadIdx.x / DSK_WAVE;
  const int incl = wave_incl_scan_i(v, lane);
  __syncthreads();                                    // earlier readers of sm_wave are done
  if (lane == DSK_WAVE - 1) sm_wave[wave] = incl;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kImpWaves; ++w) {
    before += w < wave ? sm_wave[w] : 0;
    all += sm_wave[w];
  }
  *total = all;
  return before + incl - v;
}

// logits of a key tile against one row tile: kf[u] = channels [64*hf + 8u, +8) of key `col`
__device__ __forceinline__ f32x16_t imp_product(const bf16x8_t (&kf)[8], const bf16x8_t (&qf)[8]) {
  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u], qf[u], acc, 0, 0, 0);
  return acc;
}

__device__ __forceinline__ float imp_tile_sum(const f32x16_t& acc, float scale_log2, float m) {
  float e[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) e[r] = __builtin_amdgcn_exp2f(fmaf(acc[r], scale_log2, -m));
  float a = e[0], b = e[1], c = e[2], d = e[3];       // four chains of four, fixed order
#pragma unroll
  for (int r = 4; r < 16; r += 4) { a += e[r]; b += e[r + 1]; c += e[r + 2]; d += e[r + 3]; }
  return (a + b) + (c + d);
}

struct RowAcc {          // of one lane: 16 keys in 32 of one query row
  float m, zf;           // reference; mass of tiles that lie wholly in the discarded region
  float zt, zo, zd;      // masses from the other tiles
};

// the tile's sum is too large for the reference (or there is none yet): move it above the largest logit
__device__ __forceinline__ void imp_move_reference(RowAcc& st, const f32x16_t& acc, float scale_log2) {
  float top = acc[0] * scale_log2;
#pragma unroll
  for (int r = 1; r < 16; ++r) top = fmaxf(top, acc[r] * scale_log2);
  const float mn = top > st.m ? top + kImpHeadroom : st.m;
  const float f = mn == st.m ? 1.0f : __builtin_amdgcn_exp2f(st.m - mn);   // 0 while there is none
  st.zf *= f; st.zt *= f; st.zo *= f; st.zd *= f;
  st.m = mn;
}

__device__ __forceinline__ bool imp_too_large(float sum) { return __any(!(sum <= kImpRescaleAt)); }

// a tile that crosses a region's edge, the causal edge or the end of the sequence.  Bounds count from
// the lane's first key of the tile: keys <= kmax exist, >= o_lo and <= t are retained, <= d_hi discarded.
__device__ __forceinline__ void imp_masked_tile(RowAcc& st, f32x16_t z, float scale_log2, int kmax, int o_lo, int t,
                                                int d_hi) {
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = kmax >= 8 * (r / 4) + (r % 4) ? z[r] : -__builtin_inff();
  float zt, zo, zd;
  auto sums = [&]() {
    zt = zo = zd = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int k = 8 * (r / 4) + (r % 4);
      float e = __builtin_amdgcn_exp2f(fmaf(z[r], scale_log2, -st.m));
      zt += e;
      zd += d_hi >= k ? e : 0.0f;
      e = t >= k ? e : 0.0f;
      zo += o_lo <= k ? e : 0.0f;
    }
  };
  sums();
  if (imp_too_large(zt)) {
    imp_move_reference(st, z, scale_log2);
    sums();
    // a lane without any key so far still has no reference and no number here; it adds nothing
    if (st.m == -__builtin_inff()) zt = zo = zd = 0.0f;
  }
  st.zt += zt; st.zo += zo; st.zd += zd;
}

// The plan, in the workspace (ints):
//   head [0] stages of all items of one KV head, [1] pieces, [2] items of one KV head
//   n_valid [nseq], first item of each sequence [nseq + 1], first unit of each item [items + 1]
//   rank of each sample [nseq * n_samp] (-1 = absent), samples by rank [nseq * n_samp], their positions
struct ImpPlan {
  int32_t *head, *n_valid, *item_base, *item_at, *rank, *order, *pos;
};
__host__ __device__ __forceinline__ ImpPlan imp_plan(int32_t* w, int nseq, int n_samp, int items) {
  ImpPlan p;
  p.head = w;
  p.n_valid = w + 4;
  p.item_base = p.n_valid + nseq;
  p.item_at = p.item_base + nseq + 1;
  p.rank = p.item_at + items + 1;
  p.order = p.rank + (int64_t)nseq * n_samp;
  p.pos = p.order + (int64_t)nseq * n_samp;
  return p;
}

// sort key of a sample at position t: position, then the smaller index; 0 = absent
__device__ __forceinline__ uint32_t imp_key(bool have, int t, int slack, int i) {
  return have ? (((uint32_t)t >> slack) + 1u) << 12 | (uint32_t)(4095 - i) : 0u;
}

// keys among quads [lo, hi) of a table that are larger than `key`
__device__ __forceinline__ int imp_count_larger(const uint32_t* table, int lo, int hi, uint32_t key) {
  const uint4* keys = reinterpret_cast<const uint4*>(table);
  int c = 0;
  for (int j = lo; j < hi; ++j) {
    const uint4 o = keys[j];
    c += (o.x > key ? 1 : 0) + (o.y > key ? 1 : 0) + (o.z > key ? 1 : 0) + (o.w > key ? 1 : 0);
  }
  return c;
}

// The samples of a sequence ranked by position, latest first: 64 samples per workgroup, counted by its
// four wavefronts against a quarter of the sequence's samples each.  grid: (64 samples, sequence)
__global__ __launch_bounds__(kImpThreads) void importance_rank_kernel(
    const int32_t* __restrict__ samp_pos, const int32_t* __restrict__ cu_seqlens, int seq_first, int nseq, int n_samp,
    int items, int32_t* __restrict__ plan) {
  __shared__ __attribute__((aligned(16))) uint32_t sm_key[kImpMaxSamples];
  __shared__ int sm_rank[DSK_WAVE], sm_n;
  const ImpPlan pl = imp_plan(plan, nseq, n_samp, items);
  const int s = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid & (DSK_WAVE - 1), wave = tid / DSK_WAVE;
  const int ns4 = (n_samp + 3) & ~3;
  const int seq0 = cu_seqlens[seq_first + s];
  const int L = cu_seqlens[seq_first + s + 1] - seq0;
  const int slack = imp_slack(L);
  const int32_t* pos = samp_pos + (int64_t)(seq_first + s) * n_samp;
  if (tid < DSK_WAVE) sm_rank[tid] = 0;
  if (tid == 0) sm_n = 0;
  __syncthreads();
  int n = 0;
  for (int i = tid; i < ns4; i += kImpThreads) {
    const int tg = i < n_samp ? pos[i] : -1;
    const bool have = tg >= 0 && tg - seq0 >= 0 && tg - seq0 < L;
    sm_key[i] = imp_key(have, tg - seq0, slack, i);
    n += have ? 1 : 0;
  }
  if (n > 0) atomicAdd(&sm_n, n);
  __syncthreads();
  const int i = blockIdx.x * DSK_WAVE + lane;
  const uint32_t key = i < n_samp ? sm_key[i] : 0u;
  const int quads = ns4 / 4;
  const int c = imp_count_larger(sm_key, wave * quads / kImpWaves, (wave + 1) * quads / kImpWaves, key);
  atomicAdd(&sm_rank[lane], c);
  __syncthreads();
  if (wave == 0 && i < n_samp) {
    const int r = sm_rank[lane];
    pl.rank[s * n_samp + i] = key != 0 ? r : -1;
    if (key != 0) {
      pl.order[s * n_samp + r] = i;
      pl.pos[s * n_samp + r] = pos[i] - seq0;
    }
  }
  if (blockIdx.x == 0 && tid == 0) pl.n_valid[s] = sm_n;
}

// grid: persistent workgroups, one piece of the work line each.  OWN_RANK (one sequence of at most
// kImpThreads samples): every workgroup ranks the samples itself, which takes it 1 us, instead of a
// launch in front (63.0 -> 57.7 us for the stage at 128 samples of a 128K sequence, 32 heads).
template <bool OWN_RANK>
__global__ __launch_bounds__(kImpThreads, 2) void importance_kernel(
    const uint16_t* __restrict__ K, int64_t kst, int64_t ksh, const uint16_t* __restrict__ qwin,
    const int32_t* __restrict__ samp_pos, const int32_t* __restrict__ cu_seqlens, int seq_first, int nseq, int n_samp, int items, int W, int R, int Hq, int G,
    int Hkv, float scale_log2, int32_t* __restrict__ plan, float4* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint16_t sm_k[2][kImpStage][DSK_HEAD_DIM];
  __shared__ int sm_ib[kImpMaxSeqs + 1];         // first item of each sequence
  __shared__ int sm_nv[kImpMaxSeqs];             // its samples
  __shared__ int sm_wave[kImpWaves];
  __shared__ int sm_cur[2];

  const ImpPlan pl = imp_plan(plan, nseq, n_samp, items);
  const int tid = threadIdx.x;
  const int lane = tid & (DSK_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / DSK_WAVE);
  const int rps = W * G;                          // query rows of one (sample, KV head)

  __shared__ uint16_t sm_order[OWN_RANK ? kImpThreads : 1];   // the plan's order and positions
  __shared__ int sm_pos[OWN_RANK ? kImpThreads : 1];
  auto order_of = [&](int s, int j) { return OWN_RANK ? (int)sm_order[j] : pl.order[s * n_samp + j]; };
  auto pos_of = [&](int s, int j) { return OWN_RANK ? sm_pos[j] : pl.pos[s * n_samp + j]; };
  int own_valid = 0;
  if constexpr (OWN_RANK) {
    uint32_t* sm_key = reinterpret_cast<uint32_t*>(&sm_k[0][0][0]);
    const int seq0 = cu_seqlens[seq_first];
    const int L = cu_seqlens[seq_first + 1] - seq0;
    const int tg = tid < n_samp ? samp_pos[(int64_t)seq_first * n_samp + tid] : -1;
    const int t = tg - seq0;
    const bool have = tg >= 0 && t >= 0 && t < L;
    const uint32_t key = imp_key(have, t, imp_slack(L), tid);
    sm_key[tid] = key;
    const int in_wave = __popcll(__ballot(have));
    if (lane == 0) sm_wave[wave] = in_wave;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kImpWaves; ++w) own_valid += sm_wave[w];
    const int rank = imp_count_larger(sm_key, 0, (n_samp + 3) / 4, key);
    if (have) { sm_order[rank] = (uint16_t)tid; sm_pos[rank] = t; }
    if (blockIdx.x == 0 && tid < n_samp) pl.rank[tid] = have ? rank : -1;
    __syncthreads();
  }

  // ---- the work line, the same in every workgroup ----------------------------------------------
  int n_list;                                     // items of one KV head
  {
    const int nv = OWN_RANK ? (tid == 0 ? own_valid : 0) : (tid < nseq ? pl.n_valid[tid] : 0);
    const int at = block_excl_scan((nv * rps + kImpRows - 1) / kImpRows, sm_wave, &n_list);
    if (tid < nseq) { sm_ib[tid] = at; sm_nv[tid] = nv; }
    if (tid == 0) sm_ib[nseq] = n_list;
  }
  __syncthreads();
  if (n_list == 0) {                              // no sample anywhere
    if (blockIdx.x == 0 && tid < 4) pl.head[tid] = 0;
    return;
  }
  auto seq_of = [&](int item) {
    int a = 0, b = nseq - 1;
    while (a < b) {
      const int mid = (a + b + 1) >> 1;
      if (sm_ib[mid] <= item) a = mid; else b = mid - 1;
    }
    return a;
  };
  // stages of 64 keys up to the item's latest query, and its length on the line
  auto stages_of = [&](int item, int s) {
    const int j0 = (item - sm_ib[s]) * kImpRows / rps;
    const int L = cu_seqlens[seq_first + s + 1] - cu_seqlens[seq_first + s];
    const int t = pos_of(s, j0) | ((1 << imp_slack(L)) - 1);   // no later one in the item
    return (t < L - 1 - W ? t + W : L - 1) / kImpStage + 1;
  };
  const int per_thread = (n_list + kImpThreads - 1) / kImpThreads;
  const int item_lo = tid * per_thread < n_list ? tid * per_thread : n_list;
  const int item_hi = item_lo + per_thread < n_list ? item_lo + per_thread : n_list;
  int own = 0;
  for (int it = item_lo; it < item_hi; ++it) own += stages_of(it, seq_of(it)) + kImpItemCost;
  int T1;
  const int own_at = block_excl_scan(own, sm_wave, &T1);
  const uint64_t T = (uint64_t)T1 * Hkv;
  uint32_t nw = gridDim.x;
  if (T / kImpMinStages < nw) nw = T / kImpMinStages > 0 ? (uint32_t)(T / kImpMinStages) : 1u;
  if (nw >= 8) nw &= ~7u;
  ImpLine line;
  line.per = (uint32_t)(T / nw);
  line.extra = (uint32_t)(T % nw);
  if (blockIdx.x == 0) {
    if (tid == 0) { pl.head[0] = T1; pl.head[1] = (int)nw; pl.head[2] = n_list; }
    for (int s = tid; s <= nseq; s += kImpThreads) pl.item_base[s] = sm_ib[s];
    int at = own_at;
    for (int it = item_lo; it < item_hi; ++it) { pl.item_at[it] = at; at += stages_of(it, seq_of(it)) + kImpItemCost; }
    if (tid == 0) pl.item_at[n_list] = T1;
  }
  if (blockIdx.x >= nw) return;                   // uniform over the workgroup
  // workgroup 8j + i runs on XCD i: neighbouring pieces, which read the same keys, go to one L2
  const uint32_t piece = nw >= 8 ? (blockIdx.x & 7) * (nw >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  uint64_t x = line.lo(piece);
  const uint64_t x_end = line.lo(piece + 1);
  int hk = (int)(x / (uint32_t)T1);
  {
    const int rem = (int)(x - (uint64_t)hk * T1);
    if (rem >= own_at && rem < own_at + own) {
      int at = own_at;
      for (int it = item_lo; it < item_hi; ++it) {
        const int len = stages_of(it, seq_of(it)) + kImpItemCost;
        if (rem < at + len) { sm_cur[0] = it; sm_cur[1] = rem - at; break; }
        at += len;
      }
    }
  }
  __syncthreads();
  int item = __builtin_amdgcn_readfirstlane(sm_cur[0]);
  int at = __builtin_amdgcn_readfirstlane(sm_cur[1]);        // units into the item

  // the later row tiles of an item have fewer keys: the second workgroup of a CU deals its tiles to the
  // SIMDs the other way round
  const int own_tile = (blockIdx.x * 2 >= gridDim.x ? kImpWaves - 1 - wave : wave) * kImpNS;
  // Most likely the second workgroup of its CU, which goes first in three stages of four (below): where a row tile holds rows
  // of one sample and pieces are long.  Row tiles that samples share leave much work behind the stages, at each wavefront's
  // own pace, and a priority then costs as often as it gains.  600 random calls, time against none, mean / largest: 32, 64 ..
  // rows a sample, pieces of 8 stages and more 0.97 / 0.99, shorter ones 1.00 / 1.02; up to 20 rows, 64 stages and more 0.985
  // / 1.01 (1.09 among 52 others), fewer 0.99 / 1.07; 40, 56, 72 .. rows 1.00 / 1.10.
  const bool young = rps % 32 == 0 && line.per >= 8 && blockIdx.x * 2 >= gridDim.x;
  const int col = lane & 31;        // query row of the tile this lane accumulates; key row of its A operand
  const int hf = lane >> 5;         // channel half / key sub-row selector
  // LDS: chunk c (16 bytes) of key row r lies in slot c ^ (r & 15) of the row
  const int ld_row = tid >> 4, ld_slot = ((tid & 15) ^ ld_row) * 8;   // rows ld_row + 0, 16, 32, 48
  const unsigned ld_off = ((unsigned)ld_row * (unsigned)kst + (unsigned)(tid & 15) * 8u) * 2u;
  static_assert(kImpThreads == 256 && kImpStage == 64, "a thread stages four 16-byte chunks");
  const int rd_slot = (hf * 8) ^ (col & 15);

  while (x < x_end) {
    const int s = __builtin_amdgcn_readfirstlane(seq_of(item));
    const int seq = seq_first + s;
    const int seq0 = __builtin_amdgcn_readfirstlane(cu_seqlens[seq]);
    const int L = __builtin_amdgcn_readfirstlane(cu_seqlens[seq + 1]) - seq0;
    const int item_st = __builtin_amdgcn_readfirstlane(stages_of(item, s));
    // a cut among the units of the item's cost, behind its stages, leaves the next piece no stage of it
    const int end = (uint64_t)(item_st + kImpItemCost - at) < x_end - x ? item_st + kImpItemCost : at + (int)(x_end - x);
    const int st_at = at < item_st ? at : item_st;
    const int st_end = end < item_st ? end : item_st;
    const char* Kh = reinterpret_cast<const char*>(K + (int64_t)hk * ksh + (int64_t)seq0 * kst);     // uniform

    // first stage -> registers
    uint4 kreg0, kreg1, kreg2, kreg3;
    auto load_stage = [&](int st) {
      if ((st + 1) * kImpStage <= L) {            // uniform bases + one 32-bit lane offset (kst <= 2^24, host-checked)
        const char* base = Kh + (int64_t)st * kImpStage * kst * 2;
        kreg0 = *reinterpret_cast<const uint4*>(base + ld_off);
        kreg1 = *reinterpret_cast<const uint4*>(base + 32 * kst + ld_off);
        kreg2 = *reinterpret_cast<const uint4*>(base + 64 * kst + ld_off);
        kreg3 = *reinterpret_cast<const uint4*>(base + 96 * kst + ld_off);
      } else {                                    // stay inside the sequence (the stage may lie behind it); masked below
        auto row_at = [&](int row) {
          row += st * kImpStage;
          return *reinterpret_cast<const uint4*>(Kh + ((int64_t)(row < L ? row : L - 1) * kst + (tid & 15) * 8) * 2);
        };
        kreg0 = row_at(ld_row);
        kreg1 = row_at(ld_row + 16);
        kreg2 = row_at(ld_row + 32);
        kreg3 = row_at(ld_row + 48);
      }
    };
    auto store_stage = [&](int buf) {
      *reinterpret_cast<uint4*>(&sm_k[buf][ld_row][ld_slot]) = kreg0;
      *reinterpret_cast<uint4*>(&sm_k[buf][ld_row + 16][ld_slot]) = kreg1;
      *reinterpret_cast<uint4*>(&sm_k[buf][ld_row + 32][ld_slot]) = kreg2;
      *reinterpret_cast<uint4*>(&sm_k[buf][ld_row + 48][ld_slot]) = kreg3;
    };
    load_stage(st_at);

    // this wavefront's row tiles: row rho of the sequence's packed rows is row rho % rps of the
    // (rho / rps)-th latest sample -- window position w = r / G, head g = r % G
    bf16x8_t qf[kImpNS][8];
    int tt[kImpNS], kmax[kImpNS];                 // per lane: position of the sample, last key of the row (-1: no row)
    int t_lo[kImpNS], t_hi[kImpNS], last[kImpNS]; // per tile: smallest and largest position, last key of any row
    // (first qf[p][i] = row 4i + lane / 16 of the tile, chunk lane % 16)
#pragma unroll
    for (int p = 0; p < kImpNS; ++p) {
      const int rho = (item - sm_ib[s]) * kImpRows + (own_tile + p) * 32 + col;
      const int j = rho / rps;
      const bool ok = j < sm_nv[s];               // the packed rows end with the last sample's
      const int jn = ok ? order_of(s, j) : 0;
      const int t = ok ? pos_of(s, j) : 0;
      const int r = rho - j * rps;
      const int w = ok ? r / G : 0, g = ok ? r - (r / G) * G : 0;
      tt[p] = t;
      kmax[p] = ok ? (t < L - 2 - w ? t + 1 + w : L - 1) : -1;
      t_lo[p] = (int)wave_min_u(ok ? (uint32_t)t : 0x7FFFFFFFu);
      t_hi[p] = (int)wave_max_u((uint32_t)t);
      last[p] = (int)wave_max_u((uint32_t)(kmax[p] + 1)) - 1;
      // the row among all query rows
      const int64_t row_at = (((int64_t)seq * n_samp + jn) * W + w) * Hq + hk * G + g;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int from = 4 * i + (lane >> 4);
        const int64_t at_i = (int64_t)__shfl((int)(row_at >> 32), from, DSK_WAVE) << 32 |
                             (uint32_t)__shfl((int)row_at, from, DSK_WAVE);
        qf[p][i] = *reinterpret_cast<const bf16x8_t*>(qwin + at_i * DSK_HEAD_DIM + (lane & 15) * 8);
      }
    }
    __syncthreads();                              // readers of the previous piece are done
    // rows -> operand layout through the wavefront's own quarter of the key buffers
    uint16_t* sm_own = &sm_k[0][0][0] + wave * (32 * DSK_HEAD_DIM);
    static_assert(sizeof(sm_k) == kImpWaves * 32 * DSK_HEAD_DIM * sizeof(uint16_t), "a row tile per wavefront");
#pragma unroll
    for (int p = 0; p < kImpNS; ++p) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int row = 4 * i + (lane >> 4);
        *reinterpret_cast<bf16x8_t*>(sm_own + row * DSK_HEAD_DIM + ((lane & 15) ^ (row & 15)) * 8) = qf[p][i];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < 8; ++u)
        qf[p][u] = *reinterpret_cast<const bf16x8_t*>(sm_own + col * DSK_HEAD_DIM + (rd_slot ^ u) * 8);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    RowAcc acc_st[kImpNS];
#pragma unroll
    for (int p = 0; p < kImpNS; ++p) {
      acc_st[p].m = -__builtin_inff();
      acc_st[p].zf = acc_st[p].zt = acc_st[p].zo = acc_st[p].zd = 0.0f;
    }

    __syncthreads();
    store_stage(0);
    if (st_at + 1 < st_end) load_stage(st_at + 1);
    __syncthreads();

    auto read_keys = [&](bf16x8_t (&kf)[8], int buf, int tile) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
        kf[u] = *reinterpret_cast<const bf16x8_t*>(&sm_k[buf][tile * 32 + col][(rd_slot ^ u) * 8]);
    };
    // what a tile is to row tile p: nothing (0), wholly discarded (1) or retained (2) by all rows, mixed (3)
    auto kind_of = [&](int p, int k0) {
      if (k0 > last[p]) return 0;
      if (k0 + 31 <= (t_lo[p] - R > 0 ? t_lo[p] - R : 0)) return 1;
      return k0 > t_hi[p] - R && k0 + 31 <= t_lo[p] && k0 > 0 ? 2 : 3;   // key 0 may be in both regions
    };
    // statistics of the tile at key k0 for row tile p (logits cur) in the shadow of the products that the
    // caller's next half step needs: nxt = keys kf against row tile o.  FRESH: kf was only just requested
    // from LDS, so the products are held back behind the first exponentials.
    auto half_step = [&](auto fresh, int p, int o, int k0, const f32x16_t& cur, f32x16_t& nxt, const bf16x8_t (&kf)[8]) {
      const int kind = kind_of(p, k0);
      if (kind == 1 || kind == 2) {
        // no masks: one sum per row feeds the total and one of the regions
        nxt = imp_product(kf, qf[o]);
        float sum = imp_tile_sum(cur, scale_log2, acc_st[p].m);
        if constexpr (decltype(fresh)::value) {
          __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);      // vector ALU
          __builtin_amdgcn_sched_group_barrier(0x400, 6, 0);    // exponentials
          __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);    // MFMA
            __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
          }
        }
        if (imp_too_large(sum)) {
          imp_move_reference(acc_st[p], cur, scale_log2);
          sum = imp_tile_sum(cur, scale_log2, acc_st[p].m);
        }
        if (kind == 1) {
          acc_st[p].zf += sum;
        } else {
          acc_st[p].zt += sum;
          acc_st[p].zo += sum;
        }
      } else if (k0 <= last[o]) {
        nxt = imp_product(kf, qf[o]);
      }
    };
    constexpr std::true_type kFresh{};
    constexpr std::false_type kReady{};
    bf16x8_t kf[8];
    f32x16_t c0, c1;
    read_keys(kf, 0, 0);
    c0 = imp_product(kf, qf[0]);
    c1 = c0;
    for (int st = st_at; st < st_end; ++st) {
      const int buf = (st - st_at) & 1;
      const int k0 = st * kImpStage;
      // The older of two wavefronts issues first: pieces of the second workgroup of a CU took a third longer than those
      // of the first, which then left it alone.  Three stages in four the younger one goes first: 57.8 -> 55.0 us,
      // 232 -> 222 for the two cases above; 212 calls with 32, 64 and 128 rows a sample 0.99 -> 0.97 of the time with
      // multiplied addresses in the mean, 1.02 at most.
      if (young) {
        if ((st & 3) != 0) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
      }
      half_step(kReady, 0, 1, k0, c0, c1, kf);
      read_keys(kf, buf, 1);
      half_step(kFresh, 1, 0, k0, c1, c0, kf);
      half_step(kReady, 0, 1, k0 + 32, c0, c1, kf);
      if (st + 1 < st_end) store_stage(buf ^ 1);  // read last before the previous barrier
      __syncthreads();
      if (st + 2 < st_end) load_stage(st + 2);
      read_keys(kf, buf ^ 1, 0);                  // past the end: old keys, their products are not used
      half_step(kFresh, 1, 0, k0 + 32, c1, c0, kf);
    }
    __builtin_amdgcn_s_setprio(0);
    // the mixed tiles: each wavefront on its own, so that it holds up no other one
    auto next_mixed = [&](int p, int tile) {
      while (tile < 2 * st_end && tile * 32 <= last[p] && kind_of(p, tile * 32) != 3) ++tile;
      return tile < 2 * st_end && tile * 32 <= last[p] ? tile : -1;
    };
    auto first_mixed = [&](int p) {
      const int open = ((t_lo[p] - R > 0 ? t_lo[p] - R : 0) + 1) >> 5;      // the first that is not discarded
      return next_mixed(p, open > 2 * st_at ? open : 2 * st_at);
    };
    auto fetch_keys = [&](int tile) {
      int row = tile * 32 + col;
      row = row < L ? row : L - 1;
      const uint16_t* kp = K + (int64_t)hk * ksh + (int64_t)(seq0 + row) * kst + hf * 64;
#pragma unroll
      for (int u = 0; u < 8; ++u) kf[u] = *reinterpret_cast<const bf16x8_t*>(kp + u * 8);
    };
    int m0 = first_mixed(0), m1 = first_mixed(1);
    if (m0 >= 0 || m1 >= 0) fetch_keys(m0 >= 0 ? m0 : m1);
    // tile m of row tile p, whose keys are in kf; the keys of the next one are requested behind its products
    auto mixed_tile = [&](int p, int& m, const int& other) {
      c0 = imp_product(kf, qf[p]);
      const int tile = m;
      m = next_mixed(p, tile + 1);
      if (m >= 0 || other >= 0) fetch_keys(other >= 0 ? other : m);
      const int key0 = tile * 32 + 4 * hf;
      imp_masked_tile(acc_st[p], c0, scale_log2, kmax[p] - key0, (tt[p] - R + 1 > 0 ? tt[p] - R + 1 : 0) - key0,
                      tt[p] - key0, (tt[p] - R > 0 ? tt[p] - R : 0) - key0);
    };
    while (m0 >= 0 || m1 >= 0) {
      if (m0 >= 0) mixed_tile(0, m0, m1);
      if (m1 >= 0) mixed_tile(1, m1, m0);
    }

    // halves of a wave hold disjoint keys of the same row
    float4* out = part + ((int64_t)piece + (int64_t)hk * n_list + item) * kImpRows;
#pragma unroll
    for (int p = 0; p < kImpNS; ++p) {
      RowStat a, o;
      a.m = acc_st[p].m;
      a.zt = acc_st[p].zt + acc_st[p].zf;
      a.zo = acc_st[p].zo;
      a.zd = acc_st[p].zd + acc_st[p].zf;
      o.m = shfl_xor_f(a.m, 32);
      o.zt = shfl_xor_f(a.zt, 32);
      o.zo = shfl_xor_f(a.zo, 32);
      o.zd = shfl_xor_f(a.zd, 32);
      stat_merge(a, o);
      if (hf == 0) out[(own_tile + p) * 32 + col] = make_float4(a.m, a.zt, a.zo, a.zd);
    }
    x += (uint64_t)(end - at);
    at = 0;
    if (++item == n_list) { item = 0; ++hk; }
  }
}

// ---- calls with few query rows ------------------------------------------------------------------
constexpr int kImpQRow = DSK_HEAD_DIM + 8;   // bf16 elements per query row in LDS: 16 rows' 16-byte reads cover all banks

// key ranges that hold keys of a sample
__device__ __forceinline__ int imp_few_ranges(int last_key, int ranges, int range_keys) {
  const int n = last_key / range_keys + 1;
  return n < ranges ? n : ranges;
}

// The packed kernel pays for its plan, and shares key tiles among kImpRows query rows of a sequence.  Where a
// sequence has far fewer rows, or few keys, one workgroup per kSamples samples of one KV head does better: its
// wavefronts take every kWaves-th key tile, straight from memory (one key row per lane), against the
// samples' operands in LDS.  What bounds it is the latency of that chain, so the keys are cut into
// ranges of `range_keys` that workgroups of their own take.  A range in which none of the samples has a key
// ends at once.  A sample that ends in the first range is finished here (imp_part), of the others the
// statistics of their rows (part) are left to the finishing kernel.
// grid: (group of kSamples samples, KV head, range x sequence): the ranges are the slowest, so that the few
// workgroups with work, the first range's, spread over all XCDs
template <int kThreads, int kSamples, bool SPLIT>
__global__ __launch_bounds__(kThreads) void importance_few_kernel(
    const uint16_t* __restrict__ K, int64_t kst, int64_t ksh, const uint16_t* __restrict__ qwin,
    const int32_t* __restrict__ samp_pos, const int32_t* __restrict__ cu_seqlens, int n_samp, int ranges,
    int range_keys, int W, int R, int Hq, int G, int Hkv, float alpha, float scale_log2, int B,
    double* __restrict__ imp_part, float4* __restrict__ part) {
  constexpr int kWaves = kThreads / DSK_WAVE;
  __shared__ RowStat sm_stat[kSamples][kWaves][32];
  __shared__ __attribute__((aligned(16))) uint16_t sm_q[kSamples][32][kImpQRow];
  const int group = blockIdx.x;
  const int hk = blockIdx.y;
  const int range = SPLIT ? blockIdx.z / B : 0, s = SPLIT ? blockIdx.z - range * B : blockIdx.z;
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = threadIdx.x / DSK_WAVE;
  const int col = lane & 31;        // query row of the tile this lane accumulates
  const int hf = lane >> 5;         // channel half / key sub-row selector

  const int seq0 = cu_seqlens[s];
  const int L = cu_seqlens[s + 1] - seq0;
  int jn[kSamples], t[kSamples], o_lo[kSamples], d_hi[kSamples], last_key[kSamples];
  int n_tiles = 0;
#pragma unroll
  for (int p = 0; p < kSamples; ++p) {
    jn[p] = group * kSamples + p;
    const int tg = jn[p] < n_samp ? samp_pos[(int64_t)s * n_samp + jn[p]] : -1;
    t[p] = tg - seq0;
    const bool have = tg >= 0 && t[p] >= 0 && t[p] < L;
    if (!have) t[p] = 0;
    o_lo[p] = t[p] - R + 1 > 0 ? t[p] - R + 1 : 0;          // retained region [o_lo, t]
    d_hi[p] = t[p] - R > 0 ? t[p] - R : 0;                  // discarded region [0, d_hi]
    last_key[p] = have ? (t[p] < L - 1 - W ? t[p] + W : L - 1) : -1;
    if (have && last_key[p] / 32 + 1 > n_tiles) n_tiles = last_key[p] / 32 + 1;
  }
  // the last range takes what is left, whatever the host expected
  const int tile0 = range * (range_keys / 32);
  if (SPLIT && range + 1 < ranges && n_tiles > tile0 + range_keys / 32) n_tiles = tile0 + range_keys / 32;
  if (tile0 >= n_tiles) return;                             // uniform over the workgroup
  const int rows = W * G;                                   // query rows of one (sample, kv head)
  const uint16_t* Kh = K + (int64_t)hk * ksh + (int64_t)seq0 * kst + hf * 64;
  // of sample threadIdx / 32: the row values are near -alpha each, so 32-bit sums would round away a bit of the mean
  double total = 0.0;

  for (int row0 = 0; row0 < rows; row0 += 32) {
    // Q^T operands of the group's samples -> LDS: row r of sample p is query row row0 + r (window
    // position w = row / G, head g = row % G), zero for rows or samples that do not exist
    for (int idx = threadIdx.x; idx < kSamples * 32 * 16; idx += kThreads) {
      const int p = idx / (32 * 16);
      const int r = (idx / 16) & 31;
      const int c16 = idx & 15;
      const int rowq = row0 + r;
      uint4 raw = make_uint4(0, 0, 0, 0);
      if (rowq < rows && last_key[p] >= 0) {
        const int wq_ = rowq / G, gq_ = rowq % G;
        raw = *reinterpret_cast<const uint4*>(
            qwin + ((((int64_t)s * n_samp + jn[p]) * W + wq_) * Hq + hk * G + gq_) * DSK_HEAD_DIM + c16 * 8);
      }
      *reinterpret_cast<uint4*>(&sm_q[p][r][c16 * 8]) = raw;
    }
    const int row = row0 + col;
    const int w = row < rows ? row / G : 0;
    int qpos[kSamples];
    RowStat st[kSamples];
#pragma unroll
    for (int p = 0; p < kSamples; ++p) {
      qpos[p] = t[p] + 1 + w;               // position of this query; attends keys 0..qpos
      st[p].m = -__builtin_inff();
      st[p].zt = st[p].zo = st[p].zd = 0.0f;
    }
    __syncthreads();
    // the rows of the wave's next tile are requested before the current tile is multiplied
    uint4 knext[8];
    auto request = [&](int tile) {
      int krow = tile * 32 + col;           // A operand row of this lane
      krow = krow < L ? krow : L - 1;       // stay inside the sequence; masked below, or past the last tile
      const uint16_t* kp = Kh + (int64_t)krow * kst;
#pragma unroll
      for (int u = 0; u < 8; ++u) knext[u] = *reinterpret_cast<const uint4*>(kp + u * 8);
    };
    request(tile0 + wave);
    for (int tile = tile0 + wave; tile < n_tiles; tile += kWaves) {
      const int k0 = tile * 32;
      uint4 kraw[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) kraw[u] = knext[u];
      request(tile + kWaves);
#pragma unroll
      for (int p = 0; p < kSamples; ++p) {
        if (k0 > last_key[p]) continue;     // this sample's keys ended before the tile (uniform)
        f32x16_t acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          // lane (col, hf) supplies channels [64*hf + 8u, +8) of query row col
          const bf16x8_t qb = *reinterpret_cast<const bf16x8_t*>(&sm_q[p][col][hf * 64 + u * 8]);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8_t*>(&kraw[u]), qb, acc, 0, 0, 0);
        }
        // acc[r] = logit of key k0 + 8*(r/4) + 4*hf + r%4 against query row `col`
        if (k0 + 31 <= d_hi[p]) {
          // the whole tile lies in the discarded region (hence before every query of the window
          // and outside the retained region): no masks, one sum feeds both totals
          float amax = acc[0];
#pragma unroll
          for (int r = 1; r < 16; ++r) amax = fmaxf(amax, acc[r]);
          const float mn = fmaxf(st[p].m, amax * scale_log2);
          const float f = __builtin_amdgcn_exp2f(st[p].m - mn);   // 0 while st.m is still -inf
          const float esum = imp_tile_sum(acc, scale_log2, mn);
          st[p].zt = fmaf(st[p].zt, f, esum);
          st[p].zd = fmaf(st[p].zd, f, esum);
          st[p].zo *= f;
          st[p].m = mn;
          continue;
        }
        float z[16];
        float tmax = -__builtin_inff();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int kpos = k0 + 8 * (r / 4) + 4 * hf + (r % 4);
          z[r] = (kpos <= qpos[p] && kpos <= last_key[p]) ? acc[r] * scale_log2 : -__builtin_inff();
          tmax = fmaxf(tmax, z[r]);
        }
        if (tmax != -__builtin_inff()) {
          const float mn = fmaxf(st[p].m, tmax);
          const float f = st[p].m == -__builtin_inff() ? 0.0f : exp2f(st[p].m - mn);
          st[p].zt *= f; st[p].zo *= f; st[p].zd *= f;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int kpos = k0 + 8 * (r / 4) + 4 * hf + (r % 4);
            const float e = __builtin_amdgcn_exp2f(z[r] - mn);   // z <= mn; 0 for masked keys (-inf)
            st[p].zt += e;
            st[p].zo += (kpos >= o_lo[p] && kpos <= t[p]) ? e : 0.0f;
            st[p].zd += (kpos <= d_hi[p]) ? e : 0.0f;
          }
          st[p].m = mn;
        }
      }
    }
    // halves of a wave hold disjoint keys of the same row; then waves; fixed order
#pragma unroll
    for (int p = 0; p < kSamples; ++p) {
      RowStat other;
      other.m = shfl_xor_f(st[p].m, 32);
      other.zt = shfl_xor_f(st[p].zt, 32);
      other.zo = shfl_xor_f(st[p].zo, 32);
      other.zd = shfl_xor_f(st[p].zd, 32);
      if (hf == 0) {
        stat_merge(st[p], other);
        sm_stat[p][wave][col] = st[p];
      }
    }
    __syncthreads();
    if (threadIdx.x < 32 * kSamples) {
      const int p = threadIdx.x >> 5;
      RowStat a = sm_stat[p][0][col];
#pragma unroll
      for (int wv = 1; wv < kWaves; ++wv) stat_merge(a, sm_stat[p][wv][col]);
      double v = row0 + col < rows && a.zt > 0.0f ? (a.zo - alpha * a.zd) / a.zt : 0.0f;
#pragma unroll
      for (int m = 1; m < 32; m <<= 1) v += __shfl_xor(v, m, DSK_WAVE);   // the sample's 32 rows, in a fixed order
      total += v;
      if constexpr (SPLIT) {
        int j = 0, last = -1;
#pragma unroll
        for (int i = 0; i < kSamples; ++i)
          if (i == p) { j = jn[i]; last = last_key[i]; }
        if (row0 + col < rows && last >= tile0 * 32 && imp_few_ranges(last, ranges, range_keys) > 1)
          part[((((int64_t)s * n_samp + j) * Hkv + hk) * rows + row0 + col) * ranges + range] =
              make_float4(a.m, a.zt, a.zo, a.zd);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 32 * kSamples && col == 0) {
    int j = 0, last = -1;
#pragma unroll
    for (int i = 0; i < kSamples; ++i)
      if (i == (int)threadIdx.x >> 5) { j = jn[i]; last = last_key[i]; }
    if (last >= 0 && (!SPLIT || (range == 0 && imp_few_ranges(last, ranges, range_keys) == 1)))
      imp_part[((int64_t)s * n_samp + j) * Hkv + hk] = total;
  }
}

// what the finishing kernels end with, on the sum of a sample's rows (thread m < M <= 64: the class's m-th
// sample, have: its position is not -1): sample scores, class mean, class weight; sums in sample order.  The first
// wavefront alone: with the scores in LDS, a barrier and one thread that adds them this took 2400 cycles instead of 1600.
__device__ __forceinline__ void imp_class_weight(double sum_rows, bool have, int c, int s, int n_class, int M, int n_rows,
                                                 float alpha, uint8_t* class_weight_q, float* class_mean,
                                                 float* samp_score, float* samp_score_sum, int layers) {
  static_assert(kMaxSamplesPerClass <= DSK_WAVE, "a lane per sample");
  if (threadIdx.x >= DSK_WAVE) return;
  float st = 0.0f;
  if ((int)threadIdx.x < M) {
    const int64_t js = ((int64_t)s * n_class + c) * M + threadIdx.x;
    st = (float)(sum_rows / n_rows);
    if (samp_score) samp_score[js] = have ? st : __builtin_nanf("");
    if (samp_score_sum != nullptr && have) {      // expectation over layers: this layer joins the running sum
      const float tot = samp_score_sum[js] + st;
      samp_score_sum[js] = tot;
      st = tot / (float)layers;
    }
  }
  unsigned long long left = __ballot((int)threadIdx.x < M && have);
  const int cnt = __popcll(left);
  float sum = 0.0f;
  for (; left != 0; left &= left - 1) sum += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st), __builtin_ctzll(left)));
  if (threadIdx.x != 0) return;
  const int64_t cs = (int64_t)s * n_class + c;
  if (cnt > 0) {
    const float mean = sum / (float)cnt;
    float w = (mean + alpha) / (1.0f + alpha);
    w = fminf(1.0f, fmaxf(0.0f, w));
    class_weight_q[cs] = (uint8_t)floorf(10.0f * w + 0.5f);
    if (class_mean) class_mean[cs] = mean;
  } else if (class_mean) {
    class_mean[cs] = __builtin_nanf("");
  }
}

// grid: (class, sequence), one lane per sample (M <= 64): the samples that importance_few_kernel finished
__global__ __launch_bounds__(DSK_WAVE) void importance_few_finalize_kernel(
    const double* __restrict__ imp_part, const int32_t* __restrict__ samp_pos, const int32_t* __restrict__ cu_seqlens,
    int n_class, int M, int Hkv, int G, int W, float alpha, uint8_t* __restrict__ class_weight_q,
    float* __restrict__ class_mean, float* __restrict__ samp_score, float* __restrict__ samp_score_sum, int layers) {
  const int c = blockIdx.x, s = blockIdx.y, m = threadIdx.x;
  const int seq0 = cu_seqlens[s], end = cu_seqlens[s + 1];
  double st = 0.0;
  bool have = false;
  if (m < M) {
    const int64_t js = ((int64_t)s * n_class + c) * M + m;
    const int tg = samp_pos[js];
    have = tg >= 0;
    if (have && tg >= seq0 && tg < end)           // a position outside the sequence counts with 0
      for (int hk = 0; hk < Hkv; ++hk) st += imp_part[js * Hkv + hk];
  }
  imp_class_weight(st, have, c, s, n_class, M, G * Hkv * W, alpha, class_weight_q, class_mean, samp_score,
                   samp_score_sum, layers);
}

constexpr int kImpFinThreads = 1024;
constexpr int kImpFinWaves = kImpFinThreads / DSK_WAVE;
constexpr int kImpFinRows = 2;       // rows of a lane in flight together
// The rows idx, idx + stride .. of a sample's n_rows: their pieces' statistics merged, the row values summed.
// locate(row, n): the first of the row's n pieces, `pitch` entries apart.
// What bounds it is how fast one CU takes them in, so no more pieces are requested than some row of the wavefront has, to
// the next even number: with 8 at a time whatever there is, this was 9100 of the finishing kernel's 15500 cycles (128
// samples of 128K tokens, 5 pieces a row), now 8100 of 13600; 8600 of 14700 and 6500 of 11500 (eight sequences, 2 pieces).
template <typename Locate>
__device__ __forceinline__ float imp_rows_sum(Locate locate, int pitch, int idx, int stride, int n_rows, float alpha) {
  float sum = 0.0f;
  while (__any(idx < n_rows)) {
    const float4* rows[kImpFinRows];
    int n[kImpFinRows];
    int most = 0;
    RowStat a[kImpFinRows];
#pragma unroll
    for (int i = 0; i < kImpFinRows; ++i) {
      const bool own = idx + i * stride < n_rows;
      rows[i] = locate(own ? idx + i * stride : 0, n[i]);
      n[i] = own ? n[i] : 0;
      most = n[i] > most ? n[i] : most;
      a[i] = {-__builtin_inff(), 0.0f, 0.0f, 0.0f};
    }
    most = (int)wave_max_u((uint32_t)most);
    auto merge = [&](auto batch, int w) {                // pieces w .. of each row
      constexpr int kBatch = decltype(batch)::value;
      float4 v[kImpFinRows][kBatch];
#pragma unroll
      for (int i = 0; i < kImpFinRows; ++i)
#pragma unroll
        for (int j = 0; j < kBatch; ++j) v[i][j] = rows[i][(int64_t)(w + j < n[i] ? w + j : 0) * pitch];
#pragma unroll
      for (int i = 0; i < kImpFinRows; ++i)
#pragma unroll
        for (int j = 0; j < kBatch; ++j) pin_loaded(v[i][j]);
#pragma unroll
      for (int i = 0; i < kImpFinRows; ++i) {
        float m = a[i].m;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) m = fmaxf(m, w + j < n[i] ? v[i][j].x : -__builtin_inff());
        const float ref = m == -__builtin_inff() ? 0.0f : m;     // no key anywhere yet: all factors 0
        const float f = __builtin_amdgcn_exp2f(a[i].m - ref);
        a[i] = {m, a[i].zt * f, a[i].zo * f, a[i].zd * f};
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
          const float g = w + j < n[i] ? __builtin_amdgcn_exp2f(v[i][j].x - ref) : 0.0f;
          a[i].zt = fmaf(v[i][j].y, g, a[i].zt);
          a[i].zo = fmaf(v[i][j].z, g, a[i].zo);
          a[i].zd = fmaf(v[i][j].w, g, a[i].zd);
        }
      }
    };
    int w = 0;
    for (; most - w > 6; w += 8) merge(std::integral_constant<int, 8>{}, w);
    if (most - w > 4) merge(std::integral_constant<int, 6>{}, w);
    else if (most - w > 2) merge(std::integral_constant<int, 4>{}, w);
    else if (most > w) merge(std::integral_constant<int, 2>{}, w);
#pragma unroll
    for (int i = 0; i < kImpFinRows; ++i) sum += a[i].zt > 0.0f ? (a[i].zo - alpha * a[i].zd) / a[i].zt : 0.0f;
    idx += kImpFinRows * stride;
  }
  return sum;
}

// grid: (class, sequence).  The wavefronts are dealt to the class's samples; their lanes merge the pieces
// of the sample's rows over all KV heads and sum the row values, the first wavefront then adds the sample
// scores in sample order (every sum in a fixed order).
constexpr int kImpFinItems = 1024;   // items whose places on the line are fetched ahead
__global__ __launch_bounds__(kImpFinThreads) void importance_finalize_kernel(
    int32_t* __restrict__ plan, const float4* __restrict__ part, const int32_t* __restrict__ samp_pos,
    int seq_first, int nseq, int items, int n_class, int M, int Hkv, int G, int W, float alpha,
    uint8_t* __restrict__ class_weight_q, float* __restrict__ class_mean, float* __restrict__ samp_score,
    float* __restrict__ samp_score_sum, int layers) {
  __shared__ float sm_sum[kMaxSamplesPerClass * kImpFinWaves];
  __shared__ int sm_item[kImpFinItems];
  const int c = blockIdx.x;
  const int sl = blockIdx.y, s = seq_first + sl;
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DSK_WAVE);
  const int n_samp = n_class * M;
  const int rps = W * G;
  const ImpPlan pl = imp_plan(plan, nseq, n_samp, items);
  const int T1 = pl.head[0], n_list = pl.head[2];
  const uint32_t nw = (uint32_t)pl.head[1];
  const int ib = pl.item_base[sl];
  const int32_t* rank = pl.rank + (int64_t)sl * n_samp;
  // everything that does not depend on the plan's values goes out in one round trip
  if (threadIdx.x <= items && threadIdx.x < kImpFinItems) sm_item[threadIdx.x] = pl.item_at[threadIdx.x];
  const bool have = (int)threadIdx.x < M && samp_pos[(int64_t)s * n_samp + c * M + threadIdx.x] >= 0;
  const int per_sample = M < kImpFinWaves ? kImpFinWaves / M : 1;   // wavefronts of one sample
  const int m_first = wave / per_sample;
  const int rk_first = m_first < M ? rank[c * M + m_first] : -1;
  static_assert(kImpFinItems <= kImpFinThreads, "one load each");
  auto item_at = [&](int i) { return (uint32_t)(i < kImpFinItems ? sm_item[i] : pl.item_at[i]); };
  ImpLine line;
  line.per = line.extra = 0;
  if (nw > 0) {
    const uint64_t T = (uint64_t)T1 * Hkv;
    line.per = (uint32_t)(T / nw);
    line.extra = (uint32_t)(T % nw);
  }
  __syncthreads();
  for (int m = m_first; m < M; m += kImpFinWaves / per_sample) {
    const int rk = m == m_first ? rk_first : rank[c * M + m];
    float sum = 0.0f;
    if (rk >= 0 && nw > 0) {
      sum = imp_rows_sum(
          [&](int x, int& n) {
            const int hk = x / rps;
            const int rho = rk * rps + (x - hk * rps);
            const int item = ib + rho / kImpRows;
            const uint64_t x0 = (uint64_t)hk * T1 + item_at(item), x1 = (uint64_t)hk * T1 + item_at(item + 1);
            const uint32_t w0 = line.piece_of(x0);
            n = (int)(line.piece_of(x1 - 1) - w0) + 1;
            return part + ((int64_t)w0 + (int64_t)hk * n_list + item) * kImpRows + rho % kImpRows;
          },
          kImpRows, (wave % per_sample) * DSK_WAVE + lane, per_sample * DSK_WAVE, rps * Hkv, alpha);
    }
    sum = wave_sum(sum);
    if (lane == 0) sm_sum[m * kImpFinWaves + wave % per_sample] = sum;
  }
  __syncthreads();
  float st = 0.0f;
  if ((int)threadIdx.x < M)
    for (int i = 0; i < per_sample; ++i) st += sm_sum[threadIdx.x * kImpFinWaves + i];
  imp_class_weight(st, have, c, s, n_class, M, G * Hkv * W, alpha, class_weight_q, class_mean, samp_score, samp_score_sum,
                   layers);
}

// grid: (class, sequence): the same behind importance_few_kernel with several key ranges
constexpr int kImpFewWaves = 4;
__global__ __launch_bounds__(kImpFewWaves * DSK_WAVE) void importance_few_merge_kernel(
    const double* __restrict__ imp_part, const float4* __restrict__ part, const int32_t* __restrict__ samp_pos,
    const int32_t* __restrict__ cu_seqlens, int ranges, int range_keys, int n_class, int M, int Hkv, int G, int W,
    float alpha, uint8_t* __restrict__ class_weight_q, float* __restrict__ class_mean, float* __restrict__ samp_score,
    float* __restrict__ samp_score_sum, int layers) {
  __shared__ double sm_sum[kMaxSamplesPerClass * kImpFewWaves];
  const int c = blockIdx.x, s = blockIdx.y;
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DSK_WAVE);
  const int n_rows = W * G * Hkv;
  const int seq0 = cu_seqlens[s], L = cu_seqlens[s + 1] - seq0;
  const int64_t js = ((int64_t)s * n_class + c) * M;
  const bool have = (int)threadIdx.x < M && samp_pos[js + threadIdx.x] >= 0;
  const int per_sample = M < kImpFewWaves ? kImpFewWaves / M : 1;   // wavefronts of one sample
  for (int m = wave / per_sample; m < M; m += kImpFewWaves / per_sample) {
    const int tg = samp_pos[js + m], t = tg - seq0, part_of = wave % per_sample;
    double sum = 0.0;
    if (tg >= 0 && t >= 0 && t < L) {             // a position outside the sequence counts with 0
      const int n_ranges = imp_few_ranges(t < L - 1 - W ? t + W : L - 1, ranges, range_keys);
      if (n_ranges == 1) {
        for (int hk = part_of * DSK_WAVE + lane; hk < Hkv; hk += per_sample * DSK_WAVE) sum += imp_part[(js + m) * Hkv + hk];
      } else {
        sum = imp_rows_sum(
            [&](int x, int& n) {
              n = n_ranges;
              return part + ((js + m) * n_rows + x) * ranges;
            },
            1, part_of * DSK_WAVE + lane, per_sample * DSK_WAVE, n_rows, alpha);
      }
    }
#pragma unroll
    for (int i = 1; i < DSK_WAVE; i <<= 1) sum += __shfl_xor(sum, i, DSK_WAVE);
    if (lane == 0) sm_sum[m * kImpFewWaves + part_of] = sum;
  }
  __syncthreads();
  double st = 0.0;
  if ((int)threadIdx.x < M)
    for (int i = 0; i < per_sample; ++i) st += sm_sum[threadIdx.x * kImpFewWaves + i];
  imp_class_weight(st, have, c, s, n_class, M, G * Hkv * W, alpha, class_weight_q, class_mean, samp_score, samp_score_sum,
                   layers);
}

ImpLayout importance_layout(int B, int n_samp, int W, int Hq, int Hkv) {
  ImpLayout l;
  const int64_t rps = (int64_t)W * (Hq / Hkv);
  const int64_t per_seq = ((int64_t)n_samp * rps + kImpRows - 1) / kImpRows;
  int64_t seqs = kImpMaxItems / (per_seq * Hkv > 0 ? per_seq * Hkv : 1);    // bounds the workspace
  if (seqs < 1) seqs = 1;
  if (seqs > kImpMaxSeqs) seqs = kImpMaxSeqs;
  if (seqs > B) seqs = B;
  l.seqs = (int)seqs;
  l.items = (int)(seqs * per_seq);
  // sequences and items of a launch at most, for these arguments and for smaller ones (fewer rows per sequence can
  // mean more sequences in a launch, and more items)
  const int64_t most_seqs = B < kImpMaxSeqs ? B : kImpMaxSeqs;
  int64_t most_items = kImpMaxItems / Hkv > per_seq ? kImpMaxItems / Hkv : per_seq;
  if (most_items > most_seqs * per_seq) most_items = most_seqs * per_seq;
  l.plan_ints = (size_t)(4 + 2 * most_seqs + 1 + most_items + 1 + 3 * most_seqs * n_samp);
  l.part_rows = (size_t)(kImpPieces + most_items * Hkv) * kImpRows;
  // calls with few rows: a sum of 8 bytes for each (sample, KV head) of all sequences
  l.sum_rows = ((size_t)B * n_samp * Hkv + 1) / 2;
  if (l.part_rows < l.sum_rows) l.part_rows = l.sum_rows;
  return l;
}

// The kernel for few rows: whether the call takes it, and its key ranges.
struct ImpFew {
  bool take;
  int ranges, keys;
};
static ImpFew importance_few(const dsk_compress_args& a, const ImpLayout& l) {
  ImpFew f;
  const int64_t n_samp = (int64_t)a.n_class * a.M;
  const int64_t rps = (int64_t)a.W * (a.Hq / a.Hkv), row_tiles = (rps + 31) / 32;
  const int64_t wgs = (n_samp + 3) / 4 * a.Hkv * a.B;
  // The rule bounds the work of this kernel, in products of four samples' row tiles with a key tile, and the chain of
  // samples with several row tiles.  It counts with the keys that the samples of stage CANDIDATES reach, the first
  // M occurrences of every class (delimiters are some tens of tokens apart), not with the sequence's length: on
  // positions further back this kernel is up to three times slower than the packed one, which is up to 2.9 times
  // slower than this one on early positions or short sequences.  Several sequences cost the packed kernel a
  // ranking launch and time for its plan, and items of a few rows leave most of its wavefronts idle.
  // Measured at its sides, packed against this kernel: 128 samples of 300 tokens, 32 / 8 heads 30.4 against 17.3 us;
  // 4 samples in each of 512 sequences of 300 tokens, 1 / 1 head 75 against 28, in each of 8 of 8K tokens, 32 / 32
  // heads 224 against 92; 16 samples of 128K tokens, 32 / 8 heads 24.3 against 19.2 where they lie early, 127 against
  // 183 spread over all of it (864 with one range); 128 samples spread over 8K tokens 67.6 against 77.7 (packed).
  const bool own_rank = a.B == 1 && n_samp <= kImpThreads;
  int64_t keys = (int64_t)a.R + a.W + 48 * n_samp;
  if (keys > a.max_seqlen) keys = a.max_seqlen;
  const int64_t work = wgs * row_tiles * ((keys + 31) / 32);
  f.take = (work <= (own_rank ? 16384 : 26000 + 300 * (int64_t)a.B) && (row_tiles == 1 || row_tiles * keys <= 1024)) ||
           (row_tiles == 1 && n_samp <= 8 && n_samp * rps <= 64);
  // Key ranges only where the samples alone occupy at most half of the CUs (a sequence of 128K tokens, 4 samples
  // spread over it, 8 / 8 heads: 859 us in one range, 56 in 32; 40 samples in each of 3 sequences of 5.3K, 240
  // workgroups: 53 against 62 in 2), and as far as their statistics have room.
  const int64_t rows = a.B * n_samp * rps * a.Hkv;
  int64_t ranges = ((int64_t)a.max_seqlen + kImpFewKeys - 1) / kImpFewKeys;
  if (ranges > kImpFewRanges) ranges = kImpFewRanges;
  if (wgs > 128) ranges = 1;
  else if (ranges * wgs > 1024) ranges = 1024 / wgs;
  const int64_t room = (int64_t)(l.part_rows - l.sum_rows);
  if (ranges > 1 && ranges * rows > room) ranges = room / rows;
  if (ranges < 1) ranges = 1;
  f.ranges = (int)ranges;
  f.keys = (int)((((int64_t)a.max_seqlen + ranges - 1) / ranges + 31) / 32 * 32);
  return f;
}

hipError_t launch_importance(const dsk_compress_args& a, const CompressWs& ws, hipStream_t st) {
  unsigned char* w = static_cast<unsigned char*>(a.workspace);
  int32_t* plan = reinterpret_cast<int32_t*>(w + ws.imp_plan);
  float4* part = reinterpret_cast<float4*>(w + ws.imp_part);
  const int n_samp = a.n_class * a.M;
  const int G = a.Hq / a.Hkv;
  const float scale = a.imp_scale != 0.0f ? a.imp_scale : 0.08838834764831845f;   // 128^-1/2
  const ImpLayout l = importance_layout(a.B, n_samp, a.W, a.Hq, a.Hkv);
  const int layers = a.imp_layers > 0 ? a.imp_layers : 1;
  const ImpFew few = importance_few(a, l);
  if (few.take) {
    double* sums = reinterpret_cast<double*>(part);   // of each (sample, KV head), in front of the statistics
    float4* stats = part + l.sum_rows;
#define DSK_IMP_ARGS                                                                                             \
  static_cast<const uint16_t*>(a.K), a.k_stride_tok, a.k_stride_head, static_cast<const uint16_t*>(a.qwin),      \
      a.samp_pos, a.cu_seqlens, n_samp, few.ranges, few.keys, a.W, a.R, a.Hq, G, a.Hkv, a.alpha_imp,         \
      scale * kImpLog2e, a.B, sums, stats
#define DSK_IMP_FEW(threads, samples)                                                                             \
  do {                                                                                                           \
    const dim3 grid((unsigned)((n_samp + samples - 1) / samples), (unsigned)a.Hkv, (unsigned)(a.B * few.ranges)); \
    if (few.ranges > 1) importance_few_kernel<threads, samples, true><<<grid, dim3(threads), 0, st>>>(DSK_IMP_ARGS); \
    else importance_few_kernel<threads, samples, false><<<grid, dim3(threads), 0, st>>>(DSK_IMP_ARGS);           \
  } while (0)
    // 4 samples and 8 wavefronts per workgroup where these are few, 3 and 4 where there are many
    if ((int64_t)((n_samp + 3) / 4) * a.Hkv * a.B < 1024) DSK_IMP_FEW(512, 4);
    else DSK_IMP_FEW(256, 3);
#undef DSK_IMP_FEW
#undef DSK_IMP_ARGS
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    const dim3 grid((unsigned)a.n_class, (unsigned)a.B);
    if (few.ranges == 1)
      importance_few_finalize_kernel<<<grid, dim3(DSK_WAVE), 0, st>>>(
          sums, a.samp_pos, a.cu_seqlens, a.n_class, a.M, a.Hkv, G, a.W, a.alpha_imp, a.class_weight_q, a.class_mean,
          a.samp_score, a.samp_score_sum, layers);
    else
      importance_few_merge_kernel<<<grid, dim3(kImpFewWaves * DSK_WAVE), 0, st>>>(
          sums, stats, a.samp_pos, a.cu_seqlens, few.ranges, few.keys, a.n_class, a.M, a.Hkv, G, a.W, a.alpha_imp,
          a.class_weight_q, a.class_mean, a.samp_score, a.samp_score_sum, layers);
    return hipGetLastError();
  }
  for (int s = 0; s < a.B; s += l.seqs) {
    const int nseq = a.B - s < l.seqs ? a.B - s : l.seqs;
    hipError_t err;
#define DSK_IMP_ARGS                                                                                              \
  static_cast<const uint16_t*>(a.K), a.k_stride_tok, a.k_stride_head, static_cast<const uint16_t*>(a.qwin),       \
      a.samp_pos, a.cu_seqlens, s, nseq, n_samp, l.items, a.W, a.R, a.Hq, G, a.Hkv, scale * kImpLog2e, plan, part
    if (nseq == 1 && n_samp <= kImpThreads) {
      importance_kernel<true><<<dim3(kImpPieces), dim3(kImpThreads), 0, st>>>(DSK_IMP_ARGS);
    } else {
      importance_rank_kernel<<<dim3((unsigned)((n_samp + DSK_WAVE - 1) / DSK_WAVE), (unsigned)nseq), dim3(kImpThreads), 0,
                               st>>>(a.samp_pos, a.cu_seqlens, s, nseq, n_samp, l.items, plan);
      err = hipGetLastError();
      if (err != hipSuccess) return err;
      importance_kernel<false><<<dim3(kImpPieces), dim3(kImpThreads), 0, st>>>(DSK_IMP_ARGS);
    }
#undef DSK_IMP_ARGS
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    importance_finalize_kernel<<<dim3((unsigned)a.n_class, (unsigned)nseq), dim3(kImpFinThreads), 0, st>>>(
        plan, part, a.samp_pos, s, nseq, l.items, a.n_class, a.M, a.Hkv, G, a.W, a.alpha_imp, a.class_weight_q,
        a.class_mean, a.samp_score, a.samp_score_sum, layers);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

}  // namespace dsk
