// Sparse decode attention over the K/V rows of the selected slots (App. B.2 Steps 2-3):
// a split-K flash-decode.  The gather is HBM-bound (512 B of K+V per token, ~2 flop/B), so
// there is no MFMA in the kernels per head: a 256-byte bf16 row is spread over 16 lanes x 16 B and a wavefront
// reads 4 token rows per load instruction.  A wavefront owns SPW slots of at most 4*NS rows; it
// issues every K and V load of a slot (16 x 16 B per lane, 16 KB per wavefront for 32 rows)
// before it touches the data, then folds the slot into an online-softmax state (m, l, acc).
// The wavefronts of a workgroup (8 for slots of up to 32 rows, 2 slots each) merge through LDS
// into one partial per (sequence, head, chunk of 16 slots); a second small kernel merges the
// partials of a head in a fixed order; attn_long_kernel and attn_shared_kernel below take long lists and lists that a
// KV group shares.  (Merging inside this kernel -- the workgroup of a head that
// finishes last, found with an arrival counter, folds the head's partials -- was built three ways:
// write-through partials with a device-scope counter, ordinary stores with a device-scope counter,
// ordinary stores with a counter that stays in the XCD's L2.  At 128K / 32 heads the attention call
// took 9.8 / 9.6 / 9.3 us against 9.3 us with the merge launch, whose cost in a graph is that of an
// empty kernel, about 1.5 us: the store-acknowledge, counter and reload round trips of the last
// workgroup cost as much.  Not kept.)
// The launch is a 1-D grid in which workgroup id = 8 * j + x runs on XCD x: all chunks of all
// query heads of a (sequence, KV head) group are given the same x, so that rows selected by
// several heads of the group are fetched into one L2 once (9.3 instead of 10.5 us for the call at
// 128K / 32 heads against a grid that spread a head's chunks over the XCDs; see attn_place).
#include "dsk_attn_fold.hpp"
#include "dsk_common.hpp"
#include "dsk_internal.hpp"

namespace dsk {

constexpr int kMergeBigThreads = 1024;

// slots per workgroup for a slot length bound b
__host__ __device__ constexpr int attn_slots_per_wg(int b) { return b <= 32 ? 16 : 8; }
// Launches of many workgroups (a batch) run better on workgroups of 4 wavefronts x 2 slots: the last
// round of workgroups on the CUs is finer (8 ragged sequences, b = 16: gather 28.2 -> 26.0 us, step
// 48.6 -> 47.0 us), while small launches lose to the doubled number of partials (one sequence of
// 32K or 128K tokens: step +0.2 us), so the shape follows the workgroup count.
constexpr int64_t kAttnSmallWgFrom = 1536;   // workgroups of 16 slots from which 8-slot workgroups are launched

// Shared selection: attn_shared_kernel reads every selected row once, where attn_kernel run per query head reads it once
// per head with all but the first read served by L2, which is as fast while the launch is small (step of 32 / 8 heads at
// 30K tokens, 128 slots of 16 rows, per head / shared: one sequence 16.2 / 19.3 us, two 20.4 / 21.0, three 24.5 / 22.4).
constexpr int64_t kSharedMinSlots = 3072;      // selected slots of all lists
static bool attn_shared(const dsk_attn_args& a) {
  return (a.flags & DSK_ATTN_SHARED_SELECTION) && a.Hq > a.Hkv && a.b <= 32 && (int64_t)a.B * a.Hkv * a.k >= kSharedMinSlots;
}
// heads of a group that a workgroup takes together
static int attn_shared_tile(int G) { return G <= 2 ? 2 : G <= 4 ? 4 : 8; }

// The place of a workgroup of the per-head kernels.  Workgroup id = 8 * j + x runs on XCD x.  The chunks of all heads of a
// KV group go to one XCD; where the groups are no multiple of 8, each is cut into 2^cut runs of `run` chunks, which go to
// XCDs of their own, so that all eight have about the same work (28 / 4 heads, one sequence: four groups used half of the
// chip).  Of the cuts the one with the least work on the busiest XCD, the coarsest of them: cutting until the runs are a
// multiple of 8 puts more on one where the runs are few (9 / 1 heads, six sequences, 3 chunks: 27 workgroups as they are,
// 36 in runs of 2 and 1: 10.1 against 11.9 us).
// Without grouped heads there is nothing to share: the chunks are dealt out over the XCDs in plain order (measured 2 %
// faster at 40 heads than keeping a head on one XCD).
// The index arithmetic is in front of every load, so it takes no more than three divisions (the cut is a shift): with five,
// a step of 17.4 us took 0.1 us longer.
struct AttnPlace {
  int Hkv, cut, run;
};
struct AttnAt {
  int s, hk, h, chunk;   // chunk < 0: nothing to do
};
__device__ __forceinline__ AttnAt attn_place(AttnPlace p, int Hq, int G, int n_groups, int nchunks) {
  AttnAt at;
  if (G == 1) {
    const int sh = blockIdx.x / nchunks;
    at.chunk = blockIdx.x - sh * nchunks;
    at.s = sh / Hq;
    at.h = at.hk = sh - at.s * Hq;
    return at;
  }
  const unsigned per = G * p.run;
  const unsigned j = blockIdx.x >> 3;
  const unsigned vl = j / per;
  const unsigned r = j - vl * per;
  const unsigned v = vl * 8 + (blockIdx.x & 7);      // (group, run)
  const unsigned gi = v >> p.cut;
  const unsigned gq = r / (unsigned)p.run;
  at.chunk = (int)((v - (gi << p.cut)) * p.run + r - gq * p.run);
  if ((int)gi >= n_groups || at.chunk >= nchunks) at.chunk = -1;   // padding of the last round of groups, or of the last run
  at.s = gi / (unsigned)p.Hkv;
  at.hk = gi - at.s * p.Hkv;
  at.h = at.hk * G + gq;
  return at;
}
static AttnPlace attn_placement(int G, int n_groups, int Hkv, int nchunks) {
  AttnPlace best = {Hkv, 0, nchunks};
  if (G == 1) return best;
  int64_t least = (int64_t)(n_groups + 7) / 8 * nchunks;
  for (int cut = 1; cut <= 3 && (1 << cut) <= nchunks; ++cut) {
    const int run = (nchunks + (1 << cut) - 1) >> cut;
    const int64_t most = (((int64_t)n_groups << cut) + 7) / 8 * run;
    if (most < least) { least = most; best.cut = cut; best.run = run; }
  }
  return best;
}
// workgroups on every XCD
static int64_t attn_wgs_per_xcd(int G, int n_groups, int nchunks) {
  const AttnPlace p = attn_placement(G, n_groups, 1, nchunks);
  if (G == 1) return ((int64_t)n_groups * nchunks + 7) / 8;
  return (((int64_t)n_groups << p.cut) + 7) / 8 * G * p.run;
}

// up to 4*NS rows of a slot of more than 32, the loads placed by the compiler
template <int NS>
__device__ __forceinline__ void fold_rows(WaveState& st, const QRow& qf, const uint16_t* __restrict__ kbase,
                                          const uint16_t* __restrict__ vbase, int64_t kst, int64_t vst,
                                          int nvalid, int g, float scale_log2) {
  uint4 kv[NS], vv[NS];
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    int r = 4 * u + g;
    r = r < nvalid ? r : nvalid - 1;
    kv[u] = *reinterpret_cast<const uint4*>(kbase + (int64_t)r * kst);
  }
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    int r = 4 * u + g;
    r = r < nvalid ? r : nvalid - 1;
    vv[u] = *reinterpret_cast<const uint4*>(vbase + (int64_t)r * vst);
  }
  fold_loaded<NS, true>(st, qf, kv, vv, nvalid, g, scale_log2);
}

// compile-time loop over the slots of a wave: wait for slot S's K and V, fold, recurse
template <int NS, int SPW, int S>
struct FoldSlots {
  static __device__ __forceinline__ void run(WaveState& st, const QRow& qf, uint4 (&kd)[SPW][NS],
                                             uint4 (&vd)[SPW][NS], const int (&nv)[SPW], int g,
                                             float scale_log2) {
    // loads were issued slot by slot, K rows then V rows; pinning slot S here keeps the loads of
    // the later slots in flight while this one is folded
#pragma unroll
    for (int u = 0; u < NS; ++u) pin_loaded(kd[S][u]);
#pragma unroll
    for (int u = 0; u < NS; ++u) pin_loaded(vd[S][u]);
    if (nv[S] > 0) fold_loaded<NS>(st, qf, kd[S], vd[S], nv[S], g, scale_log2);
    if constexpr (S + 1 < SPW) FoldSlots<NS, SPW, S + 1>::run(st, qf, kd, vd, nv, g, scale_log2);
  }
};

// One workgroup of WAVES wavefronts per (chunk of WAVES*SPW slots, head, sequence); writes one partial, or the
// final result when the head has a single chunk (its partial as well for a caller that merges by itself: `leave`).
// REST: slots of more than 32 rows: the first 32 of every slot of the wavefront, then those behind, 32 at a time (STAGED: slot by
// slot); half of the loads where there are no more than 16: chunks are seldom as long as such a slot.  The compiler places the
// loads: with all 32 rows requested before the first one is waited for launches of 385 workgroups and more took 2 to 4 % longer.
// A wavefront per slot where a CU has no more than one workgroup, so that the latency of its loads counts, and for lists per head
// of slots of kAttnOneSlotFrom rows and more, which keep a wavefront busy for several round trips.  Otherwise the other workgroups
// hide it, and half as many wavefronts with two slots each leave room for more of them.  Attention alone, slots of 40 to 64 rows,
// 170 random calls, time in units of two slots a wavefront, slot by slot, with each weight added to the state by itself, mean and
// largest: a wavefront per slot / two slots a wavefront up to 256 workgroups 0.91 1.00 / 0.94 0.99, 257 to 512 0.97 1.04 / 0.96
// 1.03, 513 to 1024 1.03 1.10 / 0.99 1.06, 1025 to 2048 1.03 1.13 / 0.95 1.04, more 1.09 1.14 / 0.93 1.00.  Decode steps of slots of
// 128 to 256 rows, chunks as long, 800 to 2048 workgroups: 82.5 / 86.7 us, 60.5 / 65.0, 62.4 / 76.7, 52.6 / 56.2; with chunks of 20
// to 40 tokens, or shared lists (35.2 / 31.2), the other way round.  Without grouped heads, where nothing comes from L2, slot by
// slot: 512 workgroups 28.6 / 29.2, 27.0 / 27.7 and 28.4 / 29.1 us against the first rows of both slots first; with grouped heads
// 1 to 2 % slower, or 9 % where most slots have rows behind the 32.
constexpr int kAttnWavePerSlotTo = 256;
constexpr int kAttnOneSlotFrom = 128;
template <int NS, int SPW, int WAVES, bool STAGED = false, bool REST = false>
__global__ __launch_bounds__(WAVES * DSK_WAVE) void attn_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    int64_t kst, int64_t ksh, int64_t vst, int64_t vsh, int Hq, int G, int n_groups, int k, int b, int total_tokens,
    const int32_t* __restrict__ sel_start, const int32_t* __restrict__ sel_len,
    const int32_t* __restrict__ sel_count, int sel_div, float scale_log2, AttnPlace place, int nchunks, bool leave,
    float2* __restrict__ part_ml, float* __restrict__ part_acc, float* __restrict__ out,
    uint16_t* __restrict__ out_bf16, float* __restrict__ lse) {
  constexpr int kAttnWaves = WAVES;
  __shared__ float sm_m[kAttnWaves];
  __shared__ float sm_l[kAttnWaves];
  __shared__ float sm_acc[kAttnWaves][DSK_HEAD_DIM];
  constexpr int kSlotsPerWg = kAttnWaves * SPW;

  const AttnAt at = attn_place(place, Hq, G, n_groups, nchunks);
  if (at.chunk < 0) return;
  const int s = at.s, hk = at.hk, h = at.h, chunk = at.chunk;
  const int64_t sh = (int64_t)s * Hq + h;
  // row of the selection arrays: the head's own, or its KV head's when sel_div = Hq/Hkv heads share one
  const int64_t sr = sel_div == 1 ? sh : (int64_t)s * place.Hkv + hk;
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = threadIdx.x / DSK_WAVE;
  const int slot0 = chunk * kSlotsPerWg;

  // the wave's slots: slot0 + wave + kAttnWaves * r; their spans are fetched together with the count
  int count = sel_count[sr];
  int st_[SPW], ln_[SPW];
#pragma unroll
  for (int r = 0; r < SPW; ++r) {
    const int j = slot0 + wave + kAttnWaves * r;
    st_[r] = j < k ? sel_start[sr * k + j] : 0;
    ln_[r] = j < k ? sel_len[sr * k + j] : 0;
  }
  if (count > k) count = k;
  if (total_tokens <= 0) count = 0;   // no K/V row exists: not even the redirected loads of skipped slots may run
  if (count <= 0) {   // nothing selected: chunk 0 writes the defined empty result
    if (chunk == 0 && threadIdx.x < DSK_HEAD_DIM) {
      store_attn_out(out, out_bf16, sh * DSK_HEAD_DIM + threadIdx.x, 0.0f);
      if (threadIdx.x == 0 && lse) lse[sh] = -__builtin_inff();
    }
    return;
  }
  if (slot0 >= count) return;   // uniform over the workgroup; not counted in `used` below
  const int used = (count + kSlotsPerWg - 1) / kSlotsPerWg;

  const int g = lane >> 4;
  const int c = lane & 15;
  const QRow qf = make_qrow(*reinterpret_cast<const uint4*>(q + sh * DSK_HEAD_DIM + c * 8));
  const uint16_t* Kh = K + (int64_t)hk * ksh + c * 8;
  const uint16_t* Vh = V + (int64_t)hk * vsh + c * 8;

  WaveState st;
  st.m = -__builtin_inff();
  st.l = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) st.acc[i] = 0.0f;

  if constexpr (REST) {
    // rows r0 .. r0 + 31 of a slot of len rows (r0 < len)
    auto fold_part = [&](int start, int len, int r0) {
      const int nvr = len - r0;
      const uint16_t* kb = Kh + (int64_t)(start + r0) * kst;
      const uint16_t* vb = Vh + (int64_t)(start + r0) * vst;
      if (nvr > 16) fold_rows<8>(st, qf, kb, vb, kst, vst, nvr < 32 ? nvr : 32, g, scale_log2);
      else fold_rows<4>(st, qf, kb, vb, kst, vst, nvr, g, scale_log2);
    };
#pragma unroll
    for (int r = 0; r < SPW; ++r) {
      const int j = slot0 + wave + kAttnWaves * r;
      const int start = st_[r];
      int len = ln_[r];
      if (len > b) len = b;
      ln_[r] = 0;
      if (j >= count || start < 0 || len <= 0 || start > total_tokens - len) continue;   // never read outside K/V
      if constexpr (STAGED) {
        for (int r0 = 0; r0 < len; r0 += 32) fold_part(start, len, r0);
      } else {
        fold_part(start, len, 0);
        ln_[r] = len;                    // for the rows behind
      }
    }
    if constexpr (!STAGED) {
#pragma unroll
      for (int r = 0; r < SPW; ++r)
        for (int r0 = 32; r0 < ln_[r]; r0 += 32) fold_part(st_[r], ln_[r], r0);
    }
  } else {
    // every slot has at most 4*NS rows: all K/V loads of the wave's SPW slots go out now (STAGED: of a slot)
    uint4 kd[SPW][NS], vd[SPW][NS];
    int nv[SPW];
#pragma unroll
    for (int r = 0; r < SPW; ++r) {
      const int j = slot0 + wave + kAttnWaves * r;
      int start = st_[r];
      int len = ln_[r] < b ? ln_[r] : b;
      len = len < 4 * NS ? len : 4 * NS;
      const bool ok = j < count && start >= 0 && len > 0 && start <= total_tokens - len;   // never read outside K/V
      nv[r] = ok ? len : 0;
      start = ok ? start : 0;            // a skipped slot reads row 0 (harmless) so that the loads
      len = ok ? len : 1;                // below stay unconditional
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        int row = 4 * u + g;
        row = row < len ? row : len - 1;
        kd[r][u] = *reinterpret_cast<const uint4*>(Kh + (int64_t)(start + row) * kst);
      }
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        int row = 4 * u + g;
        row = row < len ? row : len - 1;
        vd[r][u] = *reinterpret_cast<const uint4*>(Vh + (int64_t)(start + row) * vst);
      }
      if constexpr (STAGED) {
#pragma unroll
        for (int u = 0; u < NS; ++u) pin_loaded(kd[r][u]);
#pragma unroll
        for (int u = 0; u < NS; ++u) pin_loaded(vd[r][u]);
        if (nv[r] > 0) fold_loaded<NS>(st, qf, kd[r], vd[r], nv[r], g, scale_log2);
      }
    }
    if constexpr (!STAGED) FoldSlots<NS, SPW, 0>::run(st, qf, kd, vd, nv, g, scale_log2);
  }

  // lane groups -> wave
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    st.acc[i] += shfl_xor_f(st.acc[i], 16);
    st.acc[i] += shfl_xor_f(st.acc[i], 32);
  }
  st.l += shfl_xor_f(st.l, 16);
  st.l += shfl_xor_f(st.l, 32);
  if (lane == 0) { sm_m[wave] = st.m; sm_l[wave] = st.l; }
  if (g == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) sm_acc[wave][c * 8 + i] = st.acc[i];
  }
  __syncthreads();

  // waves -> workgroup partial, fixed order
  const int d = threadIdx.x;
  if (d >= DSK_HEAD_DIM) return;
  float M = sm_m[0];
#pragma unroll
  for (int w = 1; w < kAttnWaves; ++w) M = fmaxf(M, sm_m[w]);
  float l = 0.0f, a = 0.0f;
#pragma unroll
  for (int w = 0; w < kAttnWaves; ++w) {
    const float f = sm_m[w] == -__builtin_inff() ? 0.0f : exp2f(sm_m[w] - M);   // idle wave
    l = fmaf(sm_l[w], f, l);
    a = fmaf(sm_acc[w][d], f, a);
  }
  if (used == 1) {   // the only chunk of this head: finish here
    store_attn_out(out, out_bf16, sh * DSK_HEAD_DIM + d, l > 0.0f ? a / l : 0.0f);
    if (d == 0 && lse) lse[sh] = l > 0.0f ? (M + log2f(l)) * kLn2 : -__builtin_inff();
    if (!leave) return;
  }
  const int64_t pbase = sh * nchunks;
  part_acc[(pbase + chunk) * DSK_HEAD_DIM + d] = a;
  if (d == 0) part_ml[pbase + chunk] = make_float2(M, l);
}

// Long lists: one workgroup of kLongWaves wavefronts for every CU, each with many slots of one head (its whole list where
// there are that many heads, which leaves nothing to merge).  A wavefront takes every kLongWaves-th slot, one after the
// other; the spans of 64 slots lie one in each lane.  What it gains is the merge and the starts of the many workgroups:
// eight sequences, 32 / 8 heads, 128 slots of 16 rows, take 31.3 us without a merge against 32.5 and 4.8 with a workgroup per
// 8 slots, from the same 146 MB of HBM (145) with the same third of the requests served by L2; step 55.0 -> 50.4 us (8 steps
// that follow on one cache 496 -> 470).  With two slots of a wavefront in flight 51.9 / 483, with four 51.8 / 494, 4
// wavefronts 56.9 / 530, 12 wavefronts 51.8 / 483, 16 52.6 / 499.  40 / 40 heads, 128K tokens, 256 slots of 16 rows: 40.0 ->
// 38.7 with 6 chunks a head (240 workgroups), 43.5 with 7 (280: the last 24 have the card to themselves).
constexpr int kLongWaves = 8;
constexpr int kLongMinSlots = 32;       // of a workgroup; where a list of less than 256 slots is cut, 8 more: the merge takes
                                        // back what such chunks gain (2 to 8 sequences, 128 slots: 0.2 to 0.4 us slower with 32)
constexpr int kLongMinSlotsShared = 256; // of a list that a group shares: its heads meet in L2 anyway (two sequences of 30K
                                        // tokens, 28 / 4 heads, 128 slots 20.3 -> 20.8 us; one, 16 / 2, 512 slots 32.3 -> 18.9)
constexpr int kSharedChunkSlots = 16;   // of a workgroup of attn_shared_kernel
// SLOTS = 2 (slots of up to 8 rows): two slots in the 16 rows that a wavefront has in flight.  Decode steps with such slots:
// 28 / 4 heads, 130K tokens, 357 slots 23.5 -> 21.9 us; 16 / 2, eight sequences of 15K, 176 slots 27.5 -> 24.3; 32 / 32, three of
// 31K, 636 slots 63.7 -> 63.1 (at the rate of the memory).
template <int NS, int SLOTS = 1>
__global__ __launch_bounds__(kLongWaves * DSK_WAVE) void attn_long_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    int64_t kst, int64_t ksh, int64_t vst, int64_t vsh, int Hq, int G, int n_groups, int k, int b, int total_tokens,
    const int32_t* __restrict__ sel_start, const int32_t* __restrict__ sel_len,
    const int32_t* __restrict__ sel_count, int sel_div, float scale_log2, AttnPlace place, int nchunks, int slots_per_wg,
    float2* __restrict__ part_ml, float* __restrict__ part_acc, float* __restrict__ out,
    uint16_t* __restrict__ out_bf16, float* __restrict__ lse) {
  __shared__ float sm_m[kLongWaves];
  __shared__ float sm_l[kLongWaves];
  __shared__ float sm_acc[kLongWaves][DSK_HEAD_DIM];
  const AttnAt at = attn_place(place, Hq, G, n_groups, nchunks);
  if (at.chunk < 0) return;
  const int64_t sh = (int64_t)at.s * Hq + at.h;
  const int64_t sr = sel_div == 1 ? sh : (int64_t)at.s * place.Hkv + at.hk;   // row of the selection arrays
  const int slot0 = at.chunk * slots_per_wg;
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DSK_WAVE);
  const int g = lane >> 4;
  const int c = lane & 15;

  int start = 0, len = 0;                        // of the lane-th slot of the wavefront's current 64
  auto fetch_spans = [&](int first) {
    const int j = slot0 + (first + lane) * kLongWaves + wave;
    start = j < k ? sel_start[sr * k + j] : 0;
    len = j < k ? sel_len[sr * k + j] : 0;
  };
  fetch_spans(0);
  int count = sel_count[sr];
  const QRow qf = make_qrow(*reinterpret_cast<const uint4*>(q + sh * DSK_HEAD_DIM + c * 8));
  if (count > k) count = k;
  if (total_tokens <= 0) count = 0;
  if (count <= 0) {                              // nothing selected: chunk 0 writes the defined empty result
    if (at.chunk == 0 && threadIdx.x < DSK_HEAD_DIM) {
      store_attn_out(out, out_bf16, sh * DSK_HEAD_DIM + threadIdx.x, 0.0f);
      if (threadIdx.x == 0 && lse) lse[sh] = -__builtin_inff();
    }
    return;
  }
  if (slot0 >= count) return;
  const int own = count - slot0 < slots_per_wg ? count - slot0 : slots_per_wg;     // slots of this workgroup
  const int n = wave < own ? (own - wave + kLongWaves - 1) / kLongWaves : 0;       // of this wavefront
  const uint16_t* Kh = K + (int64_t)at.hk * ksh;
  const uint16_t* Vh = V + (int64_t)at.hk * vsh;
  const unsigned kst8 = (unsigned)kst >> 3, vst8 = (unsigned)vst >> 3;             // strides: multiples of 8, at most 2^24

  WaveState st;
  st.m = -__builtin_inff();
  st.l = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) st.acc[i] = 0.0f;
  for (int first = 0; first < n; first += DSK_WAVE) {
    if (first > 0) fetch_spans(first);
    len = len < b ? len : b;
    len = len < 4 * NS / SLOTS ? len : 4 * NS / SLOTS;
    // slots that exist and do not leave K/V
    unsigned long long todo = __ballot(first + lane < n && start >= 0 && len > 0 && start <= total_tokens - len);
    for (; todo != 0; todo &= todo - 1) {      // of 0: 0
      int nv[SLOTS];
      const char *kb[SLOTS], *vb[SLOTS];                                           // uniform
#pragma unroll
      for (int i = 0; i < SLOTS; ++i) {
        const bool have = i == 0 || todo != 0;
        const int r = __builtin_ctzll(have ? todo : 1ull);
        nv[i] = have ? __builtin_amdgcn_readlane(len, r) : 0;
        const int64_t row0 = __builtin_amdgcn_readlane(start, r);
        kb[i] = have ? reinterpret_cast<const char*>(Kh + row0 * kst) : kb[0];     // none left: the first one's rows again
        vb[i] = have ? reinterpret_cast<const char*>(Vh + row0 * vst) : vb[0];
        if (i + 1 < SLOTS) todo &= todo - 1;
      }
      constexpr int kPer = NS / SLOTS;
      auto row_of = [&](int u) {
        const int row = 4 * (u % kPer) + g, most = (u >= kPer && nv[SLOTS - 1] > 0 ? nv[SLOTS - 1] : nv[0]) - 1;
        return (unsigned)(row < most ? row : most);
      };
      uint4 kd[NS], vd[NS];
#pragma unroll
      for (int u = 0; u < NS; ++u)
        kd[u] = *reinterpret_cast<const uint4*>(kb[u / kPer] + (__umul24(row_of(u), kst8) + (unsigned)c) * 16u);
#pragma unroll
      for (int u = 0; u < NS; ++u)
        vd[u] = *reinterpret_cast<const uint4*>(vb[u / kPer] + (__umul24(row_of(u), vst8) + (unsigned)c) * 16u);
#pragma unroll
      for (int u = 0; u < NS; ++u) pin_loaded(kd[u]);
#pragma unroll
      for (int u = 0; u < NS; ++u) pin_loaded(vd[u]);
      fold_loaded<NS, true, SLOTS>(st, qf, kd, vd, nv[0], g, scale_log2, nv[SLOTS - 1]);
    }
  }

  // lane groups -> wave -> workgroup, as in attn_kernel
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    st.acc[i] += shfl_xor_f(st.acc[i], 16);
    st.acc[i] += shfl_xor_f(st.acc[i], 32);
  }
  st.l += shfl_xor_f(st.l, 16);
  st.l += shfl_xor_f(st.l, 32);
  if (lane == 0) { sm_m[wave] = st.m; sm_l[wave] = st.l; }
  if (g == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) sm_acc[wave][c * 8 + i] = st.acc[i];
  }
  __syncthreads();
  const int d = threadIdx.x;
  if (d >= DSK_HEAD_DIM) return;
  float M = sm_m[0];
#pragma unroll
  for (int w = 1; w < kLongWaves; ++w) M = fmaxf(M, sm_m[w]);
  float l = 0.0f, a = 0.0f;
#pragma unroll
  for (int w = 0; w < kLongWaves; ++w) {
    const float f = sm_m[w] == -__builtin_inff() ? 0.0f : exp2f(sm_m[w] - M);   // idle wave
    l = fmaf(sm_l[w], f, l);
    a = fmaf(sm_acc[w][d], f, a);
  }
  if (count <= slots_per_wg) {                   // the only chunk of this head: finish here
    store_attn_out(out, out_bf16, sh * DSK_HEAD_DIM + d, l > 0.0f ? a / l : 0.0f);
    if (d == 0 && lse) lse[sh] = l > 0.0f ? (M + log2f(l)) * kLn2 : -__builtin_inff();
    return;
  }
  part_acc[(sh * nchunks + at.chunk) * DSK_HEAD_DIM + d] = a;
  if (d == 0) part_ml[sh * nchunks + at.chunk] = make_float2(M, l);
}

// ---- shared selection: one slot list per KV head, used by all its query heads -------------------
// A row is folded into the GT = 2, 4 or 8 heads of the group, which makes the vector ALU the bound of a plain fold: 520
// instructions per slot of 16 rows and 4 heads.  Here the logits come from the matrix cores (16 rows x up to 16 heads:
// four 16x16x32 products per 16 rows, of which the heads use GT columns, repeated over the 16), which leaves a lane with
// four logits of one head instead of every lane with all of them; the weights go back to the rows' lanes by swapping
// halves and rows of the wavefront (a 4 x 4 transposition of registers and lane groups) and are broadcast inside a row of
// 16 lanes.  About 250 instructions.  The sums over V stay in fp32 on the vector ALU.
// A workgroup of kLongWaves wavefronts for every CU, as in attn_long_kernel; `leave` as in attn_kernel.  Steps at 30K tokens,
// 128 slots of 16 rows a list, before (two slots per wavefront, heads in tiles of 2 or 4, other widths per head) and now:
// eight sequences of 32 / 8 heads 33.1 -> 30.1 us, of 28 / 4 heads 36.4 -> 29.8; 512 slots of 8 rows 62.0 -> 46.8 and 75.5 ->
// 41.5.  Random calls of 3072 slots and more, now / before, mean and largest by heads a group: 2 0.90 1.01, 3 0.71 0.90, 4
// 0.75 0.86, 5 0.57 0.85, 6 0.56 0.81, 7 0.50 0.72, 8 0.62 0.79, 9 and more 0.45 0.92.
typedef __attribute__((ext_vector_type(8))) __bf16 attn_bf16x8;
typedef __attribute__((ext_vector_type(4))) float attn_f32x4;
typedef __attribute__((ext_vector_type(2))) unsigned attn_u32x2;

// the 4 x 4 transposition: register i of lane group u (16 lanes each) <-> register u of lane group i
__device__ __forceinline__ void transpose_groups(float (&p)[4]) {
  auto swap32 = [](float& x, float& y) {   // upper half of x <-> lower half of y
    const attn_u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r.x); y = __uint_as_float(r.y);
  };
  auto swap16 = [](float& x, float& y) {   // groups 1 and 3 of x <-> groups 0 and 2 of y
    const attn_u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r.x); y = __uint_as_float(r.y);
  };
  swap32(p[0], p[2]); swap32(p[1], p[3]);
  swap16(p[0], p[1]); swap16(p[2], p[3]);
}
// maximum over the four lane groups, in every lane
__device__ __forceinline__ float groups_max(float v) {
  attn_u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}
constexpr int kDppRowBcast = 0x150;        // + n: lane n of a row of 16 -> every lane of the row

// acc[j][k] *= lane j of the row: alpha;  acc[j][k] += (lane j of the row: p) * v[k]
template <int GT, int J = 0>
__device__ __forceinline__ void rescale(float (&acc)[GT][8], float alpha) {
  if constexpr (J < GT) {
    const float a = dpp_f<kDppRowBcast + J>(alpha);
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[J][k] *= a;
    rescale<GT, J + 1>(acc, alpha);
  }
}
template <int GT, int J = 0>
__device__ __forceinline__ void add_row(float (&acc)[GT][8], float p, const float (&f)[8]) {
  if constexpr (J < GT) {
    const float w = dpp_f<kDppRowBcast + J>(p);
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[J][k] = fmaf(w, f[k], acc[J][k]);
    add_row<GT, J + 1>(acc, p, f);
  }
}

// NT: 16-row tiles of a slot; GT: query heads of a tile of the group (the last tile of a group may have fewer; the columns
// of those it does not have repeat its first one).  WIDE: token strides above kMaxTokenStride, row offsets in 64 bits (the
// chunks, which a caller that merges by itself asks for, do not depend on the strides).
// grid: chunk, fastest, then head tile, KV head, sequence
// SLOTS = 2 (NT = 1, slots of up to 8 rows): a tile holds the rows of two slots: 28 / 4 heads, eight sequences of 50K tokens, 311
// slots 39.2 -> 35.8 us.
template <int NT, int GT, bool WIDE, int SLOTS = 1>
__global__ __launch_bounds__(kLongWaves * DSK_WAVE) void attn_shared_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    int64_t kst, int64_t ksh, int64_t vst, int64_t vsh, int Hq, int G, int k, int b, int total_tokens,
    const int32_t* __restrict__ sel_start, const int32_t* __restrict__ sel_len,
    const int32_t* __restrict__ sel_count, float scale_log2, int nchunks, int slots_per_wg, bool leave,
    float2* __restrict__ part_ml, float* __restrict__ part_acc, float* __restrict__ out,
    uint16_t* __restrict__ out_bf16, float* __restrict__ lse) {
  static_assert(GT <= 8 && 16 % GT == 0, "the heads repeat over the 16 columns of a product");
  static_assert(SLOTS == 1 || (SLOTS == 2 && NT == 1), "two slots in one tile");
  constexpr int kSlotRows = 16 * NT / SLOTS;
  __shared__ float sm_m[kLongWaves][GT];
  __shared__ float sm_l[kLongWaves][GT];
  __shared__ float sm_acc[kLongWaves][GT][DSK_HEAD_DIM];
  const int tiles = (G + GT - 1) / GT;
  const int list = blockIdx.x / nchunks;
  const int chunk = blockIdx.x - list * nchunks;
  const int sr = list / tiles;                              // row of the selection arrays: (sequence, KV head)
  const int hk = sr % (Hq / G);
  const int h0 = (list - sr * tiles) * GT;
  const int heads = G - h0 < GT ? G - h0 : GT;              // of this tile
  const int64_t sh0 = (int64_t)sr * G + h0;                 // first of them, over all sequences
  const int slot0 = chunk * slots_per_wg;
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DSK_WAVE);
  const int g = lane >> 4;
  const int c = lane & 15;

  int start = 0, len = 0;                        // of the lane-th slot of the wavefront's current 64
  auto fetch_spans = [&](int first) {
    const int j = slot0 + (first + lane) * kLongWaves + wave;
    start = j < k ? sel_start[(int64_t)sr * k + j] : 0;
    len = j < k ? sel_len[(int64_t)sr * k + j] : 0;
  };
  fetch_spans(0);
  int count = sel_count[sr];
  // operand of the queries: column c = head c % GT, channels 32 i + 8 g .. + 8
  attn_bf16x8 qf[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    qf[i] = *reinterpret_cast<const attn_bf16x8*>(q + (sh0 + (c % GT < heads ? c % GT : 0)) * DSK_HEAD_DIM + 32 * i + 8 * g);
  if (count > k) count = k;
  if (total_tokens <= 0) count = 0;   // no K/V row exists
  if (count <= 0) {   // nothing selected: chunk 0 writes the defined empty result of the tile's heads
    if (chunk == 0 && threadIdx.x < DSK_HEAD_DIM) {
#pragma unroll
      for (int j = 0; j < GT; ++j) {
        if (j >= heads) break;
        store_attn_out(out, out_bf16, (sh0 + j) * DSK_HEAD_DIM + threadIdx.x, 0.0f);
        if (threadIdx.x == 0 && lse) lse[sh0 + j] = -__builtin_inff();
      }
    }
    return;
  }
  if (slot0 >= count) return;
  const int own = count - slot0 < slots_per_wg ? count - slot0 : slots_per_wg;     // slots of this workgroup
  const int n = wave < own ? (own - wave + kLongWaves - 1) / kLongWaves : 0;       // of this wavefront
  const uint16_t* Kh = K + (int64_t)hk * ksh;
  const uint16_t* Vh = V + (int64_t)hk * vsh;
  const unsigned kst8 = (unsigned)kst >> 3, vst8 = (unsigned)vst >> 3;             // strides: multiples of 8, at most 2^24
  // 16 bytes at column `col` of row `row`
  auto at_row = [](const char* base, int row, int64_t stride, unsigned stride8, int col) {
    if constexpr (WIDE) return base + ((int64_t)row * stride * 2 + col * 16);
    else return base + (__umul24((unsigned)row, stride8) + (unsigned)col) * 16u;
  };

  // of head c % GT: reference, this lane group's part of the denominator; of all heads: channels 8c .. of this group's rows
  float m = -__builtin_inff(), l = 0.0f, acc[GT][8];
#pragma unroll
  for (int j = 0; j < GT; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[j][i] = 0.0f;

  for (int first = 0; first < n; first += DSK_WAVE) {
    if (first > 0) fetch_spans(first);
    len = len < b ? len : b;
    len = len < kSlotRows ? len : kSlotRows;
    // slots that exist and do not leave K/V
    unsigned long long todo = __ballot(first + lane < n && start >= 0 && len > 0 && start <= total_tokens - len);
    for (; todo != 0; todo &= todo - 1) {      // of 0: 0
      int nv[SLOTS];
      const char *kb[SLOTS], *vb[SLOTS];                                           // uniform
#pragma unroll
      for (int i = 0; i < SLOTS; ++i) {
        const bool have = i == 0 || todo != 0;
        const int r = __builtin_ctzll(have ? todo : 1ull);
        nv[i] = have ? __builtin_amdgcn_readlane(len, r) : 0;
        const int64_t row0 = __builtin_amdgcn_readlane(start, r);
        kb[i] = have ? reinterpret_cast<const char*>(Kh + row0 * kst) : kb[0];     // none left: the first one's rows again
        vb[i] = have ? reinterpret_cast<const char*>(Vh + row0 * vst) : vb[0];
        if (i + 1 < SLOTS) todo &= todo - 1;
      }
      // row of its slot for row x of the tiles, one of the second slot where x is behind the first; those behind a slot's last
      // row repeat it
      auto second = [&](int x) { return SLOTS == 2 && x >= kSlotRows; };
      auto slot_row = [&](int x) {
        const int row = SLOTS == 2 ? x & (kSlotRows - 1) : x;
        const int most = (second(x) && nv[SLOTS - 1] > 0 ? nv[SLOTS - 1] : nv[0]) - 1;
        return row < most ? row : most;
      };
      auto real_row = [&](int x) { return (SLOTS == 2 ? x & (kSlotRows - 1) : x) < (second(x) ? nv[SLOTS - 1] : nv[0]); };
      // K as operand: row c of the tile, channels 32 i + 8 g .. + 8; V as rows 4 u + g, channels 8 c .. + 8
      u32x4_t kd[NT][4], vd[4 * NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const char* from = at_row(second(c) ? kb[SLOTS - 1] : kb[0], slot_row(16 * t + c), kst, kst8, g);
#pragma unroll
        for (int i = 0; i < 4; ++i) kd[t][i] = *reinterpret_cast<const u32x4_t*>(from + 64 * i);
      }
#pragma unroll
      for (int u = 0; u < 4 * NT; ++u)
        vd[u] = *reinterpret_cast<const u32x4_t*>(at_row(SLOTS == 2 && u >= 2 ? vb[SLOTS - 1] : vb[0], slot_row(4 * u + g), vst, vst8, c));
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) pin_loaded(kd[t][i]);
#pragma unroll
      for (int u = 0; u < 4 * NT; ++u) pin_loaded(vd[u]);
      // z[t][i]: logit of row 16 t + 4 g + i against head c % GT
      float z[NT][4];
      float top = -__builtin_inff();
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        // four products of 32 channels, added here: as one chain through the accumulator the outputs are 20 % further
        // from 64 bits than with the packed dot instruction, this way 4 % nearer
        const attn_f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
        attn_f32x4 d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          d[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(attn_bf16x8, kd[t][i]), qf[i], zero, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float sum = (d[0][i] + d[1][i]) + (d[2][i] + d[3][i]);
          z[t][i] = real_row(16 * t + 4 * g + i) ? sum * scale_log2 : -__builtin_inff();
          top = fmaxf(top, z[t][i]);
        }
      }
      const float m_new = fmaxf(m, groups_max(top));      // finite: nv >= 1
      const float alpha = exp2_small(m - m_new);         // 0 on the first fold
      m = m_new;
      float part = 0.0f;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { z[t][i] = exp2_small(z[t][i] - m_new); part += z[t][i]; }   // 0 for padded rows
        transpose_groups(z[t]);                           // z[t][u]: weight of row 16 t + 4 u + g
      }
      l = fmaf(l, alpha, part);
      rescale<GT>(acc, alpha);
#pragma unroll
      for (int u = 0; u < 4 * NT; ++u) {
        float f[8];
        unpack8(make_uint4(vd[u].x, vd[u].y, vd[u].z, vd[u].w), f);
        add_row<GT>(acc, z[u / 4][u % 4], f);
      }
    }
  }

  // lane groups -> wave
#pragma unroll
  for (int j = 0; j < GT; ++j) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[j][i] += shfl_xor_f(acc[j][i], 16);
      acc[j][i] += shfl_xor_f(acc[j][i], 32);
    }
    if (g == 0) {
#pragma unroll
      for (int i = 0; i < 8; ++i) sm_acc[wave][j][c * 8 + i] = acc[j][i];
    }
  }
  l += shfl_xor_f(l, 16);
  l += shfl_xor_f(l, 32);
  if (lane < GT) { sm_m[wave][lane] = m; sm_l[wave][lane] = l; }
  __syncthreads();

  // waves -> one partial per head of the tile, fixed order
  for (int idx = threadIdx.x; idx < heads * DSK_HEAD_DIM; idx += kLongWaves * DSK_WAVE) {
    const int j = idx / DSK_HEAD_DIM;
    const int d = idx % DSK_HEAD_DIM;
    float M = sm_m[0][j];
#pragma unroll
    for (int w = 1; w < kLongWaves; ++w) M = fmaxf(M, sm_m[w][j]);
    float ls = 0.0f, a = 0.0f;
#pragma unroll
    for (int w = 0; w < kLongWaves; ++w) {
      const float f = sm_m[w][j] == -__builtin_inff() ? 0.0f : exp2f(sm_m[w][j] - M);   // idle wave
      ls = fmaf(sm_l[w][j], f, ls);
      a = fmaf(sm_acc[w][j][d], f, a);
    }
    const int64_t sh = sh0 + j;
    if (count <= slots_per_wg) {
      store_attn_out(out, out_bf16, sh * DSK_HEAD_DIM + d, ls > 0.0f ? a / ls : 0.0f);
      if (d == 0 && lse) lse[sh] = ls > 0.0f ? (M + log2f(ls)) * kLn2 : -__builtin_inff();
    }
    if (count > slots_per_wg || leave) {
      part_acc[(sh * nchunks + chunk) * DSK_HEAD_DIM + d] = a;
      if (d == 0) part_ml[sh * nchunks + chunk] = make_float2(M, ls);
    }
  }
}

// Merge of the partials of one (sequence, head) in a fixed order: 16 lane groups each fold the
// chunks ch = group, group+16, ... (all loads of a round are independent), then one pass over
// the 16 group states in LDS.  Heads with a single chunk were finished by attn_kernel.
template <int kMergeThreads>
__global__ __launch_bounds__(kMergeThreads) void attn_merge_kernel(
    const float2* __restrict__ part_ml, const float* __restrict__ part_acc,
    const int32_t* __restrict__ sel_count, const int32_t* __restrict__ cu_seqlens, int Hq, int sel_div, int k,
    int nchunks, int slots_per_wg, float* __restrict__ out, uint16_t* __restrict__ out_bf16,
    float* __restrict__ lse) {
  constexpr int kMergeGroups = kMergeThreads / 16;
  __shared__ float sm_m[kMergeGroups];
  __shared__ float sm_l[kMergeGroups];
  __shared__ float sm_acc[kMergeGroups][DSK_HEAD_DIM];
  const int64_t sh = blockIdx.x;
  const int grp = threadIdx.x >> 4;
  const int c = threadIdx.x & 15;
  const float2* ml = part_ml + sh * nchunks;
  const float* acc = part_acc + sh * nchunks * DSK_HEAD_DIM + c * 8;
  // first round of partials is fetched together with the count (the workspace always holds
  // nchunks entries per head; stale ones are discarded below by index)
  float2 v0 = make_float2(0.0f, 0.0f);
  float4 x00 = make_float4(0.f, 0.f, 0.f, 0.f), x01 = x00;
  if (grp < nchunks) {
    v0 = ml[grp];
    x00 = *reinterpret_cast<const float4*>(acc + (int64_t)grp * DSK_HEAD_DIM);
    x01 = *reinterpret_cast<const float4*>(acc + (int64_t)grp * DSK_HEAD_DIM + 4);
  }
  // units folded per head: selected slots, or (full attention) the tokens of the sequence
  int count;
  if (cu_seqlens != nullptr) {
    const int s = (int)(sh / Hq);
    count = cu_seqlens[s + 1] - cu_seqlens[s];
  } else {
    if (sel_div == 1) {
      count = sel_count[sh];
    } else {
      const int s = (int)(sh / Hq), h = (int)(sh % Hq);
      count = sel_count[(int64_t)s * (Hq / sel_div) + h / sel_div];
    }
  }
  if (count > k) count = k;
  int used = (int)(((int64_t)count + slots_per_wg - 1) / slots_per_wg);
  if (used > nchunks) used = nchunks;   // never past the partials this head owns
  if (used <= 1) return;   // empty or single-chunk heads are complete already
  float m = -__builtin_inff(), l = 0.0f, a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = 0.0f;
  for (int ch = grp; ch < used; ch += kMergeGroups) {
    float2 v;
    float4 x0, x1;
    if (ch == grp) { v = v0; x0 = x00; x1 = x01; }
    else {
      v = ml[ch];
      x0 = *reinterpret_cast<const float4*>(acc + (int64_t)ch * DSK_HEAD_DIM);
      x1 = *reinterpret_cast<const float4*>(acc + (int64_t)ch * DSK_HEAD_DIM + 4);
    }
    if (v.x == -__builtin_inff()) continue;
    const float mn = fmaxf(m, v.x);
    const float fo = exp2f(m - mn), fn = exp2f(v.x - mn);   // m = -inf -> fo = 0
    l = l * fo + v.y * fn;
    a[0] = a[0] * fo + x0.x * fn; a[1] = a[1] * fo + x0.y * fn; a[2] = a[2] * fo + x0.z * fn; a[3] = a[3] * fo + x0.w * fn;
    a[4] = a[4] * fo + x1.x * fn; a[5] = a[5] * fo + x1.y * fn; a[6] = a[6] * fo + x1.z * fn; a[7] = a[7] * fo + x1.w * fn;
    m = mn;
  }
  if (c == 0) { sm_m[grp] = m; sm_l[grp] = l; }
#pragma unroll
  for (int i = 0; i < 8; ++i) sm_acc[grp][c * 8 + i] = a[i];
  __syncthreads();
  const int d = threadIdx.x;
  if (d < DSK_HEAD_DIM) {
    float M = sm_m[0];
#pragma unroll
    for (int g2 = 1; g2 < kMergeGroups; ++g2) M = fmaxf(M, sm_m[g2]);
    float L = 0.0f, A = 0.0f;
#pragma unroll
    for (int g2 = 0; g2 < kMergeGroups; ++g2) {
      const float f = sm_m[g2] == -__builtin_inff() ? 0.0f : exp2f(sm_m[g2] - M);
      L = fmaf(sm_l[g2], f, L);
      A = fmaf(sm_acc[g2][d], f, A);
    }
    store_attn_out(out, out_bf16, sh * DSK_HEAD_DIM + d, L > 0.0f ? A / L : 0.0f);
    if (d == 0 && lse) lse[sh] = L > 0.0f ? (M + log2f(L)) * kLn2 : -__builtin_inff();
  }
}

// Chunks per list for the kernels that want a workgroup on every CU: those that occupy the CUs most evenly (in up to
// max_rounds workgroups a CU; a list that takes more by itself stays whole where several are allowed), the fewest of them
// within 6 %, with at least min_slots slots in each where there are several; 0 if none reaches min_use.
// per_xcd(ch): workgroups on the busiest XCD.
constexpr int kCusPerXcd = 32;
constexpr int kManyRounds = 4;
template <typename PerXcd>
static int attn_even_chunks(PerXcd per_xcd, int64_t lists, int k, int min_slots, double min_use, int max_rounds) {
  int best = 0;
  double best_use = 0.0;
  for (int ch = 1; ch == 1 || ch * min_slots <= k; ++ch) {
    const int64_t rounds = (per_xcd(ch) + kCusPerXcd - 1) / kCusPerXcd;
    if (rounds > max_rounds && (best > 0 || max_rounds == 1)) break;
    const double use = (double)lists * ch / ((double)rounds * kCusPerXcd * 8);
    if (use >= min_use && (best == 0 || use > best_use + 0.06)) { best = ch; best_use = use; }
    if (rounds > max_rounds) break;
  }
  return best;
}

// Lists per head on attn_long_kernel: where one workgroup a CU occupies at least 85 % of the CUs.  435 such calls with random
// heads (1 to 16 a group), batches, lists and shared rows took 0.89 times as long as on attn_kernel in the mean, 1.036 at
// most; with 75 to 85 % of them it would be 0.92, but a seventh of the calls more than 2 % longer.  (The 6 % above: no
// slack is as fast, 15 % 1.04 times as long.)  With several workgroups a CU the heads of a group are side by side no longer
// and fetch more of their common rows anew (198 -> 237 MB in the last example).  That pays, time on attn_kernel = 1, mean and
// largest,
//  - in groups of 10 heads and more: 713 calls 0.78, 1.06;
//  - for lists of up to 1024 rows: 262 calls 0.83, 1.02;
//  - for slots that leave a quarter and more of the 16 or 32 rows that both kernels have in flight empty: 1457 calls 0.85, 1.05;
//  - for whole lists (nothing to merge) of slots of up to 16 rows, 293 calls 0.90, 1.035; of larger ones up to 2700 rows, 118
//    calls 0.90, 1.02;
//  - where the lists of a group have more than 100 000 rows together, 88 calls 0.87, 1.01, or, if the last round is full to
//    95 %, more than 75 000, 102 calls 0.88, 1.04, or there are 8 heads and more, 104 calls 0.85, 1.04.
// The other 1000 took 0.97 in the mean, but a fifth of them more than 2 % longer than on attn_kernel, 13 % at most (48 / 8
// heads, six sequences, 175 slots of 16 rows 34.1 -> 38.0 us).  Slots of up to 8 rows, measured again with two of them in flight on
// both kernels: 97 calls that take this one 0.91, 1.03; with one round only 1.03 of the time as chosen, 1.40 at most.
static bool attn_long_in_rounds(const dsk_attn_args& a, int G, int chunks, double use) {
  const int64_t rows = (int64_t)a.k * a.b;
  return G >= 10 || rows <= 1024 || a.b <= 12 || (a.b > 16 && a.b <= 24) ||
         (chunks == 1 && (a.b <= 16 || rows <= 2700)) || G * rows > 100000 ||
         (use >= 0.95 && (G * rows > 75000 || G >= 8));
}

// The space asked for is that of short chunks (8 or 16 slots), whatever the call takes.
AttnWs attn_ws_layout(const dsk_attn_args& a, bool size_only) {
  AttnWs ws;
  const int short_slots = attn_slots_per_wg(a.b);
  const int G = a.Hkv > 0 ? a.Hq / a.Hkv : 1;
  const bool many = a.b <= 16 && (int64_t)a.B * a.Hq * ((a.k + short_slots - 1) / short_slots) >= kAttnSmallWgFrom;
  const bool room8 = many || ((a.flags & DSK_ATTN_SHARED_SELECTION) && (G == 2 || G == 4 || G == 8) && a.b <= 32 &&
                              (int64_t)a.B * a.Hkv * a.k >= 4096);
  auto chunks_of = [&](int slots) { return (a.k + slots - 1) / slots; };
  const int room = chunks_of(room8 ? 8 : short_slots);       // partials of a head
  const size_t n = (size_t)a.B * a.Hq * room;
  ws.part_ml = 0;
  ws.part_acc = align_up(n * sizeof(float2));
  ws.total = ws.part_acc + align_up(n * DSK_HEAD_DIM * sizeof(float));
  ws.kernel = AttnKernel::kShort;
  ws.slots_per_wg = many ? 8 : short_slots;
  ws.nchunks = chunks_of(ws.slots_per_wg);
  if (size_only || a.Hkv < 1) return ws;
  // A caller that merges the partials itself keeps short chunks of lists per query head.
  const bool own_merge = (a.flags & DSK_ATTN_PARTIALS_ONLY) != 0;
  int chunks = 0;
  if (attn_shared(a)) {
    const int tile = attn_shared_tile(G);
    const int64_t lists = (int64_t)a.B * a.Hkv * ((G + tile - 1) / tile);
    chunks = attn_even_chunks([&](int ch) { return (lists * ch + 7) / 8; }, lists, a.k, kSharedChunkSlots, 0.0,
                              kManyRounds);
    if (own_merge && chunks < 2) chunks = 2;                 // it is partials that such a caller wants
    if (chunks > room) chunks = room;
    ws.kernel = AttnKernel::kShared;
  } else if (!own_merge && a.b <= 32 && a.k >= ((a.flags & DSK_ATTN_SHARED_SELECTION) ? kLongMinSlotsShared : kLongMinSlots) &&
             a.k_stride_tok <= kMaxTokenStride && a.v_stride_tok <= kMaxTokenStride) {
    const int n_groups = a.B * a.Hkv;
    auto even = [&](int max_rounds) {
      return attn_even_chunks([&](int ch) { return attn_wgs_per_xcd(G, n_groups, ch); }, (int64_t)a.B * a.Hq, a.k,
                              a.k < 256 ? kLongMinSlots + 8 : kLongMinSlots, 0.85, max_rounds);
    };
    chunks = even(kManyRounds);
    const int64_t rounds = (attn_wgs_per_xcd(G, n_groups, chunks) + kCusPerXcd - 1) / kCusPerXcd;
    if (rounds > 1 && !attn_long_in_rounds(a, G, chunks, (double)a.B * a.Hq * chunks / (double)(rounds * kCusPerXcd * 8)))
      chunks = even(1);
    if (chunks >= ws.nchunks) chunks = 0;
    if (chunks > 0) ws.kernel = AttnKernel::kLong;
  }
  if (chunks > 0) {
    ws.slots_per_wg = (a.k + chunks - 1) / chunks;
    ws.nchunks = chunks_of(ws.slots_per_wg);
  }
  return ws;
}

hipError_t launch_attn(const dsk_attn_args& a, const AttnWs& ws, hipStream_t st) {
  unsigned char* w = static_cast<unsigned char*>(a.workspace);
  float2* part_ml = reinterpret_cast<float2*>(w + ws.part_ml);
  float* part_acc = reinterpret_cast<float*>(w + ws.part_acc);
  const float scale = a.scale != 0.0f ? a.scale : 0.08838834764831845f;   // 128^-1/2
  const int n_groups = a.B * a.Hkv;
  const AttnPlace place = attn_placement(a.Hq / a.Hkv, n_groups, a.Hkv, ws.nchunks);
  const dim3 grid(a.Hq == a.Hkv ? (unsigned)(n_groups * ws.nchunks)
                                : (unsigned)(8 * attn_wgs_per_xcd(a.Hq / a.Hkv, n_groups, ws.nchunks)));

  const uint16_t* q = static_cast<const uint16_t*>(a.q);
  const uint16_t* K = static_cast<const uint16_t*>(a.K);
  const uint16_t* V = static_cast<const uint16_t*>(a.V);
  // heads that read one row of the selection arrays; the workgroups of a group's heads gather the
  // same rows on one XCD, so only one of them misses in L2
  const int sel_div = (a.flags & DSK_ATTN_SHARED_SELECTION) ? a.Hq / a.Hkv : 1;
  // a caller that merges by itself finds the partials of every list that has a slot
  const bool leave = (a.flags & DSK_ATTN_PARTIALS_ONLY) != 0 && ws.nchunks > 1;
  if (ws.kernel != AttnKernel::kShort) {
    const dim3 block(kLongWaves * DSK_WAVE);
#define DSK_LONG_ARGS                                                                                             \
  sel_div, scale * kLog2e, place, ws.nchunks, ws.slots_per_wg, part_ml, part_acc, a.out, static_cast<uint16_t*>(a.out_bf16), a.lse
#define DSK_GATHER_ARGS(...)                                                                                      \
  q, K, V, a.k_stride_tok, a.k_stride_head, a.v_stride_tok, a.v_stride_head, a.Hq, a.Hq / a.Hkv, __VA_ARGS__ a.k, a.b, \
      a.total_tokens, a.sel_start, a.sel_len, a.sel_count
#define DSK_SHARED_ARGS                                                                                           \
  DSK_GATHER_ARGS(), scale * kLog2e, ws.nchunks, ws.slots_per_wg, leave, part_ml, part_acc, a.out,                       \
      static_cast<uint16_t*>(a.out_bf16), a.lse
    if (ws.kernel == AttnKernel::kLong) {
      if (a.b <= 8) attn_long_kernel<4, 2><<<grid, block, 0, st>>>(DSK_GATHER_ARGS(n_groups,), DSK_LONG_ARGS);
      else if (a.b <= 16) attn_long_kernel<4><<<grid, block, 0, st>>>(DSK_GATHER_ARGS(n_groups,), DSK_LONG_ARGS);
      else attn_long_kernel<8><<<grid, block, 0, st>>>(DSK_GATHER_ARGS(n_groups,), DSK_LONG_ARGS);
    } else {
      const int G = a.Hq / a.Hkv, tile = attn_shared_tile(G);
      const dim3 sgrid((unsigned)(n_groups * ((G + tile - 1) / tile) * ws.nchunks));
      const bool wide = a.k_stride_tok > kMaxTokenStride || a.v_stride_tok > kMaxTokenStride;
#define DSK_SHARED_LAUNCH(NT, GT)                                                                                 \
  do {                                                                                                            \
    if (NT == 1 && !wide && a.b <= 8) attn_shared_kernel<1, GT, false, 2><<<sgrid, block, 0, st>>>(DSK_SHARED_ARGS); \
    else if (wide) attn_shared_kernel<NT, GT, true><<<sgrid, block, 0, st>>>(DSK_SHARED_ARGS);                         \
    else attn_shared_kernel<NT, GT, false><<<sgrid, block, 0, st>>>(DSK_SHARED_ARGS);                             \
  } while (0)
      switch (tile * 64 + (a.b <= 16 ? 1 : 2)) {
        case 2 * 64 + 1: DSK_SHARED_LAUNCH(1, 2); break;
        case 2 * 64 + 2: DSK_SHARED_LAUNCH(2, 2); break;
        case 4 * 64 + 1: DSK_SHARED_LAUNCH(1, 4); break;
        case 4 * 64 + 2: DSK_SHARED_LAUNCH(2, 4); break;
        case 8 * 64 + 1: DSK_SHARED_LAUNCH(1, 8); break;
        default: DSK_SHARED_LAUNCH(2, 8);
      }
#undef DSK_SHARED_LAUNCH
    }
#undef DSK_LONG_ARGS
#undef DSK_SHARED_ARGS
#undef DSK_GATHER_ARGS
    const hipError_t lerr = hipGetLastError();
    if (lerr != hipSuccess || ws.nchunks <= 1 || (a.flags & DSK_ATTN_PARTIALS_ONLY) || a.total_tokens <= 0) return lerr;
    return launch_attn_merge(part_ml, part_acc, a.sel_count, nullptr, a.B, a.Hq, sel_div, a.k, ws.nchunks,
                             ws.slots_per_wg, a.out, static_cast<uint16_t*>(a.out_bf16), a.lse, st);
  }
#define DSK_ATTN_ARGS                                                                                          \
  q, K, V, a.k_stride_tok, a.k_stride_head, a.v_stride_tok, a.v_stride_head, a.Hq, a.Hq / a.Hkv, n_groups, a.k, a.b, \
      a.total_tokens, a.sel_start, a.sel_len, a.sel_count, sel_div, scale * kLog2e, place, ws.nchunks, leave, part_ml, part_acc, \
      a.out, static_cast<uint16_t*>(a.out_bf16), a.lse
  // Slots of at most 32 rows: workgroups of 8 wavefronts, 2 slots each (16 slots per workgroup).
  // Measured against 4 wavefronts x 2 or 4 slots, 8 x 1 or 4, 16 x 1 or 2 on all configurations:
  // the gather takes 7.3 instead of 8.6 us at 128K / b = 32, and 4.6 instead of 5.6 us at
  // 32K / b = 16 (half as many workgroups to dispatch and half as many partials to merge).
  // Slots of up to 8 rows: half of the loads (32 / 8 heads at 5.6K tokens, 54 slots 13.4 -> 12.65 us, at 11K, eight sequences
  // 21.1 -> 20.4; workgroups of 4 wavefronts x 4 slots 12.9 and 20.8).
  if (a.b <= 8 && ws.slots_per_wg == 8) attn_kernel<2, 2, 4, false><<<grid, dim3(256), 0, st>>>(DSK_ATTN_ARGS);
  else if (a.b <= 8) attn_kernel<2, 2, 8, false><<<grid, dim3(512), 0, st>>>(DSK_ATTN_ARGS);
  else if (a.b <= 16 && ws.slots_per_wg == 8) attn_kernel<4, 2, 4, false><<<grid, dim3(256), 0, st>>>(DSK_ATTN_ARGS);
  else if (a.b <= 16) attn_kernel<4, 2, 8, false><<<grid, dim3(512), 0, st>>>(DSK_ATTN_ARGS);
  else if (a.b <= 32) attn_kernel<8, 2, 8, true><<<grid, dim3(512), 0, st>>>(DSK_ATTN_ARGS);
  else if ((a.b >= kAttnOneSlotFrom && sel_div == 1) || (int64_t)a.B * a.Hq * ws.nchunks <= kAttnWavePerSlotTo)
    attn_kernel<8, 1, 8, false, true><<<grid, dim3(512), 0, st>>>(DSK_ATTN_ARGS);
  else if (a.Hq == a.Hkv) attn_kernel<8, 2, 4, true, true><<<grid, dim3(256), 0, st>>>(DSK_ATTN_ARGS);
  else attn_kernel<8, 2, 4, false, true><<<grid, dim3(256), 0, st>>>(DSK_ATTN_ARGS);
#undef DSK_ATTN_ARGS
  hipError_t err = hipGetLastError();
  // a cache without tokens: every head already holds the defined empty result, no partial exists
  if (err != hipSuccess || ws.nchunks <= 1 || (a.flags & DSK_ATTN_PARTIALS_ONLY) || a.total_tokens <= 0) return err;
  return launch_attn_merge(part_ml, part_acc, a.sel_count, nullptr, a.B, a.Hq, sel_div, a.k, ws.nchunks,
                           ws.slots_per_wg, a.out, static_cast<uint16_t*>(a.out_bf16), a.lse, st);
}

hipError_t launch_attn_merge(const float2* part_ml, const float* part_acc, const int32_t* counts,
                             const int32_t* cu_seqlens, int B, int Hq, int sel_div, int k, int nchunks, int per_chunk,
                             float* out, uint16_t* out_bf16, float* lse, hipStream_t st) {
  // one lane group of 16 per partial when there are few, several partials per group otherwise
  const dim3 grid((unsigned)(B * Hq));
  if (nchunks <= 8)
    attn_merge_kernel<128><<<grid, dim3(128), 0, st>>>(part_ml, part_acc, counts, cu_seqlens, Hq, sel_div, k, nchunks,
                                                       per_chunk, out, out_bf16, lse);
  else if (nchunks <= 32)
    attn_merge_kernel<256><<<grid, dim3(256), 0, st>>>(part_ml, part_acc, counts, cu_seqlens, Hq, sel_div, k, nchunks,
                                                       per_chunk, out, out_bf16, lse);
  else
    attn_merge_kernel<kMergeBigThreads><<<grid, dim3(kMergeBigThreads), 0, st>>>(
        part_ml, part_acc, counts, cu_seqlens, Hq, sel_div, k, nchunks, per_chunk, out, out_bf16, lse);
  return hipGetLastError();
}

}  // namespace dsk
