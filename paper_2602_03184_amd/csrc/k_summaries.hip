// V2F compression (Sec. 4.2, KVCache Compression): element-wise min and max of K (or V)
// over the tokens of every variable-length block.  One wavefront per (head, block):
// a 128-channel bf16 row is 256 B = 16 lanes x 16 B, so the 64 lanes cover 4 token rows
// per load instruction; rows stream from HBM fully coalesced and each is read once.
#include "dsk_common.hpp"
#include "dsk_internal.hpp"

namespace dsk {

constexpr int kSumThreads = 256;
constexpr int kSumWaves = kSumThreads / DSK_WAVE;
constexpr int kSumUnroll = 8;  // row-groups of 4 rows in flight per wave

// min / max (or mean) of rows [0, len) of one head, `base` pointing at row 0 of the block, written
// to the 512-byte record `o`.  All 64 lanes of a wavefront call it with wave-uniform arguments.
// STREAM (the full pass): the records are stored past the cache's replacement order.  Written through it
// they leave it one by one between the reads, which costs far more than their bytes: K and V summaries of
// eight sequences, 24K to 64K tokens, 8 heads: 361 -> 345 us for the pass from the larger grid, -> 307 us from
// these stores.  The first selection that follows reads them from memory instead of the memory-side cache: one
// sequence of 128K tokens, 8 heads, chunks of 32: pass 66.6 -> 62.6 us, pass and selection 78.4 -> 74.7; chunks of 8:
// pass unchanged, both 180 -> 183.
// STREAM_ROWS: the rows are read past the caches too.  The decode step that follows finds in the memory-side cache
// what was read last (eight sequences, all rows streamed: pass -23 us, step +30), so the launch streams only what
// would have left that cache again by its end.
// kUnroll: row-groups in flight; those behind the first kSumUnroll are left out, four at a time, where the block has no row for them.
template <bool MEAN, bool STREAM, bool STREAM_ROWS = false, int kUnroll = kSumUnroll>
__device__ __forceinline__ void summarize_block(const uint16_t* base, int len, int64_t stride_tok, unsigned ustride8,
                                                uint16_t* o, int g, int c) {
  static_assert((4 * kUnroll - 1) * kMaxTokenStride * 2 + 256 <= (int64_t)1 << 32, "byte offsets of the rows in 32 bits");
  // MEAN: mn[] holds this lane's running sums instead
  float mn[8], mx[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) { mn[k] = MEAN ? 0.0f : __builtin_inff(); mx[k] = -__builtin_inff(); }
  for (int r0 = 0; r0 < len; r0 += 4 * kUnroll) {
    // scalar 64-bit base of this row batch + 32-bit lane offsets (stride_tok <= 2^24, host-checked)
    const char* rb = reinterpret_cast<const char*>(base + (int64_t)r0 * stride_tok);
    const int last = __builtin_amdgcn_readfirstlane(len - 1 - r0);
    uint4 v[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (u >= kSumUnroll && u % 4 == 0 && 4 * u > last) break;    // uniform: no row left
      int r = 4 * u + g;
      r = r < last ? r : last;     // a repeated row changes neither min nor max
      const unsigned byte_off = (__umul24((unsigned)r, ustride8) + (unsigned)c) * 16u;   // strides are multiples of 8
      v[u] = load16<STREAM_ROWS>(rb + byte_off);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (u >= kSumUnroll && u % 4 == 0 && 4 * u > last) break;
      float f[8];
      unpack8(v[u], f);
      if constexpr (MEAN) {
        const bool real = 4 * u + g <= last;         // a repeated row must not be added again
#pragma unroll
        for (int k = 0; k < 8; ++k) mn[k] += real ? f[k] : 0.0f;
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) { mn[k] = fminf(mn[k], f[k]); mx[k] = fmaxf(mx[k], f[k]); }
      }
    }
  }
  if constexpr (MEAN) {
    // fixed order: rows of a lane group in token order, then (g0 + g1) + (g2 + g3); the mean
    // rounded to nearest-even bf16 goes into both rows of the record
    const float inv_den = (float)len;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      mn[k] += shfl_xor_f(mn[k], 16);
      mn[k] += shfl_xor_f(mn[k], 32);
      mn[k] = bf16_round_rne(mn[k] / inv_den);
      mx[k] = mn[k];
    }
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      mn[k] = fminf(mn[k], shfl_xor_f(mn[k], 16)); mx[k] = fmaxf(mx[k], shfl_xor_f(mx[k], 16));
      mn[k] = fminf(mn[k], shfl_xor_f(mn[k], 32)); mx[k] = fmaxf(mx[k], shfl_xor_f(mx[k], 32));
    }
  }
  if (g == 0) {
    store16<STREAM>(reinterpret_cast<uint4*>(o) + c,
                    make_uint4(pack_bf16_exact(mn[0], mn[1]), pack_bf16_exact(mn[2], mn[3]),
                               pack_bf16_exact(mn[4], mn[5]), pack_bf16_exact(mn[6], mn[7])));
  } else if (g == 1) {
    store16<STREAM>(reinterpret_cast<uint4*>(o) + 16 + c,
                    make_uint4(pack_bf16_exact(mx[0], mx[1]), pack_bf16_exact(mx[2], mx[3]),
                               pack_bf16_exact(mx[4], mx[5]), pack_bf16_exact(mx[6], mx[7])));
  }
}

// The same where wavefronts are few and the latency of the rows is what counts.  LONG: up to 96 rows in flight, for blocks of more
// than kSumRowsAhead where chunks are of more than that and up to kSumLongTo.  (MEAN: a lane adds its rows in token order, whatever
// is in flight.)  Steps of an update of eight sequences, 8 heads, without / with it: chunks of 33 tokens 9.74 / 9.59 us, 40 9.58 /
// 9.42, 64 9.98 / 10.02; of 84 10.6 / 11.0, 120 10.97 / 11.4, one sequence 9.34 / 9.52 (11.8, 12.0 and 10.4 when every round
// handled 96 rows, whatever a block had left); where chunks are shorter the registers are only a burden.
constexpr int kSumRowsAhead = 4 * kSumUnroll;
constexpr int kSumLongTo = 64;
template <bool MEAN, bool LONG>
__device__ __forceinline__ void summarize_few(const uint16_t* base, int len, int64_t stride_tok, unsigned ustride8,
                                              uint16_t* o, int g, int c) {
  if (!LONG || len <= kSumRowsAhead) summarize_block<MEAN, false>(base, len, stride_tok, ustride8, o, g, c);
  else summarize_block<MEAN, false, false, 3 * kSumUnroll>(base, len, stride_tok, ustride8, o, g, c);
}

// A cache to summarise: K, and V in the same launch when its summaries are wanted.
struct SumTensor {
  const uint16_t* X;
  int64_t stride_tok, stride_head;
  uint16_t* out;
};

// One wavefront per (plane, block); the planes are the heads of K, then those of V, `heads` in all and the slower index,
// so that the wavefronts for which there is no block come last.  `streamed`: planes from the first one whose rows are
// read past the caches.  WAVES: wavefronts per SIMD that the compiler schedules for, 4 (96 or 104 registers) or 6 (80).  The
// upper bound holds it to the first: of its own accord it takes one schedule or the other with any change of the code, 67.7
// or 70.5 us for the pass over one sequence of 128K tokens, 285 or 295 for K and V of eight.
template <bool MEAN, int WAVES>
__attribute__((amdgpu_waves_per_eu(WAVES, WAVES == 4 ? 4 : 8)))
__global__ __launch_bounds__(kSumThreads) void summaries_kernel(
    SumTensor k, SumTensor v, int Hkv, int heads, int streamed, const int32_t* __restrict__ block_start,
    const int32_t* __restrict__ cu_blocks, int B, int cap, int out_rows, int total_tokens, int32_t* dev_status) {
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DSK_WAVE);   // wave-uniform: scalar registers
  const int g = lane >> 4;   // row group 0..3
  const int c = lane & 15;   // 16-byte column 0..15
  int nblk = cu_blocks[B];
  if (nblk > cap) nblk = cap;
  if (nblk <= 0) return;
  const int64_t items = (int64_t)heads * nblk;
  const uint32_t nwaves = gridDim.x * kSumWaves;
  int64_t item = (int64_t)blockIdx.x * kSumWaves + wave;
  if (item >= items) return;
  // plane and block: the first by a division, the next ones by adding the quotient and remainder of the step
  // (the grid has less than 2^32 wavefronts; the results are uniform, which the compiler does not see)
  const int step_h = __builtin_amdgcn_readfirstlane((int)(nwaves / (uint32_t)nblk));
  const int step_i = (int)(nwaves - (uint32_t)step_h * (uint32_t)nblk);
  int h = __builtin_amdgcn_readfirstlane((int)((uint32_t)item / (uint32_t)nblk));
  int i = (int)((uint32_t)item - (uint32_t)h * (uint32_t)nblk);
  int s = __builtin_amdgcn_readfirstlane(block_start[i]);
  int e = __builtin_amdgcn_readfirstlane(block_start[i + 1]);
  for (;;) {
    // the bounds of this wave's next block travel with the rows of the current one
    const int64_t nitem = item + nwaves;
    const bool more = nitem < items;
    int nh = h + step_h, ni = i + step_i;
    if (ni >= nblk) { ni -= nblk; ++nh; }
    const int pi = more ? ni : i;
    const int ns = __builtin_amdgcn_readfirstlane(block_start[pi]);
    const int ne = __builtin_amdgcn_readfirstlane(block_start[pi + 1]);
    const int len = e - s;
    const bool second = h >= Hkv;
    const int64_t stride_tok = second ? v.stride_tok : k.stride_tok;
    const int64_t th = second ? h - Hkv : h;
    uint16_t* o = (second ? v.out : k.out) + (th * out_rows + i) * (2 * DSK_HEAD_DIM);   // out_rows records per head (>= cap)
    if (s < 0 || len <= 0 || e > total_tokens) {   // malformed table: defined output, flag it
      if (lane < 32) reinterpret_cast<uint4*>(o)[lane] = make_uint4(0, 0, 0, 0);
      if (lane == 0) set_status(dev_status, DSK_ERR_SHAPE);
    } else {
      const uint16_t* base = (second ? v.X : k.X) + th * (second ? v.stride_head : k.stride_head) + (int64_t)s * stride_tok;   // uniform
      const unsigned ustride8 = (unsigned)stride_tok >> 3;
      if (h < streamed) summarize_block<MEAN, true, true>(base, len, stride_tok, ustride8, o, g, c);
      else summarize_block<MEAN, true>(base, len, stride_tok, ustride8, o, g, c);
    }
    if (!more) break;
    item = nitem; h = nh; i = ni; s = ns; e = ne;
  }
}

// K's planes, then V's, are read one after the other: of those that end well before the last 256 MB nothing is left in
// the memory-side cache at the end, so their rows are read past it.  K and V of eight sequences, 362K tokens, 8 heads
// (1.5 GB), pass / first decode step behind it: 316 / 56.0 us as two launches through the cache, 308 / 56.0 as one,
// 296 / 56.0 with all but the last 400 MB past it, 294 / 57.7 with all but the last 256 MB.
constexpr int64_t kSumKeptBytes = 400ll << 20;

// wavefronts for the blocks of chunks of C tokens (C is only a hint here: a call of this stage alone may leave it unset)
static int64_t expected_waves(const dsk_compress_args& a) {
  return a.C > 0 ? (a.vsum != nullptr ? 2 : 1) * (int64_t)a.Hkv * (a.total_tokens / a.C + a.B) : 0;
}

// Wavefronts per SIMD.  Short chunks leave most of a wavefront's 32 rows in flight empty, so they want 6 of them; long ones
// lose to the scheduling that the smaller register budget forces, except in launches of few rounds.  6 against 5, 32 heads at
// 126K tokens, chunks of 15: 210 against 218 us; 8 heads at 131K, chunks of 16: 73.2 / 76.3, of 18: 74.9 / 74.8, of 20: 75.1 /
// 73.3, of 30: 74.9 / 72.8.  Chunks of 18 to 50, by wavefronts, mean of 13 to 73 launches: up to 6 K 0.97, to 18 K 0.98, to
// 30 K 0.99, to 50 K 1.015, above 1.03 (8 heads at 18K tokens, chunks of 24: 9.3 / 10.2 us).
// Where sequences have a C of their own only the largest is known here, but the capacity of the tables follows the shortest
// chunk there may be, C - delta of some sequence: against that of the largest it tells how short the shortest C is, unless
// delta leaves chunks of every C nearly alike short; half of the sum of both stands for the mean.  Two sequences of 60K
// tokens, 8 heads, C of 14 and 28: 43.4 / 47.7, 18 and 34: 41.4 / 44.4, 24 and 24: 42.6 / 40.9.
static bool six_waves(const dsk_compress_args& a) {
  if (a.C <= 0) return false;
  if (a.C <= 17 || expected_waves(a) <= 30 * 1024) return true;
  if (a.C_per_seq == nullptr) return false;
  const int64_t min_chunk = a.C - a.delta;
  if (3 * min_chunk < a.C) return a.C <= 34;
  const int64_t shortest = (int64_t)a.C * a.total_tokens / (min_chunk * a.max_blocks_total);
  return shortest <= 18 && a.C + shortest <= 52;
}

template <bool MEAN, int WAVES>
static hipError_t launch_summaries_impl(const dsk_compress_args& a, hipStream_t st) {
  const int heads = (a.vsum != nullptr ? 2 : 1) * a.Hkv;
  const int64_t max_items = (int64_t)heads * a.max_blocks_total;
  if (max_items <= 0) return hipSuccess;
  int64_t wgs = (max_items + kSumWaves - 1) / kSumWaves;
  // A wavefront per block where there are many: workgroups dealt out as others end stay close together in
  // memory, while a persistent grid of 256 * 8 drifts apart (128K tokens, 8 heads: 79 -> 73 us for the pass
  // with the streamed records).  The capacity may be a multiple of the blocks there are, and an empty workgroup
  // is not free, so the grid is bounded by wavefronts for the blocks of chunks of C tokens (twice as many
  // where sequences have a C of their own, below this bound); where there are more, wavefronts take two or three.
  // With twice these grids, 128K tokens and K and V of eight sequences: 71.1 against 70.6 us, 289.4 against 288.8.
  int64_t max_wgs = (a.C_per_seq != nullptr ? 2 : 1) * expected_waves(a) / kSumWaves;
  if (max_wgs < 256 * 8) max_wgs = 256 * 8;
  const int64_t wgs_cap = WAVES > 4 ? 256 * 128 : 256 * 256;   // 32 heads, chunks of 15: 232 -> 218 us; eight sequences 293 -> 290
  if (max_wgs > wgs_cap) max_wgs = wgs_cap;
  if (wgs > max_wgs) wgs = max_wgs;
  const int out_rows = a.sum_stride_blocks > 0 ? a.sum_stride_blocks : a.max_blocks_total;
  const SumTensor k = {static_cast<const uint16_t*>(a.K), a.k_stride_tok, a.k_stride_head, static_cast<uint16_t*>(a.ksum)};
  const SumTensor v = {static_cast<const uint16_t*>(a.V), a.v_stride_tok, a.v_stride_head, static_cast<uint16_t*>(a.vsum)};
  const int64_t plane = (int64_t)a.total_tokens * DSK_HEAD_DIM * 2;
  const int64_t kept = plane > 0 ? (kSumKeptBytes + plane - 1) / plane : 0;
  const int streamed = heads > kept ? (int)(heads - kept) : 0;
  summaries_kernel<MEAN, WAVES><<<dim3((unsigned)wgs), dim3(kSumThreads), 0, st>>>(
      k, v, a.Hkv, heads, streamed, a.block_start, a.cu_blocks, a.B, a.max_blocks_total, out_rows, a.total_tokens, a.dev_status);
  return hipGetLastError();
}

hipError_t launch_summaries(const dsk_compress_args& a, hipStream_t st) {
  if (six_waves(a))
    return a.summary_mode == DSK_SUMMARY_MEAN ? launch_summaries_impl<true, 6>(a, st) : launch_summaries_impl<false, 6>(a, st);
  return a.summary_mode == DSK_SUMMARY_MEAN ? launch_summaries_impl<true, 4>(a, st) : launch_summaries_impl<false, 4>(a, st);
}

// Summaries of the blocks [blk_range[0], blk_range[1]) that an incremental update rewrote: few, so the chain of loads in front
// of the rows is what counts.  grid: (group of kSumWaves heads, block), so that nothing has to be divided.
template <bool MEAN, bool LONG>
__global__ __launch_bounds__(kSumThreads) void summaries_range_kernel(
    const uint16_t* __restrict__ X, int64_t stride_tok, int64_t stride_head, int Hkv,
    const int32_t* __restrict__ block_start, const int32_t* __restrict__ blk_range, int cap, int total_tokens,
    uint16_t* __restrict__ out, int32_t* dev_status) {
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DSK_WAVE);
  const int g = lane >> 4, c = lane & 15;
  const int h = (int)blockIdx.x * kSumWaves + wave;
  int lo = blk_range[0], hi = blk_range[1];
  if (hi > cap) hi = cap;
  if (lo < 0) lo = 0;
  if (h >= Hkv) return;
  for (int64_t b = (int64_t)lo + blockIdx.y; b < hi; b += gridDim.y) {
    const int i = (int)b;
    const int s = __builtin_amdgcn_readfirstlane(block_start[i]);
    const int e = __builtin_amdgcn_readfirstlane(block_start[i + 1]);
    const int len = e - s;
    uint16_t* o = out + ((int64_t)h * cap + i) * (2 * DSK_HEAD_DIM);
    if (s < 0 || len <= 0 || e > total_tokens) {   // malformed table: defined output, flag it
      if (lane < 32) reinterpret_cast<uint4*>(o)[lane] = make_uint4(0, 0, 0, 0);
      if (lane == 0) set_status(dev_status, DSK_ERR_SHAPE);
    } else {
      const uint16_t* base = X + (int64_t)h * stride_head + (int64_t)s * stride_tok;
      summarize_few<MEAN, LONG>(base, len, stride_tok, (unsigned)stride_tok >> 3, o, g, c);
    }
  }
}

hipError_t launch_summaries_range(const void* X, int64_t stride_tok, int64_t stride_head, int Hkv,
                                  const int32_t* block_start, const int32_t* blk_range, int max_blocks_in_range,
                                  int cap, int total_tokens, int chunk, int summary_mode, void* out, int32_t* dev_status,
                                  hipStream_t st) {
  if (Hkv <= 0 || max_blocks_in_range <= 0) return hipSuccess;
  const int groups = (Hkv + kSumWaves - 1) / kSumWaves;
  const int most = groups < 256 * 8 ? 256 * 8 / groups : 1;    // a long range: at most about 2048 workgroups
  const dim3 grid((unsigned)groups, (unsigned)(max_blocks_in_range < most ? max_blocks_in_range : most));
#define DSK_RANGE(mean, lng)                                                                                          \
  summaries_range_kernel<mean, lng><<<grid, dim3(kSumThreads), 0, st>>>(                                                  \
      static_cast<const uint16_t*>(X), stride_tok, stride_head, Hkv, block_start, blk_range, cap, total_tokens,           \
      static_cast<uint16_t*>(out), dev_status)
  const bool lng = chunk > kSumRowsAhead && chunk <= kSumLongTo;
  if (summary_mode == DSK_SUMMARY_MEAN) { if (lng) DSK_RANGE(true, true); else DSK_RANGE(true, false); }
  else if (lng) DSK_RANGE(false, true);
  else DSK_RANGE(false, false);
#undef DSK_RANGE
  return hipGetLastError();
}

// Summaries of the blocks a batched incremental update rewrote.  ranges[s] = {first rewritten
// entry, end, first K/V row of sequence s, its length}; block_start counts from the sequence's first
// token.  grid: (rewritten block, sequence, group of kSumWaves heads): one wavefront per head.
template <bool MEAN, bool LONG>
__global__ __launch_bounds__(kSumThreads) void summaries_batch_ranges_kernel(
    const uint16_t* __restrict__ X, int64_t stride_tok, int64_t stride_head, int Hkv,
    const int32_t* __restrict__ block_start, const int4* __restrict__ ranges, int out_rows,
    uint16_t* __restrict__ out, int32_t* dev_status) {
  const int lane = threadIdx.x & (DSK_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / DSK_WAVE);
  const int g = lane >> 4, c = lane & 15;
  const int4 rg = ranges[blockIdx.y];
  const int i = rg.x + (int)blockIdx.x;
  if (i >= rg.y || i >= out_rows) return;
  const int s = __builtin_amdgcn_readfirstlane(block_start[i]);
  const int e = __builtin_amdgcn_readfirstlane(block_start[i + 1]);
  const int len = e - s;
  const int h = (int)blockIdx.z * kSumWaves + wave;
  if (h < Hkv) {
    uint16_t* o = out + ((int64_t)h * out_rows + i) * (2 * DSK_HEAD_DIM);
    if (s < 0 || len <= 0 || e > rg.w) {           // malformed table: defined output, flag it
      if (lane < 32) reinterpret_cast<uint4*>(o)[lane] = make_uint4(0, 0, 0, 0);
      if (lane == 0) set_status(dev_status, DSK_ERR_SHAPE);
    } else {
      const uint16_t* base = X + (int64_t)h * stride_head + ((int64_t)rg.z + s) * stride_tok;
      summarize_few<MEAN, LONG>(base, len, stride_tok, (unsigned)stride_tok >> 3, o, g, c);
    }
  }
}

hipError_t launch_summaries_batch_ranges(const void* X, int64_t stride_tok, int64_t stride_head, int Hkv, int B,
                                         const int32_t* block_start, const void* ranges, int max_blocks_in_range,
                                         int out_rows, int chunk, int summary_mode, void* out, int32_t* dev_status,
                                         hipStream_t st) {
  if (max_blocks_in_range <= 0 || B <= 0) return hipSuccess;
  const dim3 grid((unsigned)max_blocks_in_range, (unsigned)B, (unsigned)((Hkv + kSumWaves - 1) / kSumWaves));
#define DSK_RANGES(mean, lng)                                                                                         \
  summaries_batch_ranges_kernel<mean, lng><<<grid, dim3(kSumThreads), 0, st>>>(                                           \
      static_cast<const uint16_t*>(X), stride_tok, stride_head, Hkv, block_start, static_cast<const int4*>(ranges),       \
      out_rows, static_cast<uint16_t*>(out), dev_status)
  const bool lng = chunk > kSumRowsAhead && chunk <= kSumLongTo;
  if (summary_mode == DSK_SUMMARY_MEAN) { if (lng) DSK_RANGES(true, true); else DSK_RANGES(true, false); }
  else if (lng) DSK_RANGES(false, true);
  else DSK_RANGES(false, false);
#undef DSK_RANGES
  return hipGetLastError();
}

}  // namespace dsk
