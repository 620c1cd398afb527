// Incremental update during decoding (Sec. 4.1): chunks whose end was decided on a complete
// search range are kept; DD-Select is re-run from the first open chunk over the grown
// sequence.  The open tail is a handful of chunks, so one wavefront walks it: per chunk the
// lanes score the positions of the search range (token id -> delimiter class -> integer score)
// and a wave-wide maximum of packed (score, smaller-e-wins) keys picks the boundary.  The
// summaries of the rewritten chunks are then recomputed by the summaries kernel on that range.
#include <type_traits>

#include "dsk_common.hpp"
#include "dsk_internal.hpp"

namespace dsk {

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
  for (int m = 1; m < DSK_WAVE; m <<= 1) {
    const unsigned long long o = __shfl_xor(v, m, DSK_WAVE);
    v = o > v ? o : v;
  }
  return v;
}

// Tokens around the end of a sequence that are fetched ahead and classified once
constexpr int kAppendWindow = 1024;

// The update of one sequence by one wavefront.  token_ids, block_start and slot_base point at the
// sequence's own first entry (its tables count from its first token); *n_blocks is its block count
// (in/out; nblk is its value, already fetched, like the delimiter id and the weight of class `lane`);
// range[0..1] receives the rewritten blocks as indices into the caller's table, i.e.
// offset by blk_base.  Returns false when the table was not the one described (nothing is changed).
//
// The update is a chain of memory latencies, so everything whose address is known goes out together: the
// caller's parameters, then here the last 64 entries of both tables and the tokens that the open chunks
// search (two round trips in front of the walk instead of seven: 5.3 -> 4.8 us for a token appended to each of
// eight sequences).
__device__ __forceinline__ bool append_segment_one(
    const int32_t* __restrict__ token_ids, int my_id, int my_weight, int n_class, int nblk, int len_old, int len_new,
    int C, int delta, int a_num, int a_den, int b, int cap, int32_t* __restrict__ block_start,
    int32_t* __restrict__ n_blocks, int32_t* __restrict__ slot_base, int blk_base, int32_t* __restrict__ range,
    int32_t* __restrict__ first_recomputed, int32_t* __restrict__ first_stale_slot, int32_t* dev_status) {
  __shared__ int32_t window[kAppendWindow];                 // token ids; from the first search on offered weights
  const int lane = threadIdx.x;
  if (nblk < 0) nblk = 0;
  if (nblk > cap) nblk = cap;
  // lane l: entry nblk - l of the tables
  const int back = nblk - lane > 0 ? nblk - lane : 0;
  const int bs = block_start[back], sb = slot_base[back], first = block_start[0];
  // an open chunk starts behind len_old - C - delta, so the boundaries it searches lie behind
  // len_old - 2 * delta
  const int w0 = len_old - 2 * delta > 0 ? len_old - 2 * delta : 0;
  const bool windowed = (int64_t)len_new - w0 <= kAppendWindow;
  const int n_win = windowed ? len_new - w0 : 0;
  for (int t0 = 0; t0 < n_win; t0 += 4 * DSK_WAVE) {
    int tok[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + r * DSK_WAVE + lane;
      tok[r] = token_ids[w0 + (t < n_win ? t : n_win - 1)];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + r * DSK_WAVE + lane;
      if (t < n_win) window[t] = tok[r];
    }
  }
  __syncthreads();
  // Token id -> weight of the delimiter, -1 = none, for every token of the window, several tokens a lane side by side.
  // Left until a chunk searches, since often none does: a token appended at C = 256, delta = 128 with 64 classes takes
  // 13.1 us with the rewinds of its table, 21.1 classified ahead; at C = 600, delta = 500, where several chunks
  // search the same tokens, 34.9 against 56.7 classified by every search.
  bool classified = false;
  auto classify_rows = [&](auto rows, int t0) {              // rows * 64 tokens side by side
    constexpr int kRows = decltype(rows)::value;
    int tok[kRows], w[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int t = t0 + r * DSK_WAVE + lane;
      tok[r] = window[t < n_win ? t : n_win - 1];
      w[r] = -1;
    }
    for (int c = n_class - 1; c >= 0; --c) {               // the lowest class index wins
      const int id = __builtin_amdgcn_readlane(my_id, c), wc = __builtin_amdgcn_readlane(my_weight, c);
#pragma unroll
      for (int r = 0; r < kRows; ++r) w[r] = tok[r] == id ? wc : w[r];
    }
    __syncthreads();                                       // lanes past the end read another one's entry
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int t = t0 + r * DSK_WAVE + lane;
      if (t < n_win) window[t] = w[r];
    }
  };
  auto classify = [&]() {
    int t0 = 0;
    for (; n_win - t0 > 2 * DSK_WAVE; t0 += 4 * DSK_WAVE) classify_rows(std::integral_constant<int, 4>{}, t0);
    if (n_win - t0 > DSK_WAVE) classify_rows(std::integral_constant<int, 2>{}, t0);
    else if (n_win > t0) classify_rows(std::integral_constant<int, 1>{}, t0);
    __syncthreads();
    classified = true;
  };

  const int table_end = __builtin_amdgcn_readlane(bs, 0);
  if (table_end != len_old || first != 0) {                // not the table this call was sized for
    if (lane == 0) {
      set_status(dev_status, DSK_ERR_SHAPE);
      range[0] = blk_base; range[1] = blk_base;
      if (first_recomputed) *first_recomputed = nblk;
      if (first_stale_slot) *first_stale_slot = 0;         // the table is not trusted: nothing is reusable
    }
    return false;
  }
  // open chunks form a suffix of the table: the last 63 are at hand, more are counted 64 at a time
  const unsigned long long last63 = __ballot(lane > 0 && nblk - lane >= 0 && bs + C + delta > len_old);
  int n_open = __popcll(last63);
  if (last63 == ~1ull) {
    for (int base = nblk - DSK_WAVE; base >= 0; base -= DSK_WAVE) {
      const int i = base - lane;
      const bool open = i >= 0 && block_start[i] + C + delta > len_old;
      const unsigned long long bal = __ballot(open);
      n_open += __popcll(bal);
      if (bal != ~0ull) break;                             // a final chunk was seen: all before it are final
    }
  }
  const int i0 = nblk - n_open;
  // start of the first open chunk (len_old when there is none) and its slot (then the slot total)
  int s_c = n_open < DSK_WAVE ? __shfl(bs, n_open, DSK_WAVE) : block_start[i0];
  int slot = n_open < DSK_WAVE ? __shfl(sb, n_open, DSK_WAVE) : slot_base[i0];
  const int stale_slot = slot;
  int i = i0;
  bool overflow = false;
  const int dd = delta > 1 ? delta : 1;
  while (s_c < len_new) {
    const int s_e = s_c + C;
    int e_star;
    if (s_e >= len_new) {
      e_star = len_new;
    } else {
      const int lo = s_e - delta;                          // > s_c because delta < C
      const int hi = s_e + delta < len_new ? s_e + delta : len_new;
      unsigned long long best = 0ull;                      // 0 = nothing offered
      if (windowed && !classified) classify();
      for (int e0 = lo; e0 <= hi; e0 += DSK_WAVE) {        // all lanes stay: the class ids are read across them
        const int e = e0 + lane;
        const bool in = e <= hi;
        int w = -1;                                        // the delimiter at e-1 offers the boundary e
        if (windowed) {
          if (in) w = window[e - 1 - w0];
        } else {
          const int tok = token_ids[(in ? e : hi) - 1];
          for (int c = n_class - 1; c >= 0; --c) {
            const int id = __builtin_amdgcn_readlane(my_id, c), wc = __builtin_amdgcn_readlane(my_weight, c);
            w = in && tok == id ? wc : w;
          }
        }
        if (w >= 0) {
          const int dist = e > s_e ? e - s_e : s_e - e;
          const int score = a_num * w * dd + (a_den - a_num) * 10 * (dd - dist);   // >= 0
          const unsigned long long key =
              ((unsigned long long)(unsigned)(score + 1) << 32) | (unsigned)(0x7FFFFFFF - e);   // ties: smaller e
          best = key > best ? key : best;
        }
      }
      best = wave_max_u64(best);
      e_star = best != 0ull ? 0x7FFFFFFF - (int)(unsigned)(best & 0xFFFFFFFFull) : s_e;
    }
    if (i >= cap) { overflow = true; break; }
    slot += (e_star - s_c + b - 1) / b;
    if (lane == 0) { block_start[i + 1] = e_star; slot_base[i + 1] = slot; }
    ++i;
    s_c = e_star;
  }
  if (lane == 0) {
    *n_blocks = i;
    range[0] = blk_base + i0;
    range[1] = blk_base + i;
    if (first_recomputed) *first_recomputed = i0;
    if (first_stale_slot) *first_stale_slot = stale_slot;
    if (overflow) set_status(dev_status, DSK_ERR_CAPACITY);
  }
  return true;
}


__global__ __launch_bounds__(DSK_WAVE) void append_segment_kernel(
    const int32_t* __restrict__ token_ids, const int32_t* __restrict__ delim_ids, int n_class,
    const uint8_t* __restrict__ class_weight_q, int len_old, int len_new, int C, int delta, int a_num,
    int a_den, int b, int cap, int32_t* __restrict__ block_start, int32_t* __restrict__ cu_blocks,
    int32_t* __restrict__ slot_base, int32_t* __restrict__ range, int32_t* __restrict__ first_recomputed,
    int32_t* __restrict__ first_stale_slot, int32_t* dev_status) {
  const int lane = threadIdx.x;
  const int my_id = delim_ids[lane < n_class ? lane : 0], my_weight = class_weight_q[lane < n_class ? lane : 0];
  append_segment_one(token_ids, my_id, my_weight, n_class, cu_blocks[1], len_old, len_new, C, delta, a_num, a_den, b,
                     cap, block_start, cu_blocks + 1, slot_base, 0, range, first_recomputed, first_stale_slot, dev_status);
}

// ---- all sequences of a batch, each in its own region of the tables ---------------------------
struct AppendBatchParams {
  const int32_t* seq_row0;
  int32_t* seq_len;
  const int32_t* len_new;
  const int32_t* token_ids;
  const int32_t* delim_ids;
  const uint8_t* class_weight_q;
  const int32_t* C_per_seq;
  const int32_t* delta_per_seq;
  const int32_t* cu_blocks;
  int32_t* blocks_used;
  int32_t* block_start;
  int32_t* slot_base;
  int32_t* first_recomputed;
  int32_t* first_stale_slot;
  int32_t* dev_status;
  int n_class, C, delta, a_num, a_den, b, total_rows, max_blocks_total, max_new_tokens;
};

// workspace: int4 per sequence = {first rewritten entry, end of the rewritten entries, first K/V row
// of the sequence, its new length}
__global__ __launch_bounds__(DSK_WAVE) void append_batch_segment_kernel(AppendBatchParams p, int4* __restrict__ ranges) {
  const int s = blockIdx.x;
  const int lane = threadIdx.x;
  const int row0 = p.seq_row0[s];
  const int len_old = p.seq_len[s];
  const int len_new = p.len_new != nullptr ? p.len_new[s] : len_old + p.max_new_tokens;
  const int blk0 = p.cu_blocks[s];
  const int region = p.cu_blocks[s + 1] - blk0;
  int C = p.C_per_seq ? p.C_per_seq[s] : p.C;
  int delta = p.delta_per_seq ? p.delta_per_seq[s] : p.delta;
  const int nblk = p.blocks_used[s];
  const int my_id = p.delim_ids[lane < p.n_class ? lane : 0];
  const int my_weight = p.class_weight_q[(int64_t)s * p.n_class + (lane < p.n_class ? lane : 0)];
  bool ok = row0 >= 0 && len_old >= 0 && len_new >= len_old && len_new - len_old <= p.max_new_tokens &&
            (int64_t)row0 + len_new <= p.total_rows && blk0 >= 0 && region >= 1 &&
            (int64_t)blk0 + region <= p.max_blocks_total;
  if (C < 1 || C > p.C || delta < 0 || delta >= C || delta > p.delta) {
    if (lane == 0) set_status(p.dev_status, DSK_ERR_PARAM);
    ok = false;
  } else if (!ok && lane == 0) {
    set_status(p.dev_status, DSK_ERR_SHAPE);
  }
  __shared__ int32_t range[2];
  if (!ok) {                                               // nothing of this sequence is touched
    if (lane == 0) {
      ranges[s] = make_int4(0, 0, 0, 0);
      if (p.first_recomputed) p.first_recomputed[s] = 0;
      if (p.first_stale_slot) p.first_stale_slot[s] = 0;
    }
    return;
  }
  const bool done = append_segment_one(p.token_ids + row0, my_id, my_weight, p.n_class, nblk, len_old, len_new, C, delta, p.a_num, p.a_den, p.b, region - 1, p.block_start + blk0, p.blocks_used + s,
                     p.slot_base + blk0, blk0, range, p.first_recomputed ? p.first_recomputed + s : nullptr,
                     p.first_stale_slot ? p.first_stale_slot + s : nullptr, p.dev_status);
  __syncthreads();
  if (lane == 0) {
    ranges[s] = make_int4(range[0], range[1], row0, len_new);
    if (done) p.seq_len[s] = len_new;
  }
}

hipError_t launch_append(const dsk_append_args& a, hipStream_t st) {
  int32_t* range = static_cast<int32_t*>(a.workspace);
  append_segment_kernel<<<dim3(1), dim3(DSK_WAVE), 0, st>>>(
      a.token_ids, a.delim_ids, a.n_class, a.class_weight_q, a.len_old, a.len_new, a.C, a.delta, a.alpha_num,
      a.alpha_den, a.b, a.max_blocks_total, a.block_start, a.cu_blocks, a.slot_base, range, a.first_recomputed,
      a.first_stale_slot, a.dev_status);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  // chunks that can be rewritten: the open ones start after len_old - C - delta, and every chunk
  // but the last has at least C - delta tokens
  const int64_t span = (int64_t)(a.len_new - a.len_old) + a.C + a.delta;
  int64_t max_changed = span / (a.C - a.delta) + 2;
  if (max_changed > a.max_blocks_total) max_changed = a.max_blocks_total;
  err = launch_summaries_range(a.K, a.k_stride_tok, a.k_stride_head, a.Hkv, a.block_start, range, (int)max_changed,
                               a.max_blocks_total, a.len_new, a.C, a.summary_mode, a.ksum, a.dev_status, st);
  if (err != hipSuccess || a.vsum == nullptr) return err;
  return launch_summaries_range(a.V, a.v_stride_tok, a.v_stride_head, a.Hkv, a.block_start, range, (int)max_changed,
                                a.max_blocks_total, a.len_new, a.C, a.summary_mode, a.vsum, a.dev_status, st);
}

hipError_t launch_append_batch(const dsk_append_batch_args& a, hipStream_t st) {
  AppendBatchParams p;
  p.seq_row0 = a.seq_row0; p.seq_len = a.seq_len; p.len_new = a.len_new;
  p.token_ids = a.token_ids; p.delim_ids = a.delim_ids; p.class_weight_q = a.class_weight_q;
  p.C_per_seq = a.C_per_seq; p.delta_per_seq = a.delta_per_seq;
  p.cu_blocks = a.cu_blocks; p.blocks_used = a.blocks_used;
  p.block_start = a.block_start; p.slot_base = a.slot_base;
  p.first_recomputed = a.first_recomputed; p.first_stale_slot = a.first_stale_slot;
  p.dev_status = a.dev_status;
  p.n_class = a.n_class; p.C = a.C; p.delta = a.delta; p.a_num = a.alpha_num; p.a_den = a.alpha_den; p.b = a.b;
  p.total_rows = a.total_rows; p.max_blocks_total = a.max_blocks_total; p.max_new_tokens = a.max_new_tokens;
  int4* ranges = static_cast<int4*>(a.workspace);
  append_batch_segment_kernel<<<dim3((unsigned)a.B), dim3(DSK_WAVE), 0, st>>>(p, ranges);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  // chunks of one sequence that can be rewritten: the open ones start after len_old - C - delta,
  // and every chunk but the last has at least one token (C - delta of the sequence's own values,
  // which the host does not know when they are per sequence)
  const int min_len = (a.C_per_seq || a.delta_per_seq) ? 1 : a.C - a.delta;
  const int64_t span = (int64_t)a.max_new_tokens + a.C + a.delta;
  int64_t max_changed = span / min_len + 2;
  if (max_changed > a.max_blocks_total) max_changed = a.max_blocks_total;
  err = launch_summaries_batch_ranges(a.K, a.k_stride_tok, a.k_stride_head, a.Hkv, a.B, a.block_start, ranges,
                                      (int)max_changed, a.max_blocks_total, a.C, a.summary_mode, a.ksum, a.dev_status, st);
  if (err != hipSuccess || a.vsum == nullptr) return err;
  return launch_summaries_batch_ranges(a.V, a.v_stride_tok, a.v_stride_head, a.Hkv, a.B, a.block_start, ranges,
                                       (int)max_changed, a.max_blocks_total, a.C, a.summary_mode, a.vsum, a.dev_status, st);
}

}  // namespace dsk
