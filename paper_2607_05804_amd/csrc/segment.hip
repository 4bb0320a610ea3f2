// Segment table, validation and token weights.
//
// A segment is a maximal run of consecutive tokens with equal (trajectory id,
// turn id): turn t of a trace is its observation o_t followed by the response
// r_t (Sec. 3), and the segment's supervised count is the paper's n_t for
// that trajectory (Sec. 4.4).  The per-token weights follow the progressive
// turn-normalised blend of Sec. 5.2 / App. D Algorithm 1 expanded per token:
//   w_i = m_i / B * ((1 - alpha) / N_b + alpha / (T_b * n_bt)).
//
// Kernels, in launch order (all integer work is exact, so the table is unique;
// small batches run seg_one instead of all of them):
//   seg_count   per 1024-token tile: segment starts and the earliest id/mask
//               error of the tile; clears the per-segment counters; the first
//               workgroup resets the workspace header.
//   seg_offsets (batches of more than kFusedScanTiles tiles only) one
//               workgroup: exclusive scan of the tile counts, error key and
//               segment count of the whole batch.
//   seg_write   per tile: its first segment index (the sum of the earlier
//               tiles' counts, summed by every workgroup itself up to
//               kFusedScanTiles tiles), segment index of every token, segment
//               start / turn / trajectory / end, supervised counts (summed
//               per segment in LDS, one global atomic per tile and segment);
//               the first workgroup writes the batch's error key and segment
//               count.
//   seg_link    per segment: ordering check against the previous segment,
//               outcome-flag check against the trajectory's first segment,
//               segment length, trajectory head segment, T_b, N_b and B (the
//               segments of a wave summed per trajectory before the atomics),
//               the batch's supervised-token count, and the survivors n_t of
//               the turn-support floor.
//   seg_valid   (turn-support floor only) per segment: T_vb, the valid
//               supervised turns of each trajectory (n_t >= n_min).
//   token_weights per token: w_i and grad_scale * w_i, clears this call's
//               per-token KL and the row kernel's exchange slots.
//
// With the floor (App. D's internal-blend n_min = max(min_floor,
// ceil(min_frac * B)); the turn term covers only valid turns) the weight is
//   w_i = m_i / B * ((1 - alpha) / N_b + alpha * u_bt),
//   u_bt = [n_t >= n_min] / (T_vb * n_bt) if T_vb > 0, else 1 / N_b.

#include "block_ops.h"
#include "turnkl_internal.h"

namespace turnkl {
namespace {

struct TokenInfo {
  bool pad;
  bool start;
  unsigned long long err;
};

__device__ inline TokenInfo inspect(const SegParams& p, long long i) {
  TokenInfo r{true, false, kNoError};
  const int b = p.traj[i];
  const int t = p.turn[i];
  if (b < 0) {
    if (p.mask[i]) r.err = err_key(i, kPrioPadMask);
    return r;
  }
  r.pad = false;
  if (t < 0 || t >= p.max_turns) r.err = err_key(i, kPrioTurnRange);
  r.start = (i == 0) || p.traj[i - 1] != b || p.turn[i - 1] != t;
  // inside a segment the outcome flag must not change (segment starts are
  // checked against the trajectory's first segment in seg_link)
  if (p.success && !r.start && r.err == kNoError &&
      ((p.success[i] != 0) != (p.success[i - 1] != 0)))
    r.err = err_key(i, kPrioOutcome);
  return r;
}

__global__ __launch_bounds__(kSegThreads) void seg_count(SegParams p, Ws ws, int n_surv) {
  __shared__ int s_cnt[kSegThreads / kWave];
  __shared__ unsigned long long s_err[kSegThreads / kWave];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    volatile Header* h = ws.hdr;
    h->err_key = kNoError;
    h->ticket = 0u;
    h->n_seg = 0;
    h->b_eff = 0;
    h->n_sup = 0;
  }
  for (int t = blockIdx.x * kSegThreads + threadIdx.x; t < n_surv; t += gridDim.x * kSegThreads)
    ws.turn_surv[t] = 0;
  const long long base = (long long)blockIdx.x * kSegTile + (long long)threadIdx.x * kSegTokensPerThread;
  int cnt = 0;
  unsigned long long err = kNoError;
  for (int j = 0; j < kSegTokensPerThread; ++j) {
    const long long i = base + j;
    if (i >= p.n) break;
    const TokenInfo ti = inspect(p, i);
    cnt += ti.start ? 1 : 0;
    err = ti.err < err ? ti.err : err;
    ws.seg_nsup[i] = 0;
    ws.traj_T[i] = 0;
    ws.traj_N[i] = 0;
    ws.traj_Tv[i] = 0;
  }
  cnt = wave_sum(cnt);
  err = wave_min_u64(err);
  const int wid = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    s_cnt[wid] = cnt;
    s_err[wid] = err;
  }
  __syncthreads();
  if (threadIdx.x == 0 && (long long)blockIdx.x * kSegTile < p.n) {
    int c = 0;
    unsigned long long e = kNoError;
    for (int w = 0; w < kSegThreads / kWave; ++w) {
      c += s_cnt[w];
      e = s_err[w] < e ? s_err[w] : e;
    }
    ws.blk_cnt[blockIdx.x] = c;
    ws.blk_err[blockIdx.x] = e;
  }
}

constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void seg_offsets(Ws ws, long long nblk) {
  __shared__ int s_scan[kScanThreads / kWave];
  __shared__ unsigned long long s_err[kScanThreads / kWave];
  int carry = 0;
  unsigned long long err = kNoError;
  for (long long b0 = 0; b0 < nblk; b0 += kScanThreads) {
    const long long b = b0 + threadIdx.x;
    const int v = b < nblk ? ws.blk_cnt[b] : 0;
    if (b < nblk) err = ws.blk_err[b] < err ? ws.blk_err[b] : err;
    int total;
    const int ex = block_exclusive_scan<kScanThreads>(v, s_scan, &total);
    if (b < nblk) ws.blk_off[b] = carry + ex;
    carry += total;
  }
  err = wave_min_u64(err);
  if ((threadIdx.x & (kWave - 1)) == 0) s_err[threadIdx.x / kWave] = err;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long e = kNoError;
    for (int w = 0; w < kScanThreads / kWave; ++w) e = s_err[w] < e ? s_err[w] : e;
    volatile Header* h = ws.hdr;
    h->err_key = e;
    h->n_seg = carry;
  }
  drain_stores();
}

// The number of tiles up to which every seg_write workgroup sums the earlier
// tiles' segment counts itself (at most 8 loads per thread), which saves the
// separate scan kernel; larger batches run seg_offsets first.
constexpr long long kFusedScanTiles = 2048;

template <bool kFusedScan>
__global__ __launch_bounds__(kSegThreads) void seg_write(SegParams p, Ws ws, long long nblk) {
  __shared__ int s_scan[kSegThreads / kWave];
  __shared__ unsigned long long s_err[kSegThreads / kWave];
  __shared__ int s_nsup[kSegTile + 1];  // supervised tokens per segment of this tile
  const long long base = (long long)blockIdx.x * kSegTile + (long long)threadIdx.x * kSegTokensPerThread;
  int first;  // segment index of this tile's tokens before its first segment start
  if (kFusedScan) {
    // the earlier tiles' counts, summed in a fixed order (integers: exact);
    // the first workgroup also takes the batch's totals
    const long long upto = blockIdx.x == 0 ? nblk : (long long)blockIdx.x;
    int c = 0, before = 0;
    unsigned long long e = kNoError;
    for (long long b = threadIdx.x; b < upto; b += kSegThreads) {
      const int v = ws.blk_cnt[b];
      c += v;
      before += b < (long long)blockIdx.x ? v : 0;
      if (blockIdx.x == 0) e = ws.blk_err[b] < e ? ws.blk_err[b] : e;
    }
    before = block_sum<kSegThreads>(before, s_scan);
    if (blockIdx.x == 0) {
      c = block_sum<kSegThreads>(c, s_scan);
      e = wave_min_u64(e);
      if ((threadIdx.x & (kWave - 1)) == 0) s_err[threadIdx.x / kWave] = e;
      __syncthreads();
      if (threadIdx.x == 0) {
        for (int w = 0; w < kSegThreads / kWave; ++w) e = s_err[w] < e ? s_err[w] : e;
        volatile Header* h = ws.hdr;
        h->err_key = e;
        h->n_seg = c;
      }
    }
    first = before - 1;
  } else {
    first = ws.blk_off[blockIdx.x] - 1;
  }
  for (int k = threadIdx.x; k <= kSegTile; k += kSegThreads) s_nsup[k] = 0;
  TokenInfo ti[kSegTokensPerThread];
  int cnt = 0;
  for (int j = 0; j < kSegTokensPerThread; ++j) {
    const long long i = base + j;
    ti[j] = TokenInfo{true, false, kNoError};
    if (i < p.n) ti[j] = inspect(p, i);
    cnt += ti[j].start ? 1 : 0;
  }
  int total;
  int seg = first + block_exclusive_scan<kSegThreads>(cnt, s_scan, &total);
  // this thread's supervised tokens, counted per segment before the LDS add
  int run_seg = -1, run_n = 0;
  for (int j = 0; j < kSegTokensPerThread; ++j) {
    const long long i = base + j;
    if (i >= p.n) break;
    if (ti[j].pad) {
      ws.tok_seg[i] = -1;
      continue;
    }
    if (ti[j].start) {
      ++seg;
      ws.seg_start[seg] = (int)i;
      ws.seg_traj[seg] = p.traj[i];
      ws.seg_turn[seg] = p.turn[i];
    }
    ws.tok_seg[i] = seg;
    const bool last = (i + 1 == p.n) || p.traj[i + 1] != p.traj[i] || p.turn[i + 1] != p.turn[i];
    if (last) ws.seg_len[seg] = (int)(i + 1);  // segment end; seg_link turns it into a length
    if (p.mask[i]) {
      if (seg != run_seg) {
        if (run_n) atomicAdd(&s_nsup[run_seg - first], run_n);
        run_seg = seg;
        run_n = 0;
      }
      ++run_n;
    }
  }
  if (run_n) atomicAdd(&s_nsup[run_seg - first], run_n);
  __syncthreads();
  for (int k = threadIdx.x; k <= total; k += kSegThreads)
    if (const int n = s_nsup[k]) atomicAdd(&ws.seg_nsup[first + k], n);
}

// For each head among the wave's segments with n > 0: add(head, how many
// segments, their sum of n), in one lane.
template <typename Add>
__device__ inline void wave_by_head(int head, int n, Add add) {
  const int lane = threadIdx.x & (kWave - 1);
  unsigned long long todo = __ballot(n > 0);
  while (todo) {
    const int leader = __builtin_ctzll(todo);
    const int h = __shfl(head, leader, kWave);
    const unsigned long long same = __ballot(n > 0 && head == h);
    const int sum_n = wave_sum((same >> lane) & 1ull ? n : 0);
    if (lane == leader) add(h, __popcll(same), sum_n);
    todo &= ~same;
  }
}

__global__ __launch_bounds__(kSegThreads) void seg_link(SegParams p, Ws ws) {
  __shared__ int s_red[kSegThreads / kWave];
  const int n_seg = ws.hdr->n_seg;
  int sup_total = 0;
  // every lane of a wave runs the same iterations (the per-trajectory sums
  // below are wave-wide)
  for (int s0 = blockIdx.x * kSegThreads; s0 < n_seg; s0 += gridDim.x * kSegThreads) {
    const int s = s0 + (int)threadIdx.x;
    int head = -1, n = 0;
    if (s < n_seg) {
      const int b = ws.seg_traj[s];
      const int t = ws.seg_turn[s];
      const int start = ws.seg_start[s];
      if (s > 0) {
        const int pb = ws.seg_traj[s - 1];
        const int pt = ws.seg_turn[s - 1];
        if (b < pb || (b == pb && t <= pt)) atomicMin(&ws.hdr->err_key, err_key(start, kPrioUnsorted));
      }
      ws.seg_len[s] = ws.seg_len[s] - start;
      // first segment of this trajectory (ids are sorted when the batch is valid)
      int lo = 0, hi = s;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ws.seg_traj[mid] < b) lo = mid + 1; else hi = mid;
      }
      head = lo;
      ws.seg_head[s] = head;
      // On a sorted prefix `head` is the trajectory's first segment; otherwise
      // an ordering error at or before this segment's start outranks this one.
      if (p.success && head != s && (p.success[start] != 0) != (p.success[ws.seg_start[head]] != 0))
        atomicMin(&ws.hdr->err_key, err_key(start, kPrioOutcome));
      n = ws.seg_nsup[s];
      if (n > 0 && p.floor_on && t >= 0 && t < p.max_turns) atomicAdd(&ws.turn_surv[t], 1);
    }
    sup_total += n;
    // T_b and N_b: the wave's supervised segments summed per trajectory head,
    // one atomic pair per head; the add that lifts N_b from zero counts the
    // trajectory in B
    wave_by_head(head, n, [&](int h, int n_turns, int sum_n) {
      atomicAdd(&ws.traj_T[h], n_turns);
      if (atomicAdd(&ws.traj_N[h], sum_n) == 0) atomicAdd(&ws.hdr->b_eff, 1);
    });
  }
  sup_total = block_sum<kSegThreads>(sup_total, s_red);
  if (threadIdx.x == 0 && sup_total) atomicAdd(&ws.hdr->n_sup, sup_total);
}

__global__ __launch_bounds__(kSegThreads) void seg_valid(SegParams p, Ws ws) {
  if (ws.hdr->err_key != kNoError) return;
  const int n_seg = ws.hdr->n_seg;
  const int n_min = support_n_min(p, ws.hdr->b_eff);
  for (int s = blockIdx.x * kSegThreads + threadIdx.x; s < n_seg; s += gridDim.x * kSegThreads) {
    if (ws.seg_nsup[s] > 0 && ws.turn_surv[ws.seg_turn[s]] >= n_min)
      atomicAdd(&ws.traj_Tv[ws.seg_head[s]], 1);
  }
}

__global__ __launch_bounds__(kSegThreads) void token_weights(SegParams p, Ws ws, double alpha,
                                                             float grad_scale, int slot_words,
                                                             float* kl) {
  if (ws.hdr->err_key != kNoError) return;
  const double inv_b = ws.hdr->b_eff > 0 ? 1.0 / (double)ws.hdr->b_eff : 0.0;
  const int n_min = p.floor_on ? support_n_min(p, ws.hdr->b_eff) : 0;
  for (long long i = (long long)blockIdx.x * kSegThreads + threadIdx.x; i < p.n;
       i += (long long)gridDim.x * kSegThreads) {
    kl[i] = 0.0f;
    if (!p.mask[i]) {
      ws.w[i] = 0.0f;
      ws.wsc[i] = 0.0f;
      continue;
    }
    const int s = ws.tok_seg[i];
    const int h = ws.seg_head[s];
    const double n_bt = (double)ws.seg_nsup[s];
    const double n_b = (double)ws.traj_N[h];
    const TurnTerm u = turn_term(p, ws, s, h, n_min);
    const double w = inv_b * ((1.0 - alpha) / n_b + turn_part(alpha, u, n_bt, n_b));
    ws.w[i] = (float)w;
    ws.wsc[i] = (float)(w * (double)grad_scale);
    if (slot_words) {
      unsigned long long* sl = ws.slots + i * (long long)slot_words;
      for (int q = 0; q < slot_words; ++q) sl[q] = 0ull;
      drain_stores();
    }
  }
}

// ---------------------------------------------------------------------------
// Batches of at most kOneThreads * kOneMax tokens: all of the above in one
// kernel.  One workgroup holds the whole table in LDS (as many segments as
// tokens, 18 bytes each), the others clear the exchange slots and the per-token
// KL.  The four or five kernels above take 5 to 8 us each, nearly all of it
// launch and memory latency; this one takes 8 to 12, and 26 to 32 for the
// largest tables.  Whole calls, tiled kernels -> this one: 160 tokens of 1,024
// fp32 logits 35.8 -> 23.1 us; top-K with turns of 41 to 100 tokens, 1,000
// tokens 35.6 -> 24.2, 8,192 tokens 42.6 -> 32.6; 8,192 turns of one token, as
// many trajectories 169 -> 75 (1,024 bf16 logits), 205 trajectories 79 -> 84,
// the one layout found that loses.  At 16,384 tokens one workgroup no longer
// beats the tiled kernels (56.5 against 55.9 us).

constexpr int kOneThreads = 1024;
constexpr int kOneMax = 8;       // tokens per thread: 144 KiB of LDS
constexpr int kOneTurns = 2048;  // turn indices under a support floor

// One entry per segment; the trajectory sums are at its first segment.  Token
// indices, lengths and counts are at most 8,192: 16 bits each.  The weights (as
// bits) take the place of traj and turn, which are copied out by then.
template <int kMax>
struct SegTable {
  static constexpr int kSegs = kOneThreads * kMax;
  int traj[kSegs], turn[kSegs];
  unsigned sums[kSegs];       // T_b << 16 | N_b; under a floor then T_vb << 16 | N_b
  unsigned nsup2[kSegs / 2];  // supervised tokens, two segments to a word
  unsigned short start[kSegs], head[kSegs];

  __device__ int nsup(int s) const { return (nsup2[s >> 1] >> (16 * (s & 1))) & 0xFFFFu; }
};

// A thread's tokens r * kOneThreads + threadIdx.x, r < rounds: their ids, and bit
// r says whether the token starts a segment, is the last of one, is supervised,
// is padding (or beyond the batch).
template <int kMax>
struct OwnTokens {
  int traj[kMax], turn[kMax];
  unsigned start, last, sup, pad;
};

// an add that only this workgroup needs to see before the kernel ends
template <typename T>
__device__ inline void add_here(T* x, T n) {
  __hip_atomic_fetch_add(x, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ inline bool bit(unsigned m, int j) { return (m >> j) & 1u; }

// Everything after the segment count.  before[r * waves + w]: segments that
// start before the tokens of wave w in round r.
template <int kMax>
__device__ __forceinline__ void one_table(const SegParams& p, const Ws& ws, SegTable<kMax>& t, int* s_surv,
                                          const int* before, int n_seg, const OwnTokens<kMax>& own, int rounds,
                                          unsigned long long err, double alpha, float grad_scale) {
  constexpr int kWaves = kOneThreads / kWave;
  __shared__ unsigned long long s_err[kWaves];
  __shared__ int s_b[kWaves], s_n[kWaves];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  for (int s = tid; s < n_seg; s += kOneThreads) {
    t.sums[s] = 0u;
    t.nsup2[s >> 1] = 0u;
  }
  if (p.floor_on)
    for (int k = tid; k < p.max_turns; k += kOneThreads) s_surv[k] = 0;
  __syncthreads();
  int seg[kMax];
#pragma unroll
  for (int r = 0; r < kMax; ++r) {
    if (r >= rounds) continue;
    const int i = r * kOneThreads + tid;
    const bool start = bit(own.start, r), pad = bit(own.pad, r);
    const unsigned long long starts = __ballot(start);
    const unsigned long long cuts = __ballot(start || pad);
    const unsigned long long sup = __ballot(bit(own.sup, r));
    const unsigned long long upto = ~0ull >> (kWave - 1 - lane);  // lanes 0 .. lane
    seg[r] = before[r * kWaves + tid / kWave] + __popcll(starts & upto) - 1;
    if (start) {
      t.start[seg[r]] = (unsigned short)i;
      t.traj[seg[r]] = own.traj[r];
      t.turn[seg[r]] = own.turn[r];
    }
    if (bit(own.last, r)) t.head[seg[r]] = (unsigned short)i;  // the last token, for the length below
    // the first lane of each run of one segment adds the run's supervised tokens
    const unsigned long long after = cuts & ~upto;
    const unsigned long long run = (after ? (after & -after) - 1ull : ~0ull) & ~(upto >> 1);
    const unsigned n = (unsigned)__popcll(sup & run);
    if (!pad && (start || lane == 0) && n) add_here(&t.nsup2[seg[r] >> 1], n << (16 * (seg[r] & 1)));
  }
  __syncthreads();
  int n_sup = 0;
  for (int s = tid; s < n_seg; s += kOneThreads) {
    const int b = t.traj[s];
    const int turn = t.turn[s];
    const int start = t.start[s];
    ws.seg_len[s] = t.head[s] + 1 - start;
    if (s > 0) {
      const int pb = t.traj[s - 1];
      const int pt = t.turn[s - 1];
      if (b < pb || (b == pb && turn <= pt)) {
        const unsigned long long e = err_key(start, kPrioUnsorted);
        err = e < err ? e : err;
      }
    }
    int lo = 0, hi = s;  // first segment of this trajectory, as in seg_link
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (t.traj[mid] < b) lo = mid + 1; else hi = mid;
    }
    t.head[s] = (unsigned short)lo;
    if (p.success && lo != s && (p.success[start] != 0) != (p.success[t.start[lo]] != 0)) {
      const unsigned long long e = err_key(start, kPrioOutcome);
      err = e < err ? e : err;
    }
    const int n = t.nsup(s);
    n_sup += n;
    if (n > 0) {
      add_here(&t.sums[lo], 0x10000u + (unsigned)n);
      if (p.floor_on && turn >= 0 && turn < p.max_turns) add_here(&s_surv[turn], 1);
    }
  }
  __syncthreads();
  int b_eff = 0;
  for (int s = tid; s < n_seg; s += kOneThreads) b_eff += t.sums[s] ? 1 : 0;
  b_eff = wave_sum(b_eff);
  n_sup = wave_sum(n_sup);
  err = wave_min_u64(err);
  if ((tid & (kWave - 1)) == 0) {
    s_b[tid / kWave] = b_eff;
    s_n[tid / kWave] = n_sup;
    s_err[tid / kWave] = err;
  }
  __syncthreads();
  b_eff = 0;
  n_sup = 0;
  err = kNoError;
  for (int w = 0; w < kWaves; ++w) {
    b_eff += s_b[w];
    n_sup += s_n[w];
    err = s_err[w] < err ? s_err[w] : err;
  }
  if (tid == 0) {
    volatile Header* h = ws.hdr;
    h->err_key = err;
    h->ticket = 0u;
    h->n_seg = n_seg;
    h->b_eff = b_eff;
    h->n_sup = n_sup;
  }
  const int n_min = p.floor_on ? support_n_min(p, b_eff) : 0;
  if (p.floor_on) {
    for (int k = tid; k < p.max_turns; k += kOneThreads) ws.turn_surv[k] = s_surv[k];
    for (int s = tid; s < n_seg; s += kOneThreads) {
      ws.traj_T[s] = (int)(t.sums[s] >> 16);
      t.sums[s] &= 0xFFFFu;
    }
    __syncthreads();
    for (int s = tid; s < n_seg && err == kNoError; s += kOneThreads)
      if (t.nsup(s) > 0 && s_surv[t.turn[s]] >= n_min) add_here(&t.sums[t.head[s]], 0x10000u);
    __syncthreads();
  }
  int* const turns = p.floor_on ? ws.traj_Tv : ws.traj_T;
  const double inv_b = b_eff > 0 ? 1.0 / (double)b_eff : 0.0;
  for (int s = tid; s < n_seg; s += kOneThreads) {
    const int h = t.head[s];
    const int n = t.nsup(s);
    const unsigned own_sums = t.sums[s];
    ws.seg_start[s] = t.start[s];
    ws.seg_traj[s] = t.traj[s];
    ws.seg_turn[s] = t.turn[s];
    ws.seg_nsup[s] = n;
    ws.seg_head[s] = h;
    turns[s] = (int)(own_sums >> 16);
    ws.traj_N[s] = (int)(own_sums & 0xFFFFu);
    float w = 0.0f, wsc = 0.0f;
    if (n > 0 && err == kNoError) {
      const unsigned sums = t.sums[h];
      const double n_b = (double)(sums & 0xFFFFu);
      const TurnTerm u{(double)(sums >> 16), !p.floor_on || s_surv[t.turn[s]] >= n_min};
      const double x = inv_b * ((1.0 - alpha) / n_b + turn_part(alpha, u, (double)n, n_b));
      w = (float)x;
      wsc = (float)(x * (double)grad_scale);
    }
    t.traj[s] = __float_as_int(w);
    t.turn[s] = __float_as_int(wsc);
  }
  if (err != kNoError) return;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kMax; ++r) {
    const int i = r * kOneThreads + tid;
    if (i >= (int)p.n) continue;
    const bool m = bit(own.sup, r);
    ws.w[i] = m ? __int_as_float(t.traj[seg[r]]) : 0.0f;
    ws.wsc[i] = m ? __int_as_float(t.turn[seg[r]]) : 0.0f;
  }
}

template <int kMax>
__global__ __launch_bounds__(kOneThreads) void seg_one(SegParams p, Ws ws, double alpha, float grad_scale,
                                                       int slot_words, float* kl, int rounds) {
  const int tid = threadIdx.x;
  const int n = (int)p.n;
  if (blockIdx.x > 0) {
    const long long at = (long long)(blockIdx.x - 1) * kOneThreads + tid;
    const long long step = (long long)(gridDim.x - 1) * kOneThreads;
    for (long long q = at; q < (long long)n * slot_words; q += step) ws.slots[q] = 0ull;
    for (long long q = at; q < n; q += step) kl[q] = 0.0f;
    return;
  }
  __shared__ SegTable<kMax> s_table;
  __shared__ int s_surv[kOneTurns];
  __shared__ int s_scan[kOneThreads / kWave];
  constexpr int kWaves = kOneThreads / kWave;
  __shared__ int s_before[kMax * kWaves];
  // the tokens and both neighbours, every load before the first use
  OwnTokens<kMax> own;
  own.start = own.last = own.sup = own.pad = 0u;
  const int lane = tid & (kWave - 1);
  int eb[kMax], et[kMax];  // lane 0: of the token before, lane 63: of the token after
  unsigned char m[kMax];
#pragma unroll
  for (int r = 0; r < kMax; ++r) {
    const int i = r * kOneThreads + tid;
    const int e = lane == 0 ? i - 1 : i + 1;
    const bool in = r < rounds && i < n;
    const bool edge = r < rounds && (lane == 0 || lane == kWave - 1) && e >= 0 && e < n;
    own.traj[r] = in ? p.traj[i] : -1;
    own.turn[r] = in ? p.turn[i] : 0;
    m[r] = in ? p.mask[i] : 0;
    eb[r] = edge ? p.traj[e] : -1;
    et[r] = edge ? p.turn[e] : 0;
  }
  unsigned long long err = kNoError;
#pragma unroll
  for (int r = 0; r < kMax; ++r) {
    const int i = r * kOneThreads + tid;
    const int b = own.traj[r], t = own.turn[r];
    const int ub = __shfl_up(b, 1, kWave), ut = __shfl_up(t, 1, kWave);
    const int db = __shfl_down(b, 1, kWave), dt = __shfl_down(t, 1, kWave);
    const int pb = lane == 0 ? eb[r] : ub, pt = lane == 0 ? et[r] : ut;
    const int nb = lane == kWave - 1 ? eb[r] : db, nt = lane == kWave - 1 ? et[r] : dt;
    unsigned long long e = kNoError;
    bool start = false;
    if (b < 0) {
      if (m[r]) e = err_key(i, kPrioPadMask);
      own.pad |= 1u << r;
    } else {
      if (t < 0 || t >= p.max_turns) e = err_key(i, kPrioTurnRange);
      start = i == 0 || pb != b || pt != t;
      const bool last = i + 1 == n || nb != b || nt != t;
      if (p.success && !start && e == kNoError && ((p.success[i] != 0) != (p.success[i - 1] != 0)))
        e = err_key(i, kPrioOutcome);
      own.start |= (start ? 1u : 0u) << r;
      own.last |= (last ? 1u : 0u) << r;
      own.sup |= (m[r] ? 1u : 0u) << r;
    }
    err = e < err ? e : err;
    const unsigned long long starts = __ballot(start);
    if (lane == 0) s_before[r * kWaves + tid / kWave] = __popcll(starts);
  }
  __syncthreads();
  int n_seg;
  const int k = tid < rounds * kWaves ? s_before[tid] : 0;
  const int before = block_exclusive_scan<kOneThreads>(k, s_scan, &n_seg);
  if (tid < rounds * kWaves) s_before[tid] = before;
  one_table<kMax>(p, ws, s_table, s_surv, s_before, n_seg, own, rounds, err, alpha, grad_scale);
}

int grid_for(long long items, int per_block, int cap) {
  long long g = (items + per_block - 1) / per_block;
  if (g < 1) g = 1;
  return (int)(g < cap ? g : cap);
}

}  // namespace

hipError_t launch_segments(const SegParams& p, const Ws& ws, long long nblk, hipStream_t s) {
  const int n_surv = p.floor_on ? p.max_turns : 0;
  seg_count<<<dim3((unsigned)(nblk > 0 ? nblk : 1)), dim3(kSegThreads), 0, s>>>(p, ws, n_surv);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if (nblk == 0) return hipSuccess;
  if (nblk <= kFusedScanTiles) {
    seg_write<true><<<dim3((unsigned)nblk), dim3(kSegThreads), 0, s>>>(p, ws, nblk);
  } else {
    seg_offsets<<<1, kScanThreads, 0, s>>>(ws, nblk);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    seg_write<false><<<dim3((unsigned)nblk), dim3(kSegThreads), 0, s>>>(p, ws, nblk);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  seg_link<<<grid_for(p.n, kSegThreads, 1024), kSegThreads, 0, s>>>(p, ws);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if (!p.floor_on) return hipSuccess;
  seg_valid<<<grid_for(p.n, kSegThreads, 1024), kSegThreads, 0, s>>>(p, ws);
  return hipGetLastError();
}

bool one_workgroup(const SegParams& p) {
  return p.n <= kOneThreads * kOneMax && (!p.floor_on || p.max_turns <= kOneTurns);
}

hipError_t launch_one_workgroup(const SegParams& p, const Ws& ws, double alpha, float grad_scale,
                                int n_chunks, float* kl, hipStream_t s) {
  const int slot_words = n_chunks > 1 ? n_chunks * kExchangeWords : 0;
  const int per = (int)((p.n + kOneThreads - 1) / kOneThreads);
  // a workgroup clears about 32 KiB
  const int grid = 1 + grid_for(p.n * (2 * slot_words + 1), 8 * kOneThreads, 255);
  if (per <= 4) seg_one<4><<<grid, kOneThreads, 0, s>>>(p, ws, alpha, grad_scale, slot_words, kl, per);
  else seg_one<kOneMax><<<grid, kOneThreads, 0, s>>>(p, ws, alpha, grad_scale, slot_words, kl, per);
  return hipGetLastError();
}

hipError_t launch_weights(const SegParams& p, const Ws& ws, double alpha, float grad_scale,
                          int n_chunks, float* kl, hipStream_t s) {
  if (p.n == 0) return hipSuccess;
  const int slot_words = n_chunks > 1 ? n_chunks * kExchangeWords : 0;
  token_weights<<<grid_for(p.n, kSegThreads, 4096), kSegThreads, 0, s>>>(p, ws, alpha, grad_scale,
                                                                         slot_words, kl);
  return hipGetLastError();
}

}  // namespace turnkl
