// Row kernel: per-token reverse KL over the full vocabulary and its gradient
// with respect to the student logits, fused in one read of each logit.
//
// Math (Sec. 3, Eq. opd-rkl; teacher frozen; temperature 1).  For a row with
// student logits a and teacher logits b:
//   p_s = softmax(a),  mu = <p_s, a - b>,  lse = log sum exp
//   KL  = mu - lse(a) + lse(b)
//   dKL/da_v = p_s(v) (log p_s(v) - log p_t(v) - KL) = p_s(v) ((a_v - b_v) - mu)
// so the gradient needs only lse(a) and mu, and the loss needs lse(b) too.
// All exponentials are base 2 (v_exp_f32): a chunk keeps, in log2 units,
//   M_s = max(a) log2(e),  S_s = sum 2^(a log2(e) - M_s),  A = sum 2^(...) (a - b),
//   M_t = max(b) log2(e),  S_t = sum 2^(b log2(e) - M_t).
//
// Work decomposition.  A row of V elements (V / epv packs of 16 bytes) is cut
// into n_chunks chunks whose boundaries chunk_start places on 1 KiB (or
// 128-byte) multiples from the row start when the host's tiling allows, else
// balanced; each of a workgroup's 256 threads holds up to vpt packs.  One
// workgroup owns one (row, chunk) task: it loads its chunk of both rows into
// registers, reduces the chunk's partials, publishes the seven of them as four
// 64-bit words (see the row merge below), reads its row mates' words, merges
// all chunks in chunk order (so every workgroup of the row computes
// bit-identical row scalars), and writes its chunk of the gradient straight
// from registers.  Every logit is read from HBM exactly once and every
// gradient element written once: 3 V s bytes per supervised row, V s per
// unsupervised row (zeros only).
//
// Scheduling.  A wave's priority rises with its task's progress (loads,
// partial sums, stores), and the bf16 kernel comes in two load orders, one
// of which each call runs (both explained where they are set).
//
// Rows that are no whole packs or do not start on one take the same kernel in
// another form (RowForm), compiled in rowkl_ragged.hip; its bound is the same,
// HBM, at 5.5 TB/s for 6,000 bf16 rows of 50,257 elements (2.0 TB/s with one
// element per load) and 5.85 TB/s for 3,000 fp32 rows.
//
// Rows of up to 2,048 packs (1,792 in large batches) take one workgroup each
// (kWhole, compiled in rowkl_whole.hip), of one wave up to 512 packs, handed out by the hardware's
// dispatch: their loads, sums and stores last less than the queue for the one
// ticket counter.  What bounds them is latency below about 2,000 elements
// (65,536 bf16 rows of 1,024: 94 us a call, 49 of them the other kernels), HBM
// above (8,192: 4.9 TB/s over the whole call).
//
// Longer rows' tasks are handed out by an atomic ticket in row-major order, so a
// workgroup only ever waits for tasks that running workgroups already hold
// or that the next free workgroup will take; the wait is bounded and reports
// TURNKL_ERR_SYNC_TIMEOUT instead of hanging.  An in-place gradient is safe
// because each workgroup reads its chunk completely before writing it, and
// chunks do not overlap.

#include "row_ops.h"

namespace turnkl {
namespace {

// Workgroups of a launch with one workgroup per row; beyond, each takes several.
constexpr int kWholeGrid = 1 << 22;

// How a row's packs lie.
//  kAligned: every row is whole packs and starts on one.
//  kRagged:  rows of any length (>= one pack) and start.  The packs lie on the
//            grid of the written matrix's cache lines, so that whole-wave
//            accesses cover whole lines (the same kernel with its packs
//            counted from each row's first element takes 317 instead of 277 us
//            for 6,000 bf16 rows of 50,257); the row's first and last packs
//            are moved inside the row where they would stick out, and the
//            elements they then share with their neighbours are left out of
//            the sums.  The shared elements of a gradient row are written
//            twice, with the same bits.
//  kScalar:  one element per pack (rows shorter than a 16-byte pack).
enum RowForm { kAligned, kRagged, kScalar };

// One (row, chunk) task per iteration (kWhole: one row, the whole of it, with
// rows blockIdx.x, blockIdx.x + gridDim.x, ...).  A chunk is the pack range
// [pack_lo, pack_hi) of the row; thread tid owns packs pack_lo + v * kThreads +
// tid for v < kVpt.  The host's tiling makes every chunk at least kThreads
// (kVpt - 1) packs long, so every pack v < kVpt - 1 lies inside the chunk and only the
// last one is predicated (kScalar: all of them; kRagged: the first and the
// last one, which may stick out of the row).
template <bool kBf16, int kEpv, int kVpt, RowForm kForm, bool kSplit, int kThreads, bool kWhole>
__global__ __launch_bounds__(kThreads) void rowkl_kernel(RowParams p) {
  constexpr bool kCheckAll = kForm == kScalar;
  // sums taken pack by pack: one more operation in eight, and an error against
  // 64 bits below that of a chain over all of a thread's elements
  constexpr bool kPackSums = kWhole || kForm == kRagged;
  using P = Pack<kBf16, kEpv>;
  constexpr int kEs = kBf16 ? 2 : 4;
  constexpr int kPackBytes = kEpv * kEs;
  constexpr int kWaves = kThreads / kWave;
  constexpr int kChunkSlots = kWhole ? 1 : kMaxChunks;
  constexpr int kStep = kThreads * kPackBytes;  // bytes between a thread's packs

  __shared__ float s_max[2][kWaves];
  __shared__ float s_sum[3][kWaves];
  __shared__ unsigned long long s_word[kChunkSlots * kExchangeWords];
  __shared__ float s_ref[kWaves];
  __shared__ int s_lo[kChunkSlots + 1];  // first pack of each chunk
  __shared__ unsigned s_task;
  __shared__ int s_timeout;

  // kWhole: the first row's mask is on its way while the error key is awaited
  unsigned my_row = blockIdx.x;
  const unsigned char first_mask = kWhole ? p.mask[my_row] : 0;
  if (p.hdr->err_key != kNoError) return;
  // Two launches, one per load order (see the loads below): the split order
  // runs when at most 90% of the rows are supervised, the other one exits
  // here before taking any work.
  if (p.pick_order &&
      (10ll * __builtin_amdgcn_readfirstlane(p.hdr->n_sup) < 9ll * (long long)p.n_rows) != kSplit)
    return;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wid = tid / kWave;
  const unsigned n_tasks = (unsigned)p.n_rows * (unsigned)p.n_chunks;
  // chunk c is packs [chunk_start(c), chunk_start(c + 1)) of the row
  for (int k = tid; !kWhole && k <= p.n_chunks; k += kThreads)
    s_lo[k] = (int)chunk_start(p.n_packs, p.n_chunks, p.align, k);
  // data of this wave's most recent 16-byte store, kept live until the next
  // task's loads are issued (see keep_alive)
  typename P::Data carry = P::zero();

  // Thread 0 takes the next ticket near the end of the current task: after
  // the last gradient store is issued (a masked row: after its zero stores),
  // so the atomic's latency hides behind the stores draining, and a ticket
  // is started right after it is taken.  The workgroups that take the
  // chunks of one row (consecutive tickets) then start them at nearly the
  // same time and wait little for each other; taking it right after the row
  // merge instead measured 4% slower.  A ticket is never taken before the
  // current task's row mates have all published, so a workgroup never waits
  // for row mates while it holds a ticket it has not started, which keeps
  // the row-major ticket order deadlock-free.
  constexpr unsigned kNoTicket = 0xFFFFFFFFu;
  unsigned next_task = kNoTicket;

  for (;;) {
    if (!kWhole && tid == 0) {
      s_task = next_task != kNoTicket ? next_task : take_ticket(&p.hdr->ticket);
      next_task = kNoTicket;
    }
    if (!kWhole || my_row != blockIdx.x) __syncthreads();
    // Wave priority follows the task's progress: issuing loads 0, partial
    // sums 1, gradient (or zero) stores 2.  A wave further along its task
    // wins the SIMD's issue arbitration, finishes its stores sooner and
    // starts its next loads sooner; this measured 3.5% faster than equal
    // priorities (6.97 against 7.23 ms for 65,536 rows, same process).
    __builtin_amdgcn_s_setprio(0);
    // uniform: keep it scalar
    const unsigned task = kWhole ? my_row : __builtin_amdgcn_readfirstlane(s_task);
    my_row += gridDim.x;
    if (task >= n_tasks) break;
    // s_task is rewritten only after every wave has passed a later barrier of
    // this task (pass 1's, or the masked path's), so no wave can miss it
    if (!kWhole && tid == 0) s_timeout = 0;
    const long long row = kWhole ? task : (long long)(task / (unsigned)p.n_chunks);
    const int c = kWhole ? 0 : (int)(task - (unsigned)row * (unsigned)p.n_chunks);
    const int pack_lo = kWhole ? 0 : __builtin_amdgcn_readfirstlane(s_lo[c]);
    int pack_hi = kWhole ? p.n_packs : __builtin_amdgcn_readfirstlane(s_lo[c + 1]);
    long long col = (long long)pack_lo * kEpv;  // first element of the chunk
    const int lane_off = tid * kPackBytes;
    // Ragged rows: the row's first pack begins pre / kEs elements before the
    // row, on the line that holds the row's first element; a pack that sticks
    // out of the row is moved inside it by `shift` elements, and its element j
    // belongs to it only where 0 <= j - shift < kEpv (nowhere, for a pack
    // wholly outside).  Bit j of edge_bits says so for the thread's first and
    // last pack: a mask without branches, which the sums' register budget needs.
    unsigned bits_first = 0, bits_last = 0;
    int off_first = 0, off_last = 0;  // byte offsets of those packs from the chunk's first element
    if constexpr (kForm == kRagged) {
      const char* rows = static_cast<const char*>(p.grad ? p.grad : p.zs);
      const int pre = (int)(reinterpret_cast<uintptr_t>(rows + row * (p.grad ? p.ld_g : p.ld_s) * kEs) &
                            (uintptr_t)p.line_mask);
      const int n_row = (pre + p.vocab * kEs + kPackBytes - 1) / kPackBytes;
      pack_hi = pack_hi < n_row ? pack_hi : n_row;
      col -= pre / kEs;
      const int n = pack_hi - pack_lo;
      const int e_first = (int)col + tid * kEpv;
      const int e_last = e_first + (kVpt - 1) * kThreads * kEpv;
      const int at_first = inside_row(e_first, p.vocab - kEpv);
      const int at_last = inside_row(e_last, p.vocab - kEpv);
      bits_first = tid < n ? own_bits<kEpv>(e_first - at_first) : 0u;
      bits_last = (kVpt - 1) * kThreads + tid < n ? own_bits<kEpv>(e_last - at_last) : 0u;
      off_first = (at_first - (int)col) * kEs;
      off_last = (at_last - (int)col) * kEs;
    }
    const int n_valid = pack_hi - pack_lo;  // packs in this chunk

    bool valid[kVpt];
#pragma unroll
    for (int v = 0; v < kVpt; ++v) {
      if (kForm == kRagged)
        valid[v] = v == 0 ? bits_first != 0u : (v == kVpt - 1 ? bits_last != 0u : true);
      else
        valid[v] = (kCheckAll || v == kVpt - 1) ? (v * kThreads + tid < n_valid) : true;
    }
    // the offsets of pack v's loads and stores: per-lane part and uniform part
#define TURNKL_EDGE(v) (kForm == kRagged && ((v) == 0 || (v) == kVpt - 1))
#define TURNKL_OFF_V(v) (TURNKL_EDGE(v) ? ((v) == 0 ? off_first : off_last) : lane_off)
#define TURNKL_OFF_S(v) (TURNKL_EDGE(v) ? 0 : (v) * kStep)

    if (!(kWhole && task == blockIdx.x ? first_mask : p.mask[row])) {
      if (p.lse && c == 0 && tid == 0) {  // the row is not read: no log-partition function
        p.lse[2 * row] = __builtin_nanf("");
        p.lse[2 * row + 1] = __builtin_nanf("");
      }
      if (p.grad) {
        __builtin_amdgcn_s_setprio(2);
        const typename P::Data z = P::zero();
        const auto rg = chunk_rsrc(static_cast<char*>(p.grad) + (row * p.ld_g + col) * kEs);
#pragma unroll
        for (int v = 0; v < kVpt; ++v)
          if (valid[v]) P::store(rg, TURNKL_OFF_V(v), TURNKL_OFF_S(v), z);
        __builtin_amdgcn_s_setprio(0);
        if (!kWhole && tid == 0) next_task = take_ticket(&p.hdr->ticket);
        // the zeros sit in registers the loop's phi copies may take over
        // right away: let the stores complete first
        drain_stores();
        keep_alive(carry);
      } else if (!kWhole && tid == 0) {
        next_task = take_ticket(&p.hdr->ticket);
      }
      __syncthreads();
      continue;
    }

    // ---- load the chunk of both rows into registers (an out-of-chunk pack
    // reads the chunk's first pack instead and is masked below)
    const auto rs = chunk_rsrc(static_cast<const char*>(p.zs) + (row * p.ld_s + col) * kEs);
    const auto rt = chunk_rsrc(static_cast<const char*>(p.zt) + (row * p.ld_t + col) * kEs);
    // Load order.  kSplit: the student's packs, then the teacher's; else
    // alternating.  On batches that mix masked and supervised rows the split
    // order measured 1.6% faster (6.84 against 6.96 ms for the 65,536-row
    // batch with 40% of its rows masked, 1.47 against 1.49 ms with 60%
    // masked, same process); with every row supervised it is 1.9% slower
    // (9.66 against 9.48 ms), so the host launches both orders and each
    // call runs one (see rowkl_kernel's first lines).  The two orders are
    // separate kernels: in one kernel the bf16 instantiation needs 258 VGPRs
    // (one wave per SIMD), and so does the fp32 one with the split order,
    // which therefore always alternates.
    P xs[kVpt], xt[kVpt];
    if constexpr (kSplit) {
#pragma unroll
      for (int v = 0; v < kVpt; ++v) {
        const bool sure = kForm == kRagged || (!kCheckAll && v < kVpt - 1);
        xs[v].load(rs, sure ? TURNKL_OFF_V(v) : (valid[v] ? lane_off : 0),
                   sure ? TURNKL_OFF_S(v) : (valid[v] ? v * kStep : 0));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < kVpt; ++v) {
        const bool sure = kForm == kRagged || (!kCheckAll && v < kVpt - 1);
        xt[v].load(rt, sure ? TURNKL_OFF_V(v) : (valid[v] ? lane_off : 0),
                   sure ? TURNKL_OFF_S(v) : (valid[v] ? v * kStep : 0));
      }
    } else {
#pragma unroll
      for (int v = 0; v < kVpt; ++v) {
        const bool sure = kForm == kRagged || (!kCheckAll && v < kVpt - 1);
        const int vo = sure ? TURNKL_OFF_V(v) : (valid[v] ? lane_off : 0);
        const int so = sure ? TURNKL_OFF_S(v) : (valid[v] ? v * kStep : 0);
        xs[v].load(rs, vo, so);
        xt[v].load(rt, vo, so);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    keep_alive(carry);  // the previous task's last store has long read its data

    // ---- chunk partials.  Any reference works for S = sum 2^(a log2e - M)
    // as long as no term overflows, so the fast path's reference is the
    // maximum over each thread's first pack only, folded into one FMA per
    // exponent (log2 units: the fast form of merge_chunk).  A chunk whose
    // reference is far from zero (|max| > 64), or whose sums near an overflow, is
    // redone against its exact maximum with the references subtracted per
    // element, directly in natural-reference form (uniform branch; cold for
    // ordinary logits).
#define TURNKL_BLOCK_MAX2(MS, MT)                        \
  {                                                      \
    MS = wave_max(MS);                                   \
    MT = wave_max(MT);                                   \
    if (lane == 0) {                                     \
      s_max[0][wid] = MS;                                \
      s_max[1][wid] = MT;                                \
    }                                                    \
    __syncthreads();                                     \
    MS = s_max[0][0];                                    \
    MT = s_max[1][0];                                    \
    _Pragma("unroll") for (int w = 1; w < kWaves; ++w) { \
      MS = fmaxf(MS, s_max[0][w]);                       \
      MT = fmaxf(MT, s_max[1][w]);                       \
    }                                                    \
  }
#define TURNKL_FENCE_ALL()                                \
  _Pragma("unroll") for (int v = 0; v < kVpt; ++v) {     \
    xs[v].fence();                                       \
    xt[v].fence();                                       \
  }
#define TURNKL_BLOCK_SUMS(SS, AA, ST)                                         \
  {                                                                           \
    SS = wave_sum(SS);                                                        \
    AA = wave_sum(AA);                                                        \
    ST = wave_sum(ST);                                                        \
    if (lane == 0) {                                                          \
      s_sum[0][wid] = SS;                                                     \
      s_sum[1][wid] = AA;                                                     \
      s_sum[2][wid] = ST;                                                     \
    }                                                                         \
    __syncthreads();                                                          \
    SS = s_sum[0][0];                                                         \
    AA = s_sum[1][0];                                                         \
    ST = s_sum[2][0];                                                         \
    _Pragma("unroll") for (int w = 1; w < kWaves; ++w) {                   \
      SS += s_sum[0][w];                                                      \
      AA += s_sum[1][w];                                                      \
      ST += s_sum[2][w];                                                      \
    }                                                                         \
  }
  // OFFSET (a literal): exponents against natural references RS, RT and the
  // exact difference against the double-float C2; otherwise RS, RT are
  // log2-unit references folded into the exponent FMA (C2 unused)
#define TURNKL_CHUNK_SUMS(OFFSET, RS, RT, C2, SS, AA, ST)                     \
  {                                                                           \
    SS = 0.0f;                                                                \
    AA = 0.0f;                                                                \
    ST = 0.0f;                                                                \
    _Pragma("unroll") for (int v = 0; v < kVpt; ++v) {                        \
      float ps = 0.0f, pa = 0.0f, pt = 0.0f;                                  \
      _Pragma("unroll") for (int j = 0; j < kEpv; ++j) {                      \
        const float a = xs[v].get(j);                                         \
        const float b = xt[v].get(j);                                         \
        float es, et, d;                                                      \
        if (OFFSET) {                                                         \
          es = exp2_fast((a - (RS)) * kLog2e);                                \
          et = exp2_fast((b - (RT)) * kLog2e);                                \
          d = diff_minus(a, b, (C2));                                         \
        } else {                                                              \
          es = exp2_fast(fmaf(a, kLog2e, -(RS)));                             \
          et = exp2_fast(fmaf(b, kLog2e, -(RT)));                             \
          d = a - b;                                                          \
        }                                                                     \
        if (TURNKL_EDGE(v)) {                                                 \
          const unsigned own = own_mask(v == 0 ? bits_first : bits_last, j);  \
          es = __uint_as_float(__float_as_uint(es) & own);                    \
          et = __uint_as_float(__float_as_uint(et) & own);                    \
          d = __uint_as_float(__float_as_uint(d) & own);                      \
        } else if (kCheckAll || v == kVpt - 1) {                              \
          es = valid[v] ? es : 0.0f;                                          \
          et = valid[v] ? et : 0.0f;                                          \
          d = valid[v] ? d : 0.0f;                                            \
        }                                                                     \
        if (kPackSums) {                                                      \
          ps = j ? ps + es : es;                                              \
          pa = j ? fmaf(es, d, pa) : es * d;                                  \
          pt = j ? pt + et : et;                                              \
        } else {                                                              \
          SS += es;                                                           \
          AA = fmaf(es, d, AA);                                               \
          ST += et;                                                           \
        }                                                                     \
      }                                                                       \
      if (kPackSums) {                                                        \
        SS += ps;                                                             \
        AA += pa;                                                             \
        ST += pt;                                                             \
      }                                                                       \
      /* keeps the compiler from taking one sum over all packs at a time,     \
         with every unpacked value alive: over 200 more VGPRs */              \
      if (kForm == kRagged) asm volatile("" : "+v"(SS), "+v"(AA), "+v"(ST));  \
    }                                                                         \
    TURNKL_BLOCK_SUMS(SS, AA, ST)                                             \
  }

    float ms = -INFINITY, mt = -INFINITY;
    // (one wave takes the maximum over all packs: over the first ones alone its
    // sample would be a quarter of what a chunk's usually is)
#pragma unroll
    for (int v = 0; v < (kThreads == kWave ? kVpt : 1); ++v) {
#pragma unroll
      for (int j = 0; j < kEpv; ++j) {
        ms = fmaxf(ms, valid[v] ? xs[v].get(j) : -INFINITY);
        mt = fmaxf(mt, valid[v] ? xt[v].get(j) : -INFINITY);
      }
    }
    TURNKL_BLOCK_MAX2(ms, mt)
    float m2s = ms * kLog2e;
    float m2t = mt * kLog2e;
    __builtin_amdgcn_s_setprio(1);
    TURNKL_FENCE_ALL()
    float ss, aa, st;
    float c_a = 0.0f, c_b = 0.0f;  // difference reference (offset form only)
    TURNKL_CHUNK_SUMS(false, m2s, m2t, Float2{}, ss, aa, st)
    const bool offset = !(fmaxf(fabsf(m2s), fabsf(m2t)) <= kFar2) || !sums_in_range(ss, aa, st);
    if (offset) {
      __syncthreads();  // s_max / s_sum are about to be reused
      TURNKL_FENCE_ALL()
      // exact maxima, and the teacher logit at the student's maximum (ties:
      // the larger teacher logit, so every combination order agrees)
      ms = -INFINITY;
      mt = -INFINITY;
      float bm = -INFINITY;
      if constexpr (kForm == kRagged) {
        // from memory, one pack at a time: unrolled over the registers, this
        // path costs the ragged kernel over 100 VGPRs.  (A moved pack's
        // foreign elements are the row's own too, so any may be the maximum.)
#pragma unroll 1
        for (int v = 0; v < kVpt && v * kThreads + tid < n_valid; ++v) {
          P ya, yb;
          const int off = (inside_row((int)col + (v * kThreads + tid) * kEpv, p.vocab - kEpv) - (int)col) * kEs;
          ya.load(rs, off, 0);
          yb.load(rt, off, 0);
#pragma unroll
          for (int j = 0; j < kEpv; ++j) {
            const float a = ya.get(j);
            const float b = yb.get(j);
            const bool take = (a > ms) | ((a == ms) & (b > bm));
            ms = take ? a : ms;
            bm = take ? b : bm;
            mt = fmaxf(mt, b);
          }
        }
      } else {
#pragma unroll
        for (int v = 0; v < kVpt; ++v) {
#pragma unroll
          for (int j = 0; j < kEpv; ++j) {
            const float a = valid[v] ? xs[v].get(j) : -INFINITY;
            const float b = valid[v] ? xt[v].get(j) : -INFINITY;
            const bool take = (a > ms) | ((a == ms) & (b > bm));  // branch-free
            ms = take ? a : ms;
            bm = take ? b : bm;
            mt = fmaxf(mt, b);
          }
        }
      }
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) {
        const float oa = __shfl_xor(ms, o, kWave);
        const float ob = __shfl_xor(bm, o, kWave);
        const bool take = (oa > ms) | ((oa == ms) & (ob > bm));
        ms = take ? oa : ms;
        bm = take ? ob : bm;
        mt = fmaxf(mt, __shfl_xor(mt, o, kWave));
      }
      if (lane == 0) {
        s_max[0][wid] = ms;
        s_max[1][wid] = mt;
        s_ref[wid] = bm;
      }
      __syncthreads();
      ms = s_max[0][0];
      mt = s_max[1][0];
      bm = s_ref[0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) {
        const float oa = s_max[0][w];
        const float ob = s_ref[w];
        const bool take = (oa > ms) | ((oa == ms) & (ob > bm));
        ms = take ? oa : ms;
        bm = take ? ob : bm;
        mt = fmaxf(mt, s_max[1][w]);
      }
      m2s = ms;  // from here on: natural references
      m2t = mt;
      c_a = ms;  // difference reference: (a, b) where the student peaks
      c_b = bm;
      TURNKL_FENCE_ALL()
      __syncthreads();
      if constexpr (kForm == kRagged) {
        const Float2 c2 = two_diff(c_a, c_b);
        ss = 0.0f;
        aa = 0.0f;
        st = 0.0f;
#pragma unroll 1
        for (int v = 0; v < kVpt && v * kThreads + tid < n_valid; ++v) {
          P ya, yb;
          const int e = (int)col + (v * kThreads + tid) * kEpv;
          const int at = inside_row(e, p.vocab - kEpv);
          const unsigned bits = own_bits<kEpv>(e - at);
          ya.load(rs, (at - (int)col) * kEs, 0);
          yb.load(rt, (at - (int)col) * kEs, 0);
#pragma unroll
          for (int j = 0; j < kEpv; ++j) {
            const float a = ya.get(j);
            const float b = yb.get(j);
            const bool own = (bits >> j) & 1u;
            const float es = own ? exp2_fast((a - m2s) * kLog2e) : 0.0f;
            const float et = own ? exp2_fast((b - m2t) * kLog2e) : 0.0f;
            const float d = own ? diff_minus(a, b, c2) : 0.0f;
            ss += es;
            aa = fmaf(es, d, aa);
            st += et;
          }
        }
        TURNKL_BLOCK_SUMS(ss, aa, st)
      } else {
        TURNKL_CHUNK_SUMS(true, m2s, m2t, two_diff(c_a, c_b), ss, aa, st)
      }
    }
#undef TURNKL_CHUNK_SUMS
#undef TURNKL_BLOCK_SUMS
#undef TURNKL_FENCE_ALL
#undef TURNKL_BLOCK_MAX2
#pragma unroll
    for (int v = 0; v < kVpt; ++v) {
      xs[v].fence();
      xt[v].fence();
    }

    // ---- row scalars: publish this chunk's partials, read the row mates',
    // merge all of them in chunk order against the row references (the
    // largest chunk references; see merge_chunk), so every workgroup of the
    // row computes the same bits.  If any chunk took the offset path, the
    // whole row writes its gradient with offsets too.
    RowSums r{0.0f, 0.0f, 0.0f};
    float r_s, r_t;              // row references of the exponents, logit units
    float d_s = 0.0f, d_t = 0.0f;  // row reference C* of the difference a - b
    bool row_offset = offset;
    if (!kWhole && p.n_chunks > 1) {
      const int nw = p.n_chunks * kExchangeWords;
      unsigned long long* slot = p.slots + row * (long long)nw;
      if (tid == 0) {
        const unsigned tag = offset ? kTagOffset : kTagFast;
        unsigned long long* mine = slot + c * kExchangeWords;
        const unsigned long long words[kExchangeWords] = {
            word2(enc(m2s), enc(ss)), word2(enc(aa), enc(m2t)), word2(enc(st), enc(c_a)),
            word2(enc(c_b), tag)};
#pragma unroll
        for (int q = 0; q < kExchangeWords; ++q)
          __hip_atomic_store(mine + q, words[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      // Wait for every word of the row, bounded: after spin_limit empty polls,
      // or as soon as another workgroup of the call has timed out (checked
      // every 256 polls), the task ends with the timeout error.
      for (int q = tid; q < nw; q += kThreads) {
        unsigned long long x;
        int spins = 0;
        while ((x = __hip_atomic_load(slot + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0ull) {
          if (++spins > p.spin_limit || ((spins & 255) == 0 && err_low(p.hdr) != kNoErrorLow)) {
            s_timeout = 1;
            break;
          }
          __builtin_amdgcn_s_sleep(2);
        }
        s_word[q] = x;
      }
      __syncthreads();
      if (s_timeout) {
        if (tid == 0) atomicMin(&p.hdr->err_key, err_key(0, kPrioTimeout));
        drain_stores();
        return;
      }
      // every thread merges all chunks in chunk order (uniform branches):
      // unrolled for the usual handful of chunks, a loop beyond
      constexpr int kUnrolled = 8;
#define TURNKL_TAG(K) \
  (__builtin_amdgcn_readfirstlane((unsigned)(s_word[kExchangeWords * (K) + 3] >> 32)) == kTagOffset)
      r_s = -INFINITY;
      r_t = -INFINITY;
      row_offset = false;
#define TURNKL_REFS(K)                                              \
  {                                                                 \
    const bool o = TURNKL_TAG(K);                                   \
    float w[kPartials];                                             \
    unpack_partials(s_word + kExchangeWords * (K), w);              \
    if (o && (!row_offset || w[5] > d_s)) {                         \
      d_s = w[5];                                                   \
      d_t = w[6];                                                   \
    }                                                               \
    row_offset = row_offset || o;                                   \
    r_s = fmaxf(r_s, natural_ref(o, w[0]));                         \
    r_t = fmaxf(r_t, natural_ref(o, w[3]));                         \
  }
#pragma unroll
      for (int k = 0; k < kUnrolled; ++k)
        if (k < p.n_chunks) TURNKL_REFS(k)
#pragma unroll 1
      for (int k = kUnrolled; k < p.n_chunks; ++k) TURNKL_REFS(k)
#undef TURNKL_REFS
      if (d_s < r_s) {  // a fast chunk holds the row's reference
        d_s = 0.0f;
        d_t = 0.0f;
      }
      const Float2 c_row = two_diff(d_s, d_t);
#pragma unroll
      for (int k = 0; k < kUnrolled; ++k)
        if (k < p.n_chunks) {
          float w[kPartials];
          unpack_partials(s_word + kExchangeWords * k, w);
          merge_chunk(TURNKL_TAG(k), w, r_s, r_t, c_row, r);
        }
#pragma unroll 1
      for (int k = kUnrolled; k < p.n_chunks; ++k)
      {
        float w[kPartials];
        unpack_partials(s_word + kExchangeWords * k, w);
        merge_chunk(TURNKL_TAG(k), w, r_s, r_t, c_row, r);
      }
#undef TURNKL_TAG
    } else {
      r_s = natural_ref(offset, m2s);
      r_t = natural_ref(offset, m2t);
      d_s = c_a;
      d_t = c_b;
      const float w[kPartials] = {m2s, ss, aa, m2t, st, c_a, c_b};
      merge_chunk(offset, w, r_s, r_t, two_diff(d_s, d_t), r);
    }
    // without a gradient to write the task ends here (kWhole and kScalar; the other
    // forms always have one, but with these branches taken out the compiler
    // schedules the alternating order's loads and sums worse: 8,192 rows of
    // 151,936, all supervised, 1,235 -> 1,346 us a call)
    if (!kWhole && tid == 0 && !p.grad) next_task = take_ticket(&p.hdr->ticket);

    // mu = <p_s, (a - b) - (C*_a - C*_b)>,
    // KL = <p_s, a - b> - lse(a) + lse(b) = mu + ((C*_a - R_s) - (C*_b - R_t)) + ln(S_t / S_s)
    // log sum exp of each row = R + ln S
    const float mu = r.aa / r.ss;
    if (c == 0 && tid == 0) {
      p.kl[row] = (mu + ((d_s - r_s) - (d_t - r_t))) + kLn2 * log2f(r.st / r.ss);
      if (p.lse) {
        p.lse[2 * row] = r_s + kLn2 * log2f(r.ss);
        p.lse[2 * row + 1] = r_t + kLn2 * log2f(r.st);
      }
    }

    // ---- gradient chunk, straight from registers:
    // G = grad_scale * w * 2^((a - R_s) log2e - log2 S_s) * (((a - b) - (C*_a - C*_b)) - mu),
    // with log2 |grad_scale * w| folded into the exponent and the sign applied
    // last.  Rows of fast chunks only (C* = 0) fold R_s into the exponent's
    // FMA; rows with an offset chunk subtract the references per element.
    if (p.grad) {
      __builtin_amdgcn_s_setprio(2);
      const float sc = p.wsc[row];
      const float l2 = log2f(r.ss) - log2f(fabsf(sc));
      const float l2s = row_offset ? l2 : fmaf(r_s, kLog2e, l2);
      const unsigned flip = sc < 0.0f ? 0x80008000u : 0u;
      const auto rg = chunk_rsrc(static_cast<char*>(p.grad) + (row * p.ld_g + col) * kEs);
      if (!row_offset) {
        typename P::Data prev = P::zero();
#pragma unroll
        for (int v = 0; v < kVpt; ++v) {
          float out[kEpv];
#pragma unroll
          for (int j = 0; j < kEpv; ++j) {
            const float a = xs[v].get(j);
            const float b = xt[v].get(j);
            out[j] = exp2_fast(fmaf(a, kLog2e, -l2s)) * ((a - b) - mu);
          }
          const typename P::Data cur = P::encode(out, flip);
          if (valid[v]) P::store(rg, TURNKL_OFF_V(v), TURNKL_OFF_S(v), cur);
          // keep the store here, so the next pack's work separates it from
          // any reuse of its data registers; the previous pack's data is free
          __builtin_amdgcn_sched_barrier(0);
          keep_alive(prev);
          prev = cur;
          if (!kWhole && v == kVpt - 1 && tid == 0) next_task = take_ticket(&p.hdr->ticket);
        }
        carry = prev;
        __builtin_amdgcn_s_setprio(0);
      } else {
        // Offset rows (rare): read the chunk again, one pack at a time, so
        // this loop keeps no unpacked values of the unrolled one alive.  Each
        // thread reads a pack before it writes the same pack, which keeps an
        // in-place gradient safe; every store is drained before its data
        // registers can be reused.
        const Float2 c_row = two_diff(d_s, d_t);
        const auto rs2 = chunk_rsrc(static_cast<const char*>(p.zs) + (row * p.ld_s + col) * kEs);
        const auto rt2 = chunk_rsrc(static_cast<const char*>(p.zt) + (row * p.ld_t + col) * kEs);
        keep_alive(carry);
#pragma unroll 1
        for (int v = 0; v < kVpt; ++v) {
          if (v * kThreads + tid >= n_valid) break;
          P ya, yb;
          // a ragged row's pack that sticks out of the row: only its own
          // elements are written, since a neighbour may have overwritten the
          // shared ones (in place) before this pack was read
          int shift = 0, off = lane_off + v * kStep;
          if constexpr (kForm == kRagged) {
            const int e = (int)col + (v * kThreads + tid) * kEpv;
            const int at = inside_row(e, p.vocab - kEpv);
            shift = e - at;
            off = (at - (int)col) * kEs;
          }
          ya.load(rs2, off, 0);
          yb.load(rt2, off, 0);
          float out[kEpv];
#pragma unroll
          for (int j = 0; j < kEpv; ++j) {
            const float a = ya.get(j);
            const float b = yb.get(j);
            out[j] = exp2_fast(fmaf(a - r_s, kLog2e, -l2s)) * (diff_minus(a, b, c_row) - mu);
          }
          if (kForm != kRagged || shift == 0) {
            P::store(rg, off, 0, P::encode(out, flip));
          } else if constexpr (kForm == kRagged) {
#pragma unroll
            for (int j = 0; j < kEpv; ++j)
              if (own_mask(own_bits<kEpv>(shift), j)) store_one<kBf16>(rg, off + j * kEs, out[j], flip);
          }
          drain_stores();
        }
        carry = P::zero();
      }
    }
  }
  drain_stores();
}
#undef TURNKL_EDGE
#undef TURNKL_OFF_V
#undef TURNKL_OFF_S

// ---------------------------------------------------------------------------
// launch

#ifndef TURNKL_WHOLE_ROWS
int cu_count() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 256;
  if (dev < 64 && cache[dev] > 0) return cache[dev];
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
  if (dev < 64) cache[dev] = n;
  return n;
}

// workgroups of a kernel that run on a CU at once
template <auto kKernel>
int occupancy() {
  static const int occ = [] {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kKernel, kRowThreads, 0) != hipSuccess || n < 1)
      n = 1;
    return n;
  }();
  return occ;
}

template <auto kKernel>
hipError_t launch_tasks(const RowParams& p, hipStream_t s) {
  const long long tasks = (long long)p.n_rows * p.n_chunks;
  long long grid = (long long)occupancy<kKernel>() * cu_count();
  if (grid > tasks) grid = tasks;
  if (grid < 1) return hipSuccess;
  kKernel<<<dim3((unsigned)grid), dim3(kRowThreads), 0, s>>>(p);
  return hipGetLastError();
}

template <bool kBf16, int kEpv, int kVpt, RowForm kForm, bool kSplit = false>
hipError_t launch_one(const RowParams& p, hipStream_t s) {
  return launch_tasks<rowkl_kernel<kBf16, kEpv, kVpt, kForm, kSplit, kRowThreads, false>>(p, s);
}

#ifndef TURNKL_RAGGED_ROWS
// bf16: both load orders, each kernel checking which one the call uses; small
// batches, where the launch that exits at once (4.4 us) costs more than the
// other order saves (under 2%), the split order alone.  fp32: the alternating
// order alone.
constexpr double kOneOrderBytes = 1.2e9;
template <bool kBf16, int kEpv, int kVpt>
hipError_t launch_vector(const RowParams& p, hipStream_t s) {
  if constexpr (kBf16) {
    const double bytes = 48.0 * p.n_rows * p.n_packs;  // all rows supervised
    if (bytes <= kOneOrderBytes) return launch_one<kBf16, kEpv, kVpt, kAligned, true>(p, s);
    RowParams q = p;
    q.pick_order = 1;
    if (hipError_t e = launch_one<kBf16, kEpv, kVpt, kAligned, true>(q, s); e != hipSuccess) return e;
    return launch_one<kBf16, kEpv, kVpt, kAligned, false>(q, s);
  } else {
    return launch_one<kBf16, kEpv, kVpt, kAligned, false>(p, s);
  }
}
#else
template <bool kBf16, int kEpv, int kVpt>
hipError_t launch_vector(const RowParams& p, hipStream_t s) {
  return launch_one<kBf16, kEpv, kVpt, kRagged>(p, s);
}
#endif

template <bool kBf16, int kEpv>
hipError_t launch_vpt(const RowParams& p, int vpt, hipStream_t s) {
  switch (vpt) {
#define TURNKL_CASE(n) \
    case n: return launch_vector<kBf16, kEpv, n>(p, s);
#ifndef TURNKL_RAGGED_ROWS  // shorter ragged rows take one workgroup each
    TURNKL_CASE(1) TURNKL_CASE(2) TURNKL_CASE(3) TURNKL_CASE(4) TURNKL_CASE(5) TURNKL_CASE(6)
    TURNKL_CASE(7)
#endif
    TURNKL_CASE(8) TURNKL_CASE(9) TURNKL_CASE(10) TURNKL_CASE(11) TURNKL_CASE(12)
    TURNKL_CASE(13) TURNKL_CASE(14) TURNKL_CASE(15) TURNKL_CASE(16) TURNKL_CASE(17) TURNKL_CASE(18)
    TURNKL_CASE(19) TURNKL_CASE(20) TURNKL_CASE(21) TURNKL_CASE(22)
#ifndef TURNKL_RAGGED_ROWS
    TURNKL_CASE(23) TURNKL_CASE(24) TURNKL_CASE(25)
#endif
#undef TURNKL_CASE
    default: return hipErrorInvalidValue;
  }
}

#else
template <bool kBf16, int kEpv, int kVpt, RowForm kForm, int kThreads>
hipError_t launch_whole(const RowParams& p, hipStream_t s) {
  constexpr bool kSplit = kBf16 && kForm == kAligned;
  const int grid = p.n_rows < kWholeGrid ? p.n_rows : kWholeGrid;
  rowkl_kernel<kBf16, kEpv, kVpt, kForm, kSplit, kThreads, true><<<grid, kThreads, 0, s>>>(p);
  return hipGetLastError();
}

template <bool kBf16, int kEpv, RowForm kForm>
hipError_t launch_whole_vpt(const RowParams& p, const RowTiling& t, hipStream_t s) {
  switch (t.threads * 32 + t.vpt) {
#define TURNKL_CASE(threads, n) \
    case threads * 32 + n: return launch_whole<kBf16, kEpv, n, kForm, threads>(p, s);
    TURNKL_CASE(64, 1) TURNKL_CASE(64, 2) TURNKL_CASE(64, 3) TURNKL_CASE(64, 4) TURNKL_CASE(64, 5)
    TURNKL_CASE(64, 6) TURNKL_CASE(64, 7) TURNKL_CASE(64, 8)
    TURNKL_CASE(256, 3) TURNKL_CASE(256, 4) TURNKL_CASE(256, 5) TURNKL_CASE(256, 6) TURNKL_CASE(256, 7)
    TURNKL_CASE(256, 8)
#undef TURNKL_CASE
    default: return hipErrorInvalidValue;
  }
}
#endif

}  // namespace

#if defined(TURNKL_WHOLE_ROWS)
hipError_t launch_whole_rows(const RowParams& p, const RowTiling& t, hipStream_t s) {
  if (t.ragged)
    return p.bf16 ? launch_whole_vpt<true, 8, kRagged>(p, t, s) : launch_whole_vpt<false, 4, kRagged>(p, t, s);
  return p.bf16 ? launch_whole_vpt<true, 8, kAligned>(p, t, s) : launch_whole_vpt<false, 4, kAligned>(p, t, s);
}
#elif !defined(TURNKL_RAGGED_ROWS)
hipError_t launch_rows(const RowParams& p, const RowTiling& t, hipStream_t s) {
  if (p.n_rows == 0) return hipSuccess;
  if (t.threads) return launch_whole_rows(p, t, s);
  // without a gradient: faster than the chunks at every size tried, from 64 rows
  // of 16,392 (43 us a call there, 28 here) to 65,536 of 50,176 (1,429, 1,235)
  if (!p.grad && (t.vector || t.ragged)) return launch_forward_rows(p, t, s);
  if (t.ragged) return launch_ragged_rows(p, t, s);
  if (!t.vector) {
    return p.bf16 ? launch_one<true, 1, kScalarVpt, kScalar>(p, s)
                  : launch_one<false, 1, kScalarVpt, kScalar>(p, s);
  }
  return p.bf16 ? launch_vpt<true, 8>(p, t.vpt, s) : launch_vpt<false, 4>(p, t.vpt, s);
}
#else
hipError_t launch_ragged_rows(const RowParams& p, const RowTiling& t, hipStream_t s) {
  return p.bf16 ? launch_vpt<true, 8>(p, t.vpt, s) : launch_vpt<false, 4>(p, t.vpt, s);
}
#endif

}  // namespace turnkl
