// Row kernel of calls without a gradient, for rows of more than 2,048 packs:
// per-token reverse KL and log-partition functions (the math and the forms of
// a chunk's partial sums: rowkl.hip, row_ops.h).
//
// Without a gradient nothing has to stay in registers until the row's scalars
// are known, so no workgroup waits for another: each streams its chunk of both
// rows, four packs of each at a time, publishes the chunk's partials, and the
// one that is last to arrive at the row's counter merges them (in chunk order:
// the same bits whoever it is).  No tickets either, and six workgroups per CU
// instead of two.  The bound is HBM reads: 16,384 rows of 151,936 in bf16, 60%
// supervised, 1,045 us a call in the gradient's kernel and 973 here (6.14 TB/s
// over the whole call); 65,536 of 32,000: 1,153 and 814; 4,096 of 50,257 in
// fp32: 436 and 197.
//
// Every wave sums its own packs against its own reference, the maximum of its
// first four packs of each lane.  Where that is far from zero, or a sum nears
// an overflow, the wave goes over its packs in the offset form instead, every
// lane with running maxima of its own, and the chunk is reported in that form.

#include <type_traits>

#include "row_ops.h"

namespace turnkl {
namespace {

constexpr int kFwdThreads = 256;
constexpr int kFwdWaves = kFwdThreads / kWave;
constexpr int kFwdPacks = 4;           // packs of each row in flight per lane
constexpr int kFwdGrid = 1 << 22;      // workgroups; beyond, each takes several tasks

// Six waves per SIMD (80 VGPRs): eight spill to scratch.
template <bool kBf16, int kEpv, bool kRagged>
__global__ __launch_bounds__(kFwdThreads, 6) void rowfwd_kernel(RowParams p) {
  using P = Pack<kBf16, kEpv>;
  constexpr int kEs = kBf16 ? 2 : 4;
  constexpr int kPackBytes = kEpv * kEs;
  constexpr int kStep = kFwdThreads * kPackBytes;
  __shared__ float s_part[kFwdWaves][kPartials];
  __shared__ int s_off[kFwdWaves];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(tid / kWave);
  const unsigned n_tasks = (unsigned)p.n_rows * (unsigned)p.n_chunks;
  if (p.hdr->err_key != kNoError) return;
  for (unsigned task = blockIdx.x; task < n_tasks; task += gridDim.x) {
    const long long row = (long long)(task / (unsigned)p.n_chunks);
    const int c = (int)(task - (unsigned)row * (unsigned)p.n_chunks);
    if (!p.mask[row]) {
      if (p.lse && c == 0 && tid == 0) {  // the row is not read: no log-partition function
        p.lse[2 * row] = __builtin_nanf("");
        p.lse[2 * row + 1] = __builtin_nanf("");
      }
      continue;
    }
    const int lo = (int)chunk_start(p.n_packs, p.n_chunks, p.align, c);
    int hi = (int)chunk_start(p.n_packs, p.n_chunks, p.align, c + 1);
    int col = lo * kEpv;  // first element of the chunk
    if constexpr (kRagged) {
      const char* at = static_cast<const char*>(p.zs) + row * p.ld_s * kEs;
      const int pre = (int)(reinterpret_cast<uintptr_t>(at) & (uintptr_t)p.line_mask);
      const int n_row = (pre + p.vocab * kEs + kPackBytes - 1) / kPackBytes;
      hi = hi < n_row ? hi : n_row;
      col -= pre / kEs;
    }
    const int n = hi - lo;
    const auto rs = chunk_rsrc(static_cast<const char*>(p.zs) + (row * p.ld_s + col) * kEs);
    const auto rt = chunk_rsrc(static_cast<const char*>(p.zt) + (row * p.ld_t + col) * kEs);
    const int groups = (n + kFwdThreads * kFwdPacks - 1) / (kFwdThreads * kFwdPacks);

    // Loads the lane's packs of a group: pack q is number (4 g + q) * 256 + tid
    // of the chunk.  edge (the first and the last group): some may lie beyond the
    // chunk or stick out of the row; they are read inside it, and bits[q] says
    // which elements count.
    P xs[kFwdPacks], xt[kFwdPacks];
    unsigned bits[kFwdPacks];
    auto load = [&](int g, auto edge) {
#pragma unroll
      for (int q = 0; q < kFwdPacks; ++q) {
        const int v = g * kFwdPacks + q;
        if constexpr (decltype(edge)::value) {
          const int i = v * kFwdThreads + tid;
          int off;
          if constexpr (kRagged) {
            const int e = col + i * kEpv;
            const int at = inside_row(e, p.vocab - kEpv);
            bits[q] = i < n ? own_bits<kEpv>(e - at) : 0u;
            off = (at - col) * kEs;
          } else {
            bits[q] = i < n ? (1u << kEpv) - 1u : 0u;
            off = (i < n ? i : n - 1) * kPackBytes;
          }
          xs[q].load(rs, off, 0);
          xt[q].load(rt, off, 0);
        } else {
          xs[q].load(rs, tid * kPackBytes, v * kStep);
          xt[q].load(rt, tid * kPackBytes, v * kStep);
        }
      }
    };
    float m2s, m2t;  // the wave's references, log2 units
    float ss = 0.0f, aa = 0.0f, st = 0.0f;
    auto sums = [&](auto edge) {
#pragma unroll
      for (int q = 0; q < kFwdPacks; ++q) {
        float ps = 0.0f, pa = 0.0f, pt = 0.0f;
#pragma unroll
        for (int j = 0; j < kEpv; ++j) {
          const float a = xs[q].get(j);
          const float b = xt[q].get(j);
          float es = exp2_fast(fmaf(a, kLog2e, -m2s));
          float et = exp2_fast(fmaf(b, kLog2e, -m2t));
          float d = a - b;
          if constexpr (decltype(edge)::value) {
            const unsigned own = own_mask(bits[q], j);
            es = __uint_as_float(__float_as_uint(es) & own);
            et = __uint_as_float(__float_as_uint(et) & own);
            d = __uint_as_float(__float_as_uint(d) & own);
          }
          ps = j ? ps + es : es;
          pa = j ? fmaf(es, d, pa) : es * d;
          pt = j ? pt + et : et;
        }
        ss += ps;
        aa += pa;
        st += pt;
        // one pack after the other: all unpacked at once need over 100 VGPRs
        asm volatile("" : "+v"(ss), "+v"(aa), "+v"(st));
      }
    };
    load(0, std::true_type{});
    float ms = -INFINITY, mt = -INFINITY;
#pragma unroll
    for (int q = 0; q < kFwdPacks; ++q)
#pragma unroll
      for (int j = 0; j < kEpv; ++j) {
        // (a moved pack's foreign elements are the row's own too)
        ms = fmaxf(ms, bits[q] ? xs[q].get(j) : -INFINITY);
        mt = fmaxf(mt, bits[q] ? xt[q].get(j) : -INFINITY);
      }
#pragma unroll
    for (int q = 0; q < kFwdPacks; ++q) {  // no unpacked value stays alive
      xs[q].fence();
      xt[q].fence();
    }
    m2s = wave_max(ms) * kLog2e;
    m2t = wave_max(mt) * kLog2e;
    bool offset = !(fmaxf(fabsf(m2s), fabsf(m2t)) <= kFar2);
    float c_a = 0.0f, c_b = 0.0f;
    const bool idle = wid * kWave >= n;  // no pack of the chunk is this wave's
    if (!offset) {
      sums(std::true_type{});
#pragma unroll 1
      for (int g = 1; g + 1 < groups; ++g) {
        load(g, std::false_type{});
        sums(std::false_type{});
      }
      if (groups > 1) {
        load(groups - 1, std::true_type{});
        sums(std::true_type{});
      }
      ss = wave_sum(ss);
      aa = wave_sum(aa);
      st = wave_sum(st);
      offset = !sums_in_range(ss, aa, st);
    }
    if (offset && !idle) {
      // offset form: each lane against its own maxima so far, which it moves
      // (and its sums with them) as it meets larger ones, then the wave's
      ms = -INFINITY;
      mt = -INFINITY;
      ss = 0.0f;
      aa = 0.0f;
      st = 0.0f;
#pragma unroll 1
      for (int v = 0; v < groups * kFwdPacks; ++v) {
        const int i = v * kFwdThreads + tid;
        const int e = col + i * kEpv;
        const int at = kRagged ? inside_row(e, p.vocab - kEpv) : (i < n ? e : col + (n - 1) * kEpv);
        const unsigned own = i < n ? own_bits<kEpv>(e - at) : 0u;
        P ya, yb;
        ya.load(rs, (at - col) * kEs, 0);
        yb.load(rt, (at - col) * kEs, 0);
        float na = ms, nt = mt, ca = c_a, cb = c_b;
#pragma unroll
        for (int j = 0; j < kEpv; ++j) {
          const float a = ya.get(j);
          const float b = yb.get(j);
          const bool take = own && ((a > na) | ((a == na) & (b > cb)));
          na = take ? a : na;
          ca = take ? a : ca;
          cb = take ? b : cb;
          nt = own ? fmaxf(nt, b) : nt;
        }
        const Float2 c2 = two_diff(ca, cb);
        if (na != ms || cb != c_b) {
          // (f == 0, as for masked logits before the first others: the sums so
          // far are dropped; aa, and ss times the difference, may be infinite)
          const float f = ms == -INFINITY ? 0.0f : exp2f((ms - na) * kLog2e);
          aa = f == 0.0f ? 0.0f : fmaf(ss, diff_minus(c_a, c_b, c2), aa) * f;
          ss *= f;
          ms = na;
          c_a = ca;
          c_b = cb;
        }
        if (nt != mt) {
          st *= mt == -INFINITY ? 0.0f : exp2f((mt - nt) * kLog2e);
          mt = nt;
        }
        const float us = ms == -INFINITY ? 0.0f : ms;
        const float ut = mt == -INFINITY ? 0.0f : mt;
#pragma unroll
        for (int j = 0; j < kEpv; ++j) {
          const float a = ya.get(j);
          const float b = yb.get(j);
          const bool on = (own >> j) & 1u;
          const float es = on ? exp2_fast((a - us) * kLog2e) : 0.0f;
          const float et = on ? exp2_fast((b - ut) * kLog2e) : 0.0f;
          const float d = on ? diff_minus(a, b, c2) : 0.0f;
          ss += es;
          aa = fmaf(es, d, aa);
          st += et;
        }
      }
      float wa = ms, wb = c_b, wt = wave_max(mt);
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) {
        const float oa = __shfl_xor(wa, o, kWave);
        const float ob = __shfl_xor(wb, o, kWave);
        const bool take = (oa > wa) | ((oa == wa) & (ob > wb));
        wa = take ? oa : wa;
        wb = take ? ob : wb;
      }
      const Float2 cw = two_diff(wa, wb);
      const float fs = ms == -INFINITY ? 0.0f : exp2f((ms - wa) * kLog2e);
      const float ft = mt == -INFINITY ? 0.0f : exp2f((mt - wt) * kLog2e);
      aa = fs == 0.0f ? 0.0f : fmaf(ss, diff_minus(c_a, c_b, cw), aa) * fs;
      ss = wave_sum(ss * fs);
      aa = wave_sum(aa);
      st = wave_sum(st * ft);
      m2s = wa;  // natural references from here on
      m2t = wt;
      c_a = wa;
      c_b = wb;
    }
    if (lane == 0) {
      const float w[kPartials] = {m2s, ss, aa, m2t, st, c_a, c_b};
#pragma unroll
      for (int i = 0; i < kPartials; ++i) s_part[wid][i] = w[i];
      s_off[wid] = offset && !idle;
    }
    __syncthreads();
    if (wid == 0) {
      // the waves' partials into the chunk's: in the fast form if all are, else
      // in the offset form (as chunks of a row are merged)
      const int waves = n >= kFwdThreads ? kFwdWaves : (n + kWave - 1) / kWave;
      bool c_off = false;
#pragma unroll 1
      for (int w = 0; w < waves; ++w) c_off = c_off || s_off[w];
      float x[kPartials] = {-INFINITY, 0.0f, 0.0f, -INFINITY, 0.0f, 0.0f, 0.0f};
      bool any = false;
#pragma unroll 1
      for (int w = 0; w < waves; ++w) {
        const bool o = s_off[w];
        x[0] = fmaxf(x[0], c_off ? natural_ref(o, s_part[w][0]) : s_part[w][0]);
        x[3] = fmaxf(x[3], c_off ? natural_ref(o, s_part[w][3]) : s_part[w][3]);
        if (o && (!any || s_part[w][5] > x[5])) {
          x[5] = s_part[w][5];
          x[6] = s_part[w][6];
          any = true;
        }
      }
      if (x[5] < x[0]) {  // a wave in the fast form holds the chunk's reference
        x[5] = 0.0f;
        x[6] = 0.0f;
      }
      RowSums r{0.0f, 0.0f, 0.0f};
      const Float2 c2 = two_diff(x[5], x[6]);
#pragma unroll 1
      for (int w = 0; w < waves; ++w) {
        if (c_off) {
          merge_chunk(s_off[w], s_part[w], x[0], x[3], c2, r);
        } else {
          const float fs = exp2f(s_part[w][0] - x[0]);
          r.ss = fmaf(s_part[w][1], fs, r.ss);
          r.aa = fmaf(s_part[w][2], fs, r.aa);
          r.st = fmaf(s_part[w][4], exp2f(s_part[w][3] - x[3]), r.st);
        }
      }
      x[1] = r.ss;
      x[2] = r.aa;
      x[4] = r.st;

      // the row: this workgroup's own chunk, or all of them if it is the last
      bool last = true;
      unsigned long long* const slot = p.slots + row * (long long)(p.n_chunks * kExchangeWords);
      if (p.n_chunks > 1) {
        unsigned arrived = 0;
        if (lane == 0) {
          const unsigned tag = c_off ? kTagOffset : kTagFast;
          const unsigned long long words[kExchangeWords] = {
              word2(enc(x[0]), enc(x[1])), word2(enc(x[2]), enc(x[3])), word2(enc(x[4]), enc(x[5])),
              word2(enc(x[6]), tag)};
#pragma unroll
          for (int q = 0; q < kExchangeWords; ++q)
            __hip_atomic_store(slot + c * kExchangeWords + q, words[q], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          // The words are visible before the count: agent-scope stores write
          // through the XCD's L2, so they are where the other XCDs read once
          // they are complete.  (A release fence, and an acquire fence before
          // the reads below, write back and invalidate the whole L2 for every
          // workgroup: 16,384 rows of 151,936 take 2,390 us with them, 949
          // without.)
          drain_stores();
          arrived = __hip_atomic_fetch_add(reinterpret_cast<unsigned*>(p.wsc + row), 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        }
        last = __builtin_amdgcn_readfirstlane(arrived) + 1u == (unsigned)p.n_chunks;
      }
      if (last) {
        asm volatile("" ::: "memory");  // no read below moves above the count
        float r_s = -INFINITY, r_t = -INFINITY, d_s = 0.0f, d_t = 0.0f;
        bool row_off = false;
        RowSums sum{0.0f, 0.0f, 0.0f};
        // twice over the chunks: the references, then the sums
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll 1
          for (int k = 0; k < p.n_chunks; ++k) {
            float w[kPartials];
            bool o = c_off;
            if (p.n_chunks > 1) {
              unsigned long long u[kExchangeWords];
#pragma unroll
              for (int q = 0; q < kExchangeWords; ++q)
                u[q] = __hip_atomic_load(slot + k * kExchangeWords + q, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
              unpack_partials(u, w);
              o = (unsigned)(u[kExchangeWords - 1] >> 32) == kTagOffset;
            } else {
#pragma unroll
              for (int i = 0; i < kPartials; ++i) w[i] = x[i];
            }
            if (pass == 0) {
              if (o && (!row_off || w[5] > d_s)) {
                d_s = w[5];
                d_t = w[6];
              }
              row_off = row_off || o;
              r_s = fmaxf(r_s, natural_ref(o, w[0]));
              r_t = fmaxf(r_t, natural_ref(o, w[3]));
            } else {
              merge_chunk(o, w, r_s, r_t, two_diff(d_s, d_t), sum);
            }
          }
          if (d_s < r_s) {
            d_s = 0.0f;
            d_t = 0.0f;
          }
        }
        if (lane == 0) {
          p.kl[row] = (sum.aa / sum.ss + ((d_s - r_s) - (d_t - r_t))) + kLn2 * log2f(sum.st / sum.ss);
          if (p.lse) {
            p.lse[2 * row] = r_s + kLn2 * log2f(sum.ss);
            p.lse[2 * row + 1] = r_t + kLn2 * log2f(sum.st);
          }
        }
      }
    }
    __syncthreads();  // s_part is reused by the next task
  }
}

}  // namespace

hipError_t launch_forward_rows(const RowParams& p, const RowTiling& t, hipStream_t s) {
  const long long tasks = (long long)p.n_rows * p.n_chunks;
  const int grid = (int)(tasks < kFwdGrid ? tasks : kFwdGrid);
  if (grid < 1) return hipSuccess;
  if (p.bf16 && t.ragged) rowfwd_kernel<true, 8, true><<<grid, kFwdThreads, 0, s>>>(p);
  else if (p.bf16) rowfwd_kernel<true, 8, false><<<grid, kFwdThreads, 0, s>>>(p);
  else if (t.ragged) rowfwd_kernel<false, 4, true><<<grid, kFwdThreads, 0, s>>>(p);
  else rowfwd_kernel<false, 4, false><<<grid, kFwdThreads, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace turnkl
