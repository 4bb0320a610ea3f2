// Top-K reverse KL: the teacher's top-K support S_i of each token, both
// distributions renormalised on it (the paper trains with a top-K reverse KL,
// App. D; Sec. 3, Eq. opd-rkl restricted to S_i):
//   p^_s(v) = exp(a_v) / sum_{u in S_i} exp(a_u),  p^_t likewise from the
//   teacher's values b_v on S_i,
//   KL_i = sum_{v in S_i} p^_s(v) d_v,  d_v = log p^_s(v) - log p^_t(v),
//   dKL_i/da_v = p^_s(v) (d_v - KL_i) on S_i, 0 elsewhere.
//
// topk_rows   one wave per token: gathers the K student logits at the
//             support ids (one scattered load per id), reduces max and sum
//             of both distributions with wave shuffles, writes KL_i and
//             grad_scale * w_i * dKL_i/da on the support to the stage (the
//             caller's sparse output, or the workspace);
// topk_fill   (three forms) zero-fills the vocab columns of every dense
//             gradient row with 16-byte stores;
// topk_scatter  writes the staged support values of each supervised row.
//
// Order.  An out-of-place dense gradient is zero-filled first, and topk_rows
// then writes the support values into it directly (no scatter kernel, no
// staging round trip).  In place, topk_rows reads every student logit and
// stages the values, then the fill and the scatter overwrite the rows.

#include <hip/hip_bf16.h>

#include <type_traits>

#include "block_ops.h"
#include "turnkl_internal.h"

// No implicit FMA contraction: identical student and teacher values must give
// bit-identical halves of each difference (exactly zero KL and gradient).
#pragma clang fp contract(off)

namespace turnkl {
namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / kWave;

__device__ inline float load_logit(const void* base, long long i, bool bf16) {
  if (bf16) {
    const unsigned short u = static_cast<const unsigned short*>(base)[i];
    return __uint_as_float((unsigned)u << 16);
  }
  return static_cast<const float*>(base)[i];
}

__device__ inline float wave_max_f(float v) { return wave_max(v); }

// kPer support entries per lane (K <= 64 kPer), one row per wave.  The kernel is
// bound by a chain of latencies, mask, ids, gathers and stores; many short waves
// hide it better than fewer with several rows each, whose loads were issued
// together (65,536 rows, K = 50, whole sparse call, one sweep: 85 us with one row
// per wave, 88 with two, 95 with four, 107 with eight; 4,000 rows: 26, 27, 30 and
// 37.  With the benchmark's batch and inputs the first takes 95 to 99).
// The scaled gradient on the support goes to the stage (when there is one) and,
// with p.direct, straight into a zero-filled, out-of-place dense gradient.
template <int kPer>
__global__ __launch_bounds__(kThreads) void topk_rows(TopkParams p) {
  const int lane = threadIdx.x & (kWave - 1);
  const long long wave0 = (long long)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
  const long long stride = (long long)gridDim.x * kWavesPerBlock;
  // the first row's mask is on its way while the error key is awaited
  bool sup = wave0 < p.n_rows && p.mask[wave0];
  if (p.hdr->err_key != kNoError) return;
  for (long long row = wave0; row < p.n_rows; row += stride) {
    if (row != wave0) sup = p.mask[row];
    float* stage = p.stage ? p.stage + row * p.ld_stage : nullptr;
    if (!sup) {
      if (stage && p.zero_masked_stage)
        for (int j = lane; j < p.k; j += kWave) stage[j] = 0.0f;
      if (p.lse && lane == 0) {  // the row is not read: no log-partition function
        p.lse[2 * row] = __builtin_nanf("");
        p.lse[2 * row + 1] = __builtin_nanf("");
      }
      continue;
    }
    bool bad = false, on[kPer];
    int id[kPer];
    float a[kPer], b[kPer];
    // ids, teacher values and the weight, then the student logits at the ids
    const float sc = p.wsc[row];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int j = lane + q * kWave;
      on[q] = j < p.k;
      id[q] = on[q] ? p.ids[row * p.ld_k + j] : 0;
      b[q] = on[q] ? p.vals[row * p.ld_k + j] : -INFINITY;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const bool in = id[q] >= 0 && id[q] < p.vocab;
      bad = bad || (on[q] && !in);
      on[q] = on[q] && in;
      a[q] = on[q] ? load_logit(p.zs, row * p.ld_s + id[q], p.bf16) : -INFINITY;
      b[q] = on[q] ? b[q] : -INFINITY;
    }
    if (__ballot(bad) != 0ull) {
      if (lane == 0) atomicMin(&p.hdr->err_key, err_key(row, kPrioTopkId));
      continue;
    }
    float ma = -INFINITY, mb = -INFINITY;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      ma = fmaxf(ma, a[q]);
      mb = fmaxf(mb, b[q]);
    }
    ma = wave_max_f(ma);
    mb = wave_max_f(mb);
    float sa = 0.0f, sb = 0.0f;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      sa += on[q] ? expf(a[q] - ma) : 0.0f;
      sb += on[q] ? expf(b[q] - mb) : 0.0f;
    }
    sa = wave_sum(sa);
    sb = wave_sum(sb);
    const float la = logf(sa);
    const float lb = logf(sb);
    float d[kPer], pr[kPer];
    float kl = 0.0f;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const float xa = a[q] - ma;
      d[q] = on[q] ? ((xa - (b[q] - mb)) - (la - lb)) : 0.0f;
      pr[q] = on[q] ? expf(xa - la) : 0.0f;
      kl = fmaf(pr[q], d[q], kl);
    }
    kl = wave_sum(kl);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int j = lane + q * kWave;
      if (j >= p.k) continue;
      const float g = sc * (pr[q] * (d[q] - kl));
      if (stage) stage[j] = g;
      if (p.direct && on[q]) {
        if (p.bf16) {
          reinterpret_cast<__hip_bfloat16*>(p.grad)[row * p.ld_g + id[q]] = __float2bfloat16(g);
        } else {
          reinterpret_cast<float*>(p.grad)[row * p.ld_g + id[q]] = g;
        }
      }
    }
    if (lane == 0) {
      p.kl[row] = kl;
      if (p.lse) {  // log sum exp over the support = max + ln(sum)
        p.lse[2 * row] = ma + la;
        p.lse[2 * row + 1] = mb + lb;
      }
    }
  }
}

// Zero-fill of the dense gradient, bound by HBM writes.  One 16-byte store per
// thread, 4 KiB per workgroup, workgroups in address order: the stores in
// flight then cover one moving window of a few MiB, which the memory writes at
// 6.75 TB/s (19.9 GB).  Fewer, longer-lived workgroups spread the window over
// the whole matrix and lose DRAM page locality: a grid-stride loop over 32,768
// workgroups reaches 5.7 TB/s, two stores per thread 6.0, four 5.9.  The
// stores are nontemporal: default stores fill slightly faster (6.85 TB/s) but
// leave dirty lines that the support values' stores then wait for (4,166 rows
// of 32,000 in bf16: 110 us a call, nontemporal 90, 94 before; 16,384 rows of
// 151,936: 838, 801 and 892; 6,000 of 50,257: 171, 144 and 209).
//
// Out of place the fill does not look at the error key: a load before the
// store would hold each short workgroup, and the gradient of a call with a
// data error is unspecified.  In place it must not overwrite the logits then.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr long long kFillBlocks = 1 << 23;  // a launch holds fewer than 2^32 threads

// Rows without padding between them: `n_packs` 16-byte packs from p.grad
// rounded up to one, and the elements before and after them.
template <bool kBf16>
__global__ __launch_bounds__(kThreads) void topk_fill_flat(TopkParams p, long long head, long long n_packs,
                                                           long long n_elems) {
  using E = typename std::conditional<kBf16, unsigned short, float>::type;
  constexpr int kEpv = 16 / (int)sizeof(E);
  if (!p.direct && p.hdr->err_key != kNoError) return;
  E* const g = static_cast<E*>(p.grad);
  const long long i0 = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (i0 < kEpv) {
    if (i0 < head) g[i0] = E(0);
    const long long tail = head + n_packs * kEpv + i0;
    if (tail < n_elems) g[tail] = E(0);
  }
  const u32x4 z = {0u, 0u, 0u, 0u};
  for (long long i = i0; i < n_packs; i += (long long)gridDim.x * kThreads)  // one turn up to kFillBlocks
    __builtin_nontemporal_store(z, reinterpret_cast<u32x4*>(g + head) + i);
}

// Rows at any stride and start, at least one pack long: `per_row` packs each, on
// the grid of the row's address & ~line; a pack that sticks out of the row is
// moved inside it (its neighbour's elements are zeroed twice).  The workgroups
// take the packs of all rows in order, so that short rows fill them too: 65,536
// bf16 rows of 250 at a stride of 256 take 71 us a call, 90 with workgroups of
// their own for every row.
// kStream: nontemporal, as above; matrices that the last-level cache holds are
// filled with default stores instead (see kCachedFill).
typedef unsigned u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
template <bool kBf16, bool kStream>
__global__ __launch_bounds__(kThreads) void topk_fill_rows(TopkParams p, unsigned per_row, unsigned line,
                                                           long long packs) {
  constexpr int kEs = kBf16 ? 2 : 4;
  constexpr int kEpv = 16 / kEs;
  if (!p.direct && p.hdr->err_key != kNoError) return;
  const u32x4_any z = {0u, 0u, 0u, 0u};
  for (long long i = (long long)blockIdx.x * kThreads; i < packs;
       i += (long long)gridDim.x * kThreads) {  // one turn up to kFillBlocks
    const long long row0 = i / per_row;
    unsigned q = (unsigned)(i - row0 * per_row) + threadIdx.x;
    const unsigned more = q / per_row;
    q -= more * per_row;
    if (row0 + more >= p.n_rows) continue;
    char* const g = static_cast<char*>(p.grad) + (row0 + more) * p.ld_g * kEs;
    const int pre = (int)((unsigned)reinterpret_cast<uintptr_t>(g) & line) / kEs;
    int e = (int)q * kEpv - pre;
    if (e <= -kEpv || e >= p.vocab) continue;
    e = e < 0 ? 0 : (e > p.vocab - kEpv ? p.vocab - kEpv : e);
    u32x4_any* const at = reinterpret_cast<u32x4_any*>(g + (long long)e * kEs);
    if (kStream) __builtin_nontemporal_store(z, at);
    else *at = z;
  }
}

// Bytes up to which rows at a stride are filled through the caches, out of place
// and in place (where the rows' logits have just been read).  30,000 bf16 rows of
// 3,000 at 3,001, 180 MB: 89 us a call, 99 nontemporal (in place 93, 114); 65,536
// of 2,000, 262 MB: 139, 133 (141, 154); 65,536 of 3,000, 393 MB: 213, 171 (183,
// 197); 65,536 fp32 rows of 2,000 at 2,003, 525 MB: 277, 176 (240, 203).
constexpr double kCachedFill = 192.0 * (1 << 20);
constexpr double kCachedFillInPlace = 384.0 * (1 << 20);

// Rows shorter than a pack, with padding between them.
template <bool kBf16>
__global__ __launch_bounds__(kThreads) void topk_fill_short(TopkParams p) {
  using E = typename std::conditional<kBf16, unsigned short, float>::type;
  if (p.hdr->err_key != kNoError) return;
  const long long row = (long long)blockIdx.x * kThreads + threadIdx.x;  // at most 2^31 rows
  if (row >= p.n_rows) return;
  E* const g = static_cast<E*>(p.grad) + row * p.ld_g;
  for (int v = 0; v < p.vocab; ++v) g[v] = E(0);
}

// Scatter of the staged support values into the zero-filled rows of
// supervised tokens (in place: the rows were read before the fill), kRows
// rows per wave with their loads issued together; runs after topk_fill on
// the stream.
template <bool kBf16, int kRows>
__global__ __launch_bounds__(kThreads) void topk_scatter(TopkParams p) {
  if (p.hdr->err_key != kNoError) return;
  const int lane = threadIdx.x & (kWave - 1);
  const long long wave0 = (long long)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
  const long long stride = (long long)gridDim.x * kWavesPerBlock;
  for (long long r0 = wave0 * kRows; r0 < p.n_rows; r0 += stride * kRows) {
    for (int j0 = 0; j0 < p.k; j0 += kWave) {
      const int j = j0 + lane;
      bool on[kRows];
      int id[kRows];
      float x[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const long long row = r0 + r;
        on[r] = row < p.n_rows && j < p.k && p.mask[row];
        id[r] = on[r] ? p.ids[row * p.ld_k + j] : 0;
        x[r] = on[r] ? p.stage[row * p.ld_stage + j] : 0.0f;
      }
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        if (!on[r] || id[r] < 0 || id[r] >= p.vocab) continue;  // bad ids: reported by topk_rows
        const long long at = (r0 + r) * p.ld_g + id[r];
        if (kBf16) reinterpret_cast<__hip_bfloat16*>(p.grad)[at] = __float2bfloat16(x[r]);
        else reinterpret_cast<float*>(p.grad)[at] = x[r];
      }
    }
  }
  drain_stores();
}

int grid_for(long long items, int per_block, int cap) {
  long long g = (items + per_block - 1) / per_block;
  if (g < 1) g = 1;
  return (int)(g < cap ? g : cap);
}

dim3 fill_grid(long long blocks) {
  return dim3((unsigned)(blocks < kFillBlocks ? blocks : kFillBlocks));
}

template <bool kBf16>
void launch_fill(const TopkParams& p, hipStream_t s) {
  constexpr int kEs = kBf16 ? 2 : 4;
  constexpr int kEpv = 16 / kEs;
  const long long elems = (long long)p.n_rows * p.vocab;
  // elements before the first 16-byte boundary (none when no element starts on one)
  const long long head = (long long)((16 - ((uintptr_t)p.grad & 15u)) & 15u) / kEs;
  if ((p.ld_g == p.vocab || p.n_rows == 1) && (uintptr_t)p.grad % kEs == 0 && elems >= 2 * kEpv) {
    const long long packs = (elems - head) / kEpv;
    topk_fill_flat<kBf16><<<fill_grid((packs + kThreads - 1) / kThreads), kThreads, 0, s>>>(
        p, head, packs, elems);
  } else if (p.vocab >= kEpv) {
    // on the lines' grid (then also the packs of a row that starts at the end of
    // one), unless its up to eight more packs weigh
    const bool lines = p.vocab >= 64 * kEpv;
    const unsigned per_row = (unsigned)(((lines ? 127 / kEs : 0) + (long long)p.vocab + kEpv - 1) / kEpv);
    const long long packs = (long long)p.n_rows * per_row;
    const dim3 grid = fill_grid((packs + kThreads - 1) / kThreads);
    const unsigned line = lines ? 127u : 0u;
    if ((double)elems * kEs <= (p.direct ? kCachedFill : kCachedFillInPlace))
      topk_fill_rows<kBf16, false><<<grid, kThreads, 0, s>>>(p, per_row, line, packs);
    else
      topk_fill_rows<kBf16, true><<<grid, kThreads, 0, s>>>(p, per_row, line, packs);
  } else {
    topk_fill_short<kBf16><<<dim3((unsigned)((p.n_rows + kThreads - 1) / kThreads)), kThreads, 0, s>>>(p);
  }
}

}  // namespace

hipError_t launch_topk_rows(const TopkParams& p, hipStream_t s) {
  if (p.n_rows == 0) return hipSuccess;
  const int per = (p.k + kWave - 1) / kWave;
#define TURNKL_TOPK(n)                                                                     \
  case n:                                                                                  \
    topk_rows<n><<<grid_for(p.n_rows, kWavesPerBlock, 1 << 20), kThreads, 0, s>>>(p);      \
    break;
  switch (per <= 1 ? 1 : per <= 2 ? 2 : per <= 4 ? 4 : per <= 8 ? 8 : 16) {
    TURNKL_TOPK(1) TURNKL_TOPK(2) TURNKL_TOPK(4) TURNKL_TOPK(8) TURNKL_TOPK(16)
    default: return hipErrorInvalidValue;
  }
#undef TURNKL_TOPK
  return hipGetLastError();
}

hipError_t launch_topk_fill(const TopkParams& p, hipStream_t s) {
  if (p.n_rows == 0 || !p.grad) return hipSuccess;
  if (p.bf16) launch_fill<true>(p, s);
  else launch_fill<false>(p, s);
  return hipGetLastError();
}

hipError_t launch_topk_scatter(const TopkParams& p, hipStream_t s) {
  if (p.n_rows == 0 || !p.grad) return hipSuccess;
  constexpr int kRows = 4;
  const int grid = grid_for(p.n_rows, kWavesPerBlock * kRows, 16384);
  if (p.bf16) topk_scatter<true, kRows><<<grid, kThreads, 0, s>>>(p);
  else topk_scatter<false, kRows><<<grid, kThreads, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace turnkl
