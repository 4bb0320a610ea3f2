// What the kernels over whole rows share: 16-byte packs of logits, the partial
// sums of a chunk of a row and their merge.
#pragma once

#include <hip/hip_bf16.h>

#include "block_ops.h"
#include "turnkl_internal.h"

// No implicit FMA contraction in the kernels over rows: every fused multiply-add the
// kernel wants is written as fmaf.  Contraction would evaluate the student
// and teacher halves of a difference asymmetrically (x*c - y*c becoming
// fma(x, c, -(y*c)) leaves the rounding error of y*c when x == y), so
// identical logits would no longer give exactly zero KL and gradient.
#pragma clang fp contract(off)

namespace turnkl {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// Reference magnitude (log2 units, i.e. logits times log2 e) above which a
// chunk, and then its row, subtracts its references per element.  Below it
// the fast path's error term, a few u |m_s - m_t|, stays under 1e-5.
constexpr float kFar2 = 64.0f * kLog2e;
// Sums against sampled references above which a chunk (or wave) is redone
// against its exact maxima: all of a row's chunks and waves, at most 512 of
// them, then add up inside the float range.  The sum of 2^(..) (a - b) counts
// too: it leaves the range a few units of logits before the sum of 2^(..).
constexpr float kMaxSum = 0x1p118f;

// ---------------------------------------------------------------------------
// packs of kEpv elements moved with one load/store

// Buffer resource over one row chunk (gfx9 dword-3 word for raw dword
// access).  The base is wave-uniform, so each pack's offset splits into a
// per-lane VGPR part and a compile-time SGPR step.
constexpr int kRsrcWord3 = 0x00020000;

// Cache policy of the logit loads and gradient stores: non-temporal (the nt
// bit of gfx940-family buffer instructions).  Every logit is read once and
// every gradient element written once, so nothing is gained by keeping them
// in L2; streaming them measured about 3% faster than the default policy.
constexpr int kStream = 2;

__device__ inline __amdgpu_buffer_rsrc_t chunk_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7FFFFFFF, kRsrcWord3);
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Store data must stay untouched for a while after a 16-byte store is
// issued: on gfx950 the store can read its data registers later than the
// compiler's wait states assume, so a register reused right after the store
// (observed: the first data dword) lands in memory.  The row kernel pins each
// store in program order and keeps its data live (keep_alive) across the next
// pack's work, or across the end-of-task barrier for the last pack.
__device__ inline void keep_alive(const u32x4& x) { asm volatile("" ::"v"(x)); }
__device__ inline void keep_alive(unsigned x) { asm volatile("" ::"v"(x)); }

template <bool kBf16, int kEpv>
struct Pack;

template <>
struct Pack<true, 8> {  // 8 bf16 = 16 bytes
  using Data = u32x4;
  unsigned w[4];
  __device__ void load(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    const auto u = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, kStream);
    w[0] = u[0]; w[1] = u[1]; w[2] = u[2]; w[3] = u[3];
  }
  // Opaque to the optimiser: values unpacked before the fence cannot be
  // reused after it, so only the packed words stay live between passes.
  __device__ void fence() { asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3])); }
  __device__ float get(int j) const {
    const unsigned x = w[j >> 1];
    return __uint_as_float((j & 1) ? (x & 0xFFFF0000u) : (x << 16));
  }
  // Round to bf16 (nearest even, v_cvt_pk_bf16_f32); flip = 0x80008000
  // negates both halves of every word.
  __device__ static Data encode(const float (&g)[8], unsigned flip) {
    Data o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const f32x2 x = {g[2 * k], g[2 * k + 1]};
      o[k] = __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2)) ^ flip;
    }
    return o;
  }
  __device__ static Data zero() { return Data{0u, 0u, 0u, 0u}; }
  __device__ static void store(__amdgpu_buffer_rsrc_t r, int voff, int soff, const Data& o) {
    __builtin_amdgcn_raw_buffer_store_b128(o, r, voff, soff, kStream);
  }
};

template <>
struct Pack<false, 4> {  // 4 fp32 = 16 bytes
  using Data = u32x4;
  float f[4];
  __device__ void load(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    const auto u = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, kStream);
    f[0] = __uint_as_float(u[0]); f[1] = __uint_as_float(u[1]);
    f[2] = __uint_as_float(u[2]); f[3] = __uint_as_float(u[3]);
  }
  __device__ void fence() { asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3])); }
  __device__ float get(int j) const { return f[j]; }
  __device__ static Data encode(const float (&g)[4], unsigned flip) {
    const unsigned fl = flip << 16;  // sign bit of an fp32
    Data o;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = __float_as_uint(g[k]) ^ fl;
    return o;
  }
  __device__ static Data zero() { return Data{0u, 0u, 0u, 0u}; }
  __device__ static void store(__amdgpu_buffer_rsrc_t r, int voff, int soff, const Data& o) {
    __builtin_amdgcn_raw_buffer_store_b128(o, r, voff, soff, kStream);
  }
};

template <>
struct Pack<true, 1> {  // one bf16
  using Data = unsigned;
  unsigned w;
  __device__ void load(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    w = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, kStream);
  }
  __device__ void fence() { asm volatile("" : "+v"(w)); }
  __device__ float get(int) const { return __uint_as_float(w << 16); }
  __device__ static Data encode(const float (&g)[1], unsigned flip) {
    const f32x2 x = {g[0], 0.0f};
    return (__builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2)) ^ flip) & 0xFFFFu;
  }
  __device__ static Data zero() { return 0u; }
  __device__ static void store(__amdgpu_buffer_rsrc_t r, int voff, int soff, const Data& o) {
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)o, r, voff, soff, kStream);
  }
};

template <>
struct Pack<false, 1> {  // one fp32
  using Data = unsigned;
  float f;
  __device__ void load(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    f = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, kStream));
  }
  __device__ void fence() { asm volatile("" : "+v"(f)); }
  __device__ float get(int) const { return f; }
  __device__ static Data encode(const float (&g)[1], unsigned flip) {
    return __float_as_uint(g[0]) ^ (flip << 16);
  }
  __device__ static Data zero() { return 0u; }
  __device__ static void store(__amdgpu_buffer_rsrc_t r, int voff, int soff, const Data& o) {
    __builtin_amdgcn_raw_buffer_store_b32(o, r, voff, soff, kStream);
  }
};

// one gradient element, as a pack of one element stores it
template <bool kBf16>
__device__ inline void store_one(__amdgpu_buffer_rsrc_t r, int off, float g, unsigned flip) {
  const float x[1] = {g};
  Pack<kBf16, 1>::store(r, off, 0, Pack<kBf16, 1>::encode(x, flip));
}

__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Take a ticket: an atomic increment, which the compiler issues as one plain
// global atomic whose result is waited for only where it is used (an atomic
// add from one lane is rewritten into a wave-aggregated form that waits at
// once).
__device__ inline unsigned take_ticket(unsigned* counter) {
  return __builtin_amdgcn_atomic_inc32(counter, 0xFFFFFFFFu, __ATOMIC_RELAXED, "agent");
}

// Exchange words.  A chunk's seven partials (M_s, S_s, A, M_t, S_t, C_a, C_b)
// and its form tag (kTagFast / kTagOffset, how the partials are expressed)
// travel as four 64-bit words, (M_s, S_s), (A, M_t), (S_t, C_a), (C_b, tag),
// each published with one relaxed 64-bit atomic store and read back with
// relaxed 64-bit atomic loads.  A partial is stored as the bits of v + 0 (so
// -0 becomes +0) with the sign bit flipped, which is never zero; the slots
// are cleared before the kernel, so a nonzero word is a published one.
constexpr unsigned kTagFast = 1;
constexpr unsigned kTagOffset = 2;
__device__ inline unsigned enc(float v) { return __float_as_uint(v + 0.0f) ^ 0x80000000u; }
__device__ inline float dec(unsigned u) { return __uint_as_float(u ^ 0x80000000u); }
__device__ inline unsigned long long word2(unsigned lo, unsigned hi) {
  return ((unsigned long long)hi << 32) | (unsigned long long)lo;
}
// the seven partials of one chunk's four words, in publication order
__device__ inline void unpack_partials(const unsigned long long* w, float (&out)[kPartials]) {
#pragma unroll
  for (int i = 0; i < kPartials; ++i) {
    const unsigned long long x = w[i >> 1];
    out[i] = dec((i & 1) ? (unsigned)(x >> 32) : (unsigned)x);
  }
}

// The low half of the workspace's error key, read with a relaxed atomic
// load: an error key's low nibble is a priority below 15, so the half equals
// 0xFFFFFFFF exactly while no error has been recorded (a waiting workgroup
// polls it to learn that another one has timed out).
__device__ inline unsigned err_low(Header* hdr) {
  return __hip_atomic_load(reinterpret_cast<unsigned*>(&hdr->err_key), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
constexpr unsigned kNoErrorLow = 0xFFFFFFFFu;

// Row merge.  A chunk reports (M_s, S_s, A, M_t, S_t, C_a, C_b) in one of two
// forms:
//  fast (tag kTagFast): M in log2 units (logits times log2 e), C = (0, 0),
//    S_s = sum 2^(a log2e - M_s),  A = sum 2^(a log2e - M_s) (a - b),  S_t likewise;
//  offset (kTagOffset): M = the chunk's maxima in logit units, C = (a, b)
//    where the student's logit peaks in the chunk,
//    S_s = sum 2^((a - M_s) log2e),  A = sum 2^((a - M_s) log2e) ((a - b) - (C_a - C_b)),
//    with both differences taken exactly (two_diff), so a term is accurate
//    to a few ulps of its own size whatever the magnitude of the logits.
// The maxima are the references of the exponents; C is the reference of the
// difference a - b, taken where the student's probability mass sits, so that
// a spike in the teacher (which sets its maximum) does not inflate every
// other term, and a peaked row's KL does not come from cancelling terms.
// The row works against natural references (R_s, R_t) >= every chunk's
// reference and the difference reference C* of the offset chunk with the
// largest C_a, or (0, 0) where a fast chunk's reference lies above that (all
// chunks fast; or the offset ones hold masked logits, whose difference from the
// teacher's may be of any size), and accumulates in chunk order
//   S_s = sum_v 2^((a_v - R_s) log2e),  S_t likewise,
//   A   = sum_v 2^((a_v - R_s) log2e) ((a_v - b_v) - (C*_a - C*_b)),
// so that KL = A / S_s + ((C*_a - R_s) - (C*_b - R_t)) + ln(S_t / S_s).
// A fast chunk scales by 2^(M_s - R_s log2e) (one FMA for the exponent), an
// offset chunk by 2^((M_s - R_s) log2e); both add
// S_s ((C_a - C_b) - (C*_a - C*_b)) to A (exact differences), zero for rows of
// fast chunks only.  Where the scale is zero the chunk adds nothing to A: its
// own A, and S_s times the difference of the references, may be infinite.
struct RowSums {
  float ss, aa, st;
};

// whether a chunk's (or wave's) sums in the fast form may stand
__device__ inline bool sums_in_range(float ss, float aa, float st) {
  return ss + st + fabsf(aa) <= kMaxSum;  // false for NaN
}

// Error-free difference (Knuth's TwoSum applied to x + (-y)): hi = fl(x - y)
// and hi + lo = x - y exactly.  Needs plain rounded adds, which this file
// guarantees (no contraction).
struct Float2 {
  float hi, lo;
};
__device__ inline Float2 two_diff(float x, float y) {
  const float hi = x - y;
  const float yv = hi - x;   // the part of hi that came from -y
  const float xv = hi - yv;  // the part of hi that came from x
  return Float2{hi, (x - xv) - (y + yv)};
}

// (x - y) - c for a double-float c, to within a few ulps of the result even
// when x - y and c are large and nearly equal.
__device__ inline float diff_minus(float x, float y, Float2 c) {
  const Float2 d = two_diff(x, y);
  return (d.hi - c.hi) + (d.lo - c.lo);
}

// natural reference of a chunk: a logit-unit value at or above its own
__device__ inline float natural_ref(bool offset, float m) { return offset ? m : m * kLn2; }

__device__ inline void merge_chunk(bool offset, const float* w, float rs, float rt, Float2 c_row,
                                   RowSums& r) {
  float fs, ft;
  if (offset) {
    fs = exp2f((w[0] - rs) * kLog2e);
    ft = exp2f((w[3] - rt) * kLog2e);
  } else {
    fs = exp2f(fmaf(-rs, kLog2e, w[0]));
    ft = exp2f(fmaf(-rt, kLog2e, w[3]));
  }
  const float aa = fmaf(w[1], diff_minus(w[5], w[6], c_row), w[2]);
  r.ss = fmaf(w[1], fs, r.ss);
  r.aa = fs == 0.0f ? r.aa : fmaf(aa, fs, r.aa);
  r.st = fmaf(w[4], ft, r.st);
}

// Ragged rows (RowForm): where the pack of elements [e, e + kEpv) is read and
// written (`last`: the row's last whole pack), which of the elements there are
// its own when that is `shift` elements before e, and an all-ones mask for one.
__device__ inline int inside_row(int e, int last) { return e < 0 ? 0 : (e > last ? last : e); }
template <int kEpv>
__device__ inline unsigned own_bits(int shift) {
  constexpr unsigned kAll = (1u << kEpv) - 1u;
  const int s = shift < -kEpv ? -kEpv : (shift > kEpv ? kEpv : shift);
  return (s >= 0 ? kAll << s : kAll >> -s) & kAll;
}
__device__ inline unsigned own_mask(unsigned bits, int j) {
  return (unsigned)((int)(bits << (31 - j)) >> 31);
}

}  // namespace
}  // namespace turnkl
