// Device-side helpers for the gfx950 kernels: fixed-order reductions and scans
// over 64-lane wavefronts, and the counter-based gradient generator.
#pragma once
#include "evg_internal.h"

namespace evg {

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }
__device__ __forceinline__ uint32_t wave_id() { return threadIdx.x >> 6; }

// The iteration number and decay^k of the step in flight (uniform loads).
__device__ __forceinline__ uint32_t step_k(const Tables& T, const StepArgs& A) {
  return A.from_device ? T.it->k : A.k;
}
__device__ __forceinline__ double step_decay(const Tables& T, const StepArgs& A) {
  return A.from_device ? T.it->decay_pow : A.decay_pow;
}

// Streaming (non-temporal) 16-byte accesses: every arena is far larger than the
// caches and is touched once per pass, so lines are not worth keeping.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ld4s(const float* p) {
  const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st4s(float* p, float4 a) {
  f32x4 v;
  v.x = a.x; v.y = a.y; v.z = a.z; v.w = a.w;
  __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// `bytes` bytes of memory as a buffer: lanes past them read zeros and write nothing, so a ragged end, an array that
// is not wanted this time (bytes = 0) and a lane that has nothing to write all take the same instructions,
// without a branch around a memory access (the compiler waits for a load before it leaves its branch).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t window(const void* at, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(at), 0, (int)bytes, 0x00027000);
}
// Sum over the 64 lanes by xor butterflies: every lane ends with the same value,
// and the association order is fixed, so results repeat bit for bit.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sum over a 256-thread workgroup; valid in every thread.  `ws` is 4 doubles of LDS.
__device__ __forceinline__ double block_sum(double v, double* ws) {
  v = wave_sum(v);
  if (lane_id() == 0) ws[wave_id()] = v;
  __syncthreads();
  const double total = ((ws[0] + ws[1]) + ws[2]) + ws[3];
  __syncthreads();
  return total;
}

// Inclusive prefix sum over the 64 lanes with data-parallel-primitive moves, no LDS traffic:
// shifted adds by 1, 2, 4, 8 inside each row of 16 lanes (lanes shifted in from outside a row
// read 0), then the last lane of rows 0 and 2 is added to rows 1 and 3, and lane 31 (by then the
// sum of rows 0-1) to rows 2 and 3.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);   // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);   // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, true);   // row_bcast:15 -> rows 1, 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, true);   // row_bcast:31 -> rows 2, 3
  return v;
}

// Exclusive prefix sum over the threads of a workgroup of W wavefronts (thread
// order); *total receives the workgroup sum.  `ws` is W uint32 of LDS.
template <int W>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* ws, uint32_t* total) {
  const uint32_t incl = wave_incl_scan(v);
  if (lane_id() == 63) ws[wave_id()] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const uint32_t s = ws[w];
    if ((uint32_t)w < wave_id()) before += s;
    all += s;
  }
  __syncthreads();
  *total = all;
  return before + incl - v;
}

// The same accesses with the choice left to the caller: a ring whose arenas fit the
// last-level cache is better served by ordinary cached accesses (measured 10 % per step
// on an 8-worker ResNet-20-sized ring).
template <bool STREAM>
__device__ __forceinline__ float4 ld4t(const float* p) {
  if (STREAM) return ld4s(p);
  return *reinterpret_cast<const float4*>(p);
}
template <bool STREAM>
__device__ __forceinline__ void st4t(float* p, float4 a) {
  if (STREAM) st4s(p, a);
  else *reinterpret_cast<float4*>(p) = a;
}

// Workers at the ends of a part of the ring (parts of A.part workers; one part: none).
__device__ __forceinline__ bool is_led(const Tables& T, const StepArgs& A, uint32_t s) {
  return A.part < T.P && (s % A.part == 0 || s % A.part == A.part - 1 || s == T.P - 1);
}

// The whole-tensor send of one chunk, by one workgroup.
// HAT = false: the two mailboxes (xhat takes the sent values in the update pass, which has them
// in registers).  HAT = true: xhat alone -- the receivers read it there in the update pass and
// store it into their mailboxes.
template <int SWEEPS, bool STREAM, bool HAT>
__device__ __forceinline__ void copy_chunk(const Tables& T, uint32_t r, const ChunkDesc& cd) {
  const uint32_t left = (r + T.P - 1) % T.P, right = (r + 1) % T.P;
  const float* src = T.x + (size_t)r * T.Npad + cd.off;
  float* d1 = HAT ? T.xhat + (size_t)r * T.Npad + cd.off : T.mbox_r + (size_t)left * T.Npad + cd.off;
  float* d2 = T.mbox_l + (size_t)right * T.Npad + cd.off;
#pragma unroll
  for (int it = 0; it < SWEEPS; ++it) {
    const uint32_t e = it * kSweep + threadIdx.x * kLaneElems - cd.lead;   // positions before the lead wrap around
    if (e < cd.len) {
      const float4 v = ld4t<STREAM>(src + e);
      st4t<STREAM>(d1 + e, v);
      if (!HAT) st4t<STREAM>(d2 + e, v);
    }
  }
}

// ----------------------------------------------------------------------------
// Synthetic gradients.  Philox4x32-10 (Salmon et al., SC'11): ten rounds, each
// two 32x32->64 multiplies by fixed odd constants followed by xors with the
// neighbouring words and the round key; the key advances by Weyl constants.
// ----------------------------------------------------------------------------
//
// Every transcendental step below is a fixed chain of correctly rounded operations, so that it
// gives the same bits on any IEEE machine.  The chains run on the ranges the generator feeds them
// (uniforms are odd multiples of 2^-24), which lets quotients and roots do without the scaling and
// special cases of the general operators: a hardware estimate and one correction by fused
// multiply-adds rounds as they do.  An input is 23 random bits: over all 2^23 of them a correctly rounded
// estimate never leaves a difference, and one that is off by its last bit (the estimates' accuracy) does at
// 7 of them for the normal's radius, 9 for the Student-t's (tests/test_generator_estimates.py, which also draws
// those on the GPU).  Angle and uniform take no estimate.  Cycles per wavefront for four variates, Philox
// included: normal 779 -> 530, Student-t 1737 -> 1265.
struct Rand4 { uint32_t w[4]; };

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);   // the compiler leaves two xors (248 -> 197 cycles per block)
}

__device__ __forceinline__ Rand4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                        uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t y0 = xor3(hi1, c1, k0), y2 = xor3(hi0, c3, k1);
    c0 = y0; c1 = lo1; c2 = y2; c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  Rand4 r;
  r.w[0] = c0; r.w[1] = c1; r.w[2] = c2; r.w[3] = c3;
  return r;
}

// Top 23 bits n to (n + 1/2) 2^-23, a float in (0,1); exact: 1 + n 2^-23 is put together from its
// bits, and the difference to 1 - 2^-24 has 24 significant bits.
__device__ __forceinline__ float unit_open(uint32_t w) {
  return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, w, 9u)) - 0.99999994f;
}

// Square root of a normal number: estimate, one Newton step on the root and its reciprocal.
__device__ __forceinline__ float root(float a, float estimate_at) {
  const float y = __builtin_amdgcn_rsqf(estimate_at);
  const float g = a * y, h = 0.5f * y;
  return __builtin_fmaf(__builtin_fmaf(-g, g, a), h, g);
}

// F * log(u) of a normal positive float u, F = -1 or -2 (a power of two rounds nothing differently):
// split off the exponent, fold the mantissa m into (sqrt(1/2), sqrt(2)] (0x3F3504F4 is the smallest
// float of the lower half), then the odd series of 2 atanh((m-1)/(m+1)).
template <int F>
__device__ __forceinline__ float ln_series(float u) {
  const uint32_t b = __float_as_uint(u);
  const int ne = (int)(0x3F3504F4u + 0x7FFFFFu - b) >> 23;            // minus the exponent
  const float m = __uint_as_float(((uint32_t)ne << 23) + b);
  const float t = m - 1.0f, d = m + 1.0f;
  const float r = __builtin_amdgcn_rcpf(d), q = t * r;
  const float s = __builtin_fmaf(__builtin_fmaf(-d, q, t), r, q);     // t / d
  const float w = s * s;
  float p = __builtin_fmaf(w, 0.111111112f, 0.142857149f);
  p = __builtin_fmaf(w, p, 0.2f);
  p = __builtin_fmaf(w, p, 0.333333343f);
  p = __builtin_fmaf(w, p, 1.0f);
  return __builtin_fmaf((float)ne, -F * 0.693147182f, (2 * F * s) * p);
}

// (cos, sin)(2 pi u), u = (n + 1/2) 2^-23 with n the word's top 23 bits: the nearest quarter turn is
// the top two bits of the word plus an eighth of a turn, what remains is exact, and so is its
// distance to that quarter turn; Taylor series on [-pi/4, pi/4].
__device__ __forceinline__ void turn_cos_sin(uint32_t word, float& c, float& s) {
  const uint32_t z = word + 0x20000000u;
  const uint32_t n = __builtin_amdgcn_ubfe(z, 9u, 21u);
  const float r = __uint_as_float((n << 2) | 0x3F800000u) - 1.49999976f;   // (n + 1/2) 2^-21 - 1/2
  const float th = r * 1.57079637f;
  const float q = th * th;
  float sp = __builtin_fmaf(q, 2.75573192e-6f, -1.98412701e-4f);
  sp = __builtin_fmaf(q, sp, 8.33333377e-3f);
  sp = __builtin_fmaf(q, sp, -0.166666672f);
  sp = __builtin_fmaf(q, sp, 1.0f);
  const float sn = th * sp;
  float cp = __builtin_fmaf(q, -2.75573188e-7f, 2.48015876e-5f);
  cp = __builtin_fmaf(q, cp, -1.38888892e-3f);
  cp = __builtin_fmaf(q, cp, 4.16666679e-2f);
  cp = __builtin_fmaf(q, cp, -0.5f);
  const float cs = __builtin_fmaf(q, cp, 1.0f);
  // quarter turns: odd ones swap the two series; the signs follow from the quadrant
  // (cos is negated in quadrants 1 and 2, sin in 2 and 3): a ^ (b & sign bit)
  const bool swap = (int)(z << 1) < 0;
  c = __uint_as_float(__builtin_amdgcn_bitop3_b32(__float_as_uint(swap ? sn : cs), z + 0x40000000u, 0x80000000u, 0x78));
  s = __uint_as_float(__builtin_amdgcn_bitop3_b32(__float_as_uint(swap ? cs : sn), z, 0x80000000u, 0x78));
}

// Box-Muller on words (0,1) and (2,3): radius from the first, angle from the second.
__device__ __forceinline__ void normals4(const Rand4& r, float z[4]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float a = ln_series<-2>(unit_open(r.w[2 * h]));    // at least 2^-23
    const float rad = root(a, a);
    float c, s;
    turn_cos_sin(r.w[2 * h + 1], c, s);
    z[2 * h] = rad * c;
    z[2 * h + 1] = rad * s;
  }
}

// e^y for 0 <= y < 80 with only + * fma: the nearest multiple n of ln 2 is taken out in two
// parts (high and low word of ln 2), the remainder's exponential is its Taylor polynomial of
// degree six, and 2^n is added into the exponent field.
__device__ __forceinline__ float exp_series(float y) {
  const int n = (int)(y * 1.44269502f + 0.5f);
  const float nf = (float)n;
  const float r = __builtin_fmaf(-nf, 1.42860677e-6f, __builtin_fmaf(-nf, 0.693145752f, y));
  float p = __builtin_fmaf(r, 1.38888892e-3f, 8.33333377e-3f);
  p = __builtin_fmaf(r, p, 4.16666679e-2f);
  p = __builtin_fmaf(r, p, 0.166666672f);
  p = __builtin_fmaf(r, p, 0.5f);
  p = __builtin_fmaf(r, p, 1.0f);
  p = __builtin_fmaf(r, p, 1.0f);
  return __uint_as_float(__float_as_uint(p) + ((uint32_t)n << 23));
}

// Student-t with 3 degrees of freedom from two random words by the polar method (Bailey 1994):
// a spherical bivariate t has squared radius 3 (u^(-2/3) - 1) for a uniform u, and its first
// component, radius times the cosine of a uniform angle, is Student-t(3).
__device__ __forceinline__ float student_t3(uint32_t wr, uint32_t wa) {
  const float y = 0.666666687f * ln_series<-1>(unit_open(wr));
  const float a = 3.0f * (exp_series(y) - 1.0f);             // 0 for the largest u: a finite estimate keeps the root 0
  const float rad = root(a, __builtin_fmaxf(a, 1e-30f));
  float c, s;
  turn_cos_sin(wa, c, s);
  return rad * c;
}

// The gradient of four consecutive elements, the first of them element j of its tensor: variates
// times sg (sigma of the tensor at this iteration), times the gain where the worker has a spike.
// DIST 0: normal, one Philox block per four elements.  DIST 1: Student-t(3), two blocks: variate i takes
// words 2i (radius) and 2i+1 (angle) of the eight.
template <int DIST>
__device__ __forceinline__ void draw_gradient(const StepArgs& A, uint32_t j, uint32_t layer, uint32_t k, uint32_t r,
                                              float sg, bool spike, float g[4]) {
  if (DIST == 0) {
    float z[4];
    normals4(philox(j >> 2, layer, k, r, A.key0, A.key1), z);
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = sg * z[i];
  } else {
    const uint32_t b0 = (j >> 2) << 1;
    const Rand4 ra = philox(b0, layer, k, r, A.key0, A.key1);
    const Rand4 rb = philox(b0 + 1u, layer, k, r, A.key0, A.key1);
    g[0] = sg * student_t3(ra.w[0], ra.w[1]);
    g[1] = sg * student_t3(ra.w[2], ra.w[3]);
    g[2] = sg * student_t3(rb.w[0], rb.w[1]);
    g[3] = sg * student_t3(rb.w[2], rb.w[3]);
  }
  if (spike) {
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = g[i] * A.spike_gain;
  }
}

// Does worker r have a spike in iteration k?
__device__ __forceinline__ bool has_spike(const StepArgs& A, uint32_t k, uint32_t r) {
  return A.spike_prob > 0.0f && unit_open(philox(0u, 0xFFFFFFFFu, k, r, A.key0, A.key1).w[0]) < A.spike_prob;
}

// Squared drift of the first nv lanes of a float4 pair, added in lane order.
__device__ __forceinline__ void drift_acc(double& acc, const float x[4], const float h[4], uint32_t nv) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if ((uint32_t)i < nv) {
      const float e = x[i] - h[i];
      acc += (double)e * (double)e;
    }
  }
}

// Sum of squares of the first nv lanes, added in lane order.
__device__ __forceinline__ void square_acc(double& acc, const float x[4], uint32_t nv) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if ((uint32_t)i < nv) acc += (double)x[i] * (double)x[i];
}

// Key that ranks elements for Top-K: the bit pattern of a non-negative float is
// monotone in its value, so unsigned compares order magnitudes.
__device__ __forceinline__ uint32_t rank_key(float xv, float hv, uint32_t by_value) {
  return __float_as_uint(__builtin_fabsf(by_value ? xv : xv - hv));
}

}  // namespace evg
