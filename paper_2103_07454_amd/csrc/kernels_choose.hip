// The whole Top-K selection of one tensor by one workgroup, from the trigger test to the winners' places in the message: for rings
// that live in the last-level cache, whose steps are bound by the chain of launches (the test, the pass over the tensor and
// five more on what it stages took 31 us of 53 with 8 ResNet-20 workers, 27 of 37 with 5 perceptrons of 160 000 elements).
//
// The update pass has left a key code for each element, a byte, and has counted the 128 codes in whose middle the threshold is
// expected (one addition a lane and workgroup, where the histogram of all keys took a pass of its own through LDS).  The counts
// name the code of the K-th largest key; the workgroup goes through the codes once, lists what has that one (some 0.4 % of the
// tensor), fetches those keys alone and finds the threshold among them: a histogram of their upper ten bits leaves a key or a few, which
// every wavefront ranks for itself.  Where the counts do not reach it (a tensor's first
// message; it has moved by more than an octave down or three quarters of one up) the keys are read from the arenas, in four passes.
// Tensors of at most 256 elements are a wavefront's work.
//
// Bound by latency, and by the vector ALUs where a tensor is long.  A workgroup of a ResNet-20 ring of 8 workers (its longest tensors 36 864 elements) takes
// 6.7 us: its descriptor and everything asked for 0.7, sums, counts and codes there 1.1, the codes gone through 1.4 (160 000 elements:
// 4.6), keys fetched 1.7, the histogram 0.5, ranked and added to the groups 0.8, the groups' places 0.6.  The tests' outcome is booked while the keys are on
// their way.  Before, with descriptors in two tables, the test's threshold asked for behind its sums, bytes compared in halves of registers and two
// histograms with three barriers each, 24 000 cycles.  The launch 15.8 -> 10.2 us, 160 000 elements 21.5 -> 14.4; steps: 8 ResNet-20 workers, 10 % 32.3 -> 26.8 us,
// 5 perceptrons of 160 000 elements, 5 % 27.5 -> 20.8 (in many launches 52.7 and 36.9).
#include "message_device.h"
#include "quad_device.h"
#include "trigger_device.h"

namespace evg {

constexpr uint32_t kWide = 1024;           // threads of a workgroup
constexpr uint32_t kBlock = 4;             // loads of x and of xhat that a thread has in flight
constexpr uint32_t kNearBits = 7;          // lower bits of the keys of a code that are looked at last
constexpr uint32_t kHeld = 10;             // sixteen codes each that a thread holds

// The trigger test of a tensor (test_tensor).
struct Tested { double acc; float d, dl; int32_t khat; uint32_t code, k; };

struct Chosen {                            // LDS
  Tested test;
  uint32_t hist[kHistBins];
  uint32_t wave[kWide / 64 * 2];
  uint32_t near_key[64], near_at[64];
  uint32_t bin, rem, listed, near, code, cut;
};

// The bin, from the highest down, in which the rem-th key lies, and its rank there; NB bins, a multiple of 1024 or
// fewer, in s.hist, which is empty afterwards.  false: there are fewer keys.
template <uint32_t NB>
__device__ __forceinline__ bool pick(Chosen& s, uint32_t rem) {
  constexpr uint32_t PER = NB < kWide ? 1 : NB / kWide;
  uint32_t cnt[PER], local = 0;
  const uint32_t top = NB - 1 - threadIdx.x * PER;         // (wraps around past the last bin)
  __syncthreads();
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    cnt[j] = threadIdx.x * PER < NB ? s.hist[top - j] : 0u;
    local += cnt[j];
  }
  uint32_t total;
  const uint32_t above = block_excl_scan<kWide / 64>(local, s.wave, &total);
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    if (threadIdx.x * PER < NB) s.hist[top - j] = 0;
  if (above < rem && rem <= above + local) {               // exactly one thread
    uint32_t run = above;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
      if (run < rem && rem <= run + cnt[j]) { s.bin = top - j; s.rem = rem - run; }
      run += cnt[j];
    }
  }
  __syncthreads();
  return rem <= total;
}

// The sum of the earlier wavefronts' totals, and of all sixteen.
__device__ __forceinline__ uint32_t earlier_waves(const uint32_t* totals, uint32_t* all) {
  static_assert(kWide / 64 == 16, "a row of lanes holds a workgroup's totals");
  uint32_t v = totals[lane_id() & 15u];
  const uint32_t own = v;
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);   // row_shr:1, 2, 4, 8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
  *all = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
  const int w = __builtin_amdgcn_readfirstlane((int)wave_id());
  return (uint32_t)__builtin_amdgcn_readlane((int)(v - own), w);
}

// The same where the workgroup has just passed a barrier and each thread has one bin.
__device__ __forceinline__ bool pick_at_once(Chosen& s, uint32_t rem) {
  const uint32_t bin = kWide - 1 - threadIdx.x, cnt = s.hist[bin];
  s.hist[bin] = 0;
  const uint32_t upto = wave_incl_scan(cnt);
  if (lane_id() == 63) s.wave[wave_id()] = upto;
  __syncthreads();
  uint32_t total;
  const uint32_t above = earlier_waves(s.wave, &total) + upto - cnt;
  if (above < rem && rem <= above + cnt) {                 // at most one thread
    s.bin = bin;
    s.rem = rem - above;
  }
  __syncthreads();
  return rem <= total;
}

// What the selection leaves of a tensor for the update pass.
struct Threshold { uint32_t key, ties; bool ok; };

// Running totals of winners before every group of 256 elements, for message_place; groups[g] holds group g's keys above (low half)
// and equal to (high half) the threshold.  Returns the tensor's totals.
__device__ __forceinline__ uint2 place_groups(const Tables& T, Chosen& s, uint32_t r, const ChooseDesc& ld, const uint32_t* groups) {
  const uint32_t G = T.SW * 4, ngroups = (ld.numel + 255) / 256, first = r * T.C + ld.chunk0;
  constexpr uint32_t W = kWide / 64;
  uint32_t carry_a = 0, carry_e = 0;
  for (uint32_t g0 = 0; g0 < ngroups; g0 += kWide) {       // uniform
    const uint32_t g = g0 + threadIdx.x, n = g < ngroups ? groups[g] : 0u;
    const uint32_t upto_a = wave_incl_scan(n & 0xFFFFu), upto_e = wave_incl_scan(n >> 16);
    if (g0) __syncthreads();                               // (the totals of the round before have been read)
    if (lane_id() == 63) {
      s.wave[wave_id()] = upto_a;
      s.wave[W + wave_id()] = upto_e;
    }
    __syncthreads();
    uint32_t all_a, all_e;
    const uint32_t a = carry_a + earlier_waves(s.wave, &all_a) + upto_a - (n & 0xFFFFu), e = carry_e + earlier_waves(s.wave + W, &all_e) + upto_e - (n >> 16);
    carry_a += all_a;
    carry_e += all_e;
    // a chunk's first group (64 is a multiple of a chunk's groups): its running totals are the chunk's
    const uint32_t lead = lane_id() / G * G;
    const uint32_t lead_a = (uint32_t)__shfl((int)a, (int)lead, 64), lead_e = (uint32_t)__shfl((int)e, (int)lead, 64);
    if (g < ngroups) {
      T.group[(size_t)first * G + g] = (a - lead_a) | (e - lead_e) << 16;
      if (lead == lane_id()) T.chunk_before[first + g / G] = make_uint2(a, e);
    }
  }
  return make_uint2(carry_a, carry_e);
}

// Of the keys equal to the threshold only the first `ties` win: the last of them.
__device__ __forceinline__ void cut_by_groups(const Tables& T, const StepArgs& A, Chosen& s, uint32_t r, const ChooseDesc& ld, uint32_t t,
                                              uint32_t ties, const uint32_t* groups) {
  uint32_t carry = 0;
  __syncthreads();                                         // (place_groups ends with reads of the totals that are written next)
  for (uint32_t g0 = 0; g0 < (ld.numel + 255) / 256; g0 += kWide) {       // uniform
    const uint32_t g = g0 + threadIdx.x, n = g < (ld.numel + 255) / 256 ? groups[g] >> 16 : 0u;
    uint32_t sum;
    const uint32_t before = carry + block_excl_scan<kWide / 64>(n, s.wave, &sum);
    if (before < ties && ties <= before + n) { s.bin = g; s.rem = ties - before; }      // at most one thread
    carry += sum;
  }
  __syncthreads();
  if (wave_id() == 0 && ties <= carry) {
    const size_t base = (size_t)r * T.Npad + ld.off;
    uint32_t left = s.rem;
    for (uint32_t v = 0; v < 4; ++v) {
      const uint32_t j = s.bin * 256 + 64 * v + lane_id(), at = j < ld.numel ? j : 0u;
      const bool is = j < ld.numel && rank_key(T.x[base + at], T.xhat[base + at], A.topk_key) == t;
      const uint64_t m = __ballot(is);
      if (is && lanes_below(m) + 1 == left) s.cut = j;
      const uint32_t found = (uint32_t)__popcll(m);
      left = left > found ? left - found : 0u;             // 0: behind us
    }
  }
  __syncthreads();
}

// f(first element, its four keys, how many of them are elements) for all float4s of a tensor, in order: a wavefront has a
// group of 256 at a time.
template <typename F>
__device__ __forceinline__ void for_keys(const Tables& T, const StepArgs& A, uint32_t r, const ChooseDesc& ld, F&& f) {
  const size_t base = (size_t)r * T.Npad + ld.off;
  const uint32_t bytes = (ld.numel + 3) / 4 * 16;
  const __amdgpu_buffer_rsrc_t x = window(T.x + base, bytes), h = window(T.xhat + base, A.topk_key ? 0u : bytes);
  constexpr uint32_t B = kBlock;
  for (uint32_t j0 = 0; j0 < ld.numel; j0 += B * kWide * 4) {       // uniform
    u32x4 xv[B], hv[B];
#pragma unroll
    for (uint32_t u = 0; u < B; ++u) {
      const uint32_t j = j0 + (u * kWide + threadIdx.x) * 4;
      const int byte = (int)(j < ld.numel ? j * 4 : 0xFFFFFFF0u);
      xv[u] = __builtin_amdgcn_raw_buffer_load_b128(x, byte, 0, 0);
      hv[u] = __builtin_amdgcn_raw_buffer_load_b128(h, byte, 0, 0);
    }
#pragma unroll
    for (uint32_t u = 0; u < B; ++u) {
      const uint32_t j = j0 + (u * kWide + threadIdx.x) * 4;
      uint32_t key[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) key[q] = rank_key(__uint_as_float(xv[u][q]), __uint_as_float(hv[u][q]), A.topk_key);
      f(j, key, j >= ld.numel ? 0u : ld.numel - j < 4u ? ld.numel - j : 4u);
    }
  }
}

__device__ __forceinline__ void load_codes(const Tables& T, size_t base, uint32_t numel, uint32_t j0, u32x4 held[kHeld]) {
  const __amdgpu_buffer_rsrc_t codes = window(T.codes + base, (numel + 15) / 16 * 16);       // (the array is 16 bytes longer)
#pragma unroll
  for (uint32_t u = 0; u < kHeld; ++u) {
    const uint32_t j = j0 + (u * kWide + threadIdx.x) * 16;
    held[u] = __builtin_amdgcn_raw_buffer_load_b128(codes, (int)(j < numel ? j : 0xFFFFFFF0u), 0, 0);
  }
}

// Keys from the arenas: bits 30..20, 19..9 and 8..0 in turn, then the groups.
__device__ __forceinline__ Threshold choose_by_keys(const Tables& T, const StepArgs& A, Chosen& s, uint32_t r, const ChooseDesc& ld,
                                                    uint32_t* groups) {
  auto count = [&](uint32_t shift, uint32_t left, uint32_t prefix, uint32_t mask) {
    for_keys(T, A, r, ld, [&](uint32_t, const uint32_t key[4], uint32_t nv) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if ((uint32_t)q < nv && key[q] >> left == prefix) atomicAdd(&s.hist[(key[q] >> shift) & mask], 1u);
    });
  };
  count(20, 31, 0, 2047);
  pick<kHistBins>(s, ld.K);
  uint32_t prefix = s.bin, rem = s.rem;
  count(9, 20, prefix, 2047);
  pick<kHistBins>(s, rem);
  prefix = prefix << 11 | s.bin;
  rem = s.rem;
  count(0, 9, prefix, 511);
  pick<512>(s, rem);
  const uint32_t t = prefix << 9 | s.bin, ties = s.rem;
  for_keys(T, A, r, ld, [&](uint32_t j, const uint32_t key[4], uint32_t nv) {
    uint32_t above = 0, equal = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      above += (uint32_t)__popcll(__ballot((uint32_t)q < nv && key[q] > t));
      equal += (uint32_t)__popcll(__ballot((uint32_t)q < nv && key[q] == t));
    }
    if (lane_id() == 0 && j < ld.numel) groups[j >> 8] = above | equal << 16;
  });
  __syncthreads();
  const uint2 all = place_groups(T, s, r, ld, groups);
  if (threadIdx.x == 0) s.cut = ld.numel - 1;
  __syncthreads();
  if (all.y != ties) cut_by_groups(T, A, s, r, ld, t, ties, groups);
  return {t, ties, all.x + ties == ld.K && all.y >= ties};
}

// From the codes, `code` that of the K-th largest key and `rem` its rank among those; false: too many keys have it.  `meanwhile` is done while
// the keys are on their way.
template <typename F>
__device__ __forceinline__ bool choose_by_codes(const Tables& T, const StepArgs& A, Chosen& s, uint32_t r, const ChooseDesc& ld,
                                                uint32_t anchor, uint32_t code, uint32_t rem, u32x4 held[kHeld], uint32_t* groups, uint32_t* list, uint32_t cap,
                                                Threshold* out, F&& meanwhile) {
  const size_t base = (size_t)r * T.Npad + ld.off;
  uint32_t* const key = list + cap;
  for (uint32_t j0 = 0; j0 < ld.numel; j0 += kHeld * kWide * 16) {          // uniform
    if (j0) load_codes(T, base, ld.numel, j0, held);
    uint32_t in[kHeld], mine = 0;                          // which of a thread's sixteen have the code
#pragma unroll
    for (uint32_t u = 0; u < kHeld; ++u) {
      in[u] = 0;
      const uint32_t first = j0 + u * kWide * 16, j = first + threadIdx.x * 16;
      if (first >= ld.numel) continue;                     // uniform
      if (ld.numel - first < kWide * 16) {                 // uniform: what is past the end has code 0
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
          const uint32_t left = j < ld.numel && ld.numel - j > 4 * w ? ld.numel - j - 4 * w : 0u;
          if (left < 4u) held[u][w] &= (1u << 8 * left) - 1u;
        }
      }
      const Compared c = compare_codes(held[u], code);
      in[u] = c.in;
      mine += (uint32_t)__popc(c.in);
      const uint32_t above = row_sum(c.above);             // sixteen lanes have a group of 256 elements
      if ((lane_id() & 15u) == 0 && j < ld.numel) groups[j >> 8] = above;
    }
    const uint32_t upto = wave_incl_scan(mine);
    uint32_t at = 0;
    if (lane_id() == 63) at = atomicAdd(&s.listed, upto);
    at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + upto - mine;
#pragma unroll
    for (uint32_t u = 0; u < kHeld; ++u) {
      while (in[u]) {
        const uint32_t b = (uint32_t)__ffs((int)in[u]) - 1u;
        in[u] &= in[u] - 1u;
        if (at < cap) list[at] = j0 + (u * kWide + threadIdx.x) * 16 + (b & 7u) * 4 + (b >> 3);
        ++at;
      }
    }
  }
  __syncthreads();
  const uint32_t n = s.listed;
  if (n > cap) return false;                          // uniform
  meanwhile();
  const uint32_t begin = (code + anchor) << kFineBits;
  const __amdgpu_buffer_rsrc_t x = window(T.x + base, ld.numel * 4), h = window(T.xhat + base, A.topk_key ? 0u : ld.numel * 4);
  bool moved = false;                                      // a key is not what its code says: the caller has written x since
  for (uint32_t i = threadIdx.x; i < n; i += kWide) {
    const float xv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x, (int)(list[i] * 4), 0, 0));
    const float hv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(h, (int)(list[i] * 4), 0, 0));
    const uint32_t low = rank_key(xv, hv, A.topk_key) - begin;
    moved |= low >> kFineBits != 0;
    key[i] = low & ((1u << kFineBits) - 1u);
    atomicAdd(&s.hist[key[i] >> kNearBits], 1u);
  }
  moved = __syncthreads_or(moved);
  static_assert(1u << (kFineBits - kNearBits) == kWide, "one bin a thread");
  bool ok = pick_at_once(s, rem) && !moved;
  // what shares the upper ten of their bits with the threshold: a key or a few, unless many are equal
  const uint32_t upper = s.bin, rem2 = s.rem;
  for (uint32_t i = threadIdx.x; i < n; i += kWide)
    if (key[i] >> kNearBits == upper) {
      const uint32_t at = atomicAdd(&s.near, 1u);
      if (at < 64) {
        s.near_key[at] = key[i];
        s.near_at[at] = list[i];
      }
    }
  __syncthreads();
  const uint32_t near = s.near;
  uint32_t t, ties;
  if (near <= 64) {                                        // uniform: ranked by every wavefront for itself, larger keys first, then earlier elements
    const uint32_t l = lane_id(), k = s.near_key[l], at = s.near_at[l];
    uint32_t greater = 0, before = 0;
    for (uint32_t q = 0; q < near; ++q) {
      const uint32_t kq = (uint32_t)__builtin_amdgcn_readlane((int)k, (int)q), jq = (uint32_t)__builtin_amdgcn_readlane((int)at, (int)q);
      greater += kq > k ? 1u : 0u;
      before += kq == k && jq < at ? 1u : 0u;
    }
    const uint64_t is = __ballot(l < near && greater + before + 1 == rem2);          // (no lane: the counts do not fit, `ok` says so)
    const int who = is ? __ffsll((unsigned long long)is) - 1 : 0;
    t = (uint32_t)__builtin_amdgcn_readlane((int)k, who);
    ties = rem2 - (uint32_t)__builtin_amdgcn_readlane((int)greater, who);
    ok &= is != 0;
    const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)at, who);
    if (threadIdx.x == 0) s.cut = last;
    for (uint32_t i = threadIdx.x; i < n; i += kWide)
      if (key[i] >= t) atomicAdd(&groups[list[i] >> 8], key[i] == t ? 0x10000u : 1u);
    __syncthreads();
    const uint2 all = place_groups(T, s, r, ld, groups);
    *out = {begin + t, ties, ok && all.x + ties == ld.K && all.y >= ties};
    return true;
  }
  for (uint32_t i = threadIdx.x; i < n; i += kWide)
    if (key[i] >> kNearBits == upper) atomicAdd(&s.hist[key[i] & ((1u << kNearBits) - 1u)], 1u);
  __syncthreads();
  const uint32_t last = threadIdx.x < 1u << kNearBits ? s.hist[threadIdx.x] : 0u;
  __syncthreads();
  ok &= pick<1u << kNearBits>(s, rem2);
  t = upper << kNearBits | s.bin;
  ties = s.rem;
  if (threadIdx.x == s.bin) s.code = last;                 // keys equal to the threshold
  if (threadIdx.x == 0) {
    s.cut = ld.numel - 1;
    s.near = 0;
  }
  __syncthreads();
  const uint32_t equal = s.code;
  for (uint32_t i = threadIdx.x; i < n; i += kWide) {
    const uint32_t k = key[i], j = list[i];
    if (k >= t) atomicAdd(&groups[j >> 8], k == t ? 0x10000u : 1u);
    if (k == t && equal != ties) {                         // not all of them win (common: drifts are multiples of x's spacing)
      const uint32_t at = atomicAdd(&s.near, 1u);
      if (at < 64) s.near_at[at] = j;
    }
  }
  __syncthreads();
  if (equal != ties && equal <= 64 && threadIdx.x < equal) {
    uint32_t before = 0;                                   // the last winner has ties - 1 before it
    for (uint32_t q = 0; q < equal; ++q) before += s.near_at[q] < s.near_at[threadIdx.x] ? 1u : 0u;
    if (before + 1 == ties) s.cut = s.near_at[threadIdx.x];
  }
  __syncthreads();
  const uint2 all = place_groups(T, s, r, ld, groups);
  if (equal != ties && equal > 64) cut_by_groups(T, A, s, r, ld, begin + t, ties, groups);
  *out = {begin + t, ties, ok && all.x + ties == ld.K && all.y >= ties};
  return true;
}

// The trigger test of a tensor, by a wavefront.  Threshold and last event are asked for with the sums.
__device__ __forceinline__ Tested test_tensor(const Tables& T, const StepArgs& A, uint32_t r, const ChooseDesc& ld) {
  const uint32_t seg = r * T.L + ld.layer;
  Tested t;
  t.dl = T.delta[seg];
  t.khat = T.last_event[seg];
  t.k = tested_k(T, A);
  const size_t at = (size_t)r * T.C * (T.SW * T.fine) + ld.sum0;
  auto sum = [&](const double* part) { return T.fine == 1 ? ordered_lane_sum<8, 1>(part + at, ld.sums) : ordered_lane_sum<8, kGroupSums>(part + at, ld.sums); };
  t.acc = wave_sum_dpp(sum(T.partials));
  double acc_hat = 0.0;
  if (A.norm_src == 2) acc_hat = wave_sum_dpp(sum(T.partials_hat));
  t.d = tested_norm(A, t.acc, acc_hat);
  t.code = (uint32_t)__builtin_amdgcn_readfirstlane((int)event_code(A, t.d, t.dl, t.khat, t.k));
  return t;
}

// A tensor of at most 256 elements, by a wavefront: four keys a lane, the threshold bit by bit.
__device__ __forceinline__ void choose_small(const Tables& T, const StepArgs& A, uint32_t r, const ChooseDesc& ld) {
  const uint32_t seg = r * T.L + ld.layer, lane = lane_id();
  const size_t base = (size_t)r * T.Npad + ld.off;
  const uint32_t bytes = (ld.numel + 3) / 4 * 16;
  const u32x4 xv = __builtin_amdgcn_raw_buffer_load_b128(window(T.x + base, bytes), (int)(lane * 16), 0, 0);
  const u32x4 hv = __builtin_amdgcn_raw_buffer_load_b128(window(T.xhat + base, bytes), (int)(lane * 16), 0, 0);
  const Tested test = test_tensor(T, A, r, ld);
  if (lane == 0) book_test<true>(T, A, seg, test.d, test.dl, test.khat, (uint8_t)test.code, test.acc, test.k);
  if (test.code != 2) return;
  uint32_t key[4];
  uint64_t valid[4];
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) {
    key[q] = rank_key(__uint_as_float(xv[q]), __uint_as_float(hv[q]), A.topk_key);
    valid[q] = __ballot(lane * 4 + q < ld.numel);
  }
  uint32_t t = 0;
#pragma unroll 1
  for (uint32_t b = 1u << 30; b; b >>= 1) {                // the largest t that at least K keys reach
    uint32_t n = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) n += (uint32_t)__popcll(__ballot(key[q] >= (t | b)) & valid[q]);
    if (n >= ld.K) t |= b;
  }
  uint32_t above = 0, equal = 0, before = 0;
  uint64_t eq[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    above += (uint32_t)__popcll(__ballot(key[q] > t) & valid[q]);
    eq[q] = __ballot(key[q] == t) & valid[q];
    equal += (uint32_t)__popcll(eq[q]);
    before += lanes_below(eq[q]);
  }
  const uint32_t ties = ld.K - above;
  if (lane == 0) {
    T.sel_prefix[seg] = t;
    T.sel_krem[seg] = ties;
    T.chunk_before[r * T.C + ld.chunk0] = make_uint2(0, 0);
    T.group[(size_t)(r * T.C + ld.chunk0) * (T.SW * 4)] = 0;
    if (equal == ties) T.sel_cut[seg] = ld.numel - 1;
  }
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) {
    const bool is = (eq[q] >> lane) & 1ull;
    before += is ? 1u : 0u;
    if (is && equal != ties && before == ties) T.sel_cut[seg] = lane * 4 + q;
  }
}

// tensors: by size, the `longer` of more than 256 elements first.  A workgroup has one of them, or sixteen others.
__global__ __launch_bounds__(kWide) void k_topk_choose(const ChooseDesc* tensors, uint32_t longer, uint32_t lists, uint32_t cap, StepArgs A, Tables T) {
  __shared__ Chosen s;
  extern __shared__ uint32_t groups[];                     // one a group of the longest tensor; from `lists` on `cap` listed elements and their keys
  const uint32_t r = blockIdx.y, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_id());
  if (blockIdx.x >= longer) {
    const uint32_t i = longer + (blockIdx.x - longer) * (kWide / 64) + wave;
    if (i < T.L) choose_small(T, A, r, tensors[i]);
    if (longer == 0 && blockIdx.x == 0 && r == 0 && threadIdx.x == 0) close_step(T, A);
    return;
  }
  const ChooseDesc ld = tensors[blockIdx.x];
  const uint32_t seg = r * T.L + ld.layer;
  u32x4 held[kHeld];
  load_codes(T, (size_t)r * T.Npad + ld.off, ld.numel, 0, held);
  const uint32_t anchor = T.anchor[seg];
  s.hist[threadIdx.x] = 0;
  s.hist[kWide + threadIdx.x] = 0;
  if (wave == 0) {
    const Tested test = test_tensor(T, A, r, ld);
    if (lane_id() == 0) {
      s.test = test;
      s.listed = s.near = 0;
    }
  } else if (wave == 1) {
    // the counts of codes kFirstCode + 127 .. kFirstCode, from the highest down, two a lane; those above are in the last word
    uint32_t* gh = T.hist + (size_t)seg * kHistBins;
    uint32_t higher = 0, a = 0, b = 0;
#pragma unroll
    for (uint32_t c = 0; c < kHistBins / kCodeStride; ++c) {
      higher += gh[c * kCodeStride + kCodeBins];
      a += gh[c * kCodeStride + kCodeBins - 1 - 2 * lane_id()];
      b += gh[c * kCodeStride + kCodeBins - 2 - 2 * lane_id()];
    }
    const uint32_t before = higher + wave_incl_scan(a + b) - (a + b);
    if (lane_id() == 0) s.bin = 0;                         // none of them
    if (before < ld.K && ld.K <= before + a + b) {
      const bool first = ld.K <= before + a;
      s.bin = kFirstCode + kCodeBins - 1 - 2 * lane_id() - (first ? 0 : 1);
      s.rem = ld.K - before - (first ? 0 : a);
    }
#pragma unroll
    for (uint32_t c = 0; c < kHistBins / kCodeStride; ++c) {
      gh[c * kCodeStride + kCodeBins - 1 - 2 * lane_id()] = 0;
      gh[c * kCodeStride + kCodeBins - 2 - 2 * lane_id()] = 0;
      if (lane_id() == 0) gh[c * kCodeStride + kCodeBins] = 0;
    }
  }
  __syncthreads();
  auto book = [&] {
    if (threadIdx.x != kWide - 1) return;
    book_test<true>(T, A, seg, s.test.d, s.test.dl, s.test.khat, (uint8_t)s.test.code, s.test.acc, s.test.k);
    if (blockIdx.x == 0 && r == 0) close_step(T, A);
  };
  if (s.test.code != 2) {                                  // uniform
    book();
    return;
  }
  const uint32_t code = s.bin, rem = s.rem;
  __syncthreads();                                         // (s.bin is written again further down)
  Threshold found;
  if (anchor == kNoAnchor || code == 0 || !choose_by_codes(T, A, s, r, ld, anchor, code, rem, held, groups, groups + lists, cap, &found, book)) {
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(T.not_staged, ld.nchunks);
    book();
    found = choose_by_keys(T, A, s, r, ld, groups);
  }
  if (threadIdx.x == 0) {
    T.sel_prefix[seg] = found.ok ? found.key : kNoThreshold;
    T.sel_krem[seg] = found.ties;
    T.sel_cut[seg] = s.cut;
    const uint32_t q = found.key >> kFineBits;             // in the middle of the codes
    T.anchor[seg] = q > 128u ? (q - 128u) / kPerCoarse * kPerCoarse : 0u;
  }
}

hipError_t launch_topk_choose(const Tables& t, const StepArgs& a, const ChooseTables& c, hipStream_t s) {
  const dim3 grid(c.longer + (t.L - c.longer + kWide / 64 - 1) / (kWide / 64), t.P);
  // (a list of 12 288 takes 1.2 us more where one of 4096 will do: no other workgroup is on the CU meanwhile)
  const uint32_t groups = (c.longest + 255) / 256, cap = c.longest <= 327680 ? 4096u : 12288u;
  k_topk_choose<<<grid, dim3(kWide), (groups + 2 * cap) * 4, s>>>(c.tensors, c.longer, groups, cap, a, t);
  return hipGetLastError();
}

}  // namespace evg
