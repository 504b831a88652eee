// The whole Top-K selection of one tensor by one workgroup, from the trigger test to the winners' places in the message: for rings
// that live in the last-level cache, whose steps are bound by the chain of launches (the test, the pass over the tensor and
// five more on what it stages took 31 us of 53 with 8 ResNet-20 workers, 27 of 37 with 5 perceptrons of 160 000 elements).
//
// The update pass has left a key code for each element, a byte, and has counted the 128 codes in whose middle the threshold is
// expected (one addition a lane and workgroup, where the histogram of all keys took a pass of its own through LDS).  The counts
// name the code of the K-th largest key; the workgroup goes through the codes once, lists what has that one (some 0.4 % of the
// tensor), fetches those keys alone and finds the threshold among them.  Where the counts do not reach it (a tensor's first
// message; it has moved by more than an octave down or three quarters of one up) the keys are read from the arenas, in four passes.
// Tensors of at most 256 elements are a wavefront's work.
//
// Bound by latency: some ten dependent steps of a workgroup (8 ResNet-20 workers 15 us, its longest tensors 36 864 elements; 24 000
// cycles: descriptors 4000, trigger test 5100, the pass over the codes 3500, fetching 2500, finding the threshold 4700, the groups' places
// 3600).  Steps, before -> now, with the update pass in parts of the ring: 8 ResNet-20 workers, 10 % 52.7 -> 32.7 us, 5 perceptrons of
// 160 000 elements, 5 % 36.9 -> 25.8, 3 to 12 rings of other small networks 40 - 57 -> 19 - 39.
#include "message_device.h"
#include "trigger_device.h"

namespace evg {

constexpr uint32_t kWide = 1024;           // threads of a workgroup
constexpr uint32_t kListCap = 4096;        // listed keys at most
constexpr uint32_t kBlock = 4;             // loads of x and of xhat that a thread has in flight
constexpr uint32_t kHeld = 10;             // sixteen codes each that a thread holds

struct Chosen {                            // LDS
  uint32_t hist[kHistBins];
  uint32_t list[kListCap], key[kListCap];
  uint32_t wave[kWide / 64 * 2];
  uint32_t bin, rem, listed, code, cut;
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

// What the selection leaves of a tensor for the update pass.
struct Threshold { uint32_t key, ties; bool ok; };

// Running totals of winners before every group of 256 elements, for message_place; groups[g] holds group g's keys above (low half)
// and equal to (high half) the threshold.  Returns the tensor's totals.
__device__ __forceinline__ uint2 place_groups(const Tables& T, Chosen& s, uint32_t r, const LayerDesc& ld, const uint32_t* groups) {
  const uint32_t G = T.SW * 4, ngroups = (ld.numel + 255) / 256, first = r * T.C + ld.chunk0;
  uint32_t carry_a = 0, carry_e = 0;
  for (uint32_t g0 = 0; g0 < ngroups; g0 += kWide) {       // uniform
    const uint32_t g = g0 + threadIdx.x, n = g < ngroups ? groups[g] : 0u;
    uint32_t all_a, all_e;
    const uint32_t a = carry_a + block_excl_scan<kWide / 64>(n & 0xFFFFu, s.wave, &all_a);
    const uint32_t e = carry_e + block_excl_scan<kWide / 64>(n >> 16, s.wave, &all_e);
    // a chunk's first group (1024 is a multiple of a chunk's groups): its running totals are the chunk's
    const uint32_t lead = threadIdx.x / G * G;
    s.hist[threadIdx.x] = a;
    s.hist[kWide + threadIdx.x] = e;
    __syncthreads();
    if (g < ngroups) {
      T.group[(size_t)first * G + g] = (a - s.hist[lead]) | (e - s.hist[kWide + lead]) << 16;
      if (lead == threadIdx.x) T.chunk_before[first + g / G] = make_uint2(a, e);
    }
    __syncthreads();
    carry_a += all_a;
    carry_e += all_e;
  }
  return make_uint2(carry_a, carry_e);
}

// Of the keys equal to the threshold only the first `ties` win: the last of them.
__device__ __forceinline__ void cut_by_groups(const Tables& T, const StepArgs& A, Chosen& s, uint32_t r, const LayerDesc& ld, uint32_t t,
                                              uint32_t ties, const uint32_t* groups) {
  uint32_t carry = 0;
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
__device__ __forceinline__ void for_keys(const Tables& T, const StepArgs& A, uint32_t r, const LayerDesc& ld, F&& f) {
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
#pragma unroll
    for (uint32_t w = 0; w < 4; ++w) {                     // what is past the end has code 0
      const uint32_t left = j < numel && numel - j > 4 * w ? numel - j - 4 * w : 0u;
      if (left < 4u) held[u][w] &= (1u << 8 * left) - 1u;
    }
  }
}

// Keys from the arenas: bits 30..20, 19..9 and 8..0 in turn, then the groups.
__device__ __forceinline__ Threshold choose_by_keys(const Tables& T, const StepArgs& A, Chosen& s, uint32_t r, const LayerDesc& ld,
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

// From the codes, `code` that of the K-th largest key and `rem` its rank among those; false: too many keys have it.
__device__ __forceinline__ bool choose_by_codes(const Tables& T, const StepArgs& A, Chosen& s, uint32_t r, const LayerDesc& ld,
                                                uint32_t anchor, uint32_t code, uint32_t rem, u32x4 held[kHeld], uint32_t* groups,
                                                Threshold* out) {
  const size_t base = (size_t)r * T.Npad + ld.off;
  const uint32_t more = (255u - code) * 0x10001u;          // (as in stage_by_codes)
  for (uint32_t j0 = 0; j0 < ld.numel; j0 += kHeld * kWide * 16) {          // uniform
    if (j0) load_codes(T, base, ld.numel, j0, held);
    uint32_t in[kHeld], mine = 0;                          // which of a thread's sixteen have the code
#pragma unroll
    for (uint32_t u = 0; u < kHeld; ++u) {
      in[u] = 0;
      const uint32_t j = j0 + (u * kWide + threadIdx.x) * 16;
      if (j0 + u * kWide * 16 >= ld.numel) continue;       // uniform
      uint32_t above = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t four = held[u][w], p = (four & 0x00FF00FFu) + more, q = ((four >> 8) & 0x00FF00FFu) + more;
        above += (p & 0x01000100u) + (q & 0x01000100u);
        const uint32_t ip = ((p + 0x10001u) ^ p) & 0x01000100u, iq = ((q + 0x10001u) ^ q) & 0x01000100u;
        in[u] |= (ip >> 8 | iq >> 7) << 2 * w;             // element 4 w + b: bit 2 w + (b & 1) + 16 (b >> 1)
      }
      mine += (uint32_t)__popc(in[u]);
      // sixteen lanes have a group of 256 elements
      above = (above >> 8 & 0xFu) + (above >> 24);
      above += (uint32_t)__builtin_amdgcn_mov_dpp((int)above, 0x128, 0xF, 0xF, true);   // row_ror:8, 4, 2, 1
      above += (uint32_t)__builtin_amdgcn_mov_dpp((int)above, 0x124, 0xF, 0xF, true);
      above += (uint32_t)__builtin_amdgcn_mov_dpp((int)above, 0x122, 0xF, 0xF, true);
      above += (uint32_t)__builtin_amdgcn_mov_dpp((int)above, 0x121, 0xF, 0xF, true);
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
        if (at < kListCap) s.list[at] = j0 + (u * kWide + threadIdx.x) * 16 + (b >> 1 & 7u) * 4 + (b & 1u) + (b >> 4) * 2;
        ++at;
      }
    }
  }
  __syncthreads();
  const uint32_t n = s.listed;
  if (n > kListCap) return false;                          // uniform
  const uint32_t begin = (code + anchor) << kFineBits;
  const __amdgpu_buffer_rsrc_t x = window(T.x + base, ld.numel * 4), h = window(T.xhat + base, A.topk_key ? 0u : ld.numel * 4);
  bool moved = false;                                      // a key is not what its code says: the caller has written x since
  for (uint32_t i = threadIdx.x; i < n; i += kWide) {
    const float xv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x, (int)(s.list[i] * 4), 0, 0));
    const float hv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(h, (int)(s.list[i] * 4), 0, 0));
    const uint32_t low = rank_key(xv, hv, A.topk_key) - begin;
    moved |= low >> kFineBits != 0;
    s.key[i] = low & ((1u << kFineBits) - 1u);
    atomicAdd(&s.hist[s.key[i] >> (kFineBits - 11)], 1u);
  }
  moved = __syncthreads_or(moved);
  bool ok = pick<kHistBins>(s, rem) && !moved;
  const uint32_t upper = s.bin, rem2 = s.rem;
  for (uint32_t i = threadIdx.x; i < n; i += kWide)
    if (s.key[i] >> (kFineBits - 11) == upper) atomicAdd(&s.hist[s.key[i] & ((1u << (kFineBits - 11)) - 1u)], 1u);
  __syncthreads();
  const uint32_t last = threadIdx.x < 64 ? s.hist[threadIdx.x] : 0u;        // (6 bits)
  __syncthreads();
  ok &= pick<1u << (kFineBits - 11)>(s, rem2);
  const uint32_t t = upper << (kFineBits - 11) | s.bin, ties = s.rem;
  if (threadIdx.x == s.bin) s.code = last;                 // keys equal to the threshold
  if (threadIdx.x == 0) s.cut = ld.numel - 1;
  __syncthreads();
  const uint32_t equal = s.code;
  if (threadIdx.x == 0) s.listed = 0;
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n; i += kWide) {
    const uint32_t k = s.key[i], j = s.list[i];
    if (k >= t) atomicAdd(&groups[j >> 8], k == t ? 0x10000u : 1u);
    if (k == t && equal != ties) {                         // not all of them win (common: drifts are multiples of x's spacing)
      const uint32_t at = atomicAdd(&s.listed, 1u);
      if (at < kWide) s.hist[at] = j;
    }
  }
  __syncthreads();
  if (equal != ties && equal <= 64 && threadIdx.x < equal) {
    uint32_t before = 0;                                   // the last winner has ties - 1 before it
    for (uint32_t q = 0; q < equal; ++q) before += s.hist[q] < s.hist[threadIdx.x] ? 1u : 0u;
    if (before + 1 == ties) s.cut = s.hist[threadIdx.x];
  }
  __syncthreads();
  const uint2 all = place_groups(T, s, r, ld, groups);
  if (equal != ties && equal > 64) cut_by_groups(T, A, s, r, ld, begin + t, ties, groups);
  *out = {begin + t, ties, ok && all.x + ties == ld.K && all.y >= ties};
  return true;
}

// A tensor of at most 256 elements, by a wavefront: four keys a lane, the threshold bit by bit.
__device__ __forceinline__ void choose_small(const Tables& T, const StepArgs& A, uint32_t seg) {
  const uint32_t r = seg / T.L, lane = lane_id();
  const LayerDesc ld = T.layers[seg % T.L];
  const size_t base = (size_t)r * T.Npad + ld.off;
  const uint32_t bytes = (ld.numel + 3) / 4 * 16;
  const u32x4 xv = __builtin_amdgcn_raw_buffer_load_b128(window(T.x + base, bytes), (int)(lane * 16), 0, 0);
  const u32x4 hv = __builtin_amdgcn_raw_buffer_load_b128(window(T.xhat + base, bytes), (int)(lane * 16), 0, 0);
  double acc, acc_hat;
  bool hat_sums;
  segment_sums(T, A, seg, &acc, &acc_hat, &hat_sums);
  uint32_t code = 0;
  if (lane == 0) code = segment_test(T, A, seg, acc, acc_hat, hat_sums, tested_k(T, A));
  if ((uint32_t)__builtin_amdgcn_readfirstlane((int)code) != 2) return;
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

// order: the tensors by size, the `longer` of more than 256 elements first.  A workgroup has one of them, or sixteen others.
__global__ __launch_bounds__(kWide) void k_topk_choose(Tables T, StepArgs A, const uint32_t* order, uint32_t longer) {
  __shared__ Chosen s;
  extern __shared__ uint32_t groups[];                     // one a group of the longest tensor
  const uint32_t r = blockIdx.y, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_id());
  if (blockIdx.x == 0 && r == 0 && threadIdx.x == 0) close_step(T, A);
  if (blockIdx.x >= longer) {
    const uint32_t i = longer + (blockIdx.x - longer) * (kWide / 64) + wave;
    if (i < T.L) choose_small(T, A, r * T.L + order[i]);
    return;
  }
  const uint32_t layer = order[blockIdx.x], seg = r * T.L + layer;
  const LayerDesc ld = T.layers[layer];
  const uint32_t anchor = T.anchor[seg];
  u32x4 held[kHeld];
  load_codes(T, (size_t)r * T.Npad + ld.off, ld.numel, 0, held);
  for (uint32_t b = threadIdx.x; b < (uint32_t)kHistBins; b += kWide) s.hist[b] = 0;
  if (wave == 0) {
    double acc, acc_hat;
    bool hat_sums;
    segment_sums(T, A, seg, &acc, &acc_hat, &hat_sums);
    if (lane_id() == 0) {
      s.code = segment_test(T, A, seg, acc, acc_hat, hat_sums, tested_k(T, A));
      s.listed = 0;
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
  if (s.code != 2) return;                                 // uniform
  const uint32_t code = s.bin, rem = s.rem;
  __syncthreads();                                         // (s.code and s.bin are written again further down)
  Threshold found;
  if (anchor == kNoAnchor || code == 0 || !choose_by_codes(T, A, s, r, ld, anchor, code, rem, held, groups, &found)) {
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(T.not_staged, ld.nchunks);
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
  k_topk_choose<<<grid, dim3(kWide), (c.longest + 255) / 256 * 4, s>>>(t, a, c.order, c.longer);
  return hipGetLastError();
}

}  // namespace evg
