// Top-K sparsified sends (Section 7): on an event only the K elements of largest
// rank key travel, with their indices.  The winning set is unique: keys descending,
// ties to the lower index.  Everything here is integer work on 31-bit keys (bit
// patterns of non-negative floats), so results are exact and repeatable.
//
// The selection ends with two numbers per tensor, the threshold key t and the last element that wins
// with a key equal to t: element j wins if key > t, or key == t and j <= cut.  Whoever has x and xhat in
// registers afterwards -- the update pass -- can tell the winners by itself, and where they belong
// in the message from the number of winners before its group of 256 elements.
//
//   k_topk_hist     pass A where the previous update pass has not done it: histogram of the keys per tensor, in the bins of first_bins
//   k_topk_decide   trigger test, and the bin b that holds the K-th largest key (k_topk_pick: the latter alone)
//   k_topk_stage    the one pass over the fired tensors: per group of 256 elements how many keys lie above
//                   bin b, and the keys IN bin b (a sixty-fourth of an octave where the threshold was expected, some 0.4 % of the
//                   tensor), whose next 11 bits it counts.  From the key codes of the last update pass, 1 byte an element
//                   instead of 8, where bin b has a code: only the keys in it are fetched then
//   k_topk_low      counts the last bits of the in-bin keys under the prefix found so far
//   k_topk_count    the threshold key from those counts (last_bin), and keys above and equal to it per group, as running totals over a chunk
//   k_topk_scan     the same over a tensor's chunks, and the cut
//   k_topk_apply    messages written and applied ahead of the update pass, where that pass cannot
// Codes and fine bins, steps before -> now: 16 ResNet-18 workers with given gradients, 10 % 1371 -> 1277 us (k_topk_stage 184 -> 61, the
// walk, which writes the codes, 1156 -> 1173), 64 4903 -> 4538, 8 ResNet-50 workers, 1 %, Student-t 1269 -> 1199.  Of the keys' bins
// 128 are fine: with 256 the walk merges more counts (ResNet-50 1220), with a thirty-second of an octave each the stage fetches
// more (64 workers 4647); bins of an eighth and codes that divide them cost a launch more and 1317 where 1277 is now.
// The many launches are bound by their chains of dependent reads, which go together where they can, and by vector instructions in k_topk_stage.
// 64 ResNet-18 workers, 10 %, and 8 ResNet-50 workers, 1 %, us a launch, before -> now: k_topk_decide 28 -> 21 and 10 -> 8 (bins asked for ahead of the
// test), k_topk_stage 360 -> 349 and 70 -> 60 (compare_codes, one list of a lane's two loads), k_topk_low 27 -> 21 and 9 -> 7.5, and a launch
// of 6 and 5 less (last_bin).  Steps of large rings hardly differ for it (16 ResNet-18 workers with given gradients, 10 % 1265 and 1259, 8 ResNet-50 1157 and
// 1153, 64 ResNet-18 4528 and 4520: no more than two runs do), small ones do: 42 ResNet-20 of width 18, 14 % 210 -> 204.
// (The selection used to stage every possible winner as (index, value) and to compact the messages from there;
// the update passes then scattered three messages each into LDS.)
// Cached rings whose tensors are not too long make the whole selection in one launch, kernels_choose.hip.
#include "trigger_device.h"
#include "message_device.h"

namespace evg {

struct WorkItem {
  uint32_t w, r, c, seg;
  ChunkDesc cd;
  size_t base;   // arena offset of the chunk
};

__device__ __forceinline__ WorkItem work_item(const Tables& T, uint32_t r, uint32_t c) {
  WorkItem it;
  it.w = r * T.C + c;
  it.r = r;
  it.c = c;
  it.cd = T.chunks[c];
  it.seg = it.r * T.L + it.cd.layer;
  it.base = (size_t)it.r * T.Npad + it.cd.off;
  return it;
}

// A chunk's staged keys: a quarter of its length, at most kStageCap, at a quarter of its arena offset (slots of
// neighbouring chunks cannot overlap: floor(a/16) + floor(len/16) <= floor((a + len)/16); 16-byte aligned).
__device__ __forceinline__ size_t stage_slot(const Tables& T, uint32_t r, uint32_t off) {
  return (size_t)r * T.stage_stride + (size_t)(off >> 4) * 4;
}
__device__ __forceinline__ uint32_t stage_cap(uint32_t len) {
  return (len >> 4) * 4 < kStageCap ? (len >> 4) * 4 : kStageCap;
}

// A chunk with more keys in the threshold bin than its slot holds is marked with this count and staged not
// at all: they are read from the arenas instead (exact all the same; it takes massive ties or a tiny tensor).
constexpr uint32_t kNotStaged = 0xFFFFFFFFu;

// Adds the non-empty bins of a workgroup's LDS histogram to the tensor's histogram.
template <int NB>
__device__ __forceinline__ void flush_hist(const uint32_t* h, uint32_t* gh) {
  for (uint32_t b = threadIdx.x; b < (uint32_t)NB; b += kThreads) {
    const uint32_t v = h[b];
    if (v) atomicAdd(&gh[b], v);
  }
}

// ALL: of all tensors, not only of those that send a Top-K message now, by their anchors, and their key codes: what an update pass
// leaves.
template <int SWEEPS, bool ALL>
__global__ __launch_bounds__(kThreads) void k_topk_hist(Tables T, StepArgs A) {
  __shared__ uint32_t h[kHistBins];
  const WorkItem wi = work_item(T, blockIdx.y, blockIdx.x);
  if (!ALL && T.fired[wi.seg] != 2) return;          // uniform
  for (uint32_t b = threadIdx.x; b < (uint32_t)kHistBins; b += kThreads) h[b] = 0;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < SWEEPS; ++it) {
    const uint32_t e = it * kSweep + threadIdx.x * kLaneElems - wi.cd.lead;   // positions before the lead wrap around
    if (e < wi.cd.len) {
      const float4 x4 = ld4s(T.x + wi.base + e);
      float4 h4 = make_float4(0.f, 0.f, 0.f, 0.f);
      if (!A.topk_key) h4 = ld4s(T.xhat + wi.base + e);
      const float xa[4] = {x4.x, x4.y, x4.z, x4.w}, ha[4] = {h4.x, h4.y, h4.z, h4.w};
      const uint32_t nv = wi.cd.len - e < 4u ? wi.cd.len - e : 4u;
      const Bins bins = first_bins(xa, ha, A.topk_key, T.anchor ? T.anchor[wi.seg] & kAnchorBits : kNoAnchor);
      if (ALL && T.codes) store_codes(T, wi.base, (wi.cd.len + 3) / 4 * 16, e * 4, bins.codes);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t b = T.anchor ? bins.bin[q] : rank_key(xa[q], ha[q], A.topk_key) >> kPlainBits;
        if (ALL && A.choose) {                             // what k_update_part counts
          const uint32_t c = (bins.codes >> (8 * q) & 255u) - kFirstCode;
          b = (int)c < 0 ? kFirstBins - 1 : c < kCodeBins ? c : kCodeBins;
        }
        if ((uint32_t)q < nv && !(ALL && A.choose && b == kFirstBins - 1)) atomicAdd(&h[b], 1u);
      }
    }
  }
  __syncthreads();
  flush_hist<kHistBins>(h, T.hist + (size_t)wi.seg * kHistBins);
}

// One workgroup per tensor that sends a Top-K message: find the bin that holds the krem-th largest key, append it to the
// prefix, keep what is still to be taken inside that bin, and clear the histogram for the next pass.
// PASS 0: the bins of first_bins (FINE: the ring has anchors) or a key's upper 11 bits, PASS 1: the next 11 bits.  (The rest: last_bin.)
// `counted`: the histogram, if it has been taken from T.hist.  What else it goes by is asked for by look_at, ahead of the test where there is one.
template <int PASS, bool FINE>
struct Bounds {
  static constexpr int NB = PASS == 0 && FINE ? kFirstBins : kHistBins, PER = NB / kThreads;
  uint32_t cnt[PER], krem, anchor, prefix, bits;           // (cnt: from this thread's highest bin downwards)
};
template <int PASS, bool FINE = false>
__device__ __forceinline__ Bounds<PASS, FINE> look_at(const Tables& T, uint32_t seg, bool counted) {
  Bounds<PASS, FINE> b;
  const uint32_t* gh = T.hist + (size_t)seg * kHistBins;
  if (!counted) {                                          // uniform
#pragma unroll
    for (int j = 0; j < b.PER; ++j) b.cnt[j] = gh[b.NB - 1 - threadIdx.x * b.PER - j];
  }
  b.krem = PASS == 0 ? T.layers[seg % T.L].K : T.sel_krem[seg];
  b.anchor = PASS == 0 && FINE ? T.anchor[seg] : kNoAnchor;
  b.prefix = PASS ? T.sel_prefix[seg] : 0u;
  b.bits = PASS ? T.sel_left[seg] & 255u : 0u;
  return b;
}
template <int PASS, bool FINE>
__device__ __forceinline__ void pick_bin(const Tables& T, uint32_t seg, uint32_t code, uint32_t* ws, const uint32_t* counted,
                                         Bounds<PASS, FINE> b) {
  constexpr int NB = Bounds<PASS, FINE>::NB, PER = Bounds<PASS, FINE>::PER;
  uint32_t* gh = T.hist + (size_t)seg * kHistBins;
  if (code != 2) {          // uniform for the workgroup
    // pass A histograms are built for every tensor when the update pass makes them:
    // those of tensors that stay silent are simply dropped
    if (PASS == 0 && !counted)
      for (uint32_t b = threadIdx.x; b < (uint32_t)NB; b += kThreads) gh[b] = 0;
    return;
  }
  const uint32_t krem = b.krem, anchor = b.anchor, prefix = b.prefix, bits = b.bits;
  const uint32_t top = NB - 1 - threadIdx.x * PER;   // this thread's highest bin
  uint32_t* const cnt = b.cnt;
  uint32_t local = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (PASS == 0 && counted) cnt[j] = counted[top - j];
    else gh[top - j] = 0;
    local += cnt[j];
  }
  uint32_t total;
  const uint32_t above = block_excl_scan<4>(local, ws, &total);   // keys in higher bins
  if (total < krem && threadIdx.x == 0) {
    T.sel_prefix[seg] = kNoThreshold;
    if (PASS == 0) T.sel_left[seg] = FINE ? kCoarseBits : kPlainBits;
  }
  if (above < krem && krem <= above + local) {    // exactly one thread
    uint32_t run = above, bin = top, rem = krem - above;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (run < krem && krem <= run + cnt[j]) { bin = top - j; rem = krem - run; }
      run += cnt[j];
    }
    T.sel_krem[seg] = rem;
    if (PASS == 0 && FINE) {
      uint32_t left;
      const uint32_t begin = bin_begin(bin, anchor, &left);
      T.sel_prefix[seg] = begin;
      const uint32_t fine = (begin >> kFineBits) - (anchor & kAnchorBits);
      T.sel_left[seg] = left | (T.codes && !(anchor & kUncoded) && left == kFineBits && fine > 0u && fine < 255u ? fine << 8 : 0u);
      // of the histogram and codes that the update pass will leave: this bin in the middle
      const uint32_t next = (begin >> kFineBits) + kPerCoarse / 2;
      T.anchor[seg] = next > kFineBins / 2 ? (next - kFineBins / 2) / kPerCoarse * kPerCoarse : 0u;
    } else if (PASS == 0) {
      T.sel_prefix[seg] = bin << kPlainBits;
      T.sel_left[seg] = kPlainBits;
    } else {
      // (a selection that has ended stays so)
      if (prefix != kNoThreshold) T.sel_prefix[seg] = prefix + (bin << (bits - 11u));
    }
  }
}

template <int PASS>
__global__ __launch_bounds__(kThreads) void k_topk_pick(Tables T) {
  __shared__ uint32_t ws[4];
  pick_bin<PASS, false>(T, blockIdx.x, T.fired[blockIdx.x], ws, nullptr, look_at<PASS>(T, blockIdx.x, false));
}

// Rings whose update pass has built pass A's histograms: trigger test and pass A's bin in one
// launch, one workgroup per tensor (the first wavefront runs the test).
template <bool FINE>
__global__ __launch_bounds__(kThreads) void k_topk_decide(Tables T, StepArgs A) {
  constexpr uint32_t NB = FINE ? kFirstBins : kHistBins;
  __shared__ uint32_t ws[4], code, counted[NB];
  const uint32_t seg = blockIdx.x, layer = seg % T.L;
  const bool copies = layer == T.long_layer[0] || layer == T.long_layer[1];        // uniform
  const Bounds<0, FINE> bounds = look_at<0, FINE>(T, seg, copies);
  if (wave_id() == 0) {
    double acc, acc_hat;
    bool hat_sums;
    const uint32_t anchor = bounds.anchor, k = tested_k(T, A);
    const int32_t khat = T.last_event[seg];
    segment_sums<16, 1>(T, A, seg, &acc, &acc_hat, &hat_sums);     // (no rings with sums of groups)
    if (lane_id() == 0) {
      code = segment_test(T, A, seg, acc, acc_hat, hat_sums, k);
      // Codes are a byte an element in every step, and save seven at an event: a tensor that is silent for longer leaves them out.  Steps while
      // nothing fires, without codes -> codes always -> now: 16 ResNet-18 workers 878 -> 937 -> 892 us, 30 of width 32 449 -> 479 -> 451, 8
      // ResNet-50 of width 32 294 -> 312 -> 293; where seven tenths fire none is slower than with codes always.
      if (FINE && code == 0 && !(anchor & kUncoded) && (int32_t)k - khat > (int32_t)kCodedFor) T.anchor[seg] = anchor | kUncoded;
    }
  } else if (copies) {
    // a long tensor's histograms, added up while it is tested (one after the other behind the test, which the bins need too: 8.7 us
    // instead of 5.0 with 64 perceptrons of 159 000 elements)
    uint32_t* from[kHistCopies];
#pragma unroll
    for (uint32_t i = 0; i < kHistCopies; ++i) {
      const HistAt at = first_hist(T, layer, i);
      from[i] = T.hist + (size_t)(at.first + seg / T.L * at.step) * kHistBins;
    }
#pragma unroll
    for (uint32_t u = 0; u < (NB + kThreads - 65) / (kThreads - 64); ++u) {
      const uint32_t b = u * (kThreads - 64) + threadIdx.x - 64;
      if (b < NB) {
        uint32_t n = 0;
#pragma unroll
        for (uint32_t i = 0; i < kHistCopies; ++i) n += from[i][b];
        counted[b] = n;
        if (n) {
#pragma unroll
          for (uint32_t i = 0; i < kHistCopies; ++i) from[i][b] = 0;
        }
      }
    }
  }
  __syncthreads();
  pick_bin<0, FINE>(T, seg, code, ws, copies ? counted : nullptr, bounds);
  if (seg == 0 && threadIdx.x == 0) close_step(T, A);
}

// Staging from the key codes, 1 byte an element instead of 8: what has the code of the threshold bin is listed by its
// position in the chunk, and only those keys are fetched.  A key that is not what its code says (the caller has written x
// since) ends the selection.  Sixteen codes a lane in one load, sums by rotations and one place a wavefront: four codes a
// lane with ballots and a place for each took 10 us more for 16 ResNet-18 workers.  Bound by vector instructions and the chain descriptor,
// decision, codes, keys, slot; with 10 % sent by the lines of x and xhat that hold the keys.
template <int SWEEPS>
__device__ __forceinline__ void stage_by_codes(const Tables& T, const StepArgs& A, const WorkItem& wi, uint32_t begin, uint32_t code,
                                               uint32_t* list, uint32_t* listed) {
  constexpr int LOADS = (SWEEPS + 3) / 4;                  // of 4096 positions
  const uint32_t positions = wi.cd.lead + wi.cd.len;       // (positions before the lead are codes of the tensor before)
  const __amdgpu_buffer_rsrc_t codes = window(T.codes + wi.base - wi.cd.lead, (positions + 15) / 16 * 16);
  u32x4 sixteen[LOADS];
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const uint32_t p = (u * kThreads + threadIdx.x) * 16;
    sixteen[u] = __builtin_amdgcn_raw_buffer_load_b128(codes, (int)(p < positions ? p : 0xFFFFFFF0u), 0, 2);
  }
  __syncthreads();
  static_assert(LOADS <= 2, "two loads share a register's bits");
  const bool ends = wi.cd.lead != 0 || positions < SWEEPS * (uint32_t)kSweep;      // uniform: not all positions are elements of the chunk
  uint32_t in = 0, above = 0;                              // which of a lane's have the code: bit 8 b + 4 u + w for the b-th of the w-th four
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    if (ends) {                                            // what is no element gets code 0, which no bin has that is told by codes
#pragma unroll
      for (uint32_t w = 0; w < 4; ++w) {
        const uint32_t at = (u * kThreads + threadIdx.x) * 16 + 4 * w, left = at < wi.cd.lead || at >= positions ? 0u : positions - at;
        if (left < 4u) sixteen[u][w] &= (1u << 8 * left) - 1u;
      }
    }
    const Compared c = compare_codes(sixteen[u], code);
    in |= c.in << 4 * u;
    above |= c.above << 16 * u;
  }
  above = row_sum(above);                                  // sixteen lanes have a group of 256 positions
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const uint32_t p = (u * kThreads + threadIdx.x) * 16;
    if ((lane_id() & 15u) == 0 && p < SWEEPS * (uint32_t)kSweep) T.group[(size_t)wi.w * (T.SW * 4) + (p >> 8)] = above >> 16 * u & 0xFFFFu;
  }
  const uint32_t mine = (uint32_t)__popc(in), upto = wave_incl_scan(mine);
  uint32_t next = 0;
  if (lane_id() == 63) next = atomicAdd(listed, upto);
  next = (uint32_t)__builtin_amdgcn_readlane((int)next, 63) + upto - mine;
  while (in) {
    const uint32_t b = (uint32_t)__ffs((int)in) - 1u;
    in &= in - 1u;
    if (next < kStageCap) list[next] = (b >> 2 & 1u) * (kThreads * 16) + threadIdx.x * 16 + (b & 3u) * 4 + (b >> 3);
    ++next;
  }
  __syncthreads();
  const uint32_t n = *listed;
  uint32_t* gh = T.hist + (size_t)wi.seg * kHistBins;
  const __amdgpu_buffer_rsrc_t x = window(T.x + wi.base, wi.cd.len * 4), h = window(T.xhat + wi.base, A.topk_key ? 0u : wi.cd.len * 4);
  auto low = [&](uint32_t pos) {
    const uint32_t at = (pos - wi.cd.lead) * 4;
    const float xv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x, (int)at, 0, 0));
    const float hv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(h, (int)at, 0, 0));
    const uint32_t l = rank_key(xv, hv, A.topk_key) - begin;
    if (l >> kFineBits) T.sel_prefix[wi.seg] = kNoThreshold;
    atomicAdd(&gh[(l >> (kFineBits - 11)) & 2047u], 1u);
    return l & ((1u << kFineBits) - 1u);
  };
  if (n <= kStageCap) {
    for (uint32_t i = threadIdx.x; i < n; i += kThreads) list[i] = low(list[i]) | (list[i] >> 8) << 21;
  } else {
    for (uint32_t pos = wi.cd.lead + threadIdx.x; pos < wi.cd.lead + wi.cd.len; pos += kThreads)
      if (T.codes[wi.base + pos - wi.cd.lead] == code) (void)low(pos);
  }
  __syncthreads();
}

// One workgroup per chunk; a wavefront's part of a sweep is a group of 256 elements.  Ballots give the
// counts; the keys in the threshold bin are gathered in LDS, in no particular order (each carries its
// group, in the bits from the 21st on), and leave as one run.  Bound by reading x and xhat, or by latency where it goes by codes.
// COPY: 0 nothing to do for a tensor sent whole (it lands later, or the update pass sends it), 1 its chunk goes into
// the two mailboxes, 2 into xhat, if its worker is at the end of a part of the ring (see copy_chunk): a
// Top-K tensor's first send takes no launch of its own.
template <int SWEEPS, int COPY, bool STREAM>
__global__ __launch_bounds__(kThreads) void k_topk_stage(Tables T, StepArgs A) {
  constexpr int STEP = SWEEPS >= 4 ? 4 : SWEEPS;      // sweeps whose loads are in flight together
  __shared__ __attribute__((aligned(16))) uint32_t list[kStageCap];
  __shared__ uint32_t h[kHistBins], listed;
  const WorkItem wi = work_item(T, blockIdx.y, blockIdx.x);
  const uint32_t code = T.fired[wi.seg];      // uniform
  if (COPY && code == 1 && (COPY == 1 || is_led(T, A, wi.r))) copy_chunk<SWEEPS, STREAM, COPY == 2>(T, wi.r, wi.cd);
  if (code != 2) return;
  const uint32_t begin = T.sel_prefix[wi.seg], left = T.sel_left[wi.seg] & 255u, of_bin = T.sel_left[wi.seg] >> 8;
  if (threadIdx.x == 0) listed = 0;
  if (STREAM && of_bin) {                              // uniform (cached rings whose selections are made here keep no codes)
    stage_by_codes<SWEEPS>(T, A, wi, begin, of_bin, list, &listed);
  } else {
  for (uint32_t b = threadIdx.x; b < (uint32_t)kHistBins; b += kThreads) h[b] = 0;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < SWEEPS; it += STEP) {
    uint32_t e[STEP];
    float4 x4[STEP], h4[STEP];
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
      e[u] = (it + u) * kSweep + threadIdx.x * kLaneElems - wi.cd.lead;   // positions before the lead wrap around
      x4[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      h4[u] = x4[u];
      if (e[u] < wi.cd.len) {
        x4[u] = ld4t<STREAM>(T.x + wi.base + e[u]);
        if (!A.topk_key) h4[u] = ld4t<STREAM>(T.xhat + wi.base + e[u]);
      }
    }
    uint32_t key[STEP][4], n_in[STEP], n_all = 0;
    uint64_t in[STEP][4];
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
      const float xa[4] = {x4[u].x, x4[u].y, x4[u].z, x4[u].w}, ha[4] = {h4[u].x, h4[u].y, h4[u].z, h4[u].w};
      const uint32_t nv = e[u] >= wi.cd.len ? 0u : (wi.cd.len - e[u] < 4u ? wi.cd.len - e[u] : 4u);
      uint32_t above = 0;
      n_in[u] = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        key[u][q] = rank_key(xa[q], ha[q], A.topk_key);
        const bool valid = (uint32_t)q < nv;
        const int32_t low = (int32_t)(key[u][q] - begin);          // (both have 31 bits)
        const bool is_in = valid && (uint32_t)low >> left == 0;
        key[u][q] = (uint32_t)low;
        in[u][q] = __ballot(is_in);
        above += __popcll(__ballot(valid && low >> left > 0));
        if (is_in) atomicAdd(&h[(uint32_t)low >> (left - 11u)], 1u);
        n_in[u] += __popcll(in[u][q]);
      }
      if (lane_id() == 0) T.group[(size_t)wi.w * (T.SW * 4) + (it + u) * 4 + wave_id()] = above;
      n_all += n_in[u];
    }
    uint32_t at = 0;
    if (n_all) {                                     // wave-uniform
      if (lane_id() == 0) at = atomicAdd(&listed, n_all);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    }
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t pos = at + lanes_below(in[u][q]);
        if (((in[u][q] >> lane_id()) & 1ull) && pos < kStageCap)
          list[pos] = key[u][q] | (((it + u) * 4 + wave_id()) << 21);
        at += __popcll(in[u][q]);
      }
    }
  }
  __syncthreads();
  flush_hist<kHistBins>(h, T.hist + (size_t)wi.seg * kHistBins);
  }
  const uint32_t n = listed;
  const bool over = n > stage_cap(wi.cd.len);        // uniform
  if (threadIdx.x == 0) {
    T.stage_n[wi.w] = over ? kNotStaged : n;
    if (over) atomicAdd(T.not_staged, 1u);           // running count, reported by evg_stats
  }
  if (over) return;
  uint32_t* slot = T.stage_key + stage_slot(T, wi.r, wi.cd.off);
  for (uint32_t q = threadIdx.x; q < n / 4; q += kThreads)
    *reinterpret_cast<u32x4*>(slot + 4 * q) = *reinterpret_cast<const u32x4*>(list + 4 * q);
  for (uint32_t q = n / 4 * 4 + threadIdx.x; q < n; q += kThreads) slot[q] = list[q];
}

// Rank keys of a wavefront's 256 positions of a chunk from p0 on, 64 at a time; ok: there is an element.
__device__ __forceinline__ void keys_at(const Tables& T, const StepArgs& A, uint32_t r, const ChunkDesc& pc, uint32_t p0,
                                        uint32_t key[4], bool ok[4]) {
  const size_t at = (size_t)r * T.Npad + pc.off;
  const __amdgpu_buffer_rsrc_t x = window(T.x + at, pc.len * 4), h = window(T.xhat + at, A.topk_key ? 0u : pc.len * 4);
  float xv[4], hv[4];
#pragma unroll
  for (uint32_t v = 0; v < 4; ++v) {
    const uint32_t e = p0 + 64 * v + lane_id() - pc.lead;
    ok[v] = e < pc.len;
    xv[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x, (int)(ok[v] ? e * 4 : 0xFFFFFFF0u), 0, 0));
    hv[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(h, (int)(ok[v] ? e * 4 : 0xFFFFFFF0u), 0, 0));
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) key[v] = rank_key(xv[v], hv[v], A.topk_key);
}

// The kernels below walk a chunk's staged keys, a few hundred, so one wavefront per chunk does it without
// workgroup barriers.  Four independent wavefronts share a workgroup.

// A wavefront's chunk (blockIdx.y = worker) and its first 512 keys in the threshold bin, which are asked for before it is known
// that its tensor sends a Top-K message, and so is what too(seg) does: bound by descriptor, then keys, decision and the rest at once
// instead of one behind the other.
struct Staged { WorkItem wi; uint32_t n; u32x4 e[2]; bool sends; };
__device__ __forceinline__ u32x4 four_staged(const Tables& T, const WorkItem& wi, uint32_t n, uint32_t q) {
  return __builtin_amdgcn_raw_buffer_load_b128(window(T.stage_key + stage_slot(T, wi.r, wi.cd.off), (n + 3) / 4 * 16), (int)(q * 4), 0, 0);
}
template <typename F>
__device__ __forceinline__ bool wave_item(const Tables& T, Staged* s, F&& too) {
  const uint32_t c = blockIdx.x * (kThreads / 64) + (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_id());
  if (c >= T.C) return false;
  s->wi = work_item(T, blockIdx.y, c);
  const uint32_t n = T.stage_n[s->wi.w], held = n <= stage_cap(s->wi.cd.len) ? n : 0u;      // (a silent tensor's is an earlier step's, or nobody's)
#pragma unroll
  for (uint32_t u = 0; u < 2; ++u) s->e[u] = four_staged(T, s->wi, held, 256 * u + 4 * lane_id());
  const uint32_t code = T.fired[s->wi.seg];
  too(s->wi);
  s->sends = __builtin_amdgcn_readfirstlane((int)code) == 2;
  s->n = s->sends ? n : 0u;
  return true;
}

// f(low 20 bits and group) for every key of the chunk in the threshold bin; all(key, group) instead, for every key, where
// nothing is staged.
template <typename F, typename G>
__device__ __forceinline__ void in_bin_keys(const Tables& T, const StepArgs& A, const Staged& s, F&& f, G&& all) {
  const WorkItem& wi = s.wi;
  if (s.n != kNotStaged) {                           // wave-uniform
    u32x4 e[2] = {s.e[0], s.e[1]};
    for (uint32_t q0 = 0; q0 < s.n; q0 += 512) {     // two loads of 4 entries per lane in flight
      if (q0) {
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u) e[u] = four_staged(T, wi, s.n, q0 + 256 * u + 4 * lane_id());
      }
#pragma unroll
      for (uint32_t u = 0; u < 2; ++u) {
        if (q0 + 256 * u >= s.n) break;              // uniform
#pragma unroll
        for (uint32_t v = 0; v < 4; ++v) f(e[u][v], q0 + 256 * u + 4 * lane_id() + v < s.n);
      }
    }
  } else {
#pragma unroll 1
    for (uint32_t p0 = 0; p0 < wi.cd.lead + wi.cd.len; p0 += 256) {
      uint32_t k[4];
      bool ok[4];
      keys_at(T, A, wi.r, wi.cd, p0, k, ok);
#pragma unroll
      for (int v = 0; v < 4; ++v) all(k[v], p0 >> 8, ok[v]);
    }
  }
}

// The bin that holds the krem-th largest of a tensor's last bins (6, 9 or 10 bits), and how many keys are to be taken of it, by one
// wavefront.  Every wavefront that needs the threshold finds it for itself: a launch in between took 5 us.  n: bins[63 - lane].
struct LastBin { uint32_t bin, rem; };               // rem = 0: there are not as many keys
__device__ __forceinline__ LastBin last_bin(const uint32_t* bins, uint32_t n, uint32_t bits, uint32_t krem) {
  const uint32_t lane = lane_id();
  uint32_t top = 63;                                 // highest of 64 bins, or lanes' shares of them
  auto find = [&](uint32_t n) {                      // which lane's it is in, lane 0 first; krem: left to be taken there
    const uint32_t upto = wave_incl_scan(n);
    const uint64_t m = __ballot(upto - n < krem && krem <= upto);
    if (!m) return 64u;
    const uint32_t l = (uint32_t)__ffsll((unsigned long long)m) - 1;
    krem -= (uint32_t)__builtin_amdgcn_readlane((int)(upto - n), (int)l);
    return l;
  };
  if (bits > 6) {                                    // uniform
    const uint32_t per = 1u << (bits - 6);
    n = 0;
    for (uint32_t i = 0; i < per; i += 4) {
      const u32x4 four = *reinterpret_cast<const u32x4*>(bins + (63 - lane) * per + i);
      n += four.x + four.y + four.z + four.w;
    }
    const uint32_t l = find(n);
    if (l == 64u) return {0u, 0u};
    top = (64 - l) * per - 1;
    n = lane < per ? bins[top - lane] : 0u;
  }
  const uint32_t l = find(n);
  return {top - l, l == 64u ? 0u : krem};
}

// The last 6, 9 or 10 bits of the in-bin keys that carry the prefix found so far.  Matches are
// rare (a 2^-25 to 2^-21 slice of the key range), so they go straight to the tensor's histogram,
// one atomic per distinct value per 64 entries.
__global__ __launch_bounds__(kThreads) void k_topk_low(Tables T, StepArgs A) {
  Staged s;
  uint32_t prefix = 0, bits = 0;
  if (!wave_item(T, &s, [&](const WorkItem& wi) {
        prefix = T.sel_prefix[wi.seg];
        bits = T.sel_left[wi.seg] & 255u;
        asm volatile("" : "+s"(prefix), "+s"(bits));       // (left to itself the compiler asks once the decision is known)
      })) return;
  uint32_t* gh = T.hist + (size_t)s.wi.seg * kHistBins;
  auto add = [&](uint32_t k9, bool pending) {
    uint64_t todo = __ballot(pending);
    while (todo) {                                  // uniform: every lane sees the same mask
      const uint32_t leader = __ffsll((unsigned long long)todo) - 1;
      const uint32_t v = __shfl(k9, leader, 64);
      const uint64_t same = __ballot(pending && k9 == v);
      if (lane_id() == leader) atomicAdd(&gh[v], (uint32_t)__popcll(same));
      if ((same >> lane_id()) & 1ull) pending = false;
      todo &= ~same;
    }
  };
  const uint32_t left = bits - 11u, mask = (1u << bits) - 1u, last = (1u << left) - 1u;
  in_bin_keys(T, A, s, [&](uint32_t e, bool in) { add(e & last, in && (e & mask) >> left == (prefix & mask) >> left); },
              [&](uint32_t key, uint32_t, bool in) { add(key & last, in && key >> left == prefix >> left); });
}

// Keys above (low half) and equal to (high half) the threshold: per group the sum over the chunk's earlier groups, and
// the chunk's totals.
__global__ __launch_bounds__(kThreads) void k_topk_count(Tables T, StepArgs A) {
  __shared__ uint32_t counts[kThreads / 64][64];
  Staged s;
  uint32_t* cnt = counts[wave_id()];
  const uint32_t lane = lane_id(), G = T.SW * 4;
  uint32_t above = 0, n = 0, bits = 0, prefix = 0, krem = 0;
  if (!wave_item(T, &s, [&](const WorkItem& wi) {
        above = T.group[(size_t)wi.w * G + (lane < G ? lane : 0u)];
        n = T.hist[(size_t)wi.seg * kHistBins + 63 - lane];
        bits = T.sel_left[wi.seg] & 255u;
        prefix = T.sel_prefix[wi.seg];
        krem = T.sel_krem[wi.seg];
        asm volatile("" : "+v"(n), "+v"(above), "+s"(bits), "+s"(prefix), "+s"(krem));
      }) || !s.sends) return;
  const WorkItem& wi = s.wi;
  uint32_t* group = T.group + (size_t)wi.w * G;
  const uint32_t mask = (1u << bits) - 1u;
  const uint32_t t = prefix + last_bin(T.hist + (size_t)wi.seg * kHistBins, n, bits - 11u, krem).bin;     // (no threshold: k_topk_scan ends it)
  cnt[lane] = 0;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  bool staged = true;
  in_bin_keys(T, A, s,
              [&](uint32_t e, bool in) {
                const uint32_t k = e & mask;
                if (in && k >= (t & mask)) atomicAdd(&cnt[e >> 21], k == (t & mask) ? 0x10000u : 1u);
              },
              [&](uint32_t key, uint32_t g, bool in) {
                staged = false;
                if (in && key >= t) atomicAdd(&cnt[g], key == t ? 0x10000u : 1u);
              });
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const uint32_t mine = cnt[lane] + (staged && lane < G ? above : 0u), incl = wave_incl_scan(mine);
  if (lane < G) group[lane] = incl - mine;
  if (lane == 63) T.chunk_cnt[wi.w] = make_uint2(incl & 0xFFFFu, incl >> 16);
}

// One wavefront per Top-K tensor: the threshold, clearing its bins; running totals over its chunks, in chunk order; and the last
// element that wins with a key equal to the threshold (ties that do not all win are common: differences of parameters that have moved little
// are multiples of the parameters' spacing).
__global__ __launch_bounds__(64) void k_topk_scan(Tables T, StepArgs A) {
  const uint32_t seg = blockIdx.x, lane = threadIdx.x;
  const uint32_t code = T.fired[seg];
  const uint32_t r = seg / T.L, prefix = T.sel_prefix[seg], last = (T.sel_left[seg] & 255u) - 11u, G = T.SW * 4;
  const LayerDesc ld = T.layers[seg % T.L];
  const uint32_t first = r * T.C + ld.chunk0;
  uint32_t* bins = T.hist + (size_t)seg * kHistBins;
  const uint32_t lowest = bins[63 - lane];
  uint2 n[4];
  auto ask = [&](uint32_t b) {
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t i = b + 64 * u + lane;
      n[u] = i < ld.nchunks ? T.chunk_cnt[first + i] : make_uint2(0, 0);
    }
  };
  ask(0);
  if (code != 2) return;
  const LastBin in = last_bin(bins, lowest, last, T.sel_krem[seg]);
  for (uint32_t b = lane; b < 1u << last; b += 64) bins[b] = 0;
  const uint32_t ties = in.rem, t = prefix == kNoThreshold || ties == 0 ? kNoThreshold : prefix + in.bin;
  uint32_t carry_g = 0, carry_e = 0, crossing = 0, need = 0;
  for (uint32_t b = 0; b < ld.nchunks; b += 64 * 4) {
    if (b) ask(b);
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t i = b + 64 * u + lane;
      const uint32_t ig = wave_incl_scan(n[u].x), ie = wave_incl_scan(n[u].y);
      const uint32_t gb = carry_g + ig - n[u].x, eb = carry_e + ie - n[u].y;
      if (i < ld.nchunks) T.chunk_before[first + i] = make_uint2(gb, eb);
      const uint64_t m = __ballot(eb < ties && ties <= eb + n[u].y);       // at most one chunk of the tensor
      if (m) {
        const int l = __ffsll((unsigned long long)m) - 1;
        crossing = b + 64 * u + (uint32_t)l;
        need = ties - (uint32_t)__builtin_amdgcn_readlane((int)eb, l);
      }
      carry_g += (uint32_t)__builtin_amdgcn_readlane((int)ig, 63);
      carry_e += (uint32_t)__builtin_amdgcn_readlane((int)ie, 63);
    }
  }
  if (t == kNoThreshold || carry_g + ties != ld.K || carry_e < ties) {
    if (lane == 0) T.sel_prefix[seg] = kNoThreshold;
    return;
  }
  if (lane == 0) {
    T.sel_prefix[seg] = t;
    T.sel_krem[seg] = ties;
  }
  if (carry_e == ties) {                             // all of them win
    if (lane == 0) T.sel_cut[seg] = ld.numel - 1;
    return;
  }
  // the last group that begins before the last winning tie holds it
  const ChunkDesc cd = T.chunks[ld.chunk0 + crossing];
  const uint32_t before = lane < G ? T.group[(size_t)(first + crossing) * G + lane] >> 16 : 0xFFFFu;
  const uint32_t g = (uint32_t)__popcll(__ballot(before < need)) - 1;
  uint32_t left = need - (uint32_t)__builtin_amdgcn_readlane((int)before, (int)g), k[4];
  bool ok[4];
  keys_at(T, A, r, cd, g * 256, k, ok);
#pragma unroll
  for (uint32_t v = 0; v < 4; ++v) {
    const uint64_t m = __ballot(ok[v] && k[v] == t);
    const uint32_t found = __popcll(m);
    if (((m >> lane) & 1ull) && lanes_below(m) + 1 == left) T.sel_cut[seg] = cd.j0 + g * 256 + 64 * v + lane - cd.lead;
    left = left > found ? left - found : 0u;         // 0: behind us
  }
}

// Ahead of the update pass, one workgroup per chunk: writes the Top-K messages of this iteration and applies them
//   LEAD: to xhat, for the workers at the ends of the parts in which a ring is walked;
//   else: to the neighbours' mailboxes (rings whose update pass cannot tell what a neighbour sent: it does not walk,
//   and there are no copies of x, for lack of room, or as those would be out of date or of no use: a norm pass of its own,
//   xhat reset at events).
// CODES: the ring keeps key codes.
template <int SWEEPS, bool LEAD, bool CODES>
__global__ __launch_bounds__(kThreads) void k_topk_apply(Tables T, StepArgs A) {
  const WorkItem wi = work_item(T, blockIdx.y, blockIdx.x);
  if (T.fired[wi.seg] != 2 || (LEAD && !is_led(T, A, wi.r))) return;           // uniform
  const LayerDesc ld = T.layers[wi.cd.layer];
  const uint32_t t = T.sel_prefix[wi.seg], cut = T.sel_cut[wi.seg];
  const uint32_t left = (wi.r + T.P - 1) % T.P, right = (wi.r + 1) % T.P;
#pragma unroll
  for (int it = 0; it < SWEEPS; ++it) {
    const uint32_t e = it * kSweep + threadIdx.x * kLaneElems - wi.cd.lead;   // positions before the lead wrap around
    const bool live = e < wi.cd.len;
    float4 x4 = make_float4(0.f, 0.f, 0.f, 0.f), h4 = x4;
    if (live) { x4 = ld4s(T.x + wi.base + e); h4 = ld4s(T.xhat + wi.base + e); }
    const float xa[4] = {x4.x, x4.y, x4.z, x4.w};
    float ha[4] = {h4.x, h4.y, h4.z, h4.w};
    const uint32_t nv = !live ? 0u : wi.cd.len - e < 4u ? wi.cd.len - e : 4u;
    const Place place = message_place<CODES>(T, wi.w, wi.cd, ld, it * 4 + wave_id(), T.sel_krem[wi.seg]);
    const uint32_t win = put_message<CODES>(T, wi.r, ld.msg_off, place.first, t == kNoThreshold ? 0u : place.count,
                                           winners4(xa, ha, A.topk_key, t, cut, wi.cd.j0 + e, nv), xa, wi.cd.j0 + e);
    const bool changes = any_of_line_part(win) && live;
    if (LEAD) {
      take_winners(win, xa, ha);
      if (changes) st4s(T.xhat + wi.base + e, make_float4(ha[0], ha[1], ha[2], ha[3]));
    } else if (changes) {
      float* m1 = T.mbox_r + (size_t)left * T.Npad + wi.cd.off + e;
      float* m2 = T.mbox_l + (size_t)right * T.Npad + wi.cd.off + e;
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        float* m = side ? m2 : m1;
        const float4 b = ld4s(m);
        float ba[4] = {b.x, b.y, b.z, b.w};
        take_winners(win, xa, ba);
        st4s(m, make_float4(ba[0], ba[1], ba[2], ba[3]));
      }
    }
  }
}

// Finaliser of the SplitMix64 generator (Steele, Lea, Flood, OOPSLA'14): used to turn a
// message entry into 64 well-mixed bits, so that the sum over a message's entries is a
// fingerprint of the message that does not depend on the order of summation.
__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Fingerprints of the messages of the last step, computed when asked for (evg_message_hashes):
// one workgroup per (worker, tensor) walks the packed message.  Integer sums: the order of
// summation does not change the result.
__global__ __launch_bounds__(kThreads) void k_message_hashes(Tables T) {
  __shared__ unsigned long long ws[2 * (kThreads / 64)];
  const uint32_t seg = blockIdx.x;
  unsigned long long hi = 0ull, hm = 0ull;
  if (T.fired[seg] == 2 && T.sel_prefix[seg] != kNoThreshold) {          // uniform for the workgroup
    const LayerDesc ld = T.layers[seg % T.L];
    const size_t mbase = (size_t)(seg / T.L) * T.Ktot + ld.msg_off;
    for (uint32_t q = threadIdx.x; q < ld.K; q += kThreads) {
      const unsigned long long j = T.msg_idx[mbase + q];
      if (j == kNoEntry) continue;
      hi += mix64(j);
      hm += mix64(((unsigned long long)__float_as_uint(T.msg_val[mbase + q]) << 32) | j);
    }
  }
  hi = wave_sum_u64(hi);
  hm = wave_sum_u64(hm);
  if (lane_id() == 0) { ws[wave_id()] = hi; ws[kThreads / 64 + wave_id()] = hm; }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long a = 0ull, b = 0ull;
    for (int w = 0; w < kThreads / 64; ++w) { a += ws[w]; b += ws[kThreads / 64 + w]; }
    T.idx_hash[seg] = a;
    T.msg_hash[seg] = b;
  }
}

hipError_t launch_message_hashes(const Tables& t, hipStream_t s) {
  k_message_hashes<<<dim3(t.S), dim3(kThreads), 0, s>>>(t);
  return hipGetLastError();
}

hipError_t launch_topk_decide(const Tables& t, const StepArgs& a, hipStream_t s) {
  if (t.anchor) k_topk_decide<true><<<dim3(t.S), dim3(kThreads), 0, s>>>(t, a);
  else k_topk_decide<false><<<dim3(t.S), dim3(kThreads), 0, s>>>(t, a);
  return hipGetLastError();
}

template <int SWEEPS>
static void select_s(const Tables& t, const StepArgs& a, hipStream_t s) {
  const dim3 g(t.C, t.P), gw((t.C + 3) / 4, t.P), b(kThreads), segs(t.S);
  if (!a.hist_fused) {
    k_topk_hist<SWEEPS, false><<<g, b, 0, s>>>(t, a);
    k_topk_pick<0><<<segs, b, 0, s>>>(t);
  }
  if (a.delay || a.pull || (a.walk && a.part == t.P)) {
    if (a.cached) k_topk_stage<SWEEPS, 0, false><<<g, b, 0, s>>>(t, a);
    else k_topk_stage<SWEEPS, 0, true><<<g, b, 0, s>>>(t, a);
  } else if (a.walk) k_topk_stage<SWEEPS, 2, true><<<g, b, 0, s>>>(t, a);
  else if (a.cached) k_topk_stage<SWEEPS, 1, false><<<g, b, 0, s>>>(t, a);
  else k_topk_stage<SWEEPS, 1, true><<<g, b, 0, s>>>(t, a);
  k_topk_pick<1><<<segs, b, 0, s>>>(t);
  k_topk_low<<<gw, b, 0, s>>>(t, a);
  k_topk_count<<<gw, b, 0, s>>>(t, a);
  k_topk_scan<<<segs, dim3(64), 0, s>>>(t, a);
}

template <int SWEEPS>
static void apply_s(const Tables& t, const StepArgs& a, hipStream_t s) {
  const dim3 g(t.C, t.P), b(kThreads);
  if (a.walk && t.codes) k_topk_apply<SWEEPS, true, true><<<g, b, 0, s>>>(t, a);
  else if (a.walk) k_topk_apply<SWEEPS, true, false><<<g, b, 0, s>>>(t, a);
  else if (t.codes) k_topk_apply<SWEEPS, false, true><<<g, b, 0, s>>>(t, a);
  else k_topk_apply<SWEEPS, false, false><<<g, b, 0, s>>>(t, a);
}

hipError_t launch_topk_select(const Tables& t, const StepArgs& a, uint32_t chunk_elems, hipStream_t s) {
  switch (chunk_elems / kSweep) {
    case 1: select_s<1>(t, a, s); break;
    case 2: select_s<2>(t, a, s); break;
    case 4: select_s<4>(t, a, s); break;
    case 8: select_s<8>(t, a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int SWEEPS>
static void count_s(const Tables& t, const StepArgs& a, hipStream_t s) {
  k_topk_hist<SWEEPS, true><<<dim3(t.C, t.P), dim3(kThreads), 0, s>>>(t, a);
}

hipError_t launch_topk_count_all(const Tables& t, const StepArgs& a, uint32_t chunk_elems, hipStream_t s) {
  switch (chunk_elems / kSweep) {
    case 1: count_s<1>(t, a, s); break;
    case 2: count_s<2>(t, a, s); break;
    case 4: count_s<4>(t, a, s); break;
    case 8: count_s<8>(t, a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_topk_apply(const Tables& t, const StepArgs& a, uint32_t chunk_elems, hipStream_t s) {
  switch (chunk_elems / kSweep) {
    case 1: apply_s<1>(t, a, s); break;
    case 2: apply_s<2>(t, a, s); break;
    case 4: apply_s<4>(t, a, s); break;
    case 8: apply_s<8>(t, a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace evg
