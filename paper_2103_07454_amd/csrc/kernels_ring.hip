// The update pass of cached rings of few workers, and of streaming ones that send whole tensors, of at most kRingMost (same work and results as
// k_update): one workgroup owns a window of one tensor in ALL workers, a wavefront has one worker's stretch of it (or some workers'), and what a
// worker's neighbours hold of it passes between the wavefronts through LDS.
//
// As in the walk of kernels_walk.hip, what a worker last received from a neighbour is that neighbour's xhat.  A ring cut into parts
// (kernels_parts.hip) reads what lies beyond a part's ends from xhat, and from copies of x that its passes leave; here a third of the reads
// and a tenth of the writes are not needed, a thread has one or two float4s instead of four to eight, and a worker's tests are its
// own wavefronts' work.  What a wavefront goes by is the same in all its lanes.
//
// Bound by latency and the last-level cache: 8 ResNet-20 workers (61 MB) take 9.5 us from the first workgroup's start to the last one's end and three
// before and after; a wavefront waits 1 to 2 us for its descriptor and to have asked for everything, draws for 1.9 (at the vector ALUs' rate), and
// waits 1 for the other wavefronts.  A rolled draw (a third of the code) is slower (12.6 -> 13.8 us), so are 64 registers for eight
// wavefronts a SIMD (they spill: 12.6 -> 13 and more), and kernel arguments that are there with the wavefront gain 0.1 us at most.
// Steps, kernels_parts.hip -> here: the smallest perceptron on 4 workers 6.2 -> 5.4 us, 8 ResNet-20 workers 14.5 -> 12.6, replayed 19.4 -> 18.0,
// 9 of width 24 39.5 -> 34.3, 12 ResNet-18 workers of width 8 14.2 -> 12.6 (which rings: ring_shape).
//
// Streaming rings (STREAM): memory, at 5.1 to 5.5 TB/s, where workgroups that go around the ring (kernels_walk.hip) reach 4.8 to 5.1: these take one window
// after the other, all at once, in the order of their addresses, and a ring of few windows has as many wavefronts as workers.  The
// trigger tests are a launch of their own, so that xhat is not read where the whole tensor is sent.  Walked -> here: 16 ResNet-18 workers 873 -> 817 .. 845 us,
// with given gradients 1035 -> 1010 .. 1022, 7 of width 23 with given gradients and plain SGD 54.0 -> 47.5, 13 ResNet-20 of width 24 49.6 -> 37.5; 32
// ResNet-18 workers with plain SGD 1242 and 1241 (which rings: stream_shape).  Runs of neighbouring windows for an XCD: no faster (2 or 4), 3 % slower (8 and more).
#include "message_device.h"
#include "quad_device.h"
#include "trigger_device.h"

namespace evg {

struct RingArgs {
  const WindowDesc* windows;
  PartClock* clocks;       // one a workgroup (rings whose steps can be single launches)
  double* partials[2];     // both sets of what a test reads: a step reads one and writes the other (Tables: xhat_sq)
  float* delta[2]; int32_t* last_event[2];
  float* x; float* xhat; float* vel; float* mbox_l; float* mbox_r;
  uint8_t* valid_l; uint8_t* valid_r; const uint8_t* fired;
  uint32_t P, L, threads;
  uint32_t row;            // elements of a worker's slice
  uint32_t sums_row;       // partials of a worker
  const uint32_t* thr; const uint32_t* cut; const uint32_t* ties; const uint32_t* anchor; const uint32_t* group;    // Top-K (Tables: sel_prefix ..)
  const uint2* chunk_before;
  uint32_t C, chunk_groups;                                // chunks of a worker, groups of 256 elements of a chunk (log2)
  double* xhat_sq[2];
};

// TESTS: no kernel has run the trigger tests of this iteration: each wavefront runs those of its workers, from the sums that the
// previous pass left, and the tensor's first window books the outcome.  What a test reads is not written by this launch (Tables:
// the _out arrays), so all workgroups decide alike.
// TOPK: some of the tensors send the winners of a selection (k_topk_choose has made it): they are told from x and xhat as everywhere
// (message_device.h).  The pass leaves the codes of the new rank keys and counts those about the anchor.
// G: groups of 256 elements in a window.  Q: float4s of a thread.
// R and A come first, as all workgroups wait for them; T is for the bookings.
template <int DIST, bool GRADBUF, int NORM, bool TESTS, bool TOPK, int G, int Q, bool STREAM>
__global__ __launch_bounds__(1024) void k_update_ring(RingArgs R, StepArgs A, Tables T) {
  static_assert(!(TESTS && TOPK), "selections follow the tests");
  static_assert(!(STREAM && (TESTS || TOPK)), "cached rings only");
  constexpr int WQ = Q > G ? Q / G : 1;                    // workers of a wavefront
  constexpr int GQ = Q > G ? G : Q;                        // groups of each that it has
  static_assert(GQ <= 2, "half a wavefront sums a group");
  constexpr int SPLIT = G / GQ;                            // wavefronts of a worker
  // sweeps of a test whose sums a lane asks for at once (Student-t gradients take the registers that a second one would)
  constexpr int FIRST = G == 1 || (G == 2 && Q == 2 && DIST == 1) ? 1 : 2;
  // Two wavefronts' sums of a worker are one: with one each streaming rings of 8 workers take 1.4 % longer (403 us, 397 together)
  constexpr bool TOGETHER = STREAM && G == 2;
  __shared__ double ws[TOGETHER ? kRingMost : 1][2], ws_hat[TOGETHER && NORM == 3 ? kRingMost : 1][2];
  extern __shared__ float4 held[];                         // [P][G][64] what the neighbours hold from this iteration on
  __shared__ uint32_t codes[TESTS ? kRingMost : 1];
  __shared__ uint64_t spiky;
  const WindowDesc wd = R.windows[blockIdx.x];
  const uint32_t P = R.P, layer = wd.layer, lane = lane_id();
  uint32_t* const counts = reinterpret_cast<uint32_t*>(held + P * G * 64);             // TOPK: [P][kCodeBins + 1]
  if (TOPK)
    for (uint32_t b = threadIdx.x; b < P * (kCodeBins + 1); b += R.threads) counts[b] = 0;
  // A replayable step's iteration: every workgroup keeps count by itself, so that nobody waits for another
  PartClock* const clock = R.clocks + blockIdx.x;
  const bool replayed = TESTS && A.from_device;
  PartClock now{A.k, A.step_no};
  if (replayed) now = *clock;
  if (!TESTS && A.from_device) now = PartClock{T.it->k, (uint32_t)T.it->iters - 1};     // the kernel that ran the tests has counted this step
  const uint32_t turn = now.steps & 1;                     // reads this set, writes the other
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_id()), abreast = R.threads / 64 / SPLIT;
  const uint32_t g0 = wave % SPLIT * GQ;                   // its first group
  auto worker = [&](int i) { return wave / SPLIT + i * abreast; };
  auto exists = [&](int i) { return WQ == 1 || worker(i) < P; };       // uniform
  auto some = [&](int i) { return exists(i) ? worker(i) : P - 1; };    // (loads of workers that are not there)

  // ---- everything is asked for at once ----
  SweepSums<kGroupSums> p[TESTS ? WQ : 1][FIRST];
  if (TESTS) {
#pragma unroll
    for (int i = 0; i < WQ; ++i)
#pragma unroll
      for (int q = 0; q < FIRST; ++q)
        p[i][q] = load_sweep<kGroupSums>((turn ? R.partials[1] : R.partials[0]) + (size_t)some(i) * R.sums_row + wd.sum0, wd.sums, lane + 64 * q);
  }
  // its workers' state, the same in all lanes.  Where xhat is only asked for once a flag is known it comes by scalar loads of the word it is in, as
  // loads of lanes are waited for in their order
  auto flag = [](const uint8_t* flags, uint32_t i) {
    return STREAM ? reinterpret_cast<const uint32_t*>(flags)[i >> 2] >> (8 * (i & 3u)) & 255u : (uint32_t)flags[i];
  };
  uint32_t code[WQ], from_l[WQ], from_r[WQ];
  float d[WQ], dl[WQ];
  int32_t khat[WQ];
  double acc[WQ], hat_sq[WQ];
#pragma unroll
  for (int i = 0; i < WQ; ++i) {
    const uint32_t seg = some(i) * R.L + layer;
    const uint32_t left = some(i) == 0 ? P - 1 : some(i) - 1, right = some(i) + 1 == P ? 0u : some(i) + 1;
    from_l[i] = flag(R.valid_l, seg);
    from_r[i] = flag(R.valid_r, seg);
    if (TESTS) {
      dl[i] = (turn ? R.delta[1] : R.delta[0])[seg];
      khat[i] = (turn ? R.last_event[1] : R.last_event[0])[seg];
      if (NORM == 2) hat_sq[i] = (turn ? R.xhat_sq[1] : R.xhat_sq[0])[seg];
    } else {
      code[i] = flag(R.fired, seg);
      from_l[i] |= flag(R.fired, left * R.L + layer) == 1 ? 1u : 0u;
      from_r[i] |= flag(R.fired, right * R.L + layer) == 1 ? 1u : 0u;
    }
  }
  // (two scalar registers an array; lanes past the window ask for its first element.  Tensors are padded to 4 elements)
  auto at = [&](float* arena, uint32_t r) { return arena + (size_t)r * R.row + wd.off; };
  auto elem = [&](int q) { return (g0 + q % GQ) * 256u + lane * 4; };
  auto byte = [&](int q) { return elem(q) < wd.len ? elem(q) * 4 : 0u; };
  Quad x[Q], v[Q], h[Q], g[Q];
  auto load = [](const float* a, uint32_t b) { return STREAM ? load_nt_at(a, b) : load_at(a, b); };
  auto store = [](float* a, uint32_t b, const Quad& q) { STREAM ? store_nt_at(a, b, q) : store_at(a, b, q); };
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t r = some(q / GQ);
    x[q] = load(at(R.x, r), byte(q));
    if (!STREAM) h[q] = load(at(R.xhat, r), byte(q));
    if (!STREAM || !A.plain_sgd) v[q] = load(at(A.plain_sgd ? R.x : R.vel, r), byte(q));
    if (GRADBUF) g[q] = load(at(const_cast<float*>(A.grad), r), byte(q));
  }
  if (STREAM) {                                            // xhat is not read where the whole tensor is sent: lanes past the end, all of them, get zeros
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      h[q] = load_quad<true>(at(R.xhat, some(q / GQ)), code[q / GQ] == 1 ? 0u : (wd.len + 3) / 4 * 16, elem(q) * 4);
    }
  }
  // The selections: lane q holds what float4 q of the wavefront's threads goes by, its worker's threshold and the places of its group's winners
  // and the next group's in the message (chunks have no leads here, so that a tensor's groups lie one behind the other).  By lanes, as
  // the same in all lanes would be asked for by scalar loads, which are waited for one behind the other.
  uint32_t thr = 0, cut = 0, ties = 0, anchor = 0, in_chunk = 0, in_chunk2 = 0;
  uint2 so_far = make_uint2(0, 0), so_far2 = so_far;
  uint32_t my_q = lane < Q ? lane : Q - 1;
  if (Q == 1) asm("" : "+v"(my_q));                      // (else the compiler sees that it is the same in all lanes)
  const uint32_t my_group = g0 + my_q % GQ;
  const bool more = wd.j0 + (my_group + 1) * 256 < wd.numel;          // the tensor has a group behind it
  if (TOPK) {
    const uint32_t r = worker(my_q / GQ) < P ? worker(my_q / GQ) : P - 1, seg = r * R.L + layer;
    thr = R.thr[seg];
    cut = R.cut[seg];
    ties = R.ties[seg];
    anchor = R.anchor[seg];
    const uint32_t shift = R.chunk_groups, group = (r * R.C << shift) + wd.slot + my_group, next = more ? group + 1 : group;
    in_chunk = R.group[group];
    so_far = R.chunk_before[group >> shift];
    in_chunk2 = R.group[next];
    so_far2 = R.chunk_before[next >> shift];
  }

  // ---- gradients, while all that is on its way ----
  if (!GRADBUF) {
    const double decay_pow = A.from_device ? T.decay_tab[now.k < T.decay_len ? now.k : T.decay_len - 1] : A.decay_pow;
    const float sg = (float)(wd.sig_base * decay_pow);
    uint64_t spikes = 0;                                   // bit r: worker r
    if (A.spike_prob > 0.0f) {                             // uniform; one wavefront draws for all workers (each for its own: as much again as its gradients take)
      if (wave == 0) {
        const uint64_t all = __ballot(has_spike(A, now.k, lane));
        if (lane == 0) spiky = all;
      }
      __syncthreads();
      spikes = spiky;
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (exists(q / GQ) && (g0 + q % GQ) * 256u < wd.len)             // uniform
        draw_gradient<DIST>(A, wd.j0 + elem(q), layer, now.k, worker(q / GQ), sg, ((spikes >> worker(q / GQ)) & 1u) != 0, g[q].v);
  }

  // ---- the trigger tests ----
  if (TESTS) {
#pragma unroll
    for (int i = 0; i < WQ; ++i) {
      const double* from = (turn ? R.partials[1] : R.partials[0]) + (size_t)some(i) * R.sums_row + wd.sum0;
      double s = p[i][0].added();
#pragma unroll
      for (int q = 1; q < FIRST; ++q) s += p[i][q].added();
      for (uint32_t q = FIRST * 64; q < wd.sums / kGroupSums; q += 64) s += load_sweep<kGroupSums>(from, wd.sums, q + lane).added();     // (long tensors)
      acc[i] = wave_sum_dpp(s);
      double acc_hat = 0.0;
      if (NORM == 2) {
        acc_hat = hat_sq[i];
        if (khat[i] < 0) {               // before its first event a tensor's xhat has no norm of its own: the initial pass's sums
          double s2 = 0.0;
          for (uint32_t q = 0; q < wd.sums / kGroupSums; q += 64)
            s2 += load_sweep<kGroupSums>(T.partials_hat + (size_t)some(i) * R.sums_row + wd.sum0, wd.sums, q + lane).added();
          acc_hat = wave_sum_dpp(s2);
        }
      }
      d[i] = tested_norm(A, acc[i], acc_hat);
      code[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)event_code(A, d[i], dl[i], khat[i], now.k));
      if (lane == 0 && exists(i)) codes[worker(i)] = code[i];
    }
  }

  // ---- what the neighbours hold from this iteration on ----
  uint32_t place = 0, count = 0, win[Q];
  if (TOPK) {
    const uint32_t equal = so_far.y + (in_chunk >> 16), equal2 = so_far2.y + (in_chunk2 >> 16);
    place = so_far.x + (in_chunk & 0xFFFFu) + (equal < ties ? equal : ties);
    const uint32_t end = so_far2.x + (in_chunk2 & 0xFFFFu) + (equal2 < ties ? equal2 : ties);
    count = thr == kNoThreshold || my_group * 256u >= wd.len ? 0u : (more ? end : wd.K) - place;
  }
  auto mark = [&](uint32_t v, int q) { return (uint32_t)__builtin_amdgcn_readlane((int)v, q); };
  bool puts[Q];                                            // this lane's 64 bytes are sent, or some of them
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = q / GQ;
    const uint32_t e = elem(q), nv = e >= wd.len ? 0u : wd.len - e < 4u ? wd.len - e : 4u;
    const bool whole = code[i] == 1;
#pragma unroll
    for (int n = 0; n < 4; ++n) h[q].v[n] = whole ? x[q].v[n] : h[q].v[n];
    puts[q] = whole;
    win[q] = 0;
    if (TOPK && code[i] == 2) {                            // uniform
      win[q] = counted_winners(winners4(x[q].v, h[q].v, A.topk_key, mark(thr, q), mark(cut, q), wd.j0 + e, nv), mark(count, q));
      take_winners(win[q], x[q].v, h[q].v);
      puts[q] = any_of_line_part(win[q]);
    }
    if (exists(i)) held[(worker(i) * G + g0 + q % GQ) * 64 + lane] = make_float4(h[q].v[0], h[q].v[1], h[q].v[2], h[q].v[3]);
  }
  // All loads are waited for here, ahead of the first store: a wait for a load further down would be one for the stores before it too.
  __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0)
  __syncthreads();

  // ---- update ----
  const float third = 0.333333343f;   // (float)(1/3): the ring's mixing weight
#pragma unroll
  for (int i = 0; i < WQ; ++i) {
    if (!exists(i)) break;                                 // uniform
    const uint32_t r = worker(i), left = r == 0 ? P - 1 : r - 1, right = r + 1 == P ? 0u : r + 1;
    uint32_t fl = from_l[i], fr = from_r[i];
    if (TESTS) {                                           // a neighbour's send fills a mailbox for good
      const uint32_t l = (uint32_t)__builtin_amdgcn_readfirstlane((int)codes[left]), rr = (uint32_t)__builtin_amdgcn_readfirstlane((int)codes[right]);
      if (wd.books && g0 == 0 && lane == 0) {
        const uint32_t seg = r * R.L + layer;
        T.delta_out = turn ? R.delta[0] : R.delta[1];
        T.last_event_out = turn ? R.last_event[0] : R.last_event[1];
        T.xhat_sq = turn ? R.xhat_sq[1] : R.xhat_sq[0];
        T.xhat_sq_out = turn ? R.xhat_sq[0] : R.xhat_sq[1];
        book_test<false>(T, A, seg, d[i], dl[i], khat[i], (uint8_t)code[i], acc[i], now.k);
        if (l == 1) R.valid_l[seg] = 1;
        if (rr == 1) R.valid_r[seg] = 1;
      }
      fl |= l;
      fr |= rr;
    }
    double sum[GQ], sum_hat[NORM == 3 ? GQ : 1];
#pragma unroll
    for (int gq = 0; gq < GQ; ++gq) {
      const int q = i * GQ + gq;
      const uint32_t e = elem(q), nv = e >= wd.len ? 0u : wd.len - e < 4u ? wd.len - e : 4u;
      const float4 lv4 = held[(left * G + g0 + gq) * 64 + lane], rv4 = held[(right * G + g0 + gq) * 64 + lane];
      const float lv[4] = {lv4.x, lv4.y, lv4.z, lv4.w}, rv[4] = {rv4.x, rv4.y, rv4.z, rv4.w};
      if (code[i] != 0) {                                  // uniform
        if (TOPK && code[i] == 2) (void)put_message<true>(T, r, wd.msg_off, mark(place, q), mark(count, q), win[q], x[q].v, wd.j0 + e);
        if (puts[q] && e < wd.len) {
          store(at(R.xhat, r), e * 4, h[q]);
          store(at(R.mbox_l, right), e * 4, h[q]);
          store(at(R.mbox_r, left), e * 4, h[q]);
        }
      }
      double s = 0.0, s2 = 0.0;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const bool in = (uint32_t)n < nv;                  // lanes past the tensor's end are padding: left as they are
        const float vn = A.plain_sgd ? g[q].v[n] : __builtin_fmaf(A.mu, v[q].v[n], g[q].v[n]);
        const float a = (fl ? (lv[n] - x[q].v[n]) : 0.0f) + (fr ? (rv[n] - x[q].v[n]) : 0.0f);
        const float cns = __builtin_fmaf(a, third, x[q].v[n]);
        const float xnew = __builtin_fmaf(-A.lr, vn, cns);
        x[q].v[n] = in ? xnew : x[q].v[n];
        v[q].v[n] = in ? vn : v[q].v[n];
        const float m = in ? (NORM == 1 ? x[q].v[n] - h[q].v[n] : x[q].v[n]) : 0.0f;
        s += (double)m * (double)m;                        // in lane order, padding adds zero
        if (NORM == 3) {
          const float m2 = in ? h[q].v[n] : 0.0f;
          s2 += (double)m2 * (double)m2;
        }
      }
      if (e < wd.len) {
        store(at(R.x, r), e * 4, x[q]);
        if (!A.plain_sgd) store(at(R.vel, r), e * 4, v[q]);
      }
      sum[gq] = s;
      if (NORM == 3) sum_hat[gq] = s2;
      if (TOPK) {
        const Bins bins = first_bins(x[q].v, h[q].v, A.topk_key, mark(anchor, q));
        if (e < wd.len) *reinterpret_cast<uint32_t*>(T.codes + (size_t)r * R.row + wd.off + e) = bins.codes;
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          const uint32_t c = (bins.codes >> (8 * n) & 255u) - kFirstCode;      // (past the window: one bin for all above)
          if ((uint32_t)n < nv && (int)c >= 0) atomicAdd(&counts[r * (kCodeBins + 1) + (c < kCodeBins ? c : kCodeBins)], 1u);
        }
      }
    }
    // the groups' sums are in lanes 0 and 32 (a group past the window's end: zero)
    const double total = GQ == 1 ? wave_sum_dpp(sum[0]) : wave_sums2(sum[0], sum[GQ - 1]);
    const double total_hat = NORM != 3 ? 0.0 : GQ == 1 ? wave_sum_dpp(sum_hat[0]) : wave_sums2(sum_hat[0], sum_hat[NORM == 3 ? GQ - 1 : 0]);
    if (TOGETHER) {
      if (lane == 0) {
        ws[r][g0] = total;
        if (NORM == 3) ws_hat[r][g0] = total_hat;
      }
    } else if ((GQ == 1 ? lane : lane & 31u) == 0) {
      const size_t slot = (size_t)r * R.sums_row + wd.slot + g0 + lane / 32;
      (turn ? R.partials[0] : R.partials[1])[slot] = total;
      if (NORM == 3) T.partials_hat[slot] = total_hat;
    }
  }
  if (TOGETHER || TOPK) __syncthreads();
  if (TOGETHER && threadIdx.x < P) {
    const size_t slot = (size_t)threadIdx.x * R.sums_row + wd.slot;
    (turn ? R.partials[0] : R.partials[1])[slot] = ws[threadIdx.x][0] + ws[threadIdx.x][1];
    if (NORM == 3) T.partials_hat[slot] = ws_hat[threadIdx.x][0] + ws_hat[threadIdx.x][1];
  }
  if (TOPK) {
    for (uint32_t b = threadIdx.x; b < P * (kCodeBins + 1); b += R.threads) {
      const uint32_t r = b / (kCodeBins + 1), c = counts[b];
      // (eight copies: additions to one address take some 30 ns each, and a long tensor has hundreds of windows)
      if (c) atomicAdd(T.hist + (size_t)(r * R.L + layer) * kHistBins + (blockIdx.x & 7u) * kCodeStride + (b - r * (kCodeBins + 1)), c);
    }
  }
  if (R.clocks && threadIdx.x == 0) *clock = PartClock{now.k + 1, now.steps + 1};
  if (!TESTS) end_replayable(T, A);
  if (TESTS && blockIdx.x == 0 && threadIdx.x == 0) {
    T.it->k = now.k;
    T.it->k_next = now.k + 1;
    T.it->iters = now.steps + 1;
    if (now.k >= T.decay_len && replayed) T.it->overflow = 1;
  }
}

namespace {
struct Launch { const Tables& t; const StepArgs& a; RingArgs r; uint32_t windows, dist, grad_mode; hipStream_t s; };

template <int NORM, bool TESTS, bool TOPK, int G, int Q, bool STREAM = false>
hipError_t ring_kernel(Launch l) {
  const uint32_t per = Q > G ? Q / G : 1, split = Q > G ? 1 : G / Q;
  const dim3 grid(l.windows), block((l.t.P + per - 1) / per * split * 64);
  const size_t lds = (size_t)l.t.P * (G * 1024 + (TOPK ? (kCodeBins + 1) * 4 : 0));
  if (block.x > 1024 || l.t.P > kRingMost) return hipErrorInvalidValue;
  l.r.threads = block.x;
  if (l.grad_mode == 1) k_update_ring<0, true, NORM, TESTS, TOPK, G, Q, STREAM><<<grid, block, lds, l.s>>>(l.r, l.a, l.t);
  else if (l.dist == 0) k_update_ring<0, false, NORM, TESTS, TOPK, G, Q, STREAM><<<grid, block, lds, l.s>>>(l.r, l.a, l.t);
  else k_update_ring<1, false, NORM, TESTS, TOPK, G, Q, STREAM><<<grid, block, lds, l.s>>>(l.r, l.a, l.t);
  return hipGetLastError();
}

template <int NORM, bool TESTS, bool TOPK>
hipError_t ring_of(const Launch& l, uint32_t groups, uint32_t quads) {
  if constexpr (!TESTS && !TOPK) {
    if (!l.a.cached) {
      if (groups == 2 && quads == 1) return ring_kernel<NORM, false, false, 2, 1, true>(l);
      if (groups == 1 && quads == 1) return ring_kernel<NORM, false, false, 1, 1, true>(l);
      if (groups == 1 && quads == 2) return ring_kernel<NORM, false, false, 1, 2, true>(l);
      if (groups == 1 && quads == 4) return ring_kernel<NORM, false, false, 1, 4, true>(l);
      return hipErrorInvalidValue;
    }
  }
  if (groups == 2 && quads == 2) return ring_kernel<NORM, TESTS, TOPK, 2, 2>(l);
  if constexpr (TOPK) {
    if (groups == 1 && quads == 2) return ring_kernel<NORM, TESTS, TOPK, 1, 2>(l);
  } else {
    if (groups == 4 && quads == 2) return ring_kernel<NORM, TESTS, TOPK, 4, 2>(l);
    if (groups == 2 && quads == 1) return ring_kernel<NORM, TESTS, TOPK, 2, 1>(l);
    if (groups == 1 && quads == 1) return ring_kernel<NORM, TESTS, TOPK, 1, 1>(l);
  }
  return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_ring(const Tables& t, const StepArgs& a, const PartTables& p, uint32_t dist, uint32_t grad_mode, int norm, hipStream_t s) {
  RingArgs r{};
  r.windows = p.windows;
  r.clocks = p.clocks;
  for (int i = 0; i < 2; ++i) {
    r.partials[i] = p.set[i].partials;
    r.delta[i] = p.set[i].delta;
    r.last_event[i] = p.set[i].last_event;
    r.xhat_sq[i] = p.set[i].xhat_sq;
  }
  r.x = t.x; r.xhat = t.xhat; r.vel = t.vel; r.mbox_l = t.mbox_l; r.mbox_r = t.mbox_r;
  r.valid_l = t.valid_l; r.valid_r = t.valid_r; r.fired = t.fired;
  r.row = (uint32_t)t.Npad;
  r.sums_row = t.C * t.SW * t.fine;
  r.P = t.P; r.L = t.L;
  r.thr = t.sel_prefix; r.cut = t.sel_cut; r.ties = t.sel_krem; r.anchor = t.anchor; r.group = t.group; r.chunk_before = t.chunk_before;
  r.C = t.C;
  r.chunk_groups = 33 - __builtin_clz(t.SW);               // (SW is a power of two)
  const Launch l{t, a, r, p.count, dist, grad_mode, s};
  if (a.topk_on) return norm == 1   ? ring_of<1, false, true>(l, p.groups, p.quads)
                        : norm == 3 ? ring_of<3, false, true>(l, p.groups, p.quads)
                                    : hipErrorInvalidValue;
  if (norm == 1) return a.one_launch ? ring_of<1, true, false>(l, p.groups, p.quads) : ring_of<1, false, false>(l, p.groups, p.quads);
  if (norm == 2) return a.one_launch ? ring_of<2, true, false>(l, p.groups, p.quads) : ring_of<2, false, false>(l, p.groups, p.quads);
  return hipErrorInvalidValue;
}

}  // namespace evg
