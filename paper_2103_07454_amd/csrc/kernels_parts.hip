// The update pass of rings that live in the last-level cache (same work and results as k_update):
// one workgroup owns a window of 1024 elements of one tensor in a part of the ring, up to kPartMost consecutive workers,
// whose x, velocity and xhat it loads at once.
//
// As in the walk of kernels_walk.hip, what a worker last received from a neighbour is that neighbour's xhat, so mailboxes are
// written and not read (but for Top-K, at a part's ends).  The neighbours of a part's end workers belong to other workgroups:
// what they send is read from the copy of x that the last pass left (two copies in turn, written for end workers only), what
// stays unsent from their xhat, which is written at an event only.  One part that is the whole ring needs neither.
//
// Such a pass takes some microseconds, most of it waiting: for the arguments, for the descriptor, for the arenas.  So
// everything a workgroup needs hangs on one descriptor and is asked for at once, before any of it is known to be wanted
// (xhat of a tensor that is sent, both sources of a part's neighbours); the gradients are drawn meanwhile, in a rolled loop
// into LDS, as the code too comes from memory in every launch.
#include "message_device.h"
#include "quad_device.h"
#include "trigger_device.h"

namespace evg {

struct PartArgs {
  const WindowDesc* windows;
  PartClock* clocks;       // one a workgroup (rings whose steps can be single launches)
  double* partials[2];     // both sets of what a test reads: a step reads one and writes the other (Tables: xhat_sq)
  float* delta[2]; int32_t* last_event[2];
  float* x; float* xhat; float* vel; float* mbox_l; float* mbox_r;
  float* xsnap;            // two copies of x, read and written in the same turns
  uint8_t* valid_l; uint8_t* valid_r; const uint8_t* fired;
  uint32_t row;            // elements of a worker's slice
  uint32_t sums_row;       // partials of a worker
  uint32_t P, L;
  double* xhat_sq[2];
};

__device__ __forceinline__ Quad either(bool first, const Quad& a, const Quad& b) {
  Quad q;
#pragma unroll
  for (int i = 0; i < 4; ++i) q.v[i] = first ? a.v[i] : b.v[i];
  return q;
}

// TESTS: no kernel has run the trigger tests of this iteration: the workgroup runs those of its part's workers and of
// their neighbours itself, from the sums that the previous pass left, and the tensor's first window books the outcome.  What
// a test reads is not written by this launch (Tables: the _out arrays), so all workgroups decide alike.
// TOPK: some of the tensors send the winners of a selection (k_topk_choose has made it): they are told from x and xhat as everywhere
// (message_device.h), of the part's neighbours too.  The pass leaves the codes of the new rank keys and counts those about the anchor.
// R and A come first, as all workgroups wait for them; T is for the bookings.
template <int DIST, bool GRADBUF, int NORM, bool TESTS, int N, bool TOPK>
__global__ __launch_bounds__(kThreads) void k_update_part(PartArgs R, StepArgs A, Tables T) {
  static_assert(!(TESTS && TOPK), "selections follow the tests");
  constexpr int kTests = (N + 2 + 3) / 4;                  // tests of a wavefront
  __shared__ double sums[N + 2], hats[NORM == 2 ? N + 2 : 1], ws[4 * N], ws_hat[NORM == 3 ? 4 * N : 1];
  __shared__ uint32_t counts[TOPK ? N * (kCodeBins + 1) : 1];
  __shared__ float4 draws[GRADBUF ? 1 : N * kThreads];
  const WindowDesc wd = R.windows[blockIdx.x];
  const uint32_t P = R.P, layer = wd.layer, lane = lane_id();
  // A replayable step's iteration: every workgroup keeps count by itself, so that nobody waits for another
  PartClock* const clock = R.clocks + blockIdx.y * gridDim.x + blockIdx.x;
  const bool replayed = TESTS && A.from_device;
  PartClock now{A.k, A.step_no};
  if (replayed) now = *clock;
  if (!TESTS && A.from_device) now = PartClock{T.it->k, (uint32_t)T.it->iters - 1};     // the kernel that ran the tests has counted this step
  const uint32_t turn = now.steps & 1;                     // reads this set and copy, writes the other
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_id());
  const uint32_t r0 = blockIdx.y * A.part, n = P - r0 < A.part ? P - r0 : A.part;      // workers r0 .. r0 + n - 1
  const bool closed = n == P;                              // the part is the whole ring
  // member t of the part: 1 .. n its workers, 0 and n + 1 the neighbours on either side
  const uint32_t before = r0 == 0 ? P - 1 : r0 - 1, after = r0 + n == P ? 0u : r0 + n;
  auto worker = [&](uint32_t t) { return t == 0 ? before : t <= n ? r0 + t - 1 : after; };

  // ---- everything is asked for, without a branch around a load: the compiler would wait for it there ----
  double p0[TESTS ? kTests : 1], p1[TESTS ? kTests : 1];
  if (TESTS) {
#pragma unroll
    for (int q = 0; q < kTests; ++q) {
      const uint32_t t = wave + 4 * q, np = t < n + 2 ? wd.sums : 0u;
      const double* from = (turn ? R.partials[1] : R.partials[0]) + (size_t)(worker(t) * R.sums_row + wd.sum0);
      p0[q] = load_f64(from, np * 8, lane * 8);
      p1[q] = load_f64(from, np * 8, lane * 8 + 512);
    }
  }
  // lane t holds member t's threshold, last event, mailbox flags and decision (lanes past the members: the last one's)
  const uint32_t mseg = worker(lane) * R.L + layer;
  uint32_t thr = 0, cut = 0, ties = 0, in_chunk = 0, in_chunk2 = 0, anchor = 0;
  uint2 so_far = make_uint2(0, 0), so_far2 = so_far;
  if (TOPK) {
    // member t's selection, and where the winners of this wavefront's group of 256 elements, and of the next, belong in its message
    // (chunks have no leads here, so that a tensor's groups lie one behind the other)
    thr = T.sel_prefix[mseg];
    cut = T.sel_cut[mseg];
    anchor = T.anchor[mseg];
    ties = T.sel_krem[mseg];
    const int shift = 33 - __builtin_clz(T.SW);            // groups of a chunk (a power of two)
    const uint32_t first_group = worker(lane) * T.C << shift, groups = P * T.C << shift;
    const uint32_t group = first_group + wd.slot * 4 + wave, next = group + 1 < groups ? group + 1 : group;
    so_far = T.chunk_before[group >> shift];
    in_chunk = T.group[group];
    so_far2 = T.chunk_before[next >> shift];
    in_chunk2 = T.group[next];
    for (uint32_t b = threadIdx.x; b < N * (kCodeBins + 1); b += kThreads) counts[b] = 0;
  }
  const uint32_t fl = R.valid_l[mseg], fr = R.valid_r[mseg], was = TESTS ? 0u : (uint32_t)R.fired[mseg];
  const float dl = TESTS ? (turn ? R.delta[1] : R.delta[0])[mseg] : 0.0f;
  const int32_t khat = TESTS ? (turn ? R.last_event[1] : R.last_event[0])[mseg] : 0;
  const double hat_sq = TESTS && NORM == 2 ? (turn ? R.xhat_sq[1] : R.xhat_sq[0])[mseg] : 0.0;

  // (what is not wanted is asked for at a place that is read anyway)
  const float* from_snap = closed ? R.x : R.xsnap + (size_t)turn * P * R.row;
  float* to_snap = R.xsnap + (size_t)(turn ^ 1) * P * R.row;
  const float* from_vel = A.plain_sgd ? R.x : R.vel;
  const uint32_t e = threadIdx.x * kLaneElems, nv = e >= wd.len ? 0u : wd.len - e < 4u ? wd.len - e : 4u;
  const uint32_t row = R.row * 4, here = wd.off * 4 + (e < wd.len ? e * 4 : 0u);       // (tensors are padded to 4 elements)
  const uint32_t first = r0 * row + here, to_before = closed ? first : before * row + here, to_after = closed ? first : after * row + here;
  Quad x[N], v[N], h[N], g[GRADBUF ? N : 1], end_x[2], end_h[2];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t at = first + ((uint32_t)i < n ? i : 0) * row;
    x[i] = load_at(R.x, at);
    h[i] = load_at(R.xhat, at);
    v[i] = load_at(from_vel, at);
    if (GRADBUF) g[i] = load_at(A.grad, at);
  }
  // What the part's neighbours have sent before is in their xhat, and in the mailboxes of the workers at the ends: those are read
  // where an xhat may be written in this launch although its old value is wanted (a Top-K message).
  end_x[0] = load_at(from_snap, to_before);
  end_h[0] = TOPK ? load_at(R.mbox_l, first) : load_at(R.xhat, to_before);
  end_x[1] = load_at(from_snap, to_after);
  end_h[1] = TOPK ? load_at(R.mbox_r, first + (n - 1) * row) : load_at(R.xhat, to_after);

  // ---- gradients, while all that is on its way ----
  const bool dead = wave * 256u >= wd.len;                 // wave-uniform
  if (!GRADBUF) {
    const double decay_pow = A.from_device ? T.decay_tab[now.k < T.decay_len ? now.k : T.decay_len - 1] : A.decay_pow;
    const float sg = (float)(wd.sig_base * decay_pow);
    uint64_t spikes = 0;
    if (A.spike_prob > 0.0f) spikes = __ballot(has_spike(A, now.k, worker(lane)));
    if (!dead) {
#pragma unroll 1
      for (uint32_t i = 0; i < n; ++i) {
        float z[4];
        draw_gradient<DIST>(A, wd.j0 + e, layer, now.k, r0 + i, sg, (spikes >> (i + 1)) & 1u, z);
        draws[i * kThreads + threadIdx.x] = make_float4(z[0], z[1], z[2], z[3]);
      }
    }
  }
  // (all wavefronts have cleared their share of the counts before one adds to them; the arenas are still on their way)
  if (TOPK) __syncthreads();

  // ---- the trigger tests ----
  uint32_t code = was;
  float d = 0.0f;
  if (TESTS) {
    const double sum = kTests == 1 ? wave_sum_dpp(p0[0] + p1[0])
                                   : wave_sums4(p0[0] + p1[0], p0[kTests > 1] + p1[kTests > 1], p0[kTests - 1] + p1[kTests - 1], 0.0);
    const uint32_t t = wave + 4 * (lane >> 4);             // row q: the wavefront's q-th test
    if ((lane & 15u) == 0 && lane < 16u * kTests && t < n + 2) sums[t] = sum;
    if (NORM == 2) {
      for (uint32_t q = wave; q < n + 2; q += 4) {
        double acc_hat = readlane_f64(hat_sq, q);
        if (__builtin_amdgcn_readlane(khat, (int)q) < 0) {
          // before its first event a tensor's xhat has no norm of its own: the initial pass's sums
          const double* from = T.partials_hat + (size_t)(worker(q) * R.sums_row + wd.sum0);
          acc_hat = wave_sum_dpp(load_f64(from, wd.sums * 8, lane * 8) + load_f64(from, wd.sums * 8, lane * 8 + 512));
        }
        if (lane == 0) hats[q] = acc_hat;
      }
    }
    __syncthreads();
    const uint32_t m = lane < n + 1 ? lane : n + 1;
    d = tested_norm(A, sums[m], NORM == 2 ? hats[m] : 0.0);
    code = event_code(A, d, dl, khat, now.k);
  }
  const uint64_t sent = __ballot(code == 1);               // bit t: member t
  const uint64_t some = TOPK ? __ballot(code == 2) : 0;
  uint32_t place = 0, count = 0, msg_off = 0;
  if (TOPK) {
    const uint32_t equal = so_far.y + (in_chunk >> 16), equal2 = so_far2.y + (in_chunk2 >> 16);
    place = so_far.x + (in_chunk & 0xFFFFu) + (equal < ties ? equal : ties);
    const uint32_t end = so_far2.x + (in_chunk2 & 0xFFFFu) + (equal2 < ties ? equal2 : ties);
    const LayerDesc& ld = T.layers[layer];
    count = thr == kNoThreshold ? 0u : (wd.j0 + (wave + 1) * 256 < ld.numel ? end : ld.K) - place;
    msg_off = ld.msg_off;
  }
  // a neighbour's send fills a mailbox for good (a workgroup that reads a flag after it has been booked sees what it
  // would have computed)
  const uint64_t vl = __ballot(fl != 0) | sent << 1, vr = __ballot(fr != 0) | sent >> 1;

  // ---- update ----
  auto bit = [](uint64_t m, uint32_t t) { return ((m >> t) & 1u) != 0; };
  const float third = 0.333333343f;   // (float)(1/3): the ring's mixing weight
  // what the neighbours of a worker hold of it from this iteration on: h, where h[n] is the worker's behind the part
  Quad left{};
  uint32_t touched = 0, wins[TOPK ? N : 1];                // bit t: member t sends something of this lane's 64 bytes
  auto mark = [&](uint32_t v, uint32_t t) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)t); };
  auto communicate = [&](uint32_t t, const Quad& x, Quad& h) {
    h = either(bit(sent, t), x, h);
    uint32_t win = 0;
    if (TOPK && bit(some, t)) {                            // uniform
      win = counted_winners(winners4(x.v, h.v, A.topk_key, mark(thr, t), mark(cut, t), wd.j0 + e, nv), mark(count, t));
      take_winners(win, x.v, h.v);
    }
    if (TOPK) touched |= bit(sent, t) || any_of_line_part(win) ? 1u << t : 0u;
    return win;
  };
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t win = communicate(i + 1, x[i], h[i]);
    if (TOPK) wins[i] = win;
  }
  if (!closed) {
    (void)communicate(0, end_x[0], end_h[0]);
    (void)communicate(n + 1, end_x[1], end_h[1]);
  }
  const Quad right = either(closed, h[0], end_h[1]);
  if (TOPK && closed) touched |= (touched >> n & 1u) | (touched >> 1 & 1u) << (n + 1);       // members 0 and n + 1 are n and 1
  if (closed) {
#pragma unroll
    for (int i = 0; i < N; ++i) left = either((uint32_t)i + 1 == n, h[i], left);
  } else left = end_h[0];
  if (n < (uint32_t)N) {
#pragma unroll
    for (int i = 1; i < N; ++i) h[i] = either((uint32_t)i == n, right, h[i]);
  }
  // All loads are waited for here, ahead of the first store: a wait for a load further down, in the branches, would be one for
  // the stores before it too.
  __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0)
  double acc[N], acc_hat[NORM == 3 ? N : 1];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    acc[i] = 0.0;
    if (NORM == 3) acc_hat[i] = 0.0;
    // (lanes' values are read where all lanes have them: not below, where some are switched off)
    const uint32_t my_place = TOPK ? mark(place, i + 1) : 0u, my_count = TOPK ? mark(count, i + 1) : 0u, my_anchor = TOPK ? mark(anchor, i + 1) : 0u;
    if ((uint32_t)i < n && e < wd.len) {
      const uint32_t at = first + i * row;
      const Quad& er = i + 1 < N ? h[i + 1 < N ? i + 1 : 0] : right;
      if (TOPK) {
        if (bit(some, i + 1)) (void)put_message<true>(T, r0 + i, msg_off, my_place, my_count, wins[i], x[i].v, wd.j0 + e);
        if (touched >> (i + 1) & 1u) store_at(R.xhat, at, h[i]);
        if (touched >> i & 1u) store_at(R.mbox_l, at, left);
        if (touched >> (i + 2) & 1u) store_at(R.mbox_r, at, er);
      } else {
        if (bit(sent, i + 1)) store_at(R.xhat, at, h[i]);
        if (bit(sent, i)) store_at(R.mbox_l, at, left);
        if (bit(sent, i + 2)) store_at(R.mbox_r, at, er);
      }
      Quad z = g[GRADBUF ? i : 0];
      if (!GRADBUF) {
        const float4 w = draws[i * kThreads + threadIdx.x];
        z.v[0] = w.x; z.v[1] = w.y; z.v[2] = w.z; z.v[3] = w.w;
      }
      const bool has_l = bit(vl, i + 1), has_r = bit(vr, i + 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool in = (uint32_t)q < nv;                  // lanes past the tensor's end are padding: left as they are
        const float vn = A.plain_sgd ? z.v[q] : __builtin_fmaf(A.mu, v[i].v[q], z.v[q]);
        const float a = (has_l ? (left.v[q] - x[i].v[q]) : 0.0f) + (has_r ? (er.v[q] - x[i].v[q]) : 0.0f);
        const float cns = __builtin_fmaf(a, third, x[i].v[q]);
        const float xnew = __builtin_fmaf(-A.lr, vn, cns);
        x[i].v[q] = in ? xnew : x[i].v[q];
        v[i].v[q] = in ? vn : v[i].v[q];
        const float m = in ? (NORM == 1 ? x[i].v[q] - h[i].v[q] : x[i].v[q]) : 0.0f;
        acc[i] += (double)m * (double)m;                   // in lane order, padding adds zero
        if (NORM == 3) {
          const float m2 = in ? h[i].v[q] : 0.0f;
          acc_hat[i] += (double)m2 * (double)m2;
        }
      }
      if (TOPK) {
        const Bins bins = first_bins(x[i].v, h[i].v, A.topk_key, my_anchor);
        *reinterpret_cast<uint32_t*>(T.codes + (at >> 2)) = bins.codes;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t c = (bins.codes >> (8 * q) & 255u) - kFirstCode;      // (past the window: one bin for all above)
          if ((uint32_t)q < nv && (int)c >= 0) atomicAdd(&counts[i * (kCodeBins + 1) + (c < kCodeBins ? c : kCodeBins)], 1u);
        }
      }
      store_at(R.x, at, x[i]);
      if (!A.plain_sgd) store_at(R.vel, at, v[i]);
      if (!closed && (i == 0 || (uint32_t)i + 1 == n)) store_at(to_snap, at, x[i]);
    }
    left = h[i];
  }
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    const double s = N == 1 ? wave_sum_dpp(acc[0]) : wave_sums4(acc[i], acc[i + (N > 1)], acc[i + (N > 2 ? 2 : 0)], acc[i + (N > 2 ? 3 : 0)]);
    if ((lane & 15u) == 0 && lane < 16u * (N < 4 ? N : 4)) ws[4 * (i + (lane >> 4)) + wave] = s;      // row q: worker i + q
    if (NORM == 3) {
      const double s2 = N == 1 ? wave_sum_dpp(acc_hat[0])
                               : wave_sums4(acc_hat[i], acc_hat[i + (N > 1)], acc_hat[i + (N > 2 ? 2 : 0)], acc_hat[i + (N > 2 ? 3 : 0)]);
      if ((lane & 15u) == 0 && lane < 16u * (N < 4 ? N : 4)) ws_hat[4 * (i + (lane >> 4)) + wave] = s2;
    }
  }
  __syncthreads();
  if (threadIdx.x < n) {
    const double* p = ws + 4 * threadIdx.x;
    (turn ? R.partials[0] : R.partials[1])[(size_t)(r0 + threadIdx.x) * R.sums_row + wd.slot] = ((p[0] + p[1]) + p[2]) + p[3];
    if (NORM == 3) {
      const double* ph = ws_hat + 4 * threadIdx.x;
      T.partials_hat[(size_t)(r0 + threadIdx.x) * R.sums_row + wd.slot] = ((ph[0] + ph[1]) + ph[2]) + ph[3];
    }
  }
  if (TOPK) {
    for (uint32_t b = threadIdx.x; b < n * (kCodeBins + 1); b += kThreads) {
      const uint32_t i = b / (kCodeBins + 1), c = counts[b];
      // (eight copies: additions to one address take some 30 ns each, and a long tensor has hundreds of windows)
      if (c) atomicAdd(T.hist + (size_t)((r0 + i) * R.L + layer) * kHistBins + (blockIdx.x & 7u) * kCodeStride + (b - i * (kCodeBins + 1)), c);
    }
  }

  // ---- the outcome of the tests is booked, a worker a lane ----
  if (R.clocks && threadIdx.x == 0) *clock = PartClock{now.k + 1, now.steps + 1};
  if (!TESTS) end_replayable(T, A);
  if (TESTS) {
    if (wd.books && wave == 3 && lane >= 1 && lane <= n) {
      T.delta_out = turn ? R.delta[0] : R.delta[1];
      T.last_event_out = turn ? R.last_event[0] : R.last_event[1];
      T.xhat_sq = turn ? R.xhat_sq[1] : R.xhat_sq[0];
      T.xhat_sq_out = turn ? R.xhat_sq[0] : R.xhat_sq[1];
      book_test<false>(T, A, mseg, d, dl, khat, (uint8_t)code, sums[lane], now.k);
      if (bit(sent, lane - 1)) R.valid_l[mseg] = 1;
      if (bit(sent, lane + 1)) R.valid_r[mseg] = 1;
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
      T.it->k = now.k;
      T.it->k_next = now.k + 1;
      T.it->iters = now.steps + 1;
      if (now.k >= T.decay_len && replayed) T.it->overflow = 1;
    }
  }
}

template <int NORM, bool TESTS, int N, bool TOPK>
static void part(const Tables& t, const StepArgs& a, const PartArgs& r, uint32_t count, uint32_t dist, uint32_t grad_mode,
                 hipStream_t s) {
  const dim3 grid(count, (t.P + a.part - 1) / a.part), block(kThreads);
  if (grad_mode == 1) k_update_part<0, true, NORM, TESTS, N, TOPK><<<grid, block, 0, s>>>(r, a, t);
  else if (dist == 0) k_update_part<0, false, NORM, TESTS, N, TOPK><<<grid, block, 0, s>>>(r, a, t);
  else k_update_part<1, false, NORM, TESTS, N, TOPK><<<grid, block, 0, s>>>(r, a, t);
}

template <int NORM, bool TESTS, bool TOPK = false>
static hipError_t part_of(const Tables& t, const StepArgs& a, const PartArgs& r, uint32_t count, uint32_t dist,
                          uint32_t grad_mode, hipStream_t s) {
  if (a.part <= 1) part<NORM, TESTS, 1, TOPK>(t, a, r, count, dist, grad_mode, s);
  else if (a.part <= 2) part<NORM, TESTS, 2, TOPK>(t, a, r, count, dist, grad_mode, s);
  else if (a.part <= 4) part<NORM, TESTS, 4, TOPK>(t, a, r, count, dist, grad_mode, s);
  else if (a.part <= kPartMost && !TOPK) part<NORM, TESTS, (int)kPartMost, TOPK && false>(t, a, r, count, dist, grad_mode, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_part(const Tables& t, const StepArgs& a, const PartTables& p, uint32_t dist, uint32_t grad_mode, int norm, hipStream_t s) {
  PartArgs r{};
  const uint32_t count = p.count;
  r.windows = p.windows;
  r.clocks = p.clocks;
  for (int i = 0; i < 2; ++i) {
    r.partials[i] = p.set[i].partials;
    r.delta[i] = p.set[i].delta;
    r.last_event[i] = p.set[i].last_event;
    r.xhat_sq[i] = p.set[i].xhat_sq;
  }
  r.x = t.x; r.xhat = t.xhat; r.vel = t.vel; r.mbox_l = t.mbox_l; r.mbox_r = t.mbox_r;
  r.xsnap = t.xsnap;
  r.valid_l = t.valid_l; r.valid_r = t.valid_r; r.fired = t.fired;
  r.row = (uint32_t)t.Npad;
  r.sums_row = t.C * t.SW;
  r.P = t.P; r.L = t.L;
  if (a.topk_on) return norm == 1   ? part_of<1, false, true>(t, a, r, count, dist, grad_mode, s)
                        : norm == 3 ? part_of<3, false, true>(t, a, r, count, dist, grad_mode, s)
                                    : hipErrorInvalidValue;
  if (norm == 1) return a.one_launch ? part_of<1, true>(t, a, r, count, dist, grad_mode, s)
                                     : part_of<1, false>(t, a, r, count, dist, grad_mode, s);
  if (norm == 2) return a.one_launch ? part_of<2, true>(t, a, r, count, dist, grad_mode, s)
                                     : part_of<2, false>(t, a, r, count, dist, grad_mode, s);
  return hipErrorInvalidValue;
}

}  // namespace evg
