// The update pass of rings that stream from memory and send Top-K messages, or are too large for kernels_ring.hip (same work and results as k_update): one
// workgroup owns a window of one tensor and walks it around the ring, worker by worker.
//
// What a worker last received from a neighbour IS that neighbour's xhat (same-iteration delivery, only sent entries count as
// communicated), and the walk has both neighbours' xhat in registers when it comes to a worker: x, velocity
// and xhat are read once, the mailboxes never, and a send -- whole, or the winners of a Top-K selection -- is written to
// xhat and both mailboxes from the registers that hold it, without a copy kernel.  Nobody else touches the window, so
// there is nothing to wait for.  The next worker's loads are under way while one is updated.
//
// Bound by memory: 20 bytes per element (12 read), 8 more where a tensor is sent whole, messages and the 64-byte groups they
// touch.  It moves them at 4.9 - 5.3 TB/s.  On this card a large copy reaches 4.8, two reads to a write 5.9, reads alone
// 6.3, and this pass writes about as much as it reads, or more.  Steps before (a pass per worker that read
// the neighbours through the L2, and a copy kernel) -> now: 16 ResNet-18 workers with whole sends 925 -> 868 us, 32 with plain
// SGD 1569 -> 1222, 7 of width 23 65.8 -> 54.0, 8 ResNet-50 workers of half width 343 -> 287.
// Residency: whole sends 76 - 93 vector registers and 2 KB of LDS, 5 or 6 wavefronts a SIMD; Top-K 106 - 126 and 20 or 24 KB for
// eight wavefronts, 4 a SIMD; with mailboxes read (RESET) 130 - 146, 3.  Most use 106 scalar registers and spill
// some tens of them to vector lanes: what more a Top-K walk keeps per worker costs 1 - 5 % at once, so that the number of winners in a
// group and whether codes are wanted ride with the other marks.
#include "message_device.h"
#include "quad_device.h"
#include "trigger_device.h"

namespace evg {

// Accesses are non-temporal: every line is touched once (ordinary stores: 1100 -> 1360 us with Top-K 10 % of 16 workers,
// ordinary loads: 2 .. 9 % slower).

// A copy that stays where it is written: the registers of the original are free for the next load from
// here on (left to itself the compiler loads elsewhere and moves the values at the loop's end, which
// waits there for loads that are wanted an iteration later).
__device__ __forceinline__ Quad taken(const Quad& q) {
  Quad c;
#pragma unroll
  for (int i = 0; i < 4; ++i) asm volatile("v_mov_b32 %0, %1" : "=v"(c.v[i]) : "v"(q.v[i]));
  return c;
}

// What the walk has to know of a worker; lane i of a wavefront holds the i-th worker's.
struct Marks { uint32_t f, thr, cut, place, anchor; };   // f: see below; Top-K: threshold key, last element that wins a tie, place in
                                                 // the message of the first winner of this wavefront's group, anchor of its key codes
constexpr uint32_t kCode = 3u, kLeftFilled = 4u, kRightFilled = 8u, kSpike = 16u, kLed = 32u, kCoded = 64u;
constexpr int kCountShift = 8;                   // and from bit 8 on the winners in the group

// RESET (with TOPK; the whole ring in one part): an event resets the sender's xhat to x while the mailboxes take the sent
// entries only, so a mailbox is not its sender's xhat and is read, 8 bytes more per element: its winners are taken from the
// sender's x, which the walk has at hand.  16 ResNet-18 workers with Top-K 1 % and 10 %: 1355 and 1521 us a step, where
// a pass ahead that puts the messages into the mailboxes and an update pass per worker take 1517 and 1817.
template <int DIST, bool GRADBUF, int NORM, bool TOPK, bool HISTA, int W, bool RESET = false>
__global__ __launch_bounds__(64 * W) void k_update_walk(Tables T, StepArgs A) {
  constexpr uint32_t kElems = 256 * W, SPW = W / 4;
  __shared__ double ws[NORM ? 64 * W : 1], ws_hat[NORM == 3 ? 64 * W : 1];
  __shared__ __attribute__((aligned(16))) uint32_t hist[HISTA ? 2 * kFirstBins + 4 : 4];
  const uint32_t groups = T.SW / SPW;
  // Workgroups go to the eight XCDs in turn by their number.  Where the pass counts keys, each XCD takes a contiguous
  // eighth of the windows, so that the counts of a tensor are added in one L2 (8 ResNet-50 workers 1019 -> 944 us;
  // without that work consecutive windows are better left in turn, 1249 against 1300 us).
  const uint32_t all = T.C * groups, each = (all + 7) / 8;
  const uint32_t window_no = HISTA ? (blockIdx.x & 7u) * each + (blockIdx.x >> 3) : blockIdx.x;
  if (window_no >= all || (HISTA && (blockIdx.x >> 3) >= each)) return;         // uniform
  const uint32_t c = window_no / groups, sub0 = (window_no % groups) * SPW;
  const ChunkDesc cd = T.chunks[c];
  if (sub0 * kSweep >= cd.len + cd.lead) return;                   // uniform (its sums are zero for good)
  const uint32_t P = T.P, layer = cd.layer, k_iter = step_k(T, A);
  end_replayable(T, A);
  const uint32_t r0 = blockIdx.y * A.part, n = P - r0 < A.part ? P - r0 : A.part;   // workers r0 .. r0 + n - 1
  const bool closed = n == P;                            // the part is the whole ring
  const uint32_t skip = sub0 == 0 ? cd.lead : 0u, first = sub0 * kSweep + skip - cd.lead;   // first element of the window
  const uint32_t left_over = cd.len - first;
  const uint32_t here = left_over < kElems - skip ? left_over : kElems - skip;   // elements of the window
  const uint32_t nb = (here + 3) / 4 * 16;               // its bytes (tensors are padded to 4 elements)
  const size_t off = (size_t)cd.off + first;
  const uint32_t e = threadIdx.x * kLaneElems - skip;    // positions before the first element wrap around: past the end
  const uint32_t byte = e < here ? e * 4 : kNowhere;
  const uint32_t nv = e >= here ? 0u : here - e < 4u ? here - e : 4u;
  const uint32_t j = cd.j0 + first + e;
  const float third = 0.333333343f;   // (float)(1/3): the ring's mixing weight
  const float sg = GRADBUF ? 0.0f : (float)(T.layers[layer].sig_base * step_decay(T, A));
  const uint32_t nb_vel = A.plain_sgd ? 0u : nb;
  const uint32_t msg_off = TOPK ? T.layers[layer].msg_off : 0u;
  auto at = [&](float* arena, uint32_t s) { return arena + (size_t)s * T.Npad + off; };
  auto worker = [&](uint32_t i) { return r0 + i < P ? r0 + i : r0 + i - P; };   // i <= n

  // the i-th worker of the part, i = n: the one after it
  auto marks_of = [&](uint32_t i) {
    Marks m{0u, kNoThreshold, 0u, 0u, kNoAnchor};
    if (i <= n) {
      const uint32_t s = worker(i), seg = s * T.L + layer, code = T.fired[seg];
      m.f = code | (T.valid_l[seg] ? kLeftFilled : 0u) | (T.valid_r[seg] ? kRightFilled : 0u);
      if (!GRADBUF && has_spike(A, k_iter, s)) m.f |= kSpike;
      if (HISTA) {
        m.anchor = T.anchor[seg];
        if (T.codes && !(m.anchor & kUncoded)) m.f |= kCoded;
        m.anchor &= kAnchorBits;
      }
      if (is_led(T, A, s)) m.f |= kLed;
      else if (TOPK && code == 2) {
        m.thr = T.sel_prefix[seg];
        m.cut = T.sel_cut[seg];
        const Place p = message_place<HISTA>(T, s * T.C + c, cd, T.layers[layer], sub0 * 4 + wave_id(), T.sel_krem[seg]);
        m.place = p.first;
        if (HISTA && m.thr != kNoThreshold) m.f |= p.count << kCountShift;
      }
    }
    return m;
  };
  uint32_t base = 0;
  Marks cur = marks_of(lane_id()), nxt = cur;
  if (n >= 64) nxt = marks_of(64 + lane_id());
  auto read_mark = [&](uint32_t a, uint32_t b, uint32_t i) {
    return (uint32_t)__builtin_amdgcn_readlane((int)(i - base < 64 ? a : b), (int)((i - base) & 63u));
  };

  // What worker s's neighbours hold of it from this iteration on, written to its xhat (to_hat bytes) and its
  // neighbours' mailboxes (to_right, to_left bytes) if it sends.
  // RESET: to its xhat only; `sent`, one bit per element, says what the neighbours take.
  uint32_t sent = 0;
  auto send = [&](uint32_t s, uint32_t f, uint32_t thr, uint32_t cut, uint32_t place, uint32_t to_hat, uint32_t to_left, uint32_t to_right,
                  const Quad& x, const Quad& h) {
    Quad q;
    uint32_t where = byte;
    if (RESET) {
      uint32_t win = winners4(x.v, h.v, A.topk_key, thr, cut, j, nv);
      if (to_hat) win = put_message<HISTA>(T, s, msg_off, place, f >> kCountShift, win, x.v, j);
      const bool sends = (f & kCode) != 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) q.v[i] = sends ? x.v[i] : h.v[i];
      store_quad<true>(at(T.xhat, s), sends ? to_hat : 0u, byte, q);
      sent = (f & kCode) == 1 ? (1u << nv) - 1u : win;
      return q;
    }
    const bool led = (f & kLed) != 0, whole = (f & kCode) == 1 && !led;
    if (TOPK) {
      // (workers at the ends of parts: k_topk_apply has done all this but the mailboxes)
      uint32_t win = winners4(x.v, h.v, A.topk_key, thr, cut, j, nv);
      if (to_hat) win = put_message<HISTA>(T, s, msg_off, place, f >> kCountShift, win, x.v, j);
#pragma unroll
      for (int i = 0; i < 4; ++i) q.v[i] = whole || ((win >> i) & 1u) ? x.v[i] : h.v[i];
      if (!whole && !led && !any_of_line_part(win)) where = kNowhere;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) q.v[i] = whole ? x.v[i] : h.v[i];
    }
    const bool sends = (f & kCode) != 0;
    store_quad<true>(at(T.xhat, s), sends && !led ? to_hat : 0u, where, q);
    store_quad<true>(at(T.mbox_l, s + 1 == P ? 0u : s + 1), sends ? to_right : 0u, where, q);
    store_quad<true>(at(T.mbox_r, s == 0 ? P - 1 : s - 1), sends ? to_left : 0u, where, q);
    return q;
  };
  // does the walk need xhat from memory?  (not where the whole tensor has just been sent)
  auto reads_hat = [](uint32_t f) { return (f & kCode) != 1 || (f & kLed) != 0; };

  const HistAt counts = HISTA ? first_hist(T, layer, blockIdx.x & 7u) : HistAt{0, 0};
  if (HISTA) {
    for (uint32_t b = threadIdx.x; b < 2 * kFirstBins + 4; b += 64 * W) hist[b] = 0;
    __syncthreads();
  }
  const bool dead = !HISTA && wave_id() * 256u >= here + skip;      // wave-uniform
  if (NORM && dead) {
    ws[lane_id() * W + wave_id()] = 0.0;
    if (NORM == 3) ws_hat[lane_id() * W + wave_id()] = 0.0;
  }

  // The last worker whose x / xhat the loop below loads.  A closed ring's last worker is among the
  // first two that are loaded and stays in registers, an open part ends with the xhat of the worker after it.
  const uint32_t last_x = closed ? n - 2 : n - 1, last_h = closed ? n - 2 : n;
  Quad x1{}, h1{}, v1{}, g1{}, xc{}, ec{}, el{}, x_last{}, e_last{}, e_first{};
  // RESET: the next worker's mailboxes; x before its update, and what it sent, of the worker before, the first and the last
  Quad ml1{}, mr1{}, xl{}, x_first{};
  uint32_t sent_l = 0, sent_c = 0, sent_first = 0, sent_last = 0;
  auto mailbox = [&](float* m, uint32_t s, uint32_t f, uint32_t filled) { return load_quad<true>(at(m, s), f & filled ? nb : 0u, byte); };
  auto receive = [&](float* m, uint32_t s, uint32_t sent, const Quad& from, Quad& held) {
    take_winners(sent, from.v, held.v);
    store_quad<true>(at(m, s), nb, any_of_line_part(sent) ? byte : kNowhere, held);
  };
  if (!dead) {
    const uint32_t before = r0 == 0 ? P - 1 : r0 - 1;
    x_last = load_quad<true>(at(T.x, before), closed ? nb : 0u, byte);
    xc = load_quad<true>(at(T.x, r0), nb, byte);
    x1 = load_quad<true>(at(T.x, worker(1)), 1 <= last_x ? nb : 0u, byte);
    v1 = load_quad<true>(at(T.vel, r0), nb_vel, byte);
    if (GRADBUF) g1 = load_quad<true>(A.grad + (size_t)r0 * T.Npad + off, nb, byte);
    const uint32_t seg_b = before * T.L + layer;
    uint32_t f_b = __builtin_amdgcn_readfirstlane((int)T.fired[seg_b]);
    if (is_led(T, A, before)) f_b |= kLed;
    uint32_t thr_b = kNoThreshold, cut_b = 0u, place_b = 0u;
    if (TOPK && f_b == 2) {
      thr_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)T.sel_prefix[seg_b]);
      cut_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)T.sel_cut[seg_b]);
      const Place p = message_place<HISTA>(T, before * T.C + c, cd, T.layers[layer], sub0 * 4 + wave_id(), T.sel_krem[seg_b]);
      place_b = p.first;
      if (HISTA && thr_b != kNoThreshold) f_b |= (uint32_t)__builtin_amdgcn_readfirstlane((int)p.count) << kCountShift;
    }
    const uint32_t f0 = read_mark(cur.f, nxt.f, 0);
    const Quad h_last = load_quad<true>(at(T.xhat, before), reads_hat(f_b) ? nb : 0u, byte);
    const Quad h0 = load_quad<true>(at(T.xhat, r0), reads_hat(f0) ? nb : 0u, byte);
    h1 = load_quad<true>(at(T.xhat, worker(1)), 1 <= last_h && reads_hat(read_mark(cur.f, nxt.f, 1)) ? nb : 0u, byte);
    if (RESET) {
      ml1 = mailbox(T.mbox_l, r0, f0, kLeftFilled);
      mr1 = mailbox(T.mbox_r, r0, f0, kRightFilled);
    }
    e_last = send(before, f_b, thr_b, cut_b, place_b, closed ? nb : 0u, closed ? nb : 0u, nb, x_last, h_last);
    sent_last = sent;
    e_first = send(r0, f0, read_mark(cur.thr, nxt.thr, 0), read_mark(cur.cut, nxt.cut, 0), read_mark(cur.place, nxt.place, 0), nb, closed ? nb : 0u,
                   closed || n > 1 ? nb : 0u, xc, h0);
    sent_first = sent;
    if (RESET) {
      xl = x_last;
      x_first = xc;
      sent_l = sent_last;
      sent_c = sent_first;
    }
    el = e_last;
    ec = e_first;
  }
  uint32_t f = read_mark(cur.f, nxt.f, 0), fn = read_mark(cur.f, nxt.f, 1);     // the marks of workers i and i + 1
  for (uint32_t i = 0; i < n; ++i) {
    const uint32_t r = r0 + i;
    if (i == base + 64) {
      base += 64;
      cur = nxt;
      nxt = marks_of(base + 64 + lane_id());
    }
    if (!dead) {
      // the next worker's values have arrived: take them, and ask for those of the one after it
      Quad xn = taken(x1), hn = taken(h1), vel = taken(v1), g = GRADBUF ? taken(g1) : g1;
      Quad ml = RESET ? taken(ml1) : ml1, mr = RESET ? taken(mr1) : mr1;
      const uint32_t f2 = read_mark(cur.f, nxt.f, i + 2);
      const uint32_t s1 = worker(i + 1), s2 = i + 2 <= n ? worker(i + 2) : 0u;
      const bool another = i + 1 < n;
      x1 = load_quad<true>(at(T.x, s2), i + 2 <= last_x ? nb : 0u, byte);
      h1 = load_quad<true>(at(T.xhat, s2), i + 2 <= last_h && reads_hat(f2) ? nb : 0u, byte);
      v1 = load_quad<true>(at(T.vel, another ? r + 1 : 0), another ? nb_vel : 0u, byte);
      if (GRADBUF) g1 = load_quad<true>(A.grad + (size_t)(another ? r + 1 : 0) * T.Npad + off, another ? nb : 0u, byte);
      if (RESET) {
        ml1 = mailbox(T.mbox_l, another ? r + 1 : 0, another ? fn : 0u, kLeftFilled);
        mr1 = mailbox(T.mbox_r, another ? r + 1 : 0, another ? fn : 0u, kRightFilled);
      }
      Quad en = send(s1, fn, read_mark(cur.thr, nxt.thr, i + 1), read_mark(cur.cut, nxt.cut, i + 1),
                     read_mark(cur.place, nxt.place, i + 1), i + 1 <= last_x ? nb : 0u, i + 1 <= last_h ? nb : 0u, i + 1 <= last_x && (closed || i + 2 < n) ? nb : 0u,
                     xn, hn);
      if (closed && i + 1 > last_x) {
        en = i + 1 == n ? e_first : e_last;
        xn = RESET && i + 1 == n ? x_first : x_last;
        sent = i + 1 == n ? sent_first : sent_last;
      }
      if (RESET) {
        receive(T.mbox_l, r, sent_l, xl, ml);
        receive(T.mbox_r, r, sent, xn, mr);
        xl = xc;
        sent_l = sent_c;
        sent_c = sent;
      }
      if (!GRADBUF) draw_gradient<DIST>(A, j, layer, k_iter, r, sg, (f & kSpike) != 0, g.v);
      const bool vl = (f & kLeftFilled) != 0, vr = (f & kRightFilled) != 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = (uint32_t)i < nv;      // lanes past the tensor's end are padding: left as they are
        const float vn = A.plain_sgd ? g.v[i] : __builtin_fmaf(A.mu, vel.v[i], g.v[i]);
        const float lv = RESET ? ml.v[i] : el.v[i], rv = RESET ? mr.v[i] : en.v[i];
        const float a = (vl ? (lv - xc.v[i]) : 0.0f) + (vr ? (rv - xc.v[i]) : 0.0f);
        const float cns = __builtin_fmaf(a, third, xc.v[i]);
        const float xnew = __builtin_fmaf(-A.lr, vn, cns);
        xc.v[i] = in ? xnew : xc.v[i];
        vel.v[i] = in ? vn : vel.v[i];
      }
      store_quad<true>(at(T.x, r), nb, byte, xc);
      store_quad<true>(at(T.vel, r), nb_vel, byte, vel);
      if (NORM) {
        double acc = 0.0, acc_hat = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {          // in lane order, padding adds zero
          const bool in = (uint32_t)i < nv;
          const float d = in ? (NORM == 1 ? xc.v[i] - ec.v[i] : xc.v[i]) : 0.0f, h = in ? ec.v[i] : 0.0f;
          acc += (double)d * (double)d;
          if (NORM == 3) acc_hat += (double)h * (double)h;
        }
        acc = wave_sum_dpp(acc);
        if (NORM == 3) acc_hat = wave_sum_dpp(acc_hat);
        if (lane_id() == 0) {
          ws[(i & 63u) * W + wave_id()] = acc;
          if (NORM == 3) ws_hat[(i & 63u) * W + wave_id()] = acc_hat;
        }
      }
      if (HISTA) {
        const uint32_t anchor = read_mark(cur.anchor, nxt.anchor, i);
        const Bins bins = first_bins(xc.v, ec.v, A.topk_key, anchor);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          atomicAdd(&hist[(uint32_t)q < nv ? (i & 1u) * kFirstBins + bins.bin[q] : 2 * kFirstBins], 1u);
        if (f & kCoded) store_codes(T, (size_t)r * T.Npad + off, nb, byte, bins.codes);
      }
      if (!RESET) el = ec;
      ec = en;
      xc = xn;
      f = fn;
      fn = f2;
    }
    if (HISTA) {
      // two histograms in turn: this barrier ends worker r's counting, and the clearing of the other one
      __syncthreads();
      uint32_t* gh = T.hist + (size_t)(counts.first + r * counts.step) * kHistBins;
      for (uint32_t b = threadIdx.x * 4; b < (uint32_t)kFirstBins; b += 256 * W) {
        u32x4* p = reinterpret_cast<u32x4*>(hist + (i & 1u) * kFirstBins + b);
        const u32x4 n = *p;
        if (n.x | n.y | n.z | n.w) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (n[i]) atomicAdd(gh + b + i, n[i]);
          *p = u32x4{0u, 0u, 0u, 0u};
        }
      }
    }
    if (NORM && ((i & 63u) == 63u || i == n - 1)) {          // uniform
      __syncthreads();
      const uint32_t done = (i & 63u) + 1;
      for (uint32_t q = threadIdx.x; q < done * SPW; q += 64 * W) {
        const uint32_t rr = q / SPW, u = q % SPW;
        const size_t slot = ((size_t)(r0 + (i & ~63u) + rr) * T.C + c) * T.SW + sub0 + u;
        const double* p = ws + rr * W + 4 * u;
        T.partials_out[slot] = ((p[0] + p[1]) + p[2]) + p[3];
        if (NORM == 3) {
          const double* ph = ws_hat + rr * W + 4 * u;
          T.partials_hat_out[slot] = ((ph[0] + ph[1]) + ph[2]) + ph[3];
        }
      }
      __syncthreads();
    }
  }
}

template <int NORM, bool TOPK, bool HISTA, int W, bool RESET = false>
static void walk(const Tables& t, const StepArgs& a, uint32_t dist, uint32_t grad_mode, hipStream_t s) {
  const dim3 grid((t.C * (t.SW / (W / 4)) + 7) / 8 * 8, (t.P + a.part - 1) / a.part), block(64 * W);
  if (grad_mode == 1) k_update_walk<0, true, NORM, TOPK, HISTA, W, RESET><<<grid, block, 0, s>>>(t, a);
  else if (dist == 0) k_update_walk<0, false, NORM, TOPK, HISTA, W, RESET><<<grid, block, 0, s>>>(t, a);
  else k_update_walk<1, false, NORM, TOPK, HISTA, W, RESET><<<grid, block, 0, s>>>(t, a);
}

hipError_t launch_walk(const Tables& t, const StepArgs& a, uint32_t dist, uint32_t grad_mode, int norm, hipStream_t s) {
  if (a.topk_on) {
    // Eight wavefronts share a histogram where chunks are long enough.  4 / 8 / 16, steps in us: 64 ResNet-18 workers - / 4923 /
    // 4762, 60 of width 28 978 / 950 / 1051, 20 of width 20 219 / 220 / 262, 8 ResNet-50 workers of half width 369 / 364 / 406, with
    // Student-t gradients 390 / 404 / 451, 12 perceptrons with given gradients 188 / 138 / 119.
    const bool wide = t.SW % 2 == 0;
    if (a.xhat_reset) {
      if (norm == 0) walk<0, true, false, 4, true>(t, a, dist, grad_mode, s);
      else if (norm == 1 && a.hist_fused) wide ? walk<1, true, true, 8, true>(t, a, dist, grad_mode, s) : walk<1, true, true, 4, true>(t, a, dist, grad_mode, s);
      else if (norm == 3 && a.hist_fused) wide ? walk<3, true, true, 8, true>(t, a, dist, grad_mode, s) : walk<3, true, true, 4, true>(t, a, dist, grad_mode, s);
      else return hipErrorInvalidValue;
    } else if (norm == 0) walk<0, true, false, 4>(t, a, dist, grad_mode, s);
    else if (norm == 1 && a.hist_fused) wide ? walk<1, true, true, 8>(t, a, dist, grad_mode, s) : walk<1, true, true, 4>(t, a, dist, grad_mode, s);
    else if (norm == 3 && a.hist_fused) wide ? walk<3, true, true, 8>(t, a, dist, grad_mode, s) : walk<3, true, true, 4>(t, a, dist, grad_mode, s);
    else return hipErrorInvalidValue;
  } else if (norm == 0) walk<0, false, false, 4>(t, a, dist, grad_mode, s);
  else if (norm == 1) walk<1, false, false, 4>(t, a, dist, grad_mode, s);
  else if (norm == 2) walk<2, false, false, 4>(t, a, dist, grad_mode, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace evg
