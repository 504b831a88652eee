// The two streaming passes over every element: the fused neighbour-averaging +
// momentum-SGD update (Section 3, Eq. 2 with the last received neighbour values
// of Section 4), which also accumulates the squared drift || x - xhat ||^2 that the
// next iteration's trigger test needs, and a stand-alone drift-norm pass.
//
// Streaming rings with ordinary delivery are updated by kernels_walk.hip, cached rings by kernels_parts.hip; k_update here serves
// the others: cached Top-K rings with tensors too long for k_topk_choose, norm passes of their own, delayed delivery, xhat
// reset at events.  One workgroup (256 threads, one float4 per thread) owns one 1024-element sweep of one chunk of one
// worker; where the pass also builds the histogram of a Top-K ring, two.  With given gradients and copies of x it has 95 vector
// registers; more than 96 are too many for five wavefronts a SIMD (97: 5 perceptrons of 479 000 elements 53.5 -> 56.7 us a step).
#include "message_device.h"
#include "trigger_device.h"

namespace evg {

__device__ __forceinline__ float4 ld4(const float* p) { return ld4s(p); }

// NORMDIFF: the trigger compares ||x|| with ||xhat||: two sums instead of the drift's.
template <bool NORMDIFF>
__global__ __launch_bounds__(kThreads) void k_norm(Tables T) {
  __shared__ double ws[4];
  const uint32_t c = blockIdx.x / T.SW, sub = blockIdx.x % T.SW, r = blockIdx.y;
  const ChunkDesc cd = T.chunks[c];
  const size_t base = (size_t)r * T.Npad + cd.off;
  const uint32_t e = sub * kSweep + threadIdx.x * kLaneElems - cd.lead;   // positions before the lead wrap around
  double acc = 0.0, acc_hat = 0.0;
  if (e < cd.len) {
    const float4 x4 = ld4(T.x + base + e), h4 = ld4(T.xhat + base + e);
    const float xa[4] = {x4.x, x4.y, x4.z, x4.w}, ha[4] = {h4.x, h4.y, h4.z, h4.w};
    const uint32_t nv = cd.len - e < 4u ? cd.len - e : 4u;
    if (NORMDIFF) { square_acc(acc, xa, nv); square_acc(acc_hat, ha, nv); }
    else drift_acc(acc, xa, ha, nv);
  }
  const size_t slot = (((size_t)r * T.C + c) * T.SW + sub) * T.fine;
  const double total = block_sum(acc, ws);
  if (threadIdx.x == 0) T.partials_out[slot] = total;
  if (NORMDIFF) {
    const double total_hat = block_sum(acc_hat, ws);
    if (threadIdx.x == 0) T.partials_hat_out[slot] = total_hat;
  }
}

// Workgroup sums of SPW values at once (one barrier pair); each in the association
// order of block_sum.  `ws` is 4 * SPW doubles of LDS.
template <int SPW>
__device__ __forceinline__ void block_sums(const double v[SPW], double* ws, double total[SPW]) {
#pragma unroll
  for (int u = 0; u < SPW; ++u) {
    const double s = wave_sum(v[u]);
    if (lane_id() == 0) ws[u * 4 + wave_id()] = s;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < SPW; ++u) total[u] = ((ws[u * 4] + ws[u * 4 + 1]) + ws[u * 4 + 2]) + ws[u * 4 + 3];
  __syncthreads();
}

// DIST: 0 normal (one Philox block per float4), 1 Student-t(3) (two blocks per float4).
// GRADBUF: gradients come from a caller buffer.
// NORM: what the pass accumulates for the next trigger test: 0 nothing, 1 the sweep's squared
// drift, 2 its squared x (xhat is then not read at all), 3 its squared x and squared xhat.
// TOPK: Top-K messages of this iteration: my own is told from x and xhat as they pass through the registers, written to
// the message buffers and applied to xhat; a neighbour's (PULL) from the copy of its x and from my mailbox.
// (TOPK with NORM also leaves the codes of the new rank keys, if the ring keeps any: one that streams.)
// HISTA: also histogram the new rank keys per tensor, the first
// radix pass of the next iteration's Top-K selection, while the values are in registers.
// SPW: consecutive sweeps of a chunk per workgroup (one float4 per thread and sweep).  Two halve the cost of
// clearing and merging the histogram.
// STREAM: non-temporal accesses to the arenas (rings larger than the last-level cache).
// PULL: whole-tensor sends of this iteration have NOT been copied into the mailboxes: where a
// neighbour sent, its values are fetched from the copy of x that the previous update pass left
// (x itself is being overwritten by its owner in this very launch), used, and written into the
// mailbox here; and the new x is also written to the other of the two copies for the next
// iteration (two copies in turn: the one read now is written by nobody in this launch).  Fewer
// launches per iteration for rings that live in the cache, where launches are what costs.
// FINE: it goes by the bins of first_bins, else by the upper 11 bits of a key (cached rings without anchors).
template <int DIST, bool GRADBUF, int NORM, bool TOPK, bool HISTA, int SPW, bool STREAM, bool PULL = false, bool FINE = true>
__global__ __launch_bounds__(kThreads) void k_update(Tables T, StepArgs A) {
  __shared__ double ws[4 * SPW];
  constexpr uint32_t BINS = FINE ? kFirstBins : kHistBins;
  __shared__ uint32_t hA[HISTA ? BINS : 1];
  const uint32_t groups = T.SW / SPW;      // workgroups per chunk (SW is a multiple of SPW)
  const uint32_t c = blockIdx.x / groups, sub0 = (blockIdx.x % groups) * SPW, r = blockIdx.y;
  const ChunkDesc cd = T.chunks[c];
  const uint32_t seg = r * T.L + cd.layer;
  const bool vl = T.valid_l[seg] != 0, vr = T.valid_r[seg] != 0;
  const uint32_t lw = (r + T.P - 1) % T.P, rw = (r + 1) % T.P;
  const uint32_t my_event = T.fired[seg];
  // what did my neighbours send of this tensor in this iteration? (then vl / vr are set)
  bool from_l = false, from_r = false, some_l = false, some_r = false;   // all / some of their tensor
  if (PULL) {
    const uint32_t fl = T.fired[lw * T.L + cd.layer], fr = T.fired[rw * T.L + cd.layer];
    from_l = fl == 1;
    from_r = fr == 1;
    some_l = TOPK && fl == 2;
    some_r = TOPK && fr == 2;
  }
  // step n reads copy (n-1) & 1 of x and writes copy n & 1; the kernel that ran the tests has counted this step already
  const size_t arena = (size_t)T.P * T.Npad;
  const uint64_t step_no = PULL ? T.it->iters : 0;
  const float* snap_in = PULL ? T.xsnap + ((step_no + 1) & 1) * arena : nullptr;
  float* snap_out = PULL ? T.xsnap + (step_no & 1) * arena : nullptr;
  // xhat := x for the whole tensor: after a whole send, or after any event when a Top-K
  // event is read as resetting the tensor's xhat
  const bool sent_whole = my_event == 1 || (TOPK && A.xhat_reset && my_event == 2);
  const size_t base = (size_t)r * T.Npad + cd.off;
  const float third = 0.333333343f;   // (float)(1/3): the ring's mixing weight
  const uint32_t k_iter = step_k(T, A);
  end_replayable(T, A);
  uint32_t e[SPW];
  bool live[SPW];
#pragma unroll
  for (int u = 0; u < SPW; ++u) {
    e[u] = (sub0 + u) * kSweep + threadIdx.x * kLaneElems - cd.lead;
    live[u] = e[u] < cd.len;
  }
  double acc[SPW], acc_hat[SPW];
#pragma unroll
  for (int u = 0; u < SPW; ++u) { acc[u] = 0.0; acc_hat[u] = 0.0; }
  if (sub0 * kSweep < cd.len + cd.lead) {        // uniform: the window holds elements
    float xa[SPW][4], va[SPW][4], la[SPW][4], ra[SPW][4], ha[SPW][4], g[SPW][4];
    float hat_was[TOPK ? SPW : 1][4];                    // xhat before this iteration's event
    uint32_t nv[SPW];
    float lx[TOPK && PULL ? SPW : 1][4], rx[TOPK && PULL ? SPW : 1][4];   // the neighbours' x before this iteration's update
    // selections of mine and the neighbours' tensors, asked for early: nobody waits for them until the arenas are there
    uint32_t thr[3], cut[3], moff = 0;
    Place place[SPW];
    const uint32_t anchor = TOPK && NORM && FINE ? T.anchor[seg] : kNoAnchor;
    if (TOPK) {
      const uint32_t segs[3] = {seg, PULL ? lw * T.L + cd.layer : seg, PULL ? rw * T.L + cd.layer : seg};
#pragma unroll
      for (int i = 0; i < 3; ++i) { thr[i] = T.sel_prefix[segs[i]]; cut[i] = T.sel_cut[segs[i]]; }
      moff = T.layers[cd.layer].msg_off;
#pragma unroll
      for (int u = 0; u < SPW; ++u) place[u] = message_place<STREAM && NORM != 0>(T, r * T.C + c, cd, T.layers[cd.layer], (sub0 + u) * 4 + wave_id(), T.sel_krem[seg]);
    }
    auto receive = [&](uint32_t thr, uint32_t cut, const float (*sx)[4], float* mbox, float (*a)[4]) {
#pragma unroll
      for (int u = 0; u < SPW; ++u) {
        const uint32_t win = winners4(sx[u], a[u], A.topk_key, thr, cut, cd.j0 + e[u], nv[u]);
        take_winners(win, sx[u], a[u]);
        if (any_of_line_part(win) && live[u]) st4t<STREAM>(mbox + base + e[u], make_float4(a[u][0], a[u][1], a[u][2], a[u][3]));
      }
    };
#pragma unroll
    for (int u = 0; u < SPW; ++u) {
#pragma unroll
      for (int i = 0; i < 4; ++i) { xa[u][i] = 0.f; va[u][i] = 0.f; la[u][i] = 0.f; ra[u][i] = 0.f; ha[u][i] = 0.f; g[u][i] = 0.f; if (TOPK) hat_was[u][i] = 0.f; if (TOPK && PULL) { lx[u][i] = 0.f; rx[u][i] = 0.f; } }
      nv[u] = !live[u] ? 0u : cd.len - e[u] < 4u ? cd.len - e[u] : 4u;
      if (live[u]) {
        const float4 x4 = ld4t<STREAM>(T.x + base + e[u]);
        float4 v4 = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!A.plain_sgd) v4 = ld4t<STREAM>(T.vel + base + e[u]);   // uniform
        xa[u][0] = x4.x; xa[u][1] = x4.y; xa[u][2] = x4.z; xa[u][3] = x4.w;
        va[u][0] = v4.x; va[u][1] = v4.y; va[u][2] = v4.z; va[u][3] = v4.w;
        if (from_l) {        // the put of my left neighbour, carried out by its receiver
          const float4 t = ld4t<STREAM>(snap_in + (size_t)lw * T.Npad + cd.off + e[u]);
          la[u][0] = t.x; la[u][1] = t.y; la[u][2] = t.z; la[u][3] = t.w;
          st4t<STREAM>(T.mbox_l + base + e[u], t);
        } else if (vl) { const float4 t = ld4t<STREAM>(T.mbox_l + base + e[u]); la[u][0] = t.x; la[u][1] = t.y; la[u][2] = t.z; la[u][3] = t.w; }
        if (from_r) {
          const float4 t = ld4t<STREAM>(snap_in + (size_t)rw * T.Npad + cd.off + e[u]);
          ra[u][0] = t.x; ra[u][1] = t.y; ra[u][2] = t.z; ra[u][3] = t.w;
          st4t<STREAM>(T.mbox_r + base + e[u], t);
        } else if (vr) { const float4 t = ld4t<STREAM>(T.mbox_r + base + e[u]); ra[u][0] = t.x; ra[u][1] = t.y; ra[u][2] = t.z; ra[u][3] = t.w; }
        if (TOPK && PULL) {
          const float4 tl = ld4t<STREAM>(snap_in + (size_t)lw * T.Npad + cd.off + e[u]);
          const float4 tr = ld4t<STREAM>(snap_in + (size_t)rw * T.Npad + cd.off + e[u]);
          lx[u][0] = tl.x; lx[u][1] = tl.y; lx[u][2] = tl.z; lx[u][3] = tl.w;
          rx[u][0] = tr.x; rx[u][1] = tr.y; rx[u][2] = tr.z; rx[u][3] = tr.w;
        }
        if (TOPK && my_event == 2) {
          const float4 t = ld4t<STREAM>(T.xhat + base + e[u]);
          hat_was[u][0] = t.x; hat_was[u][1] = t.y; hat_was[u][2] = t.z; hat_was[u][3] = t.w;
        }
        if (sent_whole) {
          // the whole tensor was sent in this iteration: xhat becomes the x just read
          ha[u][0] = xa[u][0]; ha[u][1] = xa[u][1]; ha[u][2] = xa[u][2]; ha[u][3] = xa[u][3];
          st4t<STREAM>(T.xhat + base + e[u], x4);
        } else if (TOPK && my_event == 2) {
          ha[u][0] = hat_was[u][0]; ha[u][1] = hat_was[u][1]; ha[u][2] = hat_was[u][2]; ha[u][3] = hat_was[u][3];
        } else if (NORM == 1 || NORM == 3) {
          const float4 t = ld4t<STREAM>(T.xhat + base + e[u]); ha[u][0] = t.x; ha[u][1] = t.y; ha[u][2] = t.z; ha[u][3] = t.w;
        }
        if (GRADBUF) { const float4 t = ld4t<STREAM>(A.grad + base + e[u]); g[u][0] = t.x; g[u][1] = t.y; g[u][2] = t.z; g[u][3] = t.w; }
      }
    }
    if (TOPK) {
      // my own message: it is told from x and xhat, written, and applied to xhat
      if (my_event == 2) {                   // uniform
#pragma unroll
        for (int u = 0; u < SPW; ++u) {
          constexpr bool CHECK = STREAM && NORM;         // (other rings have no key codes)
          uint32_t win = winners4(xa[u], hat_was[u], A.topk_key, thr[0], cut[0], cd.j0 + e[u], nv[u]);
          const uint32_t count = thr[0] == kNoThreshold ? 0u : place[u].count;
          if (!A.applied) win = put_message<CHECK>(T, r, moff, place[u].first, count, win, xa[u], cd.j0 + e[u]);
          else if (CHECK) win = counted_winners(win, count);
          if (!sent_whole) {
            take_winners(win, xa[u], ha[u]);
            if (any_of_line_part(win) && live[u]) st4t<STREAM>(T.xhat + base + e[u], make_float4(ha[u][0], ha[u][1], ha[u][2], ha[u][3]));
          }
        }
      }
      // the neighbours': told from the copies of their x and from my mailboxes, which hold their xhat
      if (PULL && some_l) receive(thr[1], cut[1], lx, T.mbox_l, la);
      if (PULL && some_r) receive(thr[2], cut[2], rx, T.mbox_r, ra);
    }
    if (HISTA) {
      for (uint32_t b = threadIdx.x; b < BINS; b += kThreads) hA[b] = 0;
      __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < SPW; ++u) {
      if (live[u]) {
        if (!GRADBUF) {
          const float sg = (float)(T.layers[cd.layer].sig_base * step_decay(T, A));
          draw_gradient<DIST>(A, cd.j0 + e[u], cd.layer, k_iter, r, sg, has_spike(A, k_iter, r), g[u]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if ((uint32_t)i < nv[u]) {   // lanes past the tensor's end are padding: left as they are
            // momentum 0 is the paper's plain SGD: the velocity is the gradient, and the
            // velocity arena is neither read nor written
            const float vn = A.plain_sgd ? g[u][i] : __builtin_fmaf(A.mu, va[u][i], g[u][i]);
            const float a = (vl ? (la[u][i] - xa[u][i]) : 0.0f) + (vr ? (ra[u][i] - xa[u][i]) : 0.0f);
            const float cns = __builtin_fmaf(a, third, xa[u][i]);
            xa[u][i] = __builtin_fmaf(-A.lr, vn, cns);
            va[u][i] = vn;
          }
        }
        st4t<STREAM>(T.x + base + e[u], make_float4(xa[u][0], xa[u][1], xa[u][2], xa[u][3]));
        if (PULL) st4t<STREAM>(snap_out + base + e[u], make_float4(xa[u][0], xa[u][1], xa[u][2], xa[u][3]));
        if (!A.plain_sgd) st4t<STREAM>(T.vel + base + e[u], make_float4(va[u][0], va[u][1], va[u][2], va[u][3]));
        if (NORM == 1) drift_acc(acc[u], xa[u], ha[u], nv[u]);
        if (NORM >= 2) square_acc(acc[u], xa[u], nv[u]);
        if (NORM == 3) square_acc(acc_hat[u], ha[u], nv[u]);
        if (TOPK && NORM && !FINE) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (HISTA && (uint32_t)i < nv[u]) atomicAdd(&hA[rank_key(xa[u][i], ha[u][i], A.topk_key) >> kPlainBits], 1u);
        }
        if (TOPK && NORM && FINE) {
          const Bins bins = first_bins(xa[u], ha[u], A.topk_key, anchor & kAnchorBits);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (HISTA && (uint32_t)i < nv[u]) atomicAdd(&hA[bins.bin[i]], 1u);
          if (STREAM && T.codes && !(anchor & kUncoded)) store_codes(T, base, (cd.len + 3) / 4 * 16, e[u] * 4, bins.codes);
        }
      }
    }
  }
  if (HISTA && sub0 * kSweep < cd.len + cd.lead) {     // uniform
    __syncthreads();
    const HistAt counts = first_hist(T, cd.layer, FINE ? blockIdx.x & 7u : 0u);
    uint32_t* gh = T.hist + (size_t)(counts.first + r * counts.step) * kHistBins;
    for (uint32_t b = threadIdx.x; b < BINS; b += kThreads) {
      const uint32_t v = hA[b];
      if (v) atomicAdd(&gh[b], v);
    }
  }
  if (NORM) {
    const size_t slot = ((size_t)r * T.C + c) * T.SW + sub0;
    double total[SPW];
    block_sums<SPW>(acc, ws, total);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int u = 0; u < SPW; ++u) T.partials_out[slot + u] = total[u];
    }
    if (NORM == 3) {
      block_sums<SPW>(acc_hat, ws, total);
      if (threadIdx.x == 0) {
#pragma unroll
        for (int u = 0; u < SPW; ++u) T.partials_hat_out[slot + u] = total[u];
      }
    }
  }
}

// Mean over workers, one thread per float4 of a slice (last line of Algorithm B).
__global__ __launch_bounds__(kThreads) void k_average(Tables T, float* out) {
  const size_t q = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (q * 4 >= T.Npad) return;
  double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
  for (uint32_t r = 0; r < T.P; ++r) {
    const float4 v = ld4(T.x + (size_t)r * T.Npad + q * 4);
    a0 += (double)v.x; a1 += (double)v.y; a2 += (double)v.z; a3 += (double)v.w;
  }
  const double p = (double)T.P;
  st4s(out + q * 4, make_float4((float)(a0 / p), (float)(a1 / p), (float)(a2 / p), (float)(a3 / p)));
}

hipError_t launch_norm(const Tables& t, bool norm_diff, hipStream_t s) {
  const dim3 grid(t.C * t.SW, t.P), block(kThreads);
  if (norm_diff) k_norm<true><<<grid, block, 0, s>>>(t);
  else k_norm<false><<<grid, block, 0, s>>>(t);
  return hipGetLastError();
}

template <int NORM, bool TOPK, bool HISTA, int SPW>
static void launch_update_w(const Tables& t, const StepArgs& a, uint32_t dist, uint32_t grad_mode,
                            hipStream_t s) {
  const dim3 grid(t.C * (t.SW / SPW), t.P), block(kThreads);
  if (a.pull) {              // the host sets pull only for cache-resident rings
    if (grad_mode == 1) k_update<0, true, NORM, TOPK, HISTA, SPW, false, true><<<grid, block, 0, s>>>(t, a);
    else if (dist == 0) k_update<0, false, NORM, TOPK, HISTA, SPW, false, true><<<grid, block, 0, s>>>(t, a);
    else k_update<1, false, NORM, TOPK, HISTA, SPW, false, true><<<grid, block, 0, s>>>(t, a);
    return;
  }
  if (a.cached && HISTA && !t.anchor) {
    constexpr bool F = !HISTA;
    if (grad_mode == 1) k_update<0, true, NORM, TOPK, HISTA, SPW, false, false, F><<<grid, block, 0, s>>>(t, a);
    else if (dist == 0) k_update<0, false, NORM, TOPK, HISTA, SPW, false, false, F><<<grid, block, 0, s>>>(t, a);
    else k_update<1, false, NORM, TOPK, HISTA, SPW, false, false, F><<<grid, block, 0, s>>>(t, a);
    return;
  }
  if (a.cached) {
    if (grad_mode == 1) k_update<0, true, NORM, TOPK, HISTA, SPW, false><<<grid, block, 0, s>>>(t, a);
    else if (dist == 0) k_update<0, false, NORM, TOPK, HISTA, SPW, false><<<grid, block, 0, s>>>(t, a);
    else k_update<1, false, NORM, TOPK, HISTA, SPW, false><<<grid, block, 0, s>>>(t, a);
    return;
  }
  if (grad_mode == 1) k_update<0, true, NORM, TOPK, HISTA, SPW, true><<<grid, block, 0, s>>>(t, a);
  else if (dist == 0) k_update<0, false, NORM, TOPK, HISTA, SPW, true><<<grid, block, 0, s>>>(t, a);
  else k_update<1, false, NORM, TOPK, HISTA, SPW, true><<<grid, block, 0, s>>>(t, a);
}

template <int NORM, bool TOPK, bool HISTA>
static void launch_update_v(const Tables& t, const StepArgs& a, uint32_t dist, uint32_t grad_mode,
                            hipStream_t s) {
  // two sweeps per workgroup where the pass carries the Top-K extras and a chunk has them
  // (measured: four are slower again, LDS and registers then hold occupancy down)
  if (TOPK && HISTA && t.SW % 2 == 0)
    launch_update_w<NORM, TOPK, HISTA, (TOPK && HISTA) ? 2 : 1>(t, a, dist, grad_mode, s);
  else
    launch_update_w<NORM, TOPK, HISTA, 1>(t, a, dist, grad_mode, s);
}

hipError_t launch_update(const Tables& t, const StepArgs& a, uint32_t dist, uint32_t grad_mode,
                         int norm, hipStream_t s) {
  if (a.topk_on) {
    if (norm == 1 && a.hist_fused) launch_update_v<1, true, true>(t, a, dist, grad_mode, s);
    else if (norm == 3 && a.hist_fused) launch_update_v<3, true, true>(t, a, dist, grad_mode, s);
    else if (norm == 0) launch_update_v<0, true, false>(t, a, dist, grad_mode, s);
    else return hipErrorInvalidValue;
  } else {
    if (norm == 0) launch_update_v<0, false, false>(t, a, dist, grad_mode, s);
    else if (norm == 1) launch_update_v<1, false, false>(t, a, dist, grad_mode, s);
    else if (norm == 2) launch_update_v<2, false, false>(t, a, dist, grad_mode, s);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_average(const Tables& t, float* out, hipStream_t s) {
  const uint64_t quads = t.Npad / 4;
  const uint32_t grid = (uint32_t)((quads + kThreads - 1) / kThreads);
  k_average<<<dim3(grid), dim3(kThreads), 0, s>>>(t, out);
  return hipGetLastError();
}

}  // namespace evg
