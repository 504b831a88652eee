// The trigger test of one (worker, tensor) as device functions, shared by the kernels that
// run it: k_trigger / k_topk_decide (one wavefront per tensor, ahead of the update pass) and the
// update pass of rings that take a single launch per iteration (every workgroup repeats the
// tests it depends on; the tensor's first workgroup records the outcome).
// There the wavefronts sum several tensors at a time (kernels_parts.hip); test and booking are the same.
//
// What a test READS (sweep sums, delta, last_event, xhat_sq) and what an event WRITES of the
// same (delta, last_event, xhat_sq; the sweep sums are written by the update pass) go through
// two sets of pointers, T.name and T.name_out.  Normally both name the same array.  The
// single-launch step gives them different arrays, because there other workgroups of the same
// launch still have to read the values from before the event.
#pragma once
#include "evg_device.h"
#include "quad_device.h"

namespace evg {

// The sums of one sweep: one, or where windows are shorter (kernels_ring.hip) one for each group of 256 elements, or for two.  A sweep's are added up first,
// as the passes that have a whole sweep in a workgroup add theirs (block_sum): a tensor's sum is the same bits also once its sweeps' have been made
// one (evg_state_export), and, groups in their order, whichever pass has left them.
template <int F> struct SweepSums {
  double v[F];
  __device__ __forceinline__ double added() const {
    if constexpr (F == 1) return v[0];
    else if constexpr (F == 2) return v[0] + v[1];
    else return ((v[0] + v[1]) + v[2]) + v[3];
  }
};
// part: the same in all lanes, a multiple of F; past its np sums zeros
template <int F>
__device__ __forceinline__ SweepSums<F> load_sweep(const double* part, uint32_t np, uint32_t sweep) {
  static_assert(F == 1 || F == 2 || F == kGroupSums, "a sweep's, halves' or groups'");
  SweepSums<F> s;
  if constexpr (F == 1) {
    s.v[0] = load_f64(part, np * 8, sweep * 8);
  } else {
#pragma unroll
    for (int h = 0; h < F / 2; ++h) {
      const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(window(part, np * 8), (int)(sweep * (F * 8) + h * 16), 0, 0);
      s.v[2 * h] = __longlong_as_double((long long)(((uint64_t)t[1] << 32) | t[0]));
      s.v[2 * h + 1] = __longlong_as_double((long long)(((uint64_t)t[3] << 32) | t[2]));
    }
  }
  return s;
}

// A lane's sweeps in order, of np sums, MANY of which are in flight where there are more than eight: waiting for each of the 36 sweeps that a tensor
// of 2.4 M elements leaves a lane made the kernel 13 us, eight at a time 5; of the 144 sums of its groups k_trigger for 16 ResNet-18 workers 12.2 us with
// eight, 7.4 with 32 (a step with spikes 822 -> 817, with given gradients 1005 -> 1001).  k_topk_decide takes 16, as its registers cost workgroups
// beside it: 9 -> 8 and 22 -> 21 us for 8 ResNet-50 and 64 ResNet-18 workers.
template <int N, int F>
__device__ __forceinline__ void add_in_order(const double* part, uint32_t np, uint32_t first, double* acc) {
  SweepSums<F> s[N / F];
#pragma unroll
  for (uint32_t u = 0; u < N / F; ++u) s[u] = load_sweep<F>(part, np, first + 64 * u + lane_id());
#pragma unroll
  for (uint32_t u = 0; u < N / F; ++u) *acc += s[u].added();
}
template <int MANY, int F>
__device__ __forceinline__ double ordered_lane_sum(const double* part, uint32_t np) {
  double acc = 0.0;
  uint32_t i = 0;
  const uint32_t sweeps = np / F;
  if constexpr (MANY > 8)
    for (; i + 64 * (8 / F) < sweeps; i += 64 * (MANY / F)) add_in_order<MANY, F>(part, np, i, &acc);
  for (; i < sweeps; i += 64 * (8 / F)) add_in_order<8, F>(part, np, i, &acc);
  return acc;
}

// Sums of the tensor's sweep partials in a fixed order, by one whole wavefront; valid in every lane.  seg: the same in all lanes.  F: T.fine.
// *hat_sums: the squared norm of xhat comes from the arena sums (norm-difference trigger with
// Top-K, or before the tensor's first event) rather than from the scalar kept at its last event.
template <int MANY, int F>
__device__ __forceinline__ void segment_sums(const Tables& T, const StepArgs& A, uint32_t seg, double* acc_out,
                                             double* acc_hat_out, bool* hat_sums_out) {
  const uint32_t r = seg / T.L, l = seg % T.L;
  const LayerDesc ld = T.layers[l];
  const uint32_t sums = T.SW * F, np = ld.nchunks * sums;
  const double* part = T.partials + ((size_t)r * T.C + ld.chunk0) * sums;
  double acc_hat = 0.0;
  const double acc = wave_sum(ordered_lane_sum<MANY, F>(part, np));
  const bool hat_sums = A.norm_src == 2 || (A.norm_src == 1 && T.last_event[seg] < 0);
  if (hat_sums) {
    const double* ph = T.partials_hat + ((size_t)r * T.C + ld.chunk0) * sums;
    acc_hat = wave_sum(ordered_lane_sum<MANY, F>(ph, np));
  }
  *acc_out = acc;
  *acc_hat_out = acc_hat;
  *hat_sums_out = hat_sums;
}

// The tested quantity, from the tensor's sums.
__device__ __forceinline__ float tested_norm(const StepArgs& A, double acc, double acc_hat) {
  return A.norm_src == 0 ? (float)sqrt(acc) : __builtin_fabsf((float)sqrt(acc) - (float)sqrt(acc_hat));
}

// The event condition || xhat - x || >= delta (Section 4).  dl: threshold, khat: iteration of the last event.  Returns
// 0 silent, 1 the whole tensor is sent, 2 a Top-K message is sent.
__device__ __forceinline__ uint8_t event_code(const StepArgs& A, float d, float dl, int32_t khat, uint32_t k) {
  const bool fire = (A.force_first && k == 0) || (d >= dl);   // NaN never fires
  // a tensor's first message has nothing to patch on the receiving side: send it whole
  return !fire ? 0 : (!A.topk_on || khat < 0) ? 1 : 2;
}

// Books the outcome of a test, by ONE lane: norm, threshold before, near-tie flag, counters, and at an event the adaptive
// threshold (Eq. 3), the event's iteration and the event counters.
// MARK: at an event also mark the two neighbours' mailbox slots as filled.
template <bool MARK>
__device__ __forceinline__ void book_test(const Tables& T, const StepArgs& A, uint32_t seg, float d, float dl, int32_t khat,
                                          uint8_t code, double acc, uint32_t k) {
  const bool fire = code != 0;
  T.last_norm[seg] = d;
  T.delta_before[seg] = dl;
  // (additions that return nothing: nobody waits for them)
  if (!(__builtin_fabsf(d) <= 3.402823466e+38f)) atomicAdd(&T.nonfinite_cnt[seg], 1u);   // NaN or inf
  const bool near = __builtin_fabsf(d - dl) < 1e-6f * dl;
  T.near_tie[seg] = near ? 1 : 0;
  if (near) atomicAdd(&T.near_cnt[seg], 1u);
  float dl_new = dl;
  if (fire) {
    if (A.thr_mode == 1) {
      const float slope = d / (float)((int32_t)k - khat);
      if (T.hist_len <= 1) {
        dl_new = A.horizon * slope;
      } else {
        // mean of the slopes between the last hist_len consecutive events (Section 7)
        float* hs = T.slope_hist + (size_t)seg * T.hist_len;
        uint32_t cnt = T.slope_cnt[seg];
        if (cnt == T.hist_len) {
          for (uint32_t i = 1; i < cnt; ++i) hs[i - 1] = hs[i];
          cnt -= 1;
        }
        hs[cnt++] = slope;
        T.slope_cnt[seg] = cnt;
        float sum = 0.0f;
        for (uint32_t i = 0; i < cnt; ++i) sum += hs[i];
        dl_new = A.horizon * (sum / (float)cnt);
      }
    }
    atomicAdd(code == 1 ? &T.ev_full[seg] : &T.ev_topk[seg], 1u);
    if (MARK && !A.delay) {             // with delayed delivery: set when the put lands (k_deliver)
      const uint32_t r = seg / T.L, l = seg % T.L;
      const uint32_t left = (r + T.P - 1) % T.P, right = (r + 1) % T.P;
      T.valid_r[left * T.L + l] = 1;    // I am my left neighbour's right-hand source
      T.valid_l[right * T.L + l] = 1;
    }
  }
  T.delta_out[seg] = dl_new;
  T.last_event_out[seg] = fire ? (int32_t)k : khat;
  // the whole tensor is sent: xhat becomes x, and so does its squared norm
  if (A.norm_src == 1) T.xhat_sq_out[seg] = fire ? acc : T.xhat_sq[seg];
  T.fired[seg] = code;
}

// Test and booking of a tensor whose sums are at hand, by ONE lane; k: the iteration.
__device__ __forceinline__ uint8_t segment_test(const Tables& T, const StepArgs& A, uint32_t seg, double acc, double acc_hat,
                                                bool hat_sums, uint32_t k) {
  if (A.norm_src != 0 && !hat_sums) acc_hat = T.xhat_sq[seg];
  const float d = tested_norm(A, acc, acc_hat), dl = T.delta[seg];
  const int32_t khat = T.last_event[seg];
  const uint8_t code = event_code(A, d, dl, khat, k);
  book_test<true>(T, A, seg, d, dl, khat, code, acc, k);
  return code;
}

// The step's bookkeeping, once per step.  A replayable step takes its iteration from k_next, which all workgroups of the
// launch that runs the tests read; it is moved on by a later launch, the update pass (end_replayable), while the
// iteration and decay^k are left here for that pass.  (A kernel of its own ahead of the tests did this before:
// a replayed iteration of an 8-worker ResNet-20 ring took 29.2 us, now 25.3.)
__device__ __forceinline__ uint32_t tested_k(const Tables& T, const StepArgs& A) {
  return A.from_device ? T.it->k_next : A.k;
}
__device__ __forceinline__ void close_step(const Tables& T, const StepArgs& A) {
  const uint32_t k = tested_k(T, A);
  if (A.from_device) {
    T.it->k = k;
    if (k >= T.decay_len) T.it->overflow = 1;
    T.it->decay_pow = T.decay_tab[k < T.decay_len ? k : T.decay_len - 1];
  } else {
    T.it->k_next = k + 1;
  }
  atomicAdd(reinterpret_cast<unsigned long long*>(&T.it->iters), 1ull);     // (returns nothing: nobody waits for it)
}
// By the first workgroup of the update pass.
__device__ __forceinline__ void end_replayable(const Tables& T, const StepArgs& A) {
  if (A.from_device && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) T.it->k_next = T.it->k + 1;
}

}  // namespace evg
