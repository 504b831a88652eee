// Trigger test and whole-tensor sends.
//   k_trigger  one wavefront per (worker, tensor): finishes the drift norm from the
//              per-chunk partial sums in a fixed order, applies the event condition
//              || xhat - x || >= delta (Section 4), recomputes the adaptive threshold
//              at events (Eq. 3), marks the neighbours' mailbox slots as filled.
//   k_copy     x -> xhat for every chunk of a tensor that fired, where the update pass walks the ring
//              in parts: for the workers at their ends.
// The kernels that act on fired tensors have one workgroup per chunk of the ring, which leaves
// at once if its tensor stayed silent.  (Compact lists of the fired chunks, made by two more
// kernels, cost a dependent launch each, 5 + 5 us, and saved nothing in the kernels that read them.)
#include "trigger_device.h"

namespace evg {

// The trigger test of one (worker, tensor), by one whole wavefront.
template <int MANY>
__device__ __forceinline__ void trigger_segment(const Tables& T, const StepArgs& A, uint32_t seg) {
  double acc, acc_hat;
  bool hat_sums;
  if (T.fine == 1) segment_sums<MANY, 1>(T, A, seg, &acc, &acc_hat, &hat_sums);       // uniform
  else if (T.fine == 2) segment_sums<MANY, 2>(T, A, seg, &acc, &acc_hat, &hat_sums);
  else segment_sums<MANY, kGroupSums>(T, A, seg, &acc, &acc_hat, &hat_sums);
  if (lane_id() == 0) (void)segment_test(T, A, seg, acc, acc_hat, hat_sums, tested_k(T, A));
}

// MANY: sums of a lane in flight where a tensor has more than eight a lane, which takes registers: a ring without such tensors goes by MANY = 8.  14 workers of
// 5948 tensors of 700 elements 41 -> 33 us, 59 of 76 568 of 30 elements 2.29 -> 1.61 ms.
template <int MANY>
__global__ __launch_bounds__(kThreads) void k_trigger(Tables T, StepArgs A) {
  const uint32_t seg = blockIdx.x * (kThreads / 64) + (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_id());
  if (seg >= T.S) return;           // whole wavefront leaves; no workgroup barrier below
  trigger_segment<MANY>(T, A, seg);
  if (seg == 0 && lane_id() == 0) close_step(T, A);
}

template <int SWEEPS>
__global__ __launch_bounds__(kThreads) void k_copy(Tables T, StepArgs A) {
  const uint32_t c = blockIdx.x, r = blockIdx.y;
  const ChunkDesc cd = T.chunks[c];
  if (T.fired[r * T.L + cd.layer] != 1 || !is_led(T, A, r)) return;
  copy_chunk<SWEEPS, true, true>(T, r, cd);
}

hipError_t launch_trigger(const Tables& t, const StepArgs& a, uint32_t most_sums, hipStream_t s) {
  const uint32_t grid = (t.S + 3) / 4;
  if (most_sums > 64 * 8) k_trigger<32><<<dim3(grid), dim3(kThreads), 0, s>>>(t, a);
  else k_trigger<8><<<dim3(grid), dim3(kThreads), 0, s>>>(t, a);
  return hipGetLastError();
}

// Delayed delivery: after the updates, every tensor that sent in this iteration (whole
// or Top-K) lands in its neighbours' mailboxes.  What a neighbour must hold afterwards is
// exactly the sender's xhat (entries that were not sent are equal already), so each chunk
// of its xhat is copied, and the receivers' slots are marked as filled.
template <int SWEEPS>
__global__ __launch_bounds__(kThreads) void k_deliver(Tables T) {
  const uint32_t c = blockIdx.x, r = blockIdx.y;
  const ChunkDesc cd = T.chunks[c];
  if (T.fired[r * T.L + cd.layer] == 0) return;
  const uint32_t left = (r + T.P - 1) % T.P, right = (r + 1) % T.P;
  const float* src = T.xhat + (size_t)r * T.Npad + cd.off;
  float* d1 = T.mbox_r + (size_t)left * T.Npad + cd.off;
  float* d2 = T.mbox_l + (size_t)right * T.Npad + cd.off;
#pragma unroll
  for (int it = 0; it < SWEEPS; ++it) {
    const uint32_t e = it * kSweep + threadIdx.x * kLaneElems - cd.lead;
    if (e < cd.len) {
      const float4 v = ld4s(src + e);
      st4s(d1 + e, v);
      st4s(d2 + e, v);
    }
  }
  if (threadIdx.x == 0 && cd.j0 == 0) {     // the tensor's first chunk speaks for the tensor
    T.valid_r[left * T.L + cd.layer] = 1;
    T.valid_l[right * T.L + cd.layer] = 1;
  }
}

hipError_t launch_copy(const Tables& t, const StepArgs& a, uint32_t chunk_elems, hipStream_t s) {
  const dim3 g(t.C, t.P), b(kThreads);
  switch (chunk_elems / kSweep) {
    case 1: k_copy<1><<<g, b, 0, s>>>(t, a); break;
    case 2: k_copy<2><<<g, b, 0, s>>>(t, a); break;
    case 4: k_copy<4><<<g, b, 0, s>>>(t, a); break;
    case 8: k_copy<8><<<g, b, 0, s>>>(t, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_deliver(const Tables& t, uint32_t chunk_elems, hipStream_t s) {
  const dim3 g(t.C, t.P), b(kThreads);
  switch (chunk_elems / kSweep) {
    case 1: k_deliver<1><<<g, b, 0, s>>>(t); break;
    case 2: k_deliver<2><<<g, b, 0, s>>>(t); break;
    case 4: k_deliver<4><<<g, b, 0, s>>>(t); break;
    case 8: k_deliver<8><<<g, b, 0, s>>>(t); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace evg
