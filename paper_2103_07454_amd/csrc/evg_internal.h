// Internal types shared by the host side of libevg and its gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace evg {

constexpr int kThreads = 256;          // 4 wavefronts of 64 lanes
constexpr int kLaneElems = 4;          // one float4 per lane and sweep
constexpr int kSweep = kThreads * kLaneElems;   // elements one workgroup covers per sweep
constexpr uint32_t kLineElems = 32;    // floats of a 128-byte cache line
constexpr int kHistBins = 2048;        // histogram of a selection pass: the second takes 11 bits of a key, the last what is left, 6, 9 or 10
constexpr int kFirstBins = 1280;       // the first (see first_bins)
constexpr uint32_t kCoarseBits = 21, kFineBits = 17;                  // bits of a key below its coarse and fine bins
constexpr uint32_t kPlainBits = 20;                                   // below the bins of rings without anchors
constexpr uint32_t kPerCoarse = 1u << (kCoarseBits - kFineBits);      // fine bins of a coarse one
constexpr uint32_t kFineBins = 128;
constexpr uint32_t kHistCopies = 8;    // of the first histogram of a tensor that is most of a ring (Tables::long_layer)
constexpr uint32_t kHistCopiesFrom = 131072;      // elements of such a tensor at least
constexpr uint32_t kNoLayer = 0xFFFFFFFFu;
constexpr uint32_t kFirstCode = 64, kCodeBins = 128;                  // key codes that are counted where there are no such histograms,
constexpr uint32_t kCodeStride = 256;                                 // in eight copies, each of those codes and of all above
constexpr uint32_t kStageCap = 2048;   // staged keys of a chunk at most
// Threshold key that no key reaches (they have 31 bits).  A selection ends with it where it sees that it would not find exactly K
// winners: the histogram and the key codes that the last update pass left do not fit x and xhat, which the caller has written since.
// Nothing is sent then.  Where keys are counted by their codes, the update passes compare each 256 elements' winners with the count.
constexpr uint32_t kNoThreshold = 0xFFFFFFFFu;
constexpr uint32_t kNoAnchor = 0xFFFFFFFFu;
// Anchors are multiples of 16.  Bit 0 of one (and of kNoAnchor): the update pass leaves no key codes, as the tensor has been silent
// for more than kCodedFor iterations (streaming rings): its next selection reads x and xhat.
constexpr uint32_t kUncoded = 1u, kAnchorBits = ~15u;
constexpr uint32_t kCodedFor = 4;        // (some five bytes written cost what seven that need not be read save)
constexpr uint32_t kNoEntry = 0xFFFFFFFFu;       // index in a message's place that nothing was sent for

// A chunk is a run of one tensor's elements that one workgroup handles; it never
// straddles tensors, starts at a multiple of 4 elements and is at most chunk_elems long.
// In rings that stream from memory a tensor's first chunk leaves out its first `lead` positions, so that the
// sweeps of all its chunks begin on cache lines (tensors begin on multiples of 16 bytes only).
struct ChunkDesc {
  uint32_t off;    // start inside a worker's arena slice (floats, multiple of 4)
  uint32_t len;    // elements (multiple of 4 except a tensor's last chunk)
  uint32_t layer;  // tensor index
  uint32_t j0;     // start inside the tensor (multiple of 4)
  uint32_t lead;   // multiple of 4: the chunk's elements are positions lead .. lead + len - 1 of its workgroup's sweeps
};

struct LayerDesc {
  uint32_t off;      // start inside a worker's slice
  uint32_t numel;
  uint32_t chunk0;   // first chunk
  uint32_t nchunks;
  uint32_t K;        // Top-K message length (0 when Top-K is off)
  uint32_t msg_off;  // start of this tensor's message slot inside a worker's staging slice
  double sig_base;   // sigma0 [/ sqrt(fan_in)]
};

// A window of kernels_ring.hip or kernels_parts.hip: up to 1024 elements of one tensor.
struct WindowDesc {
  uint32_t off, len;   // start inside a worker's slice (multiple of 4), elements
  uint32_t layer, j0;  // tensor, start inside it
  uint32_t slot;       // where the window's sum goes, or the first of its groups', among a worker's partials
  uint32_t sum0, sums; // the tensor's partials
  uint32_t books;      // the tensor's first window
  double sig_base;     // sigma0 [/ sqrt(fan_in)]
  uint32_t numel, K, msg_off, pad;     // of the tensor; its Top-K message (see LayerDesc)
};
constexpr uint32_t kGroupSums = 4;     // sums of a sweep where each group of 256 elements has one
constexpr uint32_t kPartMost = 8;      // workers of a part of the ring there
constexpr uint32_t kRingMost = 64;     // workers of a ring whose windows are one workgroup's: 64 KB of LDS
struct PartClock { uint32_t k, steps; };       // the next iteration, and the steps completed
struct PartTables {
  const WindowDesc* windows; uint32_t count;
  uint32_t groups, quads;  // kernels_ring.hip: groups of 256 elements in a window, float4s of a thread; 0: the ring goes by kernels_parts.hip
  PartClock* clocks;       // [count * parts]
  // What the trigger tests read and an event writes exists twice: step n (from 0) reads set n & 1 and writes the other.
  struct Set { double* partials; double* xhat_sq; float* delta; int32_t* last_event; } set[2];
};

// The iteration as the device knows it.  evg_step passes the iteration by value; a step
// that must be replayable from a captured graph (evg_step_next) reads it from here instead.
struct IterState {
  uint32_t k;          // iteration of the step in flight (set with the trigger tests of replayable steps)
  uint32_t k_next;     // the iteration after the last completed step
  uint64_t iters;      // steps completed
  double decay_pow;    // decay^k for the step in flight (replayable steps)
  uint32_t overflow;   // a replayable step ran past the decay table
  uint32_t pad;
};

// Device pointers and sizes, passed to kernels by value.
struct Tables {
  const ChunkDesc* chunks;
  const LayerDesc* layers;
  float* x; float* xhat; float* mbox_l; float* mbox_r; float* vel;
  float* xsnap;            // [2][P*Npad] or null: copies of x that the update pass of one iteration leaves
                           // for the next one, two in turn (cache-resident rings with ordinary
                           // delivery: the receivers then fetch what a neighbour sends, no copy kernel)
  double* partials;        // [P*C*SW*fine] per 1024-element sweep of a chunk, or per part of it (fine): sum of squared drift, or
                           // of squared x when the trigger compares norms
  double* partials_hat;    // [P*C*SW*fine] sum of squared xhat (norm-difference trigger only)
  double* xhat_sq;         // [S] squared norm of what was last sent, kept as a scalar when whole
                           // tensors are sent (norm-difference trigger only)
  float* delta; float* last_norm; float* delta_before;
  int32_t* last_event;
  // Where a step WRITES the sweep sums, and an event the threshold, its iteration and the squared
  // norm of what was sent.  The same arrays as partials, partials_hat, delta, last_event, xhat_sq
  // (which a step reads), except in rings whose steps can be a single launch, whose workgroups must all still see the
  // values from before the step: there the two sets alternate from step to step.
  double* partials_out; double* partials_hat_out; double* xhat_sq_out;
  float* delta_out; int32_t* last_event_out;
  uint8_t* valid_l; uint8_t* valid_r; uint8_t* fired; uint8_t* near_tie;
  uint32_t* ev_full; uint32_t* ev_topk; uint32_t* near_cnt; uint32_t* nonfinite_cnt;
  float* slope_hist; uint32_t* slope_cnt;   // [S*hist_len], [S]
  uint32_t* not_staged;    // [1] chunks so far whose possible winners did not fit their staging slot
  uint32_t* hist;          // [S*kHistBins], and behind it the further copies of the long tensors' (first_hist)
  // Tensors whose first histogram, which an update pass leaves, is the sum of kHistCopies: all workgroups of a pass would add to one
  // (up to two tensors, the first, or both, may be kNoLayer).
  uint32_t long_layer[2];
  uint32_t* sel_prefix; uint32_t* sel_krem;   // [S] in the end the threshold key (or kNoThreshold), and how many of the keys equal to it win
  uint32_t* sel_cut;       // [S] the last element of the tensor that wins with a key equal to the threshold
  uint32_t* stage_n;       // [P*C] staged keys of a chunk: those in the threshold bin; 0xFFFFFFFF: more than the
                           // chunk's slot holds, nothing staged (they are then read from the arenas)
  uint32_t* stage_key;     // [P*stage_stride] their bits below the bin (at most 21), and from bit 21 on the group of the chunk they belong to
  uint64_t stage_stride;   // staging entries per worker
  uint8_t* codes;          // [P*Npad] or null: rank keys of x and xhat as the last update pass left them, in a byte: bits 30..17
                           // counted from the tensor's anchor; 0 and 255 also stand for all that is further off (see kUncoded)
  uint32_t* anchor;        // [S] or null: where the fine bins of the first pass's histogram begin; kNoAnchor: there are none
  uint32_t* sel_left;      // [S] bits of a key below the first pass's bin, and from bit 8 on the code of that bin's keys (0: none)
  uint32_t* group;         // [P*C*SW*4] per 256 elements: keys above the threshold bin; in the end, over the chunk's
                           // earlier groups, keys above (low half) and equal to (high half) the threshold
  uint2* chunk_cnt;        // [P*C] keys above and equal to the threshold per chunk
  uint2* chunk_before;     // [P*C] the same, summed over the tensor's earlier chunks
  uint32_t* msg_idx; float* msg_val;          // [P*Ktot]
  unsigned long long* idx_hash;               // [S] fingerprints of the last step's Top-K messages (sums of
  unsigned long long* msg_hash;               // mixed indices / mixed (value, index) pairs), filled on request
  IterState* it;
  const double* decay_tab;   // decay^k for k < decay_len (replayable steps only)
  uint32_t decay_len;
  uint32_t P, L, C, S;
  uint32_t SW;             // 1024-element sweeps per chunk
  uint32_t fine;           // sums of a sweep: 1, or of rings that go by kernels_ring.hip kGroupSums (streaming ones with windows of two groups: 2)
  uint32_t hist_len;
  uint32_t Ktot;           // sum of K over tensors
  uint64_t Npad;
};

struct StepArgs {
  uint32_t k;
  float lr, mu;
  uint32_t thr_mode;
  float horizon;
  uint32_t force_first;
  uint32_t topk_on;
  uint32_t topk_key;
  uint32_t norm_src;       // what k_trigger finds: 0 squared drift in partials; 1 squared x in
                           // partials, squared xhat in xhat_sq once a tensor has sent; 2 squared x
                           // and squared xhat in partials / partials_hat
  uint32_t delay;          // messages of this iteration land after its updates
  uint32_t hist_fused;     // the update pass of the previous iteration already built pass A's histograms
  uint32_t choose;         // one workgroup per tensor makes the whole selection, from key codes (k_topk_choose)
  uint32_t plain_sgd;      // momentum == 0: the velocity arena is not touched
  uint32_t from_device;    // take k and decay^k from IterState instead of the two fields here
  uint32_t xhat_reset;     // a Top-K event resets the whole tensor's xhat to x
  uint32_t cached;         // the arenas fit the last-level cache: ordinary instead of streaming accesses
  uint32_t walk;           // streaming ring whose mailboxes equal the senders' xhat: update pass of kernels_walk.hip
  uint32_t part;           // walk: workers of the ring that a workgroup goes through (P: all)
  uint32_t pull;           // sends are fetched by the receivers inside the update pass
  uint32_t applied;        // Top-K messages are written and put into the mailboxes ahead of the update pass
  uint32_t one_launch;     // ... and the update pass also runs the trigger tests (no other kernel in the step)
  uint32_t step_no;        // steps completed before this one, where the host counts them (kernels_parts.hip)
  uint32_t key0, key1;
  double decay_pow;        // decay^k
  float spike_prob, spike_gain;
  const float* grad;       // buffer mode only
};

// launchers (each enqueues on the stream and returns the launch status)
hipError_t launch_norm(const Tables& t, bool norm_diff, hipStream_t s);
// norm: 0 no norm work, 1 squared drift, 2 squared x, 3 squared x and squared xhat
hipError_t launch_update(const Tables& t, const StepArgs& a, uint32_t dist, uint32_t grad_mode,
                         int norm, hipStream_t s);
// norm as above; rings for which the host sets StepArgs::walk
hipError_t launch_walk(const Tables& t, const StepArgs& a, uint32_t dist, uint32_t grad_mode, int norm, hipStream_t s);
// norm: 1, 2 or, with Top-K, 1 or 3
hipError_t launch_part(const Tables& t, const StepArgs& a, const PartTables& p, uint32_t dist, uint32_t grad_mode, int norm, hipStream_t s);
// the same, a workgroup to a window of the whole ring
hipError_t launch_ring(const Tables& t, const StepArgs& a, const PartTables& p, uint32_t dist, uint32_t grad_mode, int norm, hipStream_t s);
// most_sums: the partials of the longest tensor
hipError_t launch_trigger(const Tables& t, const StepArgs& a, uint32_t most_sums, hipStream_t s);
hipError_t launch_copy(const Tables& t, const StepArgs& a, uint32_t chunk_elems, hipStream_t s);
hipError_t launch_deliver(const Tables& t, uint32_t chunk_elems, hipStream_t s);
hipError_t launch_topk_decide(const Tables& t, const StepArgs& a, hipStream_t s);
hipError_t launch_topk_select(const Tables& t, const StepArgs& a, uint32_t chunk_elems, hipStream_t s);
// pass A's histograms and the key codes of all tensors, as an update pass leaves them; added to the histograms that are there
hipError_t launch_topk_count_all(const Tables& t, const StepArgs& a, uint32_t chunk_elems, hipStream_t s);
// What k_topk_choose has to know of a tensor (LayerDesc; sum0, sums: its partials in a worker's).
struct ChooseDesc { uint32_t layer, off, numel, K, chunk0, nchunks, sum0, sums; };
// The tensors by size, the `longer` of more than 256 elements first; the longest's elements, at most kChooseMost.
struct ChooseTables { const ChooseDesc* tensors; uint32_t longer, longest; };
// Longer ones are too much for one workgroup.  Steps in us, in many launches / one workgroup a tensor, rings of 3, 5 (4) and 8 (9) perceptrons whose
// longest tensor has 329 000 elements 41.6 / 32.2, (43.8 / 33.6), (62.3 / 41.5); 502 000 44.6 / 38.7, 51.4 / 44.8, 75.2 / 53.0; 706 000 49.8 / 50.7, (59.5 /
// 53.4), (105.6 / 97.4); 784 000 51.7 / 54.4, 74.2 / 66.3, 104.1 / 87.2; with given gradients 329 000 39.6 / 25.9, (42.4 / 27.8), (63.4 / 43.0); 706 000
// 52.5 / 41.3, (60.7 / 47.7), (104.7 / 89.9); 784 000 55.2 / 44.5, 76.7 / 56.5, 104.2 / 79.6.  Three workers that draw their gradients: kChooseMostOf3.  With
// spikes kChooseMostSpiky: after one a tensor's threshold has left the codes, and one workgroup reads all its keys four times; 15 of 60 rings with 329 000 to
// 811 000 elements were 0.45 to 0.98 times as fast as in many launches, the others 1.02 to 1.85 (6 workers of 675 000 65 / 137 us, 9 of 461 000 63 / 128).
constexpr uint32_t kChooseMost = 819200, kChooseMostOf3 = 655360, kChooseMostSpiky = 327680;
hipError_t launch_topk_choose(const Tables& t, const StepArgs& a, const ChooseTables& c, hipStream_t s);
hipError_t launch_topk_apply(const Tables& t, const StepArgs& a, uint32_t chunk_elems, hipStream_t s);
hipError_t launch_average(const Tables& t, float* out, hipStream_t s);
hipError_t launch_message_hashes(const Tables& t, hipStream_t s);

}  // namespace evg
