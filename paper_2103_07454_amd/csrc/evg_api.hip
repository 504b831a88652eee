// Host side of libevg: argument checking, table construction, the per-iteration
// launch sequence and the counters.  See include/evg.h for the contract.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/evg.h"
#include "evg_internal.h"

using namespace evg;

namespace {

thread_local std::string g_err;

evg_status fail(evg_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

#define HIP_TRY(expr)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess)                                                               \
      return fail(e_ == hipErrorOutOfMemory ? EVG_ERR_OOM : EVG_ERR_HIP, "%s: %s", #expr, \
                  hipGetErrorString(e_));                                               \
  } while (0)

inline uint64_t pad_to(uint64_t v, uint64_t m) { return (v + m - 1) / m * m; }

struct TimerPair { hipEvent_t a, b; int phase; };

constexpr uint32_t kDecayTable = 1u << 16;   // iterations a replayable step can reach

// ---- the one block of device memory that evg_init_static hands out -------------------
// Every GPU the library runs on holds its own copy of this array from the moment the
// library is loaded until the process ends.  In host code the array's NAME is only a
// handle for hipGetSymbolAddress: the device address differs per GPU and is looked up
// once per device (scratch_base), and only that address is ever passed to kernels,
// memsets or copies.
constexpr size_t kScratchBytes = EVG_STATIC_SCRATCH_BYTES;
constexpr size_t kScratchAlign = 256;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_scratch_mu;
unsigned char* g_scratch_base[kMaxDevices] = {nullptr};   // per device: where its copy lives
evg_ctx* g_scratch_user[kMaxDevices] = {nullptr};         // per device: the context living in it

}  // namespace

struct evg_ctx {
  evg_config cfg{};
  hipStream_t stream = nullptr;
  Tables t{};
  uint32_t chunk_elems = 8192;
  uint32_t asked_SW = 8;            // sweeps of the chunks asked for (shorter ones if the static block has no room for them)
  std::vector<uint64_t> numel;      // per tensor
  std::vector<uint32_t> K;          // per tensor Top-K message length
  std::vector<uint32_t> msg_off;
  std::vector<void*> owned;         // device allocations to free
  uint64_t N = 0;                   // unpadded elements per worker
  uint64_t iters = 0;
  int64_t last_iter = -1;
  bool messages_live = false;       // the message buffers hold the last step's messages
  bool on_lines = false;            // sweeps begin on cache lines (streaming rings)
  bool walk = false;                // the update pass walks the ring
  uint32_t part = 0;                // workers of the ring that one workgroup of a walking pass goes through
  ChooseTables choose{};            // longest = 0: selections are made in many launches
  uint32_t most_sums = 0;           // partials of the longest tensor
  bool cached = false;              // the five arenas together fit the last-level cache
  bool device_ahead = false;        // evg_step_next has been used: replays of a captured graph
                                    // advance the device's iteration without the host seeing
                                    // it, so iters / last_iter are re-read whenever needed
  // Single-launch steps (cache-resident rings, whole-tensor sends, norms accumulated by the update
  // pass, no tensor longer than 128 sweeps): the update pass goes through the ring in parts of `part` workers and runs the
  // trigger tests itself.  c->t names the set of arrays that holds the current state (use_set).
  PartTables parts{};
  bool one_launch = false;          // the ring qualifies
  bool replayable_used = false;     // evg_step_next has been called: evg_step runs the tests in a kernel of their own from then on
  // evg_init_static: the tables are carved out of the device's static scratch block
  unsigned char* arena_base = nullptr;   // null = tables come from hipMalloc
  size_t arena_used = 0;
  int arena_dev = -1;
  uint64_t owned_bytes = 0;              // device memory handed out by dalloc
  // timing
  bool timing = false;
  std::vector<TimerPair> pending;
  std::vector<hipEvent_t> pool;
  double ms[EVG_PH_COUNT] = {0};
  uint64_t samples[EVG_PH_COUNT] = {0};

  uint64_t hists() const {           // first histograms: one a worker and tensor, and the long tensors' further copies
    const uint64_t longs = (t.long_layer[0] != kNoLayer) + (t.long_layer[1] != kNoLayer);
    return (uint64_t)t.S + (kHistCopies - 1) * longs * t.P;
  }

  template <typename T>
  evg_status dalloc(T** p, size_t count, bool zero) {
    void* d = nullptr;
    const size_t bytes = (count ? count : 1) * sizeof(T);
    if (arena_base) {
      const size_t at = (arena_used + kScratchAlign - 1) / kScratchAlign * kScratchAlign;
      if (at + bytes > kScratchBytes)
        return fail(EVG_ERR_INVALID, "the static scratch block holds %zu bytes; this configuration needs more",
                    kScratchBytes);
      d = arena_base + at;
      arena_used = at + bytes;
    } else {
      hipError_t e = hipMalloc(&d, bytes);
      if (e != hipSuccess) return fail(EVG_ERR_OOM, "hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(e));
      owned.push_back(d);
    }
    owned_bytes += bytes;
    if (zero) HIP_TRY(hipMemsetAsync(d, 0, bytes, stream));
    *p = static_cast<T*>(d);
    return EVG_OK;
  }

  evg_status drain_timers() {
    if (pending.empty()) return EVG_OK;
    HIP_TRY(hipStreamSynchronize(stream));
    for (const TimerPair& p : pending) {
      float m = 0.f;
      HIP_TRY(hipEventElapsedTime(&m, p.a, p.b));
      ms[p.phase] += (double)m;
      samples[p.phase] += 1;
      pool.push_back(p.a);
      pool.push_back(p.b);
    }
    pending.clear();
    return EVG_OK;
  }

  evg_status mark(hipEvent_t* ev) {
    if (pool.empty()) {
      HIP_TRY(hipEventCreate(ev));
    } else {
      *ev = pool.back();
      pool.pop_back();
    }
    HIP_TRY(hipEventRecord(*ev, stream));
    return EVG_OK;
  }
};

namespace {

// Brackets one phase with events when timing is on.
struct Phase {
  evg_ctx* c;
  int phase;
  hipEvent_t a{};
  evg_status st = EVG_OK;
  Phase(evg_ctx* c_, int ph) : c(c_), phase(ph) {
    if (c->timing) st = c->mark(&a);
  }
  evg_status end() {
    if (!c->timing || st != EVG_OK) return st;
    hipEvent_t b;
    st = c->mark(&b);
    if (st == EVG_OK) c->pending.push_back({a, b, phase});
    return st;
  }
};

evg_status check_layers(uint32_t L, const uint64_t* layer_numel) {
  if (L < 1 || !layer_numel) return fail(EVG_ERR_INVALID, "need L >= 1 tensors and their sizes");
  uint64_t total = 0;
  for (uint32_t l = 0; l < L; ++l) {
    if (layer_numel[l] < 1 || layer_numel[l] > 0x7FFFFFF8ull)
      return fail(EVG_ERR_INVALID, "tensor %u has %llu elements (1 .. 2^31-8 allowed)", l,
                  (unsigned long long)layer_numel[l]);
    total += pad_to(layer_numel[l], 4);
    if (total > 0xFFFFFF00ull) return fail(EVG_ERR_INVALID, "a worker's slice exceeds 2^32 floats");
  }
  return EVG_OK;
}

bool finite_f(float v) { return std::isfinite(v); }

// A kernel that is handed host memory, or an array shorter than the sizes say, faults
// the GPU; so ask the runtime what `p` is.  The range test sees the whole allocation
// `p` lies in (a sub-allocator's pool block counts as one), so it catches what runs
// past that; where the runtime cannot name the range the test is skipped.
evg_status check_device_array(const void* p, uint64_t bytes, const char* what) {
  hipPointerAttribute_t at;
  hipError_t e = hipPointerGetAttributes(&at, p);
  if (e != hipSuccess || (at.type != hipMemoryTypeDevice && at.type != hipMemoryTypeManaged)) {
    (void)hipGetLastError();   // a failed query must not surface after the next launch
    return fail(EVG_ERR_INVALID, "%s does not point to device memory", what);
  }
  int dev = -1;
  if (hipGetDevice(&dev) == hipSuccess && at.device != dev)
    return fail(EVG_ERR_INVALID, "%s lives on device %d, the current device is %d", what, at.device, dev);
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  e = hipMemGetAddressRange(&base, &size, const_cast<void*>(p));
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return EVG_OK;
  }
  const uintptr_t end = (uintptr_t)base + size;
  if ((uintptr_t)p < (uintptr_t)base || (uintptr_t)p + bytes > end)
    return fail(EVG_ERR_INVALID, "%s needs %llu bytes, its allocation ends after %llu", what,
                (unsigned long long)bytes, (unsigned long long)(end - (uintptr_t)p));
  return EVG_OK;
}

}  // namespace

extern "C" {

const char* evg_strerror(evg_status s) {
  switch (s) {
    case EVG_OK: return "ok";
    case EVG_ERR_INVALID: return "invalid argument";
    case EVG_ERR_ALIGN: return "misaligned device pointer";
    case EVG_ERR_OOM: return "out of memory";
    case EVG_ERR_HIP: return "HIP runtime error";
    case EVG_ERR_STATE: return "call out of order";
  }
  return "unknown status";
}

const char* evg_error_text(void) { return g_err.c_str(); }

uint64_t evg_padded_numel(uint32_t L, const uint64_t* layer_numel) {
  if (check_layers(L, layer_numel) != EVG_OK) return 0;
  uint64_t total = 0;
  for (uint32_t l = 0; l < L; ++l) total += pad_to(layer_numel[l], 4);
  return pad_to(total, 64);
}

evg_status evg_layer_offsets(uint32_t L, const uint64_t* layer_numel, uint64_t* offsets_out) {
  if (!offsets_out) return fail(EVG_ERR_INVALID, "offsets_out is NULL");
  evg_status st = check_layers(L, layer_numel);
  if (st != EVG_OK) return st;
  uint64_t total = 0;
  for (uint32_t l = 0; l < L; ++l) {
    offsets_out[l] = total;
    total += pad_to(layer_numel[l], 4);
  }
  return EVG_OK;
}

evg_status evg_destroy(evg_ctx* c) {
  if (!c) return EVG_OK;
  (void)hipStreamSynchronize(c->stream);
  if (c->arena_base) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (c->arena_dev >= 0 && g_scratch_user[c->arena_dev] == c) g_scratch_user[c->arena_dev] = nullptr;
  }
  for (void* p : c->owned) (void)hipFree(p);
  for (const TimerPair& p : c->pending) { (void)hipEventDestroy(p.a); (void)hipEventDestroy(p.b); }
  for (hipEvent_t e : c->pool) (void)hipEventDestroy(e);
  delete c;
  return EVG_OK;
}

// Sizes of a list of tables, every one rounded up to the scratch block's alignment.
struct TableSum {
  uint64_t total = 0;
  void add(uint64_t count, uint64_t elem) {
    total = (total + kScratchAlign - 1) / kScratchAlign * kScratchAlign + (count ? count : 1) * elem;
  }
};

// Bytes of library-owned device tables a configuration needs: the same list as the allocations of init_common.
static uint64_t table_bytes(uint64_t P, uint64_t L, uint64_t C, uint64_t SW, uint64_t hist_len, uint64_t Npad,
                            uint64_t ktot, bool topk, bool norm_diff, bool pull, bool one_launch, uint64_t windows, uint64_t parts, bool codes, uint64_t hists, uint64_t fine) {
  const uint64_t S = P * L, PC = P * C;
  TableSum t;
  t.add(C, sizeof(ChunkDesc)); t.add(L, sizeof(LayerDesc));
  t.add(PC * SW * fine, 8);
  if (norm_diff) { t.add(PC * SW * fine, 8); t.add(S, 8); }
  t.add(S, 4); t.add(S, 4); t.add(S, 4); t.add(S, 4);            // delta, last_norm, delta_before, last_event
  for (int i = 0; i < 4; ++i) t.add((S + 3) / 4 * 4, 1);         // valid_l, valid_r, fired (whole words are read), near_tie
  t.add(S, 4); t.add(S, 4); t.add(S, 4); t.add(S, 4);            // ev_full, ev_topk, near_cnt, nonfinite_cnt
  t.add(S * hist_len, 4); t.add(S, 4);                           // slope_hist, slope_cnt
  t.add(1, 4); t.add(1, sizeof(IterState)); t.add(kDecayTable, 8);
  if (pull) t.add(2 * P * Npad, 4);                              // xsnap
  if (one_launch) {                                              // the second set of what the trigger tests read
    t.add(PC * SW * fine, 8); t.add(S, 4); t.add(S, 4);
    if (norm_diff) t.add(S, 8);
    t.add(windows * parts, sizeof(PartClock));
  }
  if (windows) t.add(windows, sizeof(WindowDesc));
  if (topk) {
    t.add(hists * kHistBins, 4); t.add(S, 4); t.add(S, 4); t.add(S, 4); t.add(PC, 4);   // hist, selection, stage_n
    t.add(P * (Npad / 16 * 4), 4);                               // stage_key
    t.add(PC * SW * 4, 4); t.add(PC, 8); t.add(PC, 8);           // group, chunk_cnt, chunk_before
    t.add(P * ktot, 4); t.add(P * ktot, 4); t.add(S, 8); t.add(S, 8);
    t.add(S, 4); t.add(S, 4);                                     // anchor, sel_left
    if (codes) t.add(P * Npad + 16, 1);
    t.add(L, sizeof(ChooseDesc));                                  // tensors by size
  }
  return t.total;
}

// What evg_init_static admits is part of its interface, and older than the present tables: it is reckoned with those of the
// library's first version, whose tensors were cut at their own starts (C chunks a worker), with lists of fired
// chunks, and for Top-K with three words for each possible winner (one and a half times the Top-K share plus a
// sixteenth, in quarters of the ring), but without copies of x.  Whatever it admits has room, in chunks of 1024 elements if
// need be: those take 44 bytes each besides a quarter of the staging words, where the old lists took at least 48 a
// chunk and 2 more for each element (Top-K; whole sends need less than they did).
static uint64_t admitted_bytes(uint64_t P, uint64_t L, uint64_t C, uint64_t SW, uint64_t hist_len, uint64_t Npad,
                               uint64_t ktot, uint32_t topk_ppm, bool norm_diff, bool whole_copies, bool one_launch) {
  const uint64_t S = P * L, PC = P * C;
  TableSum t;
  t.add(C, 16); t.add(L, sizeof(LayerDesc));
  t.add(PC * SW, 8);
  if (norm_diff) { t.add(PC * SW, 8); t.add(S, 8); }
  for (int i = 0; i < 4; ++i) t.add(S, 4);
  for (int i = 0; i < 4; ++i) t.add(S, 1);
  for (int i = 0; i < 4; ++i) t.add(S, 4);
  t.add(S * hist_len, 4);
  for (int i = 0; i < 3; ++i) t.add(S, 4);
  t.add(4, 4); t.add(1, sizeof(IterState)); t.add(kDecayTable, 8);
  t.add(PC, 4);
  if (whole_copies) t.add(2 * P * Npad, 4);
  if (one_launch) {
    t.add(PC * SW, 8); t.add(S, 4); t.add(S, 4);
    if (norm_diff) t.add(S, 8);
  }
  if (topk_ppm) {
    t.add(PC, 4); t.add(S * kHistBins, 4); t.add(S, 4); t.add(S, 4); t.add(PC, 8);
    const uint64_t want = (3ull * topk_ppm * 8ull + 999999ull) / 1000000ull + 1ull;   // in sixteenths
    const uint64_t stage = P * (Npad / 16 * (want <= 4 ? 4 : want <= 8 ? 8 : want <= 12 ? 12 : 16));
    t.add(stage, 4); t.add(stage, 4); t.add(stage, 4);
    t.add(PC, 8); t.add(PC, 8); t.add(PC * (SW + 1), 4);
    t.add(P * ktot, 4); t.add(P * ktot, 4); t.add(S, 8); t.add(S, 8);
  }
  return t.total;
}

// The shape of the workgroups of kernels_ring.hip for a ring that is cached by its size (`windows` of 1024 elements), groups = 0: it goes by
// kernels_parts.hip, like the larger ones that are cached because that is asked for.
// With few float4s in the ring a thread has one of them and windows are short, so that there are workgroups; with more, two, as
// the sums that the tests read and the threads get many.  Four workers or fewer with long networks: whole sweeps.  A workgroup of more than twelve wavefronts leaves
// a CU too few of them beside it unless it has much to load.  Kernels_parts.hip / groups and quads 1 1 / 2 1 / 2 2 / 4 2, us a step, normal
// gradients: perceptrons of 102 windows on 4 workers 6.2 / 5.7 / 5.4 / 5.6 / 6.2, 39 on 4 5.1 / 4.5 / 4.7 / 4.9 / 5.4, 506 on 6 22.0 / 20.6 / 20.2 / 17.3 /
// 17.9; ResNet-20 of 314 on 3 8.8 / 7.4 / 7.9 / 7.8 / 8.5, on 8 14.5 / 13.6 / 16.5 / 12.6 / 15.6, of 186 on 15 13.7 / 16.3 / - / 15.3 / -;
// ResNet-18 of 729 on 4 16.9 / 18.2 / 18.6 / 17.8 / 16.8, ResNet-20 of 923 on 4 17.2 / - / - / - / 17.8; more workers have one float4 each of several: 120 windows on 24 12.7 and 15.4.  Top-K, kernels_parts.hip / 1 2 / 2 2:
// ResNet-20 of 314 windows on 8 33.6 / 32.4 / 32.3, on 16 45.1 / 43.9 / 49.6, of 426 on 10 36.5 / 37.1 / 38.6; perceptrons of 129 on 11 32.4 / - / 34.9, of
// 237 on 10 44.0 / 49.2 / 45.8; ResNet-18 of 729 on 4 39.7 / - / 41.4, ResNet-20 of 509 on 4 with given gradients 27.8 / - / 25.8.
// One ring differs by up to a fifth between allocations of its arenas.  More rings, each in four of them, how many times as fast as with kernels_parts.hip:
//   windows that are mostly empty, on 3 and 4 workers (tensors of 4, 30 and 200 elements): 4 2 0.82 .. 1.13, 1 1 1.4 .. 2.5
//   a tensor of 131 000 elements on 8: 2 1 0.92, 1 1 1.21; of 112 000 to 128 000 on 5 to 7 2 1 1.13 .. 1.15, 1 1 1.13 .. 1.18
//   7 and 8 workers, ResNets of 4000 units and more in one part of the ring: normal gradients 0.90 .. 1.00 (6 rings), Student-t's and given ones 1.00 .. 1.23; with a
//   tensor whose tests need a launch of their own, in parts of four, 1.1 and 1.2
//   9 to 12, drawn gradients: where every CU has had two workgroups and a few are left (513 to 600) and parts are of four workers 0.89 .. 0.96 (3 rings), else
//   0.98 .. 1.33 (24 rings, 1.06 in the middle)
//   13 to 16, drawn gradients, of 512 elements: normal ones, ResNets 0.78 .. 1.02 (21 rings, 0.96), perceptrons 1.08 .. 1.20; Student-t's, up to 680 workgroups 0.98 .. 1.31
//   (513 and more with spikes 0.89 .. 0.93), more 0.81 .. 1.07 (18 rings, 0.99).  Where windows are mostly empty (tensors of 4 to 1100 elements), 7 to 16 workers, 1.1 .. 1.7
//   13 to 16, given ones, where a workgroup has a CU: 1 1 of up to 256 of them 1.19 .. 1.28 (below 800 units, where it is not taken, 1.15 .. 1.21 on four rings), of more 0.81 .. 0.94 where 2 2 is 1.05 .. 1.17; 2 2 of
//   264 (ResNet-20 of width 10) 0.86 .. 0.93, of 265 to 288 in a perceptron 1.09 .. 1.11, else 0.89 .. 1.31 (53 rings, 1.11)
//   Top-K, 9 to 16, drawn gradients: of 2700 units and more 0.85 .. 1.07 (34 rings, 0.95; where windows are mostly empty 1.0 .. 1.3), fewer 1.00 .. 1.13 (with a tensor
//   of 155 000 elements 0.92)
static void ring_shape(uint32_t P, uint64_t windows, const std::vector<LayerDesc>& layers, uint64_t N, bool topk, bool tests, bool given, bool normal, bool spikes,
                       uint32_t* groups, uint32_t* quads) {
  *groups = *quads = 0;
  const uint64_t units = windows * P;
  uint64_t longest = 0, of256 = 0, of512 = 0;              // elements of the longest tensor; workgroups
  for (const LayerDesc& d : layers) {
    longest = std::max<uint64_t>(longest, d.numel);
    of256 += (d.numel + 255ull) / 256;
    of512 += (d.numel + 511ull) / 512;
  }
  const bool one_long = 2 * longest > N, thin = 10 * N < 6 * 1024 * windows;       // windows are mostly empty, or nearly so
  if (P > 16 || (P > 12 && units < (given && !topk ? 800 : 4000))) return;
  if (topk) {
    if (units < 1700 || (longest > 150000 && P > 8) || (P <= 4 && !given) || (P > 8 && !given && !thin && units >= 2700)) return;
    *groups = P > 12 ? 1 : 2;
    *quads = 2;
  } else if (P > 12) {
    if (!thin && (given ? of256 > 256 && of512 > 256 && of512 <= 288 && !one_long : normal ? !one_long : of512 > (spikes ? 512 : 680))) return;
    *groups = *quads = given && of256 <= 256 ? 1 : 2;
  } else if (P <= 4 && windows >= 700 && !given) {
    return;
  } else if (P <= 4 && windows >= 400) {
    const bool full = 5 * N >= 2 * 1024 * windows;
    *groups = full ? 4 : 1;
    *quads = full ? 2 : 1;
  } else if (units >= 1300) {
    if (!given && !one_long && !thin && (P > 8 ? of512 > 512 && of512 <= 600 && units < 3400 : P > 6 && tests && normal && units >= 4000)) return;
    *groups = *quads = 2;
  } else {
    *groups = tests && longest > 65536 && P <= 6 ? 2 : 1;
    *quads = 1;
  }
}

// The same for a ring that streams from memory and sends whole tensors; groups = 0: it is walked.  `row`: bytes of a worker's slice.
// Short windows put a CU's wavefronts to different tasks, but each has a sum that the tests read; workgroups have no more than sixteen wavefronts.
// Walked / groups and quads 1 1 / 2 1 / 1 2 / 1 4, us a step: ResNet-18 of width 23 on 7 workers 64.7 / 55.0 / 53.6 / 55.2 / 58.0, with given
// gradients and plain SGD 54.0 / 48.5 / 47.5 / 48.6 / 49.8, of width 60 on 6 275 / 271 / 267 / 272 / 286, of width 64 on 16 873 / 817 / - / 846 / 844,
// with given gradients 1035 / 1022 / - / 1025 / 1010; ResNet-50 of width 30 on 15 496 / 450 / - / 482 / 472; ResNet-20 of width 24 on 13 49.6 / 37.5 / - /
// 36.2 / 36.8, of width 21 on 23 80.0 / - / - / 47.3 / 51.0; perceptrons of 471 000 elements on 18 45.2 / - / - / 38.0 / 38.6; ResNet-50 of width 48 on 29 1584 / - /
// - / 1601 / 1500, of width 39 on 19 943 / - / - / 917 / 902; ResNet-20 of width 24 on 47 205 / - / - / - / 140, ResNet-18 of width 20 on 57 (1.2 GB) 403 / - / - / - / 367, of width 26 on 47
// (1.7 GB) 539 / - / - / - / 571, of width 42 on 35 (3.2 GB) 631 / - / - / - / 685.
// A ring differs by up to a fifth between allocations of its arenas, so that a line takes many rings and some allocations of each (four): 98 drawn ones of 3 to
// 32 workers are 0.91 to 1.64 times as fast as walked (1.07 in the middle; 52 of more than 1.5 GB 0.91 to 1.12, 1.04), 9 ResNets on 33 to 40 1.06 to
// 1.61.  Of more than 32 workers whose network is mostly one long tensor, 28 perceptrons with a tensor of 280 000 elements and more are 0.87 to 1.10 times as
// fast (0.99): walked; 9 shorter ones 1.03 to 1.37.
// All workers' stretches of a window are read and written at once.  Where they lie multiples of 8 KB apart, or nearly, those of more than eight workers can get in each
// other's way in the memory: ResNet-18 of width 39 with workers 8192 n + 0, 256, 1024, 2048 and 4096 bytes apart on 20 workers 0.83 .. 0.93, 0.95, 0.98, 0.97 and 0.97
// times as fast as walked, on 12 0.86 .. 0.91, 0.95, 1.01, 1.01 and 0.99, on 7 1.00 .. 1.08, 1.05, 1.08, 1.09 and 1.10.  (Not always: ResNet-50s of width 17 to 44 on 10 to 29
// workers, 8192 n + 0 and 256 apart, would be 1.04 to 1.18 times as fast.)  From 512 bytes on: 22 rings with
// workers 8192 n + 512 to 1280 bytes apart, or as much less, 0.94 to 1.64 times as fast (1.06 in the middle).
static void stream_shape(uint32_t P, uint64_t row, uint64_t N, uint32_t longest, uint32_t* groups, uint32_t* quads) {
  *groups = *quads = 0;
  const uint64_t bytes = 5 * P * row, apart = (row + 256) % 8192;      // (rows are multiples of 256 bytes)
  if (P > kRingMost || (P > 32 && (bytes > (1ull << 30) || (longest > 262144 && 2ull * longest > N))) || (P > 8 && apart <= 512)) return;
  *groups = P <= 8 ? 2 : 1;
  *quads = P <= 16 ? 1 : P <= 32 && bytes < (600ull << 20) ? 2 : 4;
}

static evg_status init_common(evg_ctx** out, const evg_config* cfg, void* hip_stream, bool use_scratch) {
  if (!out || !cfg) return fail(EVG_ERR_INVALID, "out and cfg must be non-NULL");
  evg_status st = check_layers(cfg->L, cfg->layer_numel);
  if (st != EVG_OK) return st;
  if (cfg->P < 3 || cfg->P > 65535)
    return fail(EVG_ERR_INVALID, "ring size P = %u (3 .. 65535: a worker needs two distinct neighbours)", cfg->P);
  if (!finite_f(cfg->lr) || !finite_f(cfg->momentum)) return fail(EVG_ERR_INVALID, "lr and momentum must be finite");
  if (cfg->thr_mode > EVG_THR_ADAPTIVE) return fail(EVG_ERR_INVALID, "unknown thr_mode %u", cfg->thr_mode);
  if (cfg->thr_mode == EVG_THR_FIXED && !(cfg->thr_fixed >= 0.0f))
    return fail(EVG_ERR_INVALID, "thr_fixed must be >= 0 (+inf allowed)");
  if (cfg->thr_mode == EVG_THR_ADAPTIVE) {
    if (!finite_f(cfg->horizon) || cfg->horizon < 0.0f) return fail(EVG_ERR_INVALID, "horizon must be finite and >= 0");
    if (!(cfg->delta_init >= 0.0f)) return fail(EVG_ERR_INVALID, "delta_init must be >= 0");
    if (cfg->hist_len < 1 || cfg->hist_len > 16) return fail(EVG_ERR_INVALID, "hist_len must be 1 .. 16");
  }
  if (cfg->topk_ppm > 1000000u) return fail(EVG_ERR_INVALID, "topk_ppm must be <= 1000000");
  if (cfg->topk_key > EVG_KEY_ABS_VALUE) return fail(EVG_ERR_INVALID, "unknown topk_key %u", cfg->topk_key);
  if (cfg->grad_mode > EVG_GRAD_BUFFER) return fail(EVG_ERR_INVALID, "unknown grad_mode %u", cfg->grad_mode);
  if (cfg->norm_mode > EVG_NORM_SEPARATE) return fail(EVG_ERR_INVALID, "unknown norm_mode %u", cfg->norm_mode);
  if (cfg->trigger_kind > EVG_TRIGGER_NORM_DIFF) return fail(EVG_ERR_INVALID, "unknown trigger_kind %u", cfg->trigger_kind);
  if (cfg->delivery_delay > 1) return fail(EVG_ERR_INVALID, "delivery_delay must be 0 or 1");
  if (cfg->xhat_reset > 1) return fail(EVG_ERR_INVALID, "xhat_reset must be 0 or 1");
  if (cfg->xhat_reset && cfg->delivery_delay)
    return fail(EVG_ERR_INVALID, "xhat_reset = 1 is not available with delivery_delay = 1");
  if (cfg->access_mode > EVG_ACCESS_CACHED) return fail(EVG_ERR_INVALID, "unknown access_mode %u", cfg->access_mode);
  if (cfg->chunk_elems != 0 && cfg->chunk_elems != 1024 && cfg->chunk_elems != 2048 &&
      cfg->chunk_elems != 4096 && cfg->chunk_elems != 8192)
    return fail(EVG_ERR_INVALID, "chunk_elems must be 0, 1024, 2048, 4096 or 8192");
  if (cfg->grad_mode == EVG_GRAD_SYNTH) {
    const evg_synth& s = cfg->synth;
    if (s.dist > EVG_DIST_STUDENT_T3) return fail(EVG_ERR_INVALID, "unknown synth.dist %u", s.dist);
    if (!std::isfinite(s.sigma0) || s.sigma0 < 0) return fail(EVG_ERR_INVALID, "synth.sigma0 must be finite and >= 0");
    if (!std::isfinite(s.decay) || s.decay <= 0) return fail(EVG_ERR_INVALID, "synth.decay must be finite and > 0");
    if (!(s.spike_prob >= 0.0f && s.spike_prob <= 1.0f)) return fail(EVG_ERR_INVALID, "synth.spike_prob must be in [0,1]");
    if (!finite_f(s.spike_gain)) return fail(EVG_ERR_INVALID, "synth.spike_gain must be finite");
    if (s.fan_in_scaling) {
      if (!cfg->layer_fan_in) return fail(EVG_ERR_INVALID, "fan_in_scaling needs layer_fan_in");
      for (uint32_t l = 0; l < cfg->L; ++l)
        if (cfg->layer_fan_in[l] < 1) return fail(EVG_ERR_INVALID, "layer_fan_in[%u] must be >= 1", l);
    }
  }
  const uint64_t Npad = evg_padded_numel(cfg->L, cfg->layer_numel);
  const uint64_t arena_bytes = (uint64_t)cfg->P * Npad * 4;
  // rings that live in the last-level cache are bound by launch and workgroup counts, not by
  // HBM: small granules leave fewer empty sweeps behind their many short tensors (measured)
  const bool small_ring = 5 * arena_bytes <= (128ull << 20);
  uint32_t ce = cfg->chunk_elems ? cfg->chunk_elems : small_ring ? 2048u : 8192u;
  const float* arenas[5] = {cfg->x, cfg->xhat, cfg->mbox_l, cfg->mbox_r, cfg->vel};
  static const char* names[5] = {"x", "xhat", "mbox_l", "mbox_r", "vel"};
  for (int i = 0; i < 5; ++i) {
    if (!arenas[i]) return fail(EVG_ERR_INVALID, "arena %s is NULL", names[i]);
    if ((uintptr_t)arenas[i] % 16) return fail(EVG_ERR_ALIGN, "arena %s is not 16-byte aligned", names[i]);
  }
  for (int i = 0; i < 5; ++i)
    for (int j = i + 1; j < 5; ++j) {
      const uintptr_t a = (uintptr_t)arenas[i], b = (uintptr_t)arenas[j];
      if (a < b + arena_bytes && b < a + arena_bytes)
        return fail(EVG_ERR_INVALID, "arenas %s and %s overlap", names[i], names[j]);
    }
  // everything above is plain arithmetic; from here on the HIP runtime is involved
  for (int i = 0; i < 5; ++i)
    if ((st = check_device_array(arenas[i], arena_bytes, names[i])) != EVG_OK) return st;

  // ---- host tables --------------------------------------------------------
  evg_ctx* c = new (std::nothrow) evg_ctx();
  if (!c) return fail(EVG_ERR_OOM, "host allocation failed");
  c->cfg = *cfg;
  c->cfg.layer_numel = nullptr;
  c->cfg.layer_fan_in = nullptr;
  c->stream = static_cast<hipStream_t>(hip_stream);
  const uint32_t P = cfg->P, L = cfg->L;
  std::vector<LayerDesc> layers(L);
  std::vector<ChunkDesc> chunks;
  uint64_t off = 0, ktot = 0;
  for (uint32_t l = 0; l < L; ++l) {
    const uint64_t n = cfg->layer_numel[l];
    LayerDesc& d = layers[l];
    d.off = (uint32_t)off;
    d.numel = (uint32_t)n;
    uint64_t k = 0;
    if (cfg->topk_ppm) {
      k = (n * (uint64_t)cfg->topk_ppm + 999999ull) / 1000000ull;
      if (k < 1) k = 1;
      if (k > n) k = n;
    }
    d.K = (uint32_t)k;
    d.msg_off = (uint32_t)ktot;
    ktot += k;
    d.sig_base = cfg->synth.sigma0;
    if (cfg->grad_mode == EVG_GRAD_SYNTH && cfg->synth.fan_in_scaling)
      d.sig_base = cfg->synth.sigma0 / std::sqrt((double)cfg->layer_fan_in[l]);
    c->numel.push_back(n);
    c->K.push_back(d.K);
    c->msg_off.push_back(d.msg_off);
    c->N += n;
    off += pad_to(n, 4);
  }
  // 256 MB of last-level cache on MI355X; a ring whose arenas take at most half of it is served from there and does better
  // with ordinary than with streaming accesses.  A Top-K ring with copies of x has seven arenas: asked for cached
  // accesses beyond the cache's size it is streamed all the same (8 ResNet-18 workers of width 22, 240 MB: cached and with copies
  // 153 us a step, streamed 119; of width 64 on 16 1092 instead of 2061).
  // Few windows (1024 elements of a tensor) leave a walking pass, which goes from worker to worker, short of workgroups,
  // and Top-K rings of up to 220 MB with fewer than 600 of them do better with cached accesses: 40 ResNet-18 workers of width 8 (134
  // MB) 128 us a step against 194 streamed, with messages put into the mailboxes ahead of the update pass where the
  // copies do not fit 64 of width 8 (215 MB) 197 against 262, 24 perceptrons of width 512 (186 MB) 110 against 132; but 24 of width
  // 14 (246 MB) 180 against 172, 64 perceptrons of width 256 (248 MB) 157 against 151.
  const bool topk_now = cfg->topk_ppm && !cfg->delivery_delay;
  const bool copies_fit = 7 * arena_bytes <= (256ull << 20);
  uint64_t windows = 0;
  for (const LayerDesc& d : layers) windows += ((uint64_t)d.numel + d.off % kLineElems + kSweep - 1) / kSweep;
  const bool few = topk_now && windows < 600 && 5 * arena_bytes <= (220ull << 20);
  c->cached = cfg->access_mode == EVG_ACCESS_AUTO ? small_ring || few
                                                  : cfg->access_mode == EVG_ACCESS_CACHED && (!topk_now || copies_fit || few);
  // Streaming rings: sweeps begin on cache lines.  A network whose widths are no multiples of 32 has its
  // tensors anywhere on multiples of 16 bytes; wavefronts then share the lines where they meet and write
  // parts of them.  Step times without -> with, whole sends: ResNet-18 of width 62, 16 workers 1031 -> 945 us;
  // width 28, 60 workers 843 -> 771 us; width 40, 30 workers 871 -> 796 us.  Not where the additional chunks
  // would take the tables past a limit.
  const uint32_t hist_len = cfg->thr_mode == EVG_THR_ADAPTIVE ? cfg->hist_len : 1;
  const uint32_t ce_asked = ce;
  uint32_t SW = ce / (uint32_t)kSweep;
  // Receivers fetch the sends from copies of x.  Not Top-K sends of rings whose xhat is reset at events: a mailbox then does
  // not hold what the message was told from.  Nor of rings with a norm pass of their own, in which nothing else is
  // carried from step to step: a caller may have written x since the copies were made, and the sender goes by x.
  bool pull = c->cached && !cfg->delivery_delay &&
              !(cfg->topk_ppm && (cfg->xhat_reset || cfg->norm_mode == EVG_NORM_SEPARATE || !copies_fit));
  bool in_parts = false, one_launch = false, one_shot = false, may_be = true, ring_may_be = true, sets_counted = false;
  bool codes = cfg->topk_ppm && cfg->norm_mode == EVG_NORM_FUSED, choose = false, hist_copies = codes;
  uint64_t need = 0, ring_windows = 0;
  // A tensor that is most of a ring has all workgroups of an update pass add their counts to one histogram, on all XCDs, at some 30 ns for each
  // addition to an address; of other rings each XCD has tensors of its own (kernels_walk.hip).  One histogram -> one for each XCD, us a
  // step: 9 perceptrons of 813 000 elements, given gradients, 152 -> 83, 30 of 556 000 225 -> 172, 3 of 461 000 (cached) 48 -> 45; streamed, 24 of 198 000
  // 89 -> 78, 64 of 135 000 115 -> 109, 64 of 79 000 79 -> 78, 24 of 119 000 68.4 -> 68.7 (with copies from 16 384 elements on).  Tensors of more than an
  // eighth of a ring, ResNet-18 of width 16 to 64 on 8 and 16 workers, the two longest: within 0.5 %.
  std::vector<uint32_t> long_layers;
  uint32_t ring_part = 0;
  uint32_t longest = 0, groups = 0, quads = 0, fine = 1;
  for (const LayerDesc& d : layers) longest = std::max(longest, d.numel);
  const uint32_t most_chosen = cfg->grad_mode == EVG_GRAD_BUFFER ? kChooseMost : cfg->synth.spike_prob > 0.0f ? kChooseMostSpiky : P > 3 ? kChooseMost : kChooseMostOf3;
  auto cut_chunks = [&](bool on_lines) {
    chunks.clear();
    uint32_t most_sweeps = 0;
    for (uint32_t l = 0; l < L; ++l) {
      LayerDesc& d = layers[l];
      const uint32_t lead = on_lines ? d.off % kLineElems : 0u;
      d.chunk0 = (uint32_t)chunks.size();
      d.nchunks = (uint32_t)(((uint64_t)d.numel + lead + ce - 1) / ce);
      for (uint32_t i = 0; i < d.nchunks; ++i) {
        ChunkDesc cd;
        cd.lead = i == 0 ? lead : 0u;
        cd.j0 = i == 0 ? 0u : i * ce - lead;
        cd.off = d.off + cd.j0;
        cd.len = std::min(d.numel - cd.j0, ce - cd.lead);
        cd.layer = l;
        chunks.push_back(cd);
      }
      most_sweeps = std::max(most_sweeps, d.nchunks * SW);
    }
    // Cached rings that send whole tensors and accumulate the norms in the update pass are updated in parts of the ring; in
    // one launch per iteration where one wavefront sums a tensor's sweep partials with two loads per lane.
    in_parts = may_be && pull && cfg->norm_mode == EVG_NORM_FUSED && arena_bytes < (1ull << 30) && (!cfg->topk_ppm || (codes && longest <= most_chosen));
    one_launch = in_parts && !cfg->topk_ppm && most_sweeps <= 128;
    // (admission counts the second set of what the tests read also where the parts find no room, as it always has)
    sets_counted = pull && !cfg->topk_ppm && cfg->norm_mode == EVG_NORM_FUSED && most_sweeps <= 128;
    choose = in_parts && cfg->topk_ppm;
    long_layers.clear();
    for (uint32_t l = 0; l < L && hist_copies && !choose; ++l)
      if (layers[l].numel >= kHistCopiesFrom && 8ull * layers[l].numel > 3 * c->N) long_layers.push_back(l);
    ring_windows = 0;
    for (const ChunkDesc& cd : chunks) ring_windows += (cd.len + kSweep - 1) / kSweep;
    // Longer parts read less of other parts' workers and run fewer tests twice, shorter ones are more workgroups.  Parts
    // of 2 / 4 / 8, us a step: 102 windows on 4 workers 5.8 / 6.8 / -, 120 on 8 7.2 / 7.7 / 11.2, on 24 12.7 / 12.5 / 15.6; 314 on
    // 8 15.7 / 14.3 / 16.6, on 12 25.7 / 22.6 / 19.2, on 16 34.1 / 33.4 / 30.7; 438 on 8 24.9 / 21.8 / 18.4, on 16 53.3 / 48.9 / 49.0.
    groups = quads = 0;
    fine = 1;
    if (ring_may_be && in_parts && small_ring) ring_shape(P, windows, layers, c->N, cfg->topk_ppm != 0, one_launch, cfg->grad_mode == EVG_GRAD_BUFFER, cfg->synth.dist == EVG_DIST_NORMAL, cfg->synth.spike_prob > 0.0f, &groups, &quads);
    if (may_be && !c->cached && !cfg->topk_ppm && !cfg->delivery_delay && cfg->norm_mode == EVG_NORM_FUSED) stream_shape(P, Npad * 4, c->N, longest, &groups, &quads);
    one_shot = groups && !in_parts;
    if (groups) {
      fine = one_shot && groups == 2 ? 2 : kGroupSums;
      ring_windows = 0;
      for (const ChunkDesc& cd : chunks) ring_windows += (cd.lead + cd.len + 256 * groups - 1) / (256 * groups);
    }
    const uint64_t units = ring_windows * P;
    ring_part = std::min<uint32_t>(P, units < 900 ? 2 : units < 3400 ? 4 : kPartMost);
    // Top-K, parts of 1 / 2 / 4: 28 windows on 8 workers 19.9 / 21.2 / 23.9, 120 on 5 20.8 / 21.3 / 24.0, 160 on 12 38.2 / 36.8 / 37.0, 314 on
    // 8 35.2 / 32.8 / 32.6, on 24 106 / 103 / 98, 438 on 12 78 / 78 / 69.
    if (cfg->topk_ppm) ring_part = std::min<uint32_t>(P, units < 900 ? 1 : units < 1600 ? 2 : 4);
    else if (in_parts && !one_launch) ring_part = std::min<uint32_t>(ring_part, 4);
    if (groups) ring_part = P;
    need = table_bytes(P, L, chunks.size(), SW, hist_len, Npad, ktot, cfg->topk_ppm != 0,
                       cfg->trigger_kind == EVG_TRIGGER_NORM_DIFF, pull && !(in_parts && ring_part == P), one_launch,
                       in_parts || one_shot ? ring_windows : 0, (P + ring_part - 1) / ring_part, codes && (choose || !c->cached),
                       (uint64_t)P * L + (kHistCopies - 1) * P * long_layers.size(), fine);
    return (uint64_t)P * chunks.size() * (SW + 1) <= 0xFFFFFFF0ull && (uint64_t)P * ktot <= 0xFFFFFFF0ull &&
           !(use_scratch && need > kScratchBytes);
  };
  c->on_lines = !c->cached && cut_chunks(true);
  if (!c->cached && !c->on_lines && one_shot) {                 // no room for a descriptor a window
    may_be = false;
    c->on_lines = cut_chunks(true);
  }
  if (!c->on_lines) (void)cut_chunks(false);
  if (use_scratch && need > kScratchBytes && in_parts && groups) {      // thousands of short tensors: no room for a sum a group, parts of the ring
    ring_may_be = false;                                                // may have it
    (void)cut_chunks(false);
  }
  if (use_scratch && need > kScratchBytes && in_parts && !cfg->topk_ppm) {        // ... nor for what the parts take
    may_be = false;
    (void)cut_chunks(false);
  }
  if (use_scratch && need > kScratchBytes && hist_copies) {     // no room for a long tensor's histograms
    hist_copies = false;
    (void)cut_chunks(c->on_lines);
  }
  if (use_scratch && need > kScratchBytes && codes) {           // no room for key codes: x and xhat are read instead
    codes = false;
    (void)cut_chunks(c->on_lines);
  }
  if (use_scratch && need > kScratchBytes && pull && cfg->topk_ppm) {   // no room for the copies of x: messages are applied
    pull = false;                                                        // by a kernel of their own
    (void)cut_chunks(false);
  }
  if (use_scratch && need > kScratchBytes && cfg->topk_ppm && SW > 1) {   // thousands of short tensors: their chunks have as many
    ce = kSweep;                                                          // counts as long ones
    SW = 1;
    (void)cut_chunks(false);
  }
  c->chunk_elems = ce;
  c->asked_SW = ce_asked / (uint32_t)kSweep;
  // The parts in which a ring is walked (Top-K messages; whole sends of more than 64 workers, or as stream_shape leaves them; the figures of whole sends
  // on fewer workers are from before that).  One workgroup per window and the whole ring, if that is enough of them for the 256 CUs; few windows are better walked in
  // parts, although the sends of the workers at their ends need a pass of their own.  What a part costs besides grows
  // with the windows, so a part has at least `fewest` workers, and there are no more than give `aim` workgroups (Top-K: of two
  // windows each).  Measured with parts of 1 to all workers, us a step, whole sends: perceptrons of 28 windows on 15 workers 16 in
  // parts of one, 24 in one part; of 102 on 24 25 in parts of two or three, 28 of eight, 35 in one; of 300 on 64 118 in
  // parts of 6, 8 or 11, 128 in one; ResNet-20 of 326 on 64 138 of 12, 161 in one, but on 15 36 in one part, 38 of eight.  Top-K
  // 10 %: 28 windows on 15 workers 47 and 78, 102 on 24 63 of three, 111 in one; 326 on 64 266 of 12, 331 in one; ResNet-18 of 574
  // windows on 24 157 in one part, 172 of eight, on 64 342 of 12, 350 in one.  A compromise: a perceptron of 399 windows would be
  // walked in one part by 40 workers in 92 us (whole sends) where parts of eight take 100.
  uint64_t fewest = 8, aim = 2048;
  bool one_part = windows >= 600 || P <= 5;
  if (!cfg->topk_ppm && windows < 250) {
    fewest = std::min<uint64_t>(8, windows / 40);
    aim = 1536;
  } else if (cfg->topk_ppm && windows < 250 && (P < 20 || windows < 110)) {
    fewest = windows / 50;
    aim = 768;
  }
  one_part |= cfg->topk_ppm ? windows >= 390 && 16ull * P <= windows : windows >= 110 && P < 16;
  const uint64_t parts = one_part ? 1 : std::min((aim + windows - 1) / windows, std::max<uint64_t>(1, P / std::max<uint64_t>(1, fewest)));
  c->part = one_shot ? P : (uint32_t)((P + parts - 1) / parts);
  // A mailbox equals its sender's xhat wherever a message has arrived, unless messages are under way (delay).  Where xhat is
  // reset at events the walk reads the mailboxes, and does not know of messages applied ahead at the ends of parts.
  c->walk = !c->cached && !one_shot && !cfg->delivery_delay && !(cfg->xhat_reset && cfg->topk_ppm && parts > 1);
  const uint64_t C = chunks.size();
  if ((uint64_t)P * C * (SW + 1) > 0xFFFFFFF0ull || (uint64_t)P * ktot > 0xFFFFFFF0ull) {
    delete c;
    return fail(EVG_ERR_INVALID, "configuration too large: work lists and message slots are indexed with 32 bits");
  }
  const uint64_t S = (uint64_t)P * L;

  // ---- device tables ------------------------------------------------------
  Tables& t = c->t;
  t.P = P; t.L = L; t.C = (uint32_t)C; t.S = (uint32_t)S;
  t.SW = SW;
  t.fine = fine;
  for (const LayerDesc& d : layers) c->most_sums = std::max(c->most_sums, d.nchunks * SW * fine);
  t.hist_len = hist_len;
  t.Ktot = (uint32_t)ktot;
  t.Npad = Npad;
  t.stage_stride = Npad / 16 * 4;
  for (size_t i = 0; i < 2; ++i) t.long_layer[i] = i < long_layers.size() ? long_layers[i] : kNoLayer;
  t.x = cfg->x; t.xhat = cfg->xhat; t.mbox_l = cfg->mbox_l; t.mbox_r = cfg->mbox_r; t.vel = cfg->vel;
  int dev = 0;
  ChunkDesc* d_chunks = nullptr;
  LayerDesc* d_layers = nullptr;
#define TRY_OR_FREE(expr)              \
  do {                                 \
    evg_status s_ = (expr);            \
    if (s_ != EVG_OK) {                \
      evg_destroy(c);                  \
      return s_;                       \
    }                                  \
  } while (0)
#define HIP_OR_FREE(expr)                                                            \
  do {                                                                               \
    hipError_t e_ = (expr);                                                          \
    if (e_ != hipSuccess) {                                                          \
      evg_destroy(c);                                                                \
      return fail(EVG_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_));              \
    }                                                                                \
  } while (0)
  HIP_OR_FREE(hipGetDevice(&dev));
  if (use_scratch) {
    uint64_t plain_C = 0;
    for (uint64_t n : c->numel) plain_C += (n + ce_asked - 1) / ce_asked;
    need = std::max(need, admitted_bytes(P, L, plain_C, c->asked_SW, hist_len, Npad, ktot, cfg->topk_ppm,
                                         cfg->trigger_kind == EVG_TRIGGER_NORM_DIFF, pull && !cfg->topk_ppm, sets_counted));
    if (need > kScratchBytes) {
      evg_destroy(c);
      return fail(EVG_ERR_INVALID, "this configuration needs %llu bytes of tables; the static scratch block "
                  "holds %llu (use evg_init)", (unsigned long long)need, (unsigned long long)kScratchBytes);
    }
    if (dev < 0 || dev >= kMaxDevices) {
      evg_destroy(c);
      return fail(EVG_ERR_INVALID, "device %d is beyond the %d devices evg_init_static keeps track of", dev, kMaxDevices);
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_base[dev]) {
      // once per device, with that device current: where this GPU's copy of the array lives
      void* base = nullptr;
      hipError_t e = hipGetSymbolAddress(&base, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !base) {
        delete c;
        return fail(EVG_ERR_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
      }
      g_scratch_base[dev] = static_cast<unsigned char*>(base);
    }
    if (g_scratch_user[dev]) {
      delete c;
      return fail(EVG_ERR_STATE, "the static scratch block of device %d is in use by another context: "
                  "destroy that context first", dev);
    }
    g_scratch_user[dev] = c;
    c->arena_base = g_scratch_base[dev];
    c->arena_dev = dev;
  }
  TRY_OR_FREE(c->dalloc(&d_chunks, C, false));
  TRY_OR_FREE(c->dalloc(&d_layers, L, false));
  HIP_OR_FREE(hipMemcpyAsync(d_chunks, chunks.data(), C * sizeof(ChunkDesc), hipMemcpyHostToDevice, c->stream));
  HIP_OR_FREE(hipMemcpyAsync(d_layers, layers.data(), L * sizeof(LayerDesc), hipMemcpyHostToDevice, c->stream));
  t.chunks = d_chunks;
  t.layers = d_layers;
  TRY_OR_FREE(c->dalloc(&t.partials, P * C * t.SW * fine, true));
  if (cfg->trigger_kind == EVG_TRIGGER_NORM_DIFF) {
    TRY_OR_FREE(c->dalloc(&t.partials_hat, P * C * t.SW * fine, true));
    TRY_OR_FREE(c->dalloc(&t.xhat_sq, S, true));
  }
  TRY_OR_FREE(c->dalloc(&t.delta, S, false));
  TRY_OR_FREE(c->dalloc(&t.last_norm, S, true));
  TRY_OR_FREE(c->dalloc(&t.delta_before, S, true));
  TRY_OR_FREE(c->dalloc(&t.last_event, S, false));
  TRY_OR_FREE(c->dalloc(&t.valid_l, (S + 3) / 4 * 4, true));
  TRY_OR_FREE(c->dalloc(&t.valid_r, (S + 3) / 4 * 4, true));
  TRY_OR_FREE(c->dalloc(&t.fired, (S + 3) / 4 * 4, true));
  TRY_OR_FREE(c->dalloc(&t.near_tie, S, true));
  TRY_OR_FREE(c->dalloc(&t.ev_full, S, true));
  TRY_OR_FREE(c->dalloc(&t.ev_topk, S, true));
  TRY_OR_FREE(c->dalloc(&t.near_cnt, S, true));
  TRY_OR_FREE(c->dalloc(&t.nonfinite_cnt, S, true));
  TRY_OR_FREE(c->dalloc(&t.slope_hist, S * t.hist_len, true));
  TRY_OR_FREE(c->dalloc(&t.slope_cnt, S, true));
  TRY_OR_FREE(c->dalloc(&t.not_staged, 1, true));
  TRY_OR_FREE(c->dalloc(&t.it, 1, true));
  {
    // decay^k as evg_step computes it, for the steps that take k from the device
    std::vector<double> tab(kDecayTable);
    for (uint32_t k = 0; k < kDecayTable; ++k) tab[k] = std::pow(cfg->synth.decay, (double)k);
    double* d_tab = nullptr;
    TRY_OR_FREE(c->dalloc(&d_tab, kDecayTable, false));
    HIP_OR_FREE(hipMemcpy(d_tab, tab.data(), kDecayTable * sizeof(double), hipMemcpyHostToDevice));
    t.decay_tab = d_tab;
    t.decay_len = kDecayTable;
  }
  // cache-resident ring, whole tensors, same-iteration delivery: the update pass fetches the sends
  // itself from a copy of x it keeps (one more array of the ring's size, library-owned)
  if (pull && !(in_parts && ring_part == P)) TRY_OR_FREE(c->dalloc(&t.xsnap, 2 * (uint64_t)P * Npad, false));
  std::vector<WindowDesc> ring;
  std::vector<ChooseDesc> by_size;
  if (in_parts || one_shot) {
    const uint32_t length = groups ? 256 * groups : kSweep, sums = SW * fine, step = groups ? groups * fine / kGroupSums : 1;
    for (size_t i = 0; i < chunks.size(); ++i)
      for (uint32_t u = 0; u * length < chunks[i].lead + chunks[i].len; ++u) {
        const ChunkDesc& cd = chunks[i];
        const LayerDesc& d = layers[cd.layer];
        const uint32_t first = u ? u * length - cd.lead : 0u, end = std::min<uint32_t>(cd.len, (u + 1) * length - cd.lead);
        ring.push_back({cd.off + first, end - first, cd.layer, cd.j0 + first,
                        (uint32_t)i * sums + u * step, d.chunk0 * sums, d.nchunks * sums, i == d.chunk0 && u == 0 ? 1u : 0u, d.sig_base,
                        d.numel, d.K, d.msg_off, 0u});
      }
    WindowDesc* d_ring = nullptr;
    TRY_OR_FREE(c->dalloc(&d_ring, ring.size(), false));
    HIP_OR_FREE(hipMemcpyAsync(d_ring, ring.data(), ring.size() * sizeof(WindowDesc), hipMemcpyHostToDevice, c->stream));
    c->parts.windows = d_ring;
    c->parts.count = (uint32_t)ring.size();
    c->parts.groups = groups;
    c->parts.quads = quads;
    if (in_parts) c->part = ring_part;
    c->parts.set[0] = c->parts.set[1] = {t.partials, t.xhat_sq, t.delta, t.last_event};
  }
  if (one_launch) {
    TRY_OR_FREE(c->dalloc(&c->parts.clocks, ring.size() * ((P + ring_part - 1) / ring_part), true));
    PartTables::Set& other = c->parts.set[1];
    TRY_OR_FREE(c->dalloc(&other.partials, P * C * t.SW * fine, true));
    TRY_OR_FREE(c->dalloc(&other.delta, S, true));
    TRY_OR_FREE(c->dalloc(&other.last_event, S, true));
    if (cfg->trigger_kind == EVG_TRIGGER_NORM_DIFF) TRY_OR_FREE(c->dalloc(&other.xhat_sq, S, true));
    c->one_launch = true;
  }
  // a step writes where it reads, unless it is a single-launch step (enqueue_step)
  t.partials_out = t.partials; t.partials_hat_out = t.partials_hat; t.xhat_sq_out = t.xhat_sq;
  t.delta_out = t.delta; t.last_event_out = t.last_event;
  if (cfg->topk_ppm) {
    TRY_OR_FREE(c->dalloc(&t.hist, c->hists() * kHistBins, true));
    TRY_OR_FREE(c->dalloc(&t.sel_prefix, S, true));
    TRY_OR_FREE(c->dalloc(&t.sel_krem, S, true));
    TRY_OR_FREE(c->dalloc(&t.sel_cut, S, true));
    TRY_OR_FREE(c->dalloc(&t.stage_n, P * C, true));
    TRY_OR_FREE(c->dalloc(&t.stage_key, (uint64_t)P * t.stage_stride, false));
    TRY_OR_FREE(c->dalloc(&t.group, P * C * t.SW * 4, true));
    TRY_OR_FREE(c->dalloc(&t.chunk_cnt, P * C, true));
    TRY_OR_FREE(c->dalloc(&t.chunk_before, P * C, true));
    TRY_OR_FREE(c->dalloc(&t.msg_idx, (uint64_t)P * ktot, true));
    TRY_OR_FREE(c->dalloc(&t.msg_val, (uint64_t)P * ktot, true));
    TRY_OR_FREE(c->dalloc(&t.sel_left, S, true));
    // Cached rings that put their messages ahead or late and have short tensors only count their keys by the upper 11 bits: finer bins about the
    // threshold cost the update pass more than they save with a tensor's few keys (64 ResNet-18 workers of width 8 223 -> 213 us a step, given
    // gradients 211 -> 208; of perceptrons of 159 000 elements 122 -> 129).
    if (cfg->norm_mode == EVG_NORM_FUSED && (pull || !c->cached || !long_layers.empty())) {
      TRY_OR_FREE(c->dalloc(&t.anchor, S, false));
      HIP_OR_FREE(hipMemsetAsync(t.anchor, 0xFF, S * 4, c->stream));      // kNoAnchor
    }
    // (cached rings that make their selections in many launches read x and xhat as fast)
    if (codes && (choose || !c->cached)) TRY_OR_FREE(c->dalloc(&t.codes, (uint64_t)P * Npad + 16, true));
    if (choose) {
      for (uint32_t l = 0; l < L; ++l) {
        const LayerDesc& d = layers[l];
        by_size.push_back({l, d.off, d.numel, d.K, d.chunk0, d.nchunks, d.chunk0 * SW * fine, d.nchunks * SW * fine});
      }
      std::stable_sort(by_size.begin(), by_size.end(), [&](const ChooseDesc& a, const ChooseDesc& b) { return a.numel > b.numel; });
      ChooseDesc* d_by_size = nullptr;
      TRY_OR_FREE(c->dalloc(&d_by_size, L, false));
      HIP_OR_FREE(hipMemcpyAsync(d_by_size, by_size.data(), L * sizeof(ChooseDesc), hipMemcpyHostToDevice, c->stream));
      c->choose.tensors = d_by_size;
      c->choose.longest = longest;
      for (const LayerDesc& d : layers) c->choose.longer += d.numel > 256;
    }
    TRY_OR_FREE(c->dalloc(&t.idx_hash, S, true));
    TRY_OR_FREE(c->dalloc(&t.msg_hash, S, true));
  }
  // nothing sent yet: xhat = x, khat = -1, delta = its starting value, v = 0
  const float d0 = cfg->thr_mode == EVG_THR_FIXED ? cfg->thr_fixed : cfg->delta_init;
  std::vector<float> dinit(S, d0);
  HIP_OR_FREE(hipMemcpyAsync(t.delta, dinit.data(), S * sizeof(float), hipMemcpyHostToDevice, c->stream));
  HIP_OR_FREE(hipMemsetAsync(t.last_event, 0xFF, S * sizeof(int32_t), c->stream));
  HIP_OR_FREE(hipMemcpyAsync(t.xhat, t.x, arena_bytes, hipMemcpyDeviceToDevice, c->stream));
  if (t.xsnap) {     // step 1 reads copy 0; both are set so that either parity finds x
    HIP_OR_FREE(hipMemcpyAsync(t.xsnap, t.x, arena_bytes, hipMemcpyDeviceToDevice, c->stream));
    HIP_OR_FREE(hipMemcpyAsync(t.xsnap + (uint64_t)P * Npad, t.x, arena_bytes, hipMemcpyDeviceToDevice, c->stream));
  }
  HIP_OR_FREE(hipMemsetAsync(t.vel, 0, arena_bytes, c->stream));
  HIP_OR_FREE(launch_norm(t, cfg->trigger_kind == EVG_TRIGGER_NORM_DIFF, c->stream));
  HIP_OR_FREE(hipStreamSynchronize(c->stream));   // host staging buffers above go out of scope
#undef TRY_OR_FREE
#undef HIP_OR_FREE
  *out = c;
  return EVG_OK;
}

evg_status evg_init(evg_ctx** out, const evg_config* cfg, void* hip_stream) {
  return init_common(out, cfg, hip_stream, false);
}

evg_status evg_init_static(evg_ctx** out, const evg_config* cfg, void* hip_stream) {
  return init_common(out, cfg, hip_stream, true);
}

// Single-launch rings: c->t names the set that the next step reads.
static void use_set(evg_ctx* c) {
  if (!c->one_launch) return;
  Tables& t = c->t;
  const PartTables::Set& now = c->parts.set[c->iters & 1];
  t.partials = t.partials_out = now.partials;
  t.xhat_sq = t.xhat_sq_out = now.xhat_sq;
  t.delta = t.delta_out = now.delta;
  t.last_event = t.last_event_out = now.last_event;
}

// Brings iters / last_iter up to date with the device after replayable steps.
static evg_status refresh_iteration(evg_ctx* c) {
  if (!c->device_ahead) return EVG_OK;
  HIP_TRY(hipStreamSynchronize(c->stream));
  IterState it{};
  HIP_TRY(hipMemcpy(&it, c->t.it, sizeof it, hipMemcpyDeviceToHost));
  if (it.overflow)
    return fail(EVG_ERR_STATE, "evg_step_next ran past iteration %u, the end of its decay table", kDecayTable - 1);
  c->iters = it.iters;
  c->last_iter = (int64_t)it.k_next - 1;
  use_set(c);
  return EVG_OK;
}

// The launch sequence of one iteration.  `timed`: bracket the phases with events.
static evg_status enqueue_step(evg_ctx* c, const StepArgs& args, bool timed) {
  const evg_config& g = c->cfg;
  Tables t = c->t;
  StepArgs a = args;
  const bool fused = g.norm_mode == EVG_NORM_FUSED;
  const bool norm_diff = g.trigger_kind == EVG_TRIGGER_NORM_DIFF;
  const bool was_timing = c->timing;
  c->timing = was_timing && timed;
  struct Restore { evg_ctx* c; bool v; ~Restore() { c->timing = v; } } restore{c, was_timing};
  evg_status st;
  // single launch: the update pass runs the trigger tests
  const bool single = c->one_launch && (a.from_device || !c->replayable_used);
  a.one_launch = single;
  a.step_no = (uint32_t)c->iters;
  if (c->one_launch) {
    const PartTables::Set& next = c->parts.set[(c->iters + 1) & 1];
    t.partials_out = next.partials;
    t.xhat_sq_out = next.xhat_sq; t.delta_out = next.delta; t.last_event_out = next.last_event;
  }
  if (!fused) {
    Phase ph(c, EVG_PH_NORM);
    HIP_TRY(launch_norm(t, norm_diff, c->stream));
    if ((st = ph.end()) != EVG_OK) return st;
  }
  if (!single) {
    Phase ph(c, EVG_PH_TRIGGER);
    HIP_TRY(a.choose       ? launch_topk_choose(t, a, c->choose, c->stream)
            : a.hist_fused ? launch_topk_decide(t, a, c->stream)
                           : launch_trigger(t, a, c->most_sums, c->stream));
    if ((st = ph.end()) != EVG_OK) return st;
  }
  // Whole sends: with delayed delivery the mailboxes are written after the update, a cache-resident ring's receivers
  // fetch them in the update pass, a Top-K ring's few ride in the selection's first kernel, and a walking pass has
  // them in registers -- but for the workers at the ends of the parts it is walked in.
  if (!a.topk_on && a.walk && a.part < t.P) {
    Phase ph(c, EVG_PH_SEND_FULL);
    HIP_TRY(launch_copy(t, a, c->chunk_elems, c->stream));
    if ((st = ph.end()) != EVG_OK) return st;
  }
  if (a.topk_on && !a.choose) {
    {
      Phase ph(c, EVG_PH_TOPK_SELECT);
      HIP_TRY(launch_topk_select(t, a, c->chunk_elems, c->stream));
      if ((st = ph.end()) != EVG_OK) return st;
    }
    if (a.applied || (a.walk && a.part < t.P)) {
      Phase ph(c, EVG_PH_TOPK_SEND);
      HIP_TRY(launch_topk_apply(t, a, c->chunk_elems, c->stream));
      if ((st = ph.end()) != EVG_OK) return st;
    }
  }
  {
    Phase ph(c, EVG_PH_UPDATE);
    const int norm = !fused ? 0 : !norm_diff ? 1 : g.topk_ppm ? 3 : 2;
    HIP_TRY(a.walk          ? launch_walk(t, a, g.synth.dist, g.grad_mode, norm, c->stream)
            : c->parts.groups ? launch_ring(t, a, c->parts, g.synth.dist, g.grad_mode, norm, c->stream)
            : c->parts.count ? launch_part(t, a, c->parts, g.synth.dist, g.grad_mode, norm, c->stream)
                            : launch_update(t, a, g.synth.dist, g.grad_mode, norm, c->stream));
    if ((st = ph.end()) != EVG_OK) return st;
  }
  if (a.delay) {
    Phase ph(c, EVG_PH_DELIVER);
    HIP_TRY(launch_deliver(t, c->chunk_elems, c->stream));
    if ((st = ph.end()) != EVG_OK) return st;
  }
  c->messages_live = true;
  return EVG_OK;
}

// Everything of StepArgs that does not depend on the iteration.
static evg_status fixed_args(evg_ctx* c, const float* grad, StepArgs* out) {
  const evg_config& g = c->cfg;
  if (g.grad_mode == EVG_GRAD_BUFFER) {
    if (!grad) return fail(EVG_ERR_INVALID, "grad_mode is EVG_GRAD_BUFFER but grad is NULL");
    if ((uintptr_t)grad % 16) return fail(EVG_ERR_ALIGN, "grad is not 16-byte aligned");
    evg_status gs = check_device_array(grad, (uint64_t)c->t.P * c->t.Npad * 4, "grad");
    if (gs != EVG_OK) return gs;
  }
  StepArgs a{};
  a.lr = g.lr;
  a.mu = g.momentum;
  a.plain_sgd = g.momentum == 0.0f ? 1u : 0u;
  a.thr_mode = g.thr_mode;
  a.horizon = g.horizon;
  a.force_first = g.force_first ? 1u : 0u;
  a.topk_on = g.topk_ppm ? 1u : 0u;
  a.topk_key = g.topk_key;
  a.delay = g.delivery_delay;
  a.hist_fused = (g.topk_ppm && g.norm_mode == EVG_NORM_FUSED) ? 1u : 0u;
  a.choose = c->choose.longest ? 1u : 0u;
  a.cached = c->cached ? 1u : 0u;
  a.pull = c->t.xsnap ? 1u : 0u;
  a.walk = c->walk ? 1u : 0u;
  a.part = c->part;
  a.applied = (g.topk_ppm && !g.delivery_delay && !a.walk && !a.pull) ? 1u : 0u;
  a.xhat_reset = (g.xhat_reset && g.topk_ppm) ? 1u : 0u;
  const bool norm_diff = g.trigger_kind == EVG_TRIGGER_NORM_DIFF;
  // fused + whole-tensor sends: xhat's norm is a scalar per tensor and xhat is never read
  a.norm_src = !norm_diff ? 0u : (g.norm_mode == EVG_NORM_FUSED && !g.topk_ppm) ? 1u : 2u;
  a.key0 = (uint32_t)g.synth.seed;
  a.key1 = (uint32_t)(g.synth.seed >> 32);
  a.spike_prob = g.synth.spike_prob;
  a.spike_gain = g.synth.spike_gain;
  a.grad = grad;
  *out = a;
  return EVG_OK;
}

evg_status evg_step(evg_ctx* c, uint64_t iter, const float* grad) {
  if (!c) return fail(EVG_ERR_INVALID, "context is NULL");
  evg_status st = refresh_iteration(c);
  if (st != EVG_OK) return st;
  if ((int64_t)iter <= c->last_iter || iter >= 0x7FFFFFFFull)
    return fail(EVG_ERR_STATE, "iteration %llu does not follow %lld", (unsigned long long)iter,
                (long long)c->last_iter);
  StepArgs a{};
  if ((st = fixed_args(c, grad, &a)) != EVG_OK) return st;
  a.k = (uint32_t)iter;
  a.decay_pow = std::pow(c->cfg.synth.decay, (double)iter);
  if (c->timing && c->pending.size() > 4096 && (st = c->drain_timers()) != EVG_OK) return st;
  if ((st = enqueue_step(c, a, true)) != EVG_OK) return st;
  c->last_iter = (int64_t)iter;
  c->iters += 1;
  use_set(c);
  return EVG_OK;
}

evg_status evg_step_next(evg_ctx* c, const float* grad) {
  if (!c) return fail(EVG_ERR_INVALID, "context is NULL");
  StepArgs a{};
  evg_status st = fixed_args(c, grad, &a);
  if (st != EVG_OK) return st;
  a.from_device = 1;
  c->replayable_used = true;
  if ((st = enqueue_step(c, a, false)) != EVG_OK) return st;
  c->device_ahead = true;
  return EVG_OK;
}

evg_status evg_stats(evg_ctx* c, evg_stats_t* out) {
  if (!c || !out) return fail(EVG_ERR_INVALID, "context and out must be non-NULL");
  const Tables& t = c->t;
  const size_t S = t.S;
  HIP_TRY(hipStreamSynchronize(c->stream));
  evg_status rs = refresh_iteration(c);
  if (rs != EVG_OK) return rs;
  std::vector<uint32_t> ef(S), et(S), nt(S), nf(S);
  HIP_TRY(hipMemcpy(ef.data(), t.ev_full, S * 4, hipMemcpyDeviceToHost));
  HIP_TRY(hipMemcpy(et.data(), t.ev_topk, S * 4, hipMemcpyDeviceToHost));
  HIP_TRY(hipMemcpy(nt.data(), t.near_cnt, S * 4, hipMemcpyDeviceToHost));
  HIP_TRY(hipMemcpy(nf.data(), t.nonfinite_cnt, S * 4, hipMemcpyDeviceToHost));
  if (out->last_norm) HIP_TRY(hipMemcpy(out->last_norm, t.last_norm, S * 4, hipMemcpyDeviceToHost));
  if (out->delta) HIP_TRY(hipMemcpy(out->delta, t.delta, S * 4, hipMemcpyDeviceToHost));
  if (out->last_event_iter) HIP_TRY(hipMemcpy(out->last_event_iter, t.last_event, S * 4, hipMemcpyDeviceToHost));
  if (out->valid_l) HIP_TRY(hipMemcpy(out->valid_l, t.valid_l, S, hipMemcpyDeviceToHost));
  if (out->valid_r) HIP_TRY(hipMemcpy(out->valid_r, t.valid_r, S, hipMemcpyDeviceToHost));
  if (out->events_full_rl) std::memcpy(out->events_full_rl, ef.data(), S * 4);
  if (out->events_topk_rl) std::memcpy(out->events_topk_rl, et.data(), S * 4);
  uint64_t e_full = 0, e_topk = 0, vw = 0, iw = 0, near = 0, nonf = 0;
  for (uint32_t r = 0; r < t.P; ++r)
    for (uint32_t l = 0; l < t.L; ++l) {
      const size_t s = (size_t)r * t.L + l;
      e_full += ef[s];
      e_topk += et[s];
      vw += (uint64_t)ef[s] * c->numel[l] + (uint64_t)et[s] * c->K[l];
      iw += (uint64_t)et[s] * c->K[l];
      near += nt[s];
      nonf += nf[s];
    }
  out->iters = c->iters;
  out->events_full = e_full;
  out->events_topk = e_topk;
  out->events_total = e_full + e_topk;
  out->value_words = vw;
  out->index_words = iw;
  out->bytes_sent = 2ull * 4ull * (vw + iw);
  out->regular_events = (uint64_t)t.P * t.L * c->iters;
  out->regular_words = (uint64_t)t.P * c->N * c->iters;
  out->near_tie_flags = near;
  out->nonfinite_norms = nonf;
  uint32_t not_staged = 0;
  HIP_TRY(hipMemcpy(&not_staged, t.not_staged, 4, hipMemcpyDeviceToHost));
  out->chunks_not_staged = not_staged;
  out->library_bytes = c->owned_bytes;
  return EVG_OK;
}

evg_status evg_update_pass(evg_ctx* c, uint32_t* pass, uint32_t* workers, uint32_t* elements) {
  if (!c) return fail(EVG_ERR_INVALID, "context is NULL");
  const uint32_t which = c->walk ? EVG_PASS_WALK : c->parts.groups ? EVG_PASS_RING : c->parts.count ? EVG_PASS_PART : EVG_PASS_CHUNK;
  if (pass) *pass = which;
  if (workers) *workers = which == EVG_PASS_CHUNK ? 1 : c->part;
  if (elements) *elements = which == EVG_PASS_RING ? 256 * c->parts.groups : which == EVG_PASS_PART ? (uint32_t)kSweep : 0;
  return EVG_OK;
}

evg_status evg_last_decisions(evg_ctx* c, uint8_t* fired, uint8_t* near_tie, float* norm, float* delta_before) {
  if (!c) return fail(EVG_ERR_INVALID, "context is NULL");
  const Tables& t = c->t;
  HIP_TRY(hipStreamSynchronize(c->stream));
  if (fired) HIP_TRY(hipMemcpy(fired, t.fired, t.S, hipMemcpyDeviceToHost));
  if (near_tie) HIP_TRY(hipMemcpy(near_tie, t.near_tie, t.S, hipMemcpyDeviceToHost));
  if (norm) HIP_TRY(hipMemcpy(norm, t.last_norm, t.S * 4, hipMemcpyDeviceToHost));
  if (delta_before) HIP_TRY(hipMemcpy(delta_before, t.delta_before, t.S * 4, hipMemcpyDeviceToHost));
  return EVG_OK;
}

evg_status evg_message(evg_ctx* c, uint32_t r, uint32_t l, uint32_t* idx, float* val, uint64_t cap,
                       uint64_t* count) {
  if (!c || !count) return fail(EVG_ERR_INVALID, "context and count must be non-NULL");
  const Tables& t = c->t;
  if (r >= t.P || l >= t.L) return fail(EVG_ERR_INVALID, "no worker %u / tensor %u", r, l);
  HIP_TRY(hipStreamSynchronize(c->stream));
  uint8_t code = 0;
  HIP_TRY(hipMemcpy(&code, t.fired + (size_t)r * t.L + l, 1, hipMemcpyDeviceToHost));
  uint32_t threshold = 0;
  if (code == 2 && c->cfg.topk_ppm)
    HIP_TRY(hipMemcpy(&threshold, t.sel_prefix + (size_t)r * t.L + l, 4, hipMemcpyDeviceToHost));
  if (code != 2 || !c->cfg.topk_ppm || !c->messages_live || threshold == kNoThreshold) {
    *count = 0;
    return EVG_OK;
  }
  const uint64_t K = c->K[l];
  const size_t base = (size_t)r * t.Ktot + c->msg_off[l];
  if (!t.codes) {
    const uint64_t n = K < cap ? K : cap;
    if (idx && n) HIP_TRY(hipMemcpy(idx, t.msg_idx + base, n * 4, hipMemcpyDeviceToHost));
    if (val && n) HIP_TRY(hipMemcpy(val, t.msg_val + base, n * 4, hipMemcpyDeviceToHost));
    *count = K;
    return EVG_OK;
  }
  // where keys are counted by their codes, places of a message that nothing was sent for are left out
  constexpr uint64_t kBlock = 1 << 16;
  std::unique_ptr<uint32_t[]> at(new (std::nothrow) uint32_t[kBlock]);
  std::unique_ptr<float[]> values(new (std::nothrow) float[kBlock]);
  if (!at || !values) return fail(EVG_ERR_OOM, "host allocation failed");
  uint64_t n = 0;
  for (uint64_t i0 = 0; i0 < K; i0 += kBlock) {
    const uint64_t m = std::min(kBlock, K - i0);
    HIP_TRY(hipMemcpy(at.get(), t.msg_idx + base + i0, m * 4, hipMemcpyDeviceToHost));
    if (val && n < cap) HIP_TRY(hipMemcpy(values.get(), t.msg_val + base + i0, m * 4, hipMemcpyDeviceToHost));
    for (uint64_t i = 0; i < m; ++i) {
      if (at[i] == kNoEntry) continue;
      if (idx && n < cap) idx[n] = at[i];
      if (val && n < cap) val[n] = values[i];
      ++n;
    }
  }
  *count = n;
  return EVG_OK;
}

evg_status evg_message_hashes(evg_ctx* c, uint64_t* idx_hash, uint64_t* msg_hash) {
  if (!c) return fail(EVG_ERR_INVALID, "context is NULL");
  const Tables& t = c->t;
  const bool live = c->cfg.topk_ppm && c->messages_live;
  if (live) HIP_TRY(launch_message_hashes(t, c->stream));    // from the message buffers of the last step
  HIP_TRY(hipStreamSynchronize(c->stream));
  if (idx_hash) {
    if (live) HIP_TRY(hipMemcpy(idx_hash, t.idx_hash, (size_t)t.S * 8, hipMemcpyDeviceToHost));
    else std::memset(idx_hash, 0, (size_t)t.S * 8);
  }
  if (msg_hash) {
    if (live) HIP_TRY(hipMemcpy(msg_hash, t.msg_hash, (size_t)t.S * 8, hipMemcpyDeviceToHost));
    else std::memset(msg_hash, 0, (size_t)t.S * 8);
  }
  return EVG_OK;
}

evg_status evg_average(evg_ctx* c, float* out) {
  if (!c || !out) return fail(EVG_ERR_INVALID, "context and out must be non-NULL");
  if ((uintptr_t)out % 16) return fail(EVG_ERR_ALIGN, "out is not 16-byte aligned");
  evg_status st = check_device_array(out, c->t.Npad * 4, "out");
  if (st != EVG_OK) return st;
  HIP_TRY(launch_average(c->t, out, c->stream));
  return EVG_OK;
}

}  // extern "C"

namespace {

struct StateHeader {
  char magic[8];
  uint32_t version, P, L, C, SW, S, hist_len, topk_ppm, trigger_kind, norm_mode, thr_mode, pad;
  uint64_t Npad, iters;
  int64_t last_iter;
};

constexpr uint32_t kCutOnLines = 1u << 16, kCutFiner = 1u << 17;   // StateHeader::pad, from version 5 on

struct Piece { void* dev; size_t bytes; };

// Every library-owned array a later step reads before writing it.
std::vector<Piece> state_pieces(evg_ctx* c) {
  const Tables& t = c->t;
  const size_t S = t.S, sweeps = (size_t)t.P * t.C * t.SW;
  std::vector<Piece> v = {
      {t.delta, S * 4}, {t.last_norm, S * 4}, {t.delta_before, S * 4}, {t.last_event, S * 4},
      {t.valid_l, S}, {t.valid_r, S}, {t.fired, S}, {t.near_tie, S},
      {t.ev_full, S * 4}, {t.ev_topk, S * 4}, {t.near_cnt, S * 4}, {t.nonfinite_cnt, S * 4},
      {t.slope_hist, S * t.hist_len * 4}, {t.slope_cnt, S * 4}, {t.partials, sweeps * 8},
      {t.it, sizeof(IterState)}, {t.not_staged, sizeof(uint32_t)}};
  if (t.partials_hat) { v.push_back({t.partials_hat, sweeps * 8}); v.push_back({t.xhat_sq, S * 8}); }
  if (t.hist) v.push_back({t.hist, S * kHistBins * 4});
  return v;
}

// Does the update pass count the keys of the next selection?
bool carries_keys(const evg_ctx* c) { return c->cfg.topk_ppm && c->cfg.norm_mode == EVG_NORM_FUSED; }

StateHeader state_header(evg_ctx* c) {
  StateHeader h{};
  std::memcpy(h.magic, "EVGSTATE", 8);
  h.version = 6;
  h.P = c->t.P; h.L = c->t.L; h.C = c->t.C; h.SW = c->t.SW; h.S = c->t.S;
  h.hist_len = c->t.hist_len;
  h.topk_ppm = c->cfg.topk_ppm;
  h.trigger_kind = c->cfg.trigger_kind;
  h.norm_mode = c->cfg.norm_mode;
  h.thr_mode = c->cfg.thr_mode;
  h.pad = c->cfg.delivery_delay | (c->cfg.xhat_reset << 8) | (c->on_lines ? kCutOnLines : 0u) |
          (c->t.SW != c->asked_SW ? kCutFiner : 0u);
  h.Npad = c->t.Npad;
  h.iters = c->iters;
  h.last_iter = c->last_iter;
  return h;
}

}  // namespace

extern "C" {

uint64_t evg_state_size(evg_ctx* c) {
  if (!c) return 0;
  uint64_t n = sizeof(StateHeader);
  for (const Piece& p : state_pieces(c)) n += p.bytes;
  return n;
}

evg_status evg_state_export(evg_ctx* c, void* blob, uint64_t capacity) {
  if (!c || !blob) return fail(EVG_ERR_INVALID, "context and blob must be non-NULL");
  if (capacity < evg_state_size(c))
    return fail(EVG_ERR_INVALID, "blob holds %llu bytes, %llu needed", (unsigned long long)capacity,
                (unsigned long long)evg_state_size(c));
  HIP_TRY(hipStreamSynchronize(c->stream));
  evg_status rs = refresh_iteration(c);
  if (rs != EVG_OK) return rs;
  const StateHeader h = state_header(c);
  char* out = static_cast<char*>(blob);
  std::memcpy(out, &h, sizeof h);
  out += sizeof h;
  const Tables& t = c->t;
  for (const Piece& p : state_pieces(c)) {
    if (t.fine > 1 && (p.dev == t.partials || p.dev == t.partials_hat)) {      // blobs hold a sum a sweep, added as every test adds it (SweepSums)
      const size_t sweeps = p.bytes / 8;
      std::unique_ptr<double[]> parts(new (std::nothrow) double[sweeps * t.fine]);
      if (!parts) return fail(EVG_ERR_OOM, "host allocation failed");
      HIP_TRY(hipMemcpy(parts.get(), p.dev, p.bytes * t.fine, hipMemcpyDeviceToHost));
      for (size_t i = 0; i < sweeps; ++i, out += 8) {
        double sum = 0.0;
        for (uint32_t u = 0; u < t.fine; ++u) sum += parts[i * t.fine + u];
        std::memcpy(out, &sum, 8);
      }
      continue;
    }
    HIP_TRY(hipMemcpy(out, p.dev, p.bytes, hipMemcpyDeviceToHost));
    out += p.bytes;
  }
  if (carries_keys(c)) {       // (see evg_state_import)
    std::unique_ptr<uint32_t[]> anchors(new (std::nothrow) uint32_t[c->t.S]);
    if (!anchors) return fail(EVG_ERR_OOM, "host allocation failed");
    std::fill_n(anchors.get(), c->t.S, kNoAnchor);
    if (c->t.anchor) HIP_TRY(hipMemcpy(anchors.get(), c->t.anchor, (size_t)c->t.S * 4, hipMemcpyDeviceToHost));
    char* hists = out - (size_t)c->t.S * kHistBins * 4;
    for (size_t i = 0; i < c->t.S; ++i) if (anchors[i] != kNoAnchor) anchors[i] &= kAnchorBits;      // (an import makes the codes)
    for (size_t i = 0; i < c->t.S; ++i) std::memcpy(hists + (i * kHistBins + kHistBins - 1) * 4, &anchors[i], 4);
  }
  return EVG_OK;
}

evg_status evg_state_import(evg_ctx* c, const void* blob, uint64_t size) {
  if (!c || !blob) return fail(EVG_ERR_INVALID, "context and blob must be non-NULL");
  // A tensor's sums are only ever added up, so a blob serves however its ring cut the tensors: at their own starts or on cache
  // lines, or into shorter chunks than were asked for.  A tensor's sums in chunks of SW sweeps:
  const Tables& t = c->t;
  const size_t L = c->numel.size();
  auto sums_of = [&](size_t l, uint64_t off, uint64_t SW, bool on_lines) {
    const uint64_t granule = SW * kSweep;
    return (c->numel[l] + (on_lines ? off % kLineElems : 0) + granule - 1) / granule * SW;
  };
  StateHeader got;
  if (size < sizeof got) return fail(EVG_ERR_INVALID, "blob size does not match this configuration");
  std::memcpy(&got, blob, sizeof got);
  const uint32_t flags = got.version > 4 ? got.pad & (kCutOnLines | kCutFiner) : 0u;
  if (got.SW != t.SW && !(flags & kCutFiner && got.SW == 1) && got.SW != c->asked_SW)
    return fail(EVG_ERR_INVALID, "blob was exported from a different configuration or version");
  uint64_t plain = 0, lines = 0, off = 0;        // sums per worker
  for (size_t l = 0; l < L; ++l) {
    plain += sums_of(l, off, got.SW, false);
    lines += sums_of(l, off, got.SW, true);
    off += pad_to(c->numel[l], 4);
  }
  const uint64_t here = (uint64_t)t.C * t.SW, there = (uint64_t)got.C * got.SW;
  // (a pass in parts writes no sum where a chunk has no window, so what another ring has there is moved in any case)
  const bool same_cut = got.C == t.C && got.SW == t.SW && !c->parts.count, from_lines = there != plain;
  const bool maybe_lines = got.version == 4 || (flags & kCutOnLines);     // (version 4 does not say)
  if (there != plain && !(maybe_lines && there == lines))
    return fail(EVG_ERR_INVALID, "blob was exported from a different configuration or version");
  // version 3 has three more words, lengths of lists that are no longer kept, ahead of the count of chunks not staged
  const uint64_t list_bytes = got.version == 3 ? 12 : 0, per_sum = (uint64_t)t.P * 8 * (t.partials_hat ? 2 : 1);
  if (size != evg_state_size(c) - here * per_sum + there * per_sum + list_bytes)
    return fail(EVG_ERR_INVALID, "blob size does not match this configuration");
  StateHeader want = state_header(c);
  want.C = got.C;
  want.SW = got.SW;
  if (got.version >= 3 && got.version < 6) want.version = got.version;
  want.pad = (want.pad & ~(kCutOnLines | kCutFiner)) | flags;
  want.iters = got.iters;
  want.last_iter = got.last_iter;
  if (std::memcmp(&got, &want, sizeof got) != 0)
    return fail(EVG_ERR_INVALID, "blob was exported from a different configuration or version");
  const size_t sum_count = (size_t)t.P * here * t.fine;
  std::unique_ptr<double[]> moved(same_cut ? nullptr : new (std::nothrow) double[sum_count]);
  if (!same_cut && !moved) return fail(EVG_ERR_OOM, "host allocation failed");
  const size_t clock_count = c->one_launch ? (size_t)c->parts.count * ((t.P + c->part - 1) / c->part) : 0;
  std::unique_ptr<PartClock[]> clocks(new (std::nothrow) PartClock[clock_count + 1]);
  if (!clocks) return fail(EVG_ERR_OOM, "host allocation failed");
  // anchors of key codes, if the exporter had any: in the last word of a tensor's saved histogram, from version 6 on
  std::unique_ptr<uint32_t[]> anchors(new (std::nothrow) uint32_t[t.S]);
  if (!anchors) return fail(EVG_ERR_OOM, "host allocation failed");
  const char* hists = static_cast<const char*>(blob) + size - (size_t)t.S * kHistBins * 4;      // (the last piece, if there is one)
  for (size_t i = 0; t.anchor && i < t.S; ++i) {
    anchors[i] = kNoAnchor;
    if (got.version >= 6) std::memcpy(&anchors[i], hists + (i * kHistBins + kHistBins - 1) * 4, 4);
  }
  std::fill_n(clocks.get(), clock_count, PartClock{(uint32_t)(got.last_iter + 1), (uint32_t)got.iters});
  c->iters = got.iters;
  c->last_iter = got.last_iter;
  use_set(c);
  // Everything goes through the context's stream, and is waited for: steps on a non-blocking stream do not wait for copies
  // on the default stream, and a copy from device to device does not make the host wait.
  const char* in = static_cast<const char*>(blob) + sizeof got;
  for (const Piece& p : state_pieces(c)) {
    if (p.dev == t.not_staged) in += list_bytes;
    if (!same_cut && (p.dev == t.partials || p.dev == t.partials_hat)) {
      // sums of the exporter's sweeps to the places of this ring's; what is beyond the last place in use here (a
      // streaming ring's passes never write there) joins the sum before
      double* to = moved.get();
      std::fill_n(to, sum_count, 0.0);
      for (uint32_t r = 0; r < t.P; ++r) {
        off = 0;
        for (size_t l = 0; l < L; ++l) {
          const uint64_t from = sums_of(l, off, got.SW, from_lines);
          const uint64_t used = (c->numel[l] + (c->on_lines ? off % kLineElems : 0) + kSweep - 1) / kSweep;
          for (uint64_t i = 0; i < from; ++i) {
            double v;
            std::memcpy(&v, in, 8);
            in += 8;
            to[std::min(i, used - 1) * t.fine] += v;
          }
          to += sums_of(l, off, t.SW, c->on_lines) * t.fine;
          off += pad_to(c->numel[l], 4);
        }
      }
      HIP_TRY(hipMemcpyAsync(p.dev, moved.get(), sum_count * 8, hipMemcpyHostToDevice, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));        // `moved` is filled again
      continue;
    }
    HIP_TRY(hipMemcpyAsync(p.dev, in, p.bytes, hipMemcpyHostToDevice, c->stream));
    in += p.bytes;
  }
  if (clock_count)
    HIP_TRY(hipMemcpyAsync(c->parts.clocks, clocks.get(), clock_count * sizeof(PartClock), hipMemcpyHostToDevice, c->stream));
  if (carries_keys(c)) {
    // Histograms and key codes are counted again, from the arenas: the saved ones have the exporter's bins.
    StepArgs a{};
    a.topk_key = c->cfg.topk_key;
    a.choose = c->choose.longest ? 1u : 0u;
    if (t.anchor) HIP_TRY(hipMemcpyAsync(t.anchor, anchors.get(), (size_t)t.S * 4, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipMemsetAsync(t.hist, 0, c->hists() * kHistBins * 4, c->stream));
    HIP_TRY(launch_topk_count_all(t, a, c->chunk_elems, c->stream));
  }
  // the library's copy of x follows the caller's arena, which holds the saved parameters again
  if (c->t.xsnap) {
    const size_t arena = (size_t)c->t.P * c->t.Npad;
    HIP_TRY(hipMemcpyAsync(c->t.xsnap, c->t.x, arena * 4, hipMemcpyDeviceToDevice, c->stream));
    HIP_TRY(hipMemcpyAsync(c->t.xsnap + arena, c->t.x, arena * 4, hipMemcpyDeviceToDevice, c->stream));
  }
  HIP_TRY(hipStreamSynchronize(c->stream));
  c->messages_live = false;         // message buffers are scratch and are not part of the blob
  return EVG_OK;
}

evg_status evg_timing(evg_ctx* c, int enable) {
  if (!c) return fail(EVG_ERR_INVALID, "context is NULL");
  evg_status st = c->drain_timers();
  if (st != EVG_OK) return st;
  for (int i = 0; i < EVG_PH_COUNT; ++i) { c->ms[i] = 0; c->samples[i] = 0; }
  c->timing = enable != 0;
  return EVG_OK;
}

evg_status evg_timing_read(evg_ctx* c, double ms_out[EVG_PH_COUNT], uint64_t samples_out[EVG_PH_COUNT]) {
  if (!c || !ms_out || !samples_out) return fail(EVG_ERR_INVALID, "NULL argument");
  evg_status st = c->drain_timers();
  if (st != EVG_OK) return st;
  for (int i = 0; i < EVG_PH_COUNT; ++i) { ms_out[i] = c->ms[i]; samples_out[i] = c->samples[i]; }
  return EVG_OK;
}

}  // extern "C"
