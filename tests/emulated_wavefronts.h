// A workgroup of a kernel, on the CPU: what the device code of csrc/ takes from HIP and the compiler, for a plain C++ compiler (clang).
// Every lane is a coroutine.  The lanes of a wavefront meet wherever one reads another's register; wavefronts meet at barriers only, and
// between two barriers they run in an order that the caller chooses (emu::Order).  What one of them writes to LDS without a barrier
// behind another's read of it therefore shows in the results, in one of the orders, each time.
#pragma once
#include <stdint.h>
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <new>
#include <vector>

#define __device__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(n)
typedef int hipError_t;
typedef void* hipStream_t;
struct float4 { float x, y, z, w; };
struct uint2 { uint32_t x, y; };
struct dim3 { uint32_t x = 1, y = 1, z = 1; };
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }

namespace emu {
enum class Order { kAscending, kDescending, kRandom };       // which wavefront goes on first
struct Lane { dim3 thread; ucontext_t at; bool done = false, in_barrier = false; };
struct Wave { uint32_t arrived = 0, round = 0; uint64_t value[2][64]; };
inline std::vector<Lane> lanes;
inline std::vector<Wave> waves;
inline Lane* now;
inline dim3 block_idx, grid_dim;
inline ucontext_t scheduler;
inline uint32_t in_barrier, barriers, live, arrivals;
inline uint32_t or_value[2];
inline std::function<void()> body;
inline std::vector<uint32_t> dynamic_lds;

inline void yield() { swapcontext(&now->at, &scheduler); }
inline uint32_t lane() { return now->thread.x & 63u; }
// The values that the wavefront's lanes have brought.
inline const uint64_t* meet(uint64_t v) {
  Wave& w = waves[now->thread.x >> 6];
  const uint32_t round = w.round;
  w.value[round & 1][lane()] = v;
  ++arrivals;
  if (++w.arrived == 64) {
    w.arrived = 0;
    ++w.round;
  } else {
    while (w.round == round) yield();
  }
  return w.value[round & 1];
}
inline void open_barrier() {
  in_barrier = 0;
  or_value[(barriers + 1) & 1] = 0;
  ++barriers;
  for (Lane& l : lanes) l.in_barrier = false;
}
inline bool barrier(bool mine) {
  const uint32_t which = barriers;
  or_value[which & 1] |= mine ? 1u : 0u;
  ++arrivals;
  if (++in_barrier == live) {
    open_barrier();
  } else {
    now->in_barrier = true;
    while (barriers == which) yield();
  }
  return or_value[which & 1] != 0;
}
inline void start() {
  body();
  now->done = true;
  ++arrivals;
  if (--live && in_barrier == live) open_barrier();          // the others wait for nobody else
}
// One workgroup of `threads`, a multiple of 64.
inline void run(uint32_t threads, Order order, uint32_t seed, std::function<void()> f) {
  constexpr size_t kStack = 96 << 10;
  static std::vector<unsigned char> stacks;
  stacks.resize(kStack * threads);
  lanes.assign(threads, Lane());
  waves.assign(threads / 64, Wave());
  body = std::move(f);
  live = threads;
  in_barrier = 0;
  or_value[0] = or_value[1] = 0;
  for (uint32_t t = 0; t < threads; ++t) {
    lanes[t].thread.x = t;
    getcontext(&lanes[t].at);
    lanes[t].at.uc_stack.ss_sp = stacks.data() + kStack * t;
    lanes[t].at.uc_stack.ss_size = kStack;
    lanes[t].at.uc_link = &scheduler;
    makecontext(&lanes[t].at, start, 0);
  }
  const uint32_t n = threads / 64;
  while (live) {
    // the first wavefront, in the order asked for, that is not waiting in a barrier: a turn of all its lanes
    uint32_t picked = n;
    const uint32_t first = order == Order::kRandom ? (seed = seed * 1664525u + 1013904223u) >> 8 : 0u;
    for (uint32_t i = 0; i < n && picked == n; ++i) {
      const uint32_t w = order == Order::kDescending ? n - 1 - i : (first + i) % n;
      for (uint32_t l = 0; l < 64; ++l)
        if (!lanes[w * 64 + l].done && !lanes[w * 64 + l].in_barrier) picked = w;
    }
    if (picked == n) {
      std::printf("all wavefronts wait\n");
      std::exit(1);
    }
    const uint32_t before = arrivals;
    for (uint32_t l = 0; l < 64; ++l) {
      now = &lanes[picked * 64 + l];
      if (!now->done) swapcontext(&scheduler, &now->at);
    }
    if (arrivals == before) {
      std::printf("the lanes of a wavefront do not meet\n");
      std::exit(1);
    }
  }
}

struct Buffer { char* at; uint32_t bytes; };
inline Buffer make_buffer(void* at, short, int bytes, int) { return {static_cast<char*>(at), (uint32_t)bytes}; }
template <typename V, int N>
inline V load(Buffer b, int byte) {
  V v;
  for (int i = 0; i < N; ++i) {
    uint32_t word = 0;
    const uint64_t o = (uint64_t)(uint32_t)byte + 4 * i;
    if (o + 4 <= b.bytes) std::memcpy(&word, b.at + o, 4);
    v[i] = word;
  }
  return v;
}
template <typename V, int N>
inline void store(const V& v, Buffer b, int byte) {
  for (int i = 0; i < N; ++i) {
    uint32_t word;
    std::memcpy(&word, reinterpret_cast<const char*>(&v) + 4 * i, 4);
    const uint64_t o = (uint64_t)(uint32_t)byte + 4 * i;
    if (o + 4 <= b.bytes) std::memcpy(b.at + o, &word, 4);
  }
}
inline int dpp(int old, int v, int ctrl, int row_mask, int, bool) {
  const uint64_t* all = meet((uint32_t)v);
  const uint32_t l = lane(), row = l / 16, in = l % 16;
  if (!((row_mask >> row) & 1)) return old;
  if (ctrl < 0x100) return (int)all[l / 4 * 4 + ((ctrl >> (2 * (l % 4))) & 3)];                     // quad_perm
  if (ctrl > 0x110 && ctrl < 0x120) return in >= (uint32_t)(ctrl & 15) ? (int)all[l - (ctrl & 15)] : 0;      // row_shr
  if (ctrl > 0x120 && ctrl < 0x130) return (int)all[row * 16 + (in + 16 - (ctrl & 15)) % 16];       // row_ror
  if (ctrl == 0x142) return row ? (int)all[row * 16 - 1] : 0;                                        // row_bcast:15
  if (ctrl == 0x143) return row > 1 ? (int)all[31] : 0;                                              // row_bcast:31
  std::abort();
}
struct Pair { uint32_t v[2]; uint32_t operator[](int i) const { return v[i]; } };
// The odd ones of a's stretches of `span` lanes change places with the even ones of b's.
inline Pair swap(uint32_t a, uint32_t b, uint32_t span) {
  const uint64_t* all = meet((uint64_t)b << 32 | a);
  const uint32_t l = lane();
  const bool odd = l / span & 1;
  return {{odd ? (uint32_t)(all[l - span] >> 32) : a, odd ? b : (uint32_t)all[l + span]}};
}
inline uint32_t bitop3(uint32_t a, uint32_t b, uint32_t c, uint32_t table) {
  uint32_t v = 0;
  for (int i = 0; i < 8; ++i)
    if (table >> i & 1) v |= (i & 4 ? a : ~a) & (i & 2 ? b : ~b) & (i & 1 ? c : ~c);
  return v;
}
inline uint32_t perm(uint32_t a, uint32_t b, uint32_t select) {
  const uint64_t both = (uint64_t)a << 32 | b;
  uint32_t v = 0;
  for (int i = 0; i < 4; ++i) v |= (uint32_t)(both >> (8 * (select >> (8 * i) & 7)) & 255) << (8 * i);
  return v;
}
inline uint64_t ballot(bool p) {
  const uint64_t* all = meet(p);
  uint64_t m = 0;
  for (int i = 0; i < 64; ++i) m |= (all[i] & 1) << i;
  return m;
}
inline uint64_t below(uint32_t l, uint64_t mask) { return (uint64_t)__builtin_popcountll(mask & ((1ull << l) - 1)); }
template <typename T>
inline T from(T v, uint32_t l) {
  uint64_t bits = 0;
  std::memcpy(&bits, &v, sizeof v);
  bits = meet(bits)[l & 63];
  std::memcpy(&v, &bits, sizeof v);
  return v;
}
template <typename T, typename U>
inline T add(T* at, U v) { const T old = *at; *at = old + (T)v; return old; }
}  // namespace emu

#define threadIdx (emu::now->thread)
#define blockIdx emu::block_idx
#define gridDim emu::grid_dim
#define __syncthreads() ((void)emu::barrier(false))
#define __syncthreads_or(p) emu::barrier(p)
#define __ballot(p) emu::ballot(p)
#define __shfl(v, l, n) emu::from(v, (uint32_t)(l))
#define __shfl_xor(v, o, n) emu::from(v, emu::lane() ^ (uint32_t)(o))
#define __popc __builtin_popcount
#define __popcll __builtin_popcountll
#define __ffs __builtin_ffs
#define __ffsll(v) __builtin_ffsll((long long)(v))
#define atomicAdd emu::add
#define __float_as_uint(f) __builtin_bit_cast(uint32_t, (float)(f))
#define __uint_as_float(u) __builtin_bit_cast(float, (uint32_t)(u))
#define __double_as_longlong(d) __builtin_bit_cast(long long, (double)(d))
#define __longlong_as_double(l) __builtin_bit_cast(double, (long long)(l))
typedef uint32_t emu_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t emu_u32x4 __attribute__((ext_vector_type(4)));
#define __amdgpu_buffer_rsrc_t emu::Buffer
#define __builtin_amdgcn_make_buffer_rsrc emu::make_buffer
#define __builtin_amdgcn_raw_buffer_load_b128(b, at, s, c) emu::load<emu_u32x4, 4>(b, at)
#define __builtin_amdgcn_raw_buffer_load_b64(b, at, s, c) emu::load<emu_u32x2, 2>(b, at)
#define __builtin_amdgcn_raw_buffer_load_b32(b, at, s, c) (emu::load<emu_u32x4, 1>(b, at)[0])
#define __builtin_amdgcn_raw_buffer_store_b128(v, b, at, s, c) emu::store<decltype(v), 4>(v, b, at)
#define __builtin_amdgcn_raw_buffer_store_b32(v, b, at, s, c) emu::store<uint32_t, 1>(v, b, at)
#define __builtin_amdgcn_update_dpp emu::dpp
#define __builtin_amdgcn_mov_dpp(v, ctrl, row, bank, bound) emu::dpp(0, v, ctrl, row, bank, bound)
#define __builtin_amdgcn_readlane(v, l) emu::from((int)(v), (uint32_t)(l))
#define __builtin_amdgcn_readfirstlane(v) emu::from((int)(v), 0u)
#define __builtin_amdgcn_permlane32_swap(a, b, x, y) emu::swap(a, b, 32)
#define __builtin_amdgcn_permlane16_swap(a, b, x, y) emu::swap(a, b, 16)
#define __builtin_amdgcn_bitop3_b32 emu::bitop3
#define __builtin_amdgcn_perm emu::perm
#define __builtin_amdgcn_alignbit(a, b, n) ((uint32_t)((((uint64_t)(a) << 32) | (b)) >> (n)))
#define __builtin_amdgcn_ubfe(v, at, n) ((uint32_t)(v) >> (at) & ((1u << (n)) - 1u))
#define __builtin_amdgcn_rcpf(v) (1.0f / (v))
#define __builtin_amdgcn_rsqf(v) (1.0f / std::sqrt(v))
#define __builtin_amdgcn_mbcnt_lo(mask, n) ((uint32_t)(n) + (uint32_t)emu::below(std::min(emu::lane(), 32u), (uint32_t)(mask)))
#define __builtin_amdgcn_mbcnt_hi(mask, n) ((uint32_t)(n) + (emu::lane() < 32 ? 0u : (uint32_t)emu::below(emu::lane() - 32, (uint32_t)(mask))))
#define __builtin_amdgcn_s_waitcnt(n)
