// Who wins in a Top-K selection, told from x, xhat and the selection's outcome, and where a winner belongs in
// the message.
#pragma once
#include "evg_device.h"

namespace evg {

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The first pass's bins, by ascending keys: a quarter of an octave each (bits 30..21), but a sixty-fourth (bits 30..17) in the two
// octaves from the anchor on, bits 30..17 of a key (a multiple of 16), in whose middle the threshold is expected.  A bin holds some
// 0.4 % of a tensor's keys there; with an eighth of an octave everywhere (rings without anchors) 3 to 12 %.
// (Four keys at a time, two in a register, in 16-bit arithmetic: 25 instructions instead of 40.)
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
struct Bins { uint32_t bin[4], codes; };     // codes: see Tables::codes
__device__ __forceinline__ Bins first_bins(const float x[4], const float h[4], uint32_t by_value, uint32_t anchor) {
  const unsigned short f = (unsigned short)anchor, a = f / (unsigned short)kPerCoarse;               // (kNoAnchor: past every key)
  Bins b;
  uint32_t codes[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t k0 = rank_key(x[2 * i], h[2 * i], by_value), k1 = rank_key(x[2 * i + 1], h[2 * i + 1], by_value);
    const u16x2 q = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(k1, k0, 0x07060302u)) >> (u16x2)(unsigned short)(kFineBits - 16);      // bits 30..kFineBits
    const u16x2 coarse = q >> (u16x2)(unsigned short)(kCoarseBits - kFineBits), fine = __builtin_elementwise_sub_sat(q, (u16x2)f);
    const u16x2 bin = __builtin_elementwise_min(coarse, (u16x2)a) + __builtin_elementwise_min(fine, (u16x2)(unsigned short)kFineBins) +
                      __builtin_elementwise_sub_sat(coarse, (u16x2)(unsigned short)(a + kFineBins / kPerCoarse));
    b.bin[2 * i] = bin.x;
    b.bin[2 * i + 1] = bin.y;
    codes[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(fine, (u16x2)(unsigned short)255));
  }
  b.codes = __builtin_amdgcn_perm(codes[1], codes[0], 0x06040200u);
  return b;
}
// Where an update pass counts the keys of a tensor: worker r's histogram is number first + r * step of those in T.hist.
struct HistAt { uint32_t first, step; };
__device__ __forceinline__ HistAt first_hist(const Tables& T, uint32_t layer, uint32_t copy) {
  const uint32_t which = layer == T.long_layer[0] ? 0u : layer == T.long_layer[1] ? 1u : 2u;
  if (copy == 0 || which == 2) return {layer, T.L};
  return {T.S + (which * (kHistCopies - 1) + copy - 1) * T.P, 1u};
}
// The smallest key of a bin, and how many bits its keys have below it.
__device__ __forceinline__ uint32_t bin_begin(uint32_t bin, uint32_t anchor, uint32_t* left) {
  const uint32_t a = anchor / kPerCoarse;
  *left = bin >= a && bin < a + kFineBins ? kFineBits : kCoarseBits;
  return bin < a ? bin << kCoarseBits : bin < a + kFineBins ? (bin - a + (anchor & kAnchorBits)) << kFineBits
                                                          : (bin - (kFineBins - kFineBins / kPerCoarse)) << kCoarseBits;
}
// Codes of four elements at bytes `byte` .. of a window of `bytes` bytes of an arena that starts at element `first` of it.
__device__ __forceinline__ void store_codes(const Tables& T, size_t first, uint32_t bytes, uint32_t byte, uint32_t four) {
  __builtin_amdgcn_raw_buffer_store_b32(four, window(T.codes + first, bytes >> 2), (int)(byte >> 2), 0, 2);     // non-temporal
}

// Sixteen codes against one (1 .. 254): how many are above it, and which are equal, bit 8 b + w for the b-th of the w-th four.
// Four bytes at a time: with bit 7 set, a byte less the lower seven bits of k keeps that bit where its own seven are no less.  (44 instructions;
// taking bytes apart into halves of registers 70.)
struct Compared { uint32_t above, in; };
__device__ __forceinline__ Compared compare_codes(const u32x4& sixteen, uint32_t code) {
  const uint32_t k = code * 0x01010101u, k1 = k + 0x01010101u, m = 0x80808080u;
  Compared c{0u, 0u};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t four = sixteen[w], with = four | m;
    // (a & ~b) | (~(a ^ b) & c): bit 7 of each byte says whether it is at least the code, or above it
    const uint32_t ge = __builtin_amdgcn_bitop3_b32(four, k, with - (k & ~m), 0xB2);
    const uint32_t gt = __builtin_amdgcn_bitop3_b32(four, k1, with - (k1 & ~m), 0xB2);
    c.above += (uint32_t)__popc(gt & m);
    const uint32_t eq = __builtin_amdgcn_bitop3_b32(ge, gt, m, 0x20);                 // a & ~b & c
    c.in |= eq >> (7 - w);
  }
  return c;
}
// Sum over the lane's sixteen lanes.
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);   // row_ror:8, 4, 2, 1
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x122, 0xF, 0xF, true);
  v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x121, 0xF, 0xF, true);
  return v;
}

// One bit per element of a float4, the first of them element j of the tensor.  thr = kNoThreshold: none.
// nv: how many of the four are elements of the tensor.
__device__ __forceinline__ uint32_t winners4(const float x[4], const float h[4], uint32_t by_value, uint32_t thr,
                                             uint32_t cut, uint32_t j, uint32_t nv) {
  uint32_t win = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t key = rank_key(x[i], h[i], by_value);
    win |= key > thr || (key == thr && j + i <= cut) ? 1u << i : 0u;
  }
  return win & ((1u << nv) - 1u);
}

__device__ __forceinline__ void take_winners(uint32_t win, const float x[4], float h[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) h[i] = (win >> i) & 1u ? x[i] : h[i];
}

// Is `any` non-zero in one of the four lanes whose float4s make up an aligned 64 bytes?  Those are written
// together: scattered 16-byte writes cost far more in HBM than the unchanged bytes (128 bytes: 3 % slower
// where 10 % is sent, 2 % faster at 1 %).
__device__ __forceinline__ bool any_of_line_part(uint32_t any) {
  any |= (uint32_t)__builtin_amdgcn_mov_dpp((int)any, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
  any |= (uint32_t)__builtin_amdgcn_mov_dpp((int)any, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
  return any != 0;
}

// Winners of the tensor before a group of 256 elements (chunk w of all workers' chunks, group g of the chunk; ties: how
// many keys equal to the threshold win).
__device__ __forceinline__ uint32_t winners_before(const Tables& T, uint32_t w, uint32_t g, uint32_t ties) {
  const uint2 before = T.chunk_before[w];
  const uint32_t in_chunk = T.group[(size_t)w * (T.SW * 4) + g], equal = before.y + (in_chunk >> 16);
  return before.x + (in_chunk & 0xFFFFu) + (equal < ties ? equal : ties);
}

// Where a group has its entries in its tensor's message, and (CHECK, see put_message) how many.
struct Place { uint32_t first, count; };

// w, cd: the chunk.
template <bool CHECK>
__device__ __forceinline__ Place message_place(const Tables& T, uint32_t w, const ChunkDesc& cd, const LayerDesc& ld, uint32_t g, uint32_t ties) {
  const uint32_t first = winners_before(T, w, g, ties);
  if (!CHECK) return {first, 0u};
  const uint32_t G = T.SW * 4, beyond = cd.j0 + (g + 1) * 256 - cd.lead;        // the next group's first element
  const bool same = g + 1 < G;                        // it is in this chunk
  // (what is past the tensor's last chunk, and past its last group, is not read: the tensor ends with its K-th entry)
  const uint32_t w2 = same || beyond >= ld.numel ? w : w + 1, g2 = same && beyond < ld.numel ? g + 1 : 0u;
  const uint32_t end = winners_before(T, w2, g2, ties);
  return {first, beyond < ld.numel ? end - first : beyond < ld.numel + 256 ? ld.K - first : 0u};       // (past the tensor's end: none)
}

// How many winners a wavefront's group has, and how many come before a lane's first.
__device__ __forceinline__ uint32_t count_winners(uint32_t win, uint32_t* rank) {
  uint32_t n = 0;
  *rank = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t m = __ballot((win >> i) & 1u);
    n += (uint32_t)__popcll(m);
    *rank += lanes_below(m);
  }
  return n;
}

// The winners of a wavefront's group, none if there are not as many as the selection has counted in it: the selection goes by key
// codes, and the caller has written x since the last update pass left them.
__device__ __forceinline__ uint32_t counted_winners(uint32_t win, uint32_t count) {
  uint32_t rank;
  return count_winners(win, &rank) == count ? win : 0u;
}

// Writes the winners of a wavefront's group to their places in worker r's message, ascending indices; `first` is the
// first one's, `count` how many the selection has counted in the group (the same in all lanes).  CHECK: where there is another number
// (see above) all of these places are marked as empty instead.  Returns who is sent.  The stretch of the group is a buffer of just its
// entries, past which the other lanes' stores fall.
template <bool CHECK>
__device__ __forceinline__ uint32_t put_message(const Tables& T, uint32_t r, uint32_t msg_off, uint32_t first, uint32_t count, uint32_t win,
                                                const float x[4], uint32_t j) {
  uint32_t rank;
  const uint32_t n = count_winners(win, &rank);
  if (!CHECK) count = n;
  if ((n | count) == 0) return 0;                     // wave-uniform
  const bool fits = n == count;
  win = fits ? win : 0u;
  const size_t at = (size_t)r * T.Ktot + msg_off + (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
  const __amdgpu_buffer_rsrc_t idx = window(T.msg_idx + at, count * 4), val = window(T.msg_val + at, count * 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool w = (win >> i) & 1u;
    const int byte = (int)(!fits ? lane_id() * 16 + 4 * i : w ? rank * 4 : 0xFFFFFFF0u);
    __builtin_amdgcn_raw_buffer_store_b32(fits ? j + i : kNoEntry, idx, byte, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[i]), val, byte, 0, 0);
    rank += w ? 1u : 0u;
  }
  return win;
}

}  // namespace evg
