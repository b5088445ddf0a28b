// Wide lane-split sponge: one Keccak-f[1600] state per wave, one 32-bit half
// of a state word per lane, held bit-interleaved: half 0 of a word is its even
// bits, half 1 its odd bits.  The serial absorb chain of one message (Section
// 3.2) then costs each lane about a dozen VALU instructions and five lane
// reads per round.
//
// Bit-interleaving (a published technique of 32-bit Keccak code: Bertoni et
// al., "Keccak implementation overview") makes every rotation local: rotating
// a word by 2k rotates both halves by k; rotating it by 2k + 1 swaps the
// halves, the even ones rotated by k and the odd ones by k + 1 before.  A swap
// is only a different source lane.  So no lane ever needs its partner half.
//
// Lane layout: the five words of column x, half h, sit in five neighbouring
// lanes of one 16-lane row, group g = 2x + h in row g / 3 at lanes
// 5 (g % 3) + y.  Per round (eq. 10):
//   theta  column parities by three row shifts (DPP), complete in the lane of
//          y = 4; every lane then reads C[x-1] and, of the other half,
//          C[x+1] from those lanes (ds_bpermute) and applies
//          D = C[x-1] ^ rot(C[x+1], 1) (eqs. 2-4);
//   rho    one rotation by the lane's own amount (eq. 5);
//   pi     is where chi reads from (eq. 6);
//   chi    reads words x, x + 1, x + 2 of its row (three ds_bpermute, eq. 7);
//   iota   is linear, so that of round r is folded into round r + 1's theta:
//          the constant reaches word (0, 0) and, through the parity of column
//          0, the columns 1 and 4, one xor off the critical path (eqs. 8-9).
// What bounds it is latency: two lane-read round trips of 56 cycles and a
// chain of about ten dependent VALU instructions (6.5 cycles each, 13 through
// DPP).  Measured on one wave alone, per permutation: 2.15 us, against 3.03
// for one 64-bit word per lane with both exchanges through LDS memory (two
// states per wave); with 2048 states on the chip (two waves per SIMD against
// one) 2.79 against 3.75, with 4096 5.6 against 5.5.  Column parities through
// LDS memory instead of DPP: 2.07 alone, but 4.1 with two waves per SIMD (the
// reads of ten words per lane fill the LDS).
#pragma once

#include "sponge_device.h"

namespace kb {
namespace wide {

constexpr int kStateLanes = 64;  // lanes per state

// Bits h, h + 2, h + 4, ... of a 64-bit word.
constexpr uint32_t half_bits(uint64_t v, int h) {
  uint32_t r = 0;
  for (int i = 0; i < 32; ++i) r |= static_cast<uint32_t>((v >> (2 * i + h)) & 1u) << i;
  return r;
}

struct HalfConstants {
  uint32_t e[24], o[24];
};
constexpr HalfConstants make_half_constants() {
  HalfConstants t{};
  for (int r = 0; r < 24; ++r) {
    const uint64_t v = (static_cast<uint64_t>(kRC.hi[r]) << 32) | kRC.lo[r];
    t.e[r] = half_bits(v, 0);
    t.o[r] = half_bits(v, 1);
  }
  return t;
}
constexpr HalfConstants kHalfRC = make_half_constants();

// The 25 rotation amounts, ten 6-bit fields to a constant, and their parities.
struct RotTable {
  uint64_t six[3];
  uint32_t odd;
};
constexpr RotTable make_rot_table() {
  RotTable t{};
  for (int i = 0; i < 25; ++i) {
    t.six[i / 10] |= static_cast<uint64_t>(kMaps.rot[i]) << (6 * (i % 10));
    t.odd |= static_cast<uint32_t>(kMaps.rot[i] & 1) << i;
  }
  return t;
}
constexpr RotTable kRot = make_rot_table();

// Per-lane constants of the wide form.
struct WideLane {
  uint32_t word;        // state word of this lane (25: idle lane)
  uint32_t half;        // 0: its even bits, 1: its odd bits
  uint32_t cm, cp;      // lane reads (byte addresses): C[x-1] of this half, C[x+1] of the other
  uint32_t b0, b1, b2;  // words x, x + 1, x + 2 of this row after rho and pi
  uint32_t partner;     // the other half of this word
  uint32_t one;         // theta's rotation by one, as a v_alignbit amount
  uint32_t sh;          // rho's
  uint32_t m1, m2, m3;  // lanes whose folded iota constant is RC's even bits, odd bits, odd bits rotated
  uint32_t origin;      // all ones on word (0, 0)
};

// Byte address of the lane that holds half h of word i.
__device__ __forceinline__ uint32_t lane_address(uint32_t i, uint32_t h) {
  const uint32_t g = (i % 5u) * 2u + h;
  return 4u * ((g / 3u) * 16u + (g % 3u) * 5u + i / 5u);
}

__device__ __forceinline__ void setup(WideLane& L, uint32_t lane) {
  const uint32_t s = lane & 15u, g0 = (lane >> 4) * 3u + s / 5u;
  const bool on = s < 15u && g0 < 10u;
  const uint32_t g = on ? g0 : 0u, y = on ? s % 5u : 0u;
  const uint32_t x = g >> 1, h = g & 1u, i = x + 5u * y;
  L.word = on ? i : 25u;
  L.half = h;
  const uint64_t six = i < 10u ? kRot.six[0] : i < 20u ? kRot.six[1] : kRot.six[2];
  const uint32_t n = static_cast<uint32_t>(six >> (6u * (i % 10u))) & 63u;
  // n = 2k: by k; n = 2k + 1: the even bits by k, the odd ones by k + 1
  const uint32_t amount = (n + ((n & 1u) & h)) >> 1;
  L.sh = (32u - amount) & 31u;
  // rotl(C, 1): its even bits are C's odd ones rotated by one, its odd bits C's even ones
  L.one = h == 0u ? 31u : 0u;
  L.cm = lane_address((x + 4u) % 5u + 20u, h);
  L.cp = lane_address((x + 1u) % 5u + 20u, h ^ 1u);
  // pi sends word (y, 2x' + 3y) = (X, Y) from (x', y): x' = 3Y + X mod 5, y = X;
  // an odd rotation moves the half across
  auto source = [&](uint32_t X) -> uint32_t {
    const uint32_t j = (3u * y + X) % 5u + 5u * X;
    return lane_address(j, h ^ ((kRot.odd >> j) & 1u));
  };
  L.b0 = source(x);
  L.b1 = source((x + 1u) % 5u);
  L.b2 = source((x + 2u) % 5u);
  L.partner = lane_address(i, h ^ 1u);
  const bool direct = i == 0u || x == 1u, rotated = x == 4u;
  L.m1 = on && ((direct && h == 0u) || (rotated && h == 1u)) ? ~0u : 0u;
  L.m2 = on && direct && h == 1u ? ~0u : 0u;
  L.m3 = on && rotated && h == 0u ? ~0u : 0u;
  L.origin = on && i == 0u ? ~0u : 0u;
}

__device__ __forceinline__ uint32_t read_lane(uint32_t address, uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(static_cast<int>(address), static_cast<int>(v)));
}

// w ^ (v shifted up N lanes within its row of 16)
template <int N>
__device__ __forceinline__ uint32_t xor_row_shift(uint32_t w, uint32_t v) {
  return w ^ static_cast<uint32_t>(
                 __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x110 + N, 0xf, 0xf, true));
}

// One round (eq. 10), its iota left to the next one; `r` must fold to a
// constant.  Round 0 takes a state whose last iota has been applied.
__device__ __forceinline__ void wide_round(uint32_t& a, const WideLane& L, int r) {
  // theta (eqs. 2-4): in the lane of y = 4, pairs (3, 4) and 0, then (1, 2)
  const uint32_t q = xor_row_shift<1>(a, a);
  const uint32_t p = xor_row_shift<4>(q, a);
  const uint32_t c = xor_row_shift<2>(p, q);
  const uint32_t cp = read_lane(L.cp, c);
  const uint32_t cm = read_lane(L.cm, c);
  uint32_t ak = a;
  if (r > 0) {
    const uint32_t e = kHalfRC.e[r - 1], o = kHalfRC.o[r - 1];
    uint32_t m1 = L.m1, m2 = L.m2, m3 = L.m3;
    // (through an empty asm so that the masked constants are formed round by
    // round, not hoisted into registers)
    __asm__ volatile("" : "+v"(m1), "+v"(m2), "+v"(m3));
    if (e) ak ^= m1 & e;
    if (o) ak ^= (m2 & o) | (m3 & ((o << 1) | (o >> 31)));
  }
  const uint32_t d = __builtin_amdgcn_alignbit(cp, cp, L.one);
  a = xor3(ak, cm, d);
  // rho (eq. 5), pi (eq. 6) and chi (eq. 7)
  const uint32_t v = __builtin_amdgcn_alignbit(a, a, L.sh);
  const uint32_t b1 = read_lane(L.b1, v);
  const uint32_t b2 = read_lane(L.b2, v);
  const uint32_t b0 = read_lane(L.b0, v);
  a = b0 ^ (~b1 & b2);
}

__device__ __forceinline__ void wide_permute(uint32_t& a, const WideLane& L) {
#pragma unroll
  for (int r = 0; r < 24; ++r) wide_round(a, L, r);
  // iota of the last round (eqs. 8-9)
  a ^= L.origin & (L.half ? kHalfRC.o[23] : kHalfRC.e[23]);
}

// This lane's half of the word (lo, hi): bits h, h + 2, ... gathered by
// swapping neighbouring bits, pairs, nibbles and bytes.
__device__ __forceinline__ uint32_t gather_half(uint32_t lo, uint32_t hi, uint32_t h) {
  uint32_t t = ((lo >> h) & 0x55555555u) | (((hi >> h) & 0x55555555u) << 1);
  uint32_t s;
  s = (t ^ (t >> 1)) & 0x22222222u;
  t ^= s ^ (s << 1);
  s = (t ^ (t >> 2)) & 0x0C0C0C0Cu;
  t ^= s ^ (s << 2);
  s = (t ^ (t >> 4)) & 0x00F000F0u;
  t ^= s ^ (s << 4);
  return __builtin_amdgcn_perm(t, t, 0x03010200u);
}

// The reverse, for output: dword h (low or high) of this lane's word.
__device__ __forceinline__ uint32_t output_dword(uint32_t a, const WideLane& L) {
  const uint32_t other = read_lane(L.partner, a);
  const uint32_t e = L.half ? other : a, o = L.half ? a : other;
  // 16 even bits and 16 odd bits, then spread
  uint32_t t = __builtin_amdgcn_perm(o, e, L.half ? 0x07060302u : 0x05040100u);
  t = __builtin_amdgcn_perm(t, t, 0x03010200u);
  uint32_t s;
  s = (t ^ (t >> 4)) & 0x00F000F0u;
  t ^= s ^ (s << 4);
  s = (t ^ (t >> 2)) & 0x0C0C0C0Cu;
  t ^= s ^ (s << 2);
  s = (t ^ (t >> 1)) & 0x22222222u;
  t ^= s ^ (s << 1);
  return t;
}

// The dwords holding the bytes of this lane's word of the block at message
// byte `boff` (message bytes [boff + 8 word, boff + 8 word + 8) that exist),
// read from aligned dwords (`sh` = message address mod 4).
struct WordDw {
  uint32_t w[3];
};

__device__ __forceinline__ void load_word(WordDw& d, const uint8_t* msg, uint32_t sh, uint64_t len,
                                          uint64_t boff, int R, const WideLane& L) {
  d.w[0] = d.w[1] = d.w[2] = 0u;
  const uint64_t o = boff + 8u * L.word;
  if (8u * L.word < static_cast<uint32_t>(R) && o < len) {
    const uint64_t left = len - o;
    const uint32_t nv = sh + (left < 8u ? static_cast<uint32_t>(left) : 8u);
    const uint32_t* base = reinterpret_cast<const uint32_t*>(msg + o - sh);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (4u * k < nv) d.w[k] = base[k];
  }
}

// Xor this lane's half of one block word into the state (eq. 12's P_i); on
// the final block (`rem` message bytes left, rem < R) only message bytes are
// kept and the suffix/pad10*1 bytes are added: `pad` at byte rem, 0x80 on
// byte R - 1.
__device__ __forceinline__ void absorb_word(uint32_t& a, const WordDw& d, uint32_t sh, int R, bool fin,
                                            uint32_t rem, uint32_t pad, const WideLane& L) {
  uint32_t lo = __builtin_amdgcn_alignbyte(d.w[1], d.w[0], sh);
  uint32_t hi = __builtin_amdgcn_alignbyte(d.w[2], d.w[1], sh);
  if (fin) {
    const int v = static_cast<int>(rem) - 8 * static_cast<int>(L.word);  // message bytes in this word
    if (v < 4) lo = v <= 0 ? 0u : lo & ((1u << (8 * v)) - 1u);
    if (v < 8) hi = v <= 4 ? 0u : hi & ((1u << (8 * (v - 4))) - 1u);
    if (v >= 0 && v < 4) lo ^= pad << (8 * v);
    if (v >= 4 && v < 8) hi ^= pad << (8 * (v - 4));
    if (8 * static_cast<int>(L.word) == R - 8) hi ^= 0x80000000u;
  }
  const uint32_t half = gather_half(lo, hi, L.half);
  if (8u * L.word < static_cast<uint32_t>(R)) a ^= half;
}

// The digest (Section 3.2, eq. 15): words 0 .. D/8 of the final state, each
// written by the lanes that hold it; with `slot_dw` = 16 (mixed form) the
// slot is filled with zeros past the digest.
__device__ __forceinline__ void store_word(uint32_t* o, uint32_t a, int dw, int slot_dw, const WideLane& L) {
  const uint32_t v = output_dword(a, L);
  const int k = 2 * static_cast<int>(L.word) + static_cast<int>(L.half);
  if (L.word < 25u && k < slot_dw) o[k] = k < dw ? v : 0u;
}

}  // namespace wide
}  // namespace kb
