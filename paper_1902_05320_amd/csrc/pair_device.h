// Pair lane-split sponge: one Keccak-f[1600] state per two adjacent lanes of
// a wave, 32 messages per wave.  Lane h = 0 of a pair holds the low 32-bit
// halves of the 25 state words, lane h = 1 the high halves (Section 3.1's
// lanes as 32-bit pairs, split across the two lanes).  Every step of a round
// is then half as many instructions per lane as one thread per message, and
// a 64-bit rotation takes the partner lane's half through one DPP move
// (quad_perm [1, 0, 3, 2]): for 0 < n < 32 both lanes compute
// alignbit(own, partner, 32 - n), for n > 32 alignbit(partner, own, 64 - n),
// and n = 32 is the partner's half itself.  About 120 VALU instructions per
// lane and round (30 of them DPP moves), against about 180 for one thread
// per message, and no exchange through memory.  What bounds a lone wave is
// issue, four cycles an instruction: 5.5 us per permutation against 8.4 for
// one thread per message (6.7 while every DPP move came with a v_mov of its
// unused old value and the moves stood right behind their sources); two waves
// per SIMD 7.8 us, for as many states as one wave of the other form.
#pragma once

#include "sponge_device.h"

namespace kb {
namespace pair {

constexpr int kPairLanes = 2;

// The partner lane's value (lanes 2k and 2k + 1 swap).
__device__ __forceinline__ uint32_t partner(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0xB1, 0xF, 0xF, true));
}

// Rotation of the 64-bit word whose half `v` this lane holds and whose other
// half is `p`, by a compile-time n.
__device__ __forceinline__ uint32_t rotl_half(uint32_t v, uint32_t p, int n) {
  if (n == 0) return v;
  if (n == 32) return p;
  if (n < 32) return __builtin_amdgcn_alignbit(v, p, 32 - n);
  return __builtin_amdgcn_alignbit(p, v, 64 - n);
}

// One round (eq. 10) on this lane's halves; `hi` is all ones on the lane
// holding the high halves.  In phases like the one-thread form: the DPP moves
// and rotations, neither of the class that pairs, run at raised priority, the
// moves ahead of the rotations that use them (a DPP move right after the
// instruction that writes its source waits two slots).
__device__ __forceinline__ void pair_round(uint32_t (&a)[25], uint32_t hi, uint32_t rc_lo, uint32_t rc_hi) {
  // theta (eqs. 2-4)
  uint32_t C[5], R[5];
#pragma unroll
  for (int x = 0; x < 5; ++x) C[x] = xor3(xor3(a[x], a[x + 5], a[x + 10]), a[x + 15], a[x + 20]);
  rot_phase_begin();
#pragma unroll
  for (int x = 0; x < 5; ++x) R[x] = partner(C[x]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int x = 0; x < 5; ++x) R[x] = rotl_half(C[x], R[x], 1);
  rot_phase_end();
#pragma unroll
  for (int y = 0; y < 5; ++y)
#pragma unroll
    for (int x = 0; x < 5; ++x) a[x + 5 * y] = xor3(a[x + 5 * y], C[(x + 4) % 5], R[(x + 1) % 5]);
  // rho and pi (eqs. 5-6)
  rot_phase_begin();
  uint32_t B[25];
#pragma unroll
  for (int i = 0; i < 25; ++i) B[kMaps.dst[i]] = kMaps.rot[i] ? partner(a[i]) : 0u;
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 25; ++i) B[kMaps.dst[i]] = rotl_half(a[i], B[kMaps.dst[i]], kMaps.rot[i]);
  rot_phase_end();
  // chi (eq. 7)
#pragma unroll
  for (int y = 0; y < 5; ++y)
#pragma unroll
    for (int x = 0; x < 5; ++x)
      a[x + 5 * y] = B[x + 5 * y] ^ (~B[(x + 1) % 5 + 5 * y] & B[(x + 2) % 5 + 5 * y]);
  // iota (eqs. 8-9): the low or high half of the round constant (the mask
  // passes through an empty asm so the selected constants are formed round
  // by round instead of being hoisted into registers)
  uint32_t m = hi;
  __asm__ volatile("" : "+v"(m));
  a[0] ^= (m & rc_hi) | (~m & rc_lo);
}

__device__ __forceinline__ void pair_permute(uint32_t (&a)[25], uint32_t hi) {
  rot_phase_end();
#pragma unroll 1
  for (int r = 0; r < 24; r += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) pair_round(a, hi, kRCTable.lo[r + q], kRCTable.hi[r + q]);
  }
}

// One block on its way into the state.  Of a whole block the two lanes of a
// pair load the 16-byte chunks in turn (lane h the chunks 2 q + h, any
// alignment: a quarter of the load instructions of dword loads, whose 17 times
// 32 lines held the wave up 1.3 us a block) and exchange halves when they
// absorb it; of the final block lane h loads its own half of word i as dword
// i of the same registers.
template <int V>
struct HalfDw {
  static constexpr int kQ = (SpongeShape<V>::kMaxRate + 31) / 32;  // chunk pairs
  uint32_t w[4 * kQ];
};

template <int V>
__device__ __forceinline__ void load_halves(HalfDw<V>& d, const uint8_t* msg, uint64_t len,
                                            uint64_t boff, int R, uint32_t h) {
  constexpr int kAll = V == kMixed ? 72 : SpongeShape<V>::kMaxRate;  // bytes every rate has
#pragma unroll
  for (int k = 0; k < 4 * HalfDw<V>::kQ; ++k) d.w[k] = 0u;
  if (len - boff >= static_cast<uint64_t>(R)) {
    const uint8_t* p = msg + boff + 16u * h;
#pragma unroll
    for (int q = 0; q < HalfDw<V>::kQ; ++q) {
      const int at = 32 * q + 16 * static_cast<int>(h);
      // (a value of its own, stored to d once: with the elements stored in the
      // branches the compiler kept d in private memory in the mixed form)
      Words4 v = {0u, 0u, 0u, 0u};
      if (32 * q + 32 <= kAll || at + 16 <= R) {
        v = *reinterpret_cast<const Words4*>(p + 32 * q);
      } else if (at + 8 == R) {
        const Words2 half = *reinterpret_cast<const Words2*>(p + 32 * q);
        v.x = half.x;
        v.y = half.y;
      }
      d.w[4 * q] = v.x;
      d.w[4 * q + 1] = v.y;
      d.w[4 * q + 2] = v.z;
      d.w[4 * q + 3] = v.w;
    }
    return;
  }
  // bytes of the message from this lane's first half on (< R)
  const uint8_t* p = msg + boff + 4u * h;
  const int left = static_cast<int>(len - boff) - 4 * static_cast<int>(h);
#pragma unroll
  for (int i = 0; i < SpongeShape<V>::kMaxRate / 8; ++i)
    if (left - 8 * i >= 4) d.w[i] = *reinterpret_cast<const Word1*>(p + 8 * i);
  if (left > 0 && (left & 7) > 0 && (left & 7) < 4) {  // a half cut off: byte by byte
    const int i8 = left & ~7;
    uint32_t x = 0u;
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (q < (left & 7)) x |= static_cast<uint32_t>(p[i8 + q]) << (8 * q);
#pragma unroll
    for (int i = 0; i < SpongeShape<V>::kMaxRate / 8; ++i)
      if (8 * i == i8) d.w[i] = x;
  }
}

// Xor this lane's halves of one block into the state; on the final block
// (`rem` message bytes, rem < R) the suffix/pad10*1 bytes too: `pad` at byte
// rem, 0x80 on byte R - 1.  `hi` is all ones on lane 1.  Both lanes of a pair
// are at the same block of the same message.
template <int V>
__device__ __forceinline__ void absorb_halves(uint32_t (&a)[25], const HalfDw<V>& d, int R, bool fin,
                                              uint32_t rem, uint32_t pad, uint32_t h, uint32_t hi) {
  constexpr int kWords = SpongeShape<V>::kMaxRate / 8;
  if (!fin) {
    // lane 0 holds words 4q, 4q + 1 and needs the low halves of 4q .. 4q + 3,
    // lane 1 holds 4q + 2, 4q + 3 and needs the high halves
    auto pick = [&](uint32_t on1, uint32_t on0) { return (hi & on1) | (~hi & on0); };
#pragma unroll
    for (int q = 0; q < HalfDw<V>::kQ; ++q)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t lo = d.w[4 * q + 2 * j], up = d.w[4 * q + 2 * j + 1];
        const uint32_t mine = pick(up, lo), theirs = partner(pick(lo, up));
        if (4 * q + j < kWords) a[4 * q + j < 25 ? 4 * q + j : 0] ^= pick(theirs, mine);
        if (4 * q + 2 + j < kWords) a[4 * q + 2 + j < 25 ? 4 * q + 2 + j : 0] ^= pick(mine, theirs);
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < kWords; ++i) {
    uint32_t v = d.w[i];
    const int k = static_cast<int>(rem) - (8 * i + 4 * static_cast<int>(h));  // message bytes here
    if (k >= 0 && k < 4) v ^= pad << (8 * k);
    if (8 * i == R - 8 && h) v ^= 0x80000000u;
    a[i] ^= v;
  }
}

// The digest's dwords 2 i + h (Section 3.2, eq. 15) from this lane, zero past
// the digest up to `slot_dw`.
__device__ __forceinline__ void store_halves(uint32_t* o, const uint32_t (&a)[25], int dw, int slot_dw,
                                             uint32_t h) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int k = 2 * i + static_cast<int>(h);
    if (k < slot_dw) o[k] = k < dw ? a[i] : 0u;
  }
}

}  // namespace pair
}  // namespace kb
