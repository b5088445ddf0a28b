// The SHA-3 sponge (Section 3.2, eqs. 11-16) for one message per thread.
//
// A whole block is read with unaligned 16- and 8-byte loads straight into its
// words (the next one while the current one is permuted) and xored into the
// state; nothing outside the message is touched.  Staging these blocks through
// LDS like the final one cost 37 realignments, 10 LDS writes and 19 reads with
// eight-way bank conflicts a block: 32768 x 4 KiB 346 us against 313.
//
// The final block of the padded message P = M || 01 || pad10*1 is staged
// through a per-thread row of LDS:
//   1. the 16-byte-aligned chunks that hold the block's bytes are read with
//      global_load_dwordx4 and stored to the row unchanged, so a block at any
//      byte offset costs at most ceil((R + 15) / 16) vector loads;
//   2. the bytes past the message end are cleared and the suffix/padding bytes are written with byte-granular LDS stores: 0x06
//      (bits 0,1 of the suffix "01" then the first pad bit; 0x1F for the
//      SHAKE suffix "1111") at the message end, 0x80 (the last pad bit) on
//      byte R-1, or the two OR-ed when both fall on byte R-1 -- the byte form
//      of N || pad10*1 with j = (-m-2) mod r;
//   3. the row is read back as dwords and realigned with v_alignbyte.
// The data-dependent byte positions thus cost LDS address arithmetic, not
// per-dword VALU masking.
//
// Variant `V` is 0..3 (SHA3-224/256/384/512, rate fixed at compile time),
// kMixed (one of those four chosen per thread at run time), or kShake128 /
// kShake256 (the XOFs of eqs. 17-18: suffix 1111, so the byte after the
// message is 0x1F, and any output length).
#pragma once

#include "keccak_device.h"

namespace kb {

constexpr int kMixed = 4;
constexpr int kShake128 = 5;  // Keccak[256]: rate 168 bytes
constexpr int kShake256 = 6;  // Keccak[512]: rate 136 bytes

template <int V>
struct SpongeShape {
  static constexpr int kMaxRate =
      V == kMixed ? 144 : V == kShake128 ? 168 : V == kShake256 ? 136 : rate_bytes_of(V);
  static constexpr int kMaxRateDw = kMaxRate / 4;
  // 16-byte chunks that can hold R bytes starting at any offset mod 16
  static constexpr int kChunks = (kMaxRate + 15 + 15) / 16;
  // the LDS row is the chunk area; the read-back (dwords s16/4 .. s16/4 + R/4,
  // s16 < 16) stays inside it, and clearing stores past it are dropped
  static constexpr int kRowDw = kChunks * 4;
  static_assert(3 + kMaxRate / 4 < kRowDw, "read-back must stay inside the row");
  static constexpr int kMaxDigestDw = V == kMixed ? 16 : V >= kShake128 ? 0 : digest_bytes_of(V) / 4;
  // the suffix bits and the first pad bit, as the byte after the message:
  // SHA-3 "01" then 1 -> 0x06; SHAKE "1111" then 1 -> 0x1F
  static constexpr uint32_t kPadByte = V >= kShake128 ? 0x1Fu : 0x06u;
};

__device__ __forceinline__ int rate_bytes_rt(int v) { return 200 - 2 * (v == 0 ? 28 : v == 1 ? 32 : v == 2 ? 48 : 64); }
__device__ __forceinline__ int digest_bytes_rt(int v) { return v == 0 ? 28 : v == 1 ? 32 : v == 2 ? 48 : 64; }

// The bytes of one block on their way into the state: for the final block the
// 16-byte-aligned chunks that hold them (s16 = message address mod 16), for a
// whole block its words in order.
template <int V>
struct BlockChunks {
  uint4 c[SpongeShape<V>::kChunks];
  uint32_t s16;
};

// The final block's chunks: `p` points at its first message byte, `rem` =
// bytes left (< R).  Only chunks holding at least one message byte are read;
// the rest are zero.
template <int V>
__device__ __forceinline__ void load_block(BlockChunks<V>& bc, const uint8_t* p, uint32_t rem) {
  using S = SpongeShape<V>;
  bc.s16 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p) & 15u);
  // derive the aligned base by pointer arithmetic (not from an integer) so
  // the loads stay in the global address space
  const uint4* base = reinterpret_cast<const uint4*>(p - bc.s16);
  const uint32_t nv = bc.s16 + rem;
#pragma unroll
  for (int j = 0; j < S::kChunks; ++j) {
    bc.c[j] = make_uint4(0u, 0u, 0u, 0u);
    if (rem != 0u && 16u * j < nv) bc.c[j] = base[j];
  }
}

// 16, 8 and 4 bytes at any byte address (gfx950 loads and stores them unaligned).
typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t Words2 __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t Word1 __attribute__((aligned(1)));

template <int V>
__device__ __forceinline__ uint32_t& chunk_dword(BlockChunks<V>& bc, int k) {
  uint4& c = bc.c[k / 4];
  return k % 4 == 0 ? c.x : k % 4 == 1 ? c.y : k % 4 == 2 ? c.z : c.w;
}

// The 8-byte words FROM .. TO - 1 of the block at p.
template <int V, int FROM, int TO>
__device__ __forceinline__ void load_words(BlockChunks<V>& bc, const uint8_t* p) {
#pragma unroll
  for (int i = FROM; i < TO; i += 2) {
    if (i + 1 < TO) {
      const Words4 v = *reinterpret_cast<const Words4*>(p + 8 * i);
      chunk_dword<V>(bc, 2 * i) = v.x;
      chunk_dword<V>(bc, 2 * i + 1) = v.y;
      chunk_dword<V>(bc, 2 * i + 2) = v.z;
      chunk_dword<V>(bc, 2 * i + 3) = v.w;
    } else {
      const Words2 v = *reinterpret_cast<const Words2*>(p + 8 * i);
      chunk_dword<V>(bc, 2 * i) = v.x;
      chunk_dword<V>(bc, 2 * i + 1) = v.y;
    }
  }
}

// A whole block (R bytes at p, any alignment) straight into its words, zero
// past R: nothing is read outside the block, and its words can be xored into
// the state as they are.  In the mixed form the lanes of a wave differ in R:
// the words go in the four groups that the rates end at (72, 104, 136 and 144
// bytes), three of them under a condition, rather than a condition for each
// 16-byte chunk.
template <int V>
__device__ __forceinline__ void load_whole_block(BlockChunks<V>& bc, const uint8_t* p, int R) {
  if constexpr (V == kMixed) {
#pragma unroll
    for (int k = 18; k < 36; ++k) chunk_dword<V>(bc, k) = 0u;
    load_words<V, 0, 9>(bc, p);
    if (R >= 104) {
      load_words<V, 9, 13>(bc, p);
      if (R >= 136) {
        load_words<V, 13, 17>(bc, p);
        if (R >= 144) load_words<V, 17, 18>(bc, p);
      }
    }
  } else {
    load_words<V, 0, SpongeShape<V>::kMaxRate / 8>(bc, p);
  }
}

// Stage the final block's chunks through `row`, apply the padding (rem < R)
// and return the block as little-endian dwords w[0 .. kMaxRateDw), garbage
// past R.
template <int V>
__device__ __forceinline__ void stage_block(uint32_t* __restrict__ row, const BlockChunks<V>& bc,
                                            uint32_t rem, int R,
                                            uint32_t (&w)[SpongeShape<V>::kMaxRateDw]) {
  using S = SpongeShape<V>;
  const uint32_t s16 = bc.s16;
  const uint32_t nv = s16 + rem;  // row bytes [s16, nv) hold message bytes
  uint4* row4 = reinterpret_cast<uint4*>(row);
#pragma unroll
  for (int j = 0; j < S::kChunks; ++j) row4[j] = bc.c[j];
  // clear the tail of the last chunk: up to three whole dwords past the
  // dword holding byte nv, then bytes nv..nv+2 (suffix byte first)
  // (nv < s16 + R <= 4 kRowDw, so the suffix byte is always inside the row)
  const uint32_t d0 = (nv + 3u) >> 2;
#pragma unroll
  for (uint32_t k = 0; k < 3; ++k)
    if (d0 + k < static_cast<uint32_t>(S::kRowDw)) row[d0 + k] = 0u;
  uint8_t* rb = reinterpret_cast<uint8_t*>(row);
  rb[nv] = S::kPadByte;
  if (nv + 1u < 4u * S::kRowDw) rb[nv + 1] = 0u;
  if (nv + 2u < 4u * S::kRowDw) rb[nv + 2] = 0u;
  rb[s16 + R - 1] = rem + 1u == static_cast<uint32_t>(R) ? (S::kPadByte | 0x80u) : 0x80u;
  const uint32_t* src = row + (s16 >> 2);
  const uint32_t sh = s16 & 3u;
#pragma unroll
  for (int k = 0; k < S::kMaxRateDw; ++k) w[k] = __builtin_amdgcn_alignbyte(src[k + 1], src[k], sh);
}

// Absorb the whole message and run the permutation on every block; on return
// A holds Keccak-f[1600] of the last absorbed state, i.e. the squeezed output
// lanes (d <= r for every SHA-3 variant, so one squeeze suffices).
// With prefetch on, the chunks of block b+1 are loaded into registers before
// the permutation of block b and land while it runs, so a multi-block
// message's chain of permutations does not wait for HBM between blocks.  It
// costs the registers of one block of chunks (about 40 VGPRs).  Measured by
// interleaved A/B on one box: 4 KiB Merkle leaves 1.14 ms per 1 GiB root
// with it against 1.23 without (three waves per SIMD against four); the
// mixed-variant batch of lengths up to 16 KiB 2.40 ms against 2.52, although
// the mixed kernel then held two waves per SIMD instead of three (capping it at
// three spills); one-block messages are level either way.  With the pair and
// wide forms in them too, the hashing kernels hold 212 VGPRs (mixed), 189 and
// 185 (SHA3-224 and 256), 202 and 181 (SHAKE128 and 256), two waves per SIMD,
// and 164 and 146 (SHA3-384 and 512), three; without the prefetch 175 (mixed,
// two waves) and 132-153 (three).
// The chain of the longest message bounds a batch of uneven lengths, so the
// latency of each block matters more than the occupancy.
template <int V>
constexpr bool kPrefetch = true;

template <int V, bool PF = kPrefetch<V>>
__device__ __forceinline__ void sponge_hash(Lane (&A)[25], const uint8_t* msg, uint64_t len,
                                            int var, uint32_t* __restrict__ row) {
  using S = SpongeShape<V>;
  const int R = V == kMixed ? rate_bytes_rt(var) : S::kMaxRate;
  const int RW = R / 4;
  // blocks of the padded message: the 2 suffix bits and the pad fit after
  // any byte-aligned message, so nb = floor(L / R) + 1
  const uint64_t nb = len / static_cast<uint64_t>(R) + 1u;
  // block b's bytes into bc
  auto load = [&](BlockChunks<V>& bc, uint64_t b) {
    const uint64_t off = b * static_cast<uint64_t>(R);
    if (b + 1u == nb)
      load_block<V>(bc, msg + off, static_cast<uint32_t>(len - off));
    else
      load_whole_block<V>(bc, msg + off, R);
  };
#pragma unroll
  for (int k = 0; k < 25; ++k) A[k] = Lane{0u, 0u};
  BlockChunks<V> bc;
  if (PF) load(bc, 0u);
  for (uint64_t b = 0; b < nb; ++b) {
    const bool fin = b + 1u == nb;
    absorb_phase_begin();
    if (!PF) load(bc, b);
    uint32_t w[S::kMaxRateDw];
#pragma unroll
    for (int k = 0; k < S::kMaxRateDw; ++k) w[k] = chunk_dword<V>(bc, k);
    if (fin) {
      stage_block<V>(row, bc, static_cast<uint32_t>(len - b * static_cast<uint64_t>(R)), R, w);
      if (V == kMixed) {
#pragma unroll
        for (int k = 0; k < S::kMaxRateDw; ++k) w[k] = k < RW ? w[k] : 0u;
      }
    }
#pragma unroll
    for (int k = 0; k < S::kMaxRateDw; ++k) {
      if (k & 1)
        A[k >> 1].hi ^= w[k];
      else
        A[k >> 1].lo ^= w[k];
    }
    if (PF && !fin) load(bc, b + 1u);
    keccak_rounds_0_22_rolled(A);
    if (!fin || V >= kShake128) keccak_round(A, 23);
  }
  if (V < kShake128) keccak_round(A, 23);
}

// XOF squeeze (Section 3.2: the output is read r bits at a time, applying
// the permutation between reads, until out_len bytes are produced).  A holds
// the state after the last absorbed block's permutation.  Stores of 16 bytes
// at any alignment, then 4, then single bytes: each store instruction touches
// 64 separate lines, and with 4-byte (or, for an out_len or address that is no
// multiple of 4, 1-byte) stores their addresses took as long as the
// permutations (SHAKE128 of 65537 seeds to 1000 bytes: 122 us against 75).
template <int V>
__device__ __forceinline__ void squeeze_xof(Lane (&A)[25], uint8_t* out, uint64_t out_len) {
  constexpr int R = SpongeShape<V>::kMaxRate;
  for (uint64_t done = 0;;) {
#pragma unroll
    for (int k = 0; k < R / 4; k += 4) {
      const uint64_t at = done + 4u * k;
      if (at >= out_len) break;
      const Lane l0 = A[k / 2], l1 = A[k / 2 + 1 < 25 ? k / 2 + 1 : 24];
      const uint32_t v[4] = {l0.lo, l0.hi, l1.lo, l1.hi};
      if (k + 4 <= R / 4 && at + 16u <= out_len) {
        *reinterpret_cast<Words4*>(out + at) = Words4{v[0], v[1], v[2], v[3]};
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint64_t a4 = at + 4u * q;
          if (k + q >= R / 4 || a4 >= out_len) break;
          if (a4 + 4u <= out_len) {
            *reinterpret_cast<Word1*>(out + a4) = v[q];
          } else {
            for (int z = 0; z < 4 && a4 + z < out_len; ++z) out[a4 + z] = static_cast<uint8_t>(v[q] >> (8 * z));
          }
        }
      }
    }
    done += R;
    if (done >= out_len) break;
    keccak_rounds_0_22_rolled(A);
    keccak_round(A, 23);
  }
}

// Trunc_d of the squeezed state: the first D bytes are dwords 0..D/4-1 in
// lane order (lo, hi).  `out` must be 4-byte aligned.  In the mixed form every
// slot is 64 bytes, zero past the digest.
template <int V>
__device__ __forceinline__ void store_digest(uint8_t* out, const Lane (&A)[25], int var) {
  using S = SpongeShape<V>;
  uint32_t* o = reinterpret_cast<uint32_t*>(out);
  const int DW = V == kMixed ? digest_bytes_rt(var) / 4 : digest_bytes_of(V) / 4;
#pragma unroll
  for (int k = 0; k < S::kMaxDigestDw; ++k) {
    const uint32_t v = (k & 1) ? A[k >> 1].hi : A[k >> 1].lo;
    o[k] = k < DW ? v : 0u;
  }
}

}  // namespace kb
