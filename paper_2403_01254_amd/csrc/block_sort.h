// Stable LSD radix sort inside one workgroup, and the wave and block scans that it and the tiled radix sort
// share.
//
// Here and in the other sources, helpers that take pointers or references to LDS are inlined by force: in a function
// of its own, LDS is reached through generic pointers, and the constant part of an index can be folded into the
// instruction so that the base lies before the LDS aperture, which faults.
#pragma once

#include "rkhsba_device.h"

namespace rkhsba {

// Orders LDS accesses between the lanes of one wavefront: its LDS operations are carried out in issue order,
// so only the compiler must not move them across this point.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive add-scan over the wavefront's 64 lanes in DPP steps (row shifts, then the last lane of a row added
// to the rows after it).
__device__ inline uint32_t wave_inclusive_scan(uint32_t v) {
  int m = (int)v;
  m += __builtin_amdgcn_update_dpp(0, m, 0x111, 0xf, 0xf, true);   // row_shr:1
  m += __builtin_amdgcn_update_dpp(0, m, 0x112, 0xf, 0xf, true);   // row_shr:2
  m += __builtin_amdgcn_update_dpp(0, m, 0x114, 0xf, 0xf, true);   // row_shr:4
  m += __builtin_amdgcn_update_dpp(0, m, 0x118, 0xf, 0xf, true);   // row_shr:8
  m += __builtin_amdgcn_update_dpp(0, m, 0x142, 0xa, 0xf, false);  // row_bcast:15
  m += __builtin_amdgcn_update_dpp(0, m, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return (uint32_t)m;
}

// Exclusive scan of the 256 digit totals held by threads 0..255 (four wavefronts); every thread of the block
// takes part in the barrier.  wtot: 4 words of LDS.
__device__ __forceinline__ uint32_t digit_exclusive_scan(uint32_t v, uint32_t* wtot) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint32_t incl = wave_inclusive_scan(v);
  if (t < 256 && lane == 63) wtot[w] = incl;
  __syncthreads();
  uint32_t base = 0;
  if (t < 256)
    for (int k = 0; k < w; ++k) base += wtot[k];
  return base + incl - v;
}

// One digit pass' ranks inside a wavefront that holds IPT * 64 consecutive items in rounds of 64: rank[r] = how
// many of the wavefront's earlier items (earlier rounds, or lower lanes of the round) have item r's digit;
// cnt[256] (LDS, this wavefront's own) ends with the wavefront's digit counts.  Lanes sharing a digit find each
// other with one ballot per digit bit, so a round costs no LDS atomics and no barrier.
template <int IPT>
__device__ __forceinline__ void wave_digit_ranks(const uint32_t (&digit)[IPT], const bool (&valid)[IPT], uint32_t* cnt,
                                        uint32_t (&rank)[IPT]) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int k = 0; k < 4; ++k) cnt[lane + 64 * k] = 0u;
  wave_sync();
#pragma unroll
  for (int r = 0; r < IPT; ++r) {
    const uint32_t d = digit[r];
    uint64_t peers = __builtin_amdgcn_ballot_w64(valid[r]);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool b = ((d >> bit) & 1u) != 0u;
      const uint64_t bl = __builtin_amdgcn_ballot_w64(b);
      peers &= b ? bl : ~bl;
    }
    const uint32_t before = (uint32_t)__popcll(peers & lt);
    const uint32_t old = cnt[d];
    rank[r] = old + before;
    wave_sync();
    if (valid[r] && before == 0u) cnt[d] = old + (uint32_t)__popcll(peers);
    wave_sync();
  }
}

// Sorts count <= NT * IPT (key, local index) items of one workgroup of NT threads by key bits [0, bits), stably.
// key[r] of thread (wavefront w, lane) is item w * 64 * IPT + 64 r + lane; items from `count` on are ignored.
// On return S.val[i] holds the local index of the i-th item in order, and S.key[i] its key; all threads may
// read them (a barrier has passed).
template <int NT, int IPT>
struct BlockSort {
  static constexpr int kItems = NT * IPT;
  static constexpr int kWaves = NT / 64;
  static_assert(kItems <= 65536 && NT >= 256, "16-bit local indices; one thread per digit");
  struct Shared {
    uint32_t key[kItems];
    uint16_t val[kItems];
    uint32_t cnt[kWaves][256];
    uint32_t dig[256];
    uint32_t wtot[4];
  };
  __device__ static __forceinline__ void sort(uint32_t (&key)[IPT], int count, int bits, Shared& S) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int base = w * 64 * IPT + lane;
    uint32_t idx[IPT];
    bool valid[IPT];
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
      idx[r] = (uint32_t)(base + 64 * r);
      valid[r] = base + 64 * r < count;
    }
    for (int shift = 0; shift < bits; shift += 8) {
      uint32_t d[IPT], rank[IPT];
#pragma unroll
      for (int r = 0; r < IPT; ++r) d[r] = (key[r] >> shift) & 0xffu;
      wave_digit_ranks<IPT>(d, valid, S.cnt[w], rank);
      __syncthreads();
      // thread d: the wavefronts' offsets of digit d, and its total
      uint32_t total = 0;
      if (t < 256)
        for (int k = 0; k < kWaves; ++k) {
          const uint32_t c = S.cnt[k][t];
          S.cnt[k][t] = total;
          total += c;
        }
      const uint32_t ex = digit_exclusive_scan(total, S.wtot);
      if (t < 256) S.dig[t] = ex;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < IPT; ++r)
        if (valid[r]) {
          const uint32_t p = S.dig[d[r]] + S.cnt[w][d[r]] + rank[r];
          S.key[p] = key[r];
          S.val[p] = (uint16_t)idx[r];
        }
      __syncthreads();
      if (shift + 8 < bits) {
#pragma unroll
        for (int r = 0; r < IPT; ++r)
          if (valid[r]) {
            key[r] = S.key[base + 64 * r];
            idx[r] = S.val[base + 64 * r];
          }
        // (the next pass writes S.key and S.val only after two more barriers)
      }
    }
  }
};

}  // namespace rkhsba
