// The neighbour list of a particle as one lane of the list build writes it.
// No HIP header is needed: a test compiles this file for the CPU.
#pragma once

#include <stdint.h>

namespace mdpl {

// A list as it grows: its newest entries, up to three, in a 64-bit word that
// is stored when it is full.  Four positions are appended at a time, without
// branches: their accepted entries are moved together by byte permutations
// from a table, shifted behind those held, and what does not fit starts the
// next word.
struct Compress {
  uint2 sel[16];  // per nibble of decisions: selectors of entries 0, 1 and 2, 3
};
constexpr Compress compress_table() {
  Compress t{};
  for (unsigned nib = 0; nib < 16; ++nib) {
    uint32_t sel[2] = {0x0c0c0c0cu, 0x0c0c0c0cu};  // zero bytes
    for (unsigned j = 0, m = 0; j < 4; ++j)
      if (nib >> j & 1) {
        sel[m / 2] = m % 2 ? (sel[m / 2] & 0xffffu) | (0x0100u + 0x0202u * j) << 16
                           : (sel[m / 2] & 0xffff0000u) | (0x0100u + 0x0202u * j);
        ++m;
      }
    t.sel[nib].x = sel[0];
    t.sel[nib].y = sel[1];
  }
  return t;
}

// The most entries a lane can find: its nine rows are kListRow candidates at
// most.  A list holds fewer; those past its capacity are counted, not stored.
constexpr int kListRow = 224, kListMost = 9 * kListRow;
// Whether 32 bits hold the offset of every word that a lane may come to, the
// words past the capacity included, whose offsets tell them from the others
// (N up to about 1.06 * 10^6).
constexpr bool list_offsets_32(int64_t pitch) {
  return pitch * (kListMost / 4 + 1) < ((int64_t)1 << 32);
}

// OFF: unsigned of the width that the offsets need.
template <typename OFF>
struct ListOut {
  uint64_t acc;
  uint32_t held;      // entries in acc
  OFF at;             // where the next word goes
  OFF pitch, room;    // bytes between words; those of all words of all lists
  char* list;         // of the first slot
  // e01, e23: entries of the four positions, 16 bits each
  __device__ __forceinline__ void push4(uint32_t nib, uint2 sel, uint32_t e01, uint32_t e23) {
    const uint64_t c = (uint64_t)__builtin_amdgcn_perm(e23, e01, sel.y) << 32 |
                       __builtin_amdgcn_perm(e23, e01, sel.x);
    const uint32_t sh = held << 4;
    acc |= c << sh;
    const uint64_t rest = (c >> (48 - sh)) >> 16;
    const uint32_t sum = held + __popc(nib);
    const bool full = sum > 3;
    if (full && at < room) *(uint64_t*)(list + at) = acc;
    at += full ? pitch : 0;
    acc = full ? rest : acc;
    held = sum & 3;
  }
  // Pads the last word; returns the entries found.  `first`: where the list
  // begins; a list cut at its capacity is padded there.
  __device__ __forceinline__ int finish(OFF first, int max_nb, uint32_t pad) {
    const int m = 4 * (int)((double)(at - first) / (double)pitch + 0.5) + (int)held;
    if (held && at < room)
      *(uint64_t*)(list + at) = acc | (0x0001000100010001ull * pad) << (16 * held);
    if (m > max_nb && (max_nb & 3)) {
      uint16_t* last = (uint16_t*)(list + first + (OFF)(max_nb >> 2) * pitch);
      for (int k = max_nb & 3; k < 4; ++k) last[k] = (uint16_t)pad;
    }
    return m;
  }
};

}  // namespace mdpl
