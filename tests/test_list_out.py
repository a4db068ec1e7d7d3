"""The writer of a particle's neighbour list in the lane-per-particle list
build (csrc/list_out.h), compiled for the CPU: the stored words, the padding
and the count for lists up to twice the largest capacity, the most that a
lane can find, with word rows on both sides of the longest that 32-bit offsets
take, and of 2^24 bytes."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

PROGRAM = r"""
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <unistd.h>
#include <vector>
#define __device__
#define __forceinline__ inline
struct uint2 { uint32_t x, y; };
static int __popc(uint32_t v) { return __builtin_popcount(v); }
// v_perm_b32: byte k of the result is byte sel[k] of (hi, lo), 0 for 0x0c
static uint32_t __builtin_amdgcn_perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  const uint64_t v = (uint64_t)hi << 32 | lo;
  uint32_t r = 0;
  for (int k = 0; k < 4; ++k) {
    const uint32_t b = sel >> (8 * k) & 255;
    r |= b < 8 ? (uint32_t)(v >> (8 * b) & 255) << (8 * k) : 0;
  }
  return r;
}
#include "list_out.h"
static const mdpl::Compress pack = mdpl::compress_table();
static const uint16_t kPad = 0x2ffc;

// The list of slot s with `found` entries; every page touched must hold only
// the list's own words.
template <typename OFF>
static int check(int64_t stride, int64_t s, int found, int max_nb) {
  const int64_t pitch = 8 * stride;
  const uint32_t words = (max_nb + 3) / 4;
  const size_t page = 4096, bytes = ((size_t)words * pitch + page - 1) / page * page;
  char* list = (char*)mmap(nullptr, bytes, PROT_READ | PROT_WRITE,
                           MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (list == MAP_FAILED) { perror("mmap"); exit(2); }
  mdpl::ListOut<OFF> out{};
  out.at = (OFF)(8 * s);
  out.pitch = (OFF)pitch;
  out.room = (OFF)(words * pitch);
  out.list = list;
  std::vector<uint16_t> want;
  unsigned r = 12345u + found;
  while ((int)want.size() < found) {
    r = r * 1664525u + 1013904223u;
    uint32_t nib = r >> 28;
    while ((int)want.size() + __popc(nib) > found) nib &= nib - 1;
    uint16_t e[4];
    for (int k = 0; k < 4; ++k) {
      e[k] = (uint16_t)(4 * (1 + (want.size() + k) % 3000));
      if (nib >> k & 1) want.push_back(e[k]);
    }
    out.push4(nib, pack.sel[nib], (uint32_t)e[1] << 16 | e[0], (uint32_t)e[3] << 16 | e[2]);
  }
  const int got = out.finish((OFF)(8 * s), max_nb, kPad);
  int bad = got != found;
  const int kept = found < max_nb ? found : max_nb;
  std::vector<unsigned char> in(bytes / page);
  if (mincore(list, bytes, in.data())) { perror("mincore"); exit(2); }
  int64_t touched = 0;
  for (size_t p = 0; p < in.size(); ++p) touched += in[p] & 1;
  bad |= touched != (kept + 3) / 4;  // a page each: pitch is larger
  for (int w = 0; w < (kept + 3) / 4; ++w) {
    const size_t at = 8 * s + (size_t)w * pitch;
    const uint16_t* const q = (const uint16_t*)(list + at);
    for (int k = 0; k < 4; ++k) {
      const int m = 4 * w + k;
      bad |= q[k] != (m < kept ? want[m] : kPad);
    }
    const size_t p0 = at / page * page;
    for (size_t b = p0; b < p0 + page; b += 8)
      bad |= b != at && *(const uint64_t*)(list + b) != 0;
  }
  munmap(list, bytes);
  if (bad)
    printf("stride %lld slot %lld found %d max_nb %d: count %d, %lld pages\n", (long long)stride,
           (long long)s, found, max_nb, got, (long long)touched);
  return bad;
}

int main() {
  int bad = 0;
  for (int64_t stride : {(int64_t)1062912, (int64_t)1063168, (int64_t)2096896, (int64_t)2097152})
    for (int64_t s : {(int64_t)0, (int64_t)65536, stride - 1})
      for (int max_nb : {1024, 1021, 128, 6, 1})
        for (int found : {0, 1, 4, 127, 128, 129, 1020, 1021, 1022, 1023, 1024, 1025, 1028, 1031, 1040, 1708, 1990, mdpl::kListMost})
          bad += mdpl::list_offsets_32(stride * 8) ? check<uint32_t>(stride, s, found, max_nb)
                                        : check<uint64_t>(stride, s, found, max_nb);
  printf("%d wrong\n", bad);
  return bad != 0;
}
"""


def test_list_writer_on_the_cpu(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "list.cpp", tmp_path / "list"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_1704_03329_amd", "csrc")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", csrc, "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout[-3000:])
    assert r.returncode == 0, r.stdout[-3000:]
