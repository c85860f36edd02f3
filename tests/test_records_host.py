"""The adjoints' gradient records on the CPU: the library's own code that
claims slots, keeps ranks and places records by surfel (eag_records.h),
compiled for the host with a wave of 64 fibres in place of the GPU's lanes.
Every access is checked against its array, and the records and fallback
atomics together have to add up to what was emitted, whatever the capacity."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2601_23065_amd import build

SHIM = r"""
#include <ucontext.h>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>
#define __device__
#define __host__
#define __forceinline__ inline
struct float4 { float x, y, z, w; };
static float4 make_float4(float x, float y, float z, float w) { return float4{x, y, z, w}; }
struct Dim { unsigned x; };
static Dim threadIdx, blockIdx, gridDim, blockDim;
namespace eag {
struct D3 { double x, y, z; };
static D3 d3(double x, double y, double z) { return D3{x, y, z}; }
}

// A wave: the lanes that make a call run as fibres and meet at every wave-wide
// operation, whose operands they leave in `arg`.
static const int LANES = 64;
static ucontext_t sched, fibre[LANES];
static char stacks[LANES][1 << 16];
static bool live[LANES];
static uint64_t arg[LANES];
static int at;
static void meet(uint64_t v) {
  const int me = at;
  arg[me] = v;
  swapcontext(&fibre[me], &sched);
  at = me;
  threadIdx.x = me;
}
static uint64_t __ballot(int p) {
  meet(p ? 1 : 0);
  uint64_t m = 0;
  for (int l = 0; l < LANES; ++l) m |= live[l] && arg[l] ? 1ull << l : 0;
  return m;
}
static unsigned __shfl(unsigned v, int from) {
  meet(v);
  if (!live[from]) abort();   // an inactive lane has nothing to read
  return (unsigned)arg[from];
}
static int __ffsll(unsigned long long m) { return __builtin_ffsll((long long)m); }
static int __popcll(unsigned long long m) { return __builtin_popcountll(m); }

// Every array the code is given, and checked accesses to them.
struct Span { char* a; size_t bytes; };
static std::vector<Span> spans;
static long bad;
static bool inside(const void* p, size_t bytes) {
  for (const Span& s : spans)
    if ((char*)p >= s.a && (char*)p + bytes <= s.a + s.bytes) return true;
  ++bad;
  return false;
}
template <class T> static T atomicAdd(T* p, T v) {
  static T none;
  if (!inside(p, sizeof(T))) return none;
  const T old = *p;
  *p += v;
  return old;
}

#include "eag_records.h"
using namespace eag;

static GradRecs gr;
static GradPtrs gp;
static unsigned (*wcur)[2];
static LastRec last[16][LANES];
static int wave, call_idx[LANES];
static double call_v[LANES][GRAD_ROWS];
static void lane_main(int l) {
  at = l;
  threadIdx.x = l;
  emit_record(gr, gp, wcur[wave], last[wave][l], (uint32_t)call_idx[l], call_v[l]);
  live[l] = false;
}
// Guard bytes behind every array: what an unchecked store beyond it changes.
template <class T> static T* make(size_t n) {
  T* p = (T*)malloc(n * sizeof(T) + 256);
  for (size_t i = 0; i < n * sizeof(T) + 256; ++i) ((unsigned char*)p)[i] = 0xa5;
  spans.push_back(Span{(char*)p, n * sizeof(T)});
  return p;
}
static long guards() {
  long k = 0;
  for (const Span& s : spans)
    for (int i = 0; i < 256; ++i) k += (unsigned char)s.a[s.bytes + i] != 0xa5;
  return k;
}
// n_calls calls, call c by the lanes of mask[c] in wave wv[c], lane l with
// surfel idx[c][l] and rows v[c][l]. sums: [n][16]. Returns the number of faults.
extern "C" long run(int n, int n_chunks, int n_waves, int n_calls, const int* wv, const uint64_t* mask,
                    const int* idx, const double* v, double* sums, long* placed) {
  const size_t cap = (size_t)n_chunks * REC_CHUNK;
  spans.clear();
  bad = 0;
  gr = GradRecs{};
  gr.n_chunks = n_chunks;
  gr.rec = make<float>(cap * GRAD_ROWS);
  gr.idx = make<uint32_t>(cap);
  gr.rank = make<uint32_t>(cap);
  gr.order = make<uint32_t>(cap);
  gr.cnt = make<uint32_t>(n);
  gr.off = make<uint32_t>(n);
  gr.chunk_used = make<uint32_t>(n_chunks);
  gr.chunk_next = make<unsigned long long>(1);
  double* acc = make<double>((size_t)n * GRAD_ROWS);
  gp = GradPtrs{acc, acc + 3 * n, acc + 7 * n, acc + 9 * n, acc + 10 * n, acc + 13 * n, n};
  for (int i = 0; i < n; ++i) gr.cnt[i] = 0;
  for (int i = 0; i < n_chunks; ++i) gr.chunk_used[i] = 0;
  for (int i = 0; i < n * GRAD_ROWS; ++i) acc[i] = 0.0;
  *gr.chunk_next = 0;
  wcur = (unsigned(*)[2])make<unsigned>(2 * n_waves);
  for (wave = 0; wave < n_waves; ++wave)
    for (int l = 0; l < LANES; ++l) {
      last[wave][l] = LastRec();
      threadIdx.x = l;
      records_begin(wcur[wave]);
    }
  for (int c = 0; c < n_calls; ++c) {
    wave = wv[c];
    for (int l = 0; l < LANES; ++l) {
      live[l] = mask[c] >> l & 1;
      call_idx[l] = idx[c * LANES + l];
      for (int k = 0; k < GRAD_ROWS; ++k) call_v[l][k] = v[((size_t)c * LANES + l) * GRAD_ROWS + k];
      if (!live[l]) continue;
      getcontext(&fibre[l]);
      fibre[l].uc_stack.ss_sp = stacks[l];
      fibre[l].uc_stack.ss_size = sizeof(stacks[l]);
      fibre[l].uc_link = &sched;
      makecontext(&fibre[l], (void (*)())lane_main, 1, l);
    }
    for (bool any = true; any;) {
      // (a lane's operand is read by the others before any of them goes on)
      uint64_t now[LANES];
      any = false;
      bool on[LANES];
      for (int l = 0; l < LANES; ++l) on[l] = live[l];
      for (int l = 0; l < LANES; ++l) now[l] = arg[l];
      uint64_t next[LANES];
      for (int l = 0; l < LANES; ++l) {
        if (!on[l]) continue;
        for (int q = 0; q < LANES; ++q) {
          arg[q] = now[q];
          live[q] = on[q];
        }
        swapcontext(&sched, &fibre[l]);
        next[l] = arg[l];
        on[l] = live[l] ? on[l] : true;
        if (live[l]) any = true;
        else next[l] = ~0ull;
      }
      for (int l = 0; l < LANES; ++l) {
        if (!on[l]) continue;
        arg[l] = next[l];
        live[l] = any;
      }
    }
  }
  for (wave = 0; wave < n_waves; ++wave)
    for (int l = 0; l < LANES; ++l) {
      store_rank(gr, last[wave][l]);
      threadIdx.x = l;
      records_end(gr, wcur[wave]);
    }
  // what the placement will read and write
  const int64_t claimed = (int64_t)*gr.chunk_next < n_chunks ? (int64_t)*gr.chunk_next : n_chunks;
  uint32_t total = 0;
  for (int i = 0; i < n; ++i) {
    gr.off[i] = total;
    total += gr.cnt[i];
  }
  long used = 0;
  if (total > cap) ++bad;
  for (int64_t ch = 0; ch < claimed; ++ch) {
    if (gr.chunk_used[ch] > REC_CHUNK) { ++bad; continue; }
    for (uint32_t j = 0; j < gr.chunk_used[ch]; ++j, ++used) {
      const size_t s = ch * REC_CHUNK + j;
      if (gr.idx[s] >= (uint32_t)n || gr.rank[s] >= gr.cnt[gr.idx[s]]) ++bad;
    }
  }
  if (used != (long)total) ++bad;
  if (bad) return bad;
  for (size_t i = 0; i < cap; ++i) gr.order[i] = 0xffffffffu;
  gridDim.x = 3;
  blockDim.x = 256;
  for (blockIdx.x = 0; blockIdx.x < 3; ++blockIdx.x)
    for (threadIdx.x = 0; threadIdx.x < 256; ++threadIdx.x) place_records(gr);
  for (int i = 0; i < n; ++i)
    for (uint32_t j = 0; j < gr.cnt[i]; ++j) {
      const uint32_t s = gr.order[gr.off[i] + j];
      if (s >= cap || gr.idx[s] != (uint32_t)i) { ++bad; continue; }
      for (int k = 0; k < GRAD_ROWS; ++k) acc[(size_t)k * n + i] += gr.rec[(size_t)s * GRAD_ROWS + k];
    }
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < GRAD_ROWS; ++k) sums[(size_t)i * GRAD_ROWS + k] = acc[(size_t)k * n + i];
  *placed = used;
  bad += guards();
  for (const Span& s : spans) free(s.a);
  return bad;
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("records")
    src, lib = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", build.CSRC, src, "-o", lib], check=True,
                   capture_output=True)
    so = ctypes.CDLL(lib)
    so.run.restype = ctypes.c_long

    def call(n, chunks, waves, wv, mask, idx, v):
        sums, placed = np.zeros((n, 16)), ctypes.c_long(0)
        a = [np.ascontiguousarray(wv, np.int32), np.ascontiguousarray(mask, np.uint64),
             np.ascontiguousarray(idx, np.int32), np.ascontiguousarray(v, np.float64), sums]
        p = [x.ctypes.data_as(ctypes.c_void_p) for x in a]
        faults = so.run(n, chunks, waves, len(wv), *p, ctypes.byref(placed))
        return faults, sums, placed.value
    return call


# rows that the emulated values are multiples of 2^-8 below 2^8 in: exact in float32 and in every sum
@pytest.mark.parametrize("chunks", [1, 2, 5, 64])
@pytest.mark.parametrize("n,waves,lanes", [(1, 1, 64), (7, 3, 64), (300, 8, 64), (300, 16, 5), (40, 4, 1)])
def test_records_of_any_capacity(run, n, waves, lanes, chunks):
    rng = np.random.default_rng(n * 100 + chunks)
    calls = 400
    wv = rng.integers(0, waves, calls)
    bits = rng.random((calls, 64)) < rng.choice([0.02, 0.5, 1.0], calls)[:, None]
    bits[:, lanes:] = False
    bits[np.arange(calls), rng.integers(0, lanes, calls)] = True
    mask = (bits.astype(np.uint64) << np.arange(64, dtype=np.uint64)).sum(1, dtype=np.uint64)
    idx = rng.integers(0, n, (calls, 64))
    v = np.round(rng.uniform(-256, 256, (calls, 64, 16)) * 256) / 256
    faults, sums, placed = run(n, chunks, waves, wv, mask, idx, v)
    assert faults == 0
    want = np.zeros((n, 16))
    np.add.at(want, idx[bits], v[bits])
    assert np.array_equal(sums, want)
    assert placed <= min(chunks * 1024, int(bits.sum()))
    if chunks >= waves + bits.sum() // 960:   # (a chunk is left with at most 63 slots unused)
        assert placed == bits.sum()
