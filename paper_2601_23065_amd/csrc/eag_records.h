// Gradient accumulators and per-hit gradient records of the adjoints.
// (Uses D3 of eag_device.h and HIP's device functions only, so that a test can
// compile it for the host with its own.)
#pragma once

namespace eag {

// Gradient accumulators: double precision in the workspace (component-major,
// pos[3] rot[4] scale[2] opacity albedo[3] radiance[3] = 16 rows of n), so
// that sums of many opposing contributions keep their small results; they
// are added to the caller's float arrays once at the end.
constexpr int GRAD_ROWS = 16;
struct GradPtrs {
  double* pos;
  double* rot;
  double* scale;
  double* opacity;
  double* albedo;
  double* radiance;
  int64_t n;
};

__device__ __forceinline__ void atomic_add3(double* base, int64_t n, int64_t i, D3 v) {
  atomicAdd(base + i, v.x);
  atomicAdd(base + n + i, v.y);
  atomicAdd(base + 2 * n + i, v.z);
}

constexpr int64_t REC_CHUNK = 1024;                   // slots a wave claims at a time
struct GradRecs {
  float* rec;                   // [n_chunks * REC_CHUNK][16] accumulator rows of each hit
  uint32_t* idx;                // surfel index of each record
  uint32_t* rank;               // rank of each record among its surfel's
  uint32_t* cnt;                // [n] records per surfel
  uint32_t* off;                // [n] exclusive scan of cnt
  uint32_t* order;              // slots grouped by surfel
  uint32_t* chunk_used;         // [n_chunks] slots used in each chunk of REC_CHUNK slots
  unsigned long long* chunk_next;   // chunks claimed (set by the launch)
  int64_t n_chunks;             // records: n_chunks * REC_CHUNK
  void* scan_tmp;
  size_t scan_bytes;
};
// Per-hit gradient records of both adjoint passes. Added with atomics, a
// pass is limited by their rate (13 to 16 per hit). Instead, each hit writes
// one record of the 16 accumulator rows (64 B: each term rounded to float,
// their sums taken in double, so a surfel's sum carries an error of about
// 2^-24 of the sum of its terms' magnitudes at most) to the next slot of its
// wave's current chunk of REC_CHUNK slots, and counts itself in a per-surfel
// counter. What the atomic returns is the record's rank among its surfel's; the
// lane stores it with its next record (or at the item's end), so it never waits
// for it, and the placement needs no atomics of its own. A wave claims a
// chunk from a global counter when the lanes of a call do not fit in its
// current one (one atomic per many hits) and records how much of the chunk it
// used; its cursor lives in LDS. After the pass, an exclusive scan of the
// counters and a placement pass group the slots by surfel, and one wave per
// surfel sums its records. Hits that find the chunks exhausted fall back to
// atomics, so any capacity is correct.
constexpr unsigned REC_NO_CHUNK = 0xffffffffu;   // none claimed yet
constexpr unsigned REC_SPENT = 0xfffffffeu;      // the chunks are exhausted: atomics from here on
// A lane's last record: its slot (or NO_SLOT) and, once the atomic has returned, its rank.
constexpr uint32_t NO_SLOT = 0xffffffffu;
struct LastRec {
  uint32_t slot = NO_SLOT, rank = 0;
};
__device__ __forceinline__ void store_rank(const GradRecs& gr, LastRec& last) {
  if (last.slot != NO_SLOT) gr.rank[last.slot] = last.rank;
  last.slot = NO_SLOT;
}
// A wave's cursor: wcur[0] the slots used in its chunk, wcur[1] the chunk (or
// none). The lanes take turns as the one that moves it, so every access is
// volatile: a plain one may be answered from what the same lane wrote last, and
// then records share slots, or a chunk's use is recorded short and its surfels'
// ranges in `order` keep what was there before.
__device__ __forceinline__ void records_begin(unsigned* wcur) {
  volatile unsigned* const wc = wcur;
  if ((threadIdx.x & 63) == 0) {
    wc[0] = 0u;
    wc[1] = REC_NO_CHUNK;
  }
}
__device__ __forceinline__ void records_end(const GradRecs& gr, unsigned* wcur) {
  volatile unsigned* const wc = wcur;
  if ((threadIdx.x & 63) == 0) {
    const unsigned ch = wc[1];
    if (ch < (unsigned)gr.n_chunks) gr.chunk_used[ch] = wc[0];
  }
}
__device__ __forceinline__ void emit_record(const GradRecs& gr, const GradPtrs& gp, unsigned* wcur, LastRec& last,
                                            uint32_t idx, const double (&v)[GRAD_ROWS]) {
  store_rank(gr, last);
  const uint64_t act = __ballot(1);
  const int lane = (int)(threadIdx.x & 63);
  const int leader = __ffsll((unsigned long long)act) - 1;
  const unsigned k = (unsigned)__popcll(act);
  unsigned base = 0, chunk = REC_NO_CHUNK;
  if (lane == leader) {
    volatile unsigned* const wc = wcur;
    unsigned cur = wc[0], ch = wc[1];
    if (ch == REC_NO_CHUNK || (ch != REC_SPENT && cur + k > (unsigned)REC_CHUNK)) {
      if (ch < (unsigned)gr.n_chunks) gr.chunk_used[ch] = cur;
      const unsigned long long c = atomicAdd(gr.chunk_next, 1ull);
      ch = c < (unsigned long long)gr.n_chunks ? (unsigned)c : REC_SPENT;
      cur = 0;
    }
    base = cur;
    chunk = ch;
    wc[0] = cur + k;
    wc[1] = ch;
  }
  base = __shfl(base, leader);
  chunk = __shfl(chunk, leader);
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  if (chunk < (unsigned)gr.n_chunks) {
    const int64_t slot = (int64_t)chunk * REC_CHUNK + base + __popcll(act & below);
    float4* dst = reinterpret_cast<float4*>(gr.rec + slot * GRAD_ROWS);
#pragma unroll
    for (int q = 0; q < GRAD_ROWS / 4; ++q)
      dst[q] = make_float4((float)v[4 * q], (float)v[4 * q + 1], (float)v[4 * q + 2], (float)v[4 * q + 3]);
    gr.idx[slot] = idx;
    last.slot = (uint32_t)slot;   // (at most 2^27 records)
    last.rank = atomicAdd(gr.cnt + idx, 1u);
  } else {
    const int64_t n = gp.n;
    atomic_add3(gp.pos, n, idx, d3(v[0], v[1], v[2]));
#pragma unroll
    for (int k = 0; k < 4; ++k) atomicAdd(gp.rot + k * n + idx, v[3 + k]);
    atomicAdd(gp.scale + idx, v[7]);
    atomicAdd(gp.scale + n + idx, v[8]);
    atomicAdd(gp.opacity + idx, v[9]);
    atomic_add3(gp.albedo, n, idx, d3(v[10], v[11], v[12]));
    atomic_add3(gp.radiance, n, idx, d3(v[13], v[14], v[15]));
  }
}

// Every used slot of the claimed chunks goes to its rank in its surfel's range
// [off[i], off[i] + cnt[i]) of order. Blocks stride over the claimed chunks only.
__device__ __forceinline__ void place_records(const GradRecs& gr) {
  const unsigned long long claimed = *gr.chunk_next;
  const int64_t nc = claimed < (unsigned long long)gr.n_chunks ? (int64_t)claimed : gr.n_chunks;
  for (int64_t ch = blockIdx.x; ch < nc; ch += gridDim.x) {
    const uint32_t used = gr.chunk_used[ch];
    const int64_t s0 = ch * REC_CHUNK;
    for (uint32_t j = threadIdx.x; j < used; j += blockDim.x)
      gr.order[gr.off[gr.idx[s0 + j]] + gr.rank[s0 + j]] = (uint32_t)(s0 + j);
  }
}

}  // namespace eag
