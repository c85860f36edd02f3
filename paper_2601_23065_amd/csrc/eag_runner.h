// Persistent segment runner: the per-lane state machine that drives the
// segment engine (eag_device.h) over a stream of work items.
//
// Each lane of a wave64 carries one work item and runs its segments as a
// small state machine over the engine's steps: start a k-buffer round,
// traverse, blend the round's hits, finish the segment. Lanes advance
// independently, so a lane whose segment needs one round does not wait for a
// neighbour that needs four:
//   * idle lanes are refilled, at first with items that are the wave's own,
//     then from a global work counter (the wave ballots its idle lanes, one
//     lane claims that many work items with a single atomic, and each idle
//     lane takes base + its rank among them);
//   * lanes whose round needs the BVH traverse together; the wave leaves the
//     traversal loop once RUN_BLEND_BATCH lanes wait to blend (or no lane
//     traverses), blends those lanes' rounds, finishes the segments that have
//     ended (once FINISH_BATCH of them have, or nothing else is left to do),
//     starts the next rounds or segments, and resumes: traversal state stays
//     in registers and LDS.
// A wave exits when the items are exhausted and all its lanes are idle.
//
// The work comes from a source object, one per lane:
//   bool start(int64_t item, TraceCtx& tcl, D3& O, D3& W)
//       set up work item `item` (0 <= item < n_work); true with the first
//       segment's ray in (O, W) (and tcl.attrs set), false when the item
//       needs no tracing (the source then writes its own result);
//   bool finish(const Seg<DACC>& s, D3& O, D3& W)
//       the lane's segment has ended; true with the next segment's ray;
//   static constexpr bool kHits: whether it has
//   void operator()(const Record&, const Attr&, double t, double om,
//                   double w, double T_before, D3 O, D3 W)
//       called for every blended hit, in blending order (om = 1 - alpha).
#pragma once

#include "eag_device.h"

namespace eag {

// Lanes of a full wave waiting to blend that end a traversal stretch, and leaves
// each traversing lane waits for before a leaf phase starts. With the loads
// overlapped, bigger batches pay: 20 to 24 lanes and one leaf to two took the
// single-bounce step from 25.2 to 24.7 ms and baking from 13.4 to 13.1 ms, path
// tracing 139.7 to 140.1 ms (28 lanes or five leaves cost it 1%).
constexpr int RUN_BLEND_BATCH = 24;
constexpr int RUN_LEAVES = 2;
// Lanes with an ended segment that the source finishes together: its work (a
// bounce, a light sample) runs for few lanes otherwise. 1, 8, 16 and 24 lanes:
// emitter sampling 24.5, 24.1, 24.0 and 24.3 ms, path tracing 140.4, 140.0, 142.3
// and 146.7.
constexpr int FINISH_BATCH = 8;
// Runner kernels launch this many TRACE_BLOCK-thread blocks per CU: their
// LDS (stack and postponed leaves, 56 KB per block) admits two per CU, and
// the per-lane hit list is sized for exactly this grid.
constexpr int RUN_BLOCKS_PER_CU = 2;

// Per-lane statistics, added to a device array of 6 counters at the end:
// segments, items started, k-buffer rounds, candidate tests, blended hits,
// BVH nodes visited. Kept in 32 bits (registers are the runner's limit): a
// lane would need over 10^7 segments in one launch (about 10^12 segments
// over the grid, hours of tracing) to overflow one.
struct RunStats {
  uint32_t segments = 0, items = 0, rounds = 0, tests = 0, hits = 0, visits = 0;
  __device__ __forceinline__ void flush(unsigned long long* c) {
    atomicAdd(&c[0], (unsigned long long)segments);
    atomicAdd(&c[1], (unsigned long long)items);
    atomicAdd(&c[2], (unsigned long long)rounds);
    atomicAdd(&c[3], (unsigned long long)tests);
    atomicAdd(&c[4], (unsigned long long)hits);
    atomicAdd(&c[5], (unsigned long long)visits);
    segments = items = rounds = tests = hits = visits = 0;
  }
};

// A source that walks a tree of its own inside finish() (a light pdf, say)
// may declare a member `int* lds_stack`: it receives the lane's column of the
// traversal stack in LDS (entry i at lds_stack[i * TRACE_BLOCK], STACK_LDS
// entries), which is empty whenever finish() runs.
template <class Src>
__device__ __forceinline__ auto bind_lds_stack(Src& src, int* col, int) -> decltype(src.lds_stack = col, void()) {
  src.lds_stack = col;
}
template <class Src>
__device__ __forceinline__ void bind_lds_stack(Src&, int*, long) {}

// A wave's claims of work items. Its first ones are its own by its index
// (per_wave of them), the others come from the global counter, until that is
// past the end. Atomics on one address take 10 ns each, whoever makes them: with
// the first claims among them, and those of lanes that had found the counter at
// its end before, the counter alone set the time of short launches (Stage-0
// images of 64x64 pixels in a 100,000-surfel room 218 us, now 182; of 300x300 in
// a sparse room of 1000 surfels, where the rays themselves take little, 132, now
// 111).
struct Claims {
  unsigned long long* counter;
  int64_t n_work, own, shared;   // own: the wave's own first item; shared: the counter's
  bool first = true, exhausted = false;

  __device__ __forceinline__ Claims(unsigned long long* c, int64_t n, int per_wave) : counter(c), n_work(n) {
    // (the wave's index in a scalar register, and all that follows from it)
    const int wave = (int)blockIdx.x * (TRACE_BLOCK / 64) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    own = (int64_t)wave * per_wave;
    shared = (int64_t)gridDim.x * (TRACE_BLOCK / 64) * per_wave;
  }

  // The first of popc(m) items for the lanes of m (all lanes of the wave call
  // it, m not empty, per_wave of them the first time, and never once exhausted;
  // items at n_work or beyond do not exist).
  __device__ __forceinline__ int64_t take(uint64_t m) {
    if (first) {
      first = false;
      exhausted = shared >= n_work;
      return own;
    }
    const int leader = __ffsll((unsigned long long)m) - 1;
    unsigned long long c = 0;
    if ((int)(threadIdx.x & 63) == leader) c = atomicAdd(counter, (unsigned long long)__popcll(m));
    const int64_t base = shared + (int64_t)__shfl(c, leader);
    exhausted = base + (int64_t)__popcll(m) >= n_work;
    return base;
  }
};

// STATS: the counters are written (counters may not be null then).
template <int QMODE, bool DACC, bool STATS, class Src>
__device__ __forceinline__ void run_segments(const TraceCtx& tc, Src& src, unsigned long long* work_counter,
                                             int64_t n_work, uint64_t* hitlist, unsigned long long* counters) {
  enum { ST_IDLE = 0, ST_ROUND = 1, ST_TRAV = 2, ST_BLEND = 3, ST_DONE = 4 };
  __shared__ int s_stack[STACK_LDS * TRACE_BLOCK];
  __shared__ int s_pend[PEND * TRACE_BLOCK];
  int s_ovf[STACK_OVF];
  TravStack st;
  st.lds = s_stack + threadIdx.x;
  st.ovf = s_ovf;
  st.sp = 0;
  bind_lds_stack(src, st.lds, 0);
  int* const pend = s_pend + threadIdx.x;
  const int lane = (int)(threadIdx.x & 63);
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  TraceCtx tcl = tc;
  tcl.hl = hitlist;
  tcl.hl_at = (blockIdx.x * TRACE_BLOCK + threadIdx.x) * HL_CAP;
  tcl.hl_bytes = gridDim.x * TRACE_BLOCK * HL_CAP * 8u;   // (256 MiB on 256 CUs)

  // thresholds in lanes, scaled to the lanes that take work (all of them with at
  // most 2^10 surfels, where rays are alike and spreading them only adds waves:
  // 65,536 paths through 1000 layers 2.54 ms with 32 lanes a wave, 2.10 with 64,
  // in a cloud of 1000 surfels 0.57 and 0.49)
  const int lanes = tc.idx_bits <= 10 ? 64 : lanes_per_wave(n_work, (int64_t)gridDim.x * (TRACE_BLOCK / 64));
  const int blend_batch = (RUN_BLEND_BATCH * lanes + 63) / 64;
  const int leaf_min = (LEAF_MIN_LANES * lanes + 63) / 64;
  const int finish_batch = (FINISH_BATCH * lanes + 63) / 64;

  int stage = ST_IDLE;
  SegStats<DACC, STATS, true> s;
  seg_begin(s, d3(0.0, 0.0, 0.0), d3(0.0, 0.0, 1.0));
  Round r;
  r.cnt = 0;
  r.trav = false;
  r.np = 0;
  RunStats rs;
  D3 O = d3(0.0, 0.0, 0.0), W = d3(0.0, 0.0, 1.0);   // the next segment's ray, from the source

  Claims claims(work_counter, n_work, lanes);
  while (true) {
    // ---- refill idle lanes
    const bool need = stage == ST_IDLE && lane < lanes && !claims.exhausted;
    const uint64_t idle = __ballot(need);
    if (idle) {
      const int64_t base = claims.take(idle);
      if (need) {
        const int64_t wid = base + __popcll(idle & lt_mask);
        if (wid < n_work && src.start(wid, tcl, O, W)) {
          seg_begin(s, O, W);
          stage = ST_ROUND;
          if constexpr (STATS) {
            ++rs.items;
            ++rs.segments;
          }
        }
      }
    }
    // Every lane idle: stop once the items are exhausted, else claim again
    // (a claim can hold only items that need no tracing).
    if (__ballot(stage != ST_IDLE) == 0) {
      if (claims.exhausted) break;
      continue;
    }

    // ---- start rounds
    if (stage == ST_ROUND) stage = round_begin(tcl, s, r, st, pend) ? ST_TRAV : ST_BLEND;

    // ---- traverse until enough lanes wait to blend
    while (true) {
      if (stage == ST_TRAV) {
        while (r.trav && r.np <= PEND - 4) {
          node_visit(tcl, s, r, st, pend);
          if (__all(r.np >= RUN_LEAVES || !r.trav)) break;
        }
        leaf_phase(tcl, s, r, pend, leaf_min);
        if (!r.trav) {
          round_end_traversal(tcl, s, r);
          stage = ST_BLEND;
        }
      }
      if (__ballot(stage == ST_TRAV) == 0 || __popcll(__ballot(stage == ST_BLEND)) >= blend_batch) break;
    }

    // ---- blend
    if (stage == ST_BLEND) {
      blend_round<QMODE>(tcl, s, r, src, nullptr, 0);
      stage = s.done ? ST_DONE : ST_ROUND;
    }

    // ---- finish ended segments, once enough lanes have one (or nothing else is left to do)
    if (__popcll(__ballot(stage == ST_DONE)) >= finish_batch || __ballot(stage == ST_ROUND || stage == ST_TRAV) == 0) {
      if (stage == ST_DONE) {
        if constexpr (STATS) {
          rs.rounds += s.rounds;
          rs.tests += s.tests;
          rs.hits += s.nhits;
          rs.visits += s.visits;
        }
        if (src.finish(s, O, W)) {
          seg_begin(s, O, W);
          stage = ST_ROUND;
          if constexpr (STATS) ++rs.segments;
        } else {
          stage = ST_IDLE;
        }
      }
    }
  }
  if constexpr (STATS) rs.flush(counters);
}

// The same work by groups of lanes (group_traverse), for launches with few
// items: a wave holds group_items items, each with a group of G lanes, and its
// groups go round by round together. The first lane
// of a group is the one that carries the item: it alone runs the source.
// Rounds keep no hit list.
//
// Items a wave carries at a time. Fewer than it has to do in all (q = items /
// waves), so that a wave whose items are short takes more of them, and each
// group has more lanes. Measured with 1, 2, 4, 8 and 16 (us; 2048 waves):
//   path tracing, 100,000-surfel room: 4 k paths 492 448 535 531 532, 10 k 774
//   652 560 669 685, 19 k 1169 927 775 765 976, 50 k 2613 1883 1379 1203 1285,
//   75 k 3830 2645 1812 1515 1518; Stage-0 step: 10 k pixels 754 692 710 804 808,
//   19 k 1126 890 834 949 1241, 40 k 2101 1362 1081 1153 1424.
// With at most 2^12 surfels a forward segment ends after few visits, and the
// claims are most of its cost: there 16 items from 24 on instead of 40 (Stage-0
// images of 65,536 pixels, sparse rooms of 500 to 4000 surfels: 140 to 97 us).
__host__ __device__ inline int group_items(int64_t n_work, int64_t n_waves, bool short_items) {
  const int64_t q = (n_work + n_waves - 1) / n_waves;
  return q >= (short_items ? 24 : 40) ? 16 : (q >= 12 ? 8 : (q >= 4 ? 4 : (q >= 2 ? 2 : 1)));
}

template <int QMODE, bool DACC, bool STATS, class Src>
__device__ __forceinline__ void run_groups(const TraceCtx& tc, Src& src, unsigned long long* work_counter,
                                           int64_t n_work, unsigned long long* counters) {
  __shared__ int s_stack[STACK_LDS * TRACE_BLOCK];
  __shared__ int s_pend[PEND * TRACE_BLOCK];
  int s_ovf[STACK_OVF];
  TravStack st;
  st.lds = s_stack + threadIdx.x;
  st.ovf = s_ovf;
  st.sp = 0;
  bind_lds_stack(src, st.lds, 0);
  int* const pend = s_pend + threadIdx.x;
  const int lane = (int)(threadIdx.x & 63);
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const int G = 64 / group_items(n_work, (int64_t)gridDim.x * (TRACE_BLOCK / 64), !Src::kHits && tc.idx_bits <= 12);
  const int lead = lane & ~(G - 1);
  const bool first = lane == lead;
  TraceCtx tcl = tc;
  SegStats<DACC, STATS, false> s;
  seg_begin(s, d3(0.0, 0.0, 0.0), d3(0.0, 0.0, 1.0));
  Round r;
  RunStats rs;
  D3 O = d3(0.0, 0.0, 0.0), W = d3(0.0, 0.0, 1.0);
  bool idle = true, fresh = false;   // of the first lane's item; fresh: (O, W) is its next segment's ray
  Claims claims(work_counter, n_work, 64 / G);
  while (true) {
    const bool need = first && idle && !claims.exhausted;
    const uint64_t m = __ballot(need);
    if (m) {
      int64_t wid = claims.take(m) + __popcll(m & lt_mask);
      bool take = need;
      if constexpr (Src::kHits) {
        // a source that takes the hits is carried by every lane of the group
        wid = __shfl(wid, lead);
        take = __shfl(need ? 1 : 0, lead) != 0;
      }
      if (take) {
        if (wid < n_work && src.start(wid, tcl, O, W)) {
          idle = false;
          fresh = true;
          if constexpr (STATS) {
            ++rs.items;
            ++rs.segments;
          }
        }
      }
    }
    if (!__any(!idle)) {
      if (claims.exhausted) break;
      continue;
    }
    // the group follows its first lane: the ray of a new segment, else where
    // the last round ended
    const bool on = __shfl(idle ? 0 : 1, lead) != 0, begin = __shfl(fresh ? 1 : 0, lead) != 0;
    if (__any(begin)) {
      const D3 o = d3(__shfl(O.x, lead), __shfl(O.y, lead), __shfl(O.z, lead));
      const D3 w = d3(__shfl(W.x, lead), __shfl(W.y, lead), __shfl(W.z, lead));
      if (begin) seg_begin(s, o, w);
    }
    fresh = false;
    round_begin(tcl, s, r, st, pend);
    const bool fits = group_traverse(tcl, s, r, s_stack, s_pend, G, on);
    if (first && on && !fits) {
      round_begin(tcl, s, r, st, pend);
      traverse_round(tcl, s, r, st, pend, 1);
    }
    group_blend<QMODE>(tcl, s, r, src, s_pend, G, on, nullptr, 0);
    if constexpr (Src::kHits) {
      if (__any(on && s.done)) src.gather(G, on && s.done);
    }
    if (first && on) {
      if constexpr (STATS) {
        rs.rounds += s.rounds;
        rs.hits += s.nhits;
      }
      if (s.done) {
        fresh = src.finish(s, O, W);
        idle = !fresh;
        if constexpr (STATS) rs.segments += fresh ? 1 : 0;
      }
    }
    // (an item of a source that takes the hits is one segment)
    if constexpr (Src::kHits) {
      if (!first && on && s.done) {
        src.leave();
        idle = true;
      }
    }
    if constexpr (STATS) {
      rs.tests += s.tests;
      rs.visits += s.visits;
      s.rounds = s.tests = s.nhits = s.visits = 0;
    }
  }
  if constexpr (STATS) rs.flush(counters);
}

// Whether a launch of n_work items runs by groups (the host's choice of
// kernel: the two ways share nothing but LDS). One lane per item has the higher
// rate, and waits for its longest path at the end, 2 ms in a room; just above
// the grid's lanes its second pass is nearly empty. With few surfels there is
// little to wait for, and with 2^18 or more a group's visits miss the caches as
// a lane's do, except where roulette ends paths early: then most lanes idle,
// while a wave's groups take other items. So the line lies by the kind of launch
// and by the bits of a surfel index, in quarters of the grid's lanes. One lane
// per item against groups, ms, with 131,072 lanes:
//   paths, 90 k and 130 k of them: 20,000-surfel room 1.15 0.73, 1.29 0.91; 100,000
//   3.49 1.84, 3.32 2.30; 300,000 4.15 3.65, 4.43 4.66, with emitter sampling 7.33
//   7.00, 7.84 9.24; cloud of 2000 1.03 0.55, 1.08 0.75;
//   paths, 102 k and 124 k in the 500,000-surfel room, without roulette, depth 4: 4.37
//   5.63, 4.68 6.55, sampled 7.24 9.86, 7.52 11.6; with two rounds of it (depth 4 from 3)
//   3.59 3.78, 3.87 4.36 (the same room perturbed 5.43 4.25, 5.08 4.89), sampled 6.31
//   7.05, 6.60 8.23; with five (6 from 2) 4.66 3.59, 4.78 4.08, sampled 8.03 6.67, 8.28
//   7.47;
//   camera segments (whole Stage-0 step), 134 k, 215 k, 230 k and 246 k: cloud of 2000
//   0.82 0.70, 0.90 0.83, 1.09 1.05, 1.14 1.17, of 3800 at 215 k 1.43 1.18, at 230 k 1.72
//   1.61; 100,000-surfel room, camera pass alone, 131 k and 262 k, 0.95 0.60, 0.98 0.69;
//   300,000 1.16 1.04, 1.77 1.62; sparse rooms of 1000, 65 k and 250 k, 0.10 0.16, 0.13
//   0.25 (of 1500, whole step, 134 k and 246 k 0.32 0.44, 0.44 0.63);
//   secondary segments, 131 k, 197 k and 262 k (whole render): cloud of 4000 1.54 0.84,
//   1.60 0.97, 1.64 1.09; 300,000-surfel room 2.18 1.98, 2.35 2.57, 2.64 3.17; 1 M 3.49
//   3.54, 3.57 4.47, 3.86 5.41;
//   adjoints, 160 k: 100,000-surfel room 1.88 1.59, 300,000 3.70 3.37.
// Rays that all do the same, through many layers, gain from no group: 200 and 1000
// coplanar layers by 32 k and 65 k paths 0.90 1.40, 2.6 6.2; their adjoints 49 6.4.
enum { PATHS, ENDED_PATHS, CAMERA, SECONDARY, ADJOINTS };
inline bool by_groups(int kind, int64_t n_work, int64_t grid_lanes, int idx_bits) {
  static const int quarters[5][5] = {{1, 4, 4, 4, 3}, {1, 4, 4, 4, 4}, {1, 7, 8, 8, 8}, {1, 8, 8, 8, 4}, {8, 8, 8, 8, 8}};
  const int size = idx_bits <= 10 ? 0 : (idx_bits <= 11 ? 1 : (idx_bits <= 12 ? 2 : (idx_bits <= 17 ? 3 : 4)));
  return 4 * n_work <= quarters[kind][size] * grid_lanes;
}

// Paths of at most max_depth bounces are ended early where roulette has at
// least `rounds` of them to act on.
inline int path_kind(int32_t max_depth, int32_t rr_start, int32_t rounds) {
  return rr_start > 0 && max_depth - rr_start >= rounds - 1 ? ENDED_PATHS : PATHS;
}

template <bool GROUPS, int QMODE, bool DACC, bool STATS, class Src>
__device__ __forceinline__ void run_work(const TraceCtx& tc, Src& src, unsigned long long* work_counter,
                                         int64_t n_work, uint64_t* hitlist, unsigned long long* counters) {
  if constexpr (GROUPS) run_groups<QMODE, DACC, STATS>(tc, src, work_counter, n_work, counters);
  else run_segments<QMODE, DACC, STATS>(tc, src, work_counter, n_work, hitlist, counters);
}

// Sums into rows of doubles, one row per surfel, from the lanes that blend a
// hit together: the V values of each lane's hit are added to acc[idx * stride]
// on. The lanes put their values in LDS and share the adds out so that
// neighbouring lanes add neighbouring values of one hit: an atomic costs by the
// 64-byte piece it touches (23.5 G a second on this chip, whatever is added
// there), so that a hit's three doubles cost 1 where one lane adding its own
// hit's costs 3 (light baking's radiance gradient 11.6 to 7.8 ms).
template <int V, int CAP>
struct RowAdds {          // one per wave, in LDS
  double v[CAP * V];
  uint32_t idx[CAP];
};
template <int V, int CAP>
__device__ __forceinline__ void add_rows(RowAdds<V, CAP>* lds, double* acc, uint32_t stride, uint32_t idx,
                                         const double (&v)[V]) {
  const uint64_t act = __ballot(1);
  const uint32_t m = (uint32_t)__popcll(act);
  const uint32_t r = (uint32_t)__popcll(act & ((1ull << (threadIdx.x & 63)) - 1ull));
  // (volatile: lanes read what others wrote)
  volatile double* const lv = lds->v;
  volatile uint32_t* const li = lds->idx;
  for (uint32_t h0 = 0; h0 < m; h0 += CAP) {
    const uint32_t mh = m - h0 < (uint32_t)CAP ? m - h0 : (uint32_t)CAP;
    if (r - h0 < mh) {
#pragma unroll
      for (int k = 0; k < V; ++k) lv[(r - h0) * V + k] = v[k];
      li[r - h0] = idx;
    }
    for (uint32_t q = r; q < mh * V; q += m) {
      const uint32_t h = q / V, k = q - h * V;
      // (at most 2^23 rows: a 32-bit byte offset)
      char* const at = reinterpret_cast<char*>(acc) + (uint32_t)((li[h] * stride + k) * (uint32_t)sizeof(double));
      atomicAdd(reinterpret_cast<double*>(at), lv[q]);
    }
  }
}

}  // namespace eag
