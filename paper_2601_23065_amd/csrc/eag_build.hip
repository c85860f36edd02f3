// Linear BVH build and refit over 2D Gaussian surfels.
//
// 1. frames and k_sigma-ellipse boxes of every surfel (the surfel of
//    Sec. 3.1: centre p, tangent axes t_u, t_v from the normalised
//    quaternion, scales s_u, s_v), the scene bounds, and one 48-B geometry
//    record per surfel;
// 2. 63-bit Morton codes of the centres, sorted (eag_prim.hip), and the
//    records in that order;
// 3. a binary hierarchy by locally-ordered agglomerative clustering of the
//    sorted boxes (below), which writes each node's child boxes as it makes
//    the node and carries each cluster's height;
// 4. its collapse into a 4-wide tree, in an exact form and in the 64-B form
//    that the traversal reads.
// A refit keeps the topology and recomputes the node boxes in the order of
// the clustering iterations that made the nodes.
// Everything is enqueued on the caller's stream: the depths, node count and
// bounds stay in the device header, and the host waits for them only when
// asked (eag_bvh_get_info).
#include <hip/hip_runtime.h>

#include "eag_device.h"
#include "eag_internal.h"

#include <algorithm>

namespace eag {

namespace {

__device__ __forceinline__ uint32_t fenc(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__host__ __device__ __forceinline__ float fdec(uint32_t e) {
  const uint32_t b = (e & 0x80000000u) ? (e & 0x7fffffffu) : ~e;
  float f;
  __builtin_memcpy(&f, &b, 4);
  return f;
}

struct Frame {
  D3 tu, tv, n;
};
__device__ __forceinline__ Frame frame_of(const float (&rot)[4]) {
  double w = rot[0], x = rot[1], y = rot[2], z = rot[3];
  const double inv = 1.0 / sqrt(w * w + x * x + y * y + z * z);
  w *= inv; x *= inv; y *= inv; z *= inv;
  Frame f;
  f.tu = d3(1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y + w * z), 2.0 * (x * z - w * y));
  f.tv = d3(2.0 * (x * y - w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z + w * x));
  f.n = cross(f.tu, f.tv);
  return f;
}

// Bounds only (a refit keeps the depths and the node count).
__global__ void k_reset_bounds(BvhHeader* h) {
  if (threadIdx.x < 3) {
    h->plo[threadIdx.x] = 0xffffffffu;
    h->phi[threadIdx.x] = 0u;
    h->blo[threadIdx.x] = 0xffffffffu;
    h->bhi[threadIdx.x] = 0u;
  }
}

__global__ void k_init_header(BvhHeader* h) {
  if (threadIdx.x < 3) {
    h->plo[threadIdx.x] = 0xffffffffu;
    h->phi[threadIdx.x] = 0u;
    h->blo[threadIdx.x] = 0xffffffffu;
    h->bhi[threadIdx.x] = 0u;
  }
  if (threadIdx.x == 0) {
    h->max_depth = 0;
    h->n_nodes4 = 0;
    h->depth4 = 0;
  }
}

// Box of the k_sigma ellipse: half extent along axis a is
// k * sqrt((s_u t_u,a)^2 + (s_v t_v,a)^2), padded so that float32 rounding in
// the surfel test can never place an accepted hit outside its box. The boxes
// (lo.xyz and hi.xyz, one float4 each) and the surfels' geometry records are
// written in the caller's order, so that what later reads them through the
// sorted order finds each in one piece (the component-major arrays would cost
// a cache line per component: 203 us for the records of 1 M surfels against
// 42 from rows). Grid-stride over BOX_GRID blocks: one set of bounds atomics
// per block of 256 surfels took 184 us there, all on 12 addresses.
constexpr unsigned BOX_GRID = 512;
__global__ void __launch_bounds__(256) k_boxes(eag_surfels s, float k, float4* box, Record* raw, BvhHeader* h) {
  const int64_t n = s.n;
  // centre lo, centre hi, box lo, box hi; the upper bounds negated
  float b[12];
#pragma unroll
  for (int a = 0; a < 12; ++a) b[a] = __builtin_inff();
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float q[4] = {s.rot[i], s.rot[n + i], s.rot[2 * n + i], s.rot[3 * n + i]};
    const float sc[2] = {s.scale[i], s.scale[n + i]};
    const float p[3] = {s.pos[i], s.pos[n + i], s.pos[2 * n + i]};
    const Frame f = frame_of(q);
    const double su = sc[0], sv = sc[1];
    const float pad = 2e-5f * (1.0f + fmaxf(fmaxf(fabsf(p[0]), fabsf(p[1])), fabsf(p[2])));
    const double tu[3] = {f.tu.x, f.tu.y, f.tu.z}, tv[3] = {f.tv.x, f.tv.y, f.tv.z};
    float lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float e = (float)(k * sqrt((su * tu[a]) * (su * tu[a]) + (sv * tv[a]) * (sv * tv[a]))) + pad;
      lo[a] = p[a] - e;
      hi[a] = p[a] + e;
      b[a] = fminf(b[a], p[a]);
      b[3 + a] = fminf(b[3 + a], -p[a]);
      b[6 + a] = fminf(b[6 + a], lo[a]);
      b[9 + a] = fminf(b[9 + a], -hi[a]);
    }
    box[2 * i] = make_float4(lo[0], lo[1], lo[2], 0.0f);
    box[2 * i + 1] = make_float4(hi[0], hi[1], hi[2], 0.0f);
    float4* r = reinterpret_cast<float4*>(raw + i);
    r[0] = make_float4(p[0], p[1], p[2], s.opacity[i]);
    r[1] = make_float4(q[0], q[1], q[2], q[3]);
    r[2] = make_float4(sc[0], sc[1], __uint_as_float((uint32_t)i), 0.0f);
  }
  // block reduction of the bounds, then one atomic per block and component
  __shared__ float red[12][4];
#pragma unroll
  for (int a = 0; a < 12; ++a) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) b[a] = fminf(b[a], __shfl_xor(b[a], o));
    if ((threadIdx.x & 63) == 0) red[a][threadIdx.x >> 6] = b[a];
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    const int a = (int)threadIdx.x % 3, g = (int)threadIdx.x / 3;
    const float* r = red[threadIdx.x];
    const float v = fminf(fminf(r[0], r[1]), fminf(r[2], r[3]));
    if (g == 0) atomicMin(&h->plo[a], fenc(v));
    if (g == 1) atomicMax(&h->phi[a], fenc(-v));
    if (g == 2) atomicMin(&h->blo[a], fenc(v));
    if (g == 3) atomicMax(&h->bhi[a], fenc(-v));
  }
}

__device__ __forceinline__ uint64_t spread3(uint32_t a) {
  uint64_t x = a & 0x1fffffu;
  x = (x | x << 32) & 0x1f00000000ffffull;
  x = (x | x << 16) & 0x1f0000ff0000ffull;
  x = (x | x << 8) & 0x100f00f00f00f00full;
  x = (x | x << 4) & 0x10c30c30c30c30c3ull;
  x = (x | x << 2) & 0x1249249249249249ull;
  return x;
}

__global__ void k_morton(eag_surfels s, const BvhHeader* h, uint64_t* codes, uint32_t* ids) {
  const int64_t n = s.n;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t q[3];
  float ext = 0.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) ext = fmaxf(ext, fdec(h->phi[a]) - fdec(h->plo[a]));
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float lo = fdec(h->plo[a]);
    float x = ext > 0.0f ? (s.pos[a * n + i] - lo) / ext : 0.0f;
    x = fminf(fmaxf(x, 0.0f), 1.0f);
    q[a] = min((uint32_t)(x * 2097152.0f), 2097151u);
  }
  codes[i] = (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
  ids[i] = (uint32_t)i;
}

// ---------------------------------------------------------------------------
// Binary hierarchy by locally-ordered agglomerative clustering (PLOC, Meister
// and Bittner, TVCG 2018). The clusters start as the leaves in Morton order.
// Each iteration finds every cluster's nearest neighbour among the PLOC_R
// clusters on either side in the current order, by the surface area of the
// union of their boxes (ties to the lower position), merges every mutual pair
// into a new internal node at the lower position, and compacts the order.
// A cluster made in iteration t is at most t levels high, so there are at most
// PLOC_ITERS such iterations, then at most ceil(log2 n) halving iterations that
// pair positions 2k and 2k + 1, which bound the tree's height by PLOC_ITERS +
// ceil(log2 n) whatever the input. Internal nodes are numbered from the top:
// the k-th node made is n - 2 - k, so the last (the root) is node 0.
//
// The iterations' cost is their launches: the clusters shrink by about a third
// each time, so all but the first few iterations are small. Those first ones
// (wide_iters: enough to come near PLOC_TAIL clusters) are two launches over
// the whole chip each; one block then runs all the others in one launch, from
// LDS once a cluster per thread is left. Launching every possible iteration, as
// empty as most were, in four launches each, took 0.66 ms of a 2000-surfel build
// and 1.2 ms of a 1 M one.
// ---------------------------------------------------------------------------
constexpr int PLOC_R = 2;          // search radius (measured best of 1 to 16 for the path tracer)
constexpr int PLOC_ITERS = 64;     // iterations before the halving fallback
constexpr int PLOC_GRID = 1024;    // blocks of every clustering launch
constexpr int PLOC_TILE = 256;
constexpr int PLOC_TAIL = 1024;    // clusters (and threads) of the single block that runs the last iterations
// Clusters that the wide iterations leave to that block at most, which takes 4 us
// for each 1024 of them in each iteration. Surfels whose pairs hardly merge
// (coincident ones: the nearest of all is the lowest of the window, so two of a
// run merge at a time) come to the last of the wide iterations nearly all: those
// then halve them, each as late as the ones after it still reach this number.
// With ordinary scenes, about a third merge in each iteration and none halves.
// Left to the block as they were, 1 M coincident surfels took 24.4 ms to build and
// 6.1 ms to refit, now 1.5 and 0.5.
constexpr int PLOC_TAIL_MOST = 32768;
constexpr int PLOC_LEVELS = PLOC_ITERS + 24;   // iterations launched for up to 2^23 surfels, and more

struct PlocState {
  int32_t n;          // clusters now
  int32_t cur;        // buffer holding the current clusters
  int32_t made;       // internal nodes made so far
  int32_t pad;
};

struct Ploc {
  int32_t* cl[2];     // cluster references (node >= 0, leaf ~position)
  float4* cb[2];      // cluster boxes: [2i] lo.xyz, [2i + 1] hi.xyz
  int32_t* nn;        // nearest neighbour of each cluster
  int2* bsum;         // per block: clusters kept, nodes made
  PlocState* st;      // [2]: iteration t reads state t & 1 and writes the other
};

__device__ __forceinline__ float union_area(float4 al, float4 ah, float4 bl, float4 bh) {
  const float dx = fmaxf(ah.x, bh.x) - fminf(al.x, bl.x);
  const float dy = fmaxf(ah.y, bh.y) - fminf(al.y, bl.y);
  const float dz = fmaxf(ah.z, bh.z) - fminf(al.z, bl.z);
  return dx * dy + dy * dz + dz * dx;
}

// Iterations launched over the whole chip for n surfels.
int wide_iters(int64_t n) {
  int t = 0;
  for (double m = (double)n; m > PLOC_TAIL && t < PLOC_ITERS; m *= 0.7) ++t;
  return t;
}

// Clusters that wide iteration t of `wide` still searches; more are halved
// instead, so that those after it can bring them down to PLOC_TAIL_MOST by
// halving (n is at most PLOC_TAIL / 0.7^wide, below PLOC_TAIL_MOST 2^wide).
int search_limit(int t, int wide) {
  const int later = wide - 1 - t;
  return later < 15 ? PLOC_TAIL_MOST << later : INT32_MAX;
}

// The lower corner's w is the cluster's height (levels of internal nodes).
__global__ void k_ploc_init(int64_t n, const float4* box, const int32_t* perm, Ploc P) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j == 0) {
    PlocState s = {};
    s.n = (int32_t)n;
    *P.st = s;
  }
  if (j >= n) return;
  const int64_t i = perm[j];
  P.cl[0][j] = ~(int32_t)j;
  P.cb[0][2 * j] = box[2 * i];
  P.cb[0][2 * j + 1] = box[2 * i + 1];
}

// Merge two clusters into internal node `id`; returns the union's corners.
__device__ __forceinline__ void ploc_merge(Node* nodes, int id, int c0, int c1, float4 l0, float4 h0, float4 l1,
                                           float4 h1, float4& lo, float4& hi) {
  Node nd;
  nd.a = make_float4(l0.x, l0.y, l0.z, h0.x);
  nd.b = make_float4(h0.y, h0.z, l1.x, l1.y);
  nd.c = make_float4(l1.z, h1.x, h1.y, h1.z);
  nd.d = make_int4(c0, c1, 0, 0);
  nodes[id] = nd;
  lo = make_float4(fminf(l0.x, l1.x), fminf(l0.y, l1.y), fminf(l0.z, l1.z), 1.0f + fmaxf(l0.w, l1.w));
  hi = make_float4(fmaxf(h0.x, h1.x), fmaxf(h0.y, h1.y), fmaxf(h0.z, h1.z), 0.0f);
}

// Per position: kept (a cluster survives there) and made (a node is made
// there, at the lower position of a mutual pair).
__device__ __forceinline__ void ploc_decide(const int32_t* nn, int i, int& j, bool& keep, bool& made) {
  j = nn[i];
  const bool mutual = j != i && nn[j] == i;
  keep = !mutual || i < j;
  made = mutual && i < j;
}

// Exclusive block scan of two counts (each at most PLOC_TILE per tile),
// packed in one int; returns the block's totals in *tot.
__device__ __forceinline__ int scan_pair(int v, int* lds, int* tot) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(x, o);
    if (lane >= o) x += t;
  }
  if (lane == 63) lds[w] = x;
  __syncthreads();
  int before = 0;
  for (int k = 0; k < w; ++k) before += lds[k];
  *tot = lds[0] + lds[1] + lds[2] + lds[3];
  __syncthreads();
  return before + x - v;
}

__device__ __forceinline__ void ploc_chunk(int n, int& lo, int& hi) {
  const int chunk = (n + gridDim.x - 1) / gridDim.x;
  lo = min(n, (int)blockIdx.x * chunk);
  hi = min(n, lo + chunk);
}

// Sum of two counts over a block of PLOC_TILE threads, in every thread.
__device__ __forceinline__ int2 block_sum2(int2 v, int2* lds) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    v.x += __shfl_xor(v.x, o);
    v.y += __shfl_xor(v.y, o);
  }
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  const int2 t = make_int2(lds[0].x + lds[1].x + lds[2].x + lds[3].x, lds[0].y + lds[1].y + lds[2].y + lds[3].y);
  __syncthreads();
  return t;
}

// First half of iteration t: the partner of every cluster (nn[i]: its mutual
// nearest neighbour, or itself; with more than `limit` clusters, the other one of
// positions 2k and 2k + 1), and what each block's part of the order will
// keep and make. A tile's neighbours' neighbours are found here again rather
// than read from another launch.
__global__ void __launch_bounds__(PLOC_TILE) k_ploc_pairs(Ploc P, int t, int limit) {
  constexpr int BOXES = PLOC_TILE + 4 * PLOC_R, NEAR = PLOC_TILE + 2 * PLOC_R;
  __shared__ float4 slo[BOXES], shi[BOXES];
  __shared__ int snn[NEAR];
  __shared__ int2 lds[PLOC_TILE / 64];
  const PlocState st = P.st[t & 1];
  const int n = st.n;
  if (n <= 1) return;
  const float4* cb = P.cb[st.cur];
  int lo, hi;
  ploc_chunk(n, lo, hi);
  int2 sum = make_int2(0, 0);
  if (n > limit) {
    for (int i = lo + (int)threadIdx.x; i < hi; i += PLOC_TILE) {
      const int p = (i ^ 1) < n ? (i ^ 1) : i;
      P.nn[i] = p;
      sum.x += p >= i ? 1 : 0;
      sum.y += p > i ? 1 : 0;
    }
    lo = hi;
  }
  for (int base = lo; base < hi; base += PLOC_TILE) {
    for (int k = threadIdx.x; k < BOXES; k += PLOC_TILE) {
      const int g = base - 2 * PLOC_R + k;
      if (g >= 0 && g < n) {
        slo[k] = cb[2 * g];
        shi[k] = cb[2 * g + 1];
      }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < NEAR; k += PLOC_TILE) {
      const int i = base - PLOC_R + k, li = k + PLOC_R;
      int bj = i;
      if (i >= 0 && i < n) {
        const float4 al = slo[li], ah = shi[li];
        float best = INFINITY;
        for (int d = -PLOC_R; d <= PLOC_R; ++d) {
          const int g = i + d;
          if (d == 0 || g < 0 || g >= n) continue;
          const float a = union_area(al, ah, slo[li + d], shi[li + d]);
          if (a < best) {   // ascending g: ties keep the lower position
            best = a;
            bj = g;
          }
        }
      }
      snn[k] = bj;
    }
    __syncthreads();
    const int i = base + (int)threadIdx.x;
    if (i < hi) {
      const int j = snn[i - base + PLOC_R];
      const int p = j != i && snn[j - base + PLOC_R] == i ? j : i;
      P.nn[i] = p;
      sum.x += p >= i ? 1 : 0;
      sum.y += p > i ? 1 : 0;
    }
    __syncthreads();
  }
  const int2 tot = block_sum2(sum, lds);
  if (threadIdx.x == 0) P.bsum[blockIdx.x] = tot;
}

// Second half: the merges, and the order compacted. Each block sums up what the
// blocks before it keep and make; the first one also makes the next state.
// levels[t]: the nodes made before iteration t (iteration t makes the ids
// n - 2 - k for k in [levels[t], levels[t + 1])), kept with the tree for
// refits.
__global__ void __launch_bounds__(PLOC_TILE) k_ploc_write(Ploc P, int t, int32_t* levels, int64_t n_leaves,
                                                         Node* nodes) {
  __shared__ int lds[4];
  __shared__ int2 lds2[PLOC_TILE / 64];
  const PlocState st = P.st[t & 1];
  const int n = st.n;
  if (n <= 1) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      P.st[(t + 1) & 1] = st;
      levels[t] = st.made;
    }
    return;
  }
  const int end = blockIdx.x == 0 ? (int)gridDim.x : (int)blockIdx.x;
  int2 v = make_int2(0, 0);
  for (int k = threadIdx.x; k < end; k += PLOC_TILE) {
    const int2 q = P.bsum[k];
    v.x += q.x;
    v.y += q.y;
  }
  int2 before = block_sum2(v, lds2);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      PlocState next = {};
      next.n = before.x;
      next.cur = st.cur ^ 1;
      next.made = st.made + before.y;
      P.st[(t + 1) & 1] = next;
      levels[t] = st.made;
    }
    before = make_int2(0, 0);
  }
  const int in = st.cur, out = in ^ 1;
  const int32_t* cl = P.cl[in];
  const float4* cb = P.cb[in];
  int lo, hi;
  ploc_chunk(n, lo, hi);
  int keep_at = before.x, made_at = st.made + before.y;
  for (int base = lo; base < hi; base += PLOC_TILE) {
    const int i = base + (int)threadIdx.x;
    const int j = i < hi ? P.nn[i] : -1;
    const bool keep = i < hi && j >= i, made = keep && j > i;
    int tot;
    const int off = scan_pair((keep ? 1 : 0) | (made ? 1 << 16 : 0), lds, &tot);
    if (keep) {
      const int o = keep_at + (off & 0xffff);
      if (made) {
        const int id = (int)(n_leaves - 2) - (made_at + (off >> 16));
        float4 lo4, hi4;
        ploc_merge(nodes, id, cl[i], cl[j], cb[2 * i], cb[2 * i + 1], cb[2 * j], cb[2 * j + 1], lo4, hi4);
        P.cl[out][o] = id;
        P.cb[out][2 * o] = lo4;
        P.cb[out][2 * o + 1] = hi4;
      } else {
        P.cl[out][o] = cl[i];
        P.cb[out][2 * o] = cb[2 * i];
        P.cb[out][2 * o + 1] = cb[2 * i + 1];
      }
    }
    keep_at += tot & 0xffff;
    made_at += tot >> 16;
  }
}

// Exclusive block scan of two counts packed in one int (each at most PLOC_TAIL
// per call) over PLOC_TAIL threads; every thread gets the totals.
__device__ __forceinline__ int tail_scan(int v, int* lds, int& tot) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(x, o);
    if (lane >= o) x += t;
  }
  if (lane == 63) lds[w] = x;
  __syncthreads();
  int before = 0;
  tot = 0;
#pragma unroll
  for (int k = 0; k < PLOC_TAIL / 64; ++k) {
    before += k < w ? lds[k] : 0;
    tot += lds[k];
  }
  __syncthreads();
  return before + x - v;
}

// All iterations from t0 on, by one block. Writes the rest of levels (iteration
// t makes the ids n - 2 - k for k in [levels[t], levels[t + 1])) up to
// levels[iters], and the tree's height. Its time is latency, about 2 us an
// iteration in LDS.
__global__ void __launch_bounds__(PLOC_TAIL) k_ploc_tail(Ploc P, int64_t n_leaves, Node* nodes, int t0, int iters,
                                                         int32_t* levels, BvhHeader* h) {
  __shared__ float4 slo[PLOC_TAIL], shi[PLOC_TAIL];
  __shared__ int sref[PLOC_TAIL], snn[PLOC_TAIL], lds[PLOC_TAIL / 64];
  const int tid = (int)threadIdx.x;
  const PlocState st = P.st[t0 & 1];
  int n = st.n, made = st.made, cur = st.cur, t = t0;
  // Too many clusters for LDS: the same iteration over memory, in tiles. One
  // that merged few is followed by one that halves.
  bool few = false;
  while (n > PLOC_TAIL) {
    const bool halving = t >= PLOC_ITERS || few;
    const int32_t* cl = P.cl[cur];
    const float4* cb = P.cb[cur];
    int32_t* ol = P.cl[cur ^ 1];
    float4* ob = P.cb[cur ^ 1];
    if (tid == 0) levels[t] = made;
    for (int i = tid; i < n; i += PLOC_TAIL) {
      int bj = (i ^ 1) < n ? (i ^ 1) : i;
      if (!halving) {
        const float4 al = cb[2 * i], ah = cb[2 * i + 1];
        float best = INFINITY;
        bj = i;
        for (int d = -PLOC_R; d <= PLOC_R; ++d) {
          const int g = i + d;
          if (d == 0 || g < 0 || g >= n) continue;
          const float a = union_area(al, ah, cb[2 * g], cb[2 * g + 1]);
          if (a < best) {   // ascending g: ties keep the lower position
            best = a;
            bj = g;
          }
        }
      }
      P.nn[i] = bj;
    }
    __syncthreads();
    int kept = 0, now = made;
    for (int base = 0; base < n; base += PLOC_TAIL) {
      const int i = base + tid;
      int j = i;
      bool keep = false, mk = false;
      if (i < n) ploc_decide(P.nn, i, j, keep, mk);
      int tot;
      const int off = tail_scan((keep ? 1 : 0) | (mk ? 1 << 16 : 0), lds, tot);
      if (keep) {
        const int o = kept + (off & 0xffff);
        int ref = cl[i];
        float4 lo4 = cb[2 * i], hi4 = cb[2 * i + 1];
        if (mk) {
          const int id = (int)(n_leaves - 2) - (now + (off >> 16));
          ploc_merge(nodes, id, ref, cl[j], lo4, hi4, cb[2 * j], cb[2 * j + 1], lo4, hi4);
          ref = id;
        }
        ol[o] = ref;
        ob[2 * o] = lo4;
        ob[2 * o + 1] = hi4;
      }
      kept += tot & 0xffff;
      now += tot >> 16;
    }
    __syncthreads();
    few = kept > n - n / 8;
    n = kept;
    made = now;
    cur ^= 1;
    ++t;
  }
  if (tid < n) {
    slo[tid] = P.cb[cur][2 * tid];
    shi[tid] = P.cb[cur][2 * tid + 1];
    sref[tid] = P.cl[cur][tid];
  }
  __syncthreads();
  while (n > 1) {
    if (tid == 0) levels[t] = made;
    int j = tid;
    float4 l0 = make_float4(0.f, 0.f, 0.f, 0.f), h0 = l0;
    int ref = 0;
    if (tid < n) {
      l0 = slo[tid];
      h0 = shi[tid];
      ref = sref[tid];
      if (t >= PLOC_ITERS) {
        j = (tid ^ 1) < n ? (tid ^ 1) : tid;
      } else {
        float best = INFINITY;
        for (int d = -PLOC_R; d <= PLOC_R; ++d) {
          const int g = tid + d;
          if (d == 0 || g < 0 || g >= n) continue;
          const float a = union_area(l0, h0, slo[g], shi[g]);
          if (a < best) {   // ascending g: ties keep the lower position
            best = a;
            j = g;
          }
        }
      }
      snn[tid] = j;
    }
    __syncthreads();
    const bool mutual = tid < n && j != tid && snn[j] == tid;
    const bool keep = tid < n && (!mutual || tid < j), mk = mutual && tid < j;
    int tot;
    const int off = tail_scan((keep ? 1 : 0) | (mk ? 1 << 16 : 0), lds, tot);
    if (mk) {
      const int id = (int)(n_leaves - 2) - (made + (off >> 16));
      ploc_merge(nodes, id, ref, sref[j], l0, h0, slo[j], shi[j], l0, h0);
      ref = id;
    }
    __syncthreads();   // every merge has read its partner
    if (keep) {
      const int o = off & 0xffff;
      slo[o] = l0;
      shi[o] = h0;
      sref[o] = ref;
    }
    __syncthreads();
    n = tot & 0xffff;
    made += tot >> 16;
    ++t;
  }
  for (int k = t + tid; k <= iters; k += PLOC_TAIL) levels[k] = made;
  if (tid == 0) h->max_depth = (int)slo[0].w;
}

// Refit of one node: its children were made in earlier iterations than it, or
// are leaves.
__device__ __forceinline__ void refit_node(const float4* box, const int32_t* perm, Node* nodes, int id) {
  Node& nd = nodes[id];
  float lo[2][3], hi[2][3];
  const int ch[2] = {nd.d.x, nd.d.y};
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (ch[c] < 0) {
      const int64_t i = perm[~ch[c]];
      const float4 L = box[2 * i], H = box[2 * i + 1];
      lo[c][0] = L.x; lo[c][1] = L.y; lo[c][2] = L.z;
      hi[c][0] = H.x; hi[c][1] = H.y; hi[c][2] = H.z;
    } else {
      const Node& cn = nodes[ch[c]];
      const float4 A = cn.a, Bv = cn.b, C = cn.c;
      lo[c][0] = fminf(A.x, Bv.z);
      lo[c][1] = fminf(A.y, Bv.w);
      lo[c][2] = fminf(A.z, C.x);
      hi[c][0] = fmaxf(A.w, C.y);
      hi[c][1] = fmaxf(Bv.x, C.z);
      hi[c][2] = fmaxf(Bv.y, C.w);
    }
  }
  nd.a = make_float4(lo[0][0], lo[0][1], lo[0][2], hi[0][0]);
  nd.b = make_float4(hi[0][1], hi[0][2], lo[1][0], lo[1][1]);
  nd.c = make_float4(lo[1][2], hi[1][0], hi[1][1], hi[1][2]);
}

// The nodes made in clustering iteration t.
__global__ void __launch_bounds__(256) k_refit_level(int64_t n, const float4* box, const int32_t* perm, Node* nodes,
                                                    const int32_t* levels, int t) {
  const int k0 = levels[t], k1 = levels[t + 1];
  for (int k = k0 + (int)(blockIdx.x * blockDim.x + threadIdx.x); k < k1; k += (int)(gridDim.x * blockDim.x))
    refit_node(box, perm, nodes, (int)(n - 2) - k);
}

// The nodes made in iterations t0 to iters - 1, by one block (a launch for
// each took 2.5 us, most of them empty: 204 us of a 200,000-surfel refit).
__global__ void __launch_bounds__(PLOC_TAIL) k_refit_tail(int64_t n, const float4* box, const int32_t* perm,
                                                          Node* nodes, const int32_t* levels, int t0, int iters) {
  const int end = levels[iters];
  for (int t = t0; t < iters; ++t) {
    const int k0 = levels[t], k1 = levels[t + 1];
    if (k0 >= end) break;
    for (int k = k0 + (int)threadIdx.x; k < k1; k += PLOC_TAIL) refit_node(box, perm, nodes, (int)(n - 2) - k);
    __syncthreads();
  }
}

// Records into sorted order. (inv: written with the records of a build; null
// in a refit, which keeps the order)
__global__ void __launch_bounds__(256) k_records(int64_t n, const int32_t* perm, const Record* raw, Record* recs,
                                                 int32_t* inv) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int64_t i = perm[j];
  if (inv) inv[i] = (int32_t)j;
  const float4* src = reinterpret_cast<const float4*>(raw + i);
  float4* r = reinterpret_cast<float4*>(recs + j);
  const float4 a = src[0], b = src[1], c = src[2];
  r[0] = a;
  r[1] = b;
  r[2] = c;
}

// Attribute rows into sorted order, from the caller's order: the seven arrays
// are read in sequence and each row is one piece of 32 bytes wherever it goes.
// (Gathered in the sorted order, each component cost a cache line: 121 us for
// 1 M surfels against 39.)
__global__ void __launch_bounds__(256) k_attrs(eag_surfels s, const int32_t* inv, Attr* attrs) {
  const int64_t n = s.n;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  float4* a = reinterpret_cast<float4*>(attrs + inv[i]);
  a[0] = make_float4(s.albedo[i], s.albedo[n + i], s.albedo[2 * n + i], s.emissive[i]);
  a[1] = make_float4(s.radiance[i], s.radiance[n + i], s.radiance[2 * n + i], 0.0f);
}

// ---------------------------------------------------------------------------
// Collapse of the binary tree into a 4-wide tree, level by level. The 4-wide
// node m of a level expands the two children of binary node job[m]; while
// fewer than four children are held and one of them is an internal binary
// node, the internal child with the largest box surface area is replaced by
// its two children. Internal children left over become 4-wide nodes of the
// next level: level l holds the nodes from start(l) = sum of counts[k < l] on,
// counts[l] of them.
//
// The top levels, up to COLLAPSE_BLOCK nodes, are run by one block in one
// launch, the wide ones below by launches over the whole chip, and what is left
// of a deep tree by one block again; a level's nodes are counted with one
// atomic per block. (A launch for each possible level, two atomics for each
// node: 0.63 ms at 1 M surfels, 0.18 ms of empty launches at 2000.)
// ---------------------------------------------------------------------------
constexpr int COLLAPSE_MAXL = 128;
constexpr int COLLAPSE_BLOCK = 2048;   // the largest level the single block takes before the wide launches
struct Collapse {
  int32_t* job;       // binary node of each 4-wide node
  int32_t* counts;    // [COLLAPSE_MAXL + 1] nodes of each level
  int32_t* level;     // the first level of the wide launches
};

__device__ __forceinline__ void child_box(const Node& nd, int slot, float* lo, float* hi) {
  const float* f = reinterpret_cast<const float*>(&nd);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo[a] = f[slot * 6 + a];
    hi[a] = f[slot * 6 + 3 + a];
  }
}

__device__ __forceinline__ float half_area(const float* lo, const float* hi) {
  const float dx = hi[0] - lo[0], dy = hi[1] - lo[1], dz = hi[2] - lo[2];
  return dx * dy + dy * dz + dz * dx;
}

// The children of binary node `node` in the 4-wide tree (cnt of them).
__device__ __forceinline__ int collapse_children(const Node* bin, int node, int (&ref)[4], float (&lo)[4][3],
                                                 float (&hi)[4][3]) {
  const Node nd = bin[node];
  ref[0] = nd.d.x;
  ref[1] = nd.d.y;
  child_box(nd, 0, lo[0], hi[0]);
  child_box(nd, 1, lo[1], hi[1]);
  ref[2] = ref[3] = NODE4_EMPTY;
#pragma unroll
  for (int a = 0; a < 3; ++a) lo[2][a] = lo[3][a] = hi[2][a] = hi[3][a] = 0.0f;
  int cnt = 2;
#pragma unroll
  for (int step = 2; step < 4; ++step) {
    int best = -1;
    float area = -1.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (k < cnt && ref[k] >= 0) {
        const float a = half_area(lo[k], hi[k]);
        if (a > area) { area = a; best = k; }
      }
    }
    if (best < 0) break;
    int at = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) at = k == best ? ref[k] : at;
    const Node nb = bin[at];
    float l0[3], h0[3], l1[3], h1[3];
    child_box(nb, 0, l0, h0);
    child_box(nb, 1, l1, h1);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool first = k == best, second = k == cnt;
      if (first) ref[k] = nb.d.x;
      if (second) ref[k] = nb.d.y;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lo[k][a] = first ? l0[a] : (second ? l1[a] : lo[k][a]);
        hi[k][a] = first ? h0[a] : (second ? h1[a] : hi[k][a]);
      }
    }
    ++cnt;
  }
  return cnt;
}

// 4-wide node m: both forms written, internal children numbered from id on and
// queued.
__device__ __forceinline__ void collapse_write(Node4* out, NodeQ* outq, int32_t* job, int m, int id,
                                               const int (&src)[4], const float (&lo)[4][3], const float (&hi)[4][3]) {
  int dst[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    dst[k] = src[k];
    if (src[k] != NODE4_EMPTY && src[k] >= 0) {
      job[id] = src[k];
      dst[k] = id++;
    }
  }
  Node4 nd;
  nd.b[0] = make_float4(lo[0][0], lo[0][1], lo[0][2], hi[0][0]);
  nd.b[1] = make_float4(hi[0][1], hi[0][2], lo[1][0], lo[1][1]);
  nd.b[2] = make_float4(lo[1][2], hi[1][0], hi[1][1], hi[1][2]);
  nd.b[3] = make_float4(lo[2][0], lo[2][1], lo[2][2], hi[2][0]);
  nd.b[4] = make_float4(hi[2][1], hi[2][2], lo[3][0], lo[3][1]);
  nd.b[5] = make_float4(lo[3][2], hi[3][0], hi[3][1], hi[3][2]);
  nd.ref = make_int4(dst[0], dst[1], dst[2], dst[3]);
  nd.src = make_int4(src[0], src[1], src[2], src[3]);
  out[m] = nd;
  write_nodeq(outq + m, lo, hi, dst);
}

__device__ __forceinline__ int internal_children(const int (&ref)[4]) {
  int c = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) c += ref[k] >= 0 && ref[k] != NODE4_EMPTY ? 1 : 0;
  return c;
}

// One block: levels from *cq.level on (head: from the root, while a level has
// at most COLLAPSE_BLOCK nodes; else all that are left, then the header).
__global__ void __launch_bounds__(PLOC_TAIL) k_collapse_block(const Node* bin, Node4* out, NodeQ* outq, Collapse cq,
                                                              int head, int wide, BvhHeader* h) {
  __shared__ int lds[PLOC_TAIL / 64];
  const int tid = (int)threadIdx.x;
  int level = 0, start = 0, count = 1;
  if (head) {
    for (int k = tid; k <= COLLAPSE_MAXL; k += PLOC_TAIL) cq.counts[k] = k == 0 ? 1 : 0;
    if (tid == 0) cq.job[0] = 0;
  } else {
    level = *cq.level + wide;
    // (the wide launches may have reached past the last level)
    int l = 0;
    while (l < level && cq.counts[l] > 0) start += cq.counts[l++];
    level = l;
    count = cq.counts[level];
  }
  __syncthreads();
  while (count > 0 && !(head && count > COLLAPSE_BLOCK)) {
    int next = 0;
    for (int base = 0; base < count; base += PLOC_TAIL) {
      const int m = start + base + tid;
      const bool on = base + tid < count;
      int ref[4] = {-1, -1, -1, -1};
      float lo[4][3], hi[4][3];
      if (on) collapse_children(bin, cq.job[m], ref, lo, hi);
      int tot;
      const int off = tail_scan(on ? internal_children(ref) : 0, lds, tot);
      if (on) collapse_write(out, outq, cq.job, m, start + count + next + off, ref, lo, hi);
      next += tot;
    }
    __syncthreads();
    start += count;
    count = next;
    ++level;
    if (tid == 0) cq.counts[level] = count;
  }
  if (tid == 0) {
    if (head) *cq.level = level;
    if (count == 0) {
      h->n_nodes4 = start;
      h->depth4 = level;
    }
  }
}

// Level *cq.level + w over the whole chip.
__global__ void __launch_bounds__(256) k_collapse_level(const Node* bin, Node4* out, NodeQ* outq, Collapse cq, int w) {
  __shared__ int lds[4], first;
  const int level = *cq.level + w;
  const int count = cq.counts[level];
  int start = 0;
  for (int k = 0; k < level; ++k) start += cq.counts[k];
  for (int base = (int)blockIdx.x * 256; base < count; base += (int)gridDim.x * 256) {
    const int m = start + base + (int)threadIdx.x;
    const bool on = base + (int)threadIdx.x < count;
    int ref[4] = {-1, -1, -1, -1};
    float lo[4][3], hi[4][3];
    if (on) collapse_children(bin, cq.job[m], ref, lo, hi);
    int tot;
    const int off = scan_pair(on ? internal_children(ref) : 0, lds, &tot);
    if (threadIdx.x == 0) first = tot ? atomicAdd(&cq.counts[level + 1], tot) : 0;
    __syncthreads();
    if (on) collapse_write(out, outq, cq.job, m, start + count + first + off, ref, lo, hi);
    __syncthreads();
  }
}

// Refit of 4-wide boxes from the binary tree (internal children) and the
// surfel boxes (leaves).
__global__ void k_node4_boxes(const Node* bin, Node4* out, NodeQ* outq, const BvhHeader* h, const float4* box,
                              const int32_t* perm) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= h->n_nodes4) return;
  Node4& nd = out[m];
  const int s[4] = {nd.src.x, nd.src.y, nd.src.z, nd.src.w};
  const int ref[4] = {nd.ref.x, nd.ref.y, nd.ref.z, nd.ref.w};
  float* bf = reinterpret_cast<float*>(nd.b);
  float lo[4][3] = {}, hi[4][3] = {};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (s[k] == NODE4_EMPTY) continue;
    if (s[k] >= 0) {
      float l2[3], h2[3];
      child_box(bin[s[k]], 0, lo[k], hi[k]);
      child_box(bin[s[k]], 1, l2, h2);
      for (int a = 0; a < 3; ++a) {
        lo[k][a] = fminf(lo[k][a], l2[a]);
        hi[k][a] = fmaxf(hi[k][a], h2[a]);
      }
    } else {
      const int64_t i = perm[~s[k]];
      const float4 L = box[2 * i], H = box[2 * i + 1];
      lo[k][0] = L.x; lo[k][1] = L.y; lo[k][2] = L.z;
      hi[k][0] = H.x; hi[k][1] = H.y; hi[k][2] = H.z;
    }
    for (int a = 0; a < 3; ++a) {
      bf[k * 6 + a] = lo[k][a];
      bf[k * 6 + 3 + a] = hi[k][a];
    }
  }
  write_nodeq(outq + m, lo, hi, ref);
}

inline unsigned blocks(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

struct BuildWs {
  int32_t* cl[2];          // cluster orders; the collapse's jobs afterwards
  int32_t* counts;         // collapse: nodes of each level, then its first wide level
  float4* box;
  uint64_t* codes_in;
  uint64_t* codes_out;
  uint32_t* ids_in;
  int32_t* nn;
  float4* cbox[2];         // cluster boxes; before them, the records in the caller's order
  int2* bsum;
  PlocState* ploc;
  void* sort_tmp;
  size_t sort_bytes;
  size_t bytes;
};

BuildWs build_ws(void* base, int64_t n) {
  Carver c(base, ~size_t(0));
  BuildWs w;
  w.cl[0] = c.take<int32_t>(n);
  w.cl[1] = c.take<int32_t>(n);
  w.counts = c.take<int32_t>(COLLAPSE_MAXL + 2);
  w.box = c.take<float4>(2 * n);
  w.codes_in = c.take<uint64_t>(n);
  w.codes_out = c.take<uint64_t>(n);
  w.ids_in = c.take<uint32_t>(n);
  w.nn = c.take<int32_t>(n);
  w.cbox[0] = c.take<float4>(4 * n);
  w.cbox[1] = w.cbox[0] + 2 * n;
  w.bsum = c.take<int2>(PLOC_GRID);
  w.ploc = c.take<PlocState>(2);
  w.sort_bytes = sort_pairs_bytes(n);
  w.sort_tmp = c.take<char>(w.sort_bytes);
  w.bytes = c.bytes();
  return w;
}

static_assert(sizeof(Record) <= 4 * sizeof(float4), "the records fit the cluster boxes' memory");

// The clustering's state in the build workspace.
Ploc ploc_ws(const BuildWs& w) {
  Ploc P;
  for (int k = 0; k < 2; ++k) {
    P.cl[k] = w.cl[k];
    P.cb[k] = w.cbox[k];
  }
  P.nn = w.nn;
  P.bsum = w.bsum;
  P.st = w.ploc;
  return P;
}

// Levels the collapse launches over the whole chip: none where the single
// block takes every level, else about those with more than COLLAPSE_BLOCK
// nodes (a 4-wide level has 2 to 3 times the nodes of the one above it, and the
// tree ends some levels below its widest). Any number is right: the last block
// takes what is left.
int wide_levels(int64_t n) {
  int w = 0;
  for (double m = (double)n; m > 2 * COLLAPSE_BLOCK; m *= 0.45) ++w;
  return w ? w + 4 : 0;
}
static_assert(PLOC_ITERS + 23 < COLLAPSE_MAXL, "the collapse covers the deepest tree of 2^23 surfels");
static_assert(PLOC_ITERS + 23 <= PLOC_LEVELS, "levels has an entry per clustering iteration of 2^23 surfels");

}  // namespace

BvhLayout bvh_layout(void* base, int64_t n) {
  Carver c(base, ~size_t(0));
  BvhLayout l;
  l.hdr = c.take<BvhHeader>(1);
  l.nodes = c.take<Node>(n > 1 ? n - 1 : 1);
  l.nodes4 = c.take<Node4>(n > 1 ? n - 1 : 1);
  l.nodesq = c.take<NodeQ>(n > 1 ? n - 1 : 1);
  l.recs = c.take<Record>(n);
  l.perm = c.take<int32_t>(n);
  l.inv = c.take<int32_t>(n);
  l.levels = c.take<int32_t>(PLOC_LEVELS + 1);
  l.bytes = c.bytes();
  return l;
}

void bvh_attach(eag_bvh* b, const BvhLayout& l) {
  b->hdr = l.hdr;
  b->nodes = l.nodes;
  b->nodes4 = l.nodes4;
  b->nodesq = l.nodesq;
  b->recs = l.recs;
  b->perm = l.perm;
  b->inv = l.inv;
  b->levels = l.levels;
}

size_t build_ws_bytes(int64_t n) { return build_ws(nullptr, n).bytes; }

void validate_surfels(const eag_surfels* s) {
  if (!s) fail(EAG_ERR_INVALID_ARGUMENT, "surfels is null");
  if (s->n < 1 || s->n > (int64_t(1) << 23)) fail(EAG_ERR_INVALID_ARGUMENT, "surfel count must be in [1, 2^23]");
  if (!s->pos || !s->rot || !s->scale || !s->opacity || !s->albedo || !s->radiance || !s->emissive)
    fail(EAG_ERR_INVALID_ARGUMENT, "a surfel array pointer is null");
}

void build_bvh(const eag_surfels* s, eag_bvh* b, void* ws, size_t ws_bytes, hipStream_t st) {
  const int64_t n = s->n;
  if (!b->hdr || !b->nodes || !b->nodes4 || !b->nodesq || !b->recs || !b->perm || !b->inv || !b->levels)
    fail(EAG_ERR_INTERNAL, "bvh handle without its device arrays");
  const BuildWs w = build_ws(ws, n);
  if (ws_bytes < w.bytes) fail(EAG_ERR_WORKSPACE_TOO_SMALL, "build workspace too small");
  Record* const raw = reinterpret_cast<Record*>(w.cbox[0]);
  hipLaunchKernelGGL(k_init_header, dim3(1), dim3(64), 0, st, b->hdr);
  hipLaunchKernelGGL(k_boxes, dim3(std::min(blocks(n), BOX_GRID)), dim3(256), 0, st, *s, 3.0f, w.box, raw, b->hdr);
  hipLaunchKernelGGL(k_morton, dim3(blocks(n)), dim3(256), 0, st, *s, b->hdr, w.codes_in, w.ids_in);
  sort_pairs_u64(w.codes_in, w.codes_out, w.ids_in, reinterpret_cast<uint32_t*>(b->perm), n, 63, w.sort_tmp,
                 w.sort_bytes, st);
  // (before the clustering, which takes the records' memory for its boxes)
  hipLaunchKernelGGL(k_records, dim3(blocks(n)), dim3(256), 0, st, n, b->perm, raw, b->recs, b->inv);
  b->root = n > 1 ? 0 : ~0;
  if (n > 1) {
    const Ploc P = ploc_ws(w);
    hipLaunchKernelGGL(k_ploc_init, dim3(blocks(n)), dim3(256), 0, st, n, w.box, b->perm, P);
    const unsigned g = std::min<unsigned>(blocks(n, PLOC_TILE), (unsigned)PLOC_GRID);
    const int wide = wide_iters(n);
    for (int t = 0; t < wide; ++t) {
      hipLaunchKernelGGL(k_ploc_pairs, dim3(g), dim3(PLOC_TILE), 0, st, P, t, search_limit(t, wide));
      hipLaunchKernelGGL(k_ploc_write, dim3(g), dim3(PLOC_TILE), 0, st, P, t, b->levels, n, b->nodes);
    }
    hipLaunchKernelGGL(k_ploc_tail, dim3(1), dim3(PLOC_TAIL), 0, st, P, n, b->nodes, wide, PLOC_ITERS + b->idx_bits,
                       b->levels, b->hdr);
    const Collapse cq{w.cl[0], w.counts, w.counts + COLLAPSE_MAXL + 1};
    const int levels = wide_levels(n);
    hipLaunchKernelGGL(k_collapse_block, dim3(1), dim3(PLOC_TAIL), 0, st, b->nodes, b->nodes4, b->nodesq, cq, 1, 0,
                       b->hdr);
    for (int k = 0; k < levels; ++k)
      hipLaunchKernelGGL(k_collapse_level, dim3(std::min<unsigned>(blocks(n), 1024u)), dim3(256), 0, st, b->nodes,
                         b->nodes4, b->nodesq, cq, k);
    if (levels)
      hipLaunchKernelGGL(k_collapse_block, dim3(1), dim3(PLOC_TAIL), 0, st, b->nodes, b->nodes4, b->nodesq, cq, 0,
                         levels, b->hdr);
  }
  check_hip(hipGetLastError(), "build launch");
  check_hip(hipEventRecord(b->built, st), "build event");
}

void refit_bvh(const eag_surfels* s, eag_bvh* b, void* ws, size_t ws_bytes, hipStream_t st) {
  const int64_t n = s->n;
  if (!b->hdr || !b->nodes || !b->nodes4 || !b->nodesq || !b->recs || !b->perm || !b->levels)
    fail(EAG_ERR_INTERNAL, "bvh handle without its device arrays");
  const BuildWs w = build_ws(ws, n);
  if (ws_bytes < w.bytes) fail(EAG_ERR_WORKSPACE_TOO_SMALL, "refit workspace too small");
  BvhHeader* h = b->hdr;
  Record* const raw = reinterpret_cast<Record*>(w.cbox[0]);
  // bounds are recomputed; the depths and node count stay, since the
  // topology is unchanged
  hipLaunchKernelGGL(k_reset_bounds, dim3(1), dim3(64), 0, st, h);
  hipLaunchKernelGGL(k_boxes, dim3(std::min(blocks(n), BOX_GRID)), dim3(256), 0, st, *s, 3.0f, w.box, raw, h);
  hipLaunchKernelGGL(k_records, dim3(blocks(n)), dim3(256), 0, st, n, b->perm, raw, b->recs, (int32_t*)nullptr);
  if (n > 1) {
    // iteration by iteration of the clustering that made the tree
    const unsigned g = std::min<unsigned>(blocks(n), 1024u);
    const int iters = PLOC_ITERS + b->idx_bits, wide = wide_iters(n);
    for (int t = 0; t < wide; ++t)
      hipLaunchKernelGGL(k_refit_level, dim3(g), dim3(256), 0, st, n, w.box, b->perm, b->nodes, b->levels, t);
    hipLaunchKernelGGL(k_refit_tail, dim3(1), dim3(PLOC_TAIL), 0, st, n, w.box, b->perm, b->nodes, b->levels, wide,
                       iters);
    // (the 4-wide node count is on the device: the grid covers the n - 1 it
    // can reach)
    hipLaunchKernelGGL(k_node4_boxes, dim3(blocks(n - 1)), dim3(256), 0, st, b->nodes, b->nodes4, b->nodesq, h,
                       w.box, b->perm);
  }
  check_hip(hipGetLastError(), "refit launch");
  check_hip(hipEventRecord(b->built, st), "refit event");
}

void pack_attrs(const eag_surfels* s, const eag_bvh* b, Attr* attrs, hipStream_t st) {
  hipLaunchKernelGGL(k_attrs, dim3(blocks(s->n)), dim3(256), 0, st, *s, b->inv, attrs);
}

}  // namespace eag
