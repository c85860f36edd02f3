// Device-side building blocks shared by the build, trace, render and path
// tracing kernels: Philox4x32-10, camera rays, the hemisphere frame and
// cosine-weighted sampling, the BVH node and surfel record layouts, and the
// per-ray traversal + k-buffer + compositing core.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace eag {

constexpr int KBUF = 16;          // k-buffer depth
// Traversal stack: 3 entries per level of the deepest tree a build can make
// (64 clustering iterations plus at most 23 halving iterations, each adding
// at most one level, so at most 87 levels), so that no tree needs a check on
// the host. Entries past the LDS part live in
// private memory and are rarely touched.
constexpr int STACK_SIZE = 264;

// ---------------------------------------------------------------------------
// Layouts in HBM
// ---------------------------------------------------------------------------
// Internal node, 64 B: both children's boxes and references. A reference
// c >= 0 is an internal node, c < 0 is a leaf holding the surfel at sorted
// (Morton) position ~c.
struct __align__(16) Node {
  float4 a;   // lo0.x lo0.y lo0.z hi0.x
  float4 b;   // hi0.y hi0.z lo1.x lo1.y
  float4 c;   // lo1.z hi1.x hi1.y hi1.z
  int4 d;     // child0 child1 - -
};

// 4-wide node, 128 B, collapsed from the binary tree: child k's box is
// floats [6k, 6k+6) of b (lo.xyz, hi.xyz); ref.k >= 0 is a 4-wide node,
// ref.k < 0 a leaf holding the surfel at sorted position ~ref.k, and
// NODE4_EMPTY an unused slot. src.k is the binary-tree reference the child
// came from (used to refit boxes).
constexpr int NODE4_EMPTY = 0x7fffffff;
struct __align__(16) Node4 {
  float4 b[6];
  int4 ref;
  int4 src;
};

// What a traversal reads of a 4-wide node, 64 B: the children's boxes as
// 8-bit steps from the node's lower corner (the compression of Ylitie, Karras
// and Laine, HPG 2017), and their references. Along axis
// a, child k spans [o + qlo step, o + qhi step] with step a power of two, which
// holds its box with a margin (write_nodeq). q.a holds axis a's lower steps, q.(3 + a)
// its upper ones, child k in byte k. exps has the steps' biased exponents in
// bytes 0 to 2; 255 (step +inf, all q 0) makes every plane of the axis a NaN,
// which bounds nothing: an axis on which the box is not finite.
// A visit is limited by the L1, which takes one lane's 16-byte access a cycle
// when 64 lanes read 64 places: 4 of them here, where the exact boxes take 7.
struct __align__(16) NodeQ {
  float ox, oy, oz;
  uint32_t exps;
  uint32_t q[6];
  int32_t ref[4];
  int32_t pad[2];
};
static_assert(sizeof(NodeQ) == 64, "one node per half cache line");

// The node as the traversal reads it, from its children's boxes. node_test finds
// a plane as q (step / W) + (o - O) / W, so its error in space is, beside a few
// ulp of the plane itself and of the ray (inside the pad of the leaf box and the
// widened exit), one ulp of the corner o: a node that reaches far beyond a leaf
// would lose hits on the leaf's edge. So every plane lies at least 2^-22 of the
// node's largest coordinate (four units of rounding) outside its box. Without it
// 11, 800 and 1711 of 4000 rays through the outermost points of a leaf whose
// edge lies on a step were lost at corners 10^3, 10^4 and 10^5 away; with it
// none. An axis that is not finite (a surfel at infinity or not a number) bounds
// nothing.
__host__ __device__ __forceinline__ void write_nodeq(NodeQ* out, const float (&lo)[4][3], const float (&hi)[4][3],
                                                     const int (&ref)[4]) {
  NodeQ nq;
  float o[3];
  nq.exps = 0u;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float l = __builtin_inff(), h = -__builtin_inff();
    for (int k = 0; k < 4; ++k) {
      if (ref[k] == NODE4_EMPTY) continue;
      l = fminf(l, lo[k][a]);
      h = fmaxf(h, hi[k][a]);
    }
    uint32_t ql = 0u, qh = 0u;
    if (fabsf(l) < 1e18f && fabsf(h) < 1e18f && h >= l) {
      const double m = 0x1p-22 * (double)fmaxf(fabsf(l), fabsf(h));
      const double l_m = (double)l - m;
      o[a] = (float)l_m;
      if ((double)o[a] > l_m) o[a] = nextafterf(o[a], -__builtin_inff());
      const double ext = (double)h + m - (double)o[a];
      // the smallest step with ext <= 255 steps (at least 2^-126: a normal float)
      int e = 0;
      const double f = frexp(ext, &e);   // ext = f 2^e, f in [1/2, 1) (0 for 0)
      e = ext > 0.0 ? e - (f > 255.0 / 256.0 ? 7 : 8) : -126;
      if (e < -126) e = -126;
      const double inv = ldexp(1.0, -e);
      for (int k = 0; k < 4; ++k) {
        // an empty slot, and a box that is not a number, span the node
        double a0 = floor(((double)lo[k][a] - m - (double)o[a]) * inv), a1 = ceil(((double)hi[k][a] + m - (double)o[a]) * inv);
        if (ref[k] == NODE4_EMPTY || !(a0 >= 0.0 && a0 <= 255.0)) a0 = 0.0;
        if (ref[k] == NODE4_EMPTY || !(a1 >= 0.0 && a1 <= 255.0)) a1 = 255.0;
        ql |= (uint32_t)a0 << (8 * k);
        qh |= (uint32_t)a1 << (8 * k);
      }
      nq.exps |= (uint32_t)(e + 127) << (8 * a);
    } else {
      o[a] = 0.0f;
      nq.exps |= 255u << (8 * a);
    }
    nq.q[a] = ql;
    nq.q[3 + a] = qh;
  }
  nq.ox = o[0];
  nq.oy = o[1];
  nq.oz = o[2];
  for (int k = 0; k < 4; ++k) nq.ref[k] = ref[k];
  nq.pad[0] = nq.pad[1] = 0;
  *out = nq;
}


// Geometry record of one surfel in sorted order, 48 B (three float4 loads):
//   p.x p.y p.z sigma | q.w q.x q.y q.z | s_u s_v index -
// with q the caller's (unnormalised) quaternion and index the original surfel
// index. Frames are derived in double precision at use (surfel_geo), so the
// tracer sees exactly the float32 inputs, like the float64 definition.
struct __align__(16) Record {
  float4 p_sigma;
  float4 q;
  float4 s_idx;
};

// Attributes of one surfel in sorted order, 32 B: rho.xyz e | r.xyz -
struct __align__(16) Attr {
  float4 rho_e;
  float4 r;
};

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): published multipliers and key
// increments, ten rounds. Counter (pixel, sample, segment, stream id).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
    const uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
    c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
  }
  return c;
}
// u = (w >> 8) * 2^-24, exact in float32
__device__ __forceinline__ float to_unit(uint32_t w) { return (float)(w >> 8) * (1.0f / 16777216.0f); }

// ---------------------------------------------------------------------------
// small vector helpers
// ---------------------------------------------------------------------------
struct V3 { float x, y, z; };
__host__ __device__ __forceinline__ V3 v3(float x, float y, float z) { return V3{x, y, z}; }
__device__ __forceinline__ V3 operator+(V3 a, V3 b) { return V3{a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3 operator-(V3 a, V3 b) { return V3{a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 operator*(float s, V3 a) { return V3{s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ float dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ V3 cross(V3 a, V3 b) {
  return V3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}

// double-precision vectors for ray geometry
struct D3 { double x, y, z; };
__host__ __device__ __forceinline__ D3 d3(double x, double y, double z) { return D3{x, y, z}; }
__device__ __forceinline__ D3 operator+(D3 a, D3 b) { return D3{a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ D3 operator-(D3 a, D3 b) { return D3{a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ D3 operator*(double s, D3 a) { return D3{s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ double dot(D3 a, D3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ D3 cross(D3 a, D3 b) {
  return D3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}

// Pinhole camera prepared on the host in double precision: ray direction =
// normalize(dx * right + dy * up + fwd) with dx = 2 (x + ox) / W - 1,
// dy = 1 - 2 (y + oy) / H; right and up are pre-scaled by tan(vfov/2) * W/H
// and tan(vfov/2).
struct CamDev {
  double eye[3], right[3], up[3], fwd[3];
  int32_t width, height;
  uint32_t id;
  int32_t pad;
};

__device__ __forceinline__ D3 camera_dir(const CamDev& c, int px, int py, double ox, double oy) {
  const double dx = 2.0 * ((double)px + ox) / (double)c.width - 1.0;
  const double dy = 1.0 - 2.0 * ((double)py + oy) / (double)c.height;
  // (fused in one way, written out: a path has the same ray in every kernel)
  const D3 d = d3(fma(dy, c.up[0], dx * c.right[0]) + c.fwd[0], fma(dx, c.right[1], dy * c.up[1]) + c.fwd[1],
                  fma(dx, c.right[2], dy * c.up[2]) + c.fwd[2]);
  return (1.0 / sqrt(fma(d.z, d.z, fma(d.x, d.x, d.y * d.y)))) * d;
}

// Hemisphere frame: Gram-Schmidt of the fixed helper h = (1,2,3)/sqrt(14)
// against the unit normal n: b1 = normalize(h - (h.n) n), b2 = n x b1.
// Cosine-weighted direction (Malley): r = sqrt(u0), phi = 2 pi u1,
// w' = r cos(phi) b1 + r sin(phi) b2 + sqrt(1 - u0) n.
constexpr double HX = 0.2672612419124244, HY = 0.5345224838248488, HZ = 0.8017837257372732;
constexpr double TWO_PI = 6.283185307179586;

__device__ __forceinline__ D3 cosine_dir(D3 n, double u0, double u1) {
  const double hn = fma(HZ, n.z, fma(HX, n.x, HY * n.y));
  const D3 m = d3(fma(-hn, n.x, HX), fma(-hn, n.y, HY), fma(-hn, n.z, HZ));
  const D3 b1 = (1.0 / sqrt(fma(m.z, m.z, fma(m.x, m.x, m.y * m.y)))) * m;
  const D3 b2 = d3(fma(n.y, b1.z, -(n.z * b1.y)), fma(n.z, b1.x, -(n.x * b1.z)), fma(n.x, b1.y, -(n.y * b1.x)));
  const double r = sqrt(u0);
  double s, c;
  sincos(TWO_PI * u1, &s, &c);
  const double z = sqrt(1.0 - u0);
  return d3(fma(z, n.x, fma(r * c, b1.x, r * s * b2.x)), fma(z, n.y, fma(r * c, b1.y, r * s * b2.y)),
            fma(z, n.z, fma(r * c, b1.z, r * s * b2.z)));
}

// Element i of an array of at most 4 GiB (2^23 surfels: 1 GiB of nodes at
// most). A 32-bit byte offset beside a uniform base is an addressing mode of
// its own; a 64-bit one costs each lane its address arithmetic and registers.
template <class T>
__host__ __device__ __forceinline__ const T* elem(const T* base, uint32_t i) {
  return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (uint32_t)(i * (uint32_t)sizeof(T)));
}

// ---------------------------------------------------------------------------
// Order key: (bucket, original index) packed into 64 bits, bucket =
// floor(t / dq) (dq a power of two) or the float bits of t when dq == 0.
// Ordering keys as integers orders hits by (bucket, index); the sorted
// position that addresses the record comes from the tree's inverse
// permutation when the hit is blended. At most 32 + 23 bits are used, and bit
// 62 is set, so that every key is also the bit pattern of a positive normal
// double and doubles order like the keys: v_min_f64 and v_max_f64 compare and
// move a key in one instruction each, where a 64-bit integer comparison takes
// five with its four selects.
// ---------------------------------------------------------------------------
constexpr uint64_t KEY_BIAS = 0x4000000000000000ull;
constexpr uint64_t KEY_NONE = 0x7ff0000000000000ull;   // +inf: above every key

// (Written as instructions: from fmin the compiler makes a third one per
// operand that quiets a NaN no key can be.)
__device__ __forceinline__ uint64_t key_min(uint64_t a, uint64_t b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(__longlong_as_double((long long)a)), "v"(__longlong_as_double((long long)b)));
  return (uint64_t)__double_as_longlong(r);
}
__device__ __forceinline__ uint64_t key_max(uint64_t a, uint64_t b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(__longlong_as_double((long long)a)), "v"(__longlong_as_double((long long)b)));
  return (uint64_t)__double_as_longlong(r);
}

struct TraceCtx {
  const NodeQ* nodes;
  const Record* recs;
  const Attr* attrs;
  const int32_t* inv;      // sorted position of each surfel
  int32_t root;            // >= 0: internal node index; < 0: single leaf ~root
  int32_t idx_bits;        // bits of an index
  uint32_t max_bucket;     // largest representable bucket
  double inv_dq;           // 1 / dq, or 0 for exact-t keys
  double dq;               // the depth quantum (a power of two, so b * dq == b / inv_dq exactly), or 0
  double t_min;
  double k2;               // k_sigma^2
  double T_min;
  // Mapped host word receiving device status codes (a key beyond the last
  // bucket); null: not reported.
  unsigned int* status;
  // Per-lane hit lists (segments without one: null), HL_CAP entries each; this lane's
  // begin at entry hl_at. A lane's entries are contiguous: appends happen at
  // different times in different lanes, and a lane filling its own cache
  // lines writes each line back once.
  uint64_t* hl;
  uint32_t hl_at;
  uint32_t hl_bytes;       // of all lanes' lists
};

constexpr int HL_CAP = 256;        // entries per lane (a multiple of 8: the list is scanned 8 at a time)
static_assert(HL_CAP % 8 == 0, "hit-list scan reads 8 contiguous entries");
// An offset past every hit-list buffer (256 MiB on 256 CUs), and an operand that
// needs no register: the buffer's size in its place cost path tracing 0.4%.
constexpr uint32_t HL_DROP = 0x40000000u;

__device__ __forceinline__ void report_key_range(unsigned int* status) {
  if (status) __hip_atomic_fetch_or(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Write v to entry j of this lane's hit list if `on`. One instruction that
// every lane issues (a lane that is not on passes an offset past the buffer's
// end, which the buffer store drops by definition; not one near 2^32, whose
// second word would rest on how an address wraps): behind a branch, the
// compiler could not count the stores in flight, and would wait for all of
// them before it uses a record loaded earlier.
__device__ __forceinline__ void hl_store(const TraceCtx& tc, int j, uint64_t v, bool on) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 w = {(uint32_t)v, (uint32_t)(v >> 32)};
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(tc.hl, 0, (int)tc.hl_bytes, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b64(w, rs, (int)(on ? (tc.hl_at + (uint32_t)j) * 8u : HL_DROP), 0, 0);
}
__device__ __forceinline__ uint64_t pack_key(const TraceCtx& tc, uint32_t bucket, uint32_t idx) {
  return ((uint64_t)bucket << tc.idx_bits) | (uint64_t)idx | KEY_BIAS;
}
__device__ __forceinline__ uint64_t make_key(const TraceCtx& tc, double t, uint32_t idx) {
  // (both kinds of bucket: a branch would split the leaf test)
  const double b = floor(t * tc.inv_dq);
  const uint32_t bq = b >= (double)tc.max_bucket ? tc.max_bucket : (uint32_t)b;
  const uint32_t bt = __float_as_uint((float)t);
  return pack_key(tc, tc.inv_dq > 0.0 ? bq : bt, idx);
}
__device__ __forceinline__ uint64_t make_key_b(const TraceCtx& tc, uint32_t bucket, uint32_t idx) {
  return pack_key(tc, bucket >= tc.max_bucket ? tc.max_bucket : bucket, idx);
}
__device__ __forceinline__ uint32_t key_idx(const TraceCtx& tc, uint64_t k) {
  return (uint32_t)k & ((1u << tc.idx_bits) - 1u);
}
__device__ __forceinline__ uint32_t key_bucket(const TraceCtx& tc, uint64_t k) {
  return (uint32_t)(k >> tc.idx_bits);   // (the bias lies above the 32 bits kept)
}
// first key of the bucket after k's (saturating at the last bucket, which the
// hit list then never claims to cover)
__device__ __forceinline__ uint64_t next_bucket_key(const TraceCtx& tc, uint64_t k) {
  const uint32_t b = key_bucket(tc, k);
  return make_key_b(tc, b < tc.max_bucket ? b + 1u : tc.max_bucket, 0u);
}
// smallest t that can carry the given key's bucket (for culling)
__device__ __forceinline__ float key_tlo(const TraceCtx& tc, uint64_t k) {
  const uint32_t b = key_bucket(tc, k);
  const float tq = (float)((double)b * tc.dq);
  return tc.inv_dq > 0.0 ? tq : __uint_as_float(b);
}
// largest t whose bucket does not exceed the key's bucket
__device__ __forceinline__ float key_thi(const TraceCtx& tc, uint64_t k) {
  const uint32_t b = key_bucket(tc, k);
  const float tq = (float)((double)(b + 1u) * tc.dq);
  return tc.inv_dq > 0.0 ? tq : __uint_as_float(b);
}

// ---------------------------------------------------------------------------
// Ray-surfel geometry on the tangent plane (Eq. 1). Decisions and blended
// quantities are evaluated in double precision: the local coordinates come
// from a difference of nearly equal distances, and float32 there would cost
// ~1e-5 in u at room scale, which the bounce point and direction then
// amplify. Every candidate takes the double-precision test, straight-line:
// a wave nearly always holds some candidate whose decision a float32
// evaluation could not settle, so a float screen in front of it only added
// instructions.
// ---------------------------------------------------------------------------
__device__ __forceinline__ Record load_record(const Record* recs, uint32_t pos) {
  const float4* p = reinterpret_cast<const float4*>(elem(recs, pos));
  Record r;
  r.p_sigma = p[0];
  r.q = p[1];
  r.s_idx = p[2];
  return r;
}

__device__ __forceinline__ uint32_t rec_index(const Record& r) { return __float_as_uint(r.s_idx.z); }

// A surfel's geometry in double precision (Sec. 3.1), as the adjoint's chain
// rule needs it: centre p, tangent axes t_u, t_v = the first two columns of
// the rotation of q / |q|, normal n = t_u x t_v, scales, and the normalised
// quaternion.
struct Geo {
  D3 p, tu, tv, n;
  double su, sv, sigma;
  double qw, qx, qy, qz, iq;   // unit quaternion and 1 / |q|
};

__device__ __forceinline__ Geo surfel_geo(const Record& r) {
  Geo g;
  g.p = d3(r.p_sigma.x, r.p_sigma.y, r.p_sigma.z);
  g.sigma = r.p_sigma.w;
  double w = r.q.x, x = r.q.y, y = r.q.z, z = r.q.w;
  g.iq = 1.0 / sqrt(w * w + x * x + y * y + z * z);
  w *= g.iq; x *= g.iq; y *= g.iq; z *= g.iq;
  g.qw = w; g.qx = x; g.qy = y; g.qz = z;
  g.tu = d3(1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y + w * z), 2.0 * (x * z - w * y));
  g.tv = d3(2.0 * (x * y - w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z + w * x));
  g.n = cross(g.tu, g.tv);
  g.su = r.s_idx.x;
  g.sv = r.s_idx.y;
  return g;
}

// ---------------------------------------------------------------------------
// Segment result: the traced quantities of Eq. 3 before normalisation.
// ---------------------------------------------------------------------------
struct SegOut {
  D3 N;
  double D;
  D3 R;
  double E;
  D3 P;
  double T;
  int32_t nhits;
  int32_t rounds;
  int32_t tests;
  int32_t visits;
};

enum { Q_ALL = 0, Q_RADIANCE = 1 };

// byte k as a float (one conversion instruction)
__host__ __device__ __forceinline__ float q_byte(uint32_t w, int k) { return (float)((w >> (8 * k)) & 255u); }

// Slab test of a box against [tlo, thi]; returns the entry distance or +inf.
// (for exact boxes: the light pdf's tree; node_visit has its own over NodeQ)
// OiW = O * iW per component: each plane distance (l - O) / W is one fused
// multiply-add, l * iW - OiW. Its rounding error, in space, is a few ulp of
// |O| and |l|, far inside the pad that every leaf box carries around its
// ellipse, so no box that a ray's hit lies in is rejected.
__device__ __forceinline__ float slab(float lx, float ly, float lz, float hx, float hy, float hz, V3 OiW, V3 iW,
                                      float tlo, float thi) {
  const float ax = fmaf(lx, iW.x, -OiW.x), bx = fmaf(hx, iW.x, -OiW.x);
  const float ay = fmaf(ly, iW.y, -OiW.y), by = fmaf(hy, iW.y, -OiW.y);
  const float az = fmaf(lz, iW.z, -OiW.z), bz = fmaf(hz, iW.z, -OiW.z);
  const float tn = fmaxf(fmaxf(fminf(ax, bx), fminf(ay, by)), fmaxf(fminf(az, bz), tlo));
  // widen the exit so that rounding (and the float32 copy of the ray) never
  // rejects a box the ray touches
  const float tf = fminf(fminf(fmaxf(ax, bx), fmaxf(ay, by)), fminf(fmaxf(az, bz), thi)) * 1.000002f + 1e-6f;
  return tn <= tf ? tn : __builtin_inff();
}

// No per-hit callback (forward passes).
struct NoHit {
  static constexpr bool kHits = false;
  __device__ __forceinline__ void operator()(const Record&, const Attr&, double, double, double, double, D3, D3) const {}
};

// Traversal stack: the top STACK_LDS entries of every lane live in LDS,
// strided by the thread index so that a wave's pushes hit distinct banks;
// deeper entries (rare) spill to a private array.
constexpr int STACK_LDS = 24;
constexpr int TRACE_BLOCK = 256;   // every tracing kernel runs 256-thread blocks
constexpr int PEND = 32;           // postponed leaves per lane

// The overflow array is the caller's (a private array of the kernel): kept
// out of this struct so that the struct itself stays in registers.
constexpr int STACK_OVF = STACK_SIZE - STACK_LDS;
struct TravStack {
  int* lds;        // this lane's column: lds[i * TRACE_BLOCK]
  int* ovf;        // this lane's overflow entries, STACK_OVF of them
  int sp;
  __device__ __forceinline__ void push(int v) {
    if (sp < STACK_LDS) lds[sp * TRACE_BLOCK] = v;
    else ovf[sp - STACK_LDS] = v;
    ++sp;
  }
  __device__ __forceinline__ int pop() {
    --sp;
    if (sp < STACK_LDS) return lds[sp * TRACE_BLOCK];
    // volatile keeps the (rare) private read a load of its own, so that the
    // common LDS read is not merged with it into a generic-address load
    return static_cast<volatile int*>(ovf)[sp - STACK_LDS];
  }
};

// Accept a candidate key into the sorted k-buffer (ascending; empty =
// KEY_NONE). Entry j becomes the median of entry j - 1, entry j and the key,
// which in a sorted buffer is max(entry j - 1, min(entry j, key)): two
// instructions per entry, none waiting for another entry's. Returns the key
// that falls off the end (the old last entry, or the candidate itself when it
// is not below it).
__device__ __forceinline__ uint64_t kbuf_insert(uint64_t (&kk)[KBUF], uint64_t key) {
  const uint64_t spill = key_max(key, kk[KBUF - 1]);
#pragma unroll
  for (int j = KBUF - 1; j > 0; --j) kk[j] = key_max(kk[j - 1], key_min(kk[j], key));
  kk[0] = key_min(kk[0], key);
  return spill;
}

// Compare-exchange: afterwards a <= b.
__device__ __forceinline__ void cswap_key(uint64_t& a, uint64_t& b) {
  const uint64_t lo = key_min(a, b);
  b = key_max(a, b);
  a = lo;
}

// Sort eight keys ascending: the 19-comparator, depth-6 sorting network for
// eight inputs (checked on all 256 zero-one inputs).
__device__ __forceinline__ void sort8_keys(uint64_t (&e)[8]) {
  cswap_key(e[0], e[2]); cswap_key(e[1], e[3]); cswap_key(e[4], e[6]); cswap_key(e[5], e[7]);
  cswap_key(e[0], e[4]); cswap_key(e[1], e[5]); cswap_key(e[2], e[6]); cswap_key(e[3], e[7]);
  cswap_key(e[0], e[1]); cswap_key(e[2], e[3]); cswap_key(e[4], e[5]); cswap_key(e[6], e[7]);
  cswap_key(e[2], e[4]); cswap_key(e[3], e[5]);
  cswap_key(e[1], e[4]); cswap_key(e[3], e[6]);
  cswap_key(e[1], e[2]); cswap_key(e[3], e[4]); cswap_key(e[5], e[6]);
}

// Merge eight ascending keys into the k-buffer, keeping its KBUF smallest.
// Against the buffer's upper half, taken in reverse, the elementwise minimum
// leaves the sixteen smallest of both as a bitonic sequence, which four
// compare-exchange stages sort: 8 minima and 32 compare-exchanges in place
// of the 128 steps of eight single inserts.
static_assert(KBUF == 16, "the merge network is built for a 16-entry k-buffer");
__device__ __forceinline__ void kbuf_merge8(uint64_t (&kk)[KBUF], const uint64_t (&e)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) kk[8 + i] = key_min(e[7 - i], kk[8 + i]);
#pragma unroll
  for (int st = 8; st >= 1; st >>= 1) {
#pragma unroll
    for (int i = 0; i < KBUF; ++i)
      if ((i & st) == 0) cswap_key(kk[i], kk[i + st]);
  }
}

// Lanes of each wave that take work: 64, or fewer when the launch has fewer
// items than the grid has lanes. A wave runs as long as the longest of its
// lanes' paths through every phase, so few items are spread over all waves.
__host__ __device__ inline int lanes_per_wave(int64_t n_work, int64_t n_waves) {
  const int64_t q = (n_work + n_waves - 1) / n_waves;
  return q < 1 ? 1 : (q > 64 ? 64 : (int)q);
}

// ---------------------------------------------------------------------------
// One ray segment: multi-round k-buffer traversal and front-to-back blending.
// Round r collects the KBUF smallest keys strictly greater than the last key
// blended in round r-1, blends them in order, and stops the segment after the
// first hit with T < T_min, or when a round returns fewer than KBUF hits.
//
// With a hit list (tc.hl), a traversal round also records every accepted key
// that the k-buffer rejects or evicts and whose depth bucket does not exceed
// that of the round's KBUF-th key. Such a round has tested every surfel of
// those buckets (boxes are culled only beyond them), so after blending the
// round the list holds every hit key in (last, lhi) with lhi the first key
// of the next bucket. A later round takes its keys from the
// list when it finds KBUF of them there, and otherwise traverses only for
// keys >= lhi; when the list holds some but fewer than KBUF such keys, they
// are blended first as a round of their own, and the traversal beyond lhi
// happens only if the segment is still open. On a surface where many
// coplanar surfels share one depth
// bucket, this turns the repeated traversals of a long segment into scans
// of a short list. If the list overflows it is dropped and rounds traverse.
//
// The steps are separate functions so that a kernel can interleave them
// across lanes (the path tracer does); trace_segment_cb runs them in order.
// ---------------------------------------------------------------------------

// Segment state carried across rounds. DACC: accumulate R, E, P in double
// (the single-bounce render, whose adjoint subtracts running prefixes from
// these totals) or in float (path tracing).
template <bool DACC>
struct Seg {
  using Acc = typename std::conditional<DACC, double, float>::type;
  D3 O, W;            // the ray, double precision
  V3 OiW;             // float origin times iW, for the slab tests
  V3 iW;              // float reciprocal direction for the box tests
  D3 N;
  double D, T;
  Acc R0, R1, R2, E, P0, P1, P2;
  uint64_t last;      // keys must exceed this (0 before the first round: below every key)
  bool done;
  int nl;             // entries in the hit list
  uint64_t lhi;       // 0: list unusable; else it holds every hit key in (last, lhi)
};

// A segment with its statistics, kept only where the caller reads them: they
// cost a register each, and registers are what the runner's waves have least
// of. LIST: it has a hit list (tc.hl is not null).
template <bool DACC, bool STATS, bool LIST>
struct SegStats : Seg<DACC> {
  static constexpr bool kStats = false, kList = LIST;
};
template <bool DACC, bool LIST>
struct SegStats<DACC, true, LIST> : Seg<DACC> {
  static constexpr bool kStats = true, kList = LIST;
  int32_t nhits, rounds, tests, visits;
};

// State of one round: the k-buffer and the traversal. Internal nodes are
// visited until a lane has PEND-4 leaves postponed, its traversal ends, or
// every lane of the wave has a leaf waiting; then the postponed leaves are
// tested, so that the costly surfel test runs for many lanes at once.
struct Round {
  uint64_t kk[KBUF];  // ascending; empty = KEY_NONE
  int cnt;
  uint64_t floor_key; // keys taken must exceed this
  uint64_t cut_key;   // hit list entries must be below this
  float t_cut;        // boxes entered beyond this cannot hold a key < kk[KBUF-1]
  float tlo0;         // boxes ending before this cannot hold a key > floor_key
  bool over;          // the hit list overflowed this round
  bool partial;       // list keys below lhi only: blend them, then traverse beyond lhi if still open
  bool trav;          // internal nodes remain (ref, then the stack)
  int ref;            // next internal node
  int np;             // postponed leaves
};

template <class S>
__host__ __device__ __forceinline__ void seg_begin(S& s, D3 O, D3 W) {
  s.O = O;
  s.W = W;
  const float wx = (float)W.x, wy = (float)W.y, wz = (float)W.z;
  s.iW = v3(1.0f / (fabsf(wx) > 1e-30f ? wx : copysignf(1e-30f, wx)),
            1.0f / (fabsf(wy) > 1e-30f ? wy : copysignf(1e-30f, wy)),
            1.0f / (fabsf(wz) > 1e-30f ? wz : copysignf(1e-30f, wz)));
  s.OiW = v3((float)O.x * s.iW.x, (float)O.y * s.iW.y, (float)O.z * s.iW.z);
  s.N = d3(0.0, 0.0, 0.0);
  s.D = 0.0;
  s.T = 1.0;
  s.R0 = s.R1 = s.R2 = s.E = s.P0 = s.P1 = s.P2 = 0;
  s.last = 0;
  s.done = false;
  s.nl = 0;
  s.lhi = 0;
  if constexpr (S::kStats) s.nhits = s.rounds = s.tests = s.visits = 0;
}

// Start a round. Returns true when it must traverse (r.trav / r.np are set
// up and the stack is empty), false when the hit list alone decides it.
template <class S>
__device__ __forceinline__ bool round_begin(const TraceCtx& tc, S& s, Round& r, TravStack& st, int* pend) {
  if constexpr (S::kStats) ++s.rounds;
#pragma unroll
  for (int j = 0; j < KBUF; ++j) r.kk[j] = KEY_NONE;
  r.cnt = 0;
  r.floor_key = s.last;
  r.over = false;
  r.partial = false;
  bool traverse = true;
  if (S::kList && s.lhi > s.last + 1) {
    // keys in (last, lhi) from the list (entries at or below last were
    // blended by earlier rounds and are skipped, not removed)
    // (loaded 8 at a time: entries up to HL_CAP are this lane's, those past
    // nl are ignored)
    const uint64_t* const hl = elem(tc.hl, tc.hl_at);
    int w = 0;
    for (int j = 0; j < s.nl; j += 8) {
      uint64_t e[8];
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(hl + j + u);
        e[u] = v.x;
        e[u + 1] = v.y;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        // branch-free: a key outside (last, lhi) enters the merge as KEY_NONE
        const bool in = j + u < s.nl && e[u] > s.last && e[u] < s.lhi;
        e[u] = in ? e[u] : KEY_NONE;
        w += in ? 1 : 0;
      }
      sort8_keys(e);
      kbuf_merge8(r.kk, e);
    }
    if (w == 0) s.nl = 0;
    // every key in range is below the buffer's last entry until it is full
    r.cnt = w > KBUF ? KBUF : w;
    if (r.cnt == KBUF || s.lhi == KEY_NONE) {
      traverse = false;
    } else if (r.cnt > 0) {
      // Every key >= lhi follows these, so they can be blended first; the
      // segment often ends among them, and then nothing beyond lhi is needed.
      traverse = false;
      r.partial = true;
    } else {
      r.floor_key = s.lhi - 1;   // (above last)
    }
  } else {
    s.nl = 0;   // no list, or every key it covers is blended (last = lhi - 1)
  }
  r.cut_key = r.cnt == KBUF ? next_bucket_key(tc, r.kk[KBUF - 1]) : KEY_NONE;
  r.t_cut = r.cnt == KBUF ? key_thi(tc, r.kk[KBUF - 1]) * 1.000002f + 1e-6f : __builtin_inff();
  const float t_floor = key_tlo(tc, r.floor_key);   // (0 for floor 0)
  r.tlo0 = fmaxf((float)tc.t_min, t_floor) * 0.99999f - 1e-6f;
  st.sp = 0;
  r.ref = tc.root;
  r.np = 0;
  r.trav = traverse && tc.root >= 0;
  if (traverse && tc.root < 0) {   // the whole scene is one surfel
    pend[0] = ~tc.root;
    r.np = 1;
  }
  return traverse;
}

// A node's children for a ray: ek holds (entry, child) of the internal ones
// the ray reaches, ordered as doubles by the entry (the float's bits in the
// high word make a finite double, +inf included; +inf for the others), ni of
// them; leaf says which children are leaves the ray reaches.
struct NodeKids {
  int c[4];
  bool leaf[4];
  uint64_t ek[4];
  int ni;
};
template <bool DACC>
__host__ __device__ __forceinline__ NodeKids node_test(const TraceCtx& tc, const Seg<DACC>& s, int ref, float tlo0, float t_cut) {
  const float4* np = reinterpret_cast<const float4*>(elem(tc.nodes, (uint32_t)ref));
  const float4 h = np[0];
  const uint4 u0 = *reinterpret_cast<const uint4*>(np + 1), u1 = *reinterpret_cast<const uint4*>(np + 2);
  const uint2 u2 = *reinterpret_cast<const uint2*>(np + 3);
  const uint32_t ex = __builtin_bit_cast(uint32_t, h.w);
  // plane distances are q a + b per axis
  const float ax = __builtin_bit_cast(float, (ex & 255u) << 23) * s.iW.x, bx = fmaf(h.x, s.iW.x, -s.OiW.x);
  const float ay = __builtin_bit_cast(float, (ex & 0xff00u) << 15) * s.iW.y, by = fmaf(h.y, s.iW.y, -s.OiW.y);
  const float az = __builtin_bit_cast(float, (ex & 0xff0000u) << 7) * s.iW.z, bz = fmaf(h.z, s.iW.z, -s.OiW.z);
  const bool gx = s.iW.x < 0.0f, gy = s.iW.y < 0.0f, gz = s.iW.z < 0.0f;
  // the four children's near and far planes
  const uint32_t nx = gx ? u0.w : u0.x, fx = gx ? u0.x : u0.w;
  const uint32_t ny = gy ? u1.x : u0.y, fy = gy ? u0.y : u1.x;
  const uint32_t nz = gz ? u1.y : u0.z, fz = gz ? u0.z : u1.y;
  NodeKids kd;
  kd.c[0] = (int)u1.z;
  kd.c[1] = (int)u1.w;
  kd.c[2] = (int)u2.x;
  kd.c[3] = (int)u2.y;
  kd.ni = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float tn = fmaxf(fmaxf(fmaf(q_byte(nx, k), ax, bx), fmaf(q_byte(ny, k), ay, by)),
                           fmaxf(fmaf(q_byte(nz, k), az, bz), tlo0));
    // widen the exit so that rounding (and the float32 copy of the ray) never
    // rejects a box the ray touches
    const float tf = fminf(fminf(fmaf(q_byte(fx, k), ax, bx), fmaf(q_byte(fy, k), ay, by)),
                           fminf(fmaf(q_byte(fz, k), az, bz), t_cut)) * 1.000002f + 1e-6f;
    const bool m = kd.c[k] != NODE4_EMPTY && tn <= tf;
    const bool mi = m && kd.c[k] >= 0;
    kd.leaf[k] = m && kd.c[k] < 0;
    kd.ek[k] = ((uint64_t)__builtin_bit_cast(uint32_t, mi ? tn : __builtin_inff()) << 32) | (uint32_t)kd.c[k];
    kd.ni += mi ? 1 : 0;
  }
  return kd;
}
__device__ __forceinline__ void sort_kids(NodeKids& kd, int (&ic)[4]) {
  cswap_key(kd.ek[0], kd.ek[1]); cswap_key(kd.ek[2], kd.ek[3]); cswap_key(kd.ek[0], kd.ek[2]);
  cswap_key(kd.ek[1], kd.ek[3]); cswap_key(kd.ek[1], kd.ek[2]);
#pragma unroll
  for (int k = 0; k < 4; ++k) ic[k] = (int)(uint32_t)kd.ek[k];
}

// Visit internal node r.ref: leaves the ray reaches are postponed, internal
// children are visited nearest first (the others pushed farthest first).
template <class S>
__device__ __forceinline__ void node_visit(const TraceCtx& tc, S& s, Round& r, TravStack& st, int* pend) {
  if constexpr (S::kStats) ++s.visits;
  NodeKids kd = node_test(tc, s, r.ref, r.tlo0, r.t_cut);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    // leaves are queued without a branch: the slot past the queue is always
    // written (nodes are visited only while np <= PEND - 4, so it exists)
    pend[r.np * TRACE_BLOCK] = ~kd.c[k];
    r.np += kd.leaf[k] ? 1 : 0;
  }
  const int ni = kd.ni;
  if (ni > 0) {
    int ic[4];
    sort_kids(kd, ic);
    // push the others farthest first: bottom to top ic[ni-1] .. ic[1]
    if (st.sp + 3 <= STACK_LDS) {
      // branch-free: three slots written, the stack grows by ni - 1
      const int v0 = ni > 3 ? ic[3] : (ni > 2 ? ic[2] : ic[1]);
      const int v1 = ni > 3 ? ic[2] : ic[1];
      st.lds[(st.sp + 0) * TRACE_BLOCK] = v0;
      st.lds[(st.sp + 1) * TRACE_BLOCK] = v1;
      st.lds[(st.sp + 2) * TRACE_BLOCK] = ic[1];
      st.sp += ni - 1;
    } else {
      if (ni > 3) st.push(ic[3]);
      if (ni > 2) st.push(ic[2]);
      if (ni > 1) st.push(ic[1]);
    }
    r.ref = ic[0];
  } else if (st.sp > 0) {
    r.ref = st.pop();
  } else {
    r.trav = false;
  }
}

// The order key of a postponed leaf (its record already loaded) for the ray
// (O, W) in a round whose keys must exceed floor_key; KEY_NONE when the surfel is missed or its key cannot enter the round. cutlim: keys
// at or above it are dropped (the k-buffer's last key, or the hit list's
// cut, a bucket's first key; any larger value is also correct).
__device__ __forceinline__ uint64_t leaf_key(const TraceCtx& tc, const Record& rec, D3 O, D3 W, uint64_t floor_key,
                                             uint64_t cutlim) {
  // The surfel test in double precision, straight-line. The columns of the
  // rotation of the unnormalised quaternion are |q|^2 (t_u, t_v, n): the
  // distance t = ((p - O).n) / (W.n) needs no normalisation, and the ellipse
  // test becomes u'^2 / s_u^2 + v'^2 / s_v^2 <= k^2 |q|^4 with
  // u' = y.(|q|^2 t_u). Its rounding differs from the normalised evaluation
  // by a few ulp, well inside the margins within which rim, t_min and bucket
  // decisions are flagged.
  // Every fused product is written out: which of two products of a sum is
  // fused went with the code around it, and t, which decides the bucket, was
  // another in the kernels for groups than in those for lanes.
  const double w = rec.q.x, x = rec.q.y, y = rec.q.z, z = rec.q.w;
  const double q2n = fma(z, z, fma(y, y, fma(w, w, x * x)));
  const D3 cu = d3(fma(-z, z, fma(-y, y, fma(w, w, x * x))), 2.0 * fma(x, y, w * z), 2.0 * fma(x, z, -(w * y)));
  const D3 cv = d3(2.0 * fma(x, y, -(w * z)), fma(-z, z, fma(y, y, fma(w, w, -(x * x)))), 2.0 * fma(y, z, w * x));
  const D3 cn = d3(2.0 * fma(x, z, w * y), 2.0 * fma(y, z, -(w * x)), fma(z, z, fma(-y, y, fma(w, w, -(x * x)))));
  const D3 d = d3((double)rec.p_sigma.x - O.x, (double)rec.p_sigma.y - O.y, (double)rec.p_sigma.z - O.z);
  const double den = fma(W.z, cn.z, fma(W.x, cn.x, W.y * cn.y));
  const double t = fma(d.z, cn.z, fma(d.y, cn.y, d.x * cn.x)) / den;
  const D3 yv = d3(fma(t, W.x, -d.x), fma(t, W.y, -d.y), fma(t, W.z, -d.z));
  const double su2 = (double)rec.s_idx.x * rec.s_idx.x, sv2 = (double)rec.s_idx.y * rec.s_idx.y;
  const double up = fma(yv.z, cu.z, fma(yv.x, cu.x, yv.y * cu.y)), vp = fma(yv.z, cv.z, fma(yv.x, cv.x, yv.y * cv.y));
  // (multiplied through by s_u^2 s_v^2, all positive: no division)
  // (&, not &&: nothing is skipped, so nothing is branched around)
  const bool hit = (fabs(den) > 1e-12 * q2n) & (rec.p_sigma.w > 0.0f) & (t > tc.t_min) &
                   (fma(up * up, sv2, vp * vp * su2) <= tc.k2 * q2n * q2n * su2 * sv2);
  const uint64_t key = make_key(tc, t, rec_index(rec));
  const bool qual = hit & (key > floor_key);
  // A hit in the last bucket may stand for a farther one that the key
  // saturated into it, whose order among the others is then unknown: the
  // launch reports it (a rare branch; never taken within the range).
  if (qual && tc.inv_dq > 0.0 && key_bucket(tc, key) >= tc.max_bucket) report_key_range(tc.status);
  return qual & (key < cutlim) ? key : KEY_NONE;
}

// Take a key into the round (KEY_NONE: nothing happens). The list needs only
// keys beyond the round's final KBUF-th key: a key goes there when the
// k-buffer rejects it or later evicts it. Everything here runs without a
// branch: a wave nearly always holds a lane for either side.
template <class S>
__device__ __forceinline__ void take_key(const TraceCtx& tc, S& s, Round& r, uint64_t key) {
  // a key not below the last entry leaves the buffer unchanged and comes back
  // as the spill
  const bool ins = key < r.kk[KBUF - 1];
  const uint64_t spill = kbuf_insert(r.kk, key);   // KEY_NONE while the buffer is not full
  r.cnt = ins && r.cnt < KBUF ? r.cnt + 1 : r.cnt;
  const bool full = r.kk[KBUF - 1] != KEY_NONE;
  const float tc_new = key_thi(tc, r.kk[KBUF - 1]) * 1.000002f + 1e-6f;
  const uint64_t ck_new = next_bucket_key(tc, r.kk[KBUF - 1]);
  r.t_cut = full ? tc_new : r.t_cut;
  r.cut_key = full ? ck_new : r.cut_key;
  if constexpr (S::kList) {
    const bool app = spill < r.cut_key;   // (KEY_NONE is not)
    const bool room = s.nl < HL_CAP;
    hl_store(tc, s.nl, spill, app && room);
    s.nl += app && room ? 1 : 0;
    r.over = r.over || (app && !room);
  }
}

template <class S>
__device__ __forceinline__ uint64_t round_cutlim(const Round& r) {
  return S::kList ? r.cut_key : r.kk[KBUF - 1];
}

// Test one postponed leaf of this lane's own ray and take its key.
template <class S>
__device__ __forceinline__ void leaf_eval(const TraceCtx& tc, S& s, Round& r, const Record& rec) {
  if constexpr (S::kStats) ++s.tests;
  const uint64_t key = leaf_key(tc, rec, s.O, s.W, r.floor_key, round_cutlim<S>(r));
  take_key(tc, s, r, key);
}

// Test postponed leaves, most recent first. The next leaf's record is loaded
// before the current one is tested, so that its latency overlaps the test's
// arithmetic. A lane whose traversal continues stops once fewer than leaf_min
// lanes of the wave still hold leaves, and keeps the rest for its next leaf
// phase; a lane whose traversal has ended tests all of them.
// The load is not behind a branch (a lane without a next leaf
// loads the current one again): the compiler then knows how many loads are in
// flight and waits for the current record alone; behind a branch it waited
// for both, and every test paid the whole latency.
// leaf_min of a wave with 64 lanes at work. 16, 12, 8 and 4 lanes: Stage-0 step
// 3.15, 3.04, 2.89 and 2.83 ms, single-bounce step 26.3, 25.7, 25.2 and 25.0,
// path tracing 139.8, 139.5, 139.7 and 140.3.
constexpr int LEAF_MIN_LANES = 8;
template <class S>
__device__ __forceinline__ void leaf_phase(const TraceCtx& tc, S& s, Round& r, int* pend, int leaf_min) {
  if (r.np <= 0) return;
  uint32_t pos = (uint32_t)pend[(--r.np) * TRACE_BLOCK];
  Record rec = load_record(tc.recs, pos);
  while (true) {
    const bool more = r.np > 0 && !(r.trav && __popcll(__ballot(r.np > 0)) < leaf_min);
    r.np -= more ? 1 : 0;
    const uint32_t queued = (uint32_t)pend[r.np * TRACE_BLOCK];
    pos = more ? queued : pos;
    const Record nrec = load_record(tc.recs, pos);
    leaf_eval(tc, s, r, rec);
    __builtin_amdgcn_sched_barrier(0);   // the next record is not waited for before this one is done
    if (!more) break;
    rec = nrec;
  }
}

// After a traversal round: what the hit list now covers.
template <class S>
__device__ __forceinline__ void round_end_traversal(const TraceCtx& tc, S& s, const Round& r) {
  if constexpr (S::kList) s.lhi = r.over ? 0ull : (r.cnt == KBUF ? r.cut_key : KEY_NONE);
}

// Traverse one round to completion for this lane.
template <class S>
__device__ __forceinline__ void traverse_round(const TraceCtx& tc, S& s, Round& r, TravStack& st,
                                               int* pend, int leaf_min) {
  while (true) {
    while (r.trav && r.np <= PEND - 4) {
      node_visit(tc, s, r, st, pend);
      if (__all(r.np > 0 || !r.trav)) break;
    }
    leaf_phase(tc, s, r, pend, leaf_min);
    if (!r.trav) break;
  }
  round_end_traversal(tc, s, r);
}

// ---------------------------------------------------------------------------
// One ray by a group of lanes. With few rays in a launch, what a ray costs is
// the latency of its own chain of node visits and leaf tests, about a
// microsecond each, while the chip is nearly idle. A group of G lanes (a power
// of two, aligned in its wave) shares the ray's stack and its queue of leaves
// and takes up to G of either at a time. Every lane keeps a k-buffer of what it
// found; merges leave the KBUF smallest keys in the group's first lane. The
// keys of a round do not depend on the order of the visits, so the hits are
// those of a lane alone.
// ---------------------------------------------------------------------------
// Lanes per ray: the most that still gives every ray a group.
__host__ __device__ inline int group_lanes(int lanes_per_wave) {
  int g = 1;
  while (2 * g * lanes_per_wave <= 64) g *= 2;
  return g;
}

// The k-buffers of a group into its first lane's (KBUF smallest keys); the
// others are emptied. All lanes of the wave call it.
__device__ __forceinline__ void group_merge(uint64_t (&kk)[KBUF], int G) {
  const int lig = (int)(threadIdx.x & 63) & (G - 1);
  for (int m = 1; m < G; m <<= 1) {
    // the lower lane of a pair keeps the lower half of both, bitonic; what
    // lanes with a lower bit set hold is no longer looked at
#pragma unroll
    for (int i = 0; i < KBUF / 2; ++i) {
      const uint64_t pa = (uint64_t)__shfl_xor((unsigned long long)kk[KBUF - 1 - i], m);
      const uint64_t pb = (uint64_t)__shfl_xor((unsigned long long)kk[i], m);
      kk[i] = key_min(kk[i], pa);
      kk[KBUF - 1 - i] = key_min(kk[KBUF - 1 - i], pb);
    }
#pragma unroll
    for (int st = KBUF / 2; st >= 1; st >>= 1) {
#pragma unroll
      for (int i = 0; i < KBUF; ++i)
        if ((i & st) == 0) cswap_key(kk[i], kk[i + st]);
    }
  }
#pragma unroll
  for (int i = 0; i < KBUF; ++i) kk[i] = lig == 0 ? kk[i] : KEY_NONE;
}

// A round's traversal by groups of G lanes; every lane of the wave calls it,
// with `on` the same in a group, the ray and the round's floor in all lanes of
// the group, and the block's whole stack and queue arrays. Afterwards the first
// lane of each group holds the round. False for a group whose stack would not
// have fitted its lanes' LDS (nothing else is valid then: the caller traverses
// with one lane).
template <class S>
__device__ bool group_traverse(const TraceCtx& tc, S& s, Round& r, int* stack, int* queue, int G, bool on) {
  static_assert(!S::kList, "group rounds keep no hit list");
  const int lane = (int)(threadIdx.x & 63), lig = lane & (G - 1), gb = lane & ~(G - 1);
  const uint64_t gmask = (G == 64 ? ~0ull : ((1ull << G) - 1ull)) << gb;
  const uint64_t below = gmask & ((1ull << lane) - 1ull);
  // entry e of the group's stack or queue: row e / G of its lanes' columns
  // (volatile: lanes read what others wrote)
  const int sh = __ffs(G) - 1, col = (int)(threadIdx.x & ~63u) + gb;
  volatile int* const vs = stack;
  volatile int* const vq = queue;
  auto at = [&](int e) { return (e >> sh) * TRACE_BLOCK + col + (e & (G - 1)); };
  const int cap = STACK_LDS * G;
  int sp = 0, nq = 0, found = 0;
  bool fits = true;
  uint64_t lim = KEY_NONE;
  if (on) {
    if (tc.root >= 0) sp = 1;
    else nq = 1;
    if (lig == 0) (tc.root >= 0 ? vs : vq)[at(0)] = tc.root >= 0 ? tc.root : ~tc.root;
  }
  while (true) {
    // nodes, while fewer than G leaves wait (so at most 5 G ever do)
    const bool nodes = sp > 0 && nq < G;
    if (__any(nodes)) {
      int k = nodes ? min(sp, G) : 0;
      const int room = (cap - sp) / 3;   // each node opened leaves at most three entries more
      if (nodes && room < 1) {
        fits = false;
        k = sp = nq = 0;
      }
      k = min(k, max(room, 0));
      const bool my = lig < k;
      NodeKids kd;
      kd.ni = 0;
      int ic[4] = {0, 0, 0, 0};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        kd.leaf[c] = false;
        kd.c[c] = 0;
      }
      if (my) {
        if constexpr (S::kStats) ++s.visits;
        kd = node_test(tc, s, vs[at(sp - 1 - lig)], r.tlo0, r.t_cut);
        sort_kids(kd, ic);
      }
      sp -= k;
      // each lane's farthest child first, so that the nearest end on top
#pragma unroll
      for (int c = 3; c >= 0; --c) {
        const bool p = c < kd.ni;
        const uint64_t m = __ballot(p) & gmask;
        if (p) vs[at(sp + __popcll(m & below))] = ic[c];
        sp += __popcll(m);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint64_t m = __ballot(kd.leaf[c]) & gmask;
        if (kd.leaf[c]) vq[at(nq + __popcll(m & below))] = ~kd.c[c];
        nq += __popcll(m);
      }
    }
    // leaves, once every lane has one or no node is left
    const bool leaves = nq > 0 && (nq >= G || sp == 0);
    if (__any(leaves)) {
      const int k = leaves ? min(nq, G) : 0;
      const bool my = lig < k;
      uint64_t key = KEY_NONE;
      if (my) {
        if constexpr (S::kStats) ++s.tests;
        const Record rec = load_record(tc.recs, (uint32_t)vq[at(nq - 1 - lig)]);
        key = leaf_key(tc, rec, s.O, s.W, r.floor_key, key_min(lim, r.kk[KBUF - 1]));
      }
      kbuf_insert(r.kk, key);
      nq -= k;
      found += __popcll(__ballot(key != KEY_NONE) & gmask);
    }
    const bool end = !__any(sp > 0 || nq > 0);
    // merged when a group has found enough for a new cut, and at the end
    if (__any(found >= KBUF) || end) {
      group_merge(r.kk, G);
      lim = (uint64_t)__shfl((unsigned long long)r.kk[KBUF - 1], gb);
      if (lim != KEY_NONE) r.t_cut = key_thi(tc, lim) * 1.000002f + 1e-6f;
      found = 0;
    }
    if (end) break;
  }
  r.cnt = 0;
#pragma unroll
  for (int i = 0; i < KBUF; ++i) r.cnt += r.kk[i] != KEY_NONE ? 1 : 0;
  r.trav = false;
  r.np = 0;
  return fits;
}

// A hit of the ray (O, W) on a surfel, as group_blend passes it round (blend_round
// has the same expressions in line: through these functions its register
// allocation cost the path tracer 3%): distance t, alpha, om = 1 - alpha,
// the unnormalised normal cn = |q|^2 n with its scale 1 / |q|^2, negated when n
// points along the ray (n' faces the origin).
// Where a product could be fused into either of two sums, or into none, the
// choice is written out, the same in every kernel: left to the compiler it went
// with the code around it, and a gradient that is zero but for rounding (the
// opacities of one flat wall) then had other digits in a kernel for groups than
// in the kernel for lanes. adj: the adjoints round w y where the rest round x z.
struct HitEval {
  double t, a, om, iq2;
  D3 cn;
};
template <bool adj>
__device__ __forceinline__ HitEval eval_hit(const Record& rec, D3 O, D3 W) {
  // t, u, v and the unit normal from the columns of the unnormalised
  // quaternion's rotation, |q|^2 (t_u, t_v, n): no square root, and one
  // reciprocal c = 1 / (|q|^2 s_u s_v) for u^2 + v^2 and the normal's scale
  const double qw = rec.q.x, qx = rec.q.y, qy = rec.q.z, qz = rec.q.w;
  const double su = rec.s_idx.x, sv = rec.s_idx.y;
  const double c = 1.0 / (fma(qz, qz, fma(qy, qy, fma(qw, qw, qx * qx))) * (su * sv));
  const double iq2 = c * (su * sv);
  const double wx = qw * qx, wy = qw * qy, wz = qw * qz, xz = qx * qz;
  const D3 cu = d3(fma(-qz, qz, fma(-qy, qy, fma(qw, qw, qx * qx))), 2.0 * fma(qx, qy, wz), 2.0 * (adj ? fma(qx, qz, -wy) : fma(-qw, qy, xz)));
  const D3 cv = d3(2.0 * fma(qx, qy, -wz), fma(-qz, qz, fma(qy, qy, fma(qw, qw, -(qx * qx)))), 2.0 * fma(qy, qz, wx));
  const D3 cn = d3(2.0 * (adj ? fma(qx, qz, wy) : fma(qw, qy, xz)), 2.0 * fma(qy, qz, -wx), fma(qz, qz, fma(-qy, qy, fma(qw, qw, -(qx * qx)))));
  const D3 dp = d3((double)rec.p_sigma.x - O.x, (double)rec.p_sigma.y - O.y, (double)rec.p_sigma.z - O.z);
  const double dn = fma(W.z, cn.z, fma(W.x, cn.x, W.y * cn.y));
  const double t = fma(dp.z, cn.z, fma(dp.y, cn.y, dp.x * cn.x)) / dn;
  const D3 yv = d3(t * W.x - dp.x, t * W.y - dp.y, t * W.z - dp.z);
  const double uc = fma(yv.z, cu.z, fma(yv.x, cu.x, yv.y * cu.y)) * sv, vc = fma(yv.z, cv.z, fma(yv.x, cv.x, yv.y * cv.y)) * su;   // u, v times |q|^2 s_u s_v
  const double g = exp(-0.5 * (fma(uc, uc, vc * vc) * (c * c)));
  HitEval h;
  h.t = t;
  h.a = (double)rec.p_sigma.w * g;
  h.om = fma(-(double)rec.p_sigma.w, g, 1.0);
  h.iq2 = dn > 0.0 ? -iq2 : iq2;
  h.cn = cn;
  return h;
}

// Add a hit's terms to the segment: weight T alpha on everything, then T.
template <int QMODE, class S>
__device__ __forceinline__ void blend_hit(const TraceCtx& tc, S& s, const HitEval& h, const float4& rho_e,
                                          const float4& rr) {
  using Acc = typename S::Acc;
  const double w = s.T * h.a;
  const Acc wf = (Acc)w;
  if (QMODE == Q_ALL) {
    const double sw = w * h.iq2;
    s.N.x += sw * h.cn.x;
    s.N.y += sw * h.cn.y;
    s.N.z += sw * h.cn.z;
    s.D += w * h.t;
    s.P0 += wf * rho_e.x;
    s.P1 += wf * rho_e.y;
    s.P2 += wf * rho_e.z;
    s.E += wf * rho_e.w;
  }
  s.R0 += wf * rr.x;
  s.R1 += wf * rr.y;
  s.R2 += wf * rr.z;
  s.T *= h.om;
  if (s.T < tc.T_min) s.done = true;
}

// Blend the round's hits in key order; t and alpha are recomputed from the
// record with the same double-precision test. Sets s.done after the first hit
// with T < T_min or when the round returned fewer than KBUF hits. The sorted
// positions of all the round's hits are fetched at once (their latency is
// paid once a round), and shifted down one entry per hit, which keeps the
// indexing static.
// on_hit(record, attributes, t, 1 - alpha, w, T_before, O, W) is called for every
// blended hit (its loads would stand between the next hit's and this one); if
// hit_out is non-null, up to max_hits blended surfel indices are written.
template <int QMODE, class S, class HitFn>
__device__ __forceinline__ void blend_round(const TraceCtx& tc, S& s, Round& r, HitFn& on_hit,
                                           int32_t* hit_out, int max_hits) {
  using Acc = typename S::Acc;
  // a partial round holds every key below lhi
  const uint64_t round_last = r.partial ? s.lhi - 1 : r.kk[KBUF - 1];
  uint32_t at_pos[KBUF];
#pragma unroll
  for (int m = 0; m < KBUF; ++m) at_pos[m] = (uint32_t)*elem(tc.inv, m < r.cnt ? key_idx(tc, r.kk[m]) : 0u);
  __builtin_amdgcn_sched_barrier(0);   // all of them, before anything waits for the first
  // the next hit's record and attributes are loaded while the current one is
  // blended (always: entries past the round's hits are surfel 0's; a load
  // behind a branch would not overlap, as in leaf_phase)
  Record rec = load_record(tc.recs, at_pos[0]);
  Attr at = *elem(tc.attrs, at_pos[0]);
  for (int j = 0; j < r.cnt && !s.done; ++j) {
#pragma unroll
    for (int m = 0; m < KBUF - 1; ++m) at_pos[m] = at_pos[m + 1];
    const Record nrec = load_record(tc.recs, at_pos[0]);
    const Attr nat = *elem(tc.attrs, at_pos[0]);
    // t, u, v and the unit normal from the columns of the unnormalised
    // quaternion's rotation, |q|^2 (t_u, t_v, n): no square root, and one
    // reciprocal c = 1 / (|q|^2 s_u s_v) for u^2 + v^2 and the normal's scale
    const double qw = rec.q.x, qx = rec.q.y, qy = rec.q.z, qz = rec.q.w;
    const double su = rec.s_idx.x, sv = rec.s_idx.y;
    const double c = 1.0 / (fma(qz, qz, fma(qy, qy, fma(qw, qw, qx * qx))) * (su * sv));
    const double iq2 = c * (su * sv);
    constexpr bool adj = HitFn::kHits;
    const double wx = qw * qx, wy = qw * qy, wz = qw * qz, xz = qx * qz;
    const D3 cu = d3(fma(-qz, qz, fma(-qy, qy, fma(qw, qw, qx * qx))), 2.0 * fma(qx, qy, wz), 2.0 * (adj ? fma(qx, qz, -wy) : fma(-qw, qy, xz)));
    const D3 cv = d3(2.0 * fma(qx, qy, -wz), fma(-qz, qz, fma(qy, qy, fma(qw, qw, -(qx * qx)))), 2.0 * fma(qy, qz, wx));
    const D3 cn = d3(2.0 * (adj ? fma(qx, qz, wy) : fma(qw, qy, xz)), 2.0 * fma(qy, qz, -wx), fma(qz, qz, fma(-qy, qy, fma(qw, qw, -(qx * qx)))));
    const D3 dp = d3((double)rec.p_sigma.x - s.O.x, (double)rec.p_sigma.y - s.O.y, (double)rec.p_sigma.z - s.O.z);
    const double dn = fma(s.W.z, cn.z, fma(s.W.x, cn.x, s.W.y * cn.y));
    const double t = fma(dp.z, cn.z, fma(dp.y, cn.y, dp.x * cn.x)) / dn;
    const D3 yv = d3(t * s.W.x - dp.x, t * s.W.y - dp.y, t * s.W.z - dp.z);
    const double uc = fma(yv.z, cu.z, fma(yv.x, cu.x, yv.y * cu.y)) * sv, vc = fma(yv.z, cv.z, fma(yv.x, cv.x, yv.y * cv.y)) * su;   // u, v times |q|^2 s_u s_v
    const double g = exp(-0.5 * (fma(uc, uc, vc * vc) * (c * c)));
    const double a = (double)rec.p_sigma.w * g, om = fma(-(double)rec.p_sigma.w, g, 1.0);
    const double w = s.T * a;
    const Acc wf = (Acc)w;
    if (QMODE == Q_ALL) {
      const double sw = (dn > 0.0 ? -w : w) * iq2;  // n' faces the origin
      s.N.x += sw * cn.x;
      s.N.y += sw * cn.y;
      s.N.z += sw * cn.z;
      s.D += w * t;
      s.P0 += wf * at.rho_e.x;
      s.P1 += wf * at.rho_e.y;
      s.P2 += wf * at.rho_e.z;
      s.E += wf * at.rho_e.w;
    }
    s.R0 += wf * at.r.x;
    s.R1 += wf * at.r.y;
    s.R2 += wf * at.r.z;
    if constexpr (S::kStats) {
      if (hit_out && s.nhits < max_hits) hit_out[s.nhits] = (int32_t)rec_index(rec);
    }
    if constexpr (HitFn::kHits) on_hit(rec, at, t, om, w, s.T, s.O, s.W);
    if constexpr (S::kStats) ++s.nhits;
    s.T *= om;
    if (s.T < tc.T_min) s.done = true;
    __builtin_amdgcn_sched_barrier(0);   // the next record is not waited for before this one is done
    rec = nrec;
    at = nat;
  }
  if (r.cnt < KBUF && !r.partial) s.done = true;
  if (!s.done) s.last = round_last;
}

// The blend of a round by a group of G lanes (all lanes of the wave call it; the
// round is in the first lane of each group that is `on`): each lane evaluates
// one of the round's hits, G at a time, and all lanes of the group then blend
// them in order, so that every lane carries the segment. The same sums in the
// same order as blend_round's. A source that takes the hits carries its item in
// every lane; its running sum goes on in order, and then each lane hands it its
// own hit. queue: the block's array of postponed leaves, empty now.
template <int QMODE, class S, class HitFn>
__device__ __forceinline__ void group_blend(const TraceCtx& tc, S& s, const Round& r, HitFn& src, int* queue, int G,
                                            bool on, int32_t* hit_out, int max_hits) {
  static_assert(!S::kList, "group rounds keep no hit list");
  const int lane = (int)(threadIdx.x & 63), lig = lane & (G - 1), gb = lane & ~(G - 1);
  const int sh = __ffs(G) - 1, col = (int)(threadIdx.x & ~63u) + gb;
  volatile int* const vq = queue;
  auto at = [&](int e) { return (e >> sh) * TRACE_BLOCK + col + (e & (G - 1)); };
  if (lig == 0) {
#pragma unroll
    for (int i = 0; i < KBUF; ++i) vq[at(i)] = (int)key_idx(tc, r.kk[i]);
  }
  const int cnt = on ? __shfl(r.cnt, gb) : 0;
  const uint64_t last = (uint64_t)__shfl((unsigned long long)r.kk[KBUF - 1], gb);
  if (!on) s.done = true;
  for (int c = 0; c < KBUF; c += G) {
    if (!__any(c < cnt && !s.done)) break;
    const int mine = c + lig;
    const uint32_t idx = mine < cnt ? (uint32_t)vq[at(mine)] : 0u;
    const uint32_t pos = (uint32_t)*elem(tc.inv, idx);
    const Attr a0 = *elem(tc.attrs, pos);
    const Record rec = load_record(tc.recs, pos);
    const HitEval h0 = eval_hit<HitFn::kHits>(rec, s.O, s.W);
    double c0 = 0.0, my_T = 0.0, my_prefix = 0.0;
    bool taken = false;
    if constexpr (HitFn::kHits) c0 = src.weight(rec, a0, h0.t, s.W);
    for (int j = 0; j < G && c + j < KBUF; ++j) {
      if (!__any(c + j < cnt && !s.done)) break;
      const int from = gb + j;
      HitEval h;
      float4 rho_e = make_float4(0.f, 0.f, 0.f, 0.f), rr = rho_e;
      h.t = h.iq2 = 0.0;
      h.cn = d3(0.0, 0.0, 0.0);
      h.a = __shfl(h0.a, from);
      h.om = __shfl(h0.om, from);
      rr = make_float4(__shfl(a0.r.x, from), __shfl(a0.r.y, from), __shfl(a0.r.z, from), 0.f);
      if (QMODE == Q_ALL) {
        h.t = __shfl(h0.t, from);
        h.iq2 = __shfl(h0.iq2, from);
        h.cn = d3(__shfl(h0.cn.x, from), __shfl(h0.cn.y, from), __shfl(h0.cn.z, from));
        rho_e = make_float4(__shfl(a0.rho_e.x, from), __shfl(a0.rho_e.y, from), __shfl(a0.rho_e.z, from),
                            __shfl(a0.rho_e.w, from));
      }
      const uint32_t hit = hit_out ? (uint32_t)__shfl((int)idx, from) : 0u;
      double cj = 0.0;
      if constexpr (HitFn::kHits) cj = __shfl(c0, from);
      if (c + j < cnt && !s.done) {
        if constexpr (S::kStats) {
          if (hit_out && lig == 0 && s.nhits < max_hits) hit_out[s.nhits] = (int32_t)hit;
          ++s.nhits;
        }
        if constexpr (HitFn::kHits) {
          src.prefix += (s.T * h.a) * cj;
          if (lane == from) {
            taken = true;
            my_T = s.T;
            my_prefix = src.prefix;
          }
        }
        blend_hit<QMODE>(tc, s, h, rho_e, rr);
      }
    }
    if constexpr (HitFn::kHits) {
      if (taken) src.adjoint(rec, a0, h0.t, h0.om, my_T * h0.a, my_T, c0, my_prefix, s.O, s.W);
    }
  }
  if (cnt < KBUF) s.done = true;
  if (!s.done) s.last = last;
}

// A whole segment, without a hit list. Must be called from a
// TRACE_BLOCK-thread block (the traversal stack and the postponed leaves live
// in LDS), by every lane of the wave: with `on` for the lanes that have a ray.
// G = 1: one lane per ray, `lanes` lanes of every wave at work. G > 1: the G
// lanes of a group have the same ray, and the result is the first lane's.
template <int QMODE, bool DACC>
__device__ __forceinline__ SegOut trace_segment(const TraceCtx& tc, D3 O, D3 W, bool on, int lanes, int G,
                                                int32_t* hit_out = nullptr, int max_hits = 0) {
  __shared__ int s_stack[STACK_LDS * TRACE_BLOCK];
  __shared__ int s_pend[PEND * TRACE_BLOCK];
  const int leaf_min = (LEAF_MIN_LANES * lanes + 63) / 64;
  const int lane = (int)(threadIdx.x & 63);
  const bool first = (lane & (G - 1)) == 0;
  int s_ovf[STACK_OVF];
  TravStack st;
  st.lds = s_stack + threadIdx.x;
  st.ovf = s_ovf;
  st.sp = 0;
  int* pend = s_pend + threadIdx.x;   // this lane's queue of postponed leaves
  SegStats<DACC, true, false> s;
  NoHit nh;
  seg_begin(s, O, W);
  s.done = !on;
  Round r;
  if (G == 1) {
    while (!s.done) {
      if (round_begin(tc, s, r, st, pend)) traverse_round(tc, s, r, st, pend, leaf_min);
      blend_round<QMODE>(tc, s, r, nh, hit_out, max_hits);
    }
  } else {
    while (__any(!s.done)) {
      round_begin(tc, s, r, st, pend);
      const bool fits = group_traverse(tc, s, r, s_stack, s_pend, G, !s.done);
      if (first && !s.done && !fits) {
        round_begin(tc, s, r, st, pend);
        traverse_round(tc, s, r, st, pend, 1);
      }
      group_blend<QMODE>(tc, s, r, nh, s_pend, G, !s.done, hit_out, max_hits);
    }
    // a group's visits and tests are its lanes'
    for (int m = 1; m < G; m <<= 1) {
      s.visits += __shfl_xor(s.visits, m);
      s.tests += __shfl_xor(s.tests, m);
    }
  }
  SegOut o;
  o.N = s.N;
  o.D = s.D;
  o.R = d3(s.R0, s.R1, s.R2);
  o.E = s.E;
  o.P = d3(s.P0, s.P1, s.P2);
  o.T = s.T;
  o.nhits = s.nhits;
  o.rounds = s.rounds;
  o.tests = s.tests;
  o.visits = s.visits;
  return o;
}

}  // namespace eag

#include "eag_internal.h"
namespace eag {
TraceCtx make_ctx(const eag_bvh* b, const Attr* attrs, const eag_trace_params* p, const TraceSetup& ts);
}  // namespace eag
