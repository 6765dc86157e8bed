// rsi_device.h -- device-side records and predicates shared by the build and
// query kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rsi {

// ---------------------------------------------------------------- records --
//
// Node: one 64-byte record per internal node holding the bounding boxes of
// BOTH children next to their references, so a traversal step fetches the
// two boxes it tests with four 16-byte loads from one line.  This replaces
// the paper's per-node BVHNode with raw child pointers (Section 3.1): boxes
// move up into the parent, pointers become 32-bit indices, and a leaf is
// encoded in the reference itself.
//
//   f[0..5]   left child  lo.x lo.y lo.z hi.x hi.y hi.z
//   f[6..11]  right child lo.x lo.y lo.z hi.x hi.y hi.z
//   ref[0..1] left / right child reference
//   aux[0..1] build scratch: index-range bounds written by the children
//
// Child reference: >= 0 internal node index; < 0 leaf with
//   first sorted triangle = ref & 0x07FFFFFF, count = ((ref >> 27) & 15) + 1.
struct alignas(64) Node {
    float f[12];
    int32_t ref[2];
    int32_t aux[2];
};
static_assert(sizeof(Node) == 64, "Node must be 64 bytes");

// Node4 (64 bytes, four 16-byte loads like a binary step): the four-way
// view of binary node n, whose children are descendants of n (its two
// children, the internal one with the larger box surface replaced by its own
// two, twice), with the child boxes quantised to 8 bits per
// plane on a grid anchored at the lower corner of n's box.  Record n of the
// Node4 array belongs to binary node n, so a child reference (an internal
// node's index, or a leaf) is valid in both arrays.
//
//   ox, oy, oz   lower corner of n's box (exact)
//   sx, sy, sz   grid steps, powers of two (2^-126 .. 2^122) with 255
//                steps spanning n's box on that axis
//   lo[a]        byte c: child c's lower plane on axis a in grid steps,
//                rounded down;  hi[a] likewise for the upper plane, rounded
//                up, each at least 2^-11 steps outside the child's
//                box except a lower plane at 0, the exact corner
//   ref[c]       child reference; an unused slot (planes 255 and 0, so its
//                box is empty) names the leaf at position n_t, a record of
//                zeros that no segment crosses
//
// With exact boxes the four-way record would need 128 bytes; 64 bytes halve
// the vector-cache lookups per visited box, which bound the binary walk.  Any finite
// box is representable.
constexpr int32_t kDone = 0x7FFFFFFF;  // the four-way walk's end-of-stack mark; no reference has this value
struct alignas(64) Node4 {
    float ox, oy, oz, sz;
    uint32_t lo[3];
    uint32_t hi[3];
    float sx, sy;
    int32_t ref[4];
};
static_assert(sizeof(Node4) == 64, "Node4 must be 64 bytes");

// Tri: the three FP32 vertices of a triangle in Morton (sorted) order plus
// its original id, 48 bytes = three 16-byte loads.  Storing the vertices
// themselves (rather than edges) keeps the FP64 re-solve of reported hits
// exact with respect to the FP32 inputs.
struct alignas(16) Tri {
    float4 a;  // v0.x v0.y v0.z v1.x
    float4 b;  // v1.y v1.z v2.x v2.y
    float4 c;  // v2.z, id (int bits), 0, 1 when a vertex index was out of range (else 0)
};
static_assert(sizeof(Tri) == 48, "Tri must be 48 bytes");

constexpr int kLeafFirstBits = 27;
constexpr int32_t kLeafFirstMask = (1 << kLeafFirstBits) - 1;
constexpr int kMaxLeafSize = 16;

__host__ __device__ inline int32_t leaf_ref(int32_t first, int32_t count)
{
    return (int32_t)(0x80000000u | ((uint32_t)(count - 1) << kLeafFirstBits) | (uint32_t)first);
}
__host__ __device__ inline bool ref_is_leaf(int32_t r) { return r < 0; }
__host__ __device__ inline int32_t leaf_first(int32_t r) { return r & kLeafFirstMask; }
__host__ __device__ inline int32_t leaf_count(int32_t r) { return ((r >> kLeafFirstBits) & 15) + 1; }

// Rows of two and three floats, aligned like a float, read or written by one
// access.  (Three one-float accesses per row, 12 bytes apart across the
// lanes, visit every cache line three times.)
typedef float row2 __attribute__((ext_vector_type(2), aligned(4), may_alias));
typedef float row3 __attribute__((ext_vector_type(3), aligned(4), may_alias));
__device__ inline row3 ld3(const float *p) { return *reinterpret_cast<const row3 *>(p); }
__device__ inline row3 ld3_nt(const float *p) { return __builtin_nontemporal_load(reinterpret_cast<const row3 *>(p)); }
__device__ inline void st3(float *p, float x, float y, float z)
{
    const row3 v = {x, y, z};
    *reinterpret_cast<row3 *>(p) = v;
}
__device__ inline void st3_nt(float *p, float x, float y, float z)
{
    const row3 v = {x, y, z};
    __builtin_nontemporal_store(v, reinterpret_cast<row3 *>(p));
}
__device__ inline void st2_nt(float *p, float x, float y)
{
    const row2 v = {x, y};
    __builtin_nontemporal_store(v, reinterpret_cast<row2 *>(p));
}

// ---------------------------------------------------------------- segment --
//
// Per-lane segment state: origin o = S, direction d = E - S (t in [0, 1]
// spans the segment) and the guarded reciprocal of d for the slab test.
struct Seg {
    float ox, oy, oz;
    float dx, dy, dz;
    float ix, iy, iz;
};

__device__ inline float guarded_rcp(float d)
{
    // Components below the smallest normal FP32 value 2^-126 in magnitude
    // (zero included) use +-2^-126, so the reciprocal is finite (at most
    // 2^126) and every slab parameter is finite or +-inf, never NaN.  The
    // capped reciprocal keeps the box decision exact while every nonzero
    // coordinate difference is a normal number: then |(plane - o) * 2^126|
    // >= 1 lies outside [0, 1] on the same side as the exact parameter.
    // Only differences in the subnormal range (coordinates below about
    // 2^-102) fall short of that.  (plane == o with d == 0 is a segment
    // lying in a box face, which meets the triangles inside only on their
    // boundary.)  The hardware reciprocal is within 1 ulp, which the slack
    // of slab_hit covers.
    const float tiny = 0x1p-126f;
    const float g = fabsf(d) < tiny ? copysignf(tiny, d) : d;
    return __builtin_amdgcn_rcpf(g);
}

__device__ inline Seg make_seg(float sx, float sy, float sz, float ex, float ey, float ez)
{
    Seg r;
    r.ox = sx; r.oy = sy; r.oz = sz;
    r.dx = ex - sx; r.dy = ey - sy; r.dz = ez - sz;
    r.ix = guarded_rcp(r.dx);
    r.iy = guarded_rcp(r.dy);
    r.iz = guarded_rcp(r.dz);
    return r;
}

// Conservative segment / box test (slab method).  Each slab parameter is
// (plane - o) * (1/d): a subtraction, a reciprocal within 1 ulp and a
// product, so its relative error is at most about 4 ulp (2^-22) with no
// absolute term; accepting when near <= far * (1 + 2^-20) therefore never
// rejects a box that the exact segment touches within [0, tmax].  Returns
// the entry parameter in `tnear`.
__device__ inline bool slab_hit(const Seg &s, float lx, float ly, float lz,
                                float hx, float hy, float hz, float tmax, float &tnear)
{
    float t0x = (lx - s.ox) * s.ix, t1x = (hx - s.ox) * s.ix;
    float t0y = (ly - s.oy) * s.iy, t1y = (hy - s.oy) * s.iy;
    float t0z = (lz - s.oz) * s.iz, t1z = (hz - s.oz) * s.iz;
    float n = fmaxf(fmaxf(fminf(t0x, t1x), fminf(t0y, t1y)), fmaxf(fminf(t0z, t1z), 0.0f));
    float f = fminf(fminf(fmaxf(t0x, t1x), fmaxf(t0y, t1y)), fminf(fmaxf(t0z, t1z), tmax));
    tnear = n;
    return n <= f * (1.0f + 0x1p-20f);
}

// Conservative segment / quantised-box test of the four-way walk.  With o
// the segment's start, id the guarded reciprocal of its direction (box_rcp)
// and D = corner - o, the caller forms per node and axis
//   a  = step id,   b = fma(D, id, kStartShift),   bn = b - |b| kPlaneRel,
//   bf = b + |b| kPlaneRel,
// and grid plane q lies at parameter fma(q, a, bn) when it is the plane the
// segment meets first on that axis (the lower plane for a non-negative
// direction component) and at fma(q, a, bf) when it is the other one; qn and
// qf are those planes' quantised values as floats.  Parameters are shifted
// by kStartShift: the segment spans [2^-21, 1 + 2^-21].  Both sides are
// clamped to [0, 1] (a modifier of the max3 / min3, so the limits cost no
// instruction) and the test is near < far.
//
// Why it never rejects a touched box.  id is within 1 ulp, step is a power
// of two: the roundings of D, id, b, bn / bf and the fma add up to at most
// 2^-21.4 |b| + 2^-22.4 q |a|.  The margin is 2^-19 |b|, and for every plane
// with q > 0 also 2^-11 |a| (Wide::store places planes at least 2^-11 steps
// outside the child's box; a lower plane at q = 0 is the exact corner, and
// its parameter has no term in q).  So each parameter is strictly on the
// safe side of the exact one, by enough that (i) a box met at t <= 1 has
// near < 1: there q |a| + |b| >= 1, hence a margin of at least 2^-19 (2^-19 |b|
// + 2^-11 |a|, q <= 255) minus the shift 2^-21 and the roundings; (ii) a box
// left at t >= 0 has far >= 2^-21 minus roundings relative to it, so far > 0,
// also when the start lies exactly on its face (b = 2^-21 then); (iii) in
// between, near <= exact near <= exact far <= far with a strict step on each
// side.  Boxes past either end clamp to near = far and are rejected.
// box_rcp keeps every product finite, so no NaN arises from finite input.
constexpr float kPlaneRel = 0x1p-19f;
constexpr float kStartShift = 0x1p-21f;
constexpr double kQuantMargin = 0x1p-11 + 0x1p-40;  // grid steps between a child's box and its planes, before FP64 rounding

__device__ inline bool qslab_hit(float ax, float ay, float az, float bnx, float bny, float bnz, float bfx,
                                 float bfy, float bfz, float qnx, float qny, float qnz, float qfx, float qfy,
                                 float qfz, float &tnear)
{
    const float nx = fmaf(qnx, ax, bnx), fx = fmaf(qfx, ax, bfx);
    const float ny = fmaf(qny, ay, bny), fy = fmaf(qfy, ay, bfy);
    const float nz = fmaf(qnz, az, bnz), fz = fmaf(qfz, az, bfz);
    const float n = __builtin_amdgcn_fmed3f(fmaxf(fmaxf(nx, ny), nz), 0.0f, 1.0f);
    const float f = __builtin_amdgcn_fmed3f(fminf(fminf(fx, fy), fz), 0.0f, 1.0f);
    tnear = n;
    return n < f;
}

// Smallest |direction component| the four-way walk inverts as it is: with
// `scale` the largest |coordinate| of the mesh's box, every plane offset from
// the segment's start is at most R = scale + |o|, and a component below
// R 2^-125 is replaced by that value (with its sign), so offset times
// reciprocal stays below 2^126.  The replacement keeps the box decision
// exact while every nonzero plane offset is at least R 2^-125: its
// parameter then lies outside [0, 1] on the same side as the exact one.
__device__ inline float box_tiny(const Seg &s, float scale)
{
    const float R = scale + fmaxf(fmaxf(fabsf(s.ox), fabsf(s.oy)), fabsf(s.oz));
    return fmaf(R, 0x1p-125f, 0x1p-126f);
}

// Reciprocal direction for the four-way walk, with the segment cut at tlim
// (parameters are then fractions of the cut segment, so the box test's
// limits stay 0 and 1).
__device__ inline void box_rcp(Seg &s, float tlim, float tiny)
{
    const float c = fmaxf(tlim, 0x1p-40f);
    s.ix = __builtin_amdgcn_rcpf(copysignf(fmaxf(fabsf(s.dx) * c, tiny), s.dx));
    s.iy = __builtin_amdgcn_rcpf(copysignf(fmaxf(fabsf(s.dy) * c, tiny), s.dy));
    s.iz = __builtin_amdgcn_rcpf(copysignf(fmaxf(fabsf(s.dz) * c, tiny), s.dz));
}

// Moller-Trumbore segment / triangle test in FP32, division-free decision
// (paper Section 2 names the test: one division, four dot and two cross
// products at worst).  With e1 = v1 - v0, e2 = v2 - v0, p = d x e2,
// det = e1 . p, s = o - v0, q = s x e1:  u = s.p / det, v = d.q / det,
// t = e2.q / det.  The decision compares the numerators against |det| after
// moving det's sign onto them, so only an accepted hit pays the division.
// Closed triangle and closed segment: u >= 0, v >= 0, u + v <= 1,
// 0 <= t <= tmax; det == 0 (parallel or degenerate triangle) never hits.
struct MTHit {
    bool hit;
    float tn;   // t numerator (sign-normalised)
    float det;  // |det|
};

__device__ inline MTHit mt_test(const Seg &s, float v0x, float v0y, float v0z,
                                float v1x, float v1y, float v1z,
                                float v2x, float v2y, float v2z, float tmax)
{
    // Every fused multiply-add is written out (the library is compiled with
    // contraction off), so the decision is bit-identical in every mode.
    float e1x = v1x - v0x, e1y = v1y - v0y, e1z = v1z - v0z;
    float e2x = v2x - v0x, e2y = v2y - v0y, e2z = v2z - v0z;
    float px = fmaf(s.dy, e2z, -(s.dz * e2y));
    float py = fmaf(s.dz, e2x, -(s.dx * e2z));
    float pz = fmaf(s.dx, e2y, -(s.dy * e2x));
    float det = fmaf(e1x, px, fmaf(e1y, py, e1z * pz));
    float sx = s.ox - v0x, sy = s.oy - v0y, sz = s.oz - v0z;
    float un = fmaf(sx, px, fmaf(sy, py, sz * pz));
    float qx = fmaf(sy, e1z, -(sz * e1y));
    float qy = fmaf(sz, e1x, -(sx * e1z));
    float qz = fmaf(sx, e1y, -(sy * e1x));
    float vn = fmaf(s.dx, qx, fmaf(s.dy, qy, s.dz * qz));
    float tn = fmaf(e2x, qx, fmaf(e2y, qy, e2z * qz));
    float ad = fabsf(det);
    if (det < 0.0f) { un = -un; vn = -vn; tn = -tn; }
    MTHit h;
    h.hit = (det != 0.0f) & (un >= 0.0f) & (vn >= 0.0f) & (un + vn <= ad) & (tn >= 0.0f) &
            (tn <= ad * tmax);
    h.tn = tn;
    h.det = ad;
    return h;
}

__device__ inline void tri_load(const Tri *__restrict__ tris, int32_t k, float v[9], int32_t &id)
{
    float4 a = tris[k].a, b = tris[k].b, c = tris[k].c;
    v[0] = a.x; v[1] = a.y; v[2] = a.z;
    v[3] = a.w; v[4] = b.x; v[5] = b.y;
    v[6] = b.z; v[7] = b.w; v[8] = c.x;
    id = __float_as_int(c.y);
}

// FP64 re-solve of a reported crossing (same Moller-Trumbore algebra in
// double precision on the FP32 inputs promoted exactly).  The FP32 test
// decides WHETHER a crossing exists; this only sharpens t, u, v.
__device__ inline void mt_refine64(double sx, double sy, double sz, double ex, double ey, double ez,
                                   const float v[9], double &t, double &u, double &w)
{
    double dx = ex - sx, dy = ey - sy, dz = ez - sz;
    double v0x = v[0], v0y = v[1], v0z = v[2];
    double e1x = (double)v[3] - v0x, e1y = (double)v[4] - v0y, e1z = (double)v[5] - v0z;
    double e2x = (double)v[6] - v0x, e2y = (double)v[7] - v0y, e2z = (double)v[8] - v0z;
    double px = dy * e2z - dz * e2y;
    double py = dz * e2x - dx * e2z;
    double pz = dx * e2y - dy * e2x;
    double det = e1x * px + e1y * py + e1z * pz;
    double ox = sx - v0x, oy = sy - v0y, oz = sz - v0z;
    double qx = oy * e1z - oz * e1y;
    double qy = oz * e1x - ox * e1z;
    double qz = ox * e1y - oy * e1x;
    double inv = 1.0 / det;
    u = (ox * px + oy * py + oz * pz) * inv;
    w = (dx * qx + dy * qy + dz * qz) * inv;
    t = (e2x * qx + e2y * qy + e2z * qz) * inv;
}

// Index of the segment of a partition that holds item j: the largest m with
// off[m] <= j, for a table of M + 1 nondecreasing offsets (meshes of a batch
// over triangles, nodes or segments).
__device__ inline int32_t mesh_of(const int64_t *__restrict__ off, int32_t M, int64_t j)
{
    int32_t lo = 0, hi = M - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= j) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Order-preserving int encoding of floats for atomic min / max.
__device__ inline int32_t float_to_ordered(float f)
{
    int32_t i = __float_as_int(f);
    return i >= 0 ? i : i ^ 0x7FFFFFFF;
}
__host__ __device__ inline float ordered_to_float(int32_t i)
{
    int32_t b = i >= 0 ? i : i ^ 0x7FFFFFFF;
    union { int32_t i; float f; } u;
    u.i = b;
    return u.f;
}

}  // namespace rsi
