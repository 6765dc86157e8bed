// build.hip -- linear BVH construction on the GPU (paper Section 2 and
// Section 3.1; the steps are those timed in the paper's Table 2), for one
// mesh or for a batch of meshes in the same launches.
//
// All meshes of a handle share concatenated arrays: mesh m owns triangles,
// sorted leaves and node records [off[m], off[m+1]).  A single mesh is the
// case M = 1.
//
//   k_gather     (batches) copy every mesh's vertices and triangles into the
//                concatenated arrays, offsetting the vertex indices
//   k_init       reset per-mesh bounds, heights, roots and record flags
//   k_centroids  c_j = (v_a + v_b + v_c) / 3 per triangle, index validation,
//                and the support interval of each mesh's centroids (block
//                min/max in LDS, then one ordered-int atomic per block, mesh
//                and axis)
//   k_morton     quantise c_j to 2^21 levels per axis inside its mesh's
//                interval and interleave the three 21-bit integers into a
//                63-bit key
//   (sort.hip)   stable radix sort of (key, triangle id); with M > 1 a final
//                stable pass on the mesh id groups each mesh's leaves again
//   k_lbvh_*     agglomerative single-pass construction over the sorted
//                keys (Apetrei's scheme, as the paper follows): every leaf
//                climbs; at each step the node joins the neighbour across the
//                split whose key distance is smaller, writes its box and
//                reference into its parent, and the parent's arrival flag
//                lets only the second child continue -- so the parent's box
//                is formed exactly once, from both children.  Ranges with at
//                most `leaf_size` triangles become leaves.  Subtrees inside
//                a block of 512 sorted leaves (or a small mesh) finish in LDS
//                (k_lbvh_local), and the few that cross block boundaries are
//                joined in LDS too, by a workgroup per 64 blocks and one for
//                the rest (k_lbvh_join).
//
// The entry node of mesh m is its last record off[m+1] - 1 (unused by its
// n - 1 internal nodes): its left child is the root and its right child an
// empty far box, which mirrors the paper's convention of keeping the root as
// the left child of internalNodes[N_t - 1] and also covers n = 1.
#include <hip/hip_runtime.h>
#include <float.h>
#include <stdint.h>

#include "rsi_host.h"

namespace rsi {
namespace {

struct BuildArgs {
    int32_t M;
    const int64_t *off;    // [M+1] triangle offsets
    const float *V;        // vertices, global indexing
    int64_t n_v;
    const int32_t *T;      // triangles with global vertex indices
    int64_t n_t;
    float *cent;
    uint64_t *keys;
    uint32_t *order;
    int32_t *rank;
    Node *nodes;
    Node4 *nodes4;         // four-way records, null when the walk does not use them
    Tri *tris;
    uint8_t *laid_out;
    int32_t *joins;        // lists of the local blocks' subtrees (kListWords each)
    int32_t *bounds;       // [6M] ordered-int centroid bounds per mesh
    int32_t *mesh_height;  // [M]
    int32_t *mesh_root;    // [M]
    float *mesh_scale;     // [M]
    int32_t *scalars;
    int32_t leaf_size;
};

__global__ void k_gather(int32_t M, const float *const *__restrict__ Vp, const int32_t *const *__restrict__ Tp,
                         const int64_t *__restrict__ voff, const int64_t *__restrict__ toff, float *__restrict__ V,
                         int32_t *__restrict__ T, int32_t *__restrict__ scalars)
{
    const int64_t nv = voff[M], nt = toff[M];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nv + nt; k += stride) {
        if (k < nv) {
            const int32_t m = mesh_of(voff, M, k);
            const int64_t loc = k - voff[m];
            const row3 v = ld3(Vp[m] + 3 * loc);
            st3(V + 3 * k, v.x, v.y, v.z);
        } else {
            const int64_t j = k - nv;
            const int32_t m = mesh_of(toff, M, j);
            const int64_t loc = j - toff[m];
            const int64_t nvm = voff[m + 1] - voff[m];
            for (int c = 0; c < 3; ++c) {
                int32_t x = Tp[m][3 * loc + c];
                if (x < 0 || x >= nvm) {  // reported; a valid index keeps later reads inside V
                    atomicOr(&scalars[kBadGather], 1);
                    x = 0;
                }
                T[3 * j + c] = (int32_t)(x + voff[m]);
            }
        }
    }
}

__global__ void k_clear_gather_flag(int32_t *scalars) { scalars[kBadGather] = 0; }

__global__ void k_init(BuildArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < a.M) {
        for (int k = 0; k < 3; ++k) {
            a.bounds[6 * i + k] = float_to_ordered(FLT_MAX);
            a.bounds[6 * i + 3 + k] = float_to_ordered(-FLT_MAX);
        }
        a.mesh_height[i] = 0;
        a.mesh_root[i] = 0;
        a.mesh_scale[i] = 0.0f;
    }
    if (i == 0) {  // the record that unused four-way slots name: no segment crosses it
        const float4 z = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        a.tris[a.n_t].a = a.tris[a.n_t].b = a.tris[a.n_t].c = z;
    }
    if (i == 0) a.scalars[kBadIndex] = 0;
    if (i < a.n_t) a.laid_out[i] = 0;
}

constexpr int kCentBlock = 256;

__device__ inline int32_t wave_min(int32_t v)
{
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}

// PER triangles per thread.  The bounds end in atomics on one or a few cache
// lines, which the GPU serialises, so their number sets the time of a large
// mesh: with one triangle per thread, 499,280 triangles took 11,700 of them
// and 51 us.  PER = 8 (from 131,072 triangles on; fewer leave CUs idle at
// eight per thread) and a reduction in the wave before the LDS one.  A block
// reduces its first 4 PER meshes in LDS, one for 64 of its triangles; the
// rest go straight to device memory.  (Four with PER = 8: a batch of 1,500 meshes
// of 180 triangles, eleven to a block, took 289 us to rebuild with one triangle
// per thread, 334 with eight, 228 now.)
template <int PER>
__global__ __launch_bounds__(kCentBlock) void k_centroids(BuildArgs a)
{
    constexpr int kCentMeshes = 4 * PER;
    static_assert(kCentMeshes * 6 <= kCentBlock, "one thread per bound");
    __shared__ int32_t lb[kCentMeshes][6];  // per mesh: minima, then negated maxima (as minima)
    const int tid = threadIdx.x;
    if (tid < kCentMeshes * 6) lb[tid / 6][tid % 6] = 0x7FFFFFFF;
    const int64_t j0 = (int64_t)blockIdx.x * (kCentBlock * PER);
    const int32_t m0 = mesh_of(a.off, a.M, j0 < a.n_t ? j0 : a.n_t - 1);
    __syncthreads();
    // this thread's bounds so far, all of mesh `at` (-1: none yet)
    int32_t at = -1, b[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) b[k] = 0x7FFFFFFF;
    auto flush = [&](int32_t m, const int32_t (&v)[6]) {
        if (m - m0 < kCentMeshes) {
#pragma unroll
            for (int k = 0; k < 6; ++k) atomicMin(&lb[m - m0][k], v[k]);
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                atomicMin(&a.bounds[6 * m + k], v[k]);
                atomicMax(&a.bounds[6 * m + 3 + k], ~v[3 + k]);
            }
        }
    };
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int64_t j = j0 + r * kCentBlock + tid;
        if (j >= a.n_t) break;
        int32_t va = a.T[3 * j], vb = a.T[3 * j + 1], vc = a.T[3 * j + 2];
        const bool ok = va >= 0 && va < a.n_v && vb >= 0 && vb < a.n_v && vc >= 0 && vc < a.n_v;
        if (!ok) {
            atomicOr(&a.scalars[kBadIndex], 1);
            va = vb = vc = 0;
        }
        const row3 pa = ld3(a.V + 3 * (int64_t)va), pb = ld3(a.V + 3 * (int64_t)vb), pc = ld3(a.V + 3 * (int64_t)vc);
        const float cx = (pa.x + pb.x + pc.x) * (1.0f / 3.0f);
        const float cy = (pa.y + pb.y + pc.y) * (1.0f / 3.0f);
        const float cz = (pa.z + pb.z + pc.z) * (1.0f / 3.0f);
        a.cent[j] = cx;
        a.cent[a.n_t + j] = cy;
        a.cent[2 * a.n_t + j] = cz;
        const int32_t m = a.M > 1 ? mesh_of(a.off, a.M, j) : 0;
        const int32_t q[3] = {float_to_ordered(cx), float_to_ordered(cy), float_to_ordered(cz)};
        if (m != at && at >= 0) {
            flush(at, b);
#pragma unroll
            for (int k = 0; k < 6; ++k) b[k] = 0x7FFFFFFF;
        }
        at = m;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            b[k] = min(b[k], q[k]);
            b[3 + k] = min(b[3 + k], ~q[k]);  // ~ reverses the order of ints
        }
    }
    // a wave whose threads all end in one mesh reduces first
    const int32_t m_first = __builtin_amdgcn_readfirstlane(at);
    if (__builtin_amdgcn_ballot_w64(at != m_first && at >= 0) == 0) {
        if (m_first >= 0) {
#pragma unroll
            for (int k = 0; k < 6; ++k) b[k] = wave_min(b[k]);
            if (__lane_id() == 0) flush(m_first, b);
        }
    } else if (at >= 0) {
        flush(at, b);
    }
    __syncthreads();
    if (tid < kCentMeshes * 6) {
        const int32_t m = m0 + tid / 6, k = tid % 6;
        const int32_t v = lb[tid / 6][k];
        if (m < a.M && v != 0x7FFFFFFF) {
            if (k < 3) atomicMin(&a.bounds[6 * m + k], v);
            else atomicMax(&a.bounds[6 * m + k], ~v);
        }
    }
}

// Spread the low 21 bits of x so that bit k moves to bit 3k.
__device__ inline uint64_t spread3(uint32_t v)
{
    uint64_t x = v & 0x1FFFFFu;
    x = (x | (x << 32)) & 0x001F00000000FFFFull;
    x = (x | (x << 16)) & 0x001F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

constexpr int kCodeBits = 63;

__device__ inline uint32_t quantise21(float c, float lo, float ext)
{
    // floor((c - lo) / ext * 2^21), clamped to [0, 2^21 - 1]; a flat axis maps to 0
    if (!(ext > 0.0f)) return 0u;
    float q = (c - lo) / ext * 2097152.0f;
    q = fminf(fmaxf(q, 0.0f), 2097151.0f);
    return (uint32_t)q;
}

__global__ void k_morton(BuildArgs a)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= a.n_t) return;
    const int32_t *b = a.bounds + 6 * mesh_of(a.off, a.M, j);
    const float lx = ordered_to_float(b[0]), ly = ordered_to_float(b[1]), lz = ordered_to_float(b[2]);
    const float hx = ordered_to_float(b[3]), hy = ordered_to_float(b[4]), hz = ordered_to_float(b[5]);
    const uint32_t qx = quantise21(a.cent[j], lx, hx - lx);
    const uint32_t qy = quantise21(a.cent[a.n_t + j], ly, hy - ly);
    const uint32_t qz = quantise21(a.cent[2 * a.n_t + j], lz, hz - lz);
    a.keys[j] = (spread3(qx) << 2) | (spread3(qy) << 1) | spread3(qz);
    a.order[j] = (uint32_t)j;
}

// Common-prefix length of the augmented keys (key, index) of the sorted
// neighbours k and k+1: the leading equal key bits while the keys differ,
// else 64 plus the leading equal index bits, so equal keys are split by index
// and duplicate codes still form a valid radix tree.  A longer prefix is a
// smaller key distance.
__device__ inline uint8_t split_prefix(const uint64_t *__restrict__ keys, int32_t k)
{
    const uint64_t x = keys[k] ^ keys[k + 1];
    if (x) return (uint8_t)__clzll((long long)x);
    return (uint8_t)(64 + __clz((int)((uint32_t)k ^ (uint32_t)(k + 1))));
}

__device__ inline void write_child(Node *__restrict__ p, int side, const float bx[6], int32_t ref)
{
    float *f = p->f + 6 * side;
#pragma unroll
    for (int k = 0; k < 6; ++k) f[k] = bx[k];
    p->ref[side] = ref;
}

// State of one climbing node: its box, leaf range [l, r], reference and
// height (internal levels below it).
struct Climb {
    float box[6];
    int32_t l, r, ref, h;
};

// The neighbour to join, within the mesh's leaf range [lo, hi]: across the
// split with the longer common prefix (smaller key distance; the two splits
// around a node of the radix tree never tie).  `prefix(k)` is the prefix
// length at split k.  Returns the parent index (= that split position) and
// our side in it (0: left child, 1: right child).
template <typename Prefix>
__device__ inline int32_t choose_parent(Prefix prefix, int32_t lo, int32_t hi, int32_t l, int32_t r, int &side)
{
    if (l == lo || (r != hi && prefix(r) > prefix(l - 1))) {
        side = 0;
        return r;
    }
    side = 1;
    return l - 1;
}

__device__ inline void merge(Climb &c, const float *g, int32_t other_bound, int32_t other_h, int side,
                             int32_t parent, int32_t leaf_size)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        c.box[k] = fminf(c.box[k], g[k]);
        c.box[3 + k] = fmaxf(c.box[3 + k], g[3 + k]);
    }
    if (side == 0) c.r = other_bound;
    else c.l = other_bound;
    c.h = 1 + (c.h > other_h ? c.h : other_h);
    c.ref = (c.r - c.l + 1 <= leaf_size) ? leaf_ref(c.l, c.r - c.l + 1) : parent;
    if (c.ref < 0) c.h = 0;  // a collapsed range is a leaf
}

// Entry node `hi` (the mesh's last record): the root as its left child (the
// paper keeps the root as the left child of its last internal node record),
// an empty far box on the right.
__device__ inline void write_entry(const BuildArgs &a, int32_t m, int32_t lo, int32_t hi, const Climb &c)
{
    Node *e = a.nodes + hi;
    write_child(e, 0, c.box, c.ref);
    const float far[6] = {FLT_MAX, FLT_MAX, FLT_MAX, FLT_MAX, FLT_MAX, FLT_MAX};
    write_child(e, 1, far, leaf_ref(lo, 1));
    e->aux[0] = lo;
    e->aux[1] = hi;
    a.mesh_height[m] = c.h;
    a.mesh_root[m] = c.ref;
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < 6; ++k) s = fmaxf(s, fabsf(c.box[k]));
    a.mesh_scale[m] = s;
}

// Four-way view: record n lists the boxes and references of up to four of
// n's descendants whose subtrees make up n's, quantised inside their union
// box.  Every node gets its record, also those no traversal reaches
// (inside collapsed leaves).
//
// Grid step per axis: the smallest power of two 2^e with (255 - 2^-10) 2^e >=
// the box extent, formed in FP64 (the extent of a box of finite FP32 numbers
// can exceed the FP32 range).  Planes are placed in FP64 too: an offset from the
// corner is off by at most 2^-53 of itself, 2^-45 steps, and the scaling by a
// power of two is exact, so a plane moved outward by kQuantMargin before it is
// rounded outward (quant_plane) lies outside the child's box by 2^-11 steps at least, which
// the box test needs.
__device__ inline int quant_exponent(double ext)
{
    const double x = ext * ((1.0 + 0x1p-40) / (255.0 - 0x1p-10));
    if (!(x > 0x1p-126)) return -126;
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const int e = (int)(u >> 52) - 1023 + ((u & 0xFFFFFFFFFFFFFull) ? 1 : 0);
    return e > 127 ? 127 : e;
}

// The plane nearest to v, moved by `out` (half a step and the margin) so that
// rounding to nearest rounds outward: adding 1.5 2^52 leaves the integer in the
// low word.
__device__ inline uint32_t quant_plane(float v, float corner, double inv, double out)
{
    const double at = fma((double)v - (double)corner, inv, out) + 0x1.8p52;
    const int32_t q = (int32_t)__double_as_longlong(at);
    return (uint32_t)min(max(q, 0), 255);
}

// The children of a record, from the node's two: the internal one with the
// larger box surface gives way to its own two, twice.
struct Wide {
    float box[4][6];
    int32_t ref[4];
    int k = 0;
    __device__ inline void add(const float *b, int32_t r)
    {
        put(k, b, r);
        ++k;
    }
    __device__ inline void put(int at, const float *b, int32_t r)
    {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s == at) {
#pragma unroll
                for (int q = 0; q < 6; ++q) box[s][q] = b[q];
                ref[s] = r;
            }
        }
    }
    // `child(c, side, box)` reads node c's child: its box, and its reference
    template <typename Child>
    __device__ inline void open(Child child)
    {
#pragma unroll
        for (int turn = 0; turn < 2; ++turn) {
            int at = -1;
            int32_t c = -1;
            float most = -1.0f;
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                if (s >= k || ref[s] < 0) continue;
                const float x = box[s][3] - box[s][0], y = box[s][4] - box[s][1], z = box[s][5] - box[s][2];
                const float area = x * y + y * z + z * x;
                if (at < 0 || area > most) {
                    at = s;
                    c = ref[s];
                    most = area;
                }
            }
            if (at < 0) break;
            // in place, so the children stay in Morton order
#pragma unroll
            for (int s = 3; s > 0; --s) {
                if (s > at + 1) {
#pragma unroll
                    for (int q = 0; q < 6; ++q) box[s][q] = box[s - 1][q];
                    ref[s] = ref[s - 1];
                }
            }
            float b[6];
            int32_t r = child(c, 0, b);
            put(at, b, r);
            r = child(c, 1, b);
            put(at + 1, b, r);
            ++k;
        }
    }
    __device__ inline void store(Node4 *out, int64_t n) const
    {
        Node4 w;
        float lo[3], step[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float l = FLT_MAX, h = -FLT_MAX;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (s < k) {
                    l = fminf(l, box[s][a]);
                    h = fmaxf(h, box[s][3 + a]);
                }
            }
            l = fmaxf(l, -FLT_MAX);  // an infinite box is cut at the finite numbers
            const int e = quant_exponent((double)fminf(h, FLT_MAX) - (double)l);
            const double inv = __longlong_as_double((long long)(1023 - e) << 52);
            lo[a] = l;
            step[a] = ldexpf(1.0f, e);  // a normal float for e in [-126, 127]
            uint32_t ql = 0, qh = 0;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                uint32_t x = 255u, y = 0u;  // unused slot: an empty box
                if (s < k) {
                    x = quant_plane(box[s][a], l, inv, -0.5 - kQuantMargin);
                    y = quant_plane(fminf(box[s][3 + a], FLT_MAX), l, inv, 0.5 + kQuantMargin);
                }
                ql |= x << (8 * s);
                qh |= y << (8 * s);
            }
            w.lo[a] = ql;
            w.hi[a] = qh;
        }
        w.ox = lo[0];
        w.oy = lo[1];
        w.oz = lo[2];
        w.sx = step[0];
        w.sy = step[1];
        w.sz = step[2];
#pragma unroll
        for (int s = 0; s < 4; ++s) w.ref[s] = s < k ? ref[s] : leaf_ref((int32_t)n, 1);
        const uint4 *src = reinterpret_cast<const uint4 *>(&w);
        uint4 *dst = reinterpret_cast<uint4 *>(out);
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[q] = src[q];
    }
};

// The subtrees a workgroup has completed but cannot join to their siblings,
// which lie in other workgroups' leaves: a list per local block, in leaf
// order.  Each side of a block's range cuts a path from a mesh's root, and the
// subtrees hang off it, at most 90 per side (prefix lengths grow along a
// path).  An item: leaf range l, r, reference, height, box, and the prefix
// lengths at splits l - 1 and r.
constexpr int kListItems = 192;
constexpr int kItemWords = 12;
constexpr int kListWords = 4 + kListItems * kItemWords;  // word 0: items in use

struct Item {
    Climb c;
    int32_t pre_l, pre_r;
};

__device__ inline void put_item(const BuildArgs &a, int32_t *list, int32_t at, const Item &x)
{
    if (at >= kListItems) {  // cannot happen in a tree of at most 90 levels; never written past the list
        atomicOr(&a.scalars[kBadIndex], 2);
        return;
    }
    int4 *w = reinterpret_cast<int4 *>(list + 4 + kItemWords * at);
    w[0] = make_int4(x.c.l, x.c.r, x.c.ref, x.c.h);
    w[1] = make_int4(__float_as_int(x.c.box[0]), __float_as_int(x.c.box[1]), __float_as_int(x.c.box[2]),
                     __float_as_int(x.c.box[3]));
    w[2] = make_int4(__float_as_int(x.c.box[4]), __float_as_int(x.c.box[5]), x.pre_l, x.pre_r);
}

__device__ inline Item get_item(const int32_t *list, int32_t at)
{
    const int4 *w = reinterpret_cast<const int4 *>(list + 4 + kItemWords * at);
    const int4 u = w[0], v = w[1], t = w[2];
    Item x;
    x.c.l = u.x;
    x.c.r = u.y;
    x.c.ref = u.z;
    x.c.h = u.w;
    x.c.box[0] = __int_as_float(v.x);
    x.c.box[1] = __int_as_float(v.y);
    x.c.box[2] = __int_as_float(v.z);
    x.c.box[3] = __int_as_float(v.w);
    x.c.box[4] = __int_as_float(t.x);
    x.c.box[5] = __int_as_float(t.y);
    x.pre_l = t.z;
    x.pre_r = t.w;
    return x;
}

// Places of set bits in order: the first wave counts the bits below each of
// W <= 64 words (and all of them: the return value, in that wave).
template <int W>
__device__ inline int32_t count_below(const uint32_t *bits, int32_t *below)
{
    const int t = (int)threadIdx.x;
    const int32_t n = t < W ? __popc(bits[t]) : 0;
    int32_t x = n;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o, 64);
        if (t >= o) x += y;
    }
    if (t < W) below[t] = x - n;
    return __shfl(x, 63, 64);
}

__device__ inline int32_t place_of(const uint32_t *bits, const int32_t *below, int32_t k)
{
    return below[k >> 5] + __popc(bits[k >> 5] & ((1u << (k & 31)) - 1u));
}

// One node's two children in LDS: a climb writes its side, then counts itself
// in (bit `side` of the node's flag).
//
// A wave's LDS operations are performed in the order it issues them, so the
// child data is in place before the flag moves, and the sibling's data read
// right after the update (before its result is known; unused if we arrive
// first) is complete whenever the flag shows that the sibling arrived.  The
// signal fences keep the compiler from moving LDS accesses across the update;
// one wait then covers the update and the reads.
struct Slots {
    int32_t *flag;
    float (*box)[12];
    int32_t (*ref)[2], (*bound)[2], (*h)[2];
};

// Returns false when the sibling has not arrived (it goes on); else fills
// in the sibling's box, far bound and height.
__device__ inline bool arrive_at(const Slots &s, int32_t slot, int side, const Climb &c, float *g, int32_t &ob,
                                 int32_t &oh)
{
#pragma unroll
    for (int k = 0; k < 6; ++k) s.box[slot][6 * side + k] = c.box[k];
    s.ref[slot][side] = c.ref;
    s.bound[slot][side] = side ? c.r : c.l;
    s.h[slot][side] = c.h;
    const int other = 1 - side;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    const int32_t prev =
        __hip_atomic_fetch_or(&s.flag[slot], 1 << side, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
    for (int k = 0; k < 6; ++k) g[k] = s.box[slot][6 * other + k];
    ob = s.bound[slot][other];
    oh = s.h[slot][other];
    // an empty statement that uses the loaded values keeps the compiler
    // from sinking the reads below the branch (it emits no instruction)
    asm volatile("" : : "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "v"(g[4]), "v"(g[5]), "v"(ob), "v"(oh));
    return prev != 0;
}

__device__ inline void store_node(const Slots &s, int32_t slot, Node *q)
{
#pragma unroll
    for (int k = 0; k < 12; ++k) q->f[k] = s.box[slot][k];
    q->ref[0] = s.ref[slot][0];
    q->ref[1] = s.ref[slot][1];
    q->aux[0] = s.bound[slot][0];
    q->aux[1] = s.bound[slot][1];
}

// The one child that has arrived at a node (flag f: 1 the left one, 2 the
// right one) whose split is p.
__device__ inline Climb half_of(const Slots &s, int32_t slot, int32_t f, int32_t p)
{
    const int side = f == 1 ? 0 : 1;
    Climb c;
#pragma unroll
    for (int k = 0; k < 6; ++k) c.box[k] = s.box[slot][6 * side + k];
    c.ref = s.ref[slot][side];
    c.h = s.h[slot][side];
    c.l = side == 0 ? s.bound[slot][0] : p + 1;
    c.r = side == 0 ? p : s.bound[slot][1];
    return c;
}

// Local pass: each workgroup owns kLocal consecutive sorted leaves (512 with
// 512 threads, four workgroups to a CU; or 2048 with 1024 threads, whose LDS
// node slots fit gfx950's 160 KiB).  A node whose leaf range lies inside that block has its whole
// subtree inside it, so these subtrees are completed here with the arrival
// flags and child records in LDS.  The largest of them go to the block's list
// for the joining pass.
template <int kLocal, int kLocalThreads>
__global__ __launch_bounds__(kLocalThreads) void k_lbvh_local(BuildArgs a)
{
    constexpr int kPer = kLocal / kLocalThreads;  // leaves per thread
    __shared__ int32_t lflag[kLocal];
    __shared__ float lbox[kLocal][12];
    __shared__ int32_t lref[kLocal][2];
    __shared__ int32_t lbound[kLocal][2];
    __shared__ int32_t lh[kLocal][2];
    __shared__ uint8_t lpre[kLocal + 1];  // prefix length at split k, k = B0-1 .. B1
    __shared__ uint32_t bits[kLocal / 32];  // first leaves of the subtrees to hand over
    __shared__ int32_t below[kLocal / 32];
    const Slots slots = {lflag, lbox, lref, lbound, lh};
    const int32_t n = (int32_t)a.n_t;
    const int32_t B0 = (int32_t)blockIdx.x * kLocal;
    const int32_t B1 = (B0 + kLocal < n ? B0 + kLocal : n) - 1;  // last leaf of this block
    // split prefixes of the block (and the split before it) into LDS
    for (int t = threadIdx.x; t <= kLocal; t += kLocalThreads) {
        const int32_t k = B0 - 1 + t;
        lpre[t] = k >= 0 && k <= B1 && k < n - 1 ? split_prefix(a.keys, k) : 0;
        if (t < kLocal) lflag[t] = 0;
        if (t < kLocal / 32) bits[t] = 0;
    }
    __syncthreads();
    const auto prefix = [&](int32_t k) { return (int32_t)lpre[k - B0 + 1]; };

    // leaf set-up for all of this thread's leaves first (their loads overlap)
    Climb cl[kPer];
    int32_t lo_[kPer], hi_[kPer], m_[kPer];
    bool act[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int32_t i = B0 + (int32_t)threadIdx.x + q * kLocalThreads;
        act[q] = i < n;
        m_[q] = lo_[q] = hi_[q] = 0;
        if (!act[q]) continue;
        Climb &c = cl[q];
        const int32_t m = mesh_of(a.off, a.M, i);
        const int32_t lo = (int32_t)a.off[m];
        const int32_t hi = (int32_t)a.off[m + 1] - 1;
        m_[q] = m;
        lo_[q] = lo;
        hi_[q] = hi;
        // leaf i: pack the triangle in sorted order and form its box
        int32_t id = (int32_t)a.order[i];
        if (id < lo || id > hi) {  // cannot happen after a correct sort; never read outside T
            atomicOr(&a.scalars[kBadIndex], 2);
            id = lo;
        }
        a.rank[id] = i;
        int32_t va = a.T[3 * id], vb = a.T[3 * id + 1], vd = a.T[3 * id + 2];
        // an out-of-range index is reported by k_centroids; read vertex 0
        // instead so that no access leaves the vertex array, and mark the
        // record (the adjoint skips it)
        const bool bad = va < 0 || va >= a.n_v || vb < 0 || vb >= a.n_v || vd < 0 || vd >= a.n_v;
        if (va < 0 || va >= a.n_v) va = 0;
        if (vb < 0 || vb >= a.n_v) vb = 0;
        if (vd < 0 || vd >= a.n_v) vd = 0;
        const row3 p0 = ld3(a.V + 3 * (int64_t)va), p1 = ld3(a.V + 3 * (int64_t)vb), p2 = ld3(a.V + 3 * (int64_t)vd);
        const float v0x = p0.x, v0y = p0.y, v0z = p0.z;
        const float v1x = p1.x, v1y = p1.y, v1z = p1.z;
        const float v2x = p2.x, v2y = p2.y, v2z = p2.z;
        Tri tr;
        tr.a = make_float4(v0x, v0y, v0z, v1x);
        tr.b = make_float4(v1y, v1z, v2x, v2y);
        tr.c = make_float4(v2z, __int_as_float(id - lo), 0.0f, bad ? 1.0f : 0.0f);  // id within its mesh
        a.tris[i] = tr;
        c.box[0] = fminf(v0x, fminf(v1x, v2x));
        c.box[1] = fminf(v0y, fminf(v1y, v2y));
        c.box[2] = fminf(v0z, fminf(v1z, v2z));
        c.box[3] = fmaxf(v0x, fmaxf(v1x, v2x));
        c.box[4] = fmaxf(v0y, fmaxf(v1y, v2y));
        c.box[5] = fmaxf(v0z, fmaxf(v1z, v2z));
        c.l = c.r = i;
        c.ref = leaf_ref(i, 1);
        c.h = 0;
    }

    // each thread climbs from its leaves one after the other; a climb that
    // arrives first at a node stops, so no thread ever waits
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        Climb &c = cl[q];
        const int32_t m = m_[q], lo = lo_[q], hi = hi_[q];
        bool up = act[q];
        act[q] = false;  // from here on: handed over
        // a climb inside the block takes fewer than kLocal steps
        for (int step = 0; up; ++step) {
            if (c.l == lo && c.r == hi) {  // the whole mesh fits in this block
                write_entry(a, m, lo, hi, c);
                break;
            }
            int side;
            // inside the block [l, r] lies in [B0, B1], so both splits are in lpre
            const int32_t parent = choose_parent(prefix, lo, hi, c.l, c.r, side);
            if (parent < B0 || parent >= B1 || step >= kLocal) {
                // the sibling lies outside the block
                atomicOr(&bits[(c.l - B0) >> 5], 1u << ((c.l - B0) & 31));
                act[q] = true;
                break;
            }
            float g[6];
            int32_t ob, oh;
            if (!arrive_at(slots, parent - B0, side, c, g, ob, oh)) break;
            merge(c, g, ob, oh, side, parent, a.leaf_size);
        }
    }
    __syncthreads();
    // the subtrees to hand over: of the climbs that left the block and of the
    // nodes with one child
    if (gridDim.x > 1) {  // (one block: every mesh is complete)
        for (int tid = threadIdx.x; tid < B1 - B0; tid += kLocalThreads) {
            const int32_t p = B0 + tid, f = lflag[tid];
            if (f == 1 || f == 2) {
                const int32_t l = (f == 1 ? lbound[tid][0] : p + 1) - B0;
                atomicOr(&bits[l >> 5], 1u << (l & 31));
            }
        }
        // the block's list, in leaf order
        int32_t *const list = a.joins + (int64_t)kListWords * blockIdx.x;
        __syncthreads();
        if (threadIdx.x < 64) {
            const int32_t total = count_below<kLocal / 32>(bits, below);
            if (threadIdx.x == 0) list[0] = total < kListItems ? total : kListItems;
        }
        __syncthreads();
        const auto hand = [&](const Climb &c) {
            put_item(a, list, place_of(bits, below, c.l - B0), {c, prefix(c.l - 1), prefix(c.r)});
        };
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            if (act[q]) hand(cl[q]);
        }
        for (int tid = threadIdx.x; tid < B1 - B0; tid += kLocalThreads) {
            const int32_t f = lflag[tid];
            if (f == 1 || f == 2) hand(half_of(slots, tid, f, B0 + tid));
        }
    }
    // publish the block's completed nodes (splits B0 .. B1-1), last: the records
    // take the registers of the climbs
    for (int tid = threadIdx.x; tid < B1 - B0; tid += kLocalThreads) {
        const int32_t p = B0 + tid;
        if (lflag[tid] != 3) continue;
        store_node(slots, tid, a.nodes + p);
        if (a.nodes4) {
            // both children's subtrees lie in the block, so the four-way
            // record's boxes are here (a later pass over the node records
            // would read them all again: 45 us at 499,280 triangles)
            Wide w;
            w.add(lbox[tid], lref[tid][0]);
            w.add(lbox[tid] + 6, lref[tid][1]);
            w.open([&](int32_t c, int side, float *b) -> int32_t {
                const int slot = c - B0;
#pragma unroll
                for (int q = 0; q < 6; ++q) b[q] = lbox[slot][6 * side + q];
                return lref[slot][side];
            });
            w.store(a.nodes4 + p, n);
            a.laid_out[p] = 1;
        }
    }
}

// Joining pass: the subtrees of the local blocks' lists, in leaf order, climb
// on in LDS, one workgroup for `per` consecutive lists.  It takes as many
// lists as make kJoin items (at least five), replaces them by the list of
// what they leave, and goes on with that and the next ones until one list is
// left; with the last workgroup every mesh is complete.  Bound by the chain of
// LDS updates of the longest climb.  When the climbs met in memory, past the
// per-XCD caches, they cost about 2 us a level, and each leaf had a word that
// said whether its climb went on: 46 us at 499,280 triangles in blocks of
// 2048 (both launches here: 37, in blocks of 512 41), 29 us at 29,768 (20) and
// 111 us for the 64 meshes of 1,000 to 200,000 triangles (45, and 59).
//
// List i of the pass is block min(stride i + stride - 1, nb - 1)'s: a
// workgroup leaves its result in the place of its last list.
constexpr int kJoin = 1024;

__global__ __launch_bounds__(kJoin) void k_lbvh_join(BuildArgs a, int32_t nb, int32_t stride, int32_t per)
{
    __shared__ int32_t lflag[kJoin];
    __shared__ float lbox[kJoin][12];
    __shared__ int32_t lref[kJoin][2];
    __shared__ int32_t lbound[kJoin][2];
    __shared__ int32_t lend[kJoin][2];  // bounds as item numbers
    __shared__ int32_t lh[kJoin][2];
    __shared__ uint8_t lpre[kJoin + 1];  // prefix length before item k
    __shared__ uint32_t bits[kJoin / 32];
    __shared__ int32_t below[kJoin / 32];
    __shared__ int32_t first[65];  // first item of each list taken
    __shared__ int32_t taken;
    const Slots slots = {lflag, lbox, lref, lbound, lh};
    const int tid = (int)threadIdx.x;
    const int32_t lists = (nb + stride - 1) / stride;
    int32_t at = (int32_t)blockIdx.x * per;
    const int32_t end = at + per < lists ? at + per : lists;
    const auto list_of = [&](int32_t i) {
        const int64_t b = (int64_t)stride * i + stride - 1;
        return a.joins + kListWords * (b < nb ? b : nb - 1);
    };
    // at least one list goes with each turn
    while (at < end - 1) {
        if (tid < 64) {
            int32_t c = at + tid < end ? list_of(at + tid)[0] : 0;
            if (c < 0 || c > kListItems) c = 0;
            int32_t x = c;
            for (int o = 1; o < 64; o <<= 1) {
                const int32_t y = __shfl_up(x, o, 64);
                if (tid >= o) x += y;
            }
            first[tid + 1] = x;
            if (tid == 0) first[0] = 0;
            const uint64_t fit = __builtin_amdgcn_ballot_w64(at + tid < end && x <= kJoin);
            if (tid == 0) taken = __popcll(fit);
        }
        if (tid < kJoin / 32) bits[tid] = 0;
        lflag[tid] = 0;
        __syncthreads();
        const int32_t t = taken, K = first[t];
        Item x = {};
        int32_t m = 0, lo = 0, hi = -1;
        const bool has = tid < K;
        if (has) {
            int32_t q = 0, e = t;  // first[q] <= tid < first[e]
            while (e - q > 1) {
                const int32_t mid = (q + e) >> 1;
                if (first[mid] <= tid) q = mid;
                else e = mid;
            }
            x = get_item(list_of(at + q), tid - first[q]);
            m = mesh_of(a.off, a.M, x.c.l);
            lo = (int32_t)a.off[m];
            hi = (int32_t)a.off[m + 1] - 1;
            lpre[tid + 1] = (uint8_t)x.pre_r;
            if (tid == 0) lpre[0] = (uint8_t)x.pre_l;
        }
        const int32_t split = x.c.r;  // between this item and the next
        __syncthreads();
        Climb &c = x.c;
        int32_t il = tid, ir = tid;  // the climb's items
        bool handed = false;
        for (int step = 0; has; ++step) {
            if (c.l == lo && c.r == hi) {
                write_entry(a, m, lo, hi, c);
                break;
            }
            const int side = c.l == lo || (c.r != hi && lpre[ir + 1] > lpre[il]) ? 0 : 1;
            const int32_t slot = side == 0 ? ir : il - 1;
            if (slot < 0 || slot >= K - 1 || step >= kJoin) {
                atomicOr(&bits[il >> 5], 1u << (il & 31));
                handed = true;
                break;
            }
            lend[slot][side] = side ? ir : il;
            float g[6];
            int32_t ob, oh;
            if (!arrive_at(slots, slot, side, c, g, ob, oh)) break;
            const int32_t oe = lend[slot][1 - side];
            merge(c, g, ob, oh, side, side == 0 ? c.r : c.l - 1, a.leaf_size);
            if (side == 0) ir = oe;
            else il = oe;
        }
        __syncthreads();
        const int32_t f = tid < K - 1 ? lflag[tid] : 0;
        if (f == 3) store_node(slots, tid, a.nodes + split);
        const int32_t hl = f == 1 ? lend[tid][0] : tid + 1, hr = f == 1 ? tid : lend[tid][1];
        if (f == 1 || f == 2) atomicOr(&bits[hl >> 5], 1u << (hl & 31));
        __syncthreads();
        int32_t *const out = list_of(at + t - 1);
        if (tid < 64) {
            const int32_t total = count_below<kJoin / 32>(bits, below);
            if (tid == 0) out[0] = total < kListItems ? total : kListItems;
        }
        __syncthreads();
        if (handed) put_item(a, out, place_of(bits, below, il), {c, lpre[il], lpre[ir + 1]});
        if (f == 1 || f == 2)
            put_item(a, out, place_of(bits, below, hl), {half_of(slots, tid, f, split), lpre[hl], lpre[hr + 1]});
        at += t - 1;
        __syncthreads();
    }
}

// The records the local pass has not laid out: nodes whose subtrees cross its
// blocks, the entry nodes, and every record of a tree built without the
// four-way view.
__global__ __launch_bounds__(256) void k_widen(const Node *__restrict__ nodes, const uint8_t *__restrict__ laid_out,
                                               int64_t n, Node4 *__restrict__ out)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n || laid_out[j]) return;
    // a node no climb reached (inside a collapsed leaf) may hold anything:
    // its references are checked before use
    const auto read = [&](int64_t c, int side, float *b) -> int32_t {
#pragma unroll
        for (int q = 0; q < 6; ++q) b[q] = nodes[c].f[6 * side + q];
        const int32_t r = nodes[c].ref[side];
        return r < n ? r : leaf_ref(0, 1);
    };
    Wide w;
    for (int side = 0; side < 2; ++side) {
        float b[6];
        const int32_t r = read(j, side, b);
        // the entry record's far box (all FLT_MAX) is no child: the slot
        // stays empty
        bool far = true;
        for (int q = 0; q < 6; ++q) far = far && b[q] == FLT_MAX;
        if (!far) w.add(b, r);
    }
    w.open(read);
    w.store(out + j, n);
}

// Whether the handle's tree gets the four-way view.
bool wide_view(const rsi_bvh *h) { return h->width == 4 && h->n_t > 0 && h->nodes4; }

BuildArgs make_build_args(rsi_bvh *h, const float *V)
{
    BuildArgs a;
    a.M = h->M;
    a.off = h->tri_off;
    a.V = V;
    a.n_v = h->n_v;
    a.T = h->T;
    a.n_t = h->n_t;
    a.cent = h->cent;
    a.keys = h->keys;
    a.order = h->order;
    a.rank = h->rank;
    a.nodes = h->nodes;
    a.nodes4 = wide_view(h) ? h->nodes4 : nullptr;
    a.tris = h->tris;
    a.laid_out = h->laid_out;
    a.joins = h->joins;
    a.bounds = h->mesh_bounds;
    a.mesh_height = h->mesh_height;
    a.mesh_root = h->mesh_root;
    a.mesh_scale = h->mesh_scale;
    a.scalars = h->scalars;
    a.leaf_size = h->leaf_size;
    return a;
}

// Leaves per local block.  Up to kOneBlock one block holds the mesh whole and
// nothing is left to join.  Above that 512: four workgroups share a CU, so one
// loads or stores while another climbs, which the subtrees left to the joining
// pass (four times as many blocks' worth) cost less than.  Local pass, 2048
// leaves and 1024 threads -> 512 and 512: 499,280 triangles 53 -> 42 us, 199,712
// 42 -> 24, the 64-mesh batch 244 -> 174; with 256 threads for 512 leaves 43,
// 30 and 199.  Blocks of 256 lose as much in the joining pass as they gain
// (rebuild of 1.5M triangles 342 -> 362 us).  Rebuilds in one block and in
// blocks of 512 with a join: 1,250 triangles 53.8 and 56.4 us, 1,568 60.4 and
// 57.2, 2,048 66.8 and 52.1 (the block's four-way records take 5 us more from one
// workgroup than from the grid of a pass of their own).
constexpr int64_t kOneBlock = 1400;

int64_t local_leaves(int64_t n) { return n > kOneBlock ? 512 : 2048; }

int64_t local_blocks(int64_t n) { return (n + local_leaves(n) - 1) / local_leaves(n); }

hipError_t run_hierarchy(const BuildArgs &a, hipStream_t s)
{
    const int32_t n = (int32_t)a.n_t;
    const unsigned nb = (unsigned)local_blocks(n);
    if (local_leaves(n) == 512) {
        hipLaunchKernelGGL((k_lbvh_local<512, 512>), dim3(nb), dim3(512), 0, s, a);
    } else {
        hipLaunchKernelGGL((k_lbvh_local<2048, 1024>), dim3(nb), dim3(1024), 0, s, a);
    }
    // up to 64 lists (some 13 items each) by one workgroup, more by one per 64
    // and one for what those leave
    const int32_t lists = (int32_t)nb, groups = (lists + 63) / 64;
    if (groups > 1) {
        hipLaunchKernelGGL(k_lbvh_join, dim3((unsigned)groups), dim3(kJoin), 0, s, a, lists, 1, 64);
        hipLaunchKernelGGL(k_lbvh_join, dim3(1), dim3(kJoin), 0, s, a, lists, 64, groups);
    } else if (lists > 1) {
        hipLaunchKernelGGL(k_lbvh_join, dim3(1), dim3(kJoin), 0, s, a, lists, 1, lists);
    }
    return hipGetLastError();
}

unsigned init_grid(const BuildArgs &a)
{
    const int64_t n = a.n_t > a.M ? a.n_t : a.M;
    return (unsigned)((n + 255) / 256);
}

}  // namespace

int64_t join_words(int64_t n) { return n > 0 ? kListWords * local_blocks(n) : 0; }

hipError_t launch_gather(rsi_bvh *h, hipStream_t s)
{
    const int64_t total = h->n_v + h->n_t;
    if (total == 0) return hipSuccess;
    int64_t grid = (total + 255) / 256;
    if (grid > 65536) grid = 65536;
    hipLaunchKernelGGL(k_clear_gather_flag, dim3(1), dim3(1), 0, s, h->scalars);
    hipLaunchKernelGGL(k_gather, dim3((unsigned)grid), dim3(256), 0, s, h->M, h->src_V, h->src_T, h->vert_off,
                       h->tri_off, h->V_all, h->T, h->scalars);
    return hipGetLastError();
}

hipError_t launch_widen(rsi_bvh *h, hipStream_t s)
{
    if (!wide_view(h)) {
        h->width_built = 2;
        return hipSuccess;
    }
    hipLaunchKernelGGL(k_widen, dim3((unsigned)((h->n_t + 255) / 256)), dim3(256), 0, s, h->nodes,
                       h->laid_out, h->n_t, h->nodes4);
    h->width_built = 4;
    return hipGetLastError();
}

hipError_t launch_build(rsi_bvh *h, const float *V, hipStream_t s)
{
    const int64_t n = h->n_t;
    if (n == 0) return hipSuccess;
    const BuildArgs a = make_build_args(h, V);
    hipLaunchKernelGGL(k_init, dim3(init_grid(a)), dim3(256), 0, s, a);
    if (n >= 131072)
        hipLaunchKernelGGL(k_centroids<8>, dim3((unsigned)((n + 8 * kCentBlock - 1) / (8 * kCentBlock))),
                           dim3(kCentBlock), 0, s, a);
    else
        hipLaunchKernelGGL(k_centroids<1>, dim3((unsigned)((n + kCentBlock - 1) / kCentBlock)), dim3(kCentBlock), 0, s,
                           a);
    const int64_t *mesh_off = h->M > 1 ? h->tri_off : nullptr;
    BuildArgs km = a;  // the codes go where the sort wants its input
    hipError_t e = sort_source(h->keys, h->order, n, kCodeBits, h->sort, mesh_off, h->M, h->most_t, &km.keys, &km.order);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_morton, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, km);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    e = radix_sort_pairs(h->keys, h->order, n, kCodeBits, h->sort, s, mesh_off, h->M, h->most_t);
    if (e != hipSuccess) return e;
    e = run_hierarchy(a, s);
    if (e != hipSuccess) return e;
    return launch_widen(h, s);
}

hipError_t launch_refit(rsi_bvh *h, const float *V, hipStream_t s)
{
    if (h->n_t == 0) return hipSuccess;
    const BuildArgs a = make_build_args(h, V);
    hipLaunchKernelGGL(k_init, dim3(init_grid(a)), dim3(256), 0, s, a);
    hipError_t e = run_hierarchy(a, s);
    if (e != hipSuccess) return e;
    return launch_widen(h, s);
}

}  // namespace rsi
