// order.hip -- Morton order of segments (the paper's v2.2 step, Section 4.1:
// rays sorted so that neighbouring threads follow similar paths through the
// tree).  The key of a segment is the octant of its direction (3 bits, most
// significant) above the 30-bit Morton code of its midpoint quantised to
// 2^10 levels per axis inside the midpoints' bounding box; the radix sort of
// the build orders (key, index) pairs stably.  A caller computes the order
// once and reuses it for every mesh the segments are tested against, and
// gathers the segments into that order (rsi_gather_segments).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rsi_host.h"

namespace rsi {
namespace {

constexpr int kSegKeyBits = 33;

__global__ void k_seg_bounds_init(int32_t *b)
{
    if (threadIdx.x < 3) b[threadIdx.x] = 0x7FFFFFFF;      // ordered min
    else if (threadIdx.x < 6) b[threadIdx.x] = (int32_t)0x80000000;  // ordered max
}

// Bounding box of the midpoints: one workgroup of 1,024 threads per CU,
// reduced in registers, by wave and in LDS, then one ordered-int atomic per
// workgroup and bound.  The atomics meet on one cache line and are
// serialised: 1,024 workgroups took 25 us for them.  The arrays are read as
// streams of floats, four at a time (VEC; both pointers 16-byte aligned) or
// one; the number of threads is a multiple of 3, so every value of a thread's
// at a place in its vector belongs to the same axis.
constexpr int kBoundThreads = 960;

template <bool VEC>
__global__ __launch_bounds__(kBoundThreads) void k_seg_bounds(const float *__restrict__ S, const float *__restrict__ E,
                                                              int64_t n, int32_t *__restrict__ b)
{
    constexpr int W = VEC ? 4 : 1;
    __shared__ int32_t lb[6];
    const int tid = threadIdx.x;
    if (tid < 6) lb[tid] = 0x7FFFFFFF;
    __syncthreads();
    const int64_t total = 3 * n, threads = (int64_t)gridDim.x * kBoundThreads;
    const int64_t me = (int64_t)blockIdx.x * kBoundThreads + tid;
    int32_t mn[W], mx[W];  // minima, and minima of the reversed order (~)
#pragma unroll
    for (int k = 0; k < W; ++k) mn[k] = mx[k] = 0x7FFFFFFF;
    const int64_t whole = total / W;
#pragma unroll 4
    for (int64_t i = me; i < whole; i += threads) {
        float s[W], e[W];
        if constexpr (VEC) {
            *reinterpret_cast<float4 *>(s) = reinterpret_cast<const float4 *>(S)[i];
            *reinterpret_cast<float4 *>(e) = reinterpret_cast<const float4 *>(E)[i];
        } else {
            s[0] = S[i];
            e[0] = E[i];
        }
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const int32_t m = float_to_ordered(0.5f * (s[k] + e[k]));
            mn[k] = min(mn[k], m);
            mx[k] = min(mx[k], ~m);
        }
    }
    // by axis: the thread's value k is of axis (W me + k) mod 3
    int32_t v[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = 0x7FFFFFFF;
    const int first = (int)(W * me % 3);
#pragma unroll
    for (int k = 0; k < W; ++k) {
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            if ((first + k) % 3 == x) {
                v[x] = min(v[x], mn[k]);
                v[3 + x] = min(v[3 + x], mx[k]);
            }
        }
    }
    if (VEC && me < total - 4 * whole) {  // the last one to three floats
        const int64_t f = 4 * whole + me;
        const int32_t m = float_to_ordered(0.5f * (S[f] + E[f]));
        const int x = (int)(f % 3);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (k == x) {
                v[k] = min(v[k], m);
                v[3 + k] = min(v[3 + k], ~m);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        for (int o = 32; o > 0; o >>= 1) v[k] = min(v[k], __shfl_xor(v[k], o, 64));
        if (__lane_id() == 0) atomicMin(&lb[k], v[k]);
    }
    __syncthreads();
    if (tid < 3) atomicMin(&b[tid], lb[tid]);
    else if (tid < 6) atomicMax(&b[tid], ~lb[tid]);
}

__device__ inline uint32_t spread10(uint32_t v)
{
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x30000FFu;
    v = (v | (v << 8)) & 0x300F00Fu;
    v = (v | (v << 4)) & 0x30C30C3u;
    v = (v | (v << 2)) & 0x9249249u;
    return v;
}

__global__ __launch_bounds__(256) void k_seg_keys(const float *__restrict__ S, const float *__restrict__ E,
                                                  int64_t n, const int32_t *__restrict__ b,
                                                  uint64_t *__restrict__ keys, uint32_t *__restrict__ vals)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t q[3];
    uint32_t oct = 0;
    const row3 s = ld3(S + 3 * i), e = ld3(E + 3 * i);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float lo = ordered_to_float(b[k]), hi = ordered_to_float(b[3 + k]);
        const float m = 0.5f * (s[k] + e[k]);
        const float ext = hi - lo;
        float x = ext > 0.0f ? (m - lo) / ext * 1024.0f : 0.0f;
        x = fminf(fmaxf(x, 0.0f), 1023.0f);
        q[k] = (uint32_t)x;
        oct |= (e[k] < s[k] ? 1u : 0u) << k;
    }
    const uint32_t code = spread10(q[0]) | (spread10(q[1]) << 1) | (spread10(q[2]) << 2);
    keys[i] = ((uint64_t)oct << 30) | code;
    vals[i] = (uint32_t)i;
}

__global__ __launch_bounds__(256) void k_gather_segments(const float *__restrict__ S, const float *__restrict__ E,
                                                         const int32_t *__restrict__ order, int64_t n,
                                                         float *__restrict__ So, float *__restrict__ Eo)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int64_t i = order[k];
    if (i < 0 || i >= n) i = 0;  // every read stays inside S and E
    const row3 s = ld3(S + 3 * i), e = ld3(E + 3 * i);
    st3(So + 3 * k, s.x, s.y, s.z);
    st3(Eo + 3 * k, e.x, e.y, e.z);
}

}  // namespace

hipError_t launch_segment_order(rsi_bvh *h, const float *S, const float *E, int64_t n, int32_t *order,
                                hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipError_t e = hipSuccess;
    if (h->seg_key_cap < n) {
        if (h->seg_keys) (void)hipFree(h->seg_keys);
        h->seg_keys = nullptr;
        h->seg_key_cap = 0;
        if ((e = hipMalloc(reinterpret_cast<void **>(&h->seg_keys), sizeof(uint64_t) * (size_t)n)) != hipSuccess)
            return e;
        h->seg_key_cap = n;
    }
    uint32_t *vals = reinterpret_cast<uint32_t *>(order), *vsrc = nullptr;
    uint64_t *ksrc = nullptr;
    if ((e = sort_source(h->seg_keys, vals, n, kSegKeyBits, h->seg_sort, nullptr, 1, 0, &ksrc, &vsrc)) != hipSuccess)
        return e;
    int32_t *b = h->scalars + kSegBounds;
    hipLaunchKernelGGL(k_seg_bounds_init, dim3(1), dim3(64), 0, s, b);
    int dev = 0, n_cu = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    const bool vec = ((reinterpret_cast<uintptr_t>(S) | reinterpret_cast<uintptr_t>(E)) & 15) == 0;
    int64_t blocks = (3 * n + (vec ? 4 : 1) * kBoundThreads - 1) / ((vec ? 4 : 1) * kBoundThreads);
    if (blocks > n_cu) blocks = n_cu;
    if (vec) hipLaunchKernelGGL(k_seg_bounds<true>, dim3((unsigned)blocks), dim3(kBoundThreads), 0, s, S, E, n, b);
    else hipLaunchKernelGGL(k_seg_bounds<false>, dim3((unsigned)blocks), dim3(kBoundThreads), 0, s, S, E, n, b);
    hipLaunchKernelGGL(k_seg_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, S, E, n, b, ksrc,
                       vsrc);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return radix_sort_pairs(h->seg_keys, vals, n, kSegKeyBits, h->seg_sort, s);
}

hipError_t launch_gather_segments(rsi_bvh *h, const float *S, const float *E, const int32_t *order, int64_t n,
                                  float *So, float *Eo, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    (void)h;
    hipLaunchKernelGGL(k_gather_segments, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, S, E, order, n, So,
                       Eo);
    return hipGetLastError();
}

}  // namespace rsi
