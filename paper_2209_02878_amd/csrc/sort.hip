// sort.hip -- stable radix sort of (uint64 key, uint32 value) pairs (the
// Morton-code sorting step timed in the paper's Table 2, which there ran on
// the host): stable passes on the top 8-bit digits until the groups of equal
// prefixes are small, then one pass that orders each group by counting
// (k_finish; plan_sort says how many passes).  Groups that stay large are
// sorted by a workgroup each, in LDS or device memory; a large table in which a
// sample finds such groups gets passes on its low digits first (k_sample).
//
// One digit pass:
//   k_hist     per-tile digit histogram in LDS -> hist[digit][tile]
//   k_scan     one workgroup per digit turns its row of hist into the count
//              of that digit in earlier tiles, and its sum
//   k_scatter  per tile: stable rank of every element among equal digits
//              via wave64 ballots, reorder the tile in LDS by digit, then
//              write each digit run to its global offset (contiguous runs)
// With at most 16 tiles (inputs up to 32k elements, where the passes are
// latency bound; at 49 tiles a fused pass took 19 us, the three launches 17)
// every scatter workgroup derives its own offsets from the
// raw histograms (no k_scan) and also counts the next pass's digits of the
// elements it writes, per destination tile, so only the first pass needs
// k_hist: one launch per pass.  Three histogram buffers rotate: pass p reads
// H[p % 3], adds into H[(p + 1) % 3] and clears H[(p + 2) % 3] for pass p + 1.
// Tiles are 256 threads x 8 items in striped order (item r of thread x is
// element r*256 + x), which fixes the stable order (r, wave, lane).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rsi_host.h"
#include "rsi_rank.h"

namespace rsi {
namespace {

using rank::kThreads;
using rank::kRadix;
using rank::kWaves;
using rank::lanemask_lt;
using rank::scan256;
constexpr int kItems = 8;                // elements per thread in large sorts
constexpr int kTile = kThreads * kItems;
constexpr int kFusedTiles = 16;  // up to this many tiles each workgroup scans the histograms itself

// Digit of an element for one pass: up to 8 bits of the key, or (for batches)
// of the mesh that the element's value (a triangle index) belongs to.
struct Digit {
    const int64_t *off;  // null: key digits
    int32_t M;
    int shift;
    uint32_t mask = kRadix - 1;
    __device__ inline uint32_t operator()(uint64_t key, uint32_t val) const
    {
        if (off) return ((uint32_t)mesh_of(off, M, (int64_t)val) >> shift) & mask;
        return (uint32_t)(key >> shift) & mask;
    }
};

// GATED, here and in the next two kernels: a pass that only runs when the word
// at `gate` is set; few workgroups then take all the tiles, so that it costs
// little when it is not.
template <int IPT, bool GATED = false>
__global__ __launch_bounds__(kThreads) void k_hist(const uint64_t *__restrict__ keys,
                                                   const uint32_t *__restrict__ vals, int64_t n, Digit dg,
                                                   uint32_t *__restrict__ hist, int ntiles,
                                                   uint32_t *__restrict__ clear, const uint32_t *__restrict__ gate)
{
    if (GATED && *gate == 0) return;
    __shared__ uint32_t h[kRadix];
    const int tid = threadIdx.x;
    int tile = (int)blockIdx.x;
    do {
        // `clear` (may be null): a histogram buffer the next scatter adds into
        if (clear) clear[(int64_t)tid * ntiles + tile] = 0;
        h[tid] = 0;
        __syncthreads();
        const int64_t base = (int64_t)tile * (kThreads * IPT);
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            int64_t i = base + r * kThreads + tid;
            if (i < n) atomicAdd(&h[dg(keys[i], dg.off ? vals[i] : 0u)], 1u);
        }
        __syncthreads();
        hist[(int64_t)tid * ntiles + tile] = h[tid];
        tile += (int)gridDim.x;
    } while (GATED && tile < ntiles);
}

// Exclusive scan of every digit's counts over the tiles, in place, one
// workgroup per digit; total[d] gets the digit's sum (k_scatter turns the
// sums into the digits' offsets).  One launch; a scan of the whole table
// (block sums, their scan, a second sweep) took three, 16 us a pass.
template <bool GATED = false>
__global__ __launch_bounds__(kThreads) void k_scan(uint32_t *__restrict__ hist, int ntiles,
                                                   uint32_t *__restrict__ total, const uint32_t *__restrict__ gate)
{
    if (GATED && *gate == 0) return;
    __shared__ uint32_t ws[kWaves];
    const int tid = threadIdx.x, wave = tid >> 6;
    uint32_t *const row = hist + (int64_t)blockIdx.x * ntiles;
    uint32_t base = 0;
    for (int c0 = 0; c0 < ntiles; c0 += 4 * kThreads) {
        // four consecutive counts per thread
        const int i = c0 + 4 * tid;
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = i + k < ntiles ? row[i + k] : 0u;
        const uint32_t s = v[0] + v[1] + v[2] + v[3];
        uint32_t incl = s;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t u = __shfl_up(incl, off, 64);
            if ((int)__lane_id() >= off) incl += u;
        }
        if (__lane_id() == 63) ws[wave] = incl;
        __syncthreads();
        uint32_t run = base + incl - s;
        for (int w = 0; w < kWaves; ++w) {
            run += w < wave ? ws[w] : 0u;
            base += ws[w];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i + k < ntiles) row[i + k] = run;
            run += v[k];
        }
    }
    if (tid == 0) total[blockIdx.x] = base;
}

// FUSED: `offs` holds the raw per-tile histograms and each workgroup forms
// its own global digit offsets (few tiles: this saves the separate scan
// launch); it then also adds the next pass's digit counts of the elements it
// writes into `hnext` (per destination tile) and clears `hclear`.  They are
// counted in LDS first: a digit of few values (the mesh id of a small batch,
// keys of a cluster) puts a whole table's atomics on a few addresses, which
// take them one at a time (6 meshes, 22,000 triangles: the pass before the
// mesh id's 75 us when lanes that agree added together, @@ now).  Otherwise
// `offs` holds each digit's counts scanned over the tiles, and the digits'
// sums behind them.
template <bool FUSED, int IPT, bool GATED = false>
__global__ __launch_bounds__(kThreads) void k_scatter(const uint64_t *__restrict__ kin,
                                                      const uint32_t *__restrict__ vin,
                                                      uint64_t *__restrict__ kout, uint32_t *__restrict__ vout,
                                                      int64_t n, Digit dg, const uint32_t *__restrict__ offs,
                                                      int ntiles, Digit dnext, uint32_t *__restrict__ hnext,
                                                      uint32_t *__restrict__ hclear,
                                                      const uint32_t *__restrict__ gate)
{
    if (GATED && *gate == 0) return;
    // wcnt[r][w][d]: elements with digit d held by wave w in round r; after
    // the scan, the number of elements with digit d before (r, w) in the tile
    __shared__ uint32_t wcnt[IPT][kWaves][kRadix];
    __shared__ uint32_t run[kRadix];    // the tile's count of each digit
    __shared__ uint32_t start[kRadix];  // exclusive scan of run[]
    __shared__ uint32_t gbase[kRadix];  // global offset of (digit, this tile)
    __shared__ uint64_t skey[(kThreads * IPT)];
    __shared__ uint32_t sval[(kThreads * IPT)];

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    int tile = (int)blockIdx.x;
    do {
        const int64_t base = (int64_t)tile * (kThreads * IPT);

        // all loads first: one memory latency for the whole tile
        uint64_t key[IPT];
        uint32_t val[IPT];
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int64_t i = base + r * kThreads + tid;
            key[r] = i < n ? kin[i] : 0ull;
            val[r] = i < n ? vin[i] : 0u;
        }
        if (FUSED && hclear) hclear[(int64_t)tid * ntiles + tile] = 0;
#pragma unroll
        for (int r = 0; r < IPT; ++r)
#pragma unroll
            for (int w = 0; w < kWaves; ++w) wcnt[r][w][tid] = 0;
        if (FUSED) {
            // digit tid: elements in earlier tiles and in all tiles
            uint32_t before = 0, total = 0;
            for (int b = 0; b < ntiles; ++b) {
                const uint32_t c = offs[(int64_t)tid * ntiles + b];
                before += b < tile ? c : 0u;
                total += c;
            }
            start[tid] = total;
            __syncthreads();
            scan256(start, gbase);
            __syncthreads();
            gbase[tid] += before;
        } else {
            const uint32_t before = offs[(int64_t)tid * ntiles + tile];
            start[tid] = offs[(int64_t)kRadix * ntiles + tid];
            __syncthreads();
            scan256(start, gbase);
            __syncthreads();
            gbase[tid] += before;
        }

        // per round: the lanes of this wave holding the same digit (8 ballots);
        // the lowest of them records the group size
        uint32_t dig[IPT];
        uint32_t below[IPT];
        const uint64_t lt = lanemask_lt();
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const bool valid = base + r * kThreads + tid < n;
            const uint32_t d = valid ? dg(key[r], val[r]) : 0u;
            dig[r] = d;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            below[r] = (uint32_t)__popcll(peers & lt);
            if (valid && below[r] == 0) wcnt[r][wave][d] = (uint32_t)__popcll(peers);
        }
        __syncthreads();
        // digit tid: exclusive prefix over (round, wave) in the tile's stable order
        {
            uint32_t acc = 0;
#pragma unroll
            for (int r = 0; r < IPT; ++r)
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const uint32_t c = wcnt[r][w][tid];
                    wcnt[r][w][tid] = acc;
                    acc += c;
                }
            run[tid] = acc;
        }
        __syncthreads();
        scan256(run, start);
        __syncthreads();

#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            if (base + r * kThreads + tid < n) {
                const uint32_t p = start[dig[r]] + wcnt[r][wave][dig[r]] + below[r];
                skey[p] = key[r];
                sval[p] = val[r];
            }
        }
        __syncthreads();

        const int64_t rem = n - base;
        const int cnt = rem < (kThreads * IPT) ? (int)rem : (kThreads * IPT);
        static_assert(kFusedTiles <= IPT * kWaves, "the next pass's counts fit in wcnt");
        uint32_t *const next = &wcnt[0][0][0];  // the next pass's digits, [digit][tile], as hnext
        if (FUSED && hnext) {
            for (int i = tid; i < ntiles * kRadix; i += kThreads) next[i] = 0;
            __syncthreads();
        }
        for (int p = tid; p < cnt; p += kThreads) {
            const uint64_t k = skey[p];
            const uint32_t v = sval[p];
            const uint32_t d = dg(k, v);
            const int64_t dst = (int64_t)gbase[d] + (p - start[d]);
            kout[dst] = k;
            vout[dst] = v;
            if (FUSED && hnext) atomicAdd(&next[dnext(k, v) * ntiles + dst / (kThreads * IPT)], 1u);
        }
        if (FUSED && hnext) {
            __syncthreads();
            for (int i = tid; i < ntiles * kRadix; i += kThreads)
                if (next[i]) atomicAdd(&hnext[i], next[i]);
        }
        if (GATED) __syncthreads();
        tile += (int)gridDim.x;
    } while (GATED && tile < ntiles);
}

// Groups too large for the window below are sorted by one workgroup with
// stable passes over their low key bits, tile by tile.  Item r of lane l in
// wave w is element (w IPT + r) 64 + l of a tile.

// The digit of `low` low key bits that starts at bit `shift`.
__device__ inline uint32_t low_digit(uint64_t key, int shift, int low)
{
    return (uint32_t)(key >> shift) & (low - shift < 8 ? (1u << (low - shift)) - 1u : kRadix - 1u);
}

struct GroupRank {
    uint32_t wcnt[kWaves][kRadix];  // per wave and digit: first its items, then those of earlier waves
    uint32_t run[kRadix];           // the tile's count of each digit
    uint32_t start[kRadix];         // exclusive scan of run
};

// Places of a tile's items in stable order of their digits.  A wave counts on
// through its rounds, so the counts take 4 KB of LDS whatever IPT (a row for
// every round and wave, as k_scatter's, takes 4 KB a round; a row for a
// quarter of the rounds, a shorter chain of LDS accesses, was no faster).
template <int IPT>
__device__ __forceinline__ void rank_group(const uint32_t (&dig)[IPT], const bool (&valid)[IPT], uint32_t (&pos)[IPT],
                                  GroupRank &g)
{
    const int tid = threadIdx.x, wave = tid >> 6;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) g.wcnt[w][tid] = 0;
    __syncthreads();
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        uint64_t peers = __ballot(valid[r]);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (dig[r] >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t below = (uint32_t)__popcll(peers & lt);
        const uint32_t before = g.wcnt[wave][dig[r]];
        __builtin_amdgcn_wave_barrier();  // (a wave's LDS operations run in order)
        if (valid[r] && below == 0) g.wcnt[wave][dig[r]] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
        pos[r] = before + below;
    }
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = g.wcnt[w][tid];
        g.wcnt[w][tid] = sum;
        sum += c;
    }
    g.run[tid] = sum;
    __syncthreads();
    scan256(g.run, g.start);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; ++r) pos[r] += g.start[dig[r]] + g.wcnt[wave][dig[r]];
}

template <int IPT>
struct GroupWork {
    union {  // keys and values change places one after the other
        uint64_t key[IPT * kThreads];
        uint32_t val[IPT * kThreads];
    };
    GroupRank rank;
};

// A group of at most IPT * kThreads keys, from kin/vin to kout/vout: its
// passes in registers and LDS, over the bits in which its keys differ.  (The
// 4,000 keys of a mesh with one far vertex: 43 us; 90 by the passes in device
// memory.)  Inlined: behind a call the LDS accesses would be flat ones, 71 us.
template <int IPT, int MOST>
__device__ __forceinline__ void sort_group_lds(const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                      uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t b0, int bn,
                                      GroupWork<MOST> &g)
{
    const int tid = threadIdx.x, first = (tid >> 6) * (64 * IPT) + (int)__lane_id();
    uint64_t key[IPT];
    uint32_t val[IPT], dig[IPT], pos[IPT];
    bool valid[IPT];
    const uint64_t key0 = kin[b0];
    uint64_t differ = 0;
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int i = first + 64 * r;
        valid[r] = i < bn;
        key[r] = kin[b0 + (valid[r] ? i : 0)];
        val[r] = vin[b0 + (valid[r] ? i : 0)];
    }
    // (a use right behind each load would wait for them one by one)
#pragma unroll
    for (int r = 0; r < IPT; ++r) differ |= key[r] ^ key0;
    for (int o = 32; o > 0; o >>= 1) differ |= (uint64_t)__shfl_xor((unsigned long long)differ, o, 64);
    if (__lane_id() == 0) g.key[tid >> 6] = differ;
    __syncthreads();
    differ = g.key[0] | g.key[1] | g.key[2] | g.key[3];
    static_assert(kWaves == 4, "the waves' words above");
    __syncthreads();
    const int low = 64 - (differ ? __clzll((long long)differ) : 64);
    for (int shift = differ ? __builtin_ctzll(differ) : 0; shift < low; shift += 8) {
#pragma unroll
        for (int r = 0; r < IPT; ++r) dig[r] = low_digit(key[r], shift, low);
        rank_group<IPT>(dig, valid, pos, g.rank);
#pragma unroll
        for (int r = 0; r < IPT; ++r)
            if (valid[r]) g.key[pos[r]] = key[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; ++r)
            if (valid[r]) key[r] = g.key[first + 64 * r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; ++r)
            if (valid[r]) g.val[pos[r]] = val[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; ++r)
            if (valid[r]) val[r] = g.val[first + 64 * r];
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < IPT; ++r)
        if (valid[r]) {
            kout[b0 + first + 64 * r] = key[r];
            vout[b0 + first + 64 * r] = val[r];
        }
}

// A larger one: the passes over its `low` low key bits in device memory, one
// histogram sweep and one tile-by-tile scatter sweep per pass, alternating
// between the range in kin and in kout (the result ends in kout).
// ITEMS keys per thread and tile.
template <int ITEMS>
__device__ __forceinline__ void sort_group_global(uint64_t *__restrict__ kin, uint32_t *__restrict__ vin,
                                         uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t b0,
                                         int64_t bn, int low, GroupRank &g, uint32_t *gcount, uint32_t *gbase)
{
    const int tid = threadIdx.x, first = (tid >> 6) * (64 * ITEMS) + (int)__lane_id();
    uint64_t *ks = kin + b0, *kd = kout + b0;
    uint32_t *vs = vin + b0, *vd = vout + b0;
    for (int shift = 0; shift < low; shift += 8) {
        gcount[tid] = 0;
        __syncthreads();
        for (int64_t i = tid; i < bn; i += kThreads) atomicAdd(&gcount[low_digit(ks[i], shift, low)], 1u);
        __syncthreads();
        // a digit that every element of the group shares changes no order
        if (gcount[low_digit(ks[0], shift, low)] == (uint32_t)bn) {
            __syncthreads();
            continue;
        }
        scan256(gcount, gbase);
        __syncthreads();
        for (int64_t c0 = first; c0 - first < bn; c0 += kThreads * ITEMS) {
            uint64_t key[ITEMS];
            uint32_t val[ITEMS], dig[ITEMS], pos[ITEMS];
            bool valid[ITEMS];
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) {
                const int64_t i = c0 + 64 * r;
                valid[r] = i < bn;
                key[r] = ks[valid[r] ? i : 0];
                val[r] = vs[valid[r] ? i : 0];
            }
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) dig[r] = low_digit(key[r], shift, low);
            rank_group<ITEMS>(dig, valid, pos, g);
#pragma unroll
            for (int r = 0; r < ITEMS; ++r)
                if (valid[r]) {
                    const int64_t dst = (int64_t)gbase[dig[r]] + (pos[r] - g.start[dig[r]]);
                    kd[dst] = key[r];
                    vd[dst] = val[r];
                }
            __syncthreads();
            gbase[tid] += g.run[tid];
            __syncthreads();
        }
        uint64_t *tk = ks; ks = kd; kd = tk;
        uint32_t *tv = vs; vs = vd; vd = tv;
    }
    if (ks != kout + b0) {  // an even number of passes left the result in kin's range
        for (int64_t i = tid; i < bn; i += kThreads) {
            kout[b0 + i] = ks[i];
            vout[b0 + i] = vs[i];
        }
    }
}

// The last pass of a key sort: kin/vin are in stable order of key >> low
// (within each mesh's range of positions); each group of equal prefixes is
// put in key order into kout/vout.  The passes before it have made the
// groups small (tens of keys), so a key's place is found by counting: its
// group's start plus the keys of the group below it, equal keys by position,
// which is the place a stable sort by the whole key gives it.  A workgroup
// takes TILE consecutive keys, with HALO more on either side in LDS: a group
// of up to HALO keys is then seen whole by every tile it touches.  A larger
// one (visible extent above HALO, which every tile it touches finds alike)
// is left to the workgroup whose tile holds its first key.  (Its passes
// permute the group's range of kin while other tiles may still load it as
// their halo: those only compare its prefixes, which are all the same.)
//
// Counting replaces sorting each top-8-bit bucket in one workgroup, which at
// 499,280 keys took 189 us and at 4M 1,187 us (a 16,000-key bucket streamed
// through one workgroup).
//
// With *sorted set the passes before have put the whole table in order.
//
// The window's keys lie in LDS shifted up by 12 bits (their prefixes, equal
// within a group, may fall off) with their window position below, so keys
// are distinct and one 64-bit compare counts equal keys by position; PACKED
// false (low > 52) compares key and position.  The first keys of the groups
// are one bit each.
template <int TILE, int HALO, bool PACKED>
__global__ __launch_bounds__(kThreads)
    __attribute__((amdgpu_waves_per_eu(TILE == 256 ? 2 : 5))) void k_finish(uint64_t *__restrict__ kin,
                                                                            uint32_t *__restrict__ vin,
                                                                            uint64_t *__restrict__ kout,
                                                                            uint32_t *__restrict__ vout, int64_t n,
                                                                            int low, const int64_t *__restrict__ off,
                                                                            int32_t M,
                                                                            const uint32_t *__restrict__ sorted)
{
    constexpr int kWin = TILE + 2 * HALO;
    static_assert(kWin <= 4096 && kWin % 64 == 0, "window positions take 12 bits, group starts whole words");
    // items per thread of the largest group sorted in LDS: small sorts, of at
    // most two workgroups per CU, have LDS and registers to spare; with 8 in the
    // large ones (128 VGPRs, 96 now) the 64-mesh batch's k_finish took 54 us, 40
    // with 4
    constexpr int kMostItems = TILE == 256 ? 16 : 4;
    constexpr int kMost = TILE / HALO + 1;  // first keys of large groups lie more than HALO keys apart
    __shared__ union {
        struct {
            uint64_t key[kWin];
            uint64_t head[kWin / 64];  // bit j of word w: window position 64 w + j starts a group
            int64_t large[kMost];      // first keys of large groups
            int n_large;
        };
        GroupWork<kMostItems> work;
        struct {
            GroupRank rank;
            uint32_t gcount[kRadix], gbase[kRadix];
        };
    } sh;
    static_assert(sizeof(sh) <= 163840 / (TILE == 256 ? 4 : 6), "four or six workgroups on a CU");
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * TILE;
    if (sorted && *sorted) {
        for (int64_t i = t0 + tid; i < n && i < t0 + TILE; i += kThreads) {
            kout[i] = kin[i];
            vout[i] = vin[i];
        }
        return;
    }
    const int64_t w0 = t0 - HALO > 0 ? t0 - HALO : 0;
    const int nw = (int)((t0 + TILE + HALO < n ? t0 + TILE + HALO : n) - w0);
    if (tid == 0) sh.n_large = 0;
    // all loads first: one memory latency for the whole window
    constexpr int kPer = kWin / kThreads;
    static_assert(kWin % kThreads == 0, "whole rounds");
    uint64_t win[kPer], prev[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int p = r * kThreads + tid;
        win[r] = p < nw ? kin[w0 + p] : 0ull;
        prev[r] = p > 0 && p < nw && __lane_id() == 0 ? kin[w0 + p - 1] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int p = r * kThreads + tid;
        const uint64_t k = win[r];
        uint64_t before = __shfl_up(k, 1, 64);
        if (__lane_id() == 0) before = prev[r];
        // a position past the last key starts a group (of nothing), and so
        // does the window's first
        bool first = p == 0 || p >= nw || (before >> low) != (k >> low);
        if (off && !first) first = off[mesh_of(off, M, w0 + p)] == w0 + p;
        sh.key[p] = PACKED ? (k << 12) | (uint64_t)p : k;
        const uint64_t m = __ballot(first);
        if (__lane_id() == 0) sh.head[p >> 6] = m;
    }
    __syncthreads();
    for (int q = tid; q < TILE; q += kThreads) {
        const int64_t i = t0 + q;
        if (i >= n) break;
        const int me = (int)(i - w0);
        // the group's visible extent [b, e): the last start up to me, the
        // first one after it (or the window's end)
        int w = me >> 6;
        uint64_t m = sh.head[w] & (~0ull >> (63 - (me & 63)));
        while (m == 0) m = sh.head[--w];  // bit 0 of word 0 is set
        const int b = 64 * w + 63 - __clzll((long long)m);
        w = (me + 1) >> 6;
        m = w < kWin / 64 ? sh.head[w] & (~0ull << ((me + 1) & 63)) : 0;
        while (m == 0 && ++w < kWin / 64) m = sh.head[w];
        const int e = m ? 64 * w + __builtin_ctzll(m) : kWin;
        if (e - b > HALO) {
            // (an extent cut by the window starts before the tile)
            if (me == b) sh.large[atomicAdd(&sh.n_large, 1)] = i;
            continue;
        }
        const uint64_t k = sh.key[me];
        int below = 0;
#pragma unroll 4
        for (int j = b; j < e; ++j) {
            const uint64_t kj = sh.key[j];
            below += (PACKED ? kj < k : kj < k || (kj == k && j < me)) ? 1 : 0;
        }
        const int64_t dst = w0 + b + below;
        kout[dst] = PACKED ? kin[i] : k;
        vout[dst] = vin[i];
    }
    __syncthreads();
    const int nl = sh.n_large;
    int64_t first[kMost];
#pragma unroll
    for (int g = 0; g < kMost; ++g) first[g] = g < nl ? sh.large[g] : 0;
    __syncthreads();  // their space is the sorts' now
    for (int g = 0; g < nl; ++g) {
        int64_t b0 = first[0];
#pragma unroll
        for (int k = 1; k < kMost; ++k) b0 = g == k ? first[k] : b0;
        // the group's end: the first later key with another prefix, or its mesh's last
        int64_t lo = b0 + 1, hi = n;
        if (off) hi = off[mesh_of(off, M, b0) + 1];
        const uint64_t pre = kin[b0] >> low;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((kin[mid] >> low) <= pre) lo = mid + 1;
            else hi = mid;
        }
        const int64_t bn = lo - b0;
        if (bn <= 4 * kThreads) {
            sort_group_lds<4, kMostItems>(kin, vin, kout, vout, b0, (int)bn, sh.work);
        } else if (bn > kMostItems * kThreads) {
            sort_group_global<TILE == 256 ? 8 : 4>(kin, vin, kout, vout, b0, bn, low, sh.rank, sh.gcount, sh.gbase);
        } else if constexpr (kMostItems == 16) {
            if (bn <= 8 * kThreads) sort_group_lds<8, kMostItems>(kin, vin, kout, vout, b0, (int)bn, sh.work);
            else sort_group_lds<16, kMostItems>(kin, vin, kout, vout, b0, (int)bn, sh.work);
        }
        __syncthreads();
    }
}

// Whether a table has large groups of equal prefixes: every 64th key (jittered
// within its 64) is counted by a hash of its prefix, and *word set when an
// entry of the counts (a power of two of them, 2^bits) reaches kSampleHits: a
// group of 16,384 keys is met 256 times.  There are two to four entries to a sample (one
// at 2^30 keys), so chance meetings stay far below.
constexpr int kSampleStep = 64;
constexpr uint32_t kSampleHits = 128;

__global__ __launch_bounds__(kThreads) void k_sample_clear(uint32_t *__restrict__ count, int bits,
                                                           uint32_t *__restrict__ word)
{
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i == 0) *word = 0;
    if (i < (1u << bits)) count[i] = 0;
}

__global__ __launch_bounds__(kThreads) void k_sample(const uint64_t *__restrict__ keys,
                                                     const uint32_t *__restrict__ vals, int64_t n, int low,
                                                     const int64_t *__restrict__ off, int32_t M,
                                                     uint32_t *__restrict__ count, int bits,
                                                     uint32_t *__restrict__ word)
{
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t i = t * kSampleStep + (((uint32_t)t * 0x9E3779B1u) >> 26);
    if (i >= n) return;
    uint64_t h = keys[i] >> low;
    if (off) h ^= (uint64_t)mesh_of(off, M, (int64_t)vals[i]) << 40;
    h *= 0x9E3779B97F4A7C15ull;
    h ^= h >> 32;
    const uint32_t at = (uint32_t)((h * 0x9E3779B97F4A7C15ull) >> (64 - bits));
    // lanes that agree add together, a few groups at most: a clustered table
    // puts most of the samples on a few entries
    uint64_t left = __ballot(true);
    uint32_t add = 1;
    for (int k = 0; k < 8 && left; ++k) {
        const int lead = __builtin_ctzll(left);
        const uint64_t m = __ballot(at == (uint32_t)__builtin_amdgcn_readlane((int)at, lead)) & left;
        if ((m >> __lane_id()) & 1) add = (int)__lane_id() == lead ? (uint32_t)__popcll(m) : 0u;
        left &= ~m;
    }
    if (add && atomicAdd(&count[at], add) + add >= kSampleHits) *word = 1;
}

}  // namespace

hipError_t ensure_sort_scratch(SortScratch &sc, int64_t n)
{
    hipError_t e = hipSuccess;
    if (n > sc.cap) {
        if (sc.keys_alt) (void)hipFree(sc.keys_alt);
        if (sc.vals_alt) (void)hipFree(sc.vals_alt);
        sc.keys_alt = nullptr;
        sc.vals_alt = nullptr;
        sc.cap = 0;
        if ((e = hipMalloc(&sc.keys_alt, sizeof(uint64_t) * n)) != hipSuccess) return e;
        if ((e = hipMalloc(&sc.vals_alt, sizeof(uint32_t) * n)) != hipSuccess) return e;
        sc.cap = n;
    }
    const int64_t ntiles = (n + kTile - 1) / kTile;
    // fused path: three rotating histograms; else one table, the digits' sums and k_sample's word
    const int64_t hn = ntiles <= kFusedTiles ? 3 * kFusedTiles * kRadix : (ntiles + 1) * kRadix + 1;
    if (hn > sc.hist_cap) {
        if (sc.hist) (void)hipFree(sc.hist);
        sc.hist = nullptr;
        sc.hist_cap = 0;
        if ((e = hipMalloc(&sc.hist, sizeof(uint32_t) * hn)) != hipSuccess) return e;
        sc.hist_cap = hn;
    }
    return e;
}

void free_sort_scratch(SortScratch &sc)
{
    if (sc.keys_alt) (void)hipFree(sc.keys_alt);
    if (sc.vals_alt) (void)hipFree(sc.vals_alt);
    if (sc.hist) (void)hipFree(sc.hist);
    sc = SortScratch();
}

// The passes of a small sort (at most kFusedTiles tiles of kThreads * IPT):
// H[0] from k_hist (which also clears H[1]), then one scatter per pass.
template <int IPT>
void fused_passes(uint64_t *ka, uint32_t *va, uint64_t *kb, uint32_t *vb, int64_t n, const Digit *passes, int np,
                  SortScratch &sc, hipStream_t s)
{
    const int ntiles = (int)((n + kThreads * IPT - 1) / (kThreads * IPT));
    const int64_t hsz = (int64_t)ntiles * kRadix;
    uint32_t *H[3] = {sc.hist, sc.hist + hsz, sc.hist + 2 * hsz};
    hipLaunchKernelGGL(k_hist<IPT>, dim3(ntiles), dim3(kThreads), 0, s, ka, va, n, passes[0], H[0], ntiles,
                       np > 1 ? H[1] : nullptr, nullptr);
    for (int p = 0; p < np; ++p) {
        const Digit dn = p + 1 < np ? passes[p + 1] : passes[p];
        hipLaunchKernelGGL((k_scatter<true, IPT>), dim3(ntiles), dim3(kThreads), 0, s, ka, va, kb, vb, n, passes[p],
                           H[p % 3], ntiles, dn, p + 1 < np ? H[(p + 1) % 3] : nullptr,
                           p + 2 < np ? H[(p + 2) % 3] : nullptr, nullptr);
        uint64_t *tk = ka; ka = kb; kb = tk;
        uint32_t *tv = va; va = vb; vb = tv;
    }
}

// Above this many keys large groups are looked for, so that no workgroup is
// left alone with one: one far segment or vertex puts nearly every key in a few
// groups.  10M segments with one far are ordered in 1,007 us (4,850 when their
// groups were left to a workgroup each), 4.4M triangles with a far vertex rebuilt
// in 1,152 (9,409); a table without large groups pays for the sample and for
// launches that do not run: 932 -> 953 us for 10M segments, 795 -> 837 for the
// rebuild of 4.4M triangles.  Up to this many keys the bucket sort that came
// before left such groups to one workgroup as well, and took longer: 4M
// segments with one far 2,945 us, 1,950 now.
constexpr int64_t kAloneTotal = int64_t(1) << 22;

// Ahead of the passes on the top digits: sample the table, and when it has
// large groups, stable passes on the `low` low bits, an even number of them, so
// that the pairs are back in ka / va.  With the passes on the digits above
// them they sort the whole key.
void low_passes(uint64_t *ka, uint32_t *va, uint64_t *kb, uint32_t *vb, int64_t n, int low, const int64_t *mesh_off,
                int32_t M, uint32_t *hist, int ntiles, uint32_t *word, hipStream_t s)
{
    int bits = 63 - __builtin_clzll((unsigned long long)(n / 16));  // the counts lie in the histograms' space
    if (bits > 24) bits = 24;
    const int64_t samples = (n + kSampleStep - 1) / kSampleStep;
    hipLaunchKernelGGL(k_sample_clear, dim3((1u << bits) / kThreads), dim3(kThreads), 0, s, hist, bits, word);
    hipLaunchKernelGGL(k_sample, dim3((unsigned)((samples + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, ka, va,
                       n, low, mesh_off, M, hist, bits, word);
    const int np = (low + 15) / 16 * 2, width = (low + np - 1) / np;
    const unsigned grid = (unsigned)(ntiles < 512 ? ntiles : 512);
    for (int p = 0; p < np; ++p) {
        const int shift = p * width, left = low - shift;
        const Digit dg{nullptr, 0, shift, left <= 0 ? 0u : (1u << (left < width ? left : width)) - 1};
        hipLaunchKernelGGL((k_hist<kItems, true>), dim3(grid), dim3(kThreads), 0, s, ka, va, n, dg, hist, ntiles,
                           nullptr, word);
        hipLaunchKernelGGL(k_scan<true>, dim3(kRadix), dim3(kThreads), 0, s, hist, ntiles,
                           hist + (int64_t)ntiles * kRadix, word);
        hipLaunchKernelGGL((k_scatter<false, kItems, true>), dim3(grid), dim3(kThreads), 0, s, ka, va, kb, vb, n, dg,
                           hist, ntiles, dg, nullptr, nullptr, word);
        uint64_t *tk = ka; ka = kb; kb = tk;
        uint32_t *tv = va; va = vb; vb = tv;
    }
}

// The passes of a sort.  Key sorts (first_bit 0): `prefix` stable passes on
// the top 8-bit digits, so that the groups of equal prefixes hold tens of
// keys, then k_finish over the `low` other bits, however many they are.  The
// number of passes goes by n (by the largest mesh in a batch, whose groups lie
// inside a mesh) and the length of the keys alone: none while one group may
// hold every key (k_finish alone), one while 256 groups keep the count loop
// short (kOnePass), two up to kTwoPasses, else three.  Measured, k_finish and a
// pass: 29,768 triangles 18 us after one pass, 5 after two, a pass 10; 499,280
// triangles 45 us after two, 13 after three, a pass 19; 4M segments 189 us
// after two (the densest groups pass 512 keys), 32 after three, a pass 54.
// Rebuilds after one and two passes: sphere of 20,000 triangles 85 us and 81,
// 30,000 95 and 84.  After two and three: terrain of 200,000 triangles 140 and
// 144, 300,000 156 and 156, 500,000 192 and 182, 1M 293 and 238; sphere 139 and
// 143, 159 and 153, 197 and 182, 312 and 248.  Segments spread over a volume
// make smaller groups.  After one and two passes: 19,000 ordered in 36 to 39 us
// and 41, 32,000 in 38 to 53 and 44 (17,000 upright ones on a plane 51 and 41);
// after two and three 400,000 in 82 and 92, 1M on the terrain in 149 and 133
// (400,000 upright ones 141 and 94).  Keys
// of no more bits than that, and passes that start above bit 0 (which leave
// the lower bits unsorted), run as digit passes only.  With mesh_off (M > 1)
// the mesh id's digits follow the key's, so each mesh's elements end up
// contiguous, and k_finish works inside each mesh's range.
struct SortPlan {
    Digit pass[16];
    int np = 0;
    int low = 0;   // key bits left to k_finish (0: none)
    int moves = 0; // times the pairs change buffers
};

constexpr int64_t kOneGroup = 256;
// 63-bit codes of triangles, and keys of at most 40 bits: segments, vertices
constexpr int64_t kOnePass = 16384, kOnePassShort = 20480;
constexpr int64_t kTwoPasses = int64_t(1) << 18, kTwoPassesShort = int64_t(1) << 20;

// `most`: keys of the largest mesh (n without meshes).
static SortPlan plan_sort(int64_t n, int64_t most, int key_bits, int first_bit, const int64_t *mesh_off, int32_t M)
{
    SortPlan p;
    int from = first_bit;
    const bool batch = mesh_off && M > 1;
    if (first_bit == 0) {
        const bool wide = key_bits > 40;
        const int prefix = n <= kOneGroup                            ? 0
                           : n <= (wide ? kOnePass : kOnePassShort)  ? 1
                           : most <= (wide ? kTwoPasses : kTwoPassesShort) ? 2
                                                                     : 3;
        if (8 * prefix < key_bits) p.low = from = key_bits - 8 * prefix;
    }
    for (int b = from; b < key_bits; b += 8) p.pass[p.np++] = Digit{nullptr, 0, b};
    if (batch) {
        p.pass[p.np++] = Digit{mesh_off, M, 0};
        if (M > 256) p.pass[p.np++] = Digit{mesh_off, M, 8};
    }
    p.moves = p.np + (p.low ? 1 : 0);
    return p;
}

hipError_t sort_source(uint64_t *keys, uint32_t *vals, int64_t n, int key_bits, SortScratch &sc,
                       const int64_t *mesh_off, int32_t M, int64_t most, uint64_t **ksrc, uint32_t **vsrc)
{
    *ksrc = keys;
    *vsrc = vals;
    if (n <= 1 || key_bits <= 0) return hipSuccess;
    const hipError_t e = ensure_sort_scratch(sc, n);
    if (e != hipSuccess) return e;
    if (plan_sort(n, mesh_off && M > 1 ? most : n, key_bits, 0, mesh_off, M).moves & 1) {
        *ksrc = sc.keys_alt;
        *vsrc = sc.vals_alt;
    }
    return hipSuccess;
}

hipError_t radix_sort_pairs(uint64_t *keys, uint32_t *vals, int64_t n, int key_bits, SortScratch &sc,
                            hipStream_t s, const int64_t *mesh_off, int32_t M, int64_t most, int first_bit, uint64_t **kres,
                            uint32_t **vres)
{
    if (kres) *kres = keys;
    if (vres) *vres = vals;
    if (n <= 1 || key_bits <= first_bit) return hipSuccess;
    hipError_t e = ensure_sort_scratch(sc, n);
    if (e != hipSuccess) return e;
    const int ntiles = (int)((n + kTile - 1) / kTile);
    const SortPlan p = plan_sort(n, mesh_off && M > 1 ? most : n, key_bits, first_bit, mesh_off, M);
    uint64_t *ka = keys, *kb = sc.keys_alt;
    uint32_t *va = vals, *vb = sc.vals_alt;
    auto swap = [&]() {
        uint64_t *tk = ka; ka = kb; kb = tk;
        uint32_t *tv = va; va = vb; vb = tv;
    };
    // without kres the input is where sort_source said, so that the result
    // ends in keys / vals
    if (!kres && (p.moves & 1)) swap();
    const int64_t *off = mesh_off && M > 1 ? mesh_off : nullptr;
    uint32_t *word = nullptr;
    if (p.low && n > kAloneTotal) {
        word = sc.hist + (int64_t)(ntiles + 1) * kRadix;
        low_passes(ka, va, kb, vb, n, p.low, off, M, sc.hist, ntiles, word, s);
    }
    if (p.np > 0 && ntiles <= kFusedTiles) {
        // (smaller tiles, hence more workgroups, measured slower: each
        // workgroup then scans more histograms and the next-pass counters
        // see more atomic traffic)
        fused_passes<kItems>(ka, va, kb, vb, n, p.pass, p.np, sc, s);
        if (p.np & 1) swap();
    } else {
        for (int q = 0; q < p.np; ++q) {
            const Digit dg = p.pass[q];
            hipLaunchKernelGGL(k_hist<kItems>, dim3(ntiles), dim3(kThreads), 0, s, ka, va, n, dg, sc.hist, ntiles,
                               nullptr, nullptr);
            hipLaunchKernelGGL(k_scan<>, dim3(kRadix), dim3(kThreads), 0, s, sc.hist, ntiles,
                               sc.hist + (int64_t)ntiles * kRadix, nullptr);
            hipLaunchKernelGGL((k_scatter<false, kItems>), dim3(ntiles), dim3(kThreads), 0, s, ka, va, kb, vb, n, dg,
                               sc.hist, ntiles, dg, nullptr, nullptr, nullptr);
            swap();
        }
    }
    if (p.low) {
        auto finish = [&](auto kern, int tile) {
            hipLaunchKernelGGL(kern, dim3((unsigned)((n + tile - 1) / tile)), dim3(kThreads), 0, s, ka, va, kb, vb,
                               n, p.low, off, M, word);
        };
        // small sorts: more workgroups
        if (p.low > 52) finish(k_finish<256, 512, false>, 256);
        else if (n <= 131072) finish(k_finish<256, 512, true>, 256);
        else finish(k_finish<2048, 512, true>, 2048);
        swap();
    }
    if (kres && vres) {  // the caller takes the result where it is
        *kres = ka;
        *vres = va;
    }
    return hipGetLastError();
}

}  // namespace rsi
