// pcr_reorder.hip -- vertex orders of Sec. 4 / Sec. 5: Morton order (a 21-level
// octree traversal = 63-bit Morton code), shuffled Morton order (batches of
// the Morton sequence moved to random places) and the shuffled order.
//
// Pipeline: bounding box -> Morton codes (and the first digit's histogram) ->
// stable LSD radix sort of (key, 32-bit index) with 9-bit digits -> gather.
// The shuffle keys are SplitMix64 outputs, computed where they are needed.
// All work runs on the caller's stream in caller-provided scratch.
#include <type_traits>

#include "pcr_internal.h"

namespace pcr {
namespace {

// Sort passes.  The sort is bound by the bytes that its passes move, so the
// passes are few and narrow: 9-bit digits, keys stored without the digits
// already sorted by (4 bytes once 32 bits or fewer are left), no index read in
// the first pass and no key written in the last.  Large clouds sort by the top
// kTopBits bits of the 63-bit code only and put equal ones in order when they
// are gathered (see k_gather): 104 bytes per point, 168 for the whole code,
// where eight 8-bit passes over whole (key, index) records moved 256.
// Tiles of 512 threads x 16 keys (a 64 KiB staging buffer, two workgroups per
// CU), x 4 for inputs that fill few tiles.
constexpr uint32_t kDigit = 9;
constexpr uint32_t kBins = 1u << kDigit;
constexpr uint32_t kSortWg = kBins;                 // threads per tile, one per digit value
constexpr uint32_t kWaves = kSortWg / 64;
constexpr uint32_t kIptLarge = 16, kIptSmall = 4;   // keys per thread
static_assert(kSortWg * kIptLarge <= 65536, "tile positions are held in 16 bits");
// 100M points in shuffled Morton order 10.2 -> 4.5 ms (5.9 with the whole
// code), 1M in Morton order 0.92 -> 0.16 ms (0.19 with large tiles).
constexpr uint64_t kSmallSort = 3u << 20;           // inputs below: tiles of kIptSmall
constexpr uint32_t kTopBits = 5 * kDigit;
// Inputs from here on: kTopBits (2M points: both 0.22 ms, 4M 0.31 against 0.34,
// 32M 1.9 against 2.3).
constexpr uint64_t kTopSort = 3u << 20;

// Tile of workgroup `block` (a launch has 8 * ceil(ntiles / 8) of them; those
// past the end return ntiles).  Consecutive workgroups run on the 8 XCDs in
// turn: each XCD gets one contiguous eighth of the tiles, so that the partial
// lines at the ends of a digit's runs, which the next tile completes, meet in
// one L2.
__device__ __forceinline__ uint32_t sort_tile(uint32_t block, uint32_t ntiles) {
    const uint32_t per = (ntiles + 7) / 8;
    const uint32_t t = (block & 7u) * per + (block >> 3);
    return (block >> 3) < per && t < ntiles ? t : ntiles;
}

// Of the two sorts of a large cloud, by the top bits and by the whole code, each
// runs only if its word `go` says so (null: always).
__device__ __forceinline__ bool idle(const uint32_t *go) { return go && *go == 0; }

// ---------------------------------------------------------------------------
// Bounding box: floats mapped to unsigned integers whose order is the float
// order, so min and max are integer operations.  Every workgroup stores its own
// box and one workgroup combines them: with one atomic per wavefront and bound
// on six words, the atomics of one word queued at the memory side (about 11 ns
// each, 560 us whatever the number of points).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t ord(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unord(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Each step a thread has kBboxLoads points in flight (consecutive threads on
// consecutive points in each of them).
constexpr uint32_t kBboxLoads = 8;
constexpr uint32_t kBboxBlocks = 1024;  // at most; each leaves 6 words

__device__ __forceinline__ void bbox_add(const u32x4 &p, uint32_t (&lo)[3], uint32_t (&hi)[3]) {
    const uint32_t k[3] = {ord(__uint_as_float(p.x)), ord(__uint_as_float(p.y)), ord(__uint_as_float(p.z))};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = k[a] < lo[a] ? k[a] : lo[a];
        hi[a] = k[a] > hi[a] ? k[a] : hi[a];
    }
}

// Box of the workgroup's threads: out[0..3) minima, out[3..6) maxima.
template <uint32_t WAVES>
__device__ __forceinline__ void bbox_store(uint32_t (&lo)[3], uint32_t (&hi)[3], uint32_t *out) {
    __shared__ uint32_t sh[WAVES][6];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            uint32_t l = __shfl_xor(lo[a], o, 64), h = __shfl_xor(hi[a], o, 64);
            lo[a] = l < lo[a] ? l : lo[a];
            hi[a] = h > hi[a] ? h : hi[a];
        }
    }
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            sh[threadIdx.x >> 6][a] = lo[a];
            sh[threadIdx.x >> 6][3 + a] = hi[a];
        }
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        uint32_t x = sh[0][threadIdx.x];
        for (uint32_t w = 1; w < WAVES; ++w) {
            const uint32_t y = sh[w][threadIdx.x];
            x = (threadIdx.x < 3) == (y < x) ? y : x;
        }
        out[threadIdx.x] = x;
    }
}

__global__ __launch_bounds__(256) void k_bbox(const u32x4 *__restrict__ pts, uint64_t n, uint32_t *__restrict__ part) {
    uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + (kBboxLoads - 1) * stride < n; i += kBboxLoads * stride) {
        u32x4 p[kBboxLoads];
#pragma unroll
        for (uint32_t r = 0; r < kBboxLoads; ++r) p[r] = load_point(pts + i + r * stride);
#pragma unroll
        for (uint32_t r = 0; r < kBboxLoads; ++r) bbox_add(p[r], lo, hi);
    }
    for (; i < n; i += stride) bbox_add(load_point(pts + i), lo, hi);
    bbox_store<4>(lo, hi, part + 6 * blockIdx.x);
}

// ---------------------------------------------------------------------------
// Morton codes: cell = min(trunc(((v - lo) / size) * 2^21), 2^21 - 1) over the
// cube of edge `size` (the longest extent), interleaved x, y, z from bit 0.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t spread3(uint32_t v) {
    uint64_t x = v & 0x1FFFFFu;
    x = (x | (x << 32)) & 0x1F00000000FFFFull;
    x = (x | (x << 16)) & 0x1F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ __forceinline__ uint32_t cell21(float v, float lo, float size) {
    if (size == 0.0f) return 0u;
    float t = ((v - lo) / size) * 2097152.0f;
    uint32_t q = (uint32_t)t;
    return q > 2097151u ? 2097151u : q;
}

// Edge and corner of the cube, from the bounding box.
struct Cube {
    float lo[3], size;
    __device__ __forceinline__ explicit Cube(const uint32_t *__restrict__ bb) {
        float l0 = unord(bb[0]), l1 = unord(bb[1]), l2 = unord(bb[2]);
        float sx = unord(bb[3]) - l0, sy = unord(bb[4]) - l1, sz = unord(bb[5]) - l2;
        size = sx;
        if (sy > size) size = sy;
        if (sz > size) size = sz;
        lo[0] = l0;
        lo[1] = l1;
        lo[2] = l2;
    }
    __device__ __forceinline__ uint64_t code(const u32x4 &p) const {
        uint32_t qx = cell21(__uint_as_float(p.x), lo[0], size);
        uint32_t qy = cell21(__uint_as_float(p.y), lo[1], size);
        uint32_t qz = cell21(__uint_as_float(p.z), lo[2], size);
        return spread3(qx) | (spread3(qy) << 1) | (spread3(qz) << 2);
    }
};

// Words after the box: whether the sort by the whole code runs (set again by
// k_gather where it cannot settle a run), and the one by the top bits.
constexpr uint32_t kWhole = 8, kTop = 9;

// One workgroup: the box of `count` boxes and, for clouds that may be sorted by
// the top bits (may_top), which sort runs: points that crowd into few cells of
// the top bits (a cloud with a far outlier, copies) would make long runs of
// equal ones.  Of kSample points taken evenly over the input, a cell shared by m
// of n points on average repeats kSample^2 / 2 * m / n times; the whole code is
// sorted by from about 32 points a cell on.
constexpr uint32_t kSample = 4 * kBboxBlocks, kSampleSlots = 2 * kSample;

__global__ __launch_bounds__(kBboxBlocks) void k_bbox_join(const uint32_t *__restrict__ part, uint32_t count,
                                                           const u32x4 *__restrict__ pts, uint64_t n, bool may_top,
                                                           uint32_t *__restrict__ bb) {
    __shared__ uint32_t box[6];
    __shared__ uint32_t seen[kSampleSlots];
    __shared__ uint32_t repeats;
    uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
    if (threadIdx.x < count) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = part[6 * threadIdx.x + a];
            hi[a] = part[6 * threadIdx.x + 3 + a];
        }
    }
    bbox_store<kBboxBlocks / 64>(lo, hi, box);
    for (uint32_t k = threadIdx.x; k < kSampleSlots; k += kBboxBlocks) seen[k] = 0xFFFFFFFFu;
    if (threadIdx.x == 0) repeats = 0;
    __syncthreads();
    if (threadIdx.x < 6) bb[threadIdx.x] = box[threadIdx.x];
    if (may_top) {
        const Cube cube(box);
#pragma unroll
        for (uint32_t r = 0; r < kSample / kBboxBlocks; ++r) {
            const uint64_t i = (uint64_t)(r * kBboxBlocks + threadIdx.x) * n / kSample;
            const uint64_t c = cube.code(load_point(pts + i)) >> (63 - kTopBits);
            uint32_t tag = (uint32_t)(c * 0x9E3779B97F4A7C15ull >> 32);
            if (tag == 0xFFFFFFFFu) tag = 0;
            // The table is at most half full: the search ends.
            for (uint32_t h = tag;; ++h) {
                const uint32_t old = atomicCAS(&seen[h & (kSampleSlots - 1)], 0xFFFFFFFFu, tag);
                if (old == 0xFFFFFFFFu) break;
                if (old == tag) {
                    atomicAdd(&repeats, 1u);
                    break;
                }
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const uint64_t most = (uint64_t)kSample * kSample * 16 / n;
        const bool top = may_top && repeats <= (most < 8 ? 8 : most);
        bb[kTop] = top;
        bb[kWhole] = !top;
    }
}

// SplitMix64 (Steele, Lea, Flood 2014): output k of the stream seeded with
// `seed` is the mix of seed + (k + 1) * golden gamma.
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t k) {
    uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Random orders sort by the top kRandomBits bits of the 64-bit SplitMix64 keys
// (four passes instead of eight) and put the few keys that agree in those bits
// in order afterwards (settled()).
constexpr uint32_t kRandomBits = 4 * kDigit;
__device__ __forceinline__ uint64_t random_top(uint64_t seed, uint64_t k) {
    return splitmix64(seed, k) >> (64 - kRandomBits);
}

// Final position of entry j of `v` (indices sorted stably by random_top): its
// rank by the whole key among the neighbours that share its top bits.  The
// whole keys of different indices differ (the mix is a bijection), so the
// ranks are distinct.  A run of equal top bits is one or two entries long but
// for seeds made to collide; the scan is right for any length.
__device__ __forceinline__ uint64_t settled(const uint32_t *__restrict__ v, uint64_t n, uint64_t seed, uint64_t j) {
    const uint64_t key = splitmix64(seed, v[j]), top = key >> (64 - kRandomBits);
    uint64_t pos = j;
    for (uint64_t i = j; i > 0; --i) {
        const uint64_t o = splitmix64(seed, v[i - 1]);
        if (o >> (64 - kRandomBits) != top) break;
        pos -= o > key;
    }
    for (uint64_t i = j + 1; i < n; ++i) {
        const uint64_t o = splitmix64(seed, v[i]);
        if (o >> (64 - kRandomBits) != top) break;
        pos += o < key;
    }
    return pos;
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort pass.  A tile is kSortTile keys; wave w of the tile
// owns keys [w * 64 * kSortIpt, (w + 1) * 64 * kSortIpt) of it and visits them
// in kSortIpt rounds of 64 consecutive keys, so (wave, round, lane) order is
// the tile order.  The digit of a pass is the low kDigit bits of the stored
// key; a pass stores the key without them.
// ---------------------------------------------------------------------------

// Adds the wavefront's digits to the workgroup's counters.  A wavefront of one
// digit (the high digits of points in an order) adds once: 64 adds to one LDS
// word are taken one after another.
__device__ __forceinline__ void count_digit(uint32_t *cnt, uint32_t d, bool live) {
    const uint64_t act = __ballot(live);
    if (act == 0) return;
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, (uint32_t)__builtin_ctzll(act));
    if ((act & ~__ballot(d == d0)) == 0) {
        if (__lane_id() == 0) atomicAdd(&cnt[d0], (uint32_t)__popcll(act));
    } else if (live) {
        atomicAdd(&cnt[d], 1u);
    }
}

// hist[d * stride + tile] = number of keys of the tile with digit d.  `stride`
// (the tile count rounded up) keeps the rows 64-byte aligned for k_sort_scan.
__device__ __forceinline__ void store_hist(const uint32_t *cnt, uint32_t stride, uint32_t tile,
                                           uint32_t *__restrict__ hist) {
    __syncthreads();
    hist[(uint64_t)threadIdx.x * stride + tile] = cnt[threadIdx.x];
}

// Morton codes of a tile's points without their low `drop` bits, with the
// histogram of the first digit.
template <uint32_t IPT>
__global__ __launch_bounds__(kSortWg) void k_morton(const u32x4 *__restrict__ pts, uint64_t n,
                                                    const uint32_t *__restrict__ bb, uint32_t drop, uint32_t ntiles,
                                                    uint32_t stride, uint64_t *__restrict__ keys,
                                                    uint32_t *__restrict__ hist, const uint32_t *__restrict__ go) {
    __shared__ uint32_t cnt[kBins];
    const uint32_t tile = sort_tile(blockIdx.x, ntiles);
    if (tile >= ntiles || idle(go)) return;
    const Cube cube(bb);
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)tile * (kSortWg * IPT);
    constexpr uint32_t kStep = IPT < 8 ? IPT : 8;  // points in flight per thread
    for (uint32_t r0 = 0; r0 < IPT; r0 += kStep) {
        u32x4 p[kStep];
#pragma unroll
        for (uint32_t r = 0; r < kStep; ++r) {
            const uint64_t i = base + (r0 + r) * kSortWg + threadIdx.x;
            p[r] = load_point(pts + (i < n ? i : n - 1));
        }
#pragma unroll
        for (uint32_t r = 0; r < kStep; ++r) {
            const uint64_t i = base + (r0 + r) * kSortWg + threadIdx.x;
            const uint64_t k = cube.code(p[r]) >> drop;
            if (i < n) keys[i] = k;
            count_digit(cnt, (uint32_t)k & (kBins - 1), i < n);
        }
    }
    store_hist(cnt, stride, tile, hist);
}

// Key sources of a pass: stored keys, or the top bits of the random keys.
template <typename K>
struct StoredKeys {
    using Key = K;
    const K *keys;
    __device__ __forceinline__ K at(uint64_t i) const { return keys[i]; }
};
struct RandomKeys {
    using Key = uint64_t;
    uint64_t seed;
    __device__ __forceinline__ uint64_t at(uint64_t i) const { return random_top(seed, i); }
};

template <class Src, uint32_t IPT>
__global__ __launch_bounds__(kSortWg) void k_sort_hist(Src src, uint64_t n, uint32_t ntiles, uint32_t stride,
                                                       uint32_t *__restrict__ hist, const uint32_t *__restrict__ go) {
    __shared__ uint32_t cnt[kBins];
    const uint32_t tile = sort_tile(blockIdx.x, ntiles);
    if (tile >= ntiles || idle(go)) return;
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)tile * (kSortWg * IPT);
    uint32_t d[IPT];  // all loads issued before the first use
#pragma unroll
    for (uint32_t r = 0; r < IPT; ++r) {
        const uint64_t i = base + r * kSortWg + threadIdx.x;
        d[r] = (uint32_t)src.at(i < n ? i : n - 1) & (kBins - 1);
    }
#pragma unroll
    for (uint32_t r = 0; r < IPT; ++r) count_digit(cnt, d[r], base + r * kSortWg + threadIdx.x < n);
    store_hist(cnt, stride, tile, hist);
}

// Inclusive scan across the wavefront.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
    const uint32_t lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(x, o, 64);
        if (lane >= (uint32_t)o) x += y;
    }
    return x;
}

// One workgroup per digit: exclusive scan of the digit's tile counts in place,
// their sum to total[digit].
constexpr uint32_t kScanWg = 256, kScanPer = 4;
__global__ __launch_bounds__(kScanWg) void k_sort_scan(uint32_t *__restrict__ hist, uint32_t ntiles, uint32_t stride,
                                                       uint32_t *__restrict__ total, const uint32_t *__restrict__ go) {
    __shared__ uint32_t sh[2][kScanWg / 64];
    if (idle(go)) return;
    uint32_t *row = hist + (uint64_t)blockIdx.x * stride;
    const uint32_t lane = __lane_id(), wave = threadIdx.x / 64;
    uint32_t carry = 0, par = 0;
    for (uint32_t base = 0; base < ntiles; base += kScanWg * kScanPer, par ^= 1u) {
        const uint32_t i = base + threadIdx.x * kScanPer;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (i < stride) v = *(const u32x4 *)(row + i);  // words past ntiles hold anything: dropped below
        const uint32_t a = i < ntiles ? v.x : 0u, b = i + 1 < ntiles ? v.y : 0u, c = i + 2 < ntiles ? v.z : 0u,
                       d = i + 3 < ntiles ? v.w : 0u;
        const uint32_t s = a + b + c + d, x = wave_scan(s);
        if (lane == 63) sh[par][wave] = x;
        __syncthreads();  // the other half of sh is written by the next step only
        uint32_t before = carry;
#pragma unroll
        for (uint32_t w = 0; w < kScanWg / 64; ++w) {
            const uint32_t t = sh[par][w];
            if (w < wave) before += t;
            carry += t;
        }
        before += x - s;
        if (i < stride) *(u32x4 *)(row + i) = u32x4{before, before + a, before + a + b, before + a + b + c};
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// Lanes of the wavefront whose digit equals this lane's digit.
__device__ __forceinline__ uint64_t peers(uint32_t d) {
    uint32_t lo = ~0u, hi = ~0u;
#pragma unroll
    for (uint32_t b = 0; b < kDigit; ++b) {
        const uint64_t vb = __ballot((d >> b) & 1u);
        const uint32_t own = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // the bit in every position
        lo &= ~((uint32_t)vb ^ own);
        hi &= ~((uint32_t)(vb >> 32) ^ own);
    }
    return (uint64_t)hi << 32 | lo;
}

// Stable scatter of one pass.  off = tile counts scanned per digit, total =
// keys per digit.  The tile is first put in digit order in LDS (stably: within
// a digit, tile order), then stored from there, so that consecutive lanes store
// consecutive addresses of one digit's run; keys and indices go through the
// same LDS buffer one after the other.  KOut = void: the last pass, no keys are
// stored.  FIRST: the index of entry i is i, and vin is not read.  Entries past
// the end of the input count as keys of all ones: they come last in the last
// tile, hence last in its digit order, and are not stored.
template <class Src, typename KOut, bool FIRST, uint32_t IPT>
__global__ __launch_bounds__(kSortWg) void k_sort_scatter(Src src, const uint32_t *__restrict__ vin, uint64_t n,
                                                          uint32_t ntiles, uint32_t stride,
                                                          const uint32_t *__restrict__ off,
                                                          const uint32_t *__restrict__ total,
                                                          KOut *__restrict__ kout, uint32_t *__restrict__ vout,
                                                          const uint32_t *__restrict__ go) {
    constexpr uint32_t kSortIpt = IPT, kSortTile = kSortWg * IPT;
    using K = typename Src::Key;
    __shared__ uint16_t wcnt[kWaves][kBins];
    __shared__ uint32_t goff[kBins];
    __shared__ uint32_t scan_sh[2][kWaves];
    __shared__ K stage[kSortTile];
    const uint32_t tile = sort_tile(blockIdx.x, ntiles);
    if (tile >= ntiles || idle(go)) return;
    const uint32_t wave = threadIdx.x / 64, lane = __lane_id();
    const uint64_t tile0 = (uint64_t)tile * kSortTile;
    const uint32_t cnt = (uint32_t)(n - tile0 < kSortTile ? n - tile0 : kSortTile);
    const uint32_t mine = wave * (64 * kSortIpt) + lane;  // first entry of this thread, then steps of 64
    K k[kSortIpt];
    uint32_t v[kSortIpt];
#pragma unroll
    for (uint32_t r = 0; r < kSortIpt; ++r) {
        const uint32_t i = mine + r * 64;
        k[r] = src.at(tile0 + (i < cnt ? i : cnt - 1));
        v[r] = FIRST ? (uint32_t)tile0 + i : vin[tile0 + (i < cnt ? i : cnt - 1)];
    }
    const uint32_t before_tile = off[(uint64_t)threadIdx.x * stride + tile], in_digit = total[threadIdx.x];
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) wcnt[w][threadIdx.x] = 0;
    __syncthreads();
    const uint64_t below = ~(~0ull << lane);
    uint32_t rank[kSortIpt];
#pragma unroll
    for (uint32_t r = 0; r < kSortIpt; ++r) {
        if (mine + r * 64 >= cnt) k[r] = (K)~(K)0;
        const uint32_t d = (uint32_t)k[r] & (kBins - 1);
        const uint64_t pm = peers(d);
        const uint32_t before = (uint32_t)__popcll(pm & below);
        const uint32_t prior = wcnt[wave][d];
        rank[r] = prior + before;
        // The lowest lane of each digit group publishes the new count after
        // every lane of the group has read the old one: LDS operations of one
        // wave complete in order, and the wave barriers keep the compiler
        // from moving the read and the write across each other or across
        // rounds.
        __builtin_amdgcn_wave_barrier();
        if (before == 0) wcnt[wave][d] = (uint16_t)(prior + (uint32_t)__popcll(pm));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // Thread t = digit t: prefix of its count over the waves (wave order is
    // tile order), the start of its run in the digit-ordered tile, and the
    // start of the digit in the output (both by one scan over the threads).
    uint32_t run = 0;
    uint32_t c[kWaves];
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
        c[w] = run;
        run += wcnt[w][threadIdx.x];
    }
    const uint32_t xr = wave_scan(run), xd = wave_scan(in_digit);
    if (lane == 63) {
        scan_sh[0][wave] = xr;
        scan_sh[1][wave] = xd;
    }
    __syncthreads();
    uint32_t start = xr - run, first = xd - in_digit;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
        if (w < wave) {
            start += scan_sh[0][w];
            first += scan_sh[1][w];
        }
    }
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) wcnt[w][threadIdx.x] = (uint16_t)(start + c[w]);
    goff[threadIdx.x] = first + before_tile - start;  // entry j of the ordered tile goes to goff + j
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kSortIpt; ++r) {
        const uint32_t d = (uint32_t)k[r] & (kBins - 1);
        rank[r] += wcnt[wave][d];
        stage[rank[r]] = k[r];
    }
    __syncthreads();
    uint32_t pos[kSortIpt];
#pragma unroll
    for (uint32_t r = 0; r < kSortIpt; ++r) {
        const uint32_t j = threadIdx.x + r * kSortWg;
        const K key = stage[j];
        pos[r] = goff[(uint32_t)key & (kBins - 1)] + j;
        if (j >= cnt || pos[r] >= n) pos[r] = 0xFFFFFFFFu;  // the latter never for a consistent histogram
        if constexpr (!std::is_void<KOut>::value)
            if (pos[r] != 0xFFFFFFFFu) kout[pos[r]] = (KOut)(key >> kDigit);
    }
    __syncthreads();
    uint32_t *vstage = (uint32_t *)stage;
#pragma unroll
    for (uint32_t r = 0; r < kSortIpt; ++r) vstage[rank[r]] = v[r];
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kSortIpt; ++r)
        if (pos[r] != 0xFFFFFFFFu) vout[pos[r]] = vstage[threadIdx.x + r * kSortWg];
}

// ---------------------------------------------------------------------------
// Gathers
// ---------------------------------------------------------------------------
// Shuffled order: perm holds the random order by the top key bits (settled()).
__global__ __launch_bounds__(256) void k_gather_random(const u32x4 *__restrict__ in, const uint32_t *__restrict__ perm,
                                                       uint64_t n, uint64_t seed, u32x4 *__restrict__ out,
                                                       uint32_t *__restrict__ perm_out) {
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += stride) {
        uint32_t s = perm[j];
        if (s >= n) continue;  // never taken for a permutation
        const uint64_t to = settled(perm, n, seed, j);
        if (to >= n) continue;  // never taken
        out[to] = in[s];
        if (perm_out) perm_out[to] = s;
    }
}

// Rank (position in the shuffled batch order) of every batch: rank[b] = the
// settled position of b in `order`.
__global__ __launch_bounds__(256) void k_batch_rank(const uint32_t *__restrict__ order, uint64_t nb, uint64_t seed,
                                                    uint32_t *__restrict__ rank) {
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < nb; r += stride) {
        const uint32_t b = order[r];
        if (b < nb) rank[b] = (uint32_t)settled(order, nb, seed, r);  // always taken for a permutation
    }
}

// Where Morton position j goes: itself, or (rank != null) its place after the
// batches were shuffled: batch b goes to rank r = rank[b], batches before the
// partial last one start at r * batch and those after it `batch - len_last`
// earlier.
struct Places {
    const uint32_t *rank;
    uint32_t batch;
    uint64_t nb, len_last;
    __device__ __forceinline__ uint64_t of(uint32_t j) const {
        if (!rank) return j;
        const uint32_t b = j / batch;
        const uint64_t r = rank[b];
        return r * batch + (j - b * batch) - (r > rank[nb - 1] ? batch - len_last : 0);
    }
};

// Points in Morton order (and shuffled by batches) from their permutation.
// Workgroups take kGatherTile consecutive positions, each XCD a contiguous
// eighth of them, so that neighbouring points of the source share its L2.
// TOP: perm is the order by the top kTopBits bits of the codes, stably; the
// place of an entry among those that share its top bits is found from the whole
// codes, which are computed again from the points that are gathered anyway (so
// the sort has two passes less).  An entry with more than kRunLimit others of its
// top bits on one side (a run of more than kRunLimit entries inside a tile, of
// more than kRunLimit + 1 across tiles) sets bb[kWhole]: the sort by the whole code
// then writes the whole output again, and the workgroups that find the word set
// leave.
constexpr uint32_t kGatherPer = 4, kGatherTile = 256 * kGatherPer;
constexpr uint32_t kRunLimit = 64;

template <bool TOP>
__global__ __launch_bounds__(256) void k_gather(const u32x4 *__restrict__ in, const uint32_t *__restrict__ perm,
                                                uint64_t n, uint32_t ntiles, uint32_t *__restrict__ bb, Places places,
                                                u32x4 *__restrict__ out, uint32_t *__restrict__ perm_out,
                                                const uint32_t *__restrict__ go) {
    __shared__ uint64_t code[TOP ? kGatherTile : 1];
    __shared__ uint32_t given_up;
    const uint32_t tile = sort_tile(blockIdx.x, ntiles);
    if (tile >= ntiles || idle(go)) return;
    if constexpr (TOP) {
        // Other workgroups set the word meanwhile: one thread reads it, so that
        // the whole workgroup leaves or stays for the barriers below.
        if (threadIdx.x == 0)
            given_up = __hip_atomic_load(bb + kWhole, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (given_up) return;
    }
    const uint64_t base = (uint64_t)tile * kGatherTile;
    const uint32_t cnt = (uint32_t)(n - base < kGatherTile ? n - base : kGatherTile);
    uint32_t src[kGatherPer];
    u32x4 p[kGatherPer];
#pragma unroll
    for (uint32_t r = 0; r < kGatherPer; ++r) {
        const uint32_t j = r * 256 + threadIdx.x;
        const uint32_t v = perm[base + (j < cnt ? j : cnt - 1)];
        src[r] = v < n ? v : 0u;  // always v for a permutation
    }
#pragma unroll
    for (uint32_t r = 0; r < kGatherPer; ++r) p[r] = in[src[r]];
    if constexpr (TOP) {
        const Cube cube(bb);
        constexpr uint32_t kLow = 63 - kTopBits;
#pragma unroll
        for (uint32_t r = 0; r < kGatherPer; ++r) code[r * 256 + threadIdx.x] = cube.code(p[r]);
        __syncthreads();
        bool crowd = false;
#pragma unroll
        for (uint32_t r = 0; r < kGatherPer; ++r) {
            const uint32_t j = r * 256 + threadIdx.x;
            crowd |= j + kRunLimit < cnt && ((code[j] ^ code[j + kRunLimit]) >> kLow) == 0;
        }
        if (__syncthreads_or(crowd)) {
            if (threadIdx.x == 0) bb[kWhole] = 1;
            return;
        }
        // Code of Morton entry i, from the tile or, rarely, past its ends.
        auto code_at = [&](uint64_t i) {
            if (i >= base && i < base + cnt) return code[i - base];
            const uint32_t v = perm[i];
            return cube.code(in[v < n ? v : 0u]);
        };
#pragma unroll
        for (uint32_t r = 0; r < kGatherPer; ++r) {
            const uint32_t j = r * 256 + threadIdx.x;
            if (j >= cnt) continue;
            const uint64_t at = base + j, mine = code[j];
            uint64_t to = at;
            uint32_t left = 0, right = 0;
            for (uint64_t i = at; i > 0 && left <= kRunLimit; --i, ++left) {
                const uint64_t o = code_at(i - 1);
                if ((o ^ mine) >> kLow) break;
                to -= o > mine;
            }
            for (uint64_t i = at + 1; i < n && right <= kRunLimit; ++i, ++right) {
                const uint64_t o = code_at(i);
                if ((o ^ mine) >> kLow) break;
                to += o < mine;
            }
            if (left > kRunLimit || right > kRunLimit) {
                bb[kWhole] = 1;
                continue;
            }
            const uint64_t q = places.of((uint32_t)to);
            if (q >= n) continue;  // never taken
            out[q] = p[r];
            if (perm_out) perm_out[q] = src[r];
        }
    } else {
#pragma unroll
        for (uint32_t r = 0; r < kGatherPer; ++r) {
            const uint32_t j = r * 256 + threadIdx.x;
            if (j >= cnt) continue;
            const uint64_t q = places.of((uint32_t)(base + j));
            if (q >= n) continue;  // never taken for permutations
            out[q] = p[r];
            if (perm_out) perm_out[q] = src[r];
        }
    }
}

// ---------------------------------------------------------------------------
// Host
// ---------------------------------------------------------------------------
inline size_t a256(size_t b) { return (b + 255) & ~(size_t)255; }

struct SortBufs {
    uint64_t *k0, *k1;
    uint32_t *v0, *v1;
    uint32_t *hist, *total;
    uint32_t ipt, ntiles, stride;
};

// Carves the sort's buffers for n keys out of the memory at p; returns the end.
uintptr_t carve_sort(uintptr_t p, uint64_t n, SortBufs &sb) {
    sb.ipt = n < kSmallSort ? kIptSmall : kIptLarge;
    sb.ntiles = (uint32_t)((n + kSortWg * sb.ipt - 1) / (kSortWg * sb.ipt));
    sb.stride = (sb.ntiles + 15) / 16 * 16;
    sb.k0 = (uint64_t *)p; p += a256(8 * n);
    sb.k1 = (uint64_t *)p; p += a256(8 * n);
    sb.v0 = (uint32_t *)p; p += a256(4 * n);
    sb.v1 = (uint32_t *)p; p += a256(4 * n);
    // The room for the histogram never shrinks with n (at kSmallSort the tiles
    // become four times as large): scratch for a cloud serves every smaller one.
    constexpr uint32_t kSmallTiles = (uint32_t)(kSmallSort / (kSortWg * kIptSmall));
    const uint32_t room = n < kSmallSort || sb.stride > kSmallTiles ? sb.stride : kSmallTiles;
    sb.hist = (uint32_t *)p; p += a256((size_t)4 * kBins * room);
    sb.total = (uint32_t *)p; p += a256(4 * kBins);
    return p;
}

size_t sort_bytes(uint64_t n) {
    SortBufs sb;
    return carve_sort(0, n, sb);
}
// The boxes of k_bbox go to the histogram's place, which is not in use yet.
static_assert(6 * kBboxBlocks <= kBins * 16, "the histogram of one tile holds the boxes");

uint32_t grid_for(uint64_t n, uint32_t cap = 65536) {
    uint64_t g = (n + 255) / 256;
    return (uint32_t)(g < 1 ? 1 : (g > cap ? cap : g));
}

// Workgroups of a kernel that takes one tile each (see sort_tile).
inline uint32_t tile_grid(const SortBufs &sb) { return (sb.ntiles + 7) / 8 * 8; }

// One pass: keys from src and indices from vin to kout and vout.  The
// histogram of src's digit is taken first unless it is in sb.hist already.
template <bool FIRST, class Src, typename KOut, uint32_t IPT>
int sort_pass_ipt(const SortBufs &sb, Src src, const uint32_t *vin, uint64_t n, KOut *kout, uint32_t *vout,
                  bool have_hist, const uint32_t *go, hipStream_t s) {
    const dim3 g(tile_grid(sb)), wg(kSortWg);
    if (!have_hist)
        hipLaunchKernelGGL((k_sort_hist<Src, IPT>), g, wg, 0, s, src, n, sb.ntiles, sb.stride, sb.hist, go);
    hipLaunchKernelGGL(k_sort_scan, dim3(kBins), dim3(kScanWg), 0, s, sb.hist, sb.ntiles, sb.stride, sb.total, go);
    hipLaunchKernelGGL((k_sort_scatter<Src, KOut, FIRST, IPT>), g, wg, 0, s, src, vin, n, sb.ntiles, sb.stride,
                       sb.hist, sb.total, kout, vout, go);
    PCR_LAUNCHED();
    return PCR_OK;
}

template <bool FIRST, class Src, typename KOut>
int sort_pass(const SortBufs &sb, Src src, const uint32_t *vin, uint64_t n, KOut *kout, uint32_t *vout, bool have_hist,
              const uint32_t *go, hipStream_t s) {
    if (sb.ipt == kIptSmall)
        return sort_pass_ipt<FIRST, Src, KOut, kIptSmall>(sb, src, vin, n, kout, vout, have_hist, go, s);
    return sort_pass_ipt<FIRST, Src, KOut, kIptLarge>(sb, src, vin, n, kout, vout, have_hist, go, s);
}

using S64 = StoredKeys<uint64_t>;
using S32 = StoredKeys<uint32_t>;

// Codes of the points (without their low `drop` bits) and their stable order,
// which ends in sb.v1.
int sort_morton(const SortBufs &sb, const u32x4 *pts, uint64_t n, const uint32_t *bb, uint32_t drop,
                const uint32_t *go, hipStream_t s) {
    const dim3 g(tile_grid(sb)), wg(kSortWg);
    if (sb.ipt == kIptSmall)
        hipLaunchKernelGGL(k_morton<kIptSmall>, g, wg, 0, s, pts, n, bb, drop, sb.ntiles, sb.stride, sb.k0, sb.hist, go);
    else
        hipLaunchKernelGGL(k_morton<kIptLarge>, g, wg, 0, s, pts, n, bb, drop, sb.ntiles, sb.stride, sb.k0, sb.hist, go);
    PCR_LAUNCHED();
    uint32_t *h0 = (uint32_t *)sb.k0, *h1 = (uint32_t *)sb.k1, *none = nullptr;
    int rc;
    if (drop == 0) {
        rc = sort_pass<true>(sb, S64{sb.k0}, none, n, sb.k1, sb.v1, true, go, s);                  // 54 bits left
        if (!rc) rc = sort_pass<false>(sb, S64{sb.k1}, sb.v1, n, sb.k0, sb.v0, false, go, s);     // 45
        if (!rc) rc = sort_pass<false>(sb, S64{sb.k0}, sb.v0, n, sb.k1, sb.v1, false, go, s);     // 36
    } else {
        rc = sort_pass<true>(sb, S64{sb.k0}, none, n, sb.k1, sb.v1, true, go, s);                  // 36 of 45
    }
    if (!rc) rc = sort_pass<false>(sb, S64{sb.k1}, sb.v1, n, h0, sb.v0, false, go, s);            // 27
    if (!rc) rc = sort_pass<false>(sb, S32{h0}, sb.v0, n, h1, sb.v1, false, go, s);               // 18
    if (!rc) rc = sort_pass<false>(sb, S32{h1}, sb.v1, n, h0, sb.v0, false, go, s);               // 9
    if (!rc) rc = sort_pass<false>(sb, S32{h0}, sb.v0, n, (void *)nullptr, sb.v1, false, go, s);
    return rc;
}

// Sorts the indices [0, n) by the top bits of their random keys (stably, into
// sb.v1); settled() gives an entry's place by the whole key.
int sort_random(const SortBufs &sb, uint64_t n, uint64_t seed, hipStream_t s) {
    static_assert(kRandomBits == 4 * kDigit && 3 * kDigit <= 32, "four passes, 4-byte keys after the first");
    uint32_t *h0 = (uint32_t *)sb.k0, *h1 = (uint32_t *)sb.k1, *none = nullptr;
    int rc = sort_pass<true>(sb, RandomKeys{seed}, none, n, h0, sb.v0, false, none, s);
    if (!rc) rc = sort_pass<false>(sb, S32{h0}, sb.v0, n, h1, sb.v1, false, none, s);
    if (!rc) rc = sort_pass<false>(sb, S32{h1}, sb.v1, n, h0, sb.v0, false, none, s);
    if (!rc) rc = sort_pass<false>(sb, S32{h0}, sb.v0, n, (void *)nullptr, sb.v1, false, none, s);
    return rc;
}

size_t reorder_bytes(uint64_t n, int order, uint32_t batch) {
    if (n == 0) return 256;
    size_t b = sort_bytes(n) + 256;  // + bbox / rank word
    if (order == PCR_ORDER_MORTON_SHUFFLE) b += sort_bytes((n + batch - 1) / batch);
    return b;
}

}  // namespace
}  // namespace pcr

using namespace pcr;

extern "C" size_t pcr_reorder_scratch_bytes(uint64_t n, int order, uint32_t batch) {
    if (order < 0 || order > 2 || n >= (1ull << 32)) return 0;
    if (order == PCR_ORDER_MORTON_SHUFFLE && batch == 0) return 0;
    return reorder_bytes(n, order, batch);
}

extern "C" int pcr_reorder(const pcr_point *in, pcr_point *out, uint32_t *perm_out, uint64_t n, int order,
                           uint32_t batch, uint64_t seed, void *scratch, size_t scratch_bytes, void *stream) {
    if (order < 0 || order > 2) return fail(PCR_EINVAL, "unknown order %d", order);
    if (order == PCR_ORDER_MORTON_SHUFFLE && batch == 0) return fail(PCR_EINVAL, "batch size 0");
    if (n >= (1ull << 32)) return fail(PCR_EINVAL, "reorder needs n < 2^32 (got %llu)", (unsigned long long)n);
    if (n == 0) return PCR_OK;
    if (!in || !out || ((uintptr_t)in & 15) || ((uintptr_t)out & 15))
        return fail(PCR_EINVAL, "points must be 16-byte aligned device pointers");
    if ((uintptr_t)perm_out & 3) return fail(PCR_EINVAL, "perm_out must be 4-byte aligned");
    const char *ib = (const char *)in, *ob = (const char *)out;
    if (ib < ob + 16 * n && ob < ib + 16 * n) return fail(PCR_EINVAL, "in and out overlap");
    size_t need = reorder_bytes(n, order, batch);
    if (!scratch || ((uintptr_t)scratch & 255)) return fail(PCR_EINVAL, "scratch must be a 256-byte aligned device pointer");
    if (scratch_bytes < need) return fail(PCR_ENOMEM, "scratch has %zu bytes, %zu needed", scratch_bytes, need);

    hipStream_t s = (hipStream_t)stream;
    const u32x4 *pin = (const u32x4 *)in;
    u32x4 *pout = (u32x4 *)out;
    uintptr_t p = (uintptr_t)scratch;
    uint32_t *word = (uint32_t *)p;  // bbox[6]
    p += 256;
    SortBufs sb;
    p = carve_sort(p, n, sb);
    uint32_t g = grid_for(n);

    if (order == PCR_ORDER_SHUFFLE) {
        int rc = sort_random(sb, n, seed, s);
        if (rc) return rc;
        hipLaunchKernelGGL(k_gather_random, dim3(g), dim3(256), 0, s, pin, sb.v1, n, seed, pout, perm_out);
        PCR_LAUNCHED();
        return PCR_OK;
    }
    uint64_t want = (n + 256 * kBboxLoads - 1) / (256 * kBboxLoads);
    const uint32_t gb = (uint32_t)(want < kBboxBlocks ? want : kBboxBlocks);
    hipLaunchKernelGGL(k_bbox, dim3(gb), dim3(256), 0, s, pin, n, sb.hist);
    const bool top = n >= kTopSort;
    hipLaunchKernelGGL(k_bbox_join, dim3(1), dim3(kBboxBlocks), 0, s, sb.hist, gb, pin, n, top, word);
    PCR_LAUNCHED();
    Places places{nullptr, 1, 1, 0};
    if (order == PCR_ORDER_MORTON_SHUFFLE) {
        // Shuffled Morton (Sec. 4): the batch indices are sorted by their
        // SplitMix64 keys in a second sort whose buffers follow sb in the
        // scratch; the batches are emitted in that order.
        const uint64_t nb = (n + batch - 1) / batch;
        SortBufs bs;
        carve_sort(p, nb, bs);
        int rc = sort_random(bs, nb, seed, s);
        if (rc) return rc;
        // bs.v0 is free after the sort
        hipLaunchKernelGGL(k_batch_rank, dim3(grid_for(nb)), dim3(256), 0, s, bs.v1, nb, seed, bs.v0);
        PCR_LAUNCHED();
        places = Places{bs.v0, batch, nb, n - (nb - 1) * batch};
    }
    const uint32_t gtiles = (uint32_t)((n + kGatherTile - 1) / kGatherTile);
    const dim3 gg((gtiles + 7) / 8 * 8);
    const uint32_t *go = top ? word + kWhole : nullptr;
    if (top) {
        int rc = sort_morton(sb, pin, n, word, 63 - kTopBits, word + kTop, s);
        if (rc) return rc;
        hipLaunchKernelGGL(k_gather<true>, gg, dim3(256), 0, s, pin, sb.v1, n, gtiles, word, places, pout, perm_out,
                           word + kTop);
        PCR_LAUNCHED();
    }
    int rc = sort_morton(sb, pin, n, word, 0, go, s);
    if (rc) return rc;
    hipLaunchKernelGGL(k_gather<false>, gg, dim3(256), 0, s, pin, sb.v1, n, gtiles, word, places, pout, perm_out, go);
    PCR_LAUNCHED();
    return PCR_OK;
}
