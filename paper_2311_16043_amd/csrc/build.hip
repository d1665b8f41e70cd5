// build.hip -- LBVH construction over 3D Gaussians on gfx950 (Sec. 4.1: a
// binary radix tree built after Karras 2012; leaves are the tight boxes of the
// Gaussians, internal nodes the boxes of their two children).
//
// Pipeline on one stream, no host synchronisation:
//   up to kSmallSort Gaussians
//     sort_small        bounds, 63-bit Morton keys and the whole radix sort in
//                       one block's LDS
//   beyond
//     bounds            min/max of the means (exact in any order)
//     morton            keys in binary32 arithmetic, first digit's counts
//     sort_hist, (sort_seg_sum), sort_scatter
//                       stable LSD radix sort, seven 9-bit digits
//   leaves_karras       per sorted leaf: whitening W, 3-sigma box, origin data,
//                       box pyramid; beside it internal nodes and parents
//   (root_box), refit   per node: child boxes as unions over their sorted-leaf
//                       ranges, and the compressed four-wide record the tracer
//                       walks

#include "rv_internal.h"

namespace rv {
namespace {

// ---- bounds of the means -----------------------------------------------------

// Union of the boxes (lo[3], hi[3]) of a block's kWaves waves; the result is
// in every thread. s: [kWaves][6] of LDS.
template <int kWaves>
__device__ __forceinline__ void block_union(float (&b)[6], float (*s)[6]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            b[a] = fminf(b[a], __shfl_xor(b[a], off));
            b[3 + a] = fmaxf(b[3 + a], __shfl_xor(b[3 + a], off));
        }
    if (lane == 0) {
#pragma unroll
        for (int a = 0; a < 6; ++a) s[w][a] = b[a];
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        b[a] = s[0][a];
        b[3 + a] = s[0][3 + a];
    }
    for (int k = 1; k < kWaves; ++k)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            b[a] = fminf(b[a], s[k][a]);
            b[3 + a] = fmaxf(b[3 + a], s[k][3 + a]);
        }
}

__device__ __forceinline__ void empty_box(float (&b)[6]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        b[a] = __builtin_inff();
        b[3 + a] = -__builtin_inff();
    }
}

__device__ __forceinline__ void add_mean(const float *__restrict__ mean, int64_t i, float (&b)[6]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float x = mean[3 * i + a];
        b[a] = fminf(b[a], x);
        b[3 + a] = fmaxf(b[3 + a], x);
    }
}

// Stores of 16-byte words whose lanes each hold a whole record of R words: the
// wave's 64 records go through LDS (rows padded by one word against bank
// conflicts) and leave as R stores of 64 consecutive words. Stored straight, each
// of a record's words is a 16-byte piece of another 64-byte line in every lane.
template <int R>
struct WaveRecords {
    float4 *lds;   // 64 (R + 1) words of the wave's own
    __device__ __forceinline__ void put(int k, float4 v) { lds[(threadIdx.x & 63) * (R + 1) + k] = v; }
    // Records [0, count) to out (consecutive); every lane of the wave calls it.
    __device__ __forceinline__ void flush(float4 *__restrict__ out, int64_t count) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int j = k * 64 + (threadIdx.x & 63);
            if (j < count * R) out[j] = lds[j / R * (R + 1) + j % R];
        }
        __builtin_amdgcn_wave_barrier();
    }
};

struct Inputs {
    const float *mean, *quat, *log_scale, *opacity, *normal;
};

// partial[a][block]: the box of a block's means; with packed, each Gaussian's
// inputs also go into one 64-byte record: quaternion | mean, opacity |
// log-scale, 0 | normal, 0 (normal (0, 0, 1) where the caller has none).
__global__ __launch_bounds__(1024) void k_bounds(Inputs g, int64_t n, float *__restrict__ partial,
                                                 float4 *__restrict__ packed) {
    __shared__ float s[16][6];
    __shared__ float4 stage[16][64 * 5];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    WaveRecords<4> out{stage[w]};
    float b[6];
    empty_box(b);
    for (int64_t i0 = (int64_t)blockIdx.x * 1024 + w * 64; i0 < n; i0 += (int64_t)gridDim.x * 1024) {
        const int64_t i = i0 + lane;
        if (i < n) {
            add_mean(g.mean, i, b);
            if (packed) {
                float nx = 0.f, ny = 0.f, nz = 1.f;
                if (g.normal) {
                    nx = g.normal[3 * i]; ny = g.normal[3 * i + 1]; nz = g.normal[3 * i + 2];
                }
                out.put(0, make_float4(g.quat[4 * i], g.quat[4 * i + 1], g.quat[4 * i + 2], g.quat[4 * i + 3]));
                out.put(1, make_float4(g.mean[3 * i], g.mean[3 * i + 1], g.mean[3 * i + 2], g.opacity[i]));
                out.put(2, make_float4(g.log_scale[3 * i], g.log_scale[3 * i + 1], g.log_scale[3 * i + 2], 0.f));
                out.put(3, make_float4(nx, ny, nz, 0.f));
            }
        }
        if (packed) out.flush(packed + 4 * i0, n - i0);
    }
    block_union<16>(b, s);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int a = 0; a < 6; ++a) partial[a * kBoundsBlocks + blockIdx.x] = b[a];
    }
}

// Box of the nparts <= kBoundsBlocks partials by a block of kThreads threads.
template <int kThreads>
__device__ __forceinline__ void union_partials(const float *__restrict__ partial, int nparts, float (&b)[6],
                                               float (*s)[6]) {
    empty_box(b);
    for (int p = threadIdx.x; p < nparts; p += kThreads)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            b[a] = fminf(b[a], partial[a * kBoundsBlocks + p]);
            b[3 + a] = fmaxf(b[3 + a], partial[(3 + a) * kBoundsBlocks + p]);
        }
    block_union<kThreads / 64>(b, s);
}

// ---- Morton keys ---------------------------------------------------------------

// Spread the low 21 bits of v to every third bit (bit b -> bit 3b).
__device__ __forceinline__ uint64_t part1by2_21(uint64_t v) {
    v &= 0x1fffffull;
    v = (v | (v << 32)) & 0x001f00000000ffffull;
    v = (v | (v << 16)) & 0x001f0000ff0000ffull;
    v = (v | (v << 8)) & 0x100f00f00f00f00full;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

// Quantise one coordinate: every operation is a single correctly rounded
// binary32 operation (sub, sub, div, exact scale by 2^21, floor, clamp).
__device__ __forceinline__ uint32_t quantise21(float x, float lo, float hi) {
#pragma clang fp contract(off)
    float den = hi - lo;
    float u = den > 0.0f ? (x - lo) / den : 0.0f;
    float f = floorf(u * 2097152.0f);
    f = fminf(fmaxf(f, 0.0f), 2097151.0f);
    return (uint32_t)f;
}

__device__ __forceinline__ uint64_t morton_key(const float *__restrict__ mean, int64_t i, const float (&b)[6]) {
    const uint32_t cx = quantise21(mean[3 * i + 0], b[0], b[3]);
    const uint32_t cy = quantise21(mean[3 * i + 1], b[1], b[4]);
    const uint32_t cz = quantise21(mean[3 * i + 2], b[2], b[5]);
    return (part1by2_21(cx) << 2) | (part1by2_21(cy) << 1) | part1by2_21(cz);
}

__device__ __forceinline__ void store_bounds(float *__restrict__ header, const float (&b)[6], int64_t n) {
#pragma unroll
    for (int a = 0; a < 6; ++a) header[a] = b[a];
    header[12] = __int_as_float((int)(n & 0x7fffffff));
}

// ---- radix sort ------------------------------------------------------------------
//
// Stable LSD sort of the 63-bit keys by seven 9-bit digits. A tile is 1,024
// threads x IT items. Each digit takes two launches: the digit counts, one block
// for a group of consecutive tiles, which leaves each tile's counts before it in
// its group and each group's total; then the scatter, in which every tile sums
// the groups' totals itself: no prefix-sum launches and no waiting between
// blocks. Consecutive tiles are scattered on one XCD: their runs of a digit are
// neighbours in memory, and that XCD's L2 joins them into whole lines. At 300,000
// keys a digit takes 4.5 + 9.3 us, bound by the latency of its few dependent
// steps (loads of keys and totals, two block scans, the stores); eight passes of
// five launches with one-wave tiles took 27 + 8 us each.

struct SortTables {
    uint32_t *before;   // [tiles][kDigits]
    uint32_t *totals;   // [groups of `group` tiles][kDigits]
    int64_t tiles;
    int group;
};

__device__ __forceinline__ uint32_t digit_of(uint64_t key, int shift) {
    return (uint32_t)(key >> shift) & (uint32_t)(kDigits - 1);
}

// Mask of the lanes whose `digit` equals this lane's, among `valid` lanes (one
// ballot per digit bit).
__device__ __forceinline__ uint64_t match_digit(uint32_t digit, uint64_t valid) {
    uint32_t lo = (uint32_t)valid, hi = (uint32_t)(valid >> 32);
#pragma unroll
    for (int b = 0; b < kDigitBits; ++b) {
        const int32_t own = __builtin_amdgcn_sbfe((int)digit, b, 1);   // all ones where the bit is set
        const uint64_t m = __builtin_amdgcn_ballot_w64(own != 0);
        lo &= ~((uint32_t)m ^ (uint32_t)own);
        hi &= ~((uint32_t)(m >> 32) ^ (uint32_t)own);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Rank of each of this wave's IT x 64 items among the items of its digit in the
// wave (item order: round by round, lane by lane), counting them in cnt
// (zero on entry; one row per wave).
template <int IT>
__device__ __forceinline__ void rank_items(const uint64_t (&key)[IT], const bool (&ok)[IT], int shift,
                                           uint32_t *cnt, uint32_t (&rank)[IT]) {
    const uint64_t lt = (1ull << (threadIdx.x & 63)) - 1ull;
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t d = digit_of(key[r], shift);
        const uint64_t valid = __ballot(ok[r]);
        const uint64_t peers = match_digit(d, valid);
        const uint32_t in_round = (uint32_t)__popcll(peers & lt);
        const uint32_t before = cnt[d];
        rank[r] = before + in_round;
        __builtin_amdgcn_wave_barrier();
        // every lane has read its digit's count; the group's first lane advances it
        if (ok[r] && in_round == 0) cnt[d] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
}

// Inclusive prefix sum over the wave's lanes by DPP: within rows of 16 lanes,
// then the row totals carried over by the two row broadcasts.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
#define RV_SCAN_STEP(ctrl, rows) \
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, (ctrl), (rows), 0xf, false)
    RV_SCAN_STEP(0x111, 0xf);   // row_shr:1
    RV_SCAN_STEP(0x112, 0xf);   // row_shr:2
    RV_SCAN_STEP(0x114, 0xf);   // row_shr:4
    RV_SCAN_STEP(0x118, 0xf);   // row_shr:8
    RV_SCAN_STEP(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
    RV_SCAN_STEP(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef RV_SCAN_STEP
    return x;
}

// Exclusive prefix sum of one value per thread over the first kDigits threads
// of the block (the others take part in the barrier). ws: one word per wave.
__device__ __forceinline__ uint32_t scan_digits(uint32_t v, uint32_t *ws) {
    const int t = threadIdx.x, w = t >> 6;
    const uint32_t x = wave_scan(v);
    if ((t & 63) == 63 && t < kDigits) ws[w] = x;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int k = 0; k < kDigits / 64; ++k) before += k < w ? ws[k] : 0u;
    return before + x - v;
}

// Turns the waves' counts of digit t = threadIdx.x into their first positions:
// `base` (a function of the digit's total in the block) plus the counts of the
// waves before. Called by every thread; holds a barrier.
template <int kWaves, class Base>
__device__ __forceinline__ void place_digits(uint32_t (*cnt)[kDigits], Base base) {
    const int t = threadIdx.x;
    uint32_t c[kWaves], total = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        c[k] = t < kDigits ? cnt[k][t] : 0u;
        total += c[k];
    }
    uint32_t pos = base(total);
    if (t < kDigits) {
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            cnt[k][t] = pos;
            pos += c[k];
        }
    }
}

// Item r of this thread in a tile: each wave holds 64 IT consecutive items.
template <int IT>
__device__ __forceinline__ int64_t item_index(int64_t tile, int r) {
    return (tile * kSortThreads + (threadIdx.x & ~63)) * IT + r * 64 + (threadIdx.x & 63);
}

// Counts of digit `shift` over the tiles of group blockIdx.x: each tile's row of
// `before` gets the counts of the group's earlier tiles, the group's row of
// `totals` all of them. The next tile's keys are fetched while one is counted.
template <int IT>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const uint64_t *__restrict__ keys, int64_t n, int shift,
                                                            SortTables tb) {
    __shared__ uint32_t h[kDigits];
    const int t = threadIdx.x;
    if (t < kDigits) h[t] = 0u;
    const int64_t t0 = (int64_t)blockIdx.x * tb.group, t1 = min(tb.tiles, t0 + tb.group);
    uint64_t next[IT];
    auto fetch = [&](int64_t tile) {
#pragma unroll
        for (int r = 0; r < IT; ++r) next[r] = keys[min(item_index<IT>(tile, r), n - 1)];
    };
    fetch(t0);
    __syncthreads();
    for (int64_t tile = t0; tile < t1; ++tile) {
        if (t < kDigits) tb.before[tile * kDigits + t] = h[t];
        uint64_t key[IT];
#pragma unroll
        for (int r = 0; r < IT; ++r) key[r] = next[r];
        if (tile + 1 < t1) fetch(tile + 1);
        __syncthreads();   // the row has been read
#pragma unroll
        for (int r = 0; r < IT; ++r)
            if (item_index<IT>(tile, r) < n) atomicAdd(&h[digit_of(key[r], shift)], 1u);
        __syncthreads();
    }
    if (t < kDigits) tb.totals[(int64_t)blockIdx.x * kDigits + t] = h[t];
}

// Morton keys in original order, and the header's bounds.
__global__ __launch_bounds__(kBoxBlock) void k_morton(const float *__restrict__ mean, int64_t n,
                                                      const float *__restrict__ partial, int nparts,
                                                      float *__restrict__ header, uint64_t *__restrict__ keys) {
    __shared__ float s[kBoxBlock / 64][6];
    const int64_t i = (int64_t)blockIdx.x * kBoxBlock + threadIdx.x;
    float b[6];
    union_partials<kBoxBlock>(partial, nparts, b, s);
    if (blockIdx.x == 0 && threadIdx.x == 0) store_bounds(header, b, n);
    if (i < n) keys[i] = morton_key(mean, i, b);
}

// Threads of the scatter take four digits of every kRowGroups-th count row.
constexpr int kRowGroups = kSortThreads / (kDigits / 4);

// Sums of the group totals over this thread's digits and row group: all of
// them, and those of groups below `lim`.
__device__ __forceinline__ void sum_rows(const uint32_t *__restrict__ rows, int64_t n_rows, int64_t lim, uint4 &all,
                                         uint4 &below) {
    const int q = threadIdx.x % (kDigits / 4), g = threadIdx.x / (kDigits / 4);
#pragma unroll 8
    for (int64_t r = g; r < n_rows; r += kRowGroups) {
        const uint4 v = *reinterpret_cast<const uint4 *>(rows + r * kDigits + 4 * q);
        const bool lo = r < lim;
        all.x += v.x; all.y += v.y; all.z += v.z; all.w += v.w;
        below.x += lo ? v.x : 0u; below.y += lo ? v.y : 0u; below.z += lo ? v.z : 0u; below.w += lo ? v.w : 0u;
    }
}

// Scatter by one digit: an item goes to (items of smaller digits) + (items of
// its digit in earlier groups of tiles, and in earlier tiles of its group) +
// (those in earlier waves of its tile) + its rank in the wave. vin NULL: an
// item's value is its index. The tile is first put in digit order in LDS, so that
// a wave writes runs of consecutive places: written straight from the items,
// every lane's key and value was a memory transaction of its own (1.2M keys:
// 26.2 us a pass, now 20.2 us).
template <int IT>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(const uint64_t *__restrict__ kin,
                                                               const uint32_t *__restrict__ vin, int64_t n, int shift,
                                                               SortTables tb, uint64_t *__restrict__ kout,
                                                               uint32_t *__restrict__ vout) {
    constexpr int kWaves = kSortThreads / 64, kTile = kSortThreads * IT;
    constexpr int kRedWords = 2 * kRowGroups * kDigits, kKeyWords = 2 * kTile;
    __shared__ uint32_t cnt[kWaves][kDigits];
    // the row groups' sums, then the staged keys
    __shared__ __align__(16) uint32_t buf[kRedWords > kKeyWords ? kRedWords : kKeyWords];
    __shared__ uint32_t vs[kTile];
    __shared__ uint32_t delta[kDigits];   // a digit's first global place less its first in the tile
    __shared__ uint32_t ws[2][kWaves];
    auto red = reinterpret_cast<uint32_t (*)[kRowGroups][kDigits]>(buf);
    uint64_t *ks = reinterpret_cast<uint64_t *>(buf);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint64_t key[IT];
    uint32_t val[IT], rank[IT];
    bool ok[IT];
    const int64_t tile = xcd_block(blockIdx.x, gridDim.x);
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int64_t i = item_index<IT>(tile, r);
        ok[r] = i < n;
        const int64_t j = ok[r] ? i : n - 1;
        key[r] = kin[j];
        val[r] = vin ? vin[j] : (uint32_t)j;
    }
    uint4 all = make_uint4(0u, 0u, 0u, 0u), below = all;
    sum_rows(tb.totals, (tb.tiles + tb.group - 1) / tb.group, tile / tb.group, all, below);
    const uint32_t in_group = t < kDigits ? tb.before[tile * kDigits + t] : 0u;
    {
        const int q = t % (kDigits / 4), g = t / (kDigits / 4);
        *reinterpret_cast<uint4 *>(&red[0][g][4 * q]) = all;
        *reinterpret_cast<uint4 *>(&red[1][g][4 * q]) = below;
    }
    for (int d = lane; d < kDigits; d += 64) cnt[w][d] = 0u;   // the wave's own row
    __builtin_amdgcn_wave_barrier();
    rank_items<IT>(key, ok, shift, cnt[w], rank);
    __syncthreads();
    place_digits<kWaves>(cnt, [&](uint32_t in_tile) {
        uint32_t total = 0, before = in_group;
        if (t < kDigits) {
#pragma unroll
            for (int g = 0; g < kRowGroups; ++g) {
                total += red[0][g][t];
                before += red[1][g][t];
            }
        }
        const uint32_t global = scan_digits(total, ws[0]) + before;
        const uint32_t local = scan_digits(in_tile, ws[1]);
        if (t < kDigits) delta[t] = global - local;
        return local;
    });
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IT; ++r)
        if (ok[r]) {
            const uint32_t p = cnt[w][digit_of(key[r], shift)] + rank[r];
            ks[p] = key[r];
            vs[p] = val[r];
        }
    __syncthreads();
    const int m = (int)min(n - tile * kTile, (int64_t)kTile);
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int j = r * kSortThreads + t;
        if (j < m) {
            const uint64_t k = ks[j];
            const uint32_t p = delta[digit_of(k, shift)] + (uint32_t)j;
            kout[p] = k;
            vout[p] = vs[j];
        }
    }
}

// Bounds, keys and sort of up to 1,024 IT Gaussians in one block: the items
// stay in registers, and each pass exchanges them through LDS. One launch in
// the place of sixteen: at 2,000 Gaussians launches and their latency were
// nearly all of the build's time (256 us with one wave per tile and a three-launch
// prefix sum per digit, now 45 us, of which this kernel takes 22).
template <int IT>
__global__ __launch_bounds__(kSortThreads) void k_sort_small(const float *__restrict__ mean, int n,
                                                             float *__restrict__ header, uint64_t *__restrict__ keys,
                                                             uint32_t *__restrict__ perm) {
    constexpr int kWaves = kSortThreads / 64;
    __shared__ uint64_t ks[kSortThreads * IT];
    __shared__ uint16_t vs[kSortThreads * IT];
    __shared__ uint32_t cnt[kWaves][kDigits];
    __shared__ uint32_t ws[kWaves];
    __shared__ float s[kWaves][6];
    static_assert(kSortThreads * IT <= 65536, "item indices are kept in 16 bits");
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    float b[6];
    empty_box(b);
    for (int i = t; i < n; i += kSortThreads) add_mean(mean, i, b);
    block_union<kWaves>(b, s);
    if (t == 0) store_bounds(header, b, n);
    uint64_t key[IT];
    uint32_t val[IT], rank[IT];
    bool ok[IT];
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int i = (t & ~63) * IT + r * 64 + lane;
        ok[r] = i < n;
        val[r] = (uint32_t)(ok[r] ? i : n - 1);
        key[r] = morton_key(mean, val[r], b);
    }
    for (int pass = 0; pass < kPasses; ++pass) {
        const int shift = kDigitBits * pass;
        for (int d = lane; d < kDigits; d += 64) cnt[w][d] = 0u;
        __builtin_amdgcn_wave_barrier();
        rank_items<IT>(key, ok, shift, cnt[w], rank);
        __syncthreads();
        place_digits<kWaves>(cnt, [&](uint32_t total) { return scan_digits(total, ws); });
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IT; ++r)
            if (ok[r]) {
                const uint32_t p = cnt[w][digit_of(key[r], shift)] + rank[r];
                if (pass == kPasses - 1) {
                    keys[p] = key[r];
                    perm[p] = val[r];
                } else {
                    ks[p] = key[r];
                    vs[p] = (uint16_t)val[r];
                }
            }
        if (pass == kPasses - 1) break;   // block-uniform
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int i = (t & ~63) * IT + r * 64 + lane;
            if (ok[r]) {
                key[r] = ks[i];
                val[r] = vs[i];
            }
        }
    }
}

// ---- leaf records and their box pyramid ---------------------------------------

// Unions of 8, 64 and 512 consecutive sorted leaf boxes (six floats each).
struct BoxLevels {
    float *l8, *l64, *l512;
};

// Union of each aligned group of kGroup lanes' boxes (in every lane of it),
// from groups of kFrom.
template <int kFrom, int kGroup>
__device__ __forceinline__ void group_union(float (&b)[6]) {
#pragma unroll
    for (int off = kFrom; off < kGroup; off <<= 1)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            b[a] = fminf(b[a], __shfl_xor(b[a], off));
            b[3 + a] = fmaxf(b[3 + a], __shfl_xor(b[3 + a], off));
        }
}

// Boxes in memory are six floats at multiples of 24 bytes: moved as three float2.
__device__ __forceinline__ void store_box(float *__restrict__ out, const float (&b)[6]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) reinterpret_cast<float2 *>(out)[a] = make_float2(b[2 * a], b[2 * a + 1]);
}

__device__ __forceinline__ void load_box(const float *__restrict__ p, float (&b)[6]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float2 v = reinterpret_cast<const float2 *>(p)[a];
        b[2 * a] = v.x;
        b[2 * a + 1] = v.y;
    }
}

struct LeafArgs {
    Inputs in;
    const float4 *packed;   // 64-byte records of k_bounds, or null
    const uint32_t *perm;
    float4 *rec;
    float *box;
    float4 *origins;
    BoxLevels lv;
};

// Record (into out), box and origin data of sorted leaf m (the box also in b).
template <bool kPacked>
__device__ __forceinline__ void prepare_leaf(const LeafArgs &g, int64_t m, const float (&mb)[6], float (&b)[6],
                                             WaveRecords<kLeafF4> &out) {
    // scene scale: largest coordinate magnitude plus the diagonal of the means' box
    float scale = 0.0f, diag2 = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        scale = fmaxf(scale, fmaxf(fabsf(mb[a]), fabsf(mb[3 + a])));
        diag2 += (mb[3 + a] - mb[a]) * (mb[3 + a] - mb[a]);
    }
    const float widen_abs = (scale + sqrtf(diag2) + 1.0f) * 0x1p-20f;
    const int64_t i = g.perm[m];
    float qw, qx, qy, qz, mu[3], ls[3], op, nx = 0.f, ny = 0.f, nz = 1.f;
    if (kPacked) {
        const float4 *r = g.packed + 4 * i;
        const float4 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
        qw = r0.x; qx = r0.y; qy = r0.z; qz = r0.w;
        mu[0] = r1.x; mu[1] = r1.y; mu[2] = r1.z;
        op = r1.w;
        ls[0] = r2.x; ls[1] = r2.y; ls[2] = r2.z;
        nx = r3.x; ny = r3.y; nz = r3.z;
    } else {
        const Inputs &in = g.in;
        qw = in.quat[4 * i]; qx = in.quat[4 * i + 1]; qy = in.quat[4 * i + 2]; qz = in.quat[4 * i + 3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            mu[a] = in.mean[3 * i + a];
            ls[a] = in.log_scale[3 * i + a];
        }
        op = in.opacity[i];
        if (in.normal) {
            nx = in.normal[3 * i]; ny = in.normal[3 * i + 1]; nz = in.normal[3 * i + 2];
        }
    }
    float inv = 1.0f / sqrtf(qw * qw + qx * qx + qy * qy + qz * qz);
    qw *= inv; qx *= inv; qy *= inv; qz *= inv;
    // rotation matrix of the unit quaternion (w, x, y, z)
    float R[3][3];
    R[0][0] = 1.f - 2.f * (qy * qy + qz * qz); R[0][1] = 2.f * (qx * qy - qw * qz); R[0][2] = 2.f * (qx * qz + qw * qy);
    R[1][0] = 2.f * (qx * qy + qw * qz); R[1][1] = 1.f - 2.f * (qx * qx + qz * qz); R[1][2] = 2.f * (qy * qz - qw * qx);
    R[2][0] = 2.f * (qx * qz - qw * qy); R[2][1] = 2.f * (qy * qz + qw * qx); R[2][2] = 1.f - 2.f * (qx * qx + qy * qy);
    float s[3], is[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        s[a] = expf(ls[a]);
        is[a] = expf(-ls[a]);
    }
    // whitening W = diag(1/s) R^T: row a is column a of R divided by s_a
    float W[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) W[a][c] = is[a] * R[c][a];
    // row 2 of W is not stored: for a proper rotation, column 2 of R is
    // column 0 x column 1, so W row 2 = (s0 s1 / s2) (W row 0 x W row 1)
    out.put(0, make_float4(mu[0], mu[1], mu[2], op));
    out.put(1, make_float4(W[0][0], W[0][1], W[0][2], s[0] * s[1] * is[2]));
    out.put(2, make_float4(W[1][0], W[1][1], W[1][2], __int_as_float((int)i)));
    // 3-sigma box: half extent along world axis a is 3 sqrt(sum_m (R_am s_m)^2),
    // widened by a relative 2^-12 (rounding of R, s and the square root) and by
    // 2^-20 of the scene scale (rounding of the box and of the slab test)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float e0 = R[a][0] * s[0], e1 = R[a][1] * s[1], e2 = R[a][2] * s[2];
        float h = kBuildSigma * sqrtf(e0 * e0 + e1 * e1 + e2 * e2);
        h = h * (1.0f + 0x1p-12f) + widen_abs;
        b[a] = mu[a] - h;
        b[3 + a] = mu[a] + h;
    }
    store_box(g.box + 6 * m, b);
    if (g.in.normal) {
        float nl = sqrtf(nx * nx + ny * ny + nz * nz);
        nx /= nl; ny /= nl; nz /= nl;
    }
    float smax = expf(fmaxf(ls[0], fmaxf(ls[1], ls[2])));
    g.origins[m] = make_float4(nx, ny, nz, smax);
}

// ---- Karras internal nodes -----------------------------------------------------

// The sorted keys around a block of nodes in LDS; further keys from memory.
struct KeyWindow {
    const uint64_t *lds, *keys;
    int64_t n, w0;   // first position of the window
    __device__ __forceinline__ uint64_t at(int64_t j) const {
        const int64_t k = j - w0;
        return k >= 0 && k < kKeyWindow ? lds[k] : keys[j];
    }
    // Common-prefix length of the augmented keys (key, position) at i (whose
    // key is ki) and j; -1 when j is outside [0, n).
    __device__ __forceinline__ int prefix_len(uint64_t ki, int64_t i, int64_t j) const {
        if (j < 0 || j >= n) return -1;
        const uint64_t b = at(j);
        if (ki != b) return __clzll((long long)(ki ^ b));
        return 64 + __clz((int)((uint32_t)i ^ (uint32_t)j));
    }
};

__device__ __forceinline__ void karras_node(const KeyWindow &kw, int64_t i, float4 *__restrict__ topo,
                                            int32_t *__restrict__ parent) {
    const int64_t n = kw.n;
    const uint64_t ki = kw.at(i);
    // direction of the range: towards the neighbour sharing the longer prefix
    const int pr = kw.prefix_len(ki, i, i + 1), pl = kw.prefix_len(ki, i, i - 1);
    const int d = pr > pl ? 1 : -1;
    const int dmin = pr > pl ? pl : pr;
    // exponential search for an upper bound of the range length, then binary search
    int64_t lmax = 2;
    while (kw.prefix_len(ki, i, i + lmax * d) > dmin) lmax <<= 1;
    int64_t l = 0;
    for (int64_t t = lmax >> 1; t >= 1; t >>= 1)
        if (kw.prefix_len(ki, i, i + (l + t) * d) > dmin) l += t;
    const int64_t j = i + l * d;
    const int dnode = kw.prefix_len(ki, i, j);
    // split: the last position (counted from i) sharing more than dnode bits with i
    int64_t s = 0, t = l;
    do {
        t = (t + 1) >> 1;
        if (kw.prefix_len(ki, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    const int64_t gamma = i + s * d + (d < 0 ? -1 : 0);
    const int64_t lo = i < j ? i : j, hi = i < j ? j : i;
    const int32_t left = (lo == gamma) ? ~(int32_t)gamma : (int32_t)gamma;
    const int32_t right = (hi == gamma + 1) ? ~(int32_t)(gamma + 1) : (int32_t)(gamma + 1);
    // (words 12-15 of the binary record): the children, then the first and last
    // sorted leaf under i
    topo[i] = make_float4(__int_as_float(left), __int_as_float(right), __int_as_float((int32_t)lo),
                          __int_as_float((int32_t)hi));
    parent[left >= 0 ? left : (n - 1 + (int64_t)~left)] = (int32_t)i;
    parent[right >= 0 ? right : (n - 1 + (int64_t)~right)] = (int32_t)i;
    if (i == 0) parent[0] = -1;
}

// Leaf records, boxes and pyramid (512 sorted leaves per block) and, in a
// build, the internal nodes (512 per block): independent work that shares one
// launch, even blocks taking leaves and odd ones nodes, so that the gathers of
// the first and the searches of the second overlap (28 us at 300,000, against
// 25 and 22 us as two launches; the leaves alone 62 us at 1.2M, 110 us before their
// inputs were packed, bound by the gathers and by 106 MB of records). A refit (kRefit) launches
// leaf blocks only; it takes the means' box from the partials and leaves a blob
// whose header does not record n as it is.
template <bool kRefit, bool kPacked>
__global__ __launch_bounds__(kBoxBlock) void k_leaves_karras(LeafArgs g, int64_t n, const float *__restrict__ partial,
                                                             int nparts, float *__restrict__ header,
                                                             const uint64_t *__restrict__ keys,
                                                             float4 *__restrict__ topo,
                                                             int32_t *__restrict__ parent) {
    // (12 KB in a block of nodes, 32 KB in a block of leaves)
    __shared__ __align__(16) char lds[kBoxBlock * 16 * (kLeafF4 + 1)];
    auto kwin = reinterpret_cast<uint64_t *>(lds);
    auto stage = reinterpret_cast<float4 (*)[64 * (kLeafF4 + 1)]>(lds);
    static_assert(sizeof(lds) >= kKeyWindow * sizeof(uint64_t), "the key window must fit");
    __shared__ float s[kBoxBlock / 64][6];
    if (kRefit && !tree_matches(header, n)) return;   // block-uniform
    if (!kRefit && (blockIdx.x & 1)) {
        const int64_t base = (int64_t)(blockIdx.x >> 1) * kBoxBlock;
        KeyWindow kw;
        kw.lds = kwin;
        kw.keys = keys;
        kw.n = n;
        kw.w0 = base - (kKeyWindow - kBoxBlock) / 2;
        for (int k = threadIdx.x; k < kKeyWindow; k += kBoxBlock) {
            const int64_t j = kw.w0 + k;
            if (j >= 0 && j < n) kwin[k] = keys[j];
        }
        __syncthreads();
        const int64_t i = base + threadIdx.x;
        if (i < n - 1) karras_node(kw, i, topo, parent);
        if (n == 1 && i == 0) parent[0] = -1;
        return;
    }
    const int64_t blk = kRefit ? blockIdx.x : blockIdx.x >> 1;
    float mb[6];
    if (kRefit) {
        union_partials<kBoxBlock>(partial, nparts, mb, s);
        if (blk == 0 && threadIdx.x == 0) store_bounds(header, mb, n);
        __syncthreads();   // s is used again below
    } else {
#pragma unroll
        for (int a = 0; a < 6; ++a) mb[a] = header[a];
    }
    const int64_t m = blk * kBoxBlock + threadIdx.x;
    float b[6];
    empty_box(b);
    WaveRecords<kLeafF4> out{stage[threadIdx.x >> 6]};
    if (m < n) prepare_leaf<kPacked>(g, m, mb, b, out);
    const int64_t m0 = m & ~int64_t(63);   // the wave's first leaf
    out.flush(g.rec + kLeafF4 * m0, n - m0);
    group_union<1, 8>(b);
    if ((threadIdx.x & 7) == 0 && m < n) store_box(g.lv.l8 + 6 * (m >> 3), b);
    group_union<8, 64>(b);
    if ((threadIdx.x & 63) == 0 && m < n) store_box(g.lv.l64 + 6 * (m >> 6), b);
    block_union<kBoxBlock / 64>(b, s);
    if (threadIdx.x == 0) store_box(g.lv.l512 + 6 * blk, b);
}

// ---- child boxes and four-wide nodes --------------------------------------------
//
// Every internal node covers a contiguous range of sorted leaves (Karras), so
// the box of each child is the union of the leaf boxes over the child's range:
// min and max are exact in any order and may count a leaf twice, so this equals
// the bottom-up union of the children's boxes, with no ordering between nodes
// to arrange. The box of a range of 2^k to 2^(k+1) leaves is the union of the two
// windows of 2^k leaves at its ends: a block keeps the windows around its nodes
// in LDS and doubles them in place from one leaf to kTopWindow, every node over
// at most twice that many leaves taking its two when its size comes up (nine
// nodes in ten). Of the others, eight lanes cover one whose leaves lie in the
// block's LDS window with windows of kTopWindow, and a wave covers any other in
// one step with up to seven leaves, groups of 8 and groups of 64 at either end, a
// lane each, and its groups of 512. Boxes and four-wide records take 17 + 13 us at
// 300,000 nodes (83 us with a lane per short and a wave per long range, each child
// by itself) and 41 + 47 us at 1.2M (235 us), bound by the records' bytes there.
//
// The four-wide record of a node lists the children of its two children (a
// child that is a leaf keeps its own slot, the next slot is empty), so one
// traversal step tests up to four boxes from three 16-byte loads. Every
// internal node gets a record; a traversal from the root only lands on nodes
// an even number of binary levels down. Layout (12 words in a 64-byte slot):
//   words 0-2   origin O (float), at or below the lowest child plane
//   word 3      bytes 0-2: per-axis step exponents, step_a = 2^(byte - 127);
//               byte 3: kind of slot j in bits 2j..2j+1 (0 empty, 1 internal
//               node, 3 leaf: bit 0 = used, bit 1 = leaf)
//   words 4-9   lo_x, lo_y, lo_z, hi_x, hi_y, hi_z planes, one byte per slot
//               (byte j = slot j): plane = O_a + q step_a
//   words 10-11 index of slot 2s for side s; slot 2s + 1 holds that index + 1
//               (a node's two children always have consecutive indices)
// Planes are rounded outward from the refitted binary boxes after widening
// them by eta = (largest root-box coordinate + root diagonal + 1) 2^-20, in
// exact (double) arithmetic, so a traversal that evaluates the plane
// distances as fma(q, step/d, (O - o)/d) (error below eta / 2) never rejects
// a box the exact ray enters.

__device__ __forceinline__ void add_box(float (&b)[6], const float *__restrict__ p) {
    float v[6];
    load_box(p, v);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        b[a] = fminf(b[a], v[a]);
        b[3 + a] = fmaxf(b[3 + a], v[3 + a]);
    }
}

// Union of leaves [a, e) by one wave (in every lane of it).
__device__ __forceinline__ void wave_range(int64_t a, int64_t e, const float *__restrict__ box, const BoxLevels &lv,
                                           float (&b)[6]) {
    const int lane = threadIdx.x & 63, k = lane & 7, part = lane >> 3;
    empty_box(b);
    // parts 0, 1: leaves at the low and the high end; 2, 3: groups of 8; 4, 5: of 64
    const float *level[3] = {box, lv.l8, lv.l64};
    const float *src = nullptr;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const int64_t up = min((a + 7) & ~int64_t(7), e);       // [a, up) at the low end
        if (part == 2 * l && a + k < up) src = level[l] + 6 * (a + k);
        a = up;
        const int64_t down = max(e & ~int64_t(7), a);           // [down, e) at the high end
        if (part == 2 * l + 1 && down + k < e) src = level[l] + 6 * (down + k);
        e = down;
        // nothing left, or both are multiples of 8
        a >>= 3;
        e >>= 3;
    }
    if (src) add_box(b, src);
#pragma unroll 4
    for (int64_t g = a + lane; g < e; g += 64) add_box(b, lv.l512 + 6 * g);
    group_union<1, 64>(b);
}

// Children and leaf range of an internal node as the node kernel leaves them:
// record i is at p[i * stride].
struct Topology {
    const float4 *p;
    int stride;
    __device__ __forceinline__ float4 at(int64_t i) const { return p[i * stride]; }
};

// node_box[i]: the box of internal node i, from its leaf range (one lane per
// node but for the long ranges). copy: where the topology goes as consecutive
// records, when it comes from the binary records of a tree (a refit).
__global__ __launch_bounds__(kBoxBlock) void k_node_boxes(int64_t n, const float *__restrict__ leaf_box, BoxLevels lv,
                                                          Topology topo, float *__restrict__ header,
                                                          float *__restrict__ node_box, float4 *__restrict__ copy) {
    __shared__ float win[6][kBoxWindow];
    if (!tree_matches(header, n)) return;   // block-uniform
    const int t = threadIdx.x, lane = t & 63;
    const int64_t base = (int64_t)blockIdx.x * kBoxBlock, w0 = base - (kBoxWindow - kBoxBlock) / 2;
    const int64_t i = base + t;
    const bool live = i < n - 1;
    int64_t first = 0, end = 0;   // the node's leaves
    if (live) {
        const float4 r = topo.at(i);
        first = __float_as_int(r.z);
        end = (int64_t)__float_as_int(r.w) + 1;
        if (copy) copy[i] = r;
    }
    // this thread's windows: those from leaves w0 + t and w0 + kBoxBlock + t
    float own[2][6];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        empty_box(own[h]);
        const int64_t m = w0 + h * kBoxBlock + t;
        if (m >= 0 && m < n) add_box(own[h], leaf_box + 6 * m);
#pragma unroll
        for (int a = 0; a < 6; ++a) win[a][h * kBoxBlock + t] = own[h][a];
    }
    const bool near = first >= w0 && end <= w0 + kBoxWindow;
    const int lo = near ? (int)(first - w0) : 0, len = (int)(end - first);
    float box[6];
    empty_box(box);
    __syncthreads();
#pragma unroll
    for (int w = 1; w <= kTopWindow; w *= 2) {
        if (near && len >= w && (len < 2 * w || (w == kTopWindow && len == 2 * w))) {
            const int p = lo, q = lo + len - w;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                box[a] = fminf(win[a][p], win[a][q]);
                box[3 + a] = fmaxf(win[3 + a][p], win[3 + a][q]);
            }
        }
        if (w == kTopWindow) break;
        // the windows of 2 w leaves (those running past the LDS window are not
        // used: a range that takes them lies inside it)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int q = h * kBoxBlock + t + w;
            if (q < kBoxWindow) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    own[h][a] = fminf(own[h][a], win[a][q]);
                    own[h][3 + a] = fmaxf(own[h][3 + a], win[3 + a][q]);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < 6; ++a) win[a][h * kBoxBlock + t] = own[h][a];
        __syncthreads();
    }
    // longer ranges inside the LDS window, eight at a time, eight lanes each
    uint64_t todo = __ballot(near && len > 2 * kTopWindow);
    while (todo) {
        const int rank = __popcll(todo & ((1ull << lane) - 1ull));
        int src = 64, mine = 0;
        uint64_t rest = todo;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int f = rest ? __ffsll((unsigned long long)rest) - 1 : 64;
            src = (lane >> 3) == k ? f : src;
            rest &= rest - 1;
        }
        const int a0 = __shfl(lo, src & 63), n0 = __shfl(len, src & 63);
        float b[6];
        empty_box(b);
        if (src < 64)
            for (int k = (lane & 7) * kTopWindow; k < n0; k += 8 * kTopWindow) {
                const int p = a0 + min(k, n0 - kTopWindow);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    b[a] = fminf(b[a], win[a][p]);
                    b[3 + a] = fmaxf(b[3 + a], win[3 + a][p]);
                }
            }
        group_union<1, 8>(b);
        mine = (todo >> lane) & 1 && rank < 8;
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            const float v = __shfl(b[a], 8 * (rank & 7));
            box[a] = mine ? v : box[a];
        }
        todo = rest;
    }
    todo = __ballot(live && !near);
    while (todo) {
        const int src = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1;
        float b[6];
        wave_range(__shfl(first, src), __shfl(end, src), leaf_box, lv, b);
        if (lane == src) {
#pragma unroll
            for (int a = 0; a < 6; ++a) box[a] = b[a];
        }
    }
    if (live) store_box(node_box + 6 * i, box);
    if (i == 0) {
        // the root box; a single Gaussian's is its leaf box
        if (n == 1) add_box(box, leaf_box);
        store_box(header + 6, box);
    }
}

// One lane per internal node: its binary record (the two child boxes and the
// topology words) and its four-wide record.
__global__ __launch_bounds__(256) void k_collapse4(int64_t n, const float *__restrict__ leaf_box,
                                                   const float *__restrict__ node_box,
                                                   const float4 *__restrict__ topo, float4 *__restrict__ nodes, const float *__restrict__ header,
                                                   float *__restrict__ nodes4) {
    __shared__ float4 stage[4][64 * 5];
    if (!tree_matches(header, n)) return;   // block-uniform
    const int64_t i0 = (int64_t)blockIdx.x * 256 + (threadIdx.x & ~63);   // the wave's first node
    if (i0 >= n - 1) return;
    // lanes past the last node work on it again and store nothing
    const int64_t i = min(i0 + (threadIdx.x & 63), n - 2);
    const float4 r3 = topo[i];
    const int32_t child[2] = {__float_as_int(r3.x), __float_as_int(r3.y)};
    float box[4][6], root[6];
    uint32_t kind[4] = {0u, 0u, 0u, 0u};
    int32_t first[2];
    auto box_of = [&](int32_t c, float (&b)[6]) {
        load_box(c < 0 ? leaf_box + 6 * (int64_t)~c : node_box + 6 * (int64_t)c, b);
    };
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int32_t c = child[side];
        const int s0 = 2 * side, s1 = s0 + 1;
        if (c < 0) {
            box_of(c, box[s0]);
            kind[s0] = 3u;
            first[side] = ~c;
            // the unused slot takes the leaf's box, which keeps the node box unchanged
#pragma unroll
            for (int a = 0; a < 6; ++a) box[s1][a] = box[s0][a];
        } else {
            const float4 rc = topo[c];
            const int32_t lc = __float_as_int(rc.x), rr = __float_as_int(rc.y);
            box_of(lc, box[s0]);
            box_of(rr, box[s1]);
            kind[s0] = lc < 0 ? 3u : 1u;
            kind[s1] = rr < 0 ? 3u : 1u;
            first[side] = lc < 0 ? ~lc : lc;
        }
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) root[a] = node_box[a];
    float cb[2][6];
#pragma unroll
    for (int side = 0; side < 2; ++side)
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            const float x = box[2 * side][a], y = box[2 * side + 1][a];
            cb[side][a] = a < 3 ? fminf(x, y) : fmaxf(x, y);
        }
    WaveRecords<4> out{stage[threadIdx.x >> 6]};
    out.put(0, make_float4(cb[0][0], cb[0][1], cb[0][2], cb[0][3]));
    out.put(1, make_float4(cb[0][4], cb[0][5], cb[1][0], cb[1][1]));
    out.put(2, make_float4(cb[1][2], cb[1][3], cb[1][4], cb[1][5]));
    out.put(3, r3);
    out.flush(nodes + 4 * i0, n - 1 - i0);
    double ext = 0.0, diag2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double l = root[a], h = root[3 + a];
        ext = fmax(ext, fmax(fabs(l), fabs(h)));
        diag2 += (h - l) * (h - l);
    }
    const double eta = (ext + sqrt(diag2) + 1.0) * 0x1p-20;
    uint32_t words[12];
    uint32_t meta = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double lo = fmin((double)cb[0][a], (double)cb[1][a]);
        const double hi = fmax((double)cb[0][3 + a], (double)cb[1][3 + a]);
        // origin: a float at or below lo - eta
        const double od = lo - eta;
        float O = (float)od;
        if ((double)O > od) O = nextafterf(O, -__builtin_inff());
        // smallest power-of-two step with 255 steps reaching hi + eta
        // (the exponent of x / 255 from that of x: 255 = (255/256) 2^8)
        int e;
        const double frac = frexp(hi + eta - (double)O, &e);
        e += frac >= 255.0 / 256.0 ? -7 : -8;
        e = max(-126, min(127, e));
        // the step's reciprocal is a power of two: products with it are exact
        const double inv_step = ldexp(1.0, -e);
        uint32_t qlo = 0, qhi = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // (the conversion of a value in [0, 255] rounds down)
            const double ql = ((double)box[j][a] - eta - (double)O) * inv_step;
            const double qh = ceil(((double)box[j][3 + a] + eta - (double)O) * inv_step);
            qlo |= (uint32_t)fmin(fmax(ql, 0.0), 255.0) << (8 * j);
            qhi |= (uint32_t)fmin(fmax(qh, 0.0), 255.0) << (8 * j);
        }
        words[a] = __float_as_uint(O);
        words[4 + a] = qlo;
        words[7 + a] = qhi;
        meta |= (uint32_t)(e + 127) << (8 * a);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) meta |= kind[j] << (24 + 2 * j);
    words[3] = meta;
    words[10] = (uint32_t)first[0];
    words[11] = (uint32_t)first[1];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        out.put(k, make_float4(__uint_as_float(words[4 * k]), __uint_as_float(words[4 * k + 1]),
                               __uint_as_float(words[4 * k + 2]), __uint_as_float(words[4 * k + 3])));
    out.put(3, make_float4(0.f, 0.f, 0.f, 0.f));
    out.flush(reinterpret_cast<float4 *>(nodes4) + 4 * i0, n - 1 - i0);
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

inline int bounds_blocks(int64_t n) { return (int)std::min<int64_t>(kBoundsBlocks, (n + 1023) / 1024); }

// Boxes and four-wide records of a tree whose leaf boxes and pyramid are in
// place; its topology is in topo, or with refit in the binary records (topo then
// receives it).
void launch_refit(int64_t n, const LeafArgs &la, bool refit, float4 *topo, float *node_box, float4 *nodes,
                  float *header, float *nodes4, hipStream_t s) {
    const Topology from = refit ? Topology{nodes + 3, 4} : Topology{topo, 1};
    hipLaunchKernelGGL(k_node_boxes, dim3(grid_for(n, kBoxBlock)), dim3(kBoxBlock), 0, s, n, la.box, la.lv, from,
                       header, node_box, refit ? topo : (float4 *)nullptr);
    if (n > 1)
        hipLaunchKernelGGL(k_collapse4, dim3(grid_for(n - 1, 256)), dim3(256), 0, s, n, la.box, node_box, topo, nodes,
                           header, nodes4);
}

// Bounds, keys and radix sort of more than kSmallSort Gaussians in tiles of
// kSortThreads IT items.
template <int IT>
void launch_sort(const LeafArgs &la, int64_t n, float *partial, float *header, uint64_t *keys, uint32_t *perm,
                 uint64_t *keys_tmp, uint32_t *vals_tmp, const SortTables &tb, hipStream_t s) {
    const int nparts = bounds_blocks(n);
    const unsigned tiles = (unsigned)tb.tiles, groups = grid_for(tb.tiles, tb.group);
    hipLaunchKernelGGL(k_bounds, dim3(nparts), dim3(1024), 0, s, la.in, n, partial, const_cast<float4 *>(la.packed));
    // an odd number of passes: the unsorted keys start in the scratch, so that
    // the last pass writes the result
    static_assert(kPasses % 2 == 1, "the sorted keys must end in the blob");
    hipLaunchKernelGGL(k_morton, dim3(grid_for(n, kBoxBlock)), dim3(kBoxBlock), 0, s, la.in.mean, n, partial, nparts,
                       header, keys_tmp);
    uint64_t *ka = keys_tmp, *kb = keys;
    uint32_t *va = vals_tmp, *vb = perm;
    for (int pass = 0; pass < kPasses; ++pass) {
        const int shift = kDigitBits * pass;
        hipLaunchKernelGGL(k_sort_hist<IT>, dim3(groups), dim3(kSortThreads), 0, s, ka, n, shift, tb);
        hipLaunchKernelGGL(k_sort_scatter<IT>, dim3(tiles), dim3(kSortThreads), 0, s, ka,
                           pass == 0 ? (const uint32_t *)nullptr : va, n, shift, tb, kb, vb);
        std::swap(ka, kb);
        std::swap(va, vb);
    }
}

}  // namespace

}  // namespace rv

using namespace rv;

extern "C" size_t rv_bvh_bytes(int64_t n) { return n < 1 ? 0 : bvh_layout(n).total; }

extern "C" size_t rv_build_workspace_bytes(int64_t n) { return n < 1 ? 0 : build_ws_layout(n).total; }

extern "C" rv_status rv_bvh_view(const void *bvh, int64_t n, rv_bvh_arrays *out) {
    clear_error();
    RV_REQUIRE(bvh && out, RV_ERR_INVALID_ARG, "rv_bvh_view: null pointer");
    RV_REQUIRE(n >= 1 && n <= RV_MAX_GAUSSIANS, RV_ERR_INVALID_ARG, "rv_bvh_view: n out of range");
    BvhLayout L = bvh_layout(n);
    out->n = n;
    out->header = at<float>(bvh, L.header);
    out->keys = at<uint64_t>(bvh, L.keys);
    out->perm = at<uint32_t>(bvh, L.perm);
    out->nodes = at<float>(bvh, L.nodes);
    out->parent = at<int32_t>(bvh, L.parent);
    out->leaf_records = at<float>(bvh, L.leaf_rec);
    out->leaf_boxes = at<float>(bvh, L.leaf_box);
    out->origins = at<float>(bvh, L.origins);
    out->nodes4 = at<uint32_t>(bvh, L.nodes4);
    return RV_OK;
}

namespace {

LeafArgs leaf_args(const rv_gaussians *g, void *bvh, const BvhLayout &L, void *ws, const BuildWsLayout &W) {
    LeafArgs a;
    a.in = Inputs{g->mean, g->quat, g->log_scale, g->opacity, g->normal};
    a.packed = packs_inputs(g->n) ? at<float4>(ws, W.packed) : nullptr;
    a.perm = at<uint32_t>(bvh, L.perm);
    a.rec = at<float4>(bvh, L.leaf_rec);
    a.box = at<float>(bvh, L.leaf_box);
    a.origins = at<float4>(bvh, L.origins);
    a.lv = BoxLevels{at<float>(ws, W.box8), at<float>(ws, W.box64), at<float>(ws, W.box512)};
    return a;
}

}  // namespace

extern "C" rv_status rv_build_bvh(const rv_gaussians *g, void *bvh, size_t bvh_bytes, void *ws, size_t ws_bytes,
                                  void *stream) {
    clear_error();
    RV_REQUIRE(g && bvh && ws, RV_ERR_INVALID_ARG, "rv_build_bvh: null argument (g, bvh or ws)");
    RV_REQUIRE(g->mean && g->quat && g->log_scale && g->opacity, RV_ERR_INVALID_ARG,
               "rv_build_bvh: null Gaussian array");
    const int64_t n = g->n;
    RV_REQUIRE(n >= 1 && n <= RV_MAX_GAUSSIANS, RV_ERR_INVALID_ARG, "rv_build_bvh: n=%lld out of range",
               (long long)n);
    RV_REQUIRE(((uintptr_t)bvh % kAlign) == 0 && ((uintptr_t)ws % kAlign) == 0, RV_ERR_INVALID_ARG,
               "rv_build_bvh: bvh and ws must be 256-byte aligned");
    const BvhLayout L = bvh_layout(n);
    const BuildWsLayout W = build_ws_layout(n);
    RV_REQUIRE(bvh_bytes >= L.total, RV_ERR_WORKSPACE, "rv_build_bvh: bvh_bytes %zu < %zu", bvh_bytes, L.total);
    RV_REQUIRE(ws_bytes >= W.total, RV_ERR_WORKSPACE, "rv_build_bvh: ws_bytes %zu < %zu", ws_bytes, W.total);
    hipStream_t s = (hipStream_t)stream;

    float *header = at<float>(bvh, L.header);
    uint64_t *keys = at<uint64_t>(bvh, L.keys);
    uint32_t *perm = at<uint32_t>(bvh, L.perm);
    uint64_t *keys_tmp = at<uint64_t>(ws, W.keys_tmp);
    uint32_t *vals_tmp = at<uint32_t>(ws, W.vals_tmp);
    const SortPlan plan = sort_plan(n);
    const SortTables tb{at<uint32_t>(ws, W.before), at<uint32_t>(ws, W.totals), plan.tiles, plan.group};
    float *partial = at<float>(ws, W.bounds);

    const LeafArgs la = leaf_args(g, bvh, L, ws, W);
    if (n <= 2 * kSortThreads)
        hipLaunchKernelGGL(k_sort_small<2>, dim3(1), dim3(kSortThreads), 0, s, g->mean, (int)n, header, keys, perm);
    else if (n <= 4 * kSortThreads)
        hipLaunchKernelGGL(k_sort_small<4>, dim3(1), dim3(kSortThreads), 0, s, g->mean, (int)n, header, keys, perm);
    else if (n <= kSmallSort)
        hipLaunchKernelGGL(k_sort_small<8>, dim3(1), dim3(kSortThreads), 0, s, g->mean, (int)n, header, keys, perm);
    else if (plan.items == 1)
        launch_sort<1>(la, n, partial, header, keys, perm, keys_tmp, vals_tmp, tb, s);
    else if (plan.items == 2)
        launch_sort<2>(la, n, partial, header, keys, perm, keys_tmp, vals_tmp, tb, s);
    else if (plan.items == 4)
        launch_sort<4>(la, n, partial, header, keys, perm, keys_tmp, vals_tmp, tb, s);
    else
        launch_sort<8>(la, n, partial, header, keys, perm, keys_tmp, vals_tmp, tb, s);
    rv_status st = check_launch("morton / radix sort");
    if (st != RV_OK) return st;

    const unsigned blocks = grid_for(n, kBoxBlock);
    auto leaves = la.packed ? k_leaves_karras<false, true> : k_leaves_karras<false, false>;
    hipLaunchKernelGGL(leaves, dim3(2 * blocks), dim3(kBoxBlock), 0, s, la, n, (const float *)nullptr, 0, header, keys,
                       at<float4>(ws, W.topo), at<int32_t>(bvh, L.parent));
    launch_refit(n, la, false, at<float4>(ws, W.topo), at<float>(ws, W.node_box), at<float4>(bvh, L.nodes), header,
                 at<float>(bvh, L.nodes4), s);
    return check_launch("leaf records / karras / refit");
}

extern "C" rv_status rv_refit_bvh(const rv_gaussians *g, void *bvh, size_t bvh_bytes, void *ws, size_t ws_bytes,
                                  void *stream) {
    clear_error();
    RV_REQUIRE(g && bvh && ws, RV_ERR_INVALID_ARG, "rv_refit_bvh: null argument (g, bvh or ws)");
    RV_REQUIRE(g->mean && g->quat && g->log_scale && g->opacity, RV_ERR_INVALID_ARG,
               "rv_refit_bvh: null Gaussian array");
    const int64_t n = g->n;
    RV_REQUIRE(n >= 1 && n <= RV_MAX_GAUSSIANS, RV_ERR_INVALID_ARG, "rv_refit_bvh: n=%lld out of range",
               (long long)n);
    RV_REQUIRE(((uintptr_t)bvh % kAlign) == 0 && ((uintptr_t)ws % kAlign) == 0, RV_ERR_INVALID_ARG,
               "rv_refit_bvh: bvh and ws must be 256-byte aligned");
    const BvhLayout L = bvh_layout(n);
    const BuildWsLayout W = build_ws_layout(n);
    RV_REQUIRE(bvh_bytes >= L.total, RV_ERR_WORKSPACE, "rv_refit_bvh: bvh_bytes %zu < %zu", bvh_bytes, L.total);
    RV_REQUIRE(ws_bytes >= W.total, RV_ERR_WORKSPACE, "rv_refit_bvh: ws_bytes %zu < %zu", ws_bytes, W.total);
    hipStream_t s = (hipStream_t)stream;
    float *header = at<float>(bvh, L.header);
    float *partial = at<float>(ws, W.bounds);
    // the scene scale of the leaf widening follows the moved means; the sorted
    // order, keys and topology stay as built
    const LeafArgs la = leaf_args(g, bvh, L, ws, W);
    const int nparts = bounds_blocks(n);
    hipLaunchKernelGGL(k_bounds, dim3(nparts), dim3(1024), 0, s, la.in, n, partial, const_cast<float4 *>(la.packed));
    auto leaves = la.packed ? k_leaves_karras<true, true> : k_leaves_karras<true, false>;
    hipLaunchKernelGGL(leaves, dim3(grid_for(n, kBoxBlock)), dim3(kBoxBlock), 0, s, la, n, partial, nparts, header,
                       (const uint64_t *)nullptr, (float4 *)nullptr, (int32_t *)nullptr);
    launch_refit(n, la, true, at<float4>(ws, W.topo), at<float>(ws, W.node_box), at<float4>(bvh, L.nodes), header,
                 at<float>(bvh, L.nodes4), s);
    return check_launch("rv_refit_bvh");
}
