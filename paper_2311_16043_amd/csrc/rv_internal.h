// rv_internal.h -- shared layout, error reporting and device helpers of the
// gfx950 visibility library (internal; the public ABI is include/rvis.h).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <string>

#include "rvis.h"

namespace rv {

// ---------------------------------------------------------------------------
// error reporting
// ---------------------------------------------------------------------------
void set_error(const char *fmt, ...);
void clear_error();

#define RV_REQUIRE(cond, code, ...)      \
    do {                                 \
        if (!(cond)) {                   \
            ::rv::set_error(__VA_ARGS__); \
            return (code);               \
        }                                \
    } while (0)

// Check the launch that was just enqueued.
rv_status check_launch(const char *what);

// ---------------------------------------------------------------------------
// BVH blob layout (byte offsets, every section 256-byte aligned)
// ---------------------------------------------------------------------------
constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) & ~(kAlign - 1); }

// Half-width of the leaf boxes in standard deviations (3-sigma support).
constexpr float kBuildSigma = 3.0f;
// Header floats: lo[3], hi[3] of the means; root box lo[3], hi[3]; n (as float bits) ...
constexpr int kHeaderFloats = 16;

// Bytes per compressed four-wide node (48 used).
constexpr size_t kNode4Bytes = 64;
// Leaf record, three float4 per sorted leaf: (mu, opacity), (W row 0,
// s0 s1 / s2), (W row 1, source index bits); W row 2 = (s0 s1 / s2) (row 0 x row 1).
constexpr int kLeafF4 = 3;

struct BvhLayout {
    size_t header, keys, perm, nodes, parent, leaf_rec, leaf_box, origins, nodes4, total;
};

inline BvhLayout bvh_layout(int64_t n) {
    BvhLayout L{};
    size_t nn = (size_t)(n > 0 ? n : 1);
    size_t off = 0;
    L.header = off; off = align_up(off + kHeaderFloats * sizeof(float));
    L.keys = off; off = align_up(off + nn * 8);
    L.perm = off; off = align_up(off + nn * 4);
    L.nodes = off; off = align_up(off + (nn > 1 ? nn - 1 : 1) * 64);
    L.parent = off; off = align_up(off + (2 * nn - 1) * 4);
    L.leaf_rec = off; off = align_up(off + nn * 16 * kLeafF4);
    L.leaf_box = off; off = align_up(off + nn * 24);
    L.origins = off; off = align_up(off + nn * 16);
    L.nodes4 = off; off = align_up(off + (nn > 1 ? nn - 1 : 1) * kNode4Bytes);
    L.total = off;
    return L;
}

// Radix sort: seven 9-bit digits of the 63-bit keys.
constexpr int kDigitBits = 9, kDigits = 1 << kDigitBits, kPasses = 7;
static_assert(kDigitBits * kPasses == 63, "the passes must cover the keys");
constexpr int kSortThreads = 1024;
// Up to this many Gaussians one block sorts in LDS. The whole build so / by tiles:
// 45 / 78 us at 2,000, 82 / 100 us at 8,000; beyond, the single CU's ranking
// outweighs the fourteen launches saved.
constexpr int64_t kSmallSort = 8 * kSortThreads;
// Tiles of kSortThreads items each thread `items`, counted in groups of `group`
// tiles. Small tiles spread the sort over more CUs, large ones write longer runs
// and read fewer totals (every tile reads those of all groups). Build in us with
// 1 / 2 items: 97 / 102 at 12,000, 114 / 119 at 100,000, 141 / 142 at 200,000,
// 187 / 167 at 300,000; with 2 / 4 / 8: 202 / 219 / 300 at 520,000,
// 328 / 308 / 392 at 1M, 926 / 844 / 851 at 3M, 1,452 / 1,331 / 1,295 at 5M.
struct SortPlan {
    int items, group;
    int64_t tiles;
};
inline SortPlan sort_plan(int64_t n) {
    SortPlan p;
    p.items = n <= (int64_t(1) << 17) ? 1 : n <= (int64_t(3) << 18) ? 2 : n <= (int64_t(1) << 22) ? 4 : 8;
    p.tiles = (n + (int64_t)kSortThreads * p.items - 1) / ((int64_t)kSortThreads * p.items);
    p.group = p.items <= 4 ? 4 : 8;
    while ((p.tiles + p.group - 1) / p.group > 256) p.group *= 2;
    return p;
}

// Blocks of the means' bounds.
constexpr int kBoundsBlocks = 512;

// Leaves and nodes per block of the leaf, node and refit kernels; the leaves of
// one such block are the largest group of the box pyramid.
constexpr int kBoxBlock = 512;
// Sorted keys, and leaf boxes, held in LDS around a block of nodes.
constexpr int kKeyWindow = 3 * kBoxBlock, kBoxWindow = 2 * kBoxBlock;
// Largest power-of-two window of leaf boxes that a block of nodes builds.
constexpr int kTopWindow = 8;
// Above kPackFrom Gaussians the inputs of a leaf are gathered from packed records,
// written while the means are read for their bounds: one 64-byte line in the
// place of five partly used ones. Unpacked / packed: refit of 1.2M 211 / 178 us,
// build of 300,000 169 / 167 us, of 130,000 123 / 125 us (the inputs then fit
// the L2s). Above kPackTo (a scene of 20 GB with its tree) the records' memory counts
// more.
constexpr int64_t kPackFrom = int64_t(1) << 18, kPackTo = int64_t(1) << 26;
inline bool packs_inputs(int64_t n) { return n > kPackFrom && n <= kPackTo; }

// Bytes per Gaussian: 43.4, with packed inputs 83.4 (the sort alone needs 12.6). The
// topology is written once the sort has ended, and the node boxes once every leaf is
// prepared, so each shares the bytes of what is dead by then.
struct BuildWsLayout {
    size_t keys_tmp, vals_tmp, before, totals;   // sort; from keys_tmp on
    size_t topo;
    size_t packed;                               // inputs of the leaves, and from there on
    size_t node_box;
    size_t bounds, box8, box64, box512, total;
};

inline BuildWsLayout build_ws_layout(int64_t n) {
    BuildWsLayout W{};
    size_t nn = (size_t)(n > 0 ? n : 1);
    const SortPlan plan = sort_plan((int64_t)nn);
    size_t off = 0;
    W.keys_tmp = W.topo = off; off = align_up(off + nn * 8);
    W.vals_tmp = off; off = align_up(off + nn * 4);
    W.before = off; off = align_up(off + (size_t)plan.tiles * kDigits * 4);
    W.totals = off; off = align_up(off + (size_t)((plan.tiles + plan.group - 1) / plan.group) * kDigits * 4);
    off = std::max(off, align_up(W.topo + nn * 16));
    W.packed = W.node_box = off;
    off = align_up(off + nn * (packs_inputs((int64_t)nn) ? 64 : 6 * sizeof(float)));
    W.bounds = off; off = align_up(off + kBoundsBlocks * 6 * sizeof(float));
    W.box8 = off; off = align_up(off + (nn + 7) / 8 * 6 * sizeof(float));
    W.box64 = off; off = align_up(off + (nn + 63) / 64 * 6 * sizeof(float));
    W.box512 = off; off = align_up(off + (nn + 511) / 512 * 6 * sizeof(float));
    W.total = off;
    // a workspace that holds n Gaussians holds fewer as well
    if (n > kPackTo) W.total = std::max(W.total, build_ws_layout(kPackTo).total);
    return W;
}

template <typename T>
inline T *at(void *base, size_t off) { return reinterpret_cast<T *>(static_cast<char *>(base) + off); }
template <typename T>
inline const T *at(const void *base, size_t off) {
    return reinterpret_cast<const T *>(static_cast<const char *>(base) + off);
}

// ---------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------
struct f3 {
    float x, y, z;
};
__device__ __forceinline__ f3 mk(float x, float y, float z) { return f3{x, y, z}; }
__device__ __forceinline__ f3 operator-(f3 a, f3 b) { return mk(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ f3 operator+(f3 a, f3 b) { return mk(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ __forceinline__ f3 operator*(float s, f3 a) { return mk(s * a.x, s * a.y, s * a.z); }
__device__ __forceinline__ float dot(f3 a, f3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ f3 cross(f3 a, f3 b) {
    return mk(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

constexpr int kXcds = 8;

// Renumber blocks so that the blocks dispatched to XCD x (b % 8 == x) form a
// contiguous range of logical blocks. A bijection on [0, nb).
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb) {
    const int64_t q = nb / kXcds, r = nb % kXcds;
    const int64_t x = b % kXcds;
    return x * q + (x < r ? x : r) + b / kXcds;
}

// Header word 12 of a BVH blob holds the number of Gaussians it was built
// over. Every kernel that reads a tree compares it with the caller's n before
// touching anything else in the blob (the section offsets follow from n), so a
// blob built for another Gaussian set is never walked: traversals give NaN and
// a refit leaves the blob as it was.
__device__ __forceinline__ bool tree_matches(const float *__restrict__ header, int64_t n) {
    return __float_as_int(header[12]) == (int)(n & 0x7fffffff);
}

}  // namespace rv
