// trace.hip -- visibility pre-computation (Sec. 4.2): for every Gaussian i and
// direction k, the transmittance of the ray leaving mean_i (Sec. 4.1), and the
// per-Gaussian average over the K directions (the "averaged visibility" of the
// ablation study, Sec. 5.4).
//
// Work mapping. Rays come in pools (see the pooled traversal below): 64
// Gaussians adjacent in Morton (sorted-leaf) order times one direction for the
// all-ray kernels (the forward, which also serves the SH projection, and the
// adjoint), and 64 or 256 consecutive entries for the list kernel. In small
// launches every wave takes one pool; in larger ones a persistent grid takes them from
// eight queues, one per XCD (see Route). In the largest each queue is a
// contiguous eighth of the Morton order, so each L2 sees a compact part of the
// tree; a wave whose queue is spent takes pools from the others, so no XCD
// idles while another still holds work. A wave keeps its lanes supplied
// across pool boundaries, refilling idle lanes a dozen at a time, so the
// skewed per-ray work leaves lanes idle mainly in a wave's last pool. Each ray writes
// its own T; per-Gaussian means are FP64 row sums in a fixed order
// (deterministic, no atomics).
#include <atomic>
#include <mutex>
#include <type_traits>

#include "trace_core.h"

namespace rv {
namespace {

constexpr int kWavesPerBlock = kTraceBlock / 64;

// ---- pooled traversal -----------------------------------------------------------
//
// A wave drains pools of rays (64 Gaussians adjacent in sorted order times
// some directions, or consecutive list entries). Lanes that have no ray take
// the pool's next rays (ballot + popcount). Each iteration, lanes with
// traversal work and room in their leaf FIFO visit one node, appending pairs of
// hit leaves instead of testing them; the leaf test then runs as one block for
// all lanes with a pending leaf once enough of them have one, so the
// expensive exact test executes with most lanes active instead of inside
// every node step. Leaves are tested in discovery (FIFO) order, so each ray's
// product, and its early exit, do not depend on which pool the ray was drained
// from: the all-ray, ray-list, SH and adjoint paths give a ray the same bits.
//
// A filled chip is bound by two things at once: the vector-memory path returns
// about one 16-byte lane load per CU and cycle (340 a ray at 300,000 Gaussians),
// and the SIMDs issue instructions in nearly nine of ten cycles. Stacks and queues
// of pairs and the byte-permuted planes took the instructions of a wave's
// iteration from 321 to 275 (40.6 -> 39.8 ms at 300,000 x 256, 77.2 -> 68.0 ms at
// 3M x 16 together with the grid sizes below). Records fetched by the quad through
// LDS made a third of the vector-L1 accesses and ran slower (44.9 ms for the nodes,
// 49.0 for the leaves, 50.0 for both): direct loads into LDS return no faster, and
// their addresses are more instructions.
//
// Entries of a queued list pool, in waves.
constexpr int kPoolS = 4;
// Stack entries per lane in LDS (24 KB per block with the FIFO): with 16 fewer deep
// entries go to the private spill array than with 8 (39.8 against 40.5 ms at object
// scale).
constexpr int kStreamRing = 16;
// Directions per pool of the persistent all-ray kernel. With one, the pools
// in flight on an XCD cover the fewest Gaussians (about 256 against 1,024
// with four directions), and the tree they touch is most compact: 53.5 ms
// against 53.7 with two and 54.5 with four at object scale.
constexpr int kStreamPoolS = 1;
constexpr int kLeafMin = 32;
// Resident blocks per CU of the persistent traversal. Its waves share the CU's
// vector-memory path, which they keep full, and the caches: more of them only thin
// those out, and with few pools they also end further apart. 5 / 4 / 3 blocks:
// 40.0 / 42.0 / 50.3 ms at 300,000 Gaussians x 256; 4.48 / 4.76 / 5.44 ms at
// 100,000 x 128, 1.16 / 1.17 / 1.23 ms at 50,000 x 64, 774 / 744 / 743 us at
// 30,000 x 64 (six: 43.8 ms at 300,000 x 256; all by XcdQueue). On large trees the fewer
// directions a Gaussian has, the more Gaussians the pools in flight cover, and the
// tree they touch outgrows the L2: 5 / 4 blocks on one surface of 3M Gaussians 110 / 94 ms
// x 16, 407 / 353 x 64 and 1,621 / 1,407 x 256, of 1.2M 173 / 156 x 128 and 686 / 625 x 512; in
// 20 objects of 150,000 46.3 / 44.8 x 16, 168.4 / 169.9 x 64, 327 / 334 x 128, 643 / 664 x 256 and
// 2,525 / 2,651 x 1,024 (six: 2,820). Nothing that the host knows tells one surface from
// many objects; the line leaves the many directions of a composition's
// pre-computation five blocks, at the price of one large surface's.
constexpr int kStreamBlocksPerCu = 5, kStreamBlocksDeep = 4, kStreamBlocksFew = 3;
constexpr int64_t kFewPools = 40000, kDeepStreamGaussians = int64_t(1) << 20;
constexpr int kDeepStreamDirs = 96;

// How a launch's waves come to their pools. The counters of XcdQueue, on few lines,
// serve about one wave in 50 ns, and every wave adds to all eight to find them spent.
//   kOnePool  every wave takes one pool and the hardware hands out the blocks; the
//             lanes of a wave idle towards its end, and so do waves until their
//             block's last has ended.
//   kDealt    a persistent grid takes the pools from DealQueue.
//   kQueues   a persistent grid takes the pools from XcdQueue.
// kOnePool / kDealt in us, hemisphere directions: surfaces 79 / 85 at 1,000 Gaussians x 600
// (9,600 pools), 207 / 172 at 10,000 x 64, 256 / 200 at 14,264 x 51, 468 / 343 at 20,000 x 64;
// clouds 724 / 709 at 9,444 x 68, 1,471 / 1,149 at 12,000 x 100, and where a ray crosses
// hundreds of Gaussians (a tenth as opaque, standard deviations 0.07 to 0.37 of a side
// of 2) 16.5 / 15.4 ms at 12,000 x 64 (17.1 by queues, six blocks per CU), 36.1 / 30.6 at
// 20,000 x 64 (32.5). With the same directions for all Gaussians every pool's rays run
// side by side, and neither wins: a cloud of 9,905 x 82 706 / 760, of 12,000 x 64 763 / 723. On up
// to 256 Gaussians rays are so short that even a counter each is in the way (150 / 212
// at 64 x 20,000), and a tree that outgrows the caches wants its pools in order
// (1,889 / 2,146 at 1.2M x 1). kDealt / kQueues: surfaces 390 / 422 at 24,000 x 64 and
// 599 / 715 at 30,000 x 64, but clouds 1,414 / 1,334 at 12,000 x 128 and, as above with
// deviations divided by e, 20.1 / 17.4 ms at 30,000 x 64 (lanes taking rays after 2,048
// lane-iterations).
enum class Route { kOnePool, kDealt, kQueues };
constexpr int64_t kOnePoolWaves = 10000, kDealtPools = 24000, kFewGaussians = 256;
inline Route all_ray_route(int64_t n_pools, int64_t n, int dir_mode) {
    if (n_pools > kDealtPools) return Route::kQueues;
    const bool dealt = dir_mode == 1 && n_pools > kOnePoolWaves && n > kFewGaussians && n < kDeepStreamGaussians;
    return dealt ? Route::kDealt : Route::kOnePool;
}

// Visits that a walk makes at most between two looks at its budget (a malformed
// tree with a cycle ends then, with NaN).
constexpr uint32_t kBudgetLook = 64;

// Wave-level leaf phase condition: enough lanes hold a pending leaf, or some
// lane cannot walk for lack of FIFO room, or no lane can walk.
template <int kRing>
__device__ __forceinline__ bool leaf_phase_now(const Walk<kRing> &wk) {
    const uint64_t pend = __ballot(wk.queued());
    const uint64_t blocked = __ballot(!wk.room());
    const uint64_t trav = __ballot(wk.can_walk());
    return pend != 0 && (__popcll(pend) >= kLeafMin || blocked != 0 || trav == 0);
}

// One ray as a pool source hands it out.
struct RaySetup {
    f3 o, d;
    float tmin;
    int32_t self;       // original index of the source Gaussian
    int32_t self_leaf;  // its sorted leaf position, or -1 if not known
    bool valid;         // false: not a ray of this scene (finishes at once with NaN)
    int64_t out;        // output position of its T
};

// Pools handed to one wave. XcdQueue: the pools are cut into kXcds
// contiguous ranges, one per XCD, each drained one pool at a time through an
// atomic counter (zero at launch; kQueueStride words apart, as two on one line
// slow each other down). A wave takes from its own XCD's range
// first, so that adjacent Gaussians share that XCD's L2; once the range is
// spent it takes from the other ranges in turn, so no XCD idles while another
// still holds work.
// DealQueue: the pools are dealt to the XCDs in chunks of kChunk consecutive ones, with
// a counter each; a wave's first pool follows from its place in the grid, and it
// leaves once its XCD's pools are spent. Chunks this small share a launch out as
// evenly as taking from other ranges does, and a wave adds to one counter at its
// end instead of to eight.
// RangeQueue: a fixed run of consecutive pools.
constexpr int kQueueStride = 4;   // the eight counters fill 256 bytes
struct XcdQueue {
    unsigned long long *ctrs;  // kXcds counters
    int64_t n_pools;
    int home, turn;  // the range being drained is (home + turn) % kXcds
    __device__ __forceinline__ void init(unsigned long long *c, int64_t np, uint32_t block, uint32_t) {
        ctrs = c;
        n_pools = np;
        home = (int)(block % kXcds);
        turn = 0;
    }
    // Next pool in p, false once every range is spent. Called in wave-uniform
    // control flow; the first active lane takes the pool for the wave.
    __device__ __forceinline__ bool take(int64_t &p) {
        const int lane = threadIdx.x & 63;
        while (turn < kXcds) {
            const int x = (home + turn) % kXcds;
            unsigned long long t = 0;
            if (lane == __builtin_amdgcn_readfirstlane(lane)) t = atomicAdd(ctrs + kQueueStride * x, 1ull);
            const uint32_t tl = __builtin_amdgcn_readfirstlane((uint32_t)t);
            const uint32_t th = __builtin_amdgcn_readfirstlane((uint32_t)(t >> 32));
            p = n_pools * x / kXcds + (int64_t)(((uint64_t)th << 32) | tl);
            if (p < n_pools * (x + 1) / kXcds) return true;
            ++turn;
        }
        return false;
    }
};

template <uint32_t kChunk>
struct DealQueue {
    unsigned long long *ctr;
    int64_t n_pools;
    uint32_t xcd, own, held;   // of its XCD's pools: the wave's first; how many are a wave's first
    __device__ __forceinline__ void init(unsigned long long *c, int64_t np, uint32_t block, uint32_t blocks) {
        xcd = block % kXcds;
        ctr = c + kQueueStride * xcd;
        n_pools = np;
        own = block / kXcds * kWavesPerBlock + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        held = blocks / kXcds * kWavesPerBlock;
    }
    __device__ __forceinline__ bool take(int64_t &p) {
        uint32_t t = own;
        if (t < held) {
            own = held;
        } else {
            const int lane = threadIdx.x & 63;
            if (lane == __builtin_amdgcn_readfirstlane(lane)) t = held + (uint32_t)atomicAdd(ctr, 1ull);
            t = __builtin_amdgcn_readfirstlane(t);
        }
        const uint32_t round = t / kChunk;
        p = (int64_t)((round * kXcds + (xcd + round) % kXcds) * kChunk + t % kChunk);
        return p < n_pools;
    }
};

// The XCDs' turns shift by one from round to round: in a fixed order an XCD meets the
// same part of every Gaussian's directions (5,000 x 256 292 / 269 us). Chunks of 4 to 128
// pools take the same time so.
using RayDeal = DealQueue<64>;

struct RangeQueue {
    int64_t next, end;
    __device__ __forceinline__ bool take(int64_t &p) {
        p = next++;
        return p < end;
    }
};

// When a wave's lanes without a ray take new ones: always once no lane has a ray;
// else on a filled chip once c.refill lanes are idle, so that the ray setup runs for
// several lanes at a time.
template <class Queue>
struct Refill {
    __device__ __forceinline__ bool now(uint64_t idle, int lanes) { return __popcll(idle) >= lanes || ~idle == 0; }
    __device__ __forceinline__ void loaded(uint64_t, f3) {}
};
// From a RayDeal as the rays ask for. Rays of one pool that run side by side share
// lines, and few of them are long: mixed with another pool's they share less, and the
// long ones, which a small launch ends with, advance at the pace of a full wave. So a
// wave whose lanes took like directions waits until no lane has a ray. Rays in all
// directions share little and are long where the scene is dense: there lanes take new
// ones once the idle ones have cost as much as sixteen iterations of the wave.
// Waiting / with 1,024 / 2,048 / 4,096 idle lane-iterations, in us: surfaces 134 / 162 / 135 / 134
// at 5,000 Gaussians x 128, 362 / - / 471 / 367 at 14,824 x 89; clouds in hemispheres about
// random normals 1,390 / 1,149 / 1,266 / 1,330 at 12,000 x 100, 1,980 / 1,555 / 1,693 / 1,750 at
// 20,000 x 64 and, with deviations as under Route divided by e, 5.5 / 4.7 / 4.8 / 4.7 ms at
// 12,000 x 64.
template <>
struct Refill<RayDeal> {
    static constexpr int kIdleMost = 1024;
    int idled = 0;
    bool alike = true;   // the rays last taken run side by side
    __device__ __forceinline__ bool now(uint64_t idle, int) {
        idled += __popcll(idle);
        if ((alike || idled < kIdleMost) && ~idle != 0) return false;
        idled = 0;
        return true;
    }
    // The lanes that took a ray of direction d. Of rays in all directions every
    // fourth pair lies within 60 degrees; few lanes say nothing.
    __device__ __forceinline__ void loaded(uint64_t lanes, f3 d) {
        auto other = [](float x) {   // of the next lane or the one before
            return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xb1, 0xf, 0xf, false));
        };
        const uint64_t pairs = lanes & (((lanes >> 1) & 0x5555555555555555ull) | ((lanes & 0x5555555555555555ull) << 1));
        const int close = __popcll(__ballot(dot(d, mk(other(d.x), other(d.y), other(d.z))) > 0.5f) & pairs);
        const int n = __popcll(pairs);
        if (n >= 32) alike = 8 * close >= 5 * n;
    }
};

// Trace the rays of the pools the queue hands out with the lanes of one
// wave. With kAhead the words of a lane's next node are fetched as soon as the
// node is known, while leaves are tested: for launches that leave the chip's
// memory path idle (5,000 Gaussians x 33: 202 against 210 us; a filled chip runs up
// to 5 % slower so). Lanes without a ray
// take the next rays of the current pool (see Refill); when the pool is spent the
// wave takes the next pool at once, so lanes stay supplied across pool
// boundaries. A finished
// ray writes its T to out[r.out] (when out is given). stk and my_fifo are
// this lane's columns of the block's LDS stack ring and leaf FIFO.
template <bool kCount, bool kAhead, class Queue, class Pools>
__device__ __forceinline__ void stream_rays(const float4 *__restrict__ nodes4, const float4 *__restrict__ rec,
                                            const Cuts &c, int64_t n, Queue &queue, Pools &pools,
                                            Pair *stk, Pair *my_fifo, float *__restrict__ out, int64_t &cn,
                                            int64_t &cl, int64_t &ch) {
    const int lane = threadIdx.x & 63;
    const uint64_t lt = (1ull << lane) - 1ull;
    Walk<kStreamRing> wk;
    Pair spill[Walk<kStreamRing>::kSpill];
    wk.init(stk, my_fifo, spill);
    int64_t dst = 0;  // output position of the current ray
    RayBox rb;
    rb.set(mk(0.f, 0.f, 0.f), mk(0.f, 0.f, 0.f));
    f3 d = mk(0.f, 0.f, 0.f);
    float tmin = 0.f, T = 1.f;
    int32_t self = -1, self_leaf_m1 = -2;
    NoHit none;
    uint4 ahead[3] = {};   // kAhead: the words of wk.node
    auto node_words = [&](uint4 (&w)[3]) {
        const uint4 *r = reinterpret_cast<const uint4 *>(nodes4) + 4 * (int64_t)wk.node + 4;
#pragma unroll
        for (int k = 0; k < 3; ++k) w[k] = r[k];
    };
    // wave-uniform pool state
    int next = 0, pool_n = 0;
    bool more = true;
    Refill<Queue> refill;

    for (uint32_t round = 1;; ++round) {
        // refill idle lanes, moving on to further pools while lanes are idle
        uint64_t need = __ballot(wk.idle());
        if (!refill.now(need, c.refill)) need = 0;
        const uint64_t empty = need;
        while (need != 0 && more) {
            if (next >= pool_n) {
                int64_t p;
                more = queue.take(p);
                pool_n = more ? pools.open(p) : 0;
                next = 0;
                continue;
            }
            const int idx = next + __popcll(need & lt);
            if (wk.idle() && idx < pool_n) {
                const RaySetup r = pools(idx);
                d = r.d;
                rb.set(r.o, d);
                tmin = r.tmin;
                self = r.self;
                self_leaf_m1 = r.self_leaf - 1;
                T = r.valid ? 1.0f : __int_as_float(0x7fc00000);
                wk.start(n, r.valid);
                if (kAhead && wk.node > Walk<kStreamRing>::kDone) node_words(ahead);
                dst = r.out;
            }
            next += __popcll(need);
            need = __ballot(wk.idle());
        }
        if (empty != 0) refill.loaded(empty & ~need, d);
        if (__ballot(!wk.idle()) == 0) break;  // queue spent, every ray finished

        // node phase: one four-wide node per lane with traversal work and FIFO
        // room for the leaves of both sides
        if (wk.can_walk()) {
            if (kAhead) {
                wk.visit(ahead, rb, tmin, T);
                if (wk.node > Walk<kStreamRing>::kDone) node_words(ahead);
            } else {
                uint4 w[3];
                node_words(w);
                wk.visit(w, rb, tmin, T);
            }
            if (kCount) ++cn;
        }

        // leaf phase: test one pending leaf per lane when enough lanes have one,
        // when a lane cannot traverse for lack of FIFO room, or when no lane can traverse
        if (leaf_phase_now(wk)) {
            if (wk.queued()) {
                const int32_t m1 = wk.next_leaf();
                const float f = leaf_factor(rec, m1, rb.o, d, tmin, self, self_leaf_m1, c, none, T);
                if (kCount) {
                    ++cl;
                    ch += (f != 1.0f);
                }
                T *= f;
                if (T < c.T_stop) wk.stop();
            }
        }
        if (round % kBudgetLook == 0 && wk.budget < 0 && !wk.idle()) {
            T = __int_as_float(0x7fc00000);
            wk.stop();
        }

        if (wk.finished()) {
            if (out) out[dst] = T;
            wk.node = Walk<kStreamRing>::kIdle;
        }
    }
}

// Rays of the all-ray kernel: Gaussians m0 .. m0 + nv - 1 (sorted order) times
// directions k0 .. k0 + s - 1; pool index idx = j * nv + (m - m0). Origin data
// come from the prepared per-leaf records. The output position of ray
// (i, k) is i * K + k with i the Gaussian's original index.
struct GridSource {
    const float4 *rec, *origins;
    const float *dirs;
    int64_t m0;
    int nv, k0, dir_mode;
    float tmin_scale;
    float inv_nv;  // reciprocal of nv (within one ulp)
    int K = 0;
    // output position: i * K + k (by_leaf false), or (m - m_lo) * K + k with m
    // the Gaussian's sorted position (by_leaf true: rows of a batch)
    bool by_leaf = false;
    int64_t m_lo = 0;
    __device__ __forceinline__ RaySetup operator()(int idx) const {
        // idx / nv from the float quotient: (idx + 1/2) / nv lies at least
        // 1/(2 nv) >= 1/128 from an integer, far beyond its rounding error
        // (idx < 2^9: below 2^9 2^-22)
        const int j = (int)(((float)idx + 0.5f) * inv_nv);
        const int oi = idx - j * nv;
        const int64_t m = m0 + oi;
        const float4 r0 = rec[kLeafF4 * m];
        const float4 og = origins[m];
        const f3 nrm = mk(og.x, og.y, og.z);
        f3 b1, b2;
        onb_duff(nrm, b1, b2);
        RaySetup r;
        r.o = mk(r0.x, r0.y, r0.z);
        r.d = ray_direction(dirs, k0 + j, dir_mode, nrm, b1, b2);
        r.tmin = tmin_scale * og.w;
        r.self = __float_as_int(rec[kLeafF4 * m + 2].w);
        r.self_leaf = (int32_t)m;
        r.valid = true;
        r.out = (by_leaf ? m - m_lo : (int64_t)r.self) * K + k0 + j;
        return r;
    }
};

// All-ray pools: pool p = group * n_chunks + chunk covers the 64 Gaussians
// of the group (sorted order, groups counted from m_lo) times the chunk's
// kStreamPoolS directions.
struct GridPools : GridSource {
    int64_t m_hi;  // the pools cover sorted positions [m_lo, m_hi)
    int n_chunks;
    // Make pool p current; returns its number of rays.
    __device__ __forceinline__ int open(int64_t p) {
        const int64_t grp = p / n_chunks;
        const int chunk = (int)(p - grp * n_chunks);
        m0 = m_lo + grp * 64;
        nv = (int)min<int64_t>(64, m_hi - m0);
        inv_nv = __builtin_amdgcn_rcpf((float)nv);
        k0 = chunk * kStreamPoolS;
        return nv * min(kStreamPoolS, K - k0);
    }
};

// Rays given by id r = ids[base + idx] + id_offset = i * K + k. Origin data are
// recomputed from the input arrays with the same operations as the leaf
// preparation, so a ray gets the same bits as in the all-ray kernel.
struct ListSource {
    const float *mean, *normal, *log_scale, *dirs;
    int64_t n;
    int K, dir_mode;
    float tmin_scale;
    const int64_t *ids;
    int64_t id_offset, base;
    double inv_k;  // 1 / K
    bool out_by_value;
    bool tree_ok;  // the tree was built over these n Gaussians (else every ray is NaN)
    __device__ __forceinline__ RaySetup operator()(int idx) const {
        RaySetup r;
        const int64_t entry = ids[base + idx];
        const int64_t rid = entry + id_offset;
        r.out = out_by_value ? entry : base + idx;
        r.valid = tree_ok && rid >= 0 && rid < n * (int64_t)K;
        // rid / K from the FP64 quotient (off by at most one for rid < 2^52,
        // where rid converts exactly), corrected so that 0 <= k < K; integer
        // division beyond
        int64_t i = !r.valid ? 0 : rid < (int64_t(1) << 52) ? (int64_t)((double)rid * inv_k) : rid / K;
        int64_t k64 = r.valid ? rid - i * K : 0;
        if (k64 < 0) {
            --i;
            k64 += K;
        } else if (k64 >= K) {
            ++i;
            k64 -= K;
        }
        const int k = (int)k64;
        float nx = 0.f, ny = 0.f, nz = 1.f;
        if (normal) {
            nx = normal[3 * i]; ny = normal[3 * i + 1]; nz = normal[3 * i + 2];
            const float nl = sqrtf(nx * nx + ny * ny + nz * nz);
            nx /= nl; ny /= nl; nz /= nl;
        }
        const float smax = expf(fmaxf(log_scale[3 * i], fmaxf(log_scale[3 * i + 1], log_scale[3 * i + 2])));
        const f3 nrm = mk(nx, ny, nz);
        f3 b1, b2;
        onb_duff(nrm, b1, b2);
        r.o = mk(mean[3 * i], mean[3 * i + 1], mean[3 * i + 2]);
        r.d = ray_direction(dirs, r.valid ? k : 0, dir_mode, nrm, b1, b2);
        r.tmin = tmin_scale * smax;
        r.self = (int32_t)i;
        r.self_leaf = -1;
        return r;
    }
};

// List pools: pool p covers the kEntries list entries from p * kEntries.
template <int kEntries>
struct ListPools : ListSource {
    int64_t total;
    __device__ __forceinline__ int open(int64_t p) {
        base = p * kEntries;
        return (int)min<int64_t>(kEntries, total - base);
    }
};

// The rays of the Gaussians at sorted positions [m_lo, m_hi) (all n K rays
// for [0, n)): with kOnePool one pool per wave (consecutive blocks of pools on one
// XCD), else through per-XCD queues of pools. The grid of the latter is persistent (a
// multiple of 8 blocks, about what the device holds at once) and block b
// serves the queue of XCD b % 8 (round-robin dispatch). With kQueues its range is a
// contiguous eighth of the pools: each L2 sees a compact part of the tree
// until its range is spent and its waves help with the other ranges.
template <bool kCount, Route kRoute>
__global__ __launch_bounds__(kTraceBlock, kStreamBlocksPerCu) void k_trace_stream(const float *__restrict__ header,
                                                              const float4 *__restrict__ nodes4,
                                                              const float4 *__restrict__ rec,
                                                              const float4 *__restrict__ origins,
                                                              const float *__restrict__ dirs, int64_t n, int K,
                                                              Cuts c, int64_t m_lo, int64_t m_hi, int by_leaf,
                                                              unsigned long long *__restrict__ queues,
                                                              float *__restrict__ vis_ray,
                                                              unsigned long long *__restrict__ totals) {
    __shared__ Pair stk[kStreamRing * kTraceBlock];
    __shared__ Pair fifo[kFifo * kTraceBlock];
    if (!tree_matches(header, n)) {
        // a tree built for another Gaussian set: every ray of the range is NaN
        if (vis_ray) {
            const int64_t rows = (m_hi - m_lo) * (int64_t)K;
            for (int64_t r = (int64_t)blockIdx.x * kTraceBlock + threadIdx.x; r < rows;
                 r += (int64_t)gridDim.x * kTraceBlock)
                vis_ray[r] = __int_as_float(0x7fc00000);
        }
        return;
    }
    GridPools pools;
    pools.rec = rec;
    pools.origins = origins;
    pools.dirs = dirs;
    pools.dir_mode = c.dir_mode;
    pools.tmin_scale = c.tmin_scale;
    pools.K = K;
    pools.by_leaf = by_leaf != 0;
    pools.m_lo = m_lo;
    pools.m_hi = m_hi;
    pools.n_chunks = (K + kStreamPoolS - 1) / kStreamPoolS;
    pools.m0 = 0;
    pools.nv = 1;
    pools.k0 = 0;
    pools.inv_nv = 1.0f;
    const int64_t n_pools = ((m_hi - m_lo + 63) / 64) * (int64_t)pools.n_chunks;
    int64_t cn = 0, cl = 0, ch = 0;
    if constexpr (kRoute == Route::kOnePool) {
        RangeQueue q;
        q.next = xcd_block(blockIdx.x, gridDim.x) * kWavesPerBlock + (threadIdx.x >> 6);
        q.end = min(n_pools, q.next + 1);
        stream_rays<kCount, true>(nodes4, rec, c, n, q, pools, stk + threadIdx.x, fifo + threadIdx.x, vis_ray, cn, cl,
                                  ch);
    } else {
        std::conditional_t<kRoute == Route::kDealt, RayDeal, XcdQueue> q;
        q.init(queues, n_pools, blockIdx.x, gridDim.x);
        stream_rays<kCount, kRoute == Route::kDealt>(nodes4, rec, c, n, q, pools, stk + threadIdx.x, fifo + threadIdx.x,
                                                     vis_ray, cn, cl, ch);
    }
    if (kCount) {
        atomicAdd(totals + 0, (unsigned long long)cn);
        atomicAdd(totals + 1, (unsigned long long)cl);
        atomicAdd(totals + 2, (unsigned long long)ch);
    }
}

// Listed rays. The list holds *count entries when count is given (read on the
// device), else n_list. out_by_value: T goes to out[ids[j]] (the list holds output
// positions, the ray being id_offset + ids[j]); otherwise to out[j]. With kDealt and
// kQueues the grid is persistent and takes pools of kPoolS * 64 entries, dealt or from
// per-XCD queues (each a contiguous eighth of the list, stealing from the others once
// its own is spent), through counters at queues (kQueueBytes, zero at launch). With
// kOnePool wave w takes the run of pools [w R, (w + 1) R) of 64 entries.
template <Route kRoute>
__global__ __launch_bounds__(kTraceBlock, kStreamBlocksPerCu) void k_trace_list(
    const float *__restrict__ header, const float4 *__restrict__ nodes4, const float4 *__restrict__ rec,
    const float *__restrict__ mean, const float *__restrict__ normal, const float *__restrict__ log_scale, int64_t n, const float *__restrict__ dirs,
    int K, Cuts c, const int64_t *__restrict__ ids, int64_t n_list, const unsigned long long *__restrict__ count,
    int64_t id_offset, int out_by_value, int64_t run, unsigned long long *__restrict__ queues,
    float *__restrict__ out) {
    __shared__ Pair stk[kStreamRing * kTraceBlock];
    __shared__ Pair fifo[kFifo * kTraceBlock];
    constexpr bool kQueue = kRoute != Route::kOnePool;
    constexpr int kPool = kQueue ? kPoolS * 64 : 64;
    const int64_t total = count ? min<int64_t>(n_list, (int64_t)*count) : n_list;
    const int64_t n_pools = (total + kPool - 1) / kPool;
    using Queue = std::conditional_t<!kQueue, RangeQueue,
                                     std::conditional_t<kRoute == Route::kDealt, DealQueue<16>, XcdQueue>>;
    Queue q;
    if constexpr (kQueue) {
        q.init(queues, n_pools, blockIdx.x, gridDim.x);
    } else {
        const int64_t w = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
        q.next = w * run;
        q.end = min(n_pools, q.next + run);
        if (q.next >= q.end) return;  // wave-uniform
    }
    ListPools<kPool> pools;
    pools.mean = mean;
    pools.normal = normal;
    pools.log_scale = log_scale;
    pools.dirs = dirs;
    pools.n = n;
    pools.K = K;
    pools.dir_mode = c.dir_mode;
    pools.tmin_scale = c.tmin_scale;
    pools.ids = ids;
    pools.id_offset = id_offset;
    pools.base = 0;
    pools.inv_k = 1.0 / (double)K;
    pools.out_by_value = out_by_value != 0;
    pools.total = total;
    pools.tree_ok = tree_matches(header, n);
    int64_t cn = 0, cl = 0, ch = 0;
    stream_rays<false, !kQueue>(nodes4, rec, c, n, q, pools, stk + threadIdx.x, fifo + threadIdx.x, out, cn, cl, ch);
}

// vis_mean[i] = (1/K) sum_k vis[i K + k]: one wave per Gaussian, FP64 lane
// sums over a fixed stride and a fixed butterfly (deterministic).
__global__ __launch_bounds__(256) void k_mean_rows(const float *__restrict__ vis, int64_t n, int K,
                                                   float *__restrict__ vis_mean) {
    const int lane = threadIdx.x & 63;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * 4) {
        const float *row = vis + i * K;
        double s = 0.0;
        for (int k = lane; k < K; k += 64) s += (double)row[k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) vis_mean[i] = (float)(s / (double)K);
    }
}

// ---- visibility compressed to SH ----------------------------------------------
//
// Each Gaussian's visibility over its K directions projected onto the real
// spherical harmonics of degree <= 2 (9 coefficients, the "3-level SH" of
// Sec. 3.3) by the quadrature of Eq. (10): v_ij = sum_k V_ik Y_j(d_k) dw, with
// d_k the table's unit directions in the rays' frame (local about the normal
// in hemisphere mode). No per-ray output reaches the caller: the Gaussians are
// traced in batches of consecutive sorted positions by the persistent all-ray
// kernel into a bounded buffer of rows, and each row is projected in FP64 in a
// fixed order (deterministic).
constexpr int kShCoef = 9;
// Per-ray values held per batch: at most 2^28 (1 GiB).
constexpr int64_t kShBatchRays = int64_t(1) << 28;

// Gaussians per batch: a multiple of 64, at least 64, at most n.
inline int64_t sh_batch(int64_t n, int K) {
    int64_t b = kShBatchRays / K / 64 * 64;
    b = std::max<int64_t>(b, 64);
    return std::min<int64_t>(b, n);
}

// Real SH of degree <= 2 at the unit direction of table entry k.
__device__ __forceinline__ void sh_of_dir(const float *__restrict__ dirs, int k, float (&Y)[kShCoef]) {
    float x = dirs[3 * k], y = dirs[3 * k + 1], z = dirs[3 * k + 2];
    const float inv = 1.0f / sqrtf(x * x + y * y + z * z);
    x *= inv; y *= inv; z *= inv;
    Y[0] = 0.28209479177387814f;
    Y[1] = 0.4886025119029199f * y;
    Y[2] = 0.4886025119029199f * z;
    Y[3] = 0.4886025119029199f * x;
    Y[4] = 1.0925484305920792f * x * y;
    Y[5] = 1.0925484305920792f * y * z;
    Y[6] = 0.31539156525252005f * (3.0f * z * z - 1.0f);
    Y[7] = 1.0925484305920792f * x * z;
    Y[8] = 0.5462742152960396f * (x * x - y * y);
}

// Y[k][j] = Y_j(d_k) for the K table directions.
__global__ __launch_bounds__(256) void k_sh_table(const float *__restrict__ dirs, int K, float *__restrict__ Y) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    float y[kShCoef];
    sh_of_dir(dirs, k, y);
#pragma unroll
    for (int j = 0; j < kShCoef; ++j) Y[k * kShCoef + j] = y[j];
}

// Rows m_lo .. m_lo + n_rows - 1 (sorted positions) of a traced batch: one
// wave per row adds T_k Y_j(d_k) and T_k over k in FP64, lanes over a fixed
// stride and a fixed butterfly; vis_sh and vis_mean go to the Gaussian's
// original index.
__global__ __launch_bounds__(256) void k_sh_rows(const float *__restrict__ rows, int64_t m_lo, int64_t n_rows, int K,
                                                 const float *__restrict__ Y, const float *__restrict__ header,
                                                 const float4 *__restrict__ rec, int64_t n, double dw,
                                                 float *__restrict__ vis_sh, float *__restrict__ vis_mean) {
    const int lane = threadIdx.x & 63;
    if (!tree_matches(header, n)) {
        // a tree built for another Gaussian set: NaN for the batch's rows,
        // placed by row (the batches together cover every Gaussian)
        for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n_rows; r += (int64_t)gridDim.x * 256) {
#pragma unroll
            for (int j = 0; j < kShCoef; ++j) vis_sh[(m_lo + r) * kShCoef + j] = __int_as_float(0x7fc00000);
            if (vis_mean) vis_mean[m_lo + r] = __int_as_float(0x7fc00000);
        }
        return;
    }
    for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < n_rows; r += (int64_t)gridDim.x * 4) {
        const float *row = rows + r * K;
        double acc[kShCoef + 1];
#pragma unroll
        for (int j = 0; j <= kShCoef; ++j) acc[j] = 0.0;
        for (int k = lane; k < K; k += 64) {
            const double t = (double)row[k];
#pragma unroll
            for (int j = 0; j < kShCoef; ++j) acc[j] += t * (double)Y[k * kShCoef + j];
            acc[kShCoef] += t;
        }
#pragma unroll
        for (int j = 0; j <= kShCoef; ++j)
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc[j] += __shfl_xor(acc[j], off);
        if (lane == 0) {
            const int64_t i = __float_as_int(rec[kLeafF4 * (m_lo + r) + 2].w);
#pragma unroll
            for (int j = 0; j < kShCoef; ++j) vis_sh[i * kShCoef + j] = (float)(acc[j] * dw);
            if (vis_mean) vis_mean[i] = (float)(acc[kShCoef] / (double)K);
        }
    }
}

// ---- adjoint ----------------------------------------------------------------
//
// The adjoint traces as the forward does. A hit leaves a record in the wave's LDS
// stage: the leaf and four floats, a = (dL/dalpha) alpha and the whitened vector e,
// from which all seven gradient terms of the hit follow. A full stage is added to
// accumulators of 32 bytes per Gaussian, eight lanes to a record, so that a record
// is one request; a second kernel applies what the terms of a Gaussian share
// (1 / opacity, W^T) and adds the results to the caller's arrays.
//
// The bound is the rate of device atomics: 20.9 G requests/s of up to 64 bytes, to
// whichever addresses and from any number of waves (single floats as many, so the
// seven terms one by one would take seven times as long). 200,000 x 128 with the
// forward's T (11.8 hits a ray) takes 15.0 ms without them, 20.5 ms with one per
// hit, 17.9 ms with the records of a stage chained by leaf first. An LDS table per
// block of 1,024 rays, seven LDS atomics a hit, makes fewer device atomics but leaves
// room for three blocks per CU: 46.4 ms; the table filled from records in memory
// after the block's rays, 35.5 ms, or by a kernel of its own, 39.7 ms (LDS atomics:
// 30 cycles a hit and CU).

// Waves of one launch that take a pool each: a dispatch counts its work-items in 32
// bits, so one grid stays at 2^24 waves (2^30 work-items).
constexpr int64_t kLaunchWaves = int64_t(1) << 24;
// Up to so many pools every wave takes one (four blocks per CU, so that the next node's
// words fit the registers); beyond, pools are dealt, and from kAdjDealtPools on they
// come by queues. One / dealt in us with the
// forward's T: 286 / 322 at 5,003 x 33 (2,607 pools), surfaces 232 / 216 at 8,000 x 64 and 388 /
// 300 at 12,000 x 64, but 203 / 242 at 2,000 x 500, whose rays are short; a cloud of 9,887 x
// 75 1,407 / 1,346. A ray that is walked twice is twice as long: 264 / 301 at 4,000 x 64, 313 /
// 295 at 2,000 x 200, 625 / 476 (before either, 455) for eight objects of 1,000 x 64. Dealt /
// queues: 169 / 302 (before, 281) at 250 x 8 x 512 (16,384 pools), but a cloud of 20,000 x 64
// 3,090 / 2,920. With the same directions for all Gaussians pools are not dealt: a cloud
// of 8,935 x 79 1,094 / 1,250, of 6,647 x 69 walked twice 1,114 / 1,210.
constexpr int64_t kAdjOnePoolWaves = 8000, kAdjOnePoolWavesShort = 16000, kAdjOnePoolWavesTwice = 5000;
constexpr int64_t kAdjShortRays = 2048, kAdjDealtPools = 18000;
inline Route adjoint_route(int64_t n_pools, int64_t n, bool twice, int dir_mode) {
    if (dir_mode == 0) return n_pools <= kAdjOnePoolWavesShort ? Route::kOnePool : Route::kQueues;
    const int64_t one = twice ? kAdjOnePoolWavesTwice : n <= kAdjShortRays ? kAdjOnePoolWavesShort : kAdjOnePoolWaves;
    return n_pools <= one ? Route::kOnePool : n_pools <= kAdjDealtPools ? Route::kDealt : Route::kQueues;
}
// Up to so many rays every term goes to the caller's arrays at once: the accumulators
// are three launches more (two Gaussians x 64 54 us with them, 22 without).
constexpr int64_t kAdjDirectRays = 1024;
// Records per wave in LDS: as many as leave a CU five blocks; with chains a lane
// each. A chip that is not filled (kFewPools) is bound by the waves' own time, which
// chaining adds to: 697 / 784 us without / with at 20,000 x 64, the same at 50,000. With
// few Gaussians the same leaves come again and again: 343 / 250 us for 64 of deviation
// 0.07 to 0.37 in a cube of side 2 x 4,096 directions, 1,466 / 1,332 for 500 x 1,000 (1,205
// before), but 62.9 / 66.8 for 500 of 0.01 to 0.05 x 64.
constexpr int kAdjStageChain = 64, kAdjStage = 88;
constexpr int64_t kAdjChainGaussians = 1024;
inline bool adjoint_chains(int64_t n_pools, int64_t n) { return n <= kAdjChainGaussians || n_pools > kFewPools; }
constexpr int32_t kLinked = INT32_MIN;   // the leaf of a record that is not the head of its chain

// What the adjoint works in (null: every term goes to the caller's arrays at once).
struct AdjScratch {
    float *acc;   // [n][8] by leaf: the sums of a, a e and a e^2 (by component)
    float *org;   // [n][4] by leaf: the origin terms
};

// Seven sums of Gaussian j added with device-scope atomics.
__device__ __forceinline__ void add_grad_global(float *go, float *gm, float *gl, int64_t j, const float (&v)[7]) {
    unsafeAtomicAdd(go + j, v[0]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        unsafeAtomicAdd(gm + 3 * j + c, v[1 + c]);
        unsafeAtomicAdd(gl + 3 * j + c, v[4 + c]);
    }
}

struct GradRecord {
    bool active;        // false on the pass that only recovers T_final
    bool keep;          // records are kept; else a hit goes to the caller's arrays at once
    float g_over;       // -(dL/dT) * T_final for the current ray
    f3 origin;          // accumulated d/d(origin) of the current ray
    float *go, *gm, *gl;
    bool hit;           // the leaf under test left a record:
    float a;
    f3 e;

    __device__ __forceinline__ void operator()(const LeafHit &h, float) {
        if (!active || h.clamped) return;
        const float ga = g_over / h.one_minus;   // dL/dalpha
        a = ga * h.alpha;
        e = h.e;
        const f3 wte = e.x * h.w0 + e.y * h.w1 + e.z * h.w2;   // W^T e
        origin = origin - a * wte;
        hit = keep;
        if (keep) return;
        const float v[7] = {a / h.opacity, a * wte.x, a * wte.y, a * wte.z, a * e.x * e.x, a * e.y * e.y, a * e.z * e.z};
        add_grad_global(go, gm, gl, h.src, v);
    }
};

// A wave's stage of records: (a, e) of a hit of leaf `leaf`, or the origin terms of
// a ray (in e) of leaf ~leaf.
template <bool kChain>
struct AdjStage {
    static constexpr int kSize = kChain ? kAdjStageChain : kAdjStage;
    // (a block has an array of them, and records are stored as float4)
    struct alignas(16) Lds {
        float val[kSize * 4];
        int32_t leaf[kSize];
        int32_t next[kChain ? kSize : 1];   // the next record of a chain, -1 at its end
        int32_t last[kChain ? kSize : 1];   // the last record of a hash class; then the chains' heads
    };
    static_assert(sizeof(Lds) % 16 == 0, "every wave's records must be aligned as float4");
    Lds *s;
    int n;   // wave-uniform
    // Orders the wave's accesses to its stage.
    static __device__ __forceinline__ void sync() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
    // One record from each lane with `has` (called by the whole wave).
    __device__ __forceinline__ void put(bool has, int32_t m, float a, f3 e, const AdjScratch &sc) {
        const uint64_t lanes = __ballot(has);
        const int more = (int)__popcll(lanes);
        if (more == 0) return;
        if (n + more > kSize) flush(sc);
        if (has) {
            const int r = n + (int)__popcll(lanes & ((1ull << (threadIdx.x & 63)) - 1ull));
            *reinterpret_cast<float4 *>(s->val + 4 * r) = make_float4(a, e.x, e.y, e.z);
            s->leaf[r] = m;
        }
        n += more;
    }
    // Lane c of eight: the c-th sum of record r of leaf m.
    __device__ __forceinline__ float term(int r, int32_t m, int c, int comp) const {
        const float a = s->val[4 * r], x = s->val[4 * r + 1 + (m >= 0 ? comp : c & 3)];
        const float ax = a * x;
        return m < 0 ? x : c == 0 ? a : c < 4 ? ax : ax * x;
    }
    static __device__ __forceinline__ void add(const AdjScratch &sc, int32_t m, int c, float v) {
        if (c < (m >= 0 ? 7 : 3)) unsafeAtomicAdd((m >= 0 ? sc.acc + 8 * (int64_t)m : sc.org + 4 * (int64_t)~m) + c, v);
    }
    // Adds the records, eight lanes to one. With kChain those of one leaf are chained
    // first (through a hash of 64 classes: one that another leaf has taken starts a
    // new chain), and each chain is one addition.
    __device__ __forceinline__ void flush(const AdjScratch &sc) {
        const int lane = threadIdx.x & 63, c = lane & 7, comp = (c + 2) % 3;
        sync();
        if constexpr (kChain) {
            static_assert(kSize == 64, "a record per lane");
            const bool live = lane < n;
            s->last[lane] = -1;
            sync();
            const int32_t mine = live ? s->leaf[lane] : 0;
            const int prev = live ? atomicExch(&s->last[((uint32_t)mine * 2654435761u) >> 26], lane) : -1;
            const bool linked = prev >= 0 && s->leaf[prev] == mine;
            s->next[lane] = linked ? prev : -1;
            sync();
            if (linked) s->leaf[prev] = kLinked;
            sync();
            const bool head = live && s->leaf[lane] != kLinked;
            const uint64_t heads = __ballot(head);
            if (head) s->last[__popcll(heads & ((1ull << lane) - 1ull))] = lane;
            sync();
            const int n_heads = (int)__popcll(heads);
            for (int i = lane >> 3; i < n_heads; i += 8) {
                int r = s->last[i];
                const int32_t m = s->leaf[r];
                float sum = 0.0f;
                do {
                    sum += term(r, m, c, comp);
                    r = s->next[r];
                } while (r >= 0);
                add(sc, m, c, sum);
            }
        } else {
            for (int r = lane >> 3; r < n; r += 8) {
                const int32_t m = s->leaf[r];
                add(sc, m, c, term(r, m, c, comp));
            }
        }
        sync();
        n = 0;
    }
};

// Trace of the adjoint, pools and queues as the forward's. Each ray with a nonzero upstream gradient
// g = dL/dV_ik (grad_ray) + dL/dVbar_i / K (grad_mean) is traced once to
// recover T_final (skipped when the forward's T are given), then again
// with the same visits in the same order, recording dL/dalpha_j = -g T_final /
// (1 - alpha_j) of each included, unclamped Gaussian. The source's own term
// (through the ray origin) is summed over the ray.
template <Route kRoute, bool kChain>
__global__ __launch_bounds__(kTraceBlock, kRoute == Route::kOnePool ? 4 : kStreamBlocksPerCu) void k_adjoint_trace(
    const float *__restrict__ header, const float4 *__restrict__ nodes4, const float4 *__restrict__ rec, GridPools pools,
    int64_t first, int64_t n_pools, Cuts c,
    unsigned long long *__restrict__ queues, const float *__restrict__ grad_ray,
    const float *__restrict__ grad_mean_in, const float *__restrict__ vis_fwd, float *go, float *gm, float *gl,
    AdjScratch sc) {
    __shared__ Pair stk[kStreamRing * kTraceBlock];
    __shared__ Pair fifo[kFifo * kTraceBlock];
    __shared__ typename AdjStage<kChain>::Lds stage_lds[kWavesPerBlock];
    const int64_t n = pools.m_hi;
    if (!tree_matches(header, n)) {
        // a tree built for another Gaussian set: every gradient is NaN
        const float nan = __int_as_float(0x7fc00000);
        for (int64_t j = (int64_t)blockIdx.x * kTraceBlock + threadIdx.x; j < n; j += (int64_t)gridDim.x * kTraceBlock) {
            go[j] = nan;
#pragma unroll
            for (int x = 0; x < 3; ++x) gm[3 * j + x] = gl[3 * j + x] = nan;
        }
        return;
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    AdjStage<kChain> stage;
    stage.s = stage_lds + wv;
    stage.n = 0;
    constexpr bool kOnePool = kRoute == Route::kOnePool;
    std::conditional_t<kOnePool, RangeQueue, std::conditional_t<kRoute == Route::kDealt, RayDeal, XcdQueue>> queue;
    if constexpr (kOnePool) {
        queue.next = first + xcd_block(blockIdx.x, gridDim.x) * kWavesPerBlock + wv;
        queue.end = min(n_pools, queue.next + 1);
    } else {
        queue.init(queues, n_pools, blockIdx.x, gridDim.x);
    }

    Walk<kStreamRing> wk;
    Pair spill[Walk<kStreamRing>::kSpill];
    wk.init(stk + threadIdx.x, fifo + threadIdx.x, spill);
    RayBox rb;
    rb.set(mk(0.f, 0.f, 0.f), mk(0.f, 0.f, 0.f));
    f3 d = mk(0.f, 0.f, 0.f);
    float tmin = 0.f, T = 1.f, gk = 0.f;   // gk: upstream gradient of the current ray
    int32_t self = -1, self_leaf_m1 = -2;
    GradRecord gs;
    gs.active = false;
    gs.keep = sc.acc != nullptr;
    gs.g_over = 0.f;
    gs.origin = mk(0.f, 0.f, 0.f);
    gs.go = go;
    gs.gm = gm;
    gs.gl = gl;
    gs.a = 0.f;
    gs.e = mk(0.f, 0.f, 0.f);
    uint4 ahead[3] = {};   // kOnePool: the words of wk.node
    auto node_words = [&](uint4 (&w)[3]) {
        const uint4 *r = reinterpret_cast<const uint4 *>(nodes4) + 4 * (int64_t)wk.node + 4;
#pragma unroll
        for (int k = 0; k < 3; ++k) w[k] = r[k];
    };
    // wave-uniform pool state
    int next = 0, pool_n = 0;
    bool more = true;
    // (rays that are walked twice leave lanes idle twice as long: those are taken as on a
    // filled chip)
    Refill<RayDeal> patient;
    Refill<XcdQueue> filled;

    for (uint32_t round = 1;; ++round) {
        uint64_t need = __ballot(wk.idle());
        const bool take = kRoute == Route::kDealt && vis_fwd ? patient.now(need, c.refill) : filled.now(need, c.refill);
        if (!take) need = 0;
        const uint64_t empty = need;
        while (need != 0 && more) {
            if (next >= pool_n) {
                int64_t p;
                more = queue.take(p);
                pool_n = more ? pools.open(p) : 0;
                next = 0;
                continue;
            }
            const int idx = next + __popcll(need & lt);
            if (wk.idle() && idx < pool_n) {
                const RaySetup r = pools(idx);
                // r.out = i K + k: the ray's place in grad_ray and vis_fwd
                gk = (grad_mean_in ? grad_mean_in[r.self] / (float)pools.K : 0.0f) + (grad_ray ? grad_ray[r.out] : 0.0f);
                d = r.d;
                rb.set(r.o, d);
                tmin = r.tmin;
                self = r.self;
                self_leaf_m1 = r.self_leaf - 1;
                gs.origin = mk(0.f, 0.f, 0.f);
                // a ray with nothing to propagate ends here
                gs.active = vis_fwd != nullptr || gk == 0.0f;
                gs.g_over = vis_fwd ? -gk * vis_fwd[r.out] : 0.0f;
                T = 1.0f;
                wk.start(n, gk != 0.0f);
                if (kOnePool && wk.node > Walk<kStreamRing>::kDone) node_words(ahead);
            }
            next += __popcll(need);
            need = __ballot(wk.idle());
        }
        if (kRoute == Route::kDealt && vis_fwd && empty != 0) patient.loaded(empty & ~need, d);
        if (__ballot(!wk.idle()) == 0) break;

        if (wk.can_walk()) {
            if (kOnePool) {
                wk.visit(ahead, rb, tmin, T);
                if (wk.node > Walk<kStreamRing>::kDone) node_words(ahead);
            } else {
                uint4 w[3];
                node_words(w);
                wk.visit(w, rb, tmin, T);
            }
        }

        if (leaf_phase_now(wk)) {
            int32_t m1 = 0;
            gs.hit = false;
            if (wk.queued()) {
                m1 = wk.next_leaf();
                T *= leaf_factor(rec, m1, rb.o, d, tmin, self, self_leaf_m1, c, gs, T);
                if (T < c.T_stop) wk.stop();
            }
            stage.put(gs.hit, m1 + 1, gs.a, gs.e, sc);
        }
        if (round % kBudgetLook == 0 && wk.budget < 0 && !wk.idle()) {
            T = __int_as_float(0x7fc00000);
            wk.stop();
        }

        const bool finished = wk.finished();
        if (__ballot(finished) == 0) continue;
        const bool ended = finished && gs.active;
        const bool moved = ended && (gs.origin.x != 0.f || gs.origin.y != 0.f || gs.origin.z != 0.f);
        stage.put(moved && gs.keep, ~(self_leaf_m1 + 1), 0.f, gs.origin, sc);
        if (moved && !gs.keep) {
            unsafeAtomicAdd(gm + 3 * (int64_t)self + 0, gs.origin.x);
            unsafeAtomicAdd(gm + 3 * (int64_t)self + 1, gs.origin.y);
            unsafeAtomicAdd(gm + 3 * (int64_t)self + 2, gs.origin.z);
        }
        if (ended) wk.node = Walk<kStreamRing>::kIdle;
        if (finished && !gs.active) {
            // T_final is known: trace the same ray again, recording
            gs.g_over = -gk * T;
            gs.active = true;
            T = 1.0f;
            wk.start(n, true);
            if (kOnePool && wk.node > Walk<kStreamRing>::kDone) node_words(ahead);
        }
    }
    stage.flush(sc);
}

// The caller's gradients from the accumulators: with S the sums of a, a e and
// a e^2 over the hits of leaf m, dL/do = S_a / o, dL/dmu = W^T S_ae + the origin
// terms, dL/dlog_scale = S_ae2.
__global__ __launch_bounds__(256) void k_adjoint_add(const float *__restrict__ header, const float4 *__restrict__ rec,
                                                     int64_t n, const float4 *__restrict__ acc,
                                                     const float4 *__restrict__ org, float *go, float *gm, float *gl) {
    const int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (m >= n || !tree_matches(header, n)) return;
    const float4 s = acc[2 * m], t = acc[2 * m + 1], o = org[m];
    const float4 r0 = rec[kLeafF4 * m], r1 = rec[kLeafF4 * m + 1], r2 = rec[kLeafF4 * m + 2];
    const f3 w0 = mk(r1.x, r1.y, r1.z), w1 = mk(r2.x, r2.y, r2.z), w2 = r1.w * cross(w0, w1);
    const f3 mu = s.y * w0 + s.z * w1 + s.w * w2 + mk(o.x, o.y, o.z);
    const float v[7] = {s.x != 0.f ? s.x / r0.w : 0.f, mu.x, mu.y, mu.z, t.x, t.y, t.z};
    bool any = false;
#pragma unroll
    for (int c = 0; c < 7; ++c) any = any || v[c] != 0.f;
    if (any) add_grad_global(go, gm, gl, __float_as_int(r2.w), v);
}

// Words [0, count) to v.
__global__ __launch_bounds__(256) void k_fill_u32_wide(uint32_t *__restrict__ p, int64_t count, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) p[i] = v;
}

__global__ __launch_bounds__(64) void k_fill_u32_trace(uint32_t *__restrict__ p, int64_t count, uint32_t v) {
    for (int64_t i = threadIdx.x; i < count; i += 64) p[i] = v;
}

// The counters of the XCD queues (kQueueBytes) to zero.
void launch_clear_queues(unsigned long long *queues, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_u32_trace, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t *>(queues),
                       (int64_t)(kQueueBytes / 4), 0u);
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

rv_status validate_trace(const char *fn, const void *bvh, const rv_gaussians *g, const float *dirs, int32_t K,
                         const rv_trace_params *p) {
    RV_REQUIRE(bvh && g && dirs && p, RV_ERR_INVALID_ARG, "%s: null argument (bvh, g, dirs or params)", fn);
    RV_REQUIRE(g->mean && g->log_scale, RV_ERR_INVALID_ARG, "%s: null Gaussian mean/log_scale", fn);
    RV_REQUIRE(g->n >= 1 && g->n <= RV_MAX_GAUSSIANS, RV_ERR_INVALID_ARG, "%s: n=%lld out of range", fn,
               (long long)g->n);
    RV_REQUIRE(K >= 1, RV_ERR_INVALID_ARG, "%s: K=%d must be >= 1", fn, K);
    RV_REQUIRE(p->dir_mode == 0 || p->dir_mode == 1, RV_ERR_INVALID_ARG, "%s: dir_mode must be 0 or 1", fn);
    RV_REQUIRE(p->dir_mode == 0 || g->normal, RV_ERR_INVALID_ARG, "%s: hemisphere mode needs normals", fn);
    RV_REQUIRE(p->sigma_cut > 0.0f && p->sigma_cut <= kBuildSigma, RV_ERR_INVALID_ARG,
               "%s: sigma_cut must be in (0, %g] (the BVH boxes cover 3 sigma)", fn, (double)kBuildSigma);
    RV_REQUIRE(p->alpha_min > 0.0f && p->alpha_max < 1.0f && p->alpha_min <= p->alpha_max, RV_ERR_INVALID_ARG,
               "%s: need 0 < alpha_min <= alpha_max < 1", fn);
    RV_REQUIRE(p->T_min >= 0.0f && p->T_min < 1.0f && p->tmin_scale >= 0.0f, RV_ERR_INVALID_ARG,
               "%s: need 0 <= T_min < 1 and tmin_scale >= 0", fn);
    return RV_OK;
}


// Blocks of a persistent traversal grid: what the device holds at once, up
// to the blocks per CU above, kStreamBlocksFew with `few` (a multiple of 8, at
// least 8: every XCD queue has blocks), no more than the pools need.
int64_t stream_blocks(int64_t n_pools, int64_t n, int K, bool few) {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    int nb = (dev >= 0 && dev < 64) ? cached[dev].load() : 0;   // 256 CUs + blocks per CU
    if (nb <= 0) {
        int cus = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev < 0 ? 0 : dev) != hipSuccess ||
            cus <= 0)
            cus = 256;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_trace_stream<false, Route::kQueues>, kTraceBlock, 0) !=
                hipSuccess ||
            per_cu <= 0)
            per_cu = 4;
        (void)hipGetLastError();  // a failed query above must not surface as a launch error
        nb = cus * 256 + std::min(per_cu, kStreamBlocksPerCu);
        if (dev >= 0 && dev < 64) cached[dev].store(nb);
    }
    const int cus = nb / 256;
    const int per_cu = std::min(nb % 256, few ? kStreamBlocksFew
                                          : n >= kDeepStreamGaussians && K <= kDeepStreamDirs ? kStreamBlocksDeep
                                          : kStreamBlocksPerCu);
    int64_t want = std::min<int64_t>((int64_t)cus * per_cu, (n_pools + kWavesPerBlock - 1) / kWavesPerBlock);
    want = (want + kXcds - 1) / kXcds * kXcds;
    return std::max<int64_t>(want, kXcds);
}

// Waves of the list kernel beyond which each wave takes a run of several pools of
// 64 entries: few full waves end closer together than many that contend for the
// caches. With 2,048 / 4,096 / 16,384 waves, in ms, lists over 300,000 Gaussians x 256:
// random and sorted 0.66 / 0.68 / 0.68 for 200,000 entries, 1.55 / 1.72 / 1.90 for 1M, 11.2 /
// 12.7 / 12.5 for 10M, 31.3 / 31.7 / 31.6 for 30M; random 0.66 / 0.76 / 0.76 for 200,000,
// 13.0 / 14.7 / 15.1 for 10M; consecutive 0.74 / 0.59 / 0.59 for 200,000, 1.94 / 1.78 / 1.68 for
// 1M, 33.6 / 38.0 / 37.9 for 30M. Over 3M Gaussians x 64 sorted 6.3 / 6.6 / 6.2 for 1M, 116 / 121 /
// 118 for 30M. (32,768 waves of pools of 256: 1.21, 1.84, 13.1, 32.4 for the first four.)
constexpr int64_t kListTargetWaves = 2048;

}  // namespace

// A queued list (the surrogate's fallback) is dealt in chunks of 16 pools, on up to
// kFewPools rays by three blocks per CU. By queues and three blocks up to kFewPools pools /
// so, the whole inference of 100,000 Gaussians x 64: 2,357 / 2,217 us with nothing listed,
// 3,247 / 3,105 with 2 % of the queries, 4,204 / 3,857 with 45 %, 5,852 / 5,071 with all (5,771
// before either); of 5,003 x 33 with 45 % 239 / 220. Trees from kDeepStreamGaussians keep the former
// (1.2M x 8 with 45 % 10.6 / 12.4 ms).
void launch_trace_list(const void *bvh, const rv_gaussians *g, const float *dirs, int K, const Cuts &c,
                       const int64_t *ids, int64_t n_list, const unsigned long long *count, int64_t id_offset,
                       bool out_by_value, float *out, unsigned long long *queues, hipStream_t stream) {
    if (n_list <= 0) return;
    const BvhLayout L = bvh_layout(g->n);
    const int64_t entries = queues ? kPoolS * 64 : 64, pools = (n_list + entries - 1) / entries;
    Cuts cc = c;
    cc.refill = refill_lanes(g->n);
    auto launch = [&](auto kernel, int64_t blocks, int64_t run) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kTraceBlock), 0, stream, at<float>(bvh, L.header),
                           at<float4>(bvh, L.nodes4), at<float4>(bvh, L.leaf_rec), g->mean,
                           c.dir_mode ? g->normal : nullptr, g->log_scale, g->n, dirs, K, cc, ids, n_list, count,
                           id_offset, out_by_value ? 1 : 0, run, queues, out);
    };
    if (queues) {
        const bool deep = g->n >= kDeepStreamGaussians, dealt = pools <= kFewPools && !deep;
        launch_clear_queues(queues, stream);
        launch(dealt ? k_trace_list<Route::kDealt> : k_trace_list<Route::kQueues>,
               stream_blocks(pools, g->n, K, pools * (deep ? 1 : kPoolS) <= kFewPools), 0);
        return;
    }
    const int64_t run = (pools + kListTargetWaves - 1) / kListTargetWaves;
    launch(k_trace_list<Route::kOnePool>, ((pools + run - 1) / run + kWavesPerBlock - 1) / kWavesPerBlock, run);
}

}  // namespace rv

using namespace rv;

extern "C" size_t rv_trace_workspace_bytes(int64_t n, int32_t K) {
    if (n < 1 || K < 1) return kAlign;
    return kAlign + align_up((size_t)n * (size_t)K * sizeof(float));
}

namespace {

// The all-ray traversal: clear the XCD queues where they are used (kQueueBytes at
// ws), then trace every ray (writing vis_ray when given, counters into totals
// when counting).
template <bool kCount>
void launch_trace_stream(const void *bvh, const rv_gaussians *g, const float *dirs, int K, const Cuts &c,
                         void *ws, float *vis_ray, unsigned long long *totals, hipStream_t s, int64_t m_lo = 0,
                         int64_t m_hi = -1, bool by_leaf = false) {
    const BvhLayout L = bvh_layout(g->n);
    if (m_hi < 0) m_hi = g->n;
    const int64_t n_pools = ((m_hi - m_lo + 63) / 64) * (int64_t)((K + kStreamPoolS - 1) / kStreamPoolS);
    auto *queues = static_cast<unsigned long long *>(ws);
    Cuts cc = c;
    cc.refill = refill_lanes(g->n);
    const Route route = all_ray_route(n_pools, g->n, c.dir_mode);
    int64_t blocks = (n_pools + kWavesPerBlock - 1) / kWavesPerBlock;
    auto kernel = k_trace_stream<kCount, Route::kOnePool>;
    if (route != Route::kOnePool) {
        launch_clear_queues(queues, s);
        blocks = stream_blocks(n_pools, g->n, K, route == Route::kQueues && n_pools <= kFewPools);
        kernel = route == Route::kDealt ? k_trace_stream<kCount, Route::kDealt> : k_trace_stream<kCount, Route::kQueues>;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kTraceBlock), 0, s, at<float>(bvh, L.header),
                       at<float4>(bvh, L.nodes4), at<float4>(bvh, L.leaf_rec), at<float4>(bvh, L.origins), dirs, g->n, K,
                       cc, m_lo, m_hi, by_leaf ? 1 : 0, queues, vis_ray, totals);
}

// Enqueue the all-ray trace with its scratch at ws (256-byte aligned: the
// queue counters, then the per-ray values when vis_ray is NULL).
void trace_visibility_into(const void *bvh, const rv_gaussians *g, const float *dirs, int32_t K,
                           const rv_trace_params *p, float *vis_ray, float *vis_mean, void *ws, hipStream_t s) {
    // the per-ray values go to vis_ray, else to the workspace after the queues
    float *rays = vis_ray ? vis_ray : reinterpret_cast<float *>(static_cast<char *>(ws) + kAlign);
    launch_trace_stream<false>(bvh, g, dirs, K, make_cuts(*p), ws, rays, nullptr, s);
    if (vis_mean) {
        const int64_t blocks = std::min<int64_t>((g->n + 3) / 4, int64_t(1) << 20);
        hipLaunchKernelGGL(k_mean_rows, dim3((unsigned)blocks), dim3(256), 0, s, rays, g->n, K, vis_mean);
    }
}

// ---- scratch of the allocation-free entry point ---------------------------
//
// One array per device, held until the process ends: the queue counters and,
// for calls without per-ray output, the per-ray values. In host code the
// array's name is a host-side stand-in, never a device address: its device
// address is looked up once per device (with that device current) and only
// that address is passed on.
constexpr size_t kStaticScratchBytes = size_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];

// Device address of the current device's scratch (looked up on its first use).
rv_status static_scratch(void **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    RV_REQUIRE(e == hipSuccess && dev >= 0 && dev < kMaxDevices, RV_ERR_HIP,
               "rv_trace_visibility_static: no current device (HIP error %d)", (int)e);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        RV_REQUIRE(e == hipSuccess && ptr, RV_ERR_HIP,
                   "rv_trace_visibility_static: hipGetSymbolAddress of the scratch failed on device %d: %s", dev,
                   hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return RV_OK;
}

}  // namespace

extern "C" rv_status rv_trace_visibility(const void *bvh, const rv_gaussians *g, const float *dirs, int32_t K,
                                         const rv_trace_params *p, float *vis_ray, float *vis_mean, void *ws,
                                         size_t ws_bytes, void *stream) {
    clear_error();
    rv_status st = validate_trace("rv_trace_visibility", bvh, g, dirs, K, p);
    if (st != RV_OK) return st;
    RV_REQUIRE(vis_ray || vis_mean, RV_ERR_INVALID_ARG, "rv_trace_visibility: both outputs are NULL");
    RV_REQUIRE(ws && ((uintptr_t)ws % kAlign) == 0, RV_ERR_INVALID_ARG,
               "rv_trace_visibility: needs a 256-byte aligned workspace");
    const size_t need = vis_ray ? kAlign : rv_trace_workspace_bytes(g->n, K);
    RV_REQUIRE(ws_bytes >= need, RV_ERR_WORKSPACE, "rv_trace_visibility: ws_bytes %zu < %zu", ws_bytes, need);
    trace_visibility_into(bvh, g, dirs, K, p, vis_ray, vis_mean, ws, (hipStream_t)stream);
    return check_launch("rv_trace_visibility");
}

extern "C" size_t rv_trace_static_scratch_bytes(void) { return kStaticScratchBytes; }

extern "C" rv_status rv_trace_visibility_static(const void *bvh, const rv_gaussians *g, const float *dirs,
                                                int32_t K, const rv_trace_params *p, float *vis_ray,
                                                float *vis_mean, void *stream) {
    clear_error();
    rv_status st = validate_trace("rv_trace_visibility_static", bvh, g, dirs, K, p);
    if (st != RV_OK) return st;
    RV_REQUIRE(vis_ray || vis_mean, RV_ERR_INVALID_ARG, "rv_trace_visibility_static: both outputs are NULL");
    const size_t need = vis_ray ? kAlign : rv_trace_workspace_bytes(g->n, K);
    RV_REQUIRE(need <= kStaticScratchBytes, RV_ERR_WORKSPACE,
               "rv_trace_visibility_static: without vis_ray the %lld x %d per-ray values need %zu bytes of scratch, "
               "more than the %zu-byte static scratch (at most %zu rays; pass vis_ray or use rv_trace_visibility)",
               (long long)g->n, K, need, kStaticScratchBytes, (kStaticScratchBytes - kAlign) / sizeof(float));
    void *ws = nullptr;
    st = static_scratch(&ws);
    if (st != RV_OK) return st;
    trace_visibility_into(bvh, g, dirs, K, p, vis_ray, vis_mean, ws, (hipStream_t)stream);
    return check_launch("rv_trace_visibility_static");
}

extern "C" rv_status rv_trace_stats(const void *bvh, const rv_gaussians *g, const float *dirs, int32_t K,
                                    const rv_trace_params *p, int64_t *totals, void *ws, size_t ws_bytes,
                                    void *stream) {
    clear_error();
    rv_status st = validate_trace("rv_trace_stats", bvh, g, dirs, K, p);
    if (st != RV_OK) return st;
    RV_REQUIRE(totals, RV_ERR_INVALID_ARG, "rv_trace_stats: null totals");
    RV_REQUIRE(ws && ((uintptr_t)ws % kAlign) == 0, RV_ERR_INVALID_ARG,
               "rv_trace_stats: needs a 256-byte aligned workspace");
    RV_REQUIRE(ws_bytes >= kAlign, RV_ERR_WORKSPACE, "rv_trace_stats: ws_bytes %zu < %zu", ws_bytes, kAlign);
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_fill_u32_trace, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t *>(totals), (int64_t)6,
                       0u);
    launch_trace_stream<true>(bvh, g, dirs, K, make_cuts(*p), ws, nullptr, (unsigned long long *)totals, s);
    return check_launch("rv_trace_stats");
}

extern "C" rv_status rv_trace_rays(const void *bvh, const rv_gaussians *g, const float *dirs, int32_t K,
                                   const rv_trace_params *p, const int64_t *ray_ids, int64_t n_rays, float *out,
                                   void *stream) {
    clear_error();
    rv_status st = validate_trace("rv_trace_rays", bvh, g, dirs, K, p);
    if (st != RV_OK) return st;
    RV_REQUIRE(n_rays >= 0, RV_ERR_INVALID_ARG, "rv_trace_rays: n_rays < 0");
    if (n_rays == 0) return RV_OK;
    RV_REQUIRE(ray_ids && out, RV_ERR_INVALID_ARG, "rv_trace_rays: null ray_ids or out");
    launch_trace_list(bvh, g, dirs, K, make_cuts(*p), ray_ids, n_rays, nullptr, 0, false, out, nullptr,
                      (hipStream_t)stream);
    return check_launch("rv_trace_rays");
}

extern "C" rv_status rv_trace_visibility_backward(const void *bvh, const rv_gaussians *g, const float *dirs,
                                                  int32_t K, const rv_trace_params *p, const float *grad_vis_ray,
                                                  const float *grad_vis_mean, const float *vis_ray_fwd,
                                                  float *grad_opacity, float *grad_mean, float *grad_log_scale,
                                                  void *stream) {
    clear_error();
    rv_status st = validate_trace("rv_trace_visibility_backward", bvh, g, dirs, K, p);
    if (st != RV_OK) return st;
    RV_REQUIRE(grad_vis_ray || grad_vis_mean, RV_ERR_INVALID_ARG,
               "rv_trace_visibility_backward: both upstream gradients are NULL");
    RV_REQUIRE(grad_opacity && grad_mean && grad_log_scale, RV_ERR_INVALID_ARG,
               "rv_trace_visibility_backward: null gradient output");
    const int64_t n = g->n;
    const BvhLayout L = bvh_layout(n);
    Cuts c = make_cuts(*p);
    c.refill = refill_lanes(n);
    hipStream_t s = (hipStream_t)stream;
    GridPools pools;
    pools.rec = at<float4>(bvh, L.leaf_rec);
    pools.origins = at<float4>(bvh, L.origins);
    pools.dirs = dirs;
    pools.dir_mode = c.dir_mode;
    pools.tmin_scale = c.tmin_scale;
    pools.K = K;
    pools.m0 = 0;
    pools.nv = 1;
    pools.k0 = 0;
    pools.inv_nv = 1.0f;
    pools.m_hi = n;
    pools.n_chunks = (K + kStreamPoolS - 1) / kStreamPoolS;
    const int64_t n_pools = ((n + 63) / 64) * (int64_t)pools.n_chunks;
    // accumulators (stream-ordered, freed after the launches); without them every
    // term goes to the caller's arrays at once, by waves of one pool
    AdjScratch sc{};
    unsigned long long *queues = nullptr;
    const size_t off_acc = kQueueBytes, off_org = off_acc + (size_t)n * 8 * sizeof(float);
    const size_t bytes = off_org + (size_t)n * 4 * sizeof(float);
    void *mem = nullptr;
    if (n * (int64_t)K > kAdjDirectRays && hipMallocAsync(&mem, bytes, s) != hipSuccess) {
        mem = nullptr;
        (void)hipGetLastError();
    }
    if (mem) {
        queues = at<unsigned long long>(mem, 0);
        sc.acc = at<float>(mem, off_acc);
        sc.org = at<float>(mem, off_org);
        const int64_t words = (int64_t)(bytes / sizeof(uint32_t));
        hipLaunchKernelGGL(k_fill_u32_wide, dim3((unsigned)std::min<int64_t>((words + 255) / 256, 4096)), dim3(256), 0, s,
                           static_cast<uint32_t *>(mem), words, 0u);
    }
    const Route route = mem ? adjoint_route(n_pools, n, vis_ray_fwd == nullptr, c.dir_mode) : Route::kOnePool;
    const bool chain = adjoint_chains(n_pools, n);
    auto launch = [&](auto kernel, int64_t blocks, int64_t first) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kTraceBlock), 0, s, at<float>(bvh, L.header),
                           at<float4>(bvh, L.nodes4), at<float4>(bvh, L.leaf_rec), pools, first, n_pools, c, queues,
                           grad_vis_ray, grad_vis_mean, vis_ray_fwd, grad_opacity, grad_mean, grad_log_scale, sc);
    };
    if (route == Route::kOnePool) {
        const auto kernel = chain ? k_adjoint_trace<Route::kOnePool, true> : k_adjoint_trace<Route::kOnePool, false>;
        for (int64_t first = 0; first < n_pools; first += kLaunchWaves)
            launch(kernel, grid_for(std::min(kLaunchWaves, n_pools - first), kWavesPerBlock), first);
    } else {
        const bool dealt = route == Route::kDealt;
        const auto kernel =
            dealt ? (chain ? k_adjoint_trace<Route::kDealt, true> : k_adjoint_trace<Route::kDealt, false>)
                  : (chain ? k_adjoint_trace<Route::kQueues, true> : k_adjoint_trace<Route::kQueues, false>);
        launch(kernel, stream_blocks(n_pools, n, K, !dealt && n_pools <= kFewPools), 0);
    }
    if (mem)
        hipLaunchKernelGGL(k_adjoint_add, dim3(grid_for(n, 256)), dim3(256), 0, s, at<float>(bvh, L.header),
                           at<float4>(bvh, L.leaf_rec), n, reinterpret_cast<const float4 *>(sc.acc),
                           reinterpret_cast<const float4 *>(sc.org), grad_opacity, grad_mean, grad_log_scale);
    const rv_status st_launch = check_launch("rv_trace_visibility_backward");
    if (mem) (void)hipFreeAsync(mem, s);
    return st_launch;
}

extern "C" size_t rv_trace_sh_workspace_bytes(int64_t n, int32_t K) {
    if (n < 1 || K < 1) return 0;
    return kAlign + align_up((size_t)K * kShCoef * sizeof(float)) +
           align_up((size_t)sh_batch(n, K) * (size_t)K * sizeof(float));
}

extern "C" rv_status rv_trace_visibility_sh(const void *bvh, const rv_gaussians *g, const float *dirs, int32_t K,
                                            const rv_trace_params *p, float *vis_sh, float *vis_mean, void *ws,
                                            size_t ws_bytes, void *stream) {
    clear_error();
    rv_status st = validate_trace("rv_trace_visibility_sh", bvh, g, dirs, K, p);
    if (st != RV_OK) return st;
    RV_REQUIRE(vis_sh, RV_ERR_INVALID_ARG, "rv_trace_visibility_sh: null vis_sh");
    const size_t need = rv_trace_sh_workspace_bytes(g->n, K);
    RV_REQUIRE(ws && ((uintptr_t)ws % kAlign) == 0, RV_ERR_INVALID_ARG,
               "rv_trace_visibility_sh: ws missing or unaligned");
    RV_REQUIRE(ws_bytes >= need, RV_ERR_WORKSPACE, "rv_trace_visibility_sh: ws_bytes %zu < %zu", ws_bytes, need);
    // ws: queue counters | Y table [K][9] | rows of one batch [batch][K]
    float *Y = reinterpret_cast<float *>(static_cast<char *>(ws) + kAlign);
    float *rows = reinterpret_cast<float *>(static_cast<char *>(ws) + kAlign +
                                            align_up((size_t)K * kShCoef * sizeof(float)));
    const BvhLayout L = bvh_layout(g->n);
    const Cuts c = make_cuts(*p);
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_sh_table, dim3(grid_for(K, 256)), dim3(256), 0, s, dirs, (int)K, Y);
    const double dw = (p->dir_mode ? 2.0 : 4.0) * 3.14159265358979323846 / (double)K;
    const int64_t batch = sh_batch(g->n, K);
    for (int64_t m_lo = 0; m_lo < g->n; m_lo += batch) {
        const int64_t m_hi = std::min(g->n, m_lo + batch);
        launch_trace_stream<false>(bvh, g, dirs, K, c, ws, rows, nullptr, s, m_lo, m_hi, true);
        const int64_t blocks = std::min<int64_t>((m_hi - m_lo + 3) / 4, int64_t(1) << 20);
        hipLaunchKernelGGL(k_sh_rows, dim3((unsigned)blocks), dim3(256), 0, s, rows, m_lo, m_hi - m_lo, (int)K, Y,
                           at<float>(bvh, L.header), at<float4>(bvh, L.leaf_rec), g->n, dw, vis_sh, vis_mean);
    }
    return check_launch("rv_trace_visibility_sh");
}
