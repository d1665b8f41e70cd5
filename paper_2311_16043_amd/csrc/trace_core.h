// trace_core.h -- per-lane all-hit BVH traversal of one ray through 3D
// Gaussians (Sec. 4.1): starting at the root, test the children's boxes,
// descend into the hit ones, and at each leaf evaluate the Gaussian at its
// equivalent intersection point (Eq. (13), peak parameter Eq. (14) with
// Sigma^-1) and attenuate T by (1 - alpha) (Eq. (15)); stop early once
// T < T_min. The tree is walked through its compressed four-wide records
// (each internal node lists its grandchildren). The order of hits does not
// change the full product (Sec. 4.1), so children are taken in slot order
// without sorting by distance.
#pragma once

#include "rv_internal.h"

namespace rv {

// Deepest possible root-to-leaf path: each level consumes at least one bit of
// the 95-bit augmented key (63-bit Morton key + 32-bit position).
constexpr int kMaxDepth = 96;
// Stack bound of the four-wide walk: at most 48 wide levels on a path, each
// leaving at most two pairs of siblings (see Pair) on the stack.
constexpr int kMaxStack = 2 * (kMaxDepth / 2);

// Idle lanes that trigger the refill of a wave in the pooled traversals
// (unless no lane holds a ray). Waiting for several idle lanes runs the ray
// setup for many lanes at once at the price of a few lanes of traversal; the
// best count grows with the tree: 12 measured best at 300k and 1.2M Gaussians
// (16 equal at 1.2M, 20 slower at both), 20 at 3M (2.5 % faster than 12).
constexpr int kRefillShallow = 12, kRefillDeep = 20;
constexpr int64_t kDeepTreeGaussians = int64_t(2) << 20;
inline int refill_lanes(int64_t n) { return n >= kDeepTreeGaussians ? kRefillDeep : kRefillShallow; }

struct Cuts {
    float alpha_min, alpha_max, T_stop, q_cut, tmin_scale;
    int dir_mode;
    int refill;   // idle lanes before a refill (refill_lanes of the tree's size)
};

inline Cuts make_cuts(const rv_trace_params &p) {
    Cuts c;
    c.alpha_min = p.alpha_min;
    c.alpha_max = p.alpha_max;
    c.T_stop = p.T_min;
    c.q_cut = p.sigma_cut * p.sigma_cut;
    c.tmin_scale = p.tmin_scale;
    c.dir_mode = p.dir_mode;
    c.refill = kRefillShallow;
    return c;
}

// Orthonormal basis (b1, b2) completing the unit normal n: Duff et al.,
// "Building an Orthonormal Basis, Revisited" (JCGT 2017).
__device__ __forceinline__ void onb_duff(f3 n, f3 &b1, f3 &b2) {
    const float sign = copysignf(1.0f, n.z);
    const float a = -__builtin_amdgcn_rcpf(sign + n.z);  // |sign + n.z| in [1, 2]; one ulp
    const float b = n.x * n.y * a;
    b1 = mk(1.0f + sign * n.x * n.x * a, sign * b, -sign * n.x);
    b2 = mk(b, sign + n.y * n.y * a, -n.y);
}

// Direction k: world frame (mode 0) or local frame about n (mode 1), unit length.
__device__ __forceinline__ f3 ray_direction(const float *__restrict__ dirs, int k, int mode, f3 n, f3 b1, f3 b2) {
    const float dx = dirs[3 * k], dy = dirs[3 * k + 1], dz = dirs[3 * k + 2];
    f3 d = mode ? (dx * b1 + dy * b2 + dz * n) : mk(dx, dy, dz);
    const float inv = __builtin_amdgcn_rsqf(dot(d, d));  // one ulp; |d| is 1 up to rounding
    return inv * d;
}

// Reciprocal direction (hardware reciprocal, within one ulp) with zero
// components replaced by a tiny signed value, so every component is finite,
// nonzero and carries the sign of d. (A ray of length up to 10^12 leaves a plane
// it is parallel to by at most 10^-10 so, far inside the boxes' margin; with its
// reciprocal at 10^22, the products of visit4 stay finite for steps up to 10^9.)
__device__ __forceinline__ f3 safe_inv(f3 d) {
    auto r = [](float x) {
        const float tiny = 1e-22f;
        float y = fabsf(x) < tiny ? copysignf(tiny, x) : x;
        return __builtin_amdgcn_rcpf(y);
    };
    return mk(r(d.x), r(d.y), r(d.z));
}

// The two children on one side of a four-wide node as one word: the index of the
// first in the low 30 bits (the second has the next one; n <= 2^30), bit 30 set
// when the first counts, bit 31 when the second does. Stacks and queues of the
// walk hold pairs, so a node adds at most two entries to either.
typedef uint32_t Pair;
constexpr uint32_t kPairIndex = 0x3fffffffu;
__device__ __forceinline__ bool pair_any(Pair e) { return e > kPairIndex; }
// Index of the first child that counts, less one.
__device__ __forceinline__ int32_t pair_first_m1(Pair e) {
    return (int32_t)(e & kPairIndex) - (int32_t)((e >> 30) & 1u);
}
// The pair without its first counting child (0 when none is left).
__device__ __forceinline__ Pair pair_rest(Pair e) { return e >= 0xc0000000u ? e & ~0x40000000u : 0u; }

// Two-bit masks of a side's leaves and internal nodes for its kind bits
// (l1 u1 l0 u0), sixteen to a word.
constexpr uint32_t pair_table(bool leaf) {
    uint32_t t = 0;
    for (uint32_t v = 0; v < 16; ++v) {
        const uint32_t u = (v & 1u) | ((v >> 1) & 2u), l = ((v >> 1) & 1u) | ((v >> 2) & 2u);
        t |= (leaf ? l & u : u & ~l) << (2 * v);
    }
    return t;
}

// A ray as the box tests take it.
struct RayBox {
    f3 o, inv;           // origin, reciprocal direction
    f3 inv24;            // 2^24 inv
    uint32_t near01[3], near23[3], far01[3], far23[3];   // byte selectors, see visit4
    __device__ __forceinline__ void set(f3 origin, f3 d) {
        o = origin;
        inv = safe_inv(d);
        inv24 = 0x1p24f * inv;
        const float s[3] = {inv.x, inv.y, inv.z};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const uint32_t flip = s[a] < 0.0f ? 0x00040004u : 0u;
            near01[a] = 0x0c010c00u ^ flip;
            near23[a] = 0x0c030c02u ^ flip;
            far01[a] = 0x0c050c04u ^ flip;
            far23[a] = 0x0c070c06u ^ flip;
        }
    }
};

// Children of the compressed four-wide node at words r[0..2] whose boxes the ray
// segment [t0, inf) enters: the leaves and the internal nodes of either side. A
// box plane is P = O_a + q step_a (q one byte), so its ray distance is
// fma(q, step_a inv_a, (O_a - o_a) inv_a) with inv_a the reciprocal of d_a to
// within one ulp; step_a inv_a is exact (a power-of-two scaling). The roundings
// of inv_a (2^-23 relative), of O_a - o_a, of the product and of the fma (2^-24
// each) move a plane by at most 2^-23 (1.5 |P - o| + |O - o|) <=
// 5 2^-23 max|coordinate| in space, which is below the outward margin
// eta >= 2^-20 (max|coordinate| + 1) that the builder added to every plane. So a
// box the exact ray enters beyond t0 is never rejected, and no further
// enlargement of the exit distance is needed. The fma is monotone in q, rising
// for inv_a > 0 and falling for inv_a < 0, so the entry plane of each axis is the
// low one for a positive direction component and the high one otherwise.
//
// The walk is bound by the instructions it issues, and these tests are most of
// them. One byte permute takes two planes of an axis, low or high by the ray's
// sign, zero-extended to 16 bits each: read as an f16 a plane byte q is the
// subnormal q 2^-24, exactly, which a mixed-precision fma takes as it is with
// 2^24 inv in the scaling (in the place of a conversion per plane and a select per
// word: 36 instructions for the 24 planes instead of 57).
struct Children {
    Pair leaf[2], node[2];
};
__device__ __forceinline__ Children visit4(uint4 w0, uint4 w1, uint4 w2, const RayBox &rb, float t0) {
    typedef _Float16 half2 __attribute__((ext_vector_type(2)));
    const uint32_t meta = w0.w;
    const float ax = __uint_as_float((meta & 0xffu) << 23) * rb.inv24.x;
    const float ay = __uint_as_float(((meta >> 8) & 0xffu) << 23) * rb.inv24.y;
    const float az = __uint_as_float(((meta >> 16) & 0xffu) << 23) * rb.inv24.z;
    const float bx = (__uint_as_float(w0.x) - rb.o.x) * rb.inv.x;
    const float by = (__uint_as_float(w0.y) - rb.o.y) * rb.inv.y;
    const float bz = (__uint_as_float(w0.z) - rb.o.z) * rb.inv.z;
    auto pick = [](uint32_t lo, uint32_t hi, uint32_t sel) {
        return __builtin_bit_cast(half2, __builtin_amdgcn_perm(hi, lo, sel));
    };
    bool hit[4];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const half2 nx = pick(w1.x, w1.w, g ? rb.near23[0] : rb.near01[0]);
        const half2 ny = pick(w1.y, w2.x, g ? rb.near23[1] : rb.near01[1]);
        const half2 nz = pick(w1.z, w2.y, g ? rb.near23[2] : rb.near01[2]);
        const half2 fx = pick(w1.x, w1.w, g ? rb.far23[0] : rb.far01[0]);
        const half2 fy = pick(w1.y, w2.x, g ? rb.far23[1] : rb.far01[1]);
        const half2 fz = pick(w1.z, w2.y, g ? rb.far23[2] : rb.far01[2]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float tn = fmaxf(fmaxf(fmaf((float)nx[h], ax, bx), fmaf((float)ny[h], ay, by)),
                                   fmaxf(fmaf((float)nz[h], az, bz), t0));
            const float tf = fminf(fminf(fmaf((float)fx[h], ax, bx), fmaf((float)fy[h], ay, by)),
                                   fmaf((float)fz[h], az, bz));
            hit[2 * g + h] = tn <= tf;
        }
    }
    // a side's kind bits (l1 u1 l0 u0, zero where missed or unused) times two,
    // as the shift that brings its masks down from the tables
    Children c;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint32_t kinds = (meta >> (23 + 4 * s)) & ((hit[2 * s] ? 0x06u : 0u) | (hit[2 * s + 1] ? 0x18u : 0u));
        const uint32_t first = s ? w2.w : w2.z;
        constexpr uint32_t kLeaves = pair_table(true), kNodes = pair_table(false);
        c.leaf[s] = ((kLeaves >> kinds) << 30) | first;
        c.node[s] = ((kNodes >> kinds) << 30) | first;
    }
    return c;
}

// What a leaf test hands to a hit callback.
struct LeafHit {
    float alpha;     // unclamped alpha = o exp(-q/2)
    float one_minus; // the factor applied to T: 1 - min(alpha, alpha_max)
    bool clamped;    // alpha >= alpha_max (contribution used min(alpha, alpha_max))
    float opacity;
    int32_t src;     // original index of the Gaussian
    f3 e;            // whitened closest-approach vector p + t* v (|e|^2 = q)
    f3 w0, w1, w2;   // rows of W
};

struct NoHit {
    __device__ __forceinline__ void operator()(const LeafHit &, float) const {}
};

// e^x - 1 for x in [-1/4, 0] from its Taylor series through x^7 (the
// remainder x^8 / 8! is below 2e-9 of the result there), evaluated in
// Horner form; unlike e^x - 1 it keeps full relative precision as x -> 0.
__device__ __forceinline__ float expm1_small(float x) {
    float r = 1.0f / 5040.0f;
    r = fmaf(r, x, 1.0f / 720.0f);
    r = fmaf(r, x, 1.0f / 120.0f);
    r = fmaf(r, x, 1.0f / 24.0f);
    r = fmaf(r, x, 1.0f / 6.0f);
    r = fmaf(r, x, 0.5f);
    r = fmaf(r, x, 1.0f);
    return r * x;
}

// Evaluate leaf m = m1 + 1 for the ray (o, d) of source `self`. Returns the factor
// (1 - alpha) to multiply into T (1 when excluded); calls on_hit for included
// Gaussians with the running T before this factor. Branch-free up to the
// final decision, so the record's three rows are fetched together.
template <class OnHit>
__device__ __forceinline__ float leaf_factor(const float4 *__restrict__ rec, int32_t m1, f3 o, f3 d, float tmin,
                                             int32_t self, int32_t self_leaf_m1, const Cuts &c, OnHit &on_hit,
                                             float T_before) {
    if (m1 == self_leaf_m1) return 1.0f;   // the source's own leaf, known by sorted position
    // (in 64 bits: the record's first word passes 2^31 from leaf 715,827,883 on)
    const float4 *r = rec + ((int64_t)kLeafF4 * m1 + kLeafF4);
    const float4 r0 = r[0], r1 = r[1], r2 = r[2];
    const int32_t src = __float_as_int(r2.w);
    const f3 w0 = mk(r1.x, r1.y, r1.z), w1 = mk(r2.x, r2.y, r2.z);
    const f3 w2 = r1.w * cross(w0, w1);
    const f3 x = o - mk(r0.x, r0.y, r0.z);
    const f3 p = mk(dot(w0, x), dot(w1, x), dot(w2, x));
    const f3 v = mk(dot(w0, d), dot(w1, d), dot(w2, d));
    const float vv = dot(v, v);
    const float pv = dot(p, v);
    const f3 cp = cross(p, v);
    const float cc = dot(cp, cp);
    // peak parameter t* = -pv / vv >= t_min and squared distance at the peak
    // q = |p x v|^2 / vv <= q_cut, both decided without dividing (vv > 0); the
    // source itself (when its sorted position is not known) never counts
    const bool in_support = src != self && -pv >= tmin * vv && cc <= c.q_cut * vv;
    const float inv_vv = __builtin_amdgcn_rcpf(vv);
    const float q = cc * inv_vv;
    // alpha = o e^{-q/2} = o + o m with m = e^{-q/2} - 1. For small q, m comes
    // from the series so that 1 - alpha = (1 - o) - o m keeps full relative
    // precision when alpha approaches 1 (the adjoint divides by it).
    const float ex = -0.5f * q;
    const float m_small = expm1_small(ex), m_large = __expf(ex) - 1.0f;
    const float em1 = q < 0.5f ? m_small : m_large;
    const float op = r0.w;
    const float alpha = op + op * em1;
    if (!(in_support && alpha >= c.alpha_min)) return 1.0f;
    const bool clamped = alpha >= c.alpha_max;
    const float one_minus = clamped ? 1.0f - c.alpha_max : (1.0f - op) - op * em1;
    LeafHit h;
    h.alpha = alpha;
    h.one_minus = one_minus;
    h.clamped = clamped;
    h.opacity = op;
    h.src = src;
    h.e = p + (-pv * inv_vv) * v;
    h.w0 = w0;
    h.w1 = w1;
    h.w2 = w2;
    on_hit(h, T_before);
    return one_minus;
}

// One ray's walk: the node to visit next, the pairs of internal nodes still to
// visit (a stack) and the pairs of leaves still to test (a queue of kFifo
// entries). Both are columns of the block's LDS, entry e of lane t at
// [e kTraceBlock + t]; the top kRing entries of the stack live there and deeper
// ones in a private array owned by the kernel (kept outside this struct so that
// the scalar state stays in registers): entries [max(0, sp - kRing), sp) are in
// the ring at slot (index % kRing), entries [0, sp - kRing) in spill[].
constexpr int kTraceBlock = 256;
constexpr int kFifo = 8;

template <int kRing>
struct Walk {
    static constexpr int kSpill = kMaxStack - kRing;
    static constexpr int32_t kDone = -2, kIdle = -3;
    Pair *ring, *fifo;   // this lane's columns
    Pair *spill;         // private array of kSpill entries
    int32_t node;        // index of the node to visit next less one; kDone: none left; kIdle: no ray
    Pair cur;            // the pair below the stack's top, of which `node` was taken
    int sp;
    uint32_t head, tail; // leaf pairs queued since the ray began, and taken
    int32_t budget;      // node visits left (n <= 2^30)

    __device__ __forceinline__ void init(Pair *ring_, Pair *fifo_, Pair *spill_) {
        ring = ring_;
        fifo = fifo_;
        spill = spill_;
        node = kIdle;
        cur = 0;
        sp = 0;
        head = tail = 0;
        budget = 0;
    }
    // Start at the root of a tree over n leaves (none to walk: walk = false).
    __device__ __forceinline__ void start(int64_t n, bool walk) {
        node = walk && n > 1 ? -1 : kDone;
        cur = 0;
        sp = 0;
        head = tail = 0;
        budget = (int32_t)n;
    }
    __device__ __forceinline__ void stop() {
        node = kDone;
        head = tail;
    }
    __device__ __forceinline__ bool idle() const { return node == kIdle; }
    __device__ __forceinline__ bool queued() const { return head != tail; }
    // Room in the queue for the two pairs that a visit may add.
    __device__ __forceinline__ bool room() const { return tail - head <= (uint32_t)(kFifo - 2); }
    __device__ __forceinline__ bool can_walk() const { return node > kDone && room(); }
    __device__ __forceinline__ bool finished() const { return node == kDone && head == tail; }

    // Visit `node`: queue the leaves it enters and move to the next node in slot
    // order (the first entered child, else the most recent pair left over).
    __device__ __forceinline__ void visit(const uint4 (&w)[3], const RayBox &rb, float tmin, float &T) {
        --budget;
        const Children c = visit4(w[0], w[1], w[2], rb, tmin);
        // a visit starts with two free entries, so both are written and the
        // tail passes the ones that count
        fifo[(tail & (kFifo - 1)) * kTraceBlock] = c.leaf[0];
        tail += pair_any(c.leaf[0]);
        fifo[(tail & (kFifo - 1)) * kTraceBlock] = c.leaf[1];
        tail += pair_any(c.leaf[1]);
        const bool n0 = pair_any(c.node[0]), n1 = pair_any(c.node[1]);
        const bool push_cur = (n0 || n1) && cur != 0, push_1 = n0 && n1;
        if (sp <= kRing - 2) {
            // two free slots above the top, as above
            ring[sp * kTraceBlock] = cur;
            sp += push_cur;
            ring[sp * kTraceBlock] = c.node[1];
            sp += push_1;
        } else {
            if (sp > kMaxStack - 2) {   // a malformed tree: deeper than any valid one
                T = __int_as_float(0x7fc00000);
                stop();
                return;
            }
            if (push_cur) push(cur);
            if (push_1) push(c.node[1]);
        }
        cur = n0 ? c.node[0] : n1 ? c.node[1] : cur;
        if (cur == 0 && sp > 0) cur = pop();
        node = cur != 0 ? pair_first_m1(cur) : kDone;
        cur = pair_rest(cur);
    }

    // First queued leaf's index less one; the queue moves on.
    __device__ __forceinline__ int32_t next_leaf() {
        Pair *slot = fifo + (head & (kFifo - 1)) * kTraceBlock;
        const Pair e = *slot;
        const Pair rest = pair_rest(e);
        *slot = rest;
        head += rest == 0;
        return pair_first_m1(e);
    }

  private:
    __device__ __forceinline__ void push(Pair x) {
        Pair *slot = ring + (sp & (kRing - 1)) * kTraceBlock;
        if (sp >= kRing) spill[sp - kRing] = *slot;
        *slot = x;
        ++sp;
    }
    __device__ __forceinline__ Pair pop() {
        --sp;
        Pair *slot = ring + (sp & (kRing - 1)) * kTraceBlock;
        const Pair x = *slot;
        if (sp >= kRing) *slot = spill[sp - kRing];
        return x;
    }
};

// Scratch of the persistent traversals' queue counters.
constexpr size_t kQueueBytes = 256;

// Enqueue the pooled traversal of listed rays on `stream` (defined with the
// traversal kernels): ray j is ids[j] + id_offset = i * K + k; its T goes to
// out[ids[j]] (out_by_value) or out[j]. With count non-null, only the first
// min(n_list, *count) entries (read on the device) are traced. Ids outside
// [0, n K) give NaN. With queues (kQueueBytes of device scratch, cleared here)
// a persistent grid takes the list's pools from per-XCD queues; without, each
// wave takes a fixed run of pools.
void launch_trace_list(const void *bvh, const rv_gaussians *g, const float *dirs, int K, const Cuts &c,
                       const int64_t *ids, int64_t n_list, const unsigned long long *count, int64_t id_offset,
                       bool out_by_value, float *out, unsigned long long *queues, hipStream_t stream);

}  // namespace rv
