// surrogate.hip -- MLP visibility surrogate on the gfx950 matrix cores.
//
// Every product runs as v_mfma_f32_16x16x32_bf16 in the transposed form
//   C[16 outputs x 16 samples] += A[16 outputs x 32 inputs] * B[32 inputs x 16 samples],
// so that the accumulator layout (lane = one sample, four consecutive outputs)
// is reused unchanged as the next product's B operand: a matrix product is
// invariant under a common permutation of its summation index, so the packed
// weights (A operands) are laid out in the order in which the previous layer
// leaves its outputs in the lanes (kfeat below). Activations of a 32-sample
// wave never leave registers in inference.
//
// Parameter blob: header | FP32 master | Adam m | Adam v | BF16 forward A
// operands | BF16 backward A operands (W used as [in x out] for the
// gradient through the layer).
#include "trace_core.h"

namespace rv {
namespace {

constexpr int kHid = 256, kIn = 64, kEnc = 42;
constexpr int64_t kNParams = 214530;
__host__ __device__ constexpr int64_t off_w(int l) {  // l = 0..4 (layers 1..5)
    return l == 0 ? 0 : l == 1 ? 16640 : l == 2 ? 82432 : l == 3 ? 148224 : 214016;
}
__host__ __device__ constexpr int64_t off_b(int l) {
    return l == 0 ? 16384 : l == 1 ? 82176 : l == 2 ? 147968 : l == 3 ? 213760 : 214528;
}
__host__ __device__ constexpr int n_in(int l) { return l == 0 ? kIn : kHid; }
__host__ __device__ constexpr int n_out(int l) { return l == 4 ? 2 : kHid; }
// packed A operands, in bf16 elements: forward layer l = 0..4
__host__ __device__ constexpr int64_t fwd_off(int l) {
    return l == 0 ? 0 : l == 1 ? 16384 : l == 2 ? 81920 : l == 3 ? 147456 : 212992;
}
constexpr int64_t kFwdTotal = 217088;
// backward A operands: j = 0 for W5, 1 for W4, 2 for W3, 3 for W2
__host__ __device__ constexpr int64_t bwd_off(int j) { return j == 0 ? 0 : j == 1 ? 8192 : j == 2 ? 73728 : 139264; }
constexpr int64_t kBwdTotal = 204800;

struct SurLayout {
    size_t header, master, m, v, fwd, bwd, total;
};
inline SurLayout sur_layout() {
    SurLayout L{};
    size_t off = 0;
    L.header = off; off = align_up(off + 64 * sizeof(float));
    L.master = off; off = align_up(off + kNParams * sizeof(float));
    L.m = off; off = align_up(off + kNParams * sizeof(float));
    L.v = off; off = align_up(off + kNParams * sizeof(float));
    L.fwd = off; off = align_up(off + kFwdTotal * 2);
    L.bwd = off; off = align_up(off + kBwdTotal * 2);
    L.total = off;
    return L;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}

// bfloat16 bits of x, round to nearest even (finite inputs)
__host__ __device__ __forceinline__ uint32_t bf16_bits(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
// two bfloat16 values (round to nearest even) in one word, lo in bits 0-15:
// one v_cvt_pk_bf16_f32 on gfx950
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ float bf16_val(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// ReLU of two bf16 values in one word: read as 16-bit integers, a bf16 value
// is negative exactly when its sign bit is set, so the per-half integer max
// with 0 is the ReLU (-0 becomes +0). Rounding to bf16 preserves sign and
// zero, so this equals rounding the ReLU of the FP32 values.
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t w) {
    typedef short i16x2 __attribute__((ext_vector_type(2)));
    const i16x2 z = {0, 0};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, w), z));
}

// Feature carried by slot s (0..7) of lane group g (lane / 16) in k-block kb of
// a B operand built from accumulators: blocks 2kb and 2kb+1 of 16 outputs,
// four consecutive outputs per lane group.
__host__ __device__ constexpr int kfeat(int kb, int g, int s) { return (2 * kb + (s >> 2)) * 16 + 4 * g + (s & 3); }

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9e3779b97f4a7c15ull;
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}

// ---- encoding -----------------------------------------------------------------

// The encoding of u[0..5] has seven features of each scalar: u, sin(pi u), cos(pi u),
// sin(2 pi u), cos(2 pi u), sin(4 pi u), cos(4 pi u), features 7 a .. 7 a + 6 of u[a];
// features kEnc .. 63 are 0. A wave encodes 16 samples (lane col holds sample
// col = lane % 16's scalars in all four lane groups) as rows of bf16 features in LDS:
// lane group g evaluates u[g], groups 0 and 1 also u[4 + g]. Each value is computed
// once, by lanes that take the same path; evaluated where an operand holds it, every
// lane took both branches of its features and searched each one's scalar (a training
// step of 8,192 samples: 22.5 us in k_mlp_train, 21.6 so; inference, whose time is
// the reading of weights from LDS, is as fast either way).
constexpr int kEncRow = 68;   // bf16 elements of a row (136 bytes: 64 features + padding)

// Zeros in the rows' features past the encoding.
__device__ __forceinline__ void clear_rows(uint16_t *rows, int lane) {
    for (int i = lane; i < 16 * kEncRow / 2; i += 64) reinterpret_cast<uint32_t *>(rows)[i] = 0u;
}

__device__ __forceinline__ void encode_rows(uint16_t *rows, int lane, const float (&u)[6]) {
    const int g = lane >> 4;
    uint16_t *const row = rows + (lane & 15) * kEncRow;
    auto put = [&](int a, float v) {
        constexpr float pi = 3.14159265358979323846f;
        const float e[8] = {v, __sinf(pi * v), __cosf(pi * v), __sinf(2.0f * pi * v), __cosf(2.0f * pi * v),
                            __sinf(4.0f * pi * v), __cosf(4.0f * pi * v), 0.0f};
#pragma unroll
        for (int c = 0; c < 7; c += 2) {
            const uint32_t w = pack2(e[c], e[c + 1]);
            row[7 * a + c] = (uint16_t)w;
            if (c < 6) row[7 * a + c + 1] = (uint16_t)(w >> 16);
        }
    };
    put(g, g == 0 ? u[0] : g == 1 ? u[1] : g == 2 ? u[2] : u[3]);
    if (g < 2) put(4 + g, g == 0 ? u[4] : u[5]);
}

// k-block kb (0 or 1) of the rows' samples as a B operand (features kfeat).
__device__ __forceinline__ u32x4 row_kblock(const uint16_t *rows, int kb, int lane) {
    const uint16_t *const p = rows + (lane & 15) * kEncRow + 32 * kb + 4 * (lane >> 4);
    const uint2 lo = *reinterpret_cast<const uint2 *>(p), hi = *reinterpret_cast<const uint2 *>(p + 16);
    return u32x4{lo.x, lo.y, hi.x, hi.y};
}

// Orders a wave's accesses to its rows.
__device__ __forceinline__ void rows_sync() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// ---- forward -----------------------------------------------------------------------

enum FwdMode { kModeXd = 0, kModeGrid = 1 };

struct FwdArgs {
    const float *master;
    const u32x4 *fwd;
    const float *header;
    int64_t n;               // samples (queries) in all launches of this call
    int64_t s_off;           // first sample of this launch (a grid covers at most 2^30 samples)
    // explicit inputs (xd and train)
    const float *x, *d, *T;
    // training: sample draw and saved tensors
    int hashed;              // 1: sample index = hash(seed, step, s) mod n_samples
    int64_t n_samples;
    uint64_t seed;
    int64_t step;
    uint16_t *ht;            // activations, feature-major: section j at ht + ht_off(j) * stride
    int64_t stride;          // samples per feature row (>= padded n)
    uint16_t *dz5;           // [2][stride]
    float *loss_part;        // per wave
    // outputs
    float *vis, *unc;
    // grid queries
    const float *gmean, *gnormal, *dirs;
    int K, dir_mode;
    int64_t q_begin;
    float tau;
    uint8_t *fb_flag;  // per query: 1 = to be traced (grid mode with a BVH), else NULL
};

// Training takes the batch in blocks of kTrainNT 16-sample tiles, each block
// kTrainWaves waves that split every layer's outputs (a k-block of the next
// layer's input per wave), and covers the batch rounded up to 32
// samples: the padded samples' activations and gradients are stored as zeros
// for the weight-gradient products, which step over 32 samples at a time.
constexpr int kTrainWaves = 8, kTrainNT = 2;
constexpr int64_t kTrainPad = 16 * kTrainNT > 32 ? 16 * kTrainNT : 32;
static_assert(kTrainWaves == 8 && kTrainPad % (16 * kTrainNT) == 0 && kTrainPad <= 128,
              "training block shape");
__host__ __device__ constexpr int64_t train_pad(int64_t n) { return ((n + kTrainPad - 1) / kTrainPad) * kTrainPad; }

// feature-major activation sections: HT0 (64 rows), HT1..HT4 (256 rows each)
__host__ __device__ constexpr int64_t ht_row(int j) { return j == 0 ? 0 : 64 + (int64_t)(j - 1) * 256; }
constexpr int64_t kHtRows = 64 + 4 * 256;
constexpr int64_t kDzRows = 4 * 256 + 16;  // dZ1..dZ4 (256 rows each), dZ5 (2 rows, 16 reserved)
__host__ __device__ constexpr int64_t dz_row(int l) { return l < 4 ? (int64_t)l * 256 : 1024; }  // l = 0..4

// Output blocks 2 op and 2 op + 1 of a layer (KB k-blocks of inputs): their packed
// weights, block h and k-block kb in f[2 kb + h], and the products with act.
template <int KB>
__device__ __forceinline__ void load_pair(const u32x4 *__restrict__ A, int op, int lane, u32x4 (&f)[16]) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int h = 0; h < 2; ++h) f[2 * kb + h] = A[((2 * op + h) * KB + kb) * 64 + lane];
}
template <int KB, int NT>
__device__ __forceinline__ void multiply_pair(const u32x4 (&f)[16], const u32x4 (&act)[8][NT], f32x4 (&acc)[2][NT]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[h][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            acc[0][nt] = mfma16(f[2 * kb], act[kb][nt], acc[0][nt]);
            acc[1][nt] = mfma16(f[2 * kb + 1], act[kb][nt], acc[1][nt]);
        }
}

// The word of the lane next to this one (lanes 2c and 2c+1 swap): one DPP
// quad permute [1, 0, 3, 2].
__device__ __forceinline__ uint32_t pair_swap(uint32_t w) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, false);
}

// Feature-major rows are written and read two samples (one 32-bit word) per
// lane: in a word holding rows ra (low halves) and rb (high halves) of this
// lane's sample, the even lane of a pair (samples s, s + 1) takes row ra of
// both samples and the odd lane (samples s - 1, s) row rb of both.
__device__ __forceinline__ uint32_t pair_row_word(uint32_t own, bool odd) {
    const uint32_t nb = pair_swap(own);
    return odd ? ((nb >> 16) | (own & 0xffff0000u)) : ((own & 0xffffu) | (nb << 16));
}

// Store k-block kb of a tile's B operand (features kfeat(kb, ., .)) as
// feature-major rows of ht, samples at or past n as zeros.
__device__ __forceinline__ void store_kblock(uint16_t *__restrict__ ht, int64_t stride, const u32x4 &frag, int kb,
                                             int lane, int64_t s_base, int64_t n) {
    const int g = lane >> 4, col = lane & 15;
    const bool odd = col & 1;
    const int64_t s2 = s_base + (col & ~1);   // first sample of the lane pair
    const uint32_t keep = (s2 < n ? 0x0000ffffu : 0u) | (s2 + 1 < n ? 0xffff0000u : 0u);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t word = pair_row_word(frag[w], odd) & keep;
        const int f = kfeat(kb, g, 2 * w + (odd ? 1 : 0));
        *reinterpret_cast<uint32_t *>(ht + (int64_t)f * stride + s2) = word;
    }
}

// x mapped from [lo, hi] to [-1, 1].
__device__ __forceinline__ float to_box(float x, float lo, float hi) {
    const float span = hi - lo;
    return span > 0.f ? 2.0f * (x - lo) / span - 1.0f : 0.0f;
}

// The encoded inputs of NT tiles of 16 samples from s_base as B operands
// (k-blocks 0 and 1 of act; features kfeat), through the wave's rows.
template <int kMode, int NT>
__device__ __forceinline__ void encode_tiles(const FwdArgs &a, int64_t s_base, int lane, u32x4 (&act)[8][NT],
                                             uint16_t *rows) {
    const int col = lane & 15;
    const float lo0 = a.header[0], lo1 = a.header[1], lo2 = a.header[2];
    const float hi0 = a.header[3], hi1 = a.header[4], hi2 = a.header[5];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int64_t s = s_base + nt * 16 + col;
        const bool valid = s < a.n;
        // grid queries q = i K + k: the tile's first query is split once per
        // wave (scalar), each lane's is at most 15 further on
        int64_t gi = 0;
        int gk = 0;
        if (kMode == kModeGrid) {
            const int64_t qt = a.q_begin + s_base + nt * 16;
            const int64_t q0 = ((int64_t)__builtin_amdgcn_readfirstlane((int)(qt >> 32)) << 32) |
                               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)qt);
            const int64_t i0 = q0 / a.K;
            gi = i0;
            gk = (int)(q0 - i0 * a.K) + col;
            while (gk >= a.K) {
                gk -= a.K;
                ++gi;
            }
        }
        float x0 = 0.f, x1 = 0.f, x2 = 0.f, d0 = 0.f, d1 = 0.f, d2 = 1.f;
        if (valid) {
            if (kMode == kModeGrid) {
                const int64_t i = gi;
                const int k = gk;
                float nx = 0.f, ny = 0.f, nz = 1.f;
                if (a.gnormal) {
                    nx = a.gnormal[3 * i]; ny = a.gnormal[3 * i + 1]; nz = a.gnormal[3 * i + 2];
                    const float nl = sqrtf(nx * nx + ny * ny + nz * nz);
                    nx /= nl; ny /= nl; nz /= nl;
                }
                f3 b1, b2;
                const f3 nv = mk(nx, ny, nz);
                onb_duff(nv, b1, b2);
                const f3 dv = ray_direction(a.dirs, k, a.dir_mode, nv, b1, b2);
                x0 = a.gmean[3 * i]; x1 = a.gmean[3 * i + 1]; x2 = a.gmean[3 * i + 2];
                d0 = dv.x; d1 = dv.y; d2 = dv.z;
            } else {
                x0 = a.x[3 * s]; x1 = a.x[3 * s + 1]; x2 = a.x[3 * s + 2];
                d0 = a.d[3 * s]; d1 = a.d[3 * s + 1]; d2 = a.d[3 * s + 2];
            }
        }
        const float u[6] = {to_box(x0, lo0, hi0), to_box(x1, lo1, hi1), to_box(x2, lo2, hi2), d0, d1, d2};
        encode_rows(rows, lane, u);
        rows_sync();
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) act[kb][nt] = row_kblock(rows, kb, lane);
        rows_sync();
    }
}

// One block of eight waves takes two 16-sample tiles of the batch through the
// network and back. Of every hidden layer's 16 output blocks (8 k-blocks of the
// next layer's input) wave w produces k-block w, and of every input gradient
// likewise; the waves exchange each layer's result through LDS (double-buffered, one
// barrier per layer). Activations and gradients leave as feature-major rows for the
// weight gradients; the ReLU masks stay in the registers of the wave that made
// them. The head and its gradient are every wave's own.
//
// A block reads all 830 KB of packed weights, and with one block per CU (8,192
// samples) that and the latency between its layers are the bound: a layer's weights
// are fetched before the barrier that its inputs wait for. 21.6 us at 8,192 samples,
// against 18.9 + 20.6 us as two kernels that fetched weights after the barrier, read
// the masks back from memory and encoded every sample in all eight waves.
// Registers (227) leave a CU one block, so 8,320 samples take a second round; four whole
// steps, those kernels / this one: 222 / 144 us at 1,024 samples, 260 / 170 at 8,192, 282 / 241
// at 8,320, 341 / 273 at 16,384, 428 / 372 at 16,512, 583 / 488 at 32,768, 2,901 / 1,899 at 131,072.
__global__ __launch_bounds__(kTrainWaves * 64, 16 / kTrainWaves) void k_mlp_train(FwdArgs a, const u32x4 *__restrict__ bwd,
                                                                                 uint16_t *__restrict__ dz) {
    constexpr int NT = kTrainNT;
    static_assert(kTrainWaves == 8 && NT == 2, "the encoding is split over the waves");
    __shared__ u32x4 xb[2][8][NT][64];
    __shared__ __align__(16) uint16_t rows[NT][16 * kEncRow];
    __shared__ float target[16 * NT];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t tile = blockIdx.x;
    const int64_t s_base = tile * (16 * NT);
    if (s_base >= train_pad(a.n)) return;  // block-uniform
    const int g = lane >> 4, col = lane & 15;
    const float *master = a.master;
    u32x4 f[16], act[8][NT];   // weights and inputs of a layer
    uint64_t relu = 0;         // the wave's outputs above zero, 16 bits a hidden layer
    f32x4 acc[2][NT];
    load_pair<2>(a.fwd + fwd_off(0) / 8, w, lane, f);

    // encode: wave w < 2 tile w
    if (w < NT) {
        clear_rows(rows[w], lane);
        const int64_t s = s_base + w * 16 + col;
        float x0 = 0.f, x1 = 0.f, x2 = 0.f, d0 = 0.f, d1 = 0.f, d2 = 1.f, T = 0.f;
        if (s < a.n) {
            int64_t idx = s;
            if (a.hashed)
                idx = (int64_t)(splitmix64(a.seed ^ splitmix64((uint64_t)a.step * 0x100000000ull + (uint64_t)s)) %
                                (uint64_t)a.n_samples);
            x0 = a.x[3 * idx]; x1 = a.x[3 * idx + 1]; x2 = a.x[3 * idx + 2];
            d0 = a.d[3 * idx]; d1 = a.d[3 * idx + 1]; d2 = a.d[3 * idx + 2];
            T = a.T[idx];
        }
        const float u[6] = {to_box(x0, a.header[0], a.header[3]), to_box(x1, a.header[1], a.header[4]),
                            to_box(x2, a.header[2], a.header[5]), d0, d1, d2};
        rows_sync();
        encode_rows(rows[w], lane, u);
        if (g == 0) target[w * 16 + col] = T;
    }
    __syncthreads();
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) act[kb][nt] = row_kblock(rows[nt], kb, lane);
    if (w < 2) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            store_kblock(a.ht + ht_row(0) * a.stride, a.stride, row_kblock(rows[nt], w, lane), w, lane, s_base + 16 * nt,
                         a.n);
    }

    // the rest of hidden layer l, its products in acc: the wave's k-block for all
    // waves and the next layer's inputs. Loops over layers stay rolled: each
    // instruction is run once or thrice a block, and fetching it counts.
    auto bias_of = [&](int l, float4 (&bv)[2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            bv[h] = *reinterpret_cast<const float4 *>(master + off_b(l) + (2 * w + h) * 16 + 4 * g);
    };
    auto exchange = [&](const u32x4 (&o)[NT], int buf) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) xb[buf][w][nt][lane] = o[nt];
        __syncthreads();
#pragma unroll
        for (int kb = 0; kb < 8; ++kb)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) act[kb][nt] = xb[buf][kb][nt][lane];
    };
    auto finish = [&](int l, const float4 (&bv)[2]) {
        // bias in FP32, one v_cvt_pk_bf16_f32 per pair, then the ReLU on the packed word
        u32x4 o[NT];
        uint32_t bits = 0;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int h = q >> 1, r = 2 * (q & 1);
                const uint32_t v = relu_bf16x2(pack2(acc[h][nt][r] + (r ? bv[h].z : bv[h].x),
                                                     acc[h][nt][r + 1] + (r ? bv[h].w : bv[h].y)));
                o[nt][q] = v;
                bits |= ((v & 0xffffu) != 0u ? 1u : 0u) << (8 * nt + 2 * q) | ((v >> 16) != 0u ? 2u : 0u) << (8 * nt + 2 * q);
            }
        relu |= (uint64_t)bits << (16 * l);
        exchange(o, l & 1);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            store_kblock(a.ht + ht_row(l + 1) * a.stride, a.stride, o[nt], w, lane, s_base + 16 * nt, a.n);
    };
    float4 bv[2];
    bias_of(0, bv);
    multiply_pair<2, NT>(f, act, acc);
    load_pair<8>(a.fwd + fwd_off(1) / 8, w, lane, f);
    finish(0, bv);
#pragma unroll 1
    for (int l = 1; l < 4; ++l) {
        bias_of(l, bv);
        multiply_pair<8, NT>(f, act, acc);
        if (l < 3) {
            load_pair<8>(a.fwd + fwd_off(l + 1) / 8, w, lane, f);
        } else {
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) f[kb] = a.fwd[fwd_off(4) / 8 + kb * 64 + lane];
        }
        finish(l, bv);
    }

    // head: one block of 16 outputs, rows 0 and 1 are z0, z1
    f32x4 acc5[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc5[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc5[nt] = mfma16(f[kb], act[kb][nt], acc5[nt]);
    load_pair<1>(bwd + bwd_off(0) / 8, w, lane, f);
    const float b50 = master[off_b(4)], b51 = master[off_b(4) + 1];
    const float inv_n = 1.0f / (float)a.n;
    float lsum = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int64_t s = s_base + 16 * nt + col;
        const bool valid = s < a.n;
        const float z0 = acc5[nt][0] + b50, z1 = acc5[nt][1] + b51;
        const float V = 1.0f / (1.0f + expf(-z0));
        const float U = z1;   // predicted |T - V|, linear (no saturating activation)
        const float T = target[16 * nt + col];
        const float e = fabsf(T - V);
        // squared error of U against |T - V| (V held constant)
        const uint32_t dz0 = valid ? bf16_bits((V - T) * inv_n) : 0u;
        const uint32_t dz1 = valid ? bf16_bits(2.0f * (U - e) * inv_n) : 0u;
        // as a B operand: outputs 0 and 1 sit in slots 0, 1 of lane group 0
        act[0][nt] = u32x4{g == 0 ? (dz0 & 0xffffu) | (dz1 << 16) : 0u, 0u, 0u, 0u};
        if (w == 0 && g == 0) {
            a.dz5[s] = (uint16_t)dz0;
            a.dz5[a.stride + s] = (uint16_t)dz1;
            if (valid) {
                const float bce = -(T * logf(fmaxf(V, 1e-12f)) + (1.f - T) * logf(fmaxf(1.f - V, 1e-12f)));
                lsum += bce + (U - e) * (U - e);
            }
        }
    }
    if (w == 0) {
        for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off);
        if (lane == 0) a.loss_part[tile] = lsum;
    }

    // back: j = 0 through W5 (gradient dZ4), .., j = 3 through W2 (dZ1)
    auto back = [&](int j) {
        u32x4 o[NT];
        const uint32_t bits = (uint32_t)(relu >> (16 * (3 - j)));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            // the ReLU mask of the layer's input; none of a padded sample
            const uint32_t m = s_base + 16 * nt + col < a.n ? bits >> (8 * nt) : 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int h = q >> 1, r = 2 * (q & 1);
                o[nt][q] = pack2((m >> (2 * q)) & 1u ? acc[h][nt][r] : 0.0f, (m >> (2 * q)) & 2u ? acc[h][nt][r + 1] : 0.0f);
            }
        }
        if (j < 3) exchange(o, j & 1);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            store_kblock(dz + dz_row(3 - j) * a.stride, a.stride, o[nt], w, lane, s_base + 16 * nt, a.n);
    };
    multiply_pair<1, NT>(f, act, acc);
    load_pair<8>(bwd + bwd_off(1) / 8, w, lane, f);
    back(0);
#pragma unroll 1
    for (int j = 1; j < 4; ++j) {
        multiply_pair<8, NT>(f, act, acc);
        if (j < 3) load_pair<8>(bwd + bwd_off(j + 1) / 8, w, lane, f);
        back(j);
    }
}

// ---- inference with the weights staged through LDS ------------------------------
//
// Inference takes 32 samples per wave (two tiles) and eight waves per block,
// one block per CU (two waves per SIMD). The waves of a block share every
// weight fragment: the packed A operands are streamed layer by layer, in
// chunks of at most 64 KB, into one of two LDS buffers by direct
// global-to-LDS loads (no registers held), the next chunk loading while the
// current one is multiplied, one barrier per chunk (eight per 256 samples).
// Every A operand is then read from LDS. When each wave fetched all 424 KB of
// packed weights itself (48 samples per wave), those fetches ran at the rate
// of the CU's vector-memory path (TD busy 96 %) and held the matrix cores at
// 42 % of peak. Three tiles per wave do not fit 256 registers next to the LDS
// pipeline (the compiler spills ~150).
constexpr int kInferWaves = 8;
constexpr int kInferNT = 2;
constexpr int kInferSamples = kInferWaves * 16 * kInferNT;  // 256 per block
constexpr int kChunkVec = 4096;                             // 16-byte vectors per LDS buffer (64 KB)

typedef __attribute__((address_space(3))) void lds_void;

// This wave's share of copying `count` vectors (a multiple of 64) of packed
// operands from src to the LDS buffer dst: the 1 KB pieces wv, wv + 8, ...
// (a global_load_lds_dwordx4 writes 16 bytes per lane from the wave's LDS base).
__device__ __forceinline__ void load_chunk(const u32x4 *__restrict__ src, int count, u32x4 *dst, int wv, int lane) {
    for (int p = wv; p < count / 64; p += kInferWaves)
        __builtin_amdgcn_global_load_lds(static_cast<const void *>(src + p * 64 + lane),
                                         (lds_void *)(dst + p * 64), 16, 0, 0);
}

// This wave's loads into LDS have landed, then every wave's have, and every
// wave has finished reading the buffer the next loads will overwrite.
__device__ __forceinline__ void chunk_barrier() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// Output pairs [OP0, OP0 + NOP) of a layer (the same arithmetic as multiply_pair's)
// from the LDS chunk holding their A operands. Each k-block's two operands are read
// two k-blocks before its products: 2.93 ms for 6.4M queries with the reads right
// before the products, 2.63 one k-block ahead, 2.56 two (the scheduling groups hold
// the reads there; with half of them left out 2.01, with the epilogue left out 2.48).
template <int KB, int NT, int OP0, int NOP>
__device__ __forceinline__ void layer_ops_lds(const u32x4 *A, const float *__restrict__ bias,
                                              const u32x4 (&act)[8][NT], u32x4 (&out)[8][NT], int lane) {
    const int g = lane >> 4;
    // the operands of the next two k-blocks are read while this one is multiplied
    u32x4 n0 = A[lane], n1 = A[KB * 64 + lane], m0 = A[64 + lane], m1 = A[(KB + 1) * 64 + lane];
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int o = 0; o < NOP; ++o) {
        f32x4 acc[2][NT];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[h][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const u32x4 a0 = n0, a1 = n1;
            n0 = m0;
            n1 = m1;
            const int on = kb + 2 < KB ? o : o + 1, kn = kb + 2 < KB ? kb + 2 : kb + 2 - KB;
            if (on < NOP) {
                m0 = A[((2 * on) * KB + kn) * 64 + lane];
                m1 = A[((2 * on + 1) * KB + kn) * 64 + lane];
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                acc[0][nt] = mfma16(a0, act[kb][nt], acc[0][nt]);
                acc[1][nt] = mfma16(a1, act[kb][nt], acc[1][nt]);
            }
            if (on < NOP) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 2 * NT, 0);
        }
        // bias in FP32, then the bf16 pair, then the ReLU on the packed words
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float4 bv = *reinterpret_cast<const float4 *>(bias + (2 * (OP0 + o) + h) * 16 + 4 * g);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                out[OP0 + o][nt][2 * h + 0] = relu_bf16x2(pack2(acc[h][nt][0] + bv.x, acc[h][nt][1] + bv.y));
                out[OP0 + o][nt][2 * h + 1] = relu_bf16x2(pack2(acc[h][nt][2] + bv.z, acc[h][nt][3] + bv.w));
            }
        }
    }
}

// A 256 -> 256 layer from two LDS chunks (output pairs 0-3, then 4-7);
// `between` runs once the first half is done (the chunk hand-over). The
// output array is local, so the input array's registers are reused as soon as
// the layer ends.
template <int NT, class Between>
__device__ __forceinline__ void hidden_layer_lds(const u32x4 *A_lo, const u32x4 *A_hi, const float *__restrict__ bias,
                                                 u32x4 (&act)[8][NT], int lane, Between between) {
    u32x4 out[8][NT];
    layer_ops_lds<8, NT, 0, 4>(A_lo, bias, act, out, lane);
    between();
    layer_ops_lds<8, NT, 4, 4>(A_hi, bias, act, out, lane);
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) act[kb][nt] = out[kb][nt];
}

// Chunks, in 16-byte vectors of the packed forward operands: layer 1 whole
// (2,048), layers 2-4 in halves of four output pairs (4,096 each), the head
// (512). Chunk c is multiplied from buffer c % 2 while chunk c + 1 loads into
// the other. A k-block's two LDS reads are scheduled two k-blocks before its
// products: hoisted further, as the compiler otherwise does, they spill the
// activations.
template <int kMode>
__global__ __launch_bounds__(kInferWaves * 64, 1) void k_mlp_forward(FwdArgs a) {
    constexpr int NT = kInferNT;
    __shared__ u32x4 wbuf[2][kChunkVec];
    __shared__ __align__(16) uint16_t rows[kInferWaves][16 * kEncRow];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int g = lane >> 4, col = lane & 15;
    // every wave takes part in the loads and barriers; waves past the end
    // encode zeros and write nothing
    const int64_t s_base = a.s_off + ((int64_t)blockIdx.x * kInferWaves + wv) * (16 * NT);
    const u32x4 *F = a.fwd;
    const float *master = a.master;
    load_chunk(F + fwd_off(0) / 8, 2048, wbuf[0], wv, lane);
    u32x4 act[8][NT];
    clear_rows(rows[wv], lane);
    rows_sync();
    encode_tiles<kMode, NT>(a, s_base, lane, act, rows[wv]);
    chunk_barrier();
    // layer 1 (64 -> 256) from buffer 0; layer 2's first half loads into buffer 1
    load_chunk(F + fwd_off(1) / 8, kChunkVec, wbuf[1], wv, lane);
    {
        u32x4 out[8][NT];
        layer_ops_lds<2, NT, 0, 8>(wbuf[0], master + off_b(0), act, out, lane);
#pragma unroll
        for (int kb = 0; kb < 8; ++kb)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) act[kb][nt] = out[kb][nt];
    }
    chunk_barrier();
    // layers 2-4, each from buffer 1 (first half) then buffer 0 (second half)
    // while the following chunk loads into the other buffer
#pragma unroll
    for (int l = 1; l <= 3; ++l) {
        load_chunk(F + fwd_off(l) / 8 + kChunkVec, kChunkVec, wbuf[0], wv, lane);
        hidden_layer_lds<NT>(wbuf[1], wbuf[0], master + off_b(l), act, lane, [&]() {
            chunk_barrier();
            if (l < 3) load_chunk(F + fwd_off(l + 1) / 8, kChunkVec, wbuf[1], wv, lane);
            else load_chunk(F + fwd_off(4) / 8, 512, wbuf[1], wv, lane);
        });
        chunk_barrier();
    }
    // head: one block of 16 outputs, rows 0 and 1 are z0, z1
    f32x4 acc5[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc5[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
        const u32x4 av = wbuf[1][kb * 64 + lane];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc5[nt] = mfma16(av, act[kb][nt], acc5[nt]);
    }
    const float b50 = master[off_b(4)], b51 = master[off_b(4) + 1];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int64_t s = s_base + nt * 16 + col;
        if (g == 0 && s < a.n) {
            const float z0 = acc5[nt][0] + b50, z1 = acc5[nt][1] + b51;
            const float V = 1.0f / (1.0f + expf(-z0));
            const float U = z1;
            a.vis[s] = V;
            if (a.unc) a.unc[s] = U;
            if (kMode == kModeGrid && a.fb_flag) a.fb_flag[s] = U > a.tau ? 1 : 0;
        }
    }
}

// ---- weight gradients ----------------------------------------------------------------

// One block of eight waves: a 128 x 128 tile of dW_l[k][o] = sum_s h[k][s]
// dz[o][s] over one slice of the batch, wave w holding 64 rows k (half w / 4) by 32
// outputs o (quarter w % 4) as C[k][o] += A[k x 32 samples] B[32 samples x o], plus
// the bias gradient of its outputs when it holds the layer's first 64 rows. Each
// stage of 64 samples (two products of 32, in order; samples past the slice as
// zeros) brings the tile's 128 h rows and 128 dz rows (128 bytes each) to LDS once for
// all waves (double-buffered, one barrier per stage); rows are padded to 144 bytes
// so that a fragment read (16 rows x 16 bytes per lane group) hits 16 distinct bank
// quadruples. 8,192 samples are 256 blocks, one per CU, so what counts is the
// latency of a stage: 17.0 us, against 20.6 with four waves and 32 samples.
struct WgradArgs {
    const uint16_t *ht, *dz;
    int64_t stride;
    int64_t n_pad;       // samples covered (a multiple of 32)
    int64_t slice_len;   // multiple of 32
    int n_slices;
    float *partial;      // [n_slices][n_params]
};

// tiles per slice: l0 (64 x 256): 1 x 2, l1-3 (256 x 256): 2 x 2, l4 (256 x 2): 2 x 1 -> 16
__device__ __forceinline__ void tile_of(int t, int &l, int &kt, int &ot) {
    if (t < 2) { l = 0; kt = 0; ot = t; return; }
    t -= 2;
    if (t < 12) { l = 1 + t / 4; kt = (t % 4) / 2; ot = t % 2; return; }
    t -= 12;
    l = 4; kt = t; ot = 0;
}
constexpr int kTiles = 16;
constexpr int kWgStage = 64;   // samples of a stage
constexpr int kWgRow = 72;     // LDS row stride in bf16 elements (144 bytes: 64 samples + padding)

__global__ __launch_bounds__(512) void k_mlp_wgrad(WgradArgs a) {
    __shared__ __align__(16) uint16_t hs[2][128 * kWgRow];
    __shared__ __align__(16) uint16_t ds[2][128 * kWgRow];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int tile = (int)(blockIdx.x % kTiles);
    const int slice = (int)(blockIdx.x / kTiles);
    int l, kt, ot;
    tile_of(tile, l, kt, ot);
    const int Nin = n_in(l), Nout = n_out(l);
    const int k0 = kt * 128, o0 = ot * 128;
    const uint16_t *H = a.ht + ht_row(l) * a.stride;
    const uint16_t *D = a.dz + dz_row(l) * a.stride;
    const int64_t s0 = (int64_t)slice * a.slice_len;
    const int64_t s1 = min(a.n_pad, s0 + a.slice_len);
    // staging: thread t moves 16-byte part t % 8 of rows t / 8 and 64 + t / 8, of h
    // and of dz (rows past the layer's inputs or outputs as zeros). A stage's rows
    // are fetched into registers two stages before they are written to LDS.
    const int srow = threadIdx.x >> 3, spart = threadIdx.x & 7;
    auto fetch = [&](int64_t s, u32x4 (&r)[4]) {
        if (s >= s1) return;
        const bool in = s + 8 * spart < s1;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int row = srow + 64 * u;
            r[2 * u] = in && k0 + row < Nin
                           ? *reinterpret_cast<const u32x4 *>(H + (int64_t)(k0 + row) * a.stride + s + 8 * spart)
                           : u32x4{0u, 0u, 0u, 0u};
            r[2 * u + 1] = in && o0 + row < Nout
                               ? *reinterpret_cast<const u32x4 *>(D + (int64_t)(o0 + row) * a.stride + s + 8 * spart)
                               : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto put = [&](const u32x4 (&r)[4], int buf) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int row = srow + 64 * u;
            *reinterpret_cast<u32x4 *>(&hs[buf][row * kWgRow + 8 * spart]) = r[2 * u];
            *reinterpret_cast<u32x4 *>(&ds[buf][row * kWgRow + 8 * spart]) = r[2 * u + 1];
        }
    };
    const int wk = w >> 2, wo = w & 3;
    // a wave whose part lies past the layer's inputs or outputs only stages
    const bool live = k0 + 64 * wk < Nin && o0 + 32 * wo < Nout;
    const bool bias = live && k0 + 64 * wk == 0;
    const int g = lane >> 4, col = lane & 15;
    f32x4 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum[2] = {0.f, 0.f};
    // products of the samples staged in buffer buf
    auto stage = [&](int buf) {
        if (!live) return;
#pragma unroll
        for (int x = 0; x < kWgStage; x += 32) {
            u32x4 av[4], bv[2];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                av[i] = *reinterpret_cast<const u32x4 *>(&hs[buf][(64 * wk + 16 * i + col) * kWgRow + x + 8 * g]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                bv[j] = *reinterpret_cast<const u32x4 *>(&ds[buf][(32 * wo + 16 * j + col) * kWgRow + x + 8 * g]);
            if (bias) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) bsum[j] += bf16_val(bv[j][q] & 0xffffu) + bf16_val(bv[j][q] >> 16);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mfma16(av[i], bv[j], acc[i][j]);
        }
    };
    u32x4 ra[4], rb[4];
    fetch(s0, ra);
    fetch(s0 + kWgStage, rb);
    put(ra, 0);
    fetch(s0 + 2 * kWgStage, ra);
    __syncthreads();
    // two stages per pass: buffer 0 holds stage s, registers rb the next and ra the
    // one after
    for (int64_t s = s0; s < s1; s += 2 * kWgStage) {
        stage(0);
        if (s + kWgStage < s1) put(rb, 1);
        fetch(s + 3 * kWgStage, rb);
        __syncthreads();
        if (s + kWgStage >= s1) break;
        stage(1);
        if (s + 2 * kWgStage < s1) put(ra, 0);
        fetch(s + 4 * kWgStage, ra);
        __syncthreads();
    }
    if (!live) return;
    float *P = a.partial + (int64_t)slice * kNParams;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int o = o0 + 32 * wo + j * 16 + col;
            if (o < Nout) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = k0 + 64 * wk + i * 16 + 4 * g + r;
                    P[off_w(l) + (int64_t)k * Nout + o] = acc[i][j][r];
                }
            }
        }
    if (bias) {
        // lanes col, col+16, col+32, col+48 hold the same output: add the four groups in a fixed order
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float v = bsum[j];
            const float v1 = __shfl(v, col + 16), v2 = __shfl(v, col + 32), v3 = __shfl(v, col + 48);
            const float v0 = __shfl(v, col);
            const int o = o0 + 32 * wo + j * 16 + col;
            if (g == 0 && o < Nout) P[off_b(l) + o] = ((v0 + v1) + v2) + v3;
        }
    }
}

// grad[p] = sum over slices (in order) of partial[slice][p], eight loads in
// flight per thread; loss = sum of the wave partials / n, by the first wave of
// block 0 (lane l takes partials l, l + 64, ..., then a fixed butterfly).
__global__ __launch_bounds__(256) void k_reduce_grad(const float *__restrict__ partial, int n_slices,
                                                     float *__restrict__ grad, const float *__restrict__ loss_part,
                                                     int64_t n_waves, int64_t n, float *__restrict__ loss_out) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kNParams) {
        float s = 0.f;
        int i = 0;
        for (; i + 8 <= n_slices; i += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = partial[(int64_t)(i + u) * kNParams + p];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; i < n_slices; ++i) s += partial[(int64_t)i * kNParams + p];
        grad[p] = s;
    }
    if (blockIdx.x == 0 && threadIdx.x < 64 && loss_out) {
        double s = 0.0;
        for (int64_t w = threadIdx.x; w < n_waves; w += 64) s += loss_part[w];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (threadIdx.x == 0) *loss_out = (float)(s / (double)n);
    }
}

// ---- optimiser and packing ---------------------------------------------------------------

// BF16 A operands from the FP32 master weights (see kfeat).
__global__ __launch_bounds__(256) void k_pack(const float *__restrict__ master, uint16_t *__restrict__ fwd,
                                              uint16_t *__restrict__ bwd) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < kFwdTotal) {
        int l = 0;
        while (l < 4 && e >= fwd_off(l + 1)) ++l;
        const int64_t r = e - fwd_off(l);
        const int KB = n_in(l) / 32;
        const int s = (int)(r & 7), lane = (int)((r >> 3) & 63);
        const int64_t blk = r >> 9;
        const int kb = (int)(blk % KB), ob = (int)(blk / KB);
        const int o = ob * 16 + (lane & 15), k = kfeat(kb, lane >> 4, s);
        const float w = (o < n_out(l)) ? master[off_w(l) + (int64_t)k * n_out(l) + o] : 0.0f;
        fwd[e] = (uint16_t)bf16_bits(w);
    } else if (e < kFwdTotal + kBwdTotal) {
        const int64_t eb = e - kFwdTotal;
        int j = 0;
        while (j < 3 && eb >= bwd_off(j + 1)) ++j;
        const int l = 4 - j;  // layer index of the weights
        const int64_t r = eb - bwd_off(j);
        const int KB = (l == 4) ? 1 : 8;
        const int s = (int)(r & 7), lane = (int)((r >> 3) & 63);
        const int64_t blk = r >> 9;
        const int kb = (int)(blk % KB), mb = (int)(blk / KB);
        const int k = mb * 16 + (lane & 15), o = kfeat(kb, lane >> 4, s);
        const float w = (o < n_out(l)) ? master[off_w(l) + (int64_t)k * n_out(l) + o] : 0.0f;
        bwd[eb] = (uint16_t)bf16_bits(w);
    }
}

// Positions of weight W_l[k][o] (l = 0..4) in the packed operands: its
// forward A-operand element, and for l >= 1 its backward A-operand element
// (the inverse of the element -> weight map of k_pack).
__device__ __forceinline__ int64_t fwd_pos(int l, int k, int o) {
    const int KB = n_in(l) / 32;
    const int kb = k >> 5, g = (k & 15) >> 2, sl = ((k & 31) >> 4) * 4 + (k & 3);
    const int64_t blk = (int64_t)(o >> 4) * KB + kb;
    return fwd_off(l) + blk * 512 + (g * 16 + (o & 15)) * 8 + sl;
}
__device__ __forceinline__ int64_t bwd_pos(int l, int k, int o) {
    const int KB = (l == 4) ? 1 : 8;
    const int kb = o >> 5, g = (o & 15) >> 2, sl = ((o & 31) >> 4) * 4 + (o & 3);
    const int64_t blk = (int64_t)(k >> 4) * KB + kb;
    return bwd_off(4 - l) + blk * 512 + (g * 16 + (k & 15)) * 8 + sl;
}

// One training step's update, fused per parameter: the gradient as the
// in-order sum of the slice partials (as k_reduce_grad), the Adam update with
// bias-corrected moments (c1 = 1 - beta1^t, c2 = 1 - beta2^t), and the bf16
// copies of a weight in the packed operands (as k_pack; the padding elements
// stay the zeros written at initialisation). The loss is summed as in
// k_reduce_grad.
__global__ __launch_bounds__(256) void k_adam_pack(const float *__restrict__ partial, int n_slices,
                                                   float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                                                   uint16_t *__restrict__ fwd, uint16_t *__restrict__ bwd, float lr,
                                                   float beta1, float beta2, float eps, float c1, float c2,
                                                   const float *__restrict__ loss_part, int64_t n_waves, int64_t n,
                                                   float *__restrict__ loss_out) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kNParams) {
        float gr = 0.f;
        int i = 0;
        for (; i + 8 <= n_slices; i += 8) {
            float vs[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) vs[u] = partial[(int64_t)(i + u) * kNParams + p];
#pragma unroll
            for (int u = 0; u < 8; ++u) gr += vs[u];
        }
        for (; i < n_slices; ++i) gr += partial[(int64_t)i * kNParams + p];
        const float mm = beta1 * m[p] + (1.f - beta1) * gr;
        const float vv = beta2 * v[p] + (1.f - beta2) * gr * gr;
        m[p] = mm;
        v[p] = vv;
        const float wn = w[p] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
        w[p] = wn;
        int l = 0;
        while (l < 4 && p >= off_w(l + 1)) ++l;
        const int64_t r = p - off_w(l);
        if (r < (int64_t)n_in(l) * n_out(l)) {   // a weight (the layer's biases follow its weights)
            const int k = (int)(r / n_out(l)), o = (int)(r - (int64_t)k * n_out(l));
            const uint16_t b = (uint16_t)bf16_bits(wn);
            fwd[fwd_pos(l, k, o)] = b;
            if (l >= 1) bwd[bwd_pos(l, k, o)] = b;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < 64 && loss_out) {
        double s = 0.0;
        for (int64_t q = threadIdx.x; q < n_waves; q += 64) s += loss_part[q];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (threadIdx.x == 0) *loss_out = (float)(s / (double)n);
    }
}

// He-uniform from a counter-based hash, zero biases.
__global__ __launch_bounds__(256) void k_init_hash(float *__restrict__ master, uint64_t seed) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kNParams) return;
    int l = 0;
    while (l < 4 && p >= off_w(l + 1)) ++l;
    if (p >= off_b(l)) {
        master[p] = 0.0f;
        return;
    }
    const float lim = sqrtf(6.0f / (float)n_in(l));
    const uint64_t h = splitmix64(seed ^ splitmix64((uint64_t)p));
    const float u = (float)(h >> 40) * (1.0f / 16777216.0f);  // [0, 1)
    master[p] = (2.0f * u - 1.0f) * lim;
}

__global__ __launch_bounds__(256) void k_copy_f32(const float *__restrict__ src, float *__restrict__ dst, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

__global__ __launch_bounds__(256) void k_fill_f32(float *__restrict__ p, int64_t n, float v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ __launch_bounds__(64) void k_set_header(float *__restrict__ h, float l0, float l1, float l2, float h0,
                                                   float h1, float h2) {
    if (threadIdx.x == 0) {
        h[0] = l0; h[1] = l1; h[2] = l2; h[3] = h0; h[4] = h1; h[5] = h2;
        for (int i = 6; i < 64; ++i) h[i] = 0.0f;
    }
}

// ---- fallback tracing and ray setup -----------------------------------------------------------------

__global__ void k_store_count(const unsigned long long *__restrict__ count, int64_t *__restrict__ out) {
    if (threadIdx.x == 0) *out = (int64_t)*count;
}

// Fallback list in the BVH's leaf (Morton) order, direction by direction:
// one wave per group of 64 consecutive sorted positions (lane l holds
// Gaussian i = src(64 g + l)) appends the group's flagged queries that lie
// in [q_begin, q_begin + q_count) as positions s = q - q_begin, direction k
// by direction k and lane by lane within a direction, after one atomic
// reservation per group. A pool of consecutive list entries then holds rays
// of nearby Gaussians in the same few directions, which walk the same part of
// the tree together. The list order between groups depends on scheduling;
// each ray's result does not.
__global__ __launch_bounds__(256) void k_fallback_rows(const float *__restrict__ header,
                                                       const float4 *__restrict__ rec, int64_t n, int K,
                                                       int64_t q_begin, int64_t q_count,
                                                       const uint8_t *__restrict__ flag,
                                                       unsigned long long *__restrict__ count,
                                                       int64_t *__restrict__ list) {
    const int lane = threadIdx.x & 63;
    const uint64_t lt = (1ull << lane) - 1ull;
    const int64_t n_groups = (n + 63) / 64;
    // with a tree built for another Gaussian set the records are not read:
    // Gaussians are taken in index order (the traversal then gives NaN)
    const bool tree_ok = tree_matches(header, n);
    const bool aligned = K % 16 == 0 && q_begin % 16 == 0;
    for (int64_t grp = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); grp < n_groups; grp += (int64_t)gridDim.x * 4) {
        const int64_t m = grp * 64 + lane;
        // this lane's Gaussian and the directions of it that lie in the range
        int64_t row = 0;  // s of direction 0
        int k_lo = 0, k_hi = 0;
        if (m < n) {
            const int64_t i = tree_ok ? (int64_t)__float_as_int(rec[kLeafF4 * m + 2].w) : m;
            row = i * K - q_begin;
            // clamped to [0, K] in 64 bits: rows far outside the range give k_lo >= k_hi
            k_lo = (int)min<int64_t>(K, max<int64_t>(0, -row));
            k_hi = (int)max<int64_t>(0, min<int64_t>(K, q_count - row));
        }
        const bool any = __ballot(k_lo < k_hi) != 0;
        if (!any) continue;  // wave-uniform
        int total = 0;
        unsigned long long base = 0;
        if (aligned) {
            // rows start on 16-byte boundaries: 16 flags per lane per load
            // (the flag buffer is padded to 256 bytes, so a row's last load
            // stays inside it); two passes, counting then writing
            for (int pass = 0; pass < 2; ++pass) {
                for (int k0 = 0; k0 < K; k0 += 16) {
                    u32x4 w = u32x4{0u, 0u, 0u, 0u};
                    if (k0 + 16 > k_lo && k0 < k_hi)
                        w = *reinterpret_cast<const u32x4 *>(flag + row + k0);
#pragma unroll
                    for (int u = 0; u < 16; ++u) {
                        const int k = k0 + u;
                        const bool f = k >= k_lo && k < k_hi && ((w[u >> 2] >> (8 * (u & 3))) & 0xffu) != 0;
                        const uint64_t b = __ballot(f);
                        if (pass == 0) {
                            total += __popcll(b);
                        } else {
                            if (f) list[base + __popcll(b & lt)] = row + k;
                            base += __popcll(b);
                        }
                    }
                }
                if (pass == 0) {
                    if (total == 0) break;
                    if (lane == 0) base = atomicAdd(count, (unsigned long long)total);
                    base = __shfl(base, 0);
                }
            }
            continue;
        }
        for (int k = 0; k < K; ++k) {
            const bool f = k >= k_lo && k < k_hi && flag[row + k] != 0;
            total += __popcll(__ballot(f));
        }
        if (total == 0) continue;
        if (lane == 0) base = atomicAdd(count, (unsigned long long)total);
        base = __shfl(base, 0);
        for (int k = 0; k < K; ++k) {
            const bool f = k >= k_lo && k < k_hi && flag[row + k] != 0;
            const uint64_t b = __ballot(f);
            if (f) list[base + __popcll(b & lt)] = row + k;
            base += __popcll(b);
        }
    }
}

__global__ __launch_bounds__(256) void k_ray_setup(const float *__restrict__ mean, const float *__restrict__ normal,
                                                   int64_t n, const float *__restrict__ dirs, int K, int dir_mode,
                                                   const int64_t *__restrict__ ids, int64_t n_rays,
                                                   float *__restrict__ out_o, float *__restrict__ out_d) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_rays) return;
    const int64_t r = ids[s];
    if (r < 0 || r >= n * (int64_t)K) {
        const float nan = __int_as_float(0x7fc00000);
        for (int a = 0; a < 3; ++a) out_o[3 * s + a] = out_d[3 * s + a] = nan;
        return;
    }
    const int64_t i = r / K;
    const int k = (int)(r - i * K);
    float nx = 0.f, ny = 0.f, nz = 1.f;
    if (normal) {
        nx = normal[3 * i]; ny = normal[3 * i + 1]; nz = normal[3 * i + 2];
        const float nl = sqrtf(nx * nx + ny * ny + nz * nz);
        nx /= nl; ny /= nl; nz /= nl;
    }
    const f3 nrm = mk(nx, ny, nz);
    f3 b1, b2;
    onb_duff(nrm, b1, b2);
    const f3 d = ray_direction(dirs, k, dir_mode, nrm, b1, b2);
    out_o[3 * s] = mean[3 * i]; out_o[3 * s + 1] = mean[3 * i + 1]; out_o[3 * s + 2] = mean[3 * i + 2];
    out_d[3 * s] = d.x; out_d[3 * s + 1] = d.y; out_d[3 * s + 2] = d.z;
}

// ---- training workspace --------------------------------------------------------------------------------

// The weight gradients are summed over at most kMaxSlices slices of the
// batch (a multiple of 32 samples each), so that the 16 tiles of every slice
// give 256 blocks whatever the batch; the slice partials are added in order.
constexpr int kMaxSlices = 16;
inline int64_t slice_len_for(int64_t n_pad) {
    const int64_t per = (n_pad + kMaxSlices - 1) / kMaxSlices;
    return std::max<int64_t>(32, ((per + 31) / 32) * 32);
}
inline int slices_for(int64_t n_pad) {
    const int64_t len = slice_len_for(n_pad);
    return (int)((n_pad + len - 1) / len);
}

struct TrainWs {
    size_t ht, dz, partial, loss_part, loss, total;
    int64_t stride, n_slices, n_waves;
};

inline TrainWs train_ws(int64_t batch) {
    TrainWs W{};
    const int64_t pad = ((batch + 127) / 128) * 128;
    W.stride = pad;
    W.n_slices = kMaxSlices;
    W.n_waves = train_pad(batch) / (16 * kTrainNT);   // one loss partial per training block
    size_t off = 0;
    W.ht = off; off = align_up(off + (size_t)kHtRows * pad * 2);
    W.dz = off; off = align_up(off + (size_t)kDzRows * pad * 2);
    W.partial = off; off = align_up(off + (size_t)W.n_slices * kNParams * 4);
    W.loss_part = off; off = align_up(off + (size_t)W.n_waves * 4);
    W.loss = off; off = align_up(off + 256);
    W.total = off;
    return W;
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }
// Samples per inference launch: a dispatch counts its work-items in 32 bits,
// so one grid stays at 2^30 samples (below 2^31 work-items at 48 samples per
// wave).
constexpr int64_t kLaunchSamples = int64_t(1) << 30;

// forward (train) + backward + weight gradients + reduction on samples [0, n)
// With grad == nullptr the slice partials are left for k_adam_pack.
rv_status loss_grad_impl(const void *params, const float *x, const float *d, const float *T, int64_t n, bool hashed,
                         int64_t n_samples, uint64_t seed, int64_t step, float *grad, float *loss_out, void *ws,
                         const TrainWs &W, hipStream_t s) {
    const SurLayout L = sur_layout();
    const int64_t n_pad = train_pad(n);
    FwdArgs fa{};
    fa.master = at<float>(params, L.master);
    fa.fwd = at<u32x4>(params, L.fwd);
    fa.header = at<float>(params, L.header);
    fa.n = n;
    fa.x = x;
    fa.d = d;
    fa.T = T;
    fa.hashed = hashed ? 1 : 0;
    fa.n_samples = n_samples;
    fa.seed = seed;
    fa.step = step;
    fa.ht = at<uint16_t>(ws, W.ht);
    fa.stride = W.stride;
    fa.dz5 = at<uint16_t>(ws, W.dz) + dz_row(4) * W.stride;
    fa.loss_part = at<float>(ws, W.loss_part);
    const int64_t tiles = n_pad / (16 * kTrainNT);   // one block per kTrainNT 16-sample tiles
    hipLaunchKernelGGL(k_mlp_train, dim3((unsigned)tiles), dim3(kTrainWaves * 64), 0, s, fa, at<u32x4>(params, L.bwd),
                       at<uint16_t>(ws, W.dz));
    WgradArgs wa{};
    wa.ht = at<uint16_t>(ws, W.ht);
    wa.dz = at<uint16_t>(ws, W.dz);
    wa.stride = W.stride;
    wa.n_pad = n_pad;
    wa.slice_len = slice_len_for(n_pad);
    wa.n_slices = slices_for(n_pad);
    wa.partial = at<float>(ws, W.partial);
    hipLaunchKernelGGL(k_mlp_wgrad, dim3((unsigned)(kTiles * wa.n_slices)), dim3(512), 0, s, wa);
    if (grad)
        hipLaunchKernelGGL(k_reduce_grad, dim3(blocks_for(kNParams, 256)), dim3(256), 0, s, wa.partial, wa.n_slices,
                           grad, at<float>(ws, W.loss_part), tiles, n, loss_out);
    return check_launch("surrogate loss/gradient");
}

}  // namespace
}  // namespace rv

using namespace rv;

extern "C" int64_t rv_surrogate_n_params(void) { return kNParams; }

extern "C" size_t rv_surrogate_bytes(void) { return sur_layout().total; }

extern "C" rv_status rv_surrogate_view(const void *params, rv_surrogate_arrays *out) {
    clear_error();
    RV_REQUIRE(params && out, RV_ERR_INVALID_ARG, "rv_surrogate_view: null pointer");
    const SurLayout L = sur_layout();
    void *p = const_cast<void *>(params);
    out->header = at<float>(p, L.header);
    out->master = at<float>(p, L.master);
    out->adam_m = at<float>(p, L.m);
    out->adam_v = at<float>(p, L.v);
    out->packed = at<char>(p, L.fwd);
    return RV_OK;
}

extern "C" size_t rv_surrogate_train_workspace_bytes(int32_t batch) {
    if (batch < 1) return 0;
    return train_ws(batch).total;
}

// Inference scratch: the fallback count (256 bytes); the tracer's queue counters;
// the list of q_count int64; q_count flags.
constexpr size_t kInferList = kAlign + kQueueBytes;
extern "C" size_t rv_surrogate_infer_workspace_bytes(int64_t q_count) {
    if (q_count < 0) return 0;
    return kInferList + align_up((size_t)q_count * sizeof(int64_t)) + align_up((size_t)q_count);
}

extern "C" rv_status rv_surrogate_init(void *params, uint64_t seed, const float *box_lo_host, const float *box_hi_host,
                                       const float *init_weights, void *stream) {
    clear_error();
    RV_REQUIRE(params && box_lo_host && box_hi_host, RV_ERR_INVALID_ARG, "rv_surrogate_init: null argument");
    RV_REQUIRE(((uintptr_t)params % kAlign) == 0, RV_ERR_INVALID_ARG, "rv_surrogate_init: params not 256-byte aligned");
    const SurLayout L = sur_layout();
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_set_header, dim3(1), dim3(64), 0, s, at<float>(params, L.header), box_lo_host[0],
                       box_lo_host[1], box_lo_host[2], box_hi_host[0], box_hi_host[1], box_hi_host[2]);
    if (init_weights)
        hipLaunchKernelGGL(k_copy_f32, dim3(blocks_for(kNParams, 256)), dim3(256), 0, s, init_weights,
                           at<float>(params, L.master), kNParams);
    else
        hipLaunchKernelGGL(k_init_hash, dim3(blocks_for(kNParams, 256)), dim3(256), 0, s, at<float>(params, L.master),
                           seed);
    hipLaunchKernelGGL(k_fill_f32, dim3(blocks_for(kNParams, 256)), dim3(256), 0, s, at<float>(params, L.m), kNParams,
                       0.0f);
    hipLaunchKernelGGL(k_fill_f32, dim3(blocks_for(kNParams, 256)), dim3(256), 0, s, at<float>(params, L.v), kNParams,
                       0.0f);
    hipLaunchKernelGGL(k_pack, dim3(blocks_for(kFwdTotal + kBwdTotal, 256)), dim3(256), 0, s,
                       at<float>(params, L.master), at<uint16_t>(params, L.fwd), at<uint16_t>(params, L.bwd));
    return check_launch("rv_surrogate_init");
}

extern "C" rv_status rv_surrogate_loss_grad(const void *params, const float *x, const float *d, const float *T,
                                            int64_t n, float *grad_out, float *loss_out, void *ws, size_t ws_bytes,
                                            void *stream) {
    clear_error();
    RV_REQUIRE(params && x && d && T && grad_out && ws, RV_ERR_INVALID_ARG, "rv_surrogate_loss_grad: null argument");
    RV_REQUIRE(n >= 1 && n <= (1LL << 30), RV_ERR_INVALID_ARG, "rv_surrogate_loss_grad: n out of range");
    RV_REQUIRE(((uintptr_t)ws % kAlign) == 0, RV_ERR_INVALID_ARG, "rv_surrogate_loss_grad: ws not 256-byte aligned");
    const TrainWs W = train_ws(n);
    RV_REQUIRE(ws_bytes >= W.total, RV_ERR_WORKSPACE, "rv_surrogate_loss_grad: ws_bytes %zu < %zu", ws_bytes, W.total);
    return loss_grad_impl(params, x, d, T, n, false, n, 0, 0, grad_out, loss_out, ws, W, (hipStream_t)stream);
}

extern "C" rv_status rv_surrogate_train(void *params, const float *x, const float *d, const float *T,
                                        int64_t n_samples, const rv_train_opts *o, float *loss_log, void *ws,
                                        size_t ws_bytes, void *stream) {
    clear_error();
    RV_REQUIRE(params && x && d && T && o && ws, RV_ERR_INVALID_ARG, "rv_surrogate_train: null argument");
    RV_REQUIRE(n_samples >= 1, RV_ERR_INVALID_ARG, "rv_surrogate_train: n_samples < 1");
    RV_REQUIRE(o->steps >= 0 && o->batch >= 128 && o->batch % 128 == 0, RV_ERR_INVALID_ARG,
               "rv_surrogate_train: need steps >= 0 and batch a positive multiple of 128");
    RV_REQUIRE(o->lr >= 0.f && o->beta1 >= 0.f && o->beta1 < 1.f && o->beta2 >= 0.f && o->beta2 < 1.f && o->eps > 0.f,
               RV_ERR_INVALID_ARG, "rv_surrogate_train: bad optimiser settings");
    RV_REQUIRE(((uintptr_t)ws % kAlign) == 0, RV_ERR_INVALID_ARG, "rv_surrogate_train: ws not 256-byte aligned");
    const TrainWs W = train_ws(o->batch);
    RV_REQUIRE(ws_bytes >= W.total, RV_ERR_WORKSPACE, "rv_surrogate_train: ws_bytes %zu < %zu", ws_bytes, W.total);
    const SurLayout L = sur_layout();
    hipStream_t s = (hipStream_t)stream;
    const int64_t n_pad = train_pad(o->batch);
    const int n_slices = slices_for(n_pad);
    const int64_t n_parts = n_pad / (16 * kTrainNT);
    for (int64_t it = 0; it < o->steps; ++it) {
        const int64_t gstep = o->step0 + it;
        rv_status st = loss_grad_impl(params, x, d, T, o->batch, true, n_samples, o->seed, gstep, nullptr, nullptr,
                                      ws, W, s);
        if (st != RV_OK) return st;
        // cosine-decayed step size and bias corrections (host arithmetic, FP64)
        double lr = o->lr;
        if (o->total_steps > 0) {
            double t = (double)std::min<int64_t>(std::max<int64_t>(gstep, 0), o->total_steps) / (double)o->total_steps;
            lr = o->lr_min + 0.5 * (o->lr - o->lr_min) * (1.0 + std::cos(3.14159265358979323846 * t));
        }
        const double tt = (double)(gstep + 1);
        const float c1 = (float)(1.0 - std::pow((double)o->beta1, tt));
        const float c2 = (float)(1.0 - std::pow((double)o->beta2, tt));
        hipLaunchKernelGGL(k_adam_pack, dim3(blocks_for(kNParams, 256)), dim3(256), 0, s, at<float>(ws, W.partial),
                           n_slices, at<float>(params, L.master), at<float>(params, L.m), at<float>(params, L.v),
                           at<uint16_t>(params, L.fwd), at<uint16_t>(params, L.bwd), (float)lr, o->beta1, o->beta2,
                           o->eps, c1, c2, at<float>(ws, W.loss_part), n_parts, (int64_t)o->batch,
                           loss_log ? loss_log + it : nullptr);
        st = check_launch("rv_surrogate_train");
        if (st != RV_OK) return st;
    }
    return RV_OK;
}

extern "C" rv_status rv_surrogate_infer_xd(const void *params, const float *x, const float *d, int64_t n, float *vis,
                                           float *unc, void *stream) {
    clear_error();
    RV_REQUIRE(params && vis && (n == 0 || (x && d)), RV_ERR_INVALID_ARG, "rv_surrogate_infer_xd: null argument");
    RV_REQUIRE(n >= 0, RV_ERR_INVALID_ARG, "rv_surrogate_infer_xd: n < 0");
    if (n == 0) return RV_OK;
    const SurLayout L = sur_layout();
    FwdArgs fa{};
    fa.master = at<float>(params, L.master);
    fa.fwd = at<u32x4>(params, L.fwd);
    fa.header = at<float>(params, L.header);
    fa.n = n;
    fa.x = x;
    fa.d = d;
    fa.vis = vis;
    fa.unc = unc;
    for (int64_t off = 0; off < n; off += kLaunchSamples) {
        fa.s_off = off;
        const int64_t cnt = std::min(kLaunchSamples, n - off);
        hipLaunchKernelGGL(k_mlp_forward<kModeXd>, dim3(blocks_for(cnt, kInferSamples)), dim3(kInferWaves * 64), 0,
                           (hipStream_t)stream, fa);
    }
    return check_launch("rv_surrogate_infer_xd");
}

extern "C" rv_status rv_surrogate_infer(const void *params, const void *bvh, const rv_gaussians *g, const float *dirs,
                                        int32_t K, const rv_trace_params *p, int64_t q_begin, int64_t q_count,
                                        float tau, float *vis, float *unc, int64_t *n_fallback, void *ws,
                                        size_t ws_bytes, void *stream) {
    clear_error();
    RV_REQUIRE(params && g && dirs && p && vis, RV_ERR_INVALID_ARG, "rv_surrogate_infer: null argument");
    RV_REQUIRE(g->mean && g->log_scale && g->n >= 1 && g->n <= RV_MAX_GAUSSIANS && K >= 1, RV_ERR_INVALID_ARG,
               "rv_surrogate_infer: bad scene (null arrays, n out of range or K < 1)");
    RV_REQUIRE(p->dir_mode == 0 || (p->dir_mode == 1 && g->normal), RV_ERR_INVALID_ARG,
               "rv_surrogate_infer: bad dir_mode or missing normals");
    RV_REQUIRE(p->sigma_cut > 0.0f && p->sigma_cut <= kBuildSigma && p->alpha_min > 0.0f && p->alpha_max < 1.0f &&
                   p->T_min >= 0.0f && p->T_min < 1.0f,
               RV_ERR_INVALID_ARG, "rv_surrogate_infer: bad trace parameters");
    RV_REQUIRE(q_begin >= 0 && q_count >= 0 && q_begin + q_count <= g->n * (int64_t)K, RV_ERR_INVALID_ARG,
               "rv_surrogate_infer: query range outside [0, n*K)");
    if (q_count == 0) return RV_OK;
    RV_REQUIRE(ws && ((uintptr_t)ws % kAlign) == 0, RV_ERR_INVALID_ARG, "rv_surrogate_infer: ws missing or unaligned");
    RV_REQUIRE(ws_bytes >= rv_surrogate_infer_workspace_bytes(q_count), RV_ERR_WORKSPACE,
               "rv_surrogate_infer: ws_bytes %zu < %zu", ws_bytes, rv_surrogate_infer_workspace_bytes(q_count));
    const SurLayout L = sur_layout();
    hipStream_t s = (hipStream_t)stream;
    unsigned long long *count = at<unsigned long long>(ws, 0);
    unsigned long long *queues = at<unsigned long long>(ws, kAlign);
    int64_t *list = at<int64_t>(ws, kInferList);
    uint8_t *flag = at<uint8_t>(ws, kInferList + align_up((size_t)q_count * sizeof(int64_t)));
    hipLaunchKernelGGL(k_fill_f32, dim3(1), dim3(256), 0, s, reinterpret_cast<float *>(count), (int64_t)2, 0.0f);
    FwdArgs fa{};
    fa.master = at<float>(params, L.master);
    fa.fwd = at<u32x4>(params, L.fwd);
    fa.header = at<float>(params, L.header);
    fa.n = q_count;
    fa.vis = vis;
    fa.unc = unc;
    fa.gmean = g->mean;
    fa.gnormal = p->dir_mode ? g->normal : nullptr;
    fa.dirs = dirs;
    fa.K = K;
    fa.dir_mode = p->dir_mode;
    fa.q_begin = q_begin;
    fa.tau = tau;
    fa.fb_flag = bvh ? flag : nullptr;
    for (int64_t off = 0; off < q_count; off += kLaunchSamples) {
        fa.s_off = off;
        const int64_t cnt = std::min(kLaunchSamples, q_count - off);
        hipLaunchKernelGGL(k_mlp_forward<kModeGrid>, dim3(blocks_for(cnt, kInferSamples)), dim3(kInferWaves * 64), 0,
                           s, fa);
    }
    if (bvh) {
        const Cuts c = make_cuts(*p);
        // the compacted fallback list holds positions s; the ray is q_begin + s
        const BvhLayout BL = bvh_layout(g->n);
        const int64_t rows_blocks = std::min<int64_t>(((g->n + 63) / 64 + 3) / 4, int64_t(1) << 16);
        hipLaunchKernelGGL(k_fallback_rows, dim3((unsigned)rows_blocks), dim3(256), 0, s, at<float>(bvh, BL.header),
                           at<float4>(bvh, BL.leaf_rec),
                           g->n, (int)K, q_begin, q_count, flag, count, list);
        launch_trace_list(bvh, g, dirs, K, c, (const int64_t *)list, q_count, (const unsigned long long *)count,
                          q_begin, true, vis, queues, s);
        if (n_fallback)
            hipLaunchKernelGGL(k_store_count, dim3(1), dim3(64), 0, s, (const unsigned long long *)count, n_fallback);
    } else if (n_fallback) {
        hipLaunchKernelGGL(k_fill_f32, dim3(1), dim3(64), 0, s, reinterpret_cast<float *>(n_fallback), (int64_t)2,
                           0.0f);
    }
    return check_launch("rv_surrogate_infer");
}

extern "C" rv_status rv_ray_setup(const rv_gaussians *g, const float *dirs, int32_t K, const rv_trace_params *p,
                                  const int64_t *ray_ids, int64_t n, float *out_o, float *out_d, void *stream) {
    clear_error();
    RV_REQUIRE(g && dirs && p && g->mean, RV_ERR_INVALID_ARG, "rv_ray_setup: null argument");
    RV_REQUIRE(g->n >= 1 && g->n <= RV_MAX_GAUSSIANS && K >= 1 && n >= 0, RV_ERR_INVALID_ARG,
               "rv_ray_setup: bad sizes");
    RV_REQUIRE(p->dir_mode == 0 || (p->dir_mode == 1 && g->normal), RV_ERR_INVALID_ARG,
               "rv_ray_setup: bad dir_mode or missing normals");
    if (n == 0) return RV_OK;
    RV_REQUIRE(ray_ids && out_o && out_d, RV_ERR_INVALID_ARG, "rv_ray_setup: null ids or outputs");
    hipLaunchKernelGGL(k_ray_setup, dim3(blocks_for(n, 256)), dim3(256), 0, (hipStream_t)stream, g->mean,
                       p->dir_mode ? g->normal : nullptr, g->n, dirs, K, p->dir_mode, ray_ids, n, out_o, out_d);
    return check_launch("rv_ray_setup");
}
