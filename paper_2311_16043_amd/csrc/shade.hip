// shade.hip -- per-Gaussian physically based shading with pre-computed
// visibility (Sec. 3.3, Eq. (7)-(10)): for Gaussian i and its K incident
// directions w_k (the visibility rays' directions, Sec. 3.3 and 4.2)
//
//   c_i = sum_k (b / pi + f_s(w_o, w_k)) (V_ik L_env(w_k) + sum_j l_j Y_j(w_k)) max(n . w_k, 0) dw
//
// with f_s = D F G / (4 (n . w_k)(n . w_o)) (GGX D with alpha = r^2, Schlick F,
// separable Smith G), the 16 x 32 environment map sampled bilinearly, the
// indirect light as real SH of degree <= 2, and dw = 2 pi / K (4 pi / K on the
// sphere).
//
// Mapping: a wave takes a run of Gaussians, one after another, with lanes striding
// over the directions; the colour sums end with a wave reduction. What belongs to a
// Gaussian alone (frame, view direction, factors of the BRDF) is computed for the
// whole run at once, a lane each, and read back lane by lane. The map and the
// directions sit in LDS, padded to 16 bytes: a bilinear fetch is four loads of
// 16 bytes at fixed offsets, as a ring of texels around the map holds what lies
// beyond its edges.
//
// Bound by the vector ALUs (seven reciprocals and roots among 175 instructions a
// direction; a map read at one address is no faster): 300,000 x 256 takes 320 us, 430
// with a wave per Gaussian that set up the Gaussian and the map for four steps of
// the loop, scalar texel reads, and two octants and clamped columns per direction.
// In the Gaussian's frame the BRDF is 20 instructions shorter (285 us), but a narrow
// lobe multiplies what the directions are off by, 10^-7, up to a thousandfold, and
// the steps here give the same values as they always did. The SH sums by 4x4x1
// matrix instructions are as fast.
#include <cmath>
#include <type_traits>

#include "trace_core.h"

namespace rv {
namespace {

constexpr int kEnvRows = 16, kEnvCols = 32;
constexpr int kEnvPitch = kEnvCols + 2;   // texels of a padded row
constexpr int kShadeBlock = 256;
constexpr int kDirsLds = 512;   // directions in LDS; more are read from memory
// Gaussians of a wave's run at most, and waves below which runs are cut. Runs of
// 4 / 8 / 16 / 32: 299 / 287 / 294 / 364 us (the last waves end further apart).
constexpr int kShadeRun = 8;
constexpr int64_t kShadeWaves = 8192;
constexpr float kPi = 3.14159265358979323846f;

// Sum over the wave, in its last lane.
__device__ __forceinline__ float wave_sum(float v) {
    auto step = [&](auto ctrl, auto rows) {
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value,
                                                        decltype(rows)::value, 0xf, false));
    };
    using std::integral_constant;
    const integral_constant<int, 0xf> all{};
    step(integral_constant<int, 0x111>{}, all);                              // row_shr:1
    step(integral_constant<int, 0x112>{}, all);                              // row_shr:2
    step(integral_constant<int, 0x114>{}, all);                              // row_shr:4
    step(integral_constant<int, 0x118>{}, all);                              // row_shr:8
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});    // row_bcast:15
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});    // row_bcast:31
    return v;
}

// atan2(y, x) in units of pi / 16 (texels of the map) for y >= 0: pi / 4 + atan(t)
// with t = (y - |x|) / (y + |x|) in [-1, 1] by the hardware reciprocal, mirrored for
// x < 0. atan(t) = t P(t^2) with P of degree 7 fitted to atan on [0, 1] (least
// squares on Chebyshev nodes, reweighted toward the largest errors; at most 1.3e-7
// rad evaluated in binary32 by Horner's rule). 0 at the origin. Over 4 million random
// directions in a binary32 emulation, with a reciprocal off by up to one unit, the
// polar angle is within 2.6e-7 rad of its FP64 value and the azimuth within 4.7e-7 (4.1e-7
// and 7.7e-7 with the smaller of |x| / |y| and |y| / |x| and octants).
__device__ __forceinline__ float atan2_texels(float y, float x) {
    constexpr float s = 16.0f / kPi;
    const float ax = fmaxf(fabsf(x), 1e-30f);
    const float q = (y - ax) * __builtin_amdgcn_rcpf(y + ax);
    const float t = __uint_as_float(__float_as_uint(q) ^ (__float_as_uint(x) & 0x80000000u));
    const float u = t * t;
    float p = s * -0.004054537042975426f;
    p = fmaf(p, u, s * 0.021862857043743134f);
    p = fmaf(p, u, s * -0.05591219663619995f);
    p = fmaf(p, u, s * 0.09642188996076584f);
    p = fmaf(p, u, s * -0.1390862613916397f);
    p = fmaf(p, u, s * 0.19946564733982086f);
    p = fmaf(p, u, s * -0.33329859375953674f);
    p = fmaf(p, u, s * 0.9999993443489075f);
    return fmaf(t, p, 8.0f - copysignf(4.0f, x));
}

__device__ __forceinline__ f3 unit(f3 d) {
    return __builtin_amdgcn_rsqf(dot(d, d)) * d;   // one ulp; |d| is 1 up to rounding
}

// Value of lane j (wave-uniform).
__device__ __forceinline__ float from_lane(float v, int j) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}
// What a Gaussian brings to all its directions.
struct ShadePoint {
    f3 b1, b2, n;   // frame, as the visibility rays use it
    f3 wo;          // view direction
    float no;       // n . w_o
    float a2;       // alpha^2
    float spec;     // factor of the specular term: 2 G1(w_o) alpha^2 / (4 pi (n . w_o)); 0 seen from behind
    float kd[3];    // albedo / pi
};

template <bool kHemisphere>
__global__ __launch_bounds__(kShadeBlock) void k_shade(const float *__restrict__ mean, const float *__restrict__ normal,
                                                       int64_t n, const float *__restrict__ dirs, int K,
                                                       const float *__restrict__ vis, const float *__restrict__ albedo,
                                                       const float *__restrict__ roughness,
                                                       const float *__restrict__ sh, const float *__restrict__ env,
                                                       float cx, float cy, float cz, float f0, int64_t i_off, int run,
                                                       float *__restrict__ color) {
    __shared__ float4 env_s[(kEnvRows + 2) * kEnvPitch];
    __shared__ float4 dirs_s[kDirsLds];
    for (int t = threadIdx.x; t < (kEnvRows + 2) * kEnvPitch; t += kShadeBlock) {
        const int row = min(max(t / kEnvPitch - 1, 0), kEnvRows - 1), col = (t % kEnvPitch - 1) & (kEnvCols - 1);
        const float *e = env + (row * kEnvCols + col) * 3;
        env_s[t] = make_float4(e[0], e[1], e[2], 0.0f);
    }
    // direction k as given, on the sphere of unit length
    auto local_dir = [&](int k) {
        const f3 d = mk(dirs[3 * k], dirs[3 * k + 1], dirs[3 * k + 2]);
        return kHemisphere ? d : unit(d);
    };
    for (int k = threadIdx.x; k < min(K, kDirsLds); k += kShadeBlock) {
        const f3 d = local_dir(k);
        dirs_s[k] = make_float4(d.x, d.y, d.z, 0.0f);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t i0 = i_off + ((int64_t)__builtin_amdgcn_readfirstlane(blockIdx.x) * (kShadeBlock / 64) +
                                __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * run;
    if (i0 >= n) return;  // wave-uniform
    const int count = (int)min<int64_t>(run, n - i0);

    ShadePoint own;   // lane j: Gaussian i0 + j (the first again beyond the run)
    {
        const int64_t i = i0 + (lane < count ? lane : 0);
        float nx = normal[3 * i], ny = normal[3 * i + 1], nz = normal[3 * i + 2];
        const float nl = sqrtf(nx * nx + ny * ny + nz * nz);
        nx /= nl; ny /= nl; nz /= nl;
        own.n = mk(nx, ny, nz);
        onb_duff(own.n, own.b1, own.b2);
        f3 wo = mk(cx - mean[3 * i], cy - mean[3 * i + 1], cz - mean[3 * i + 2]);
        own.wo = (1.0f / sqrtf(dot(wo, wo))) * wo;
        const float no = own.no = dot(own.n, own.wo);
        const float r = roughness[i];
        own.a2 = (r * r) * (r * r);
        const float g1o = 2.0f * no / (no + sqrtf(own.a2 + (1.0f - own.a2) * no * no));
        own.spec = no > 0.0f ? g1o * own.a2 / (2.0f * kPi * no) : 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c) own.kd[c] = albedo[3 * i + c] * (1.0f / kPi);
    }
    const float dw = (kHemisphere ? 2.0f : 4.0f) * kPi / (float)K;
    const float f1 = 1.0f - f0;

    for (int j = 0; j < count; ++j) {
        const int64_t i = i0 + j;
        auto pick = [&](float v) { return from_lane(v, j); };
        auto pick3 = [&](f3 v) { return mk(pick(v.x), pick(v.y), pick(v.z)); };
        const f3 b1 = pick3(own.b1), b2 = pick3(own.b2), nrm = pick3(own.n), wo = pick3(own.wo);
        const float a2 = pick(own.a2), spec_k = pick(own.spec), rest = 1.0f - a2;
        const float kd[3] = {pick(own.kd[0]), pick(own.kd[1]), pick(own.kd[2])};
        const bool front = from_lane(own.no, j) > 0.0f;
        float l[9][3];
#pragma unroll
        for (int q = 0; q < 9; ++q)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) l[q][ch] = sh[(i * 9 + q) * 3 + ch];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) l[0][ch] *= 0.28209479177387814f;
        // a normal of no direction: no direction lies above the surface
        const float nn = dot(nrm, nrm);
        const int K_i = __builtin_amdgcn_readfirstlane(nn > 0.0f ? K : 0);

        float acc[3] = {0.f, 0.f, 0.f};
        for (int k = lane; k < K_i; k += 64) {
            f3 d;
            if (K <= kDirsLds) {
                const float4 q = dirs_s[k];
                d = mk(q.x, q.y, q.z);
            } else {
                d = local_dir(k);
            }
            const f3 w = kHemisphere ? unit(d.x * b1 + d.y * b2 + d.z * nrm) : d;
            const float ci = dot(nrm, w);
            if (!(ci > 0.0f)) continue;
            const float V = vis[i * K + k];
            // environment: bilinear at texel coordinates of (theta, phi);
            // u lies in [-0.5, 31.5], v in [-0.5, 15.5]
            const float xx = w.x * w.x;
            const float v = atan2_texels(__builtin_amdgcn_sqrtf(fmaf(w.y, w.y, xx)), w.z) - 0.5f;
            const float u = 15.5f + copysignf(atan2_texels(fabsf(w.y), w.x + 0.0f), w.y);
            const float uf = floorf(u), vf = floorf(v);
            const float fu = u - uf, fv = v - vf, gu = 1.0f - fu, gv = 1.0f - fv;
            const float at = fmaf(vf, 16.0f * kEnvPitch, fmaf(uf, 16.0f, 16.0f * (kEnvPitch + 1)));
            const float4 *e = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(env_s) + (int)at);
            const float4 e00 = e[0], e01 = e[1], e10 = e[kEnvPitch], e11 = e[kEnvPitch + 1];
            const float w00 = gu * gv, w01 = fu * gv, w10 = gu * fv, w11 = fu * fv;
            const float Le[3] = {fmaf(w11, e11.x, fmaf(w10, e10.x, fmaf(w01, e01.x, w00 * e00.x))),
                                 fmaf(w11, e11.y, fmaf(w10, e10.y, fmaf(w01, e01.y, w00 * e00.y))),
                                 fmaf(w11, e11.z, fmaf(w10, e10.z, fmaf(w01, e01.z, w00 * e00.z)))};
            // indirect light: real SH of degree <= 2
            const float x1 = 1.0925484305920792f * w.x, yz = 1.0925484305920792f * w.y * w.z;
            const float Y[9] = {1.0f, 0.4886025119029199f * w.y, 0.4886025119029199f * w.z, 0.4886025119029199f * w.x,
                                x1 * w.y, yz, fmaf(0.94617469575755997f * w.z, w.z, -0.31539156525252005f), x1 * w.z,
                                0.5462742152960396f * fmaf(-w.y, w.y, xx)};
            float Li[3];
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                float s = l[0][ch];
#pragma unroll
                for (int q = 1; q < 9; ++q) s = fmaf(l[q][ch], Y[q], s);
                Li[ch] = fmaf(V, Le[ch], s);
            }
            // specular times the cosine: D F G / (4 (n . w_o)); the GGX denominator
            // uses 1 - (n.h)^2 = |n x h|^2 to stay accurate for smooth surfaces.
            // Hardware reciprocals and roots (about 1 ulp): over 48 scenes the 2-norm of the
            // error against 64 bits is 1.634e-6 (geometric mean; largest 1.1249e-4), 1.637e-6
            // (1.1253e-4) with correctly rounded roots and octant angles; the roots take 3 to 5 %
            // more time each.
            float spec = 0.0f;
            if (front) {
                f3 h = w + wo;
                h = __builtin_amdgcn_rsqf(dot(h, h)) * h;
                const float nh = fmaxf(dot(nrm, h), 0.0f), vh = fmaxf(dot(wo, h), 0.0f);
                const f3 nxh = cross(nrm, h);
                const float t = dot(nxh, nxh) + nh * nh * a2;
                const float m = 1.0f - vh, m2 = m * m;
                const float F = fmaf(f1, m2 * m2 * m, f0);
                const float g = __builtin_amdgcn_rcpf(ci + __builtin_amdgcn_sqrtf(a2 + rest * ci * ci));
                // D F G1(w_i) G1(w_o) / (4 n.w_o) with D = alpha^2 / (pi t^2)
                spec = (spec_k * F) * (ci * g) * __builtin_amdgcn_rcpf(t * t);
            }
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) acc[ch] = fmaf(fmaf(kd[ch], ci, spec), Li[ch], acc[ch]);
        }
        const float c0 = wave_sum(acc[0]), c1 = wave_sum(acc[1]), c2 = wave_sum(acc[2]);
        if (lane == 63) {
            color[3 * i] = c0 * dw;
            color[3 * i + 1] = c1 * dw;
            color[3 * i + 2] = c2 * dw;
        }
    }
}

}  // namespace
}  // namespace rv

using namespace rv;

extern "C" rv_status rv_shade_pbr(const rv_gaussians *g, const float *dirs, int32_t K, const rv_trace_params *p,
                                  const float *vis_ray, const rv_pbr_material *m, float *color, void *stream) {
    clear_error();
    RV_REQUIRE(g && dirs && p && vis_ray && m && color, RV_ERR_INVALID_ARG, "rv_shade_pbr: null argument");
    RV_REQUIRE(g->mean && g->normal, RV_ERR_INVALID_ARG, "rv_shade_pbr: needs means and normals");
    RV_REQUIRE(m->albedo && m->roughness && m->sh && m->env, RV_ERR_INVALID_ARG, "rv_shade_pbr: null material array");
    RV_REQUIRE(g->n >= 1 && g->n <= RV_MAX_GAUSSIANS, RV_ERR_INVALID_ARG, "rv_shade_pbr: n=%lld out of range",
               (long long)g->n);
    RV_REQUIRE(K >= 1, RV_ERR_INVALID_ARG, "rv_shade_pbr: K=%d must be >= 1", K);
    RV_REQUIRE(p->dir_mode == 0 || p->dir_mode == 1, RV_ERR_INVALID_ARG, "rv_shade_pbr: dir_mode must be 0 or 1");
    RV_REQUIRE(m->f0 >= 0.0f && m->f0 <= 1.0f, RV_ERR_INVALID_ARG, "rv_shade_pbr: f0 must lie in [0, 1]");
    RV_REQUIRE(std::isfinite(m->camera[0]) && std::isfinite(m->camera[1]) && std::isfinite(m->camera[2]),
               RV_ERR_INVALID_ARG, "rv_shade_pbr: camera position is not finite");
    const int run = (int)std::min<int64_t>(kShadeRun, std::max<int64_t>(1, g->n / kShadeWaves));
    // at most 2^24 waves (2^30 work-items) per grid
    const int64_t per_block = (int64_t)run * (kShadeBlock / 64), per_launch = (int64_t(1) << 24) * run;
    const auto kernel = p->dir_mode ? k_shade<true> : k_shade<false>;
    for (int64_t i0 = 0; i0 < g->n; i0 += per_launch) {
        const int64_t cnt = std::min(per_launch, g->n - i0);
        hipLaunchKernelGGL(kernel, dim3((unsigned)((cnt + per_block - 1) / per_block)), dim3(kShadeBlock), 0,
                           (hipStream_t)stream, g->mean, g->normal, g->n, dirs, (int)K, vis_ray, m->albedo,
                           m->roughness, m->sh, m->env, m->camera[0], m->camera[1], m->camera[2], m->f0, i0, run, color);
    }
    return check_launch("rv_shade_pbr");
}
