"""The leaf test's addressing on the host: trace_core.h compiled for the CPU with
stand-ins for the few device built-ins it names. A tree may have 2^30 leaves of
three 16-byte words, so a leaf's first word passes 2^31 from leaf 715,827,883 on."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

HIP_STUB = r"""
#pragma once
#include <math.h>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <algorithm>
#define __device__
#define __host__
#define __forceinline__ inline
struct float4 { float x, y, z, w; };
struct uint4 { uint32_t x, y, z, w; };
typedef void *hipStream_t;
template <class To, class From> inline To bits_(From v) { To r; std::memcpy(&r, &v, 4); return r; }
inline float __int_as_float(int v) { return bits_<float>(v); }
inline int __float_as_int(float v) { return bits_<int>(v); }
inline float __uint_as_float(uint32_t v) { return bits_<float>(v); }
inline float __expf(float x) { return std::exp(x); }
inline int __lane_id() { return 0; }
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsqf(x) (1.0f / std::sqrt(x))
#define __builtin_amdgcn_perm(a, b, c) ((a) ^ (b) ^ (c))   /* box tests are not run here */
"""

PROGRAM = r"""
#include <sys/mman.h>
#include <cstdio>
#include "trace_core.h"
using namespace rv;
int main() {
    // both sides of `rec` are mapped (never touched pages take no memory), so an
    // index that wraps reads a zero record and nothing faults
    const size_t side = size_t(54) << 30;
    void *m = mmap(nullptr, 2 * side, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return 2;
    float4 *rec = reinterpret_cast<float4 *>(static_cast<char *>(m) + side);
    const int64_t leaves[] = {0, 1, 715827881, 715827882, 715827883, 715827884, (int64_t(1) << 30) - 1};
    Cuts c{};
    c.alpha_min = 1.0f / 255.0f; c.alpha_max = 0.99f; c.q_cut = 9.0f;
    NoHit none;
    for (int64_t leaf : leaves) {
        // an isotropic unit Gaussian at distance 1 on the ray
        float4 *r = rec + int64_t(3) * leaf;
        r[0] = float4{0.f, 0.f, 1.f, 0.25f};
        r[1] = float4{1.f, 0.f, 0.f, 1.f};
        r[2] = float4{0.f, 1.f, 0.f, __int_as_float(7)};
        const float f = leaf_factor(rec, (int32_t)(leaf - 1), mk(0.f, 0.f, 0.f), mk(0.f, 0.f, 1.f), 0.f, -1, -2, c, none,
                                    1.f);
        std::printf("%lld %.6f\n", (long long)leaf, f);
        r[0] = r[1] = r[2] = float4{};
    }
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm clang")
def test_leaf_records_are_reached_up_to_the_largest_tree(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP_STUB)
    (tmp_path / "main.cpp").write_text(PROGRAM)
    exe = tmp_path / "leaf_index"
    cmd = [CLANG, "-std=c++17", "-O1", "-fwrapv", "-w", "-I", str(tmp_path), "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2311_16043_amd", "csrc"), str(tmp_path / "main.cpp"), "-o", str(exe)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    if run.returncode == 2:
        pytest.skip("no address space for the sparse mapping")
    assert run.returncode == 0
    rows = [line.split() for line in run.stdout.splitlines()]
    assert len(rows) == 7
    for leaf, factor in rows:
        assert factor == "0.750000", f"leaf {leaf}: factor {factor}"
