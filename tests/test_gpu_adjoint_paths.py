"""The adjoint's routes (one pool per wave, queues, queues with chained records):
each against the oracle's analytic FP64 gradient on the rays of adjacent
Gaussians, and against each other over all rays."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_16043_amd import Gaussians, TraceParams, build_bvh, trace_visibility, trace_visibility_backward
from workloads import scenes

pytestmark = pytest.mark.gpu

NO_EXIT = TraceParams(T_min=0.0)
KAPPA_G = 8.0   # as in test_gpu_adjoint.py


# 64 Gaussians and one direction to a pool: 16,000 pools are the last that get a
# wave each, 40,000 the last whose records are not chained
@pytest.mark.parametrize("n,K,use_fwd", [(777, 33, True), (16_000, 64, False), (16_001, 64, True), (40_000, 64, False),
                                         (40_064, 64, True)])
def test_routes_match_oracle_on_adjacent_gaussians(n, K, use_fwd):
    print(f"[adjoint paths] n={n} K={K}", flush=True)
    sc = scenes.make_object_scene(n, 5)
    dirs = scenes.fibonacci_dirs(K, True)
    mean = np.asarray(sc["mean"], np.float64)
    near = np.sort(np.argsort(((mean - mean[n // 2]) ** 2).sum(1))[:150])
    rays = (near[:, None] * K + np.arange(K)[None]).reshape(-1).astype(np.int64)
    orc = oracle.trace_rays(sc, dirs, 1, rays)
    w = np.random.default_rng(n).uniform(-1.0, 1.0, rays.size)
    w[(orc["n_amb"] > 0) | (orc["n_near_clamp"] > 0)] = 0.0
    ref = oracle.grad_rays(sc, dirs, 1, rays, w)
    sens = oracle.grad_rays(sc, dirs, 1, rays, w, absolute=2)
    full = np.zeros(n * K, np.float32)
    full[rays] = w
    g = Gaussians.from_scene(sc)
    bvh = build_bvh(g)
    fwd = trace_visibility(bvh, g, dirs, NO_EXIT)[0] if use_fwd else None
    got = trace_visibility_backward(bvh, g, dirs, NO_EXIT, grad_vis_ray=torch.from_numpy(full.reshape(n, K)),
                                    vis_ray_fwd=fwd)
    for name, x in zip(("opacity", "mean", "log_scale"), got):
        exp = ref[name]
        rms = float(np.sqrt(np.mean(exp[np.nonzero(exp)] ** 2)))
        tol = 1e-3 * np.maximum(np.abs(exp), 1e-3 * rms) + KAPPA_G * sens[name]
        assert np.all(np.abs(x.cpu().numpy().astype(np.float64) - exp) <= tol), name


def test_all_rays_in_one_call_and_in_parts():
    """All directions at once (40,064 pools: chained records), or 24 and 40 of them
    (15,024 pools: one per wave; 25,040: queues), accumulated. A hit's terms are
    the same bits, so the results differ by the order of the sums: about 64 x 12
    terms of either sign per Gaussian, 2 * 768 * 2^-24 in the 2-norm."""
    n, K = 40_064, 64
    sc = scenes.make_object_scene(n, 6)
    dirs = scenes.fibonacci_dirs(K, True)
    g = Gaussians.from_scene(sc)
    bvh = build_bvh(g)
    w = torch.from_numpy(np.random.default_rng(1).uniform(-1.0, 1.0, (n, K)).astype(np.float32)).cuda()
    whole = trace_visibility_backward(bvh, g, dirs, NO_EXIT, grad_vis_ray=w)
    parts = [trace_visibility_backward(bvh, g, dirs[a:b], NO_EXIT, grad_vis_ray=w[:, a:b].contiguous())
             for a, b in ((0, 24), (24, K))]
    for x, p, q in zip(whole, *parts):
        y = p.double() + q.double()
        assert float((x.double() - y).norm() / y.norm()) <= 2 * 768 * 2.0 ** -24
        assert float(y.norm()) > 0



# 1,024 rays are the last without accumulators, 1,024 Gaussians the last whose records
# are chained in small launches; 5,000 pools (8,000 with the forward's T, 16,000 on up to
# 2,048 Gaussians) the last that get a wave each, 18,000 the last that are dealt
@pytest.mark.parametrize("n,K,use_fwd", [(256, 4, False), (257, 4, True), (1024, 312, False), (1024, 313, False),
                                         (1025, 313, True), (2048, 500, True), (2048, 501, True), (2049, 243, True),
                                         (4000, 285, False), (4000, 286, True)])
def test_routes_of_small_launches(n, K, use_fwd):
    test_routes_match_oracle_on_adjacent_gaussians(n, K, use_fwd)


@pytest.mark.parametrize("n,K", [(300, 1200), (1000, 300), (1000, 1200)])
def test_few_gaussians_in_one_call_and_in_parts(n, K):
    """A dense cloud whose hits repeat few leaves (chained records, one pool per wave or
    dealt) against the sum over calls of three directions each (1,024 rays or fewer at
    n = 300: no accumulators). Up to 10^5 terms reach a Gaussian, and roundings of
    FP32 sums of m terms grow as sqrt(m) 2^-24, 2 10^-5 of the sum: 10^-4 in the 2-norm."""
    sc = scenes.make_cube_cloud(n, 0)
    sc["log_scale"] += np.float32(2.0)
    sc["opacity"] *= np.float32(0.1)
    dirs = scenes.fibonacci_dirs(K, False)
    prm = TraceParams(T_min=0.0, dir_mode=0)
    g = Gaussians.from_scene(sc)
    bvh = build_bvh(g)
    w = torch.from_numpy(np.random.default_rng(2).uniform(0.0, 1.0, (n, K)).astype(np.float32)).cuda()
    fwd = trace_visibility(bvh, g, dirs, prm)[0]
    whole = trace_visibility_backward(bvh, g, dirs, prm, grad_vis_ray=w, vis_ray_fwd=fwd)
    again = trace_visibility_backward(bvh, g, dirs, prm, grad_vis_ray=w)
    sums = [torch.zeros_like(x, dtype=torch.float64) for x in whole]
    for a in range(0, K, 3):
        part = trace_visibility_backward(bvh, g, dirs[a:a + 3], prm, grad_vis_ray=w[:, a:a + 3].contiguous(),
                                         vis_ray_fwd=fwd[:, a:a + 3].contiguous())
        for s, x in zip(sums, part):
            s += x.double()
    for x, y, s in zip(whole, again, sums):
        assert float(s.norm()) > 0
        assert float((x.double() - s).norm() / s.norm()) <= 1e-4
        assert float((y.double() - s).norm() / s.norm()) <= 1e-4
