"""The traversal's routes (one pool per wave, queues with few or many pools,
list runs) against each other bit for bit, and against the FP64 oracle on
sampled rays; walks whose stacks leave LDS."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_16043_amd import Gaussians, TraceParams, build_bvh, trace_rays, trace_stats, trace_visibility
from workloads import scenes

from _parity import check_vis

pytestmark = pytest.mark.gpu


def _check(sc, K, mode, label, sample=256):
    n = sc["mean"].shape[0]
    print(f"[paths] {label} n={n} K={K}", flush=True)
    prm = TraceParams(dir_mode=mode)
    dirs = scenes.fibonacci_dirs(K, mode == 1)
    g = Gaussians.from_scene(sc)
    bvh = build_bvh(g)
    vr, vm = trace_visibility(bvh, g, dirs, prm)
    ids = scenes.sample_ray_ids(n, K, 300_000, seed=n + K)
    got = trace_rays(bvh, g, dirs, ids, prm)
    flat = vr.reshape(-1)
    assert torch.equal(flat[torch.from_numpy(ids).cuda()], got), "list and all-ray values differ"
    few = trace_rays(bvh, g, dirs, ids[:97], prm)
    assert torch.equal(few, got[:97])
    assert torch.allclose(vm.double(), vr.double().mean(1), rtol=0, atol=1e-7)
    st = trace_stats(bvh, g, dirs, prm)
    assert st["hits"] <= st["leaves"]
    sub = ids[:: max(1, ids.size // sample)]
    orc = oracle.trace_rays(sc, dirs, mode, sub)
    check_vis(flat.cpu().numpy()[sub], orc, label=label)


# 64 Gaussians and one direction to a pool: 24,000 pools are the last that get a
# wave each, 40,000 the last of the smallest persistent grid
@pytest.mark.parametrize("n,K", [(24_000, 64), (24_001, 64), (40_000, 64), (40_064, 64)])
def test_pool_counts_where_the_route_changes(n, K):
    _check(scenes.make_object_scene(n, 1), K, 1, f"object-{n}x{K}")


@pytest.mark.parametrize("n,K", [(4097, 24), (1, 3), (2, 1)])
def test_deep_walks_and_smallest_trees(n, K):
    sc = scenes.make_cube_cloud(n, 0)
    if n > 2:
        # clusters at halving distances from a corner give a tree of many levels;
        # wide Gaussians make a ray enter nearly all of it
        level = np.arange(n) % 20
        sc["mean"] = (sc["mean"] * np.float32(2.0) ** (-2 - level)[:, None] * np.float32(0.25)
                      + np.float32(2.0) ** (-level)[:, None]).astype(np.float32)
        sc["log_scale"][:] = np.log(np.float32(0.3))
        sc["opacity"][:] = np.float32(0.02)
    if n == 1:
        g = Gaussians.from_scene(sc)
        vr, _ = trace_visibility(build_bvh(g), g, scenes.fibonacci_dirs(K, False), TraceParams(dir_mode=0))
        assert torch.equal(vr, torch.ones_like(vr))
        return
    _check(sc, K, 0, f"comb-{n}x{K}", sample=64)


def test_few_rays_of_a_large_tree():
    sc = scenes.make_object_scene(60_000, 1)
    _check(sc, 1, 1, "object-60000x1")


# 10,000 pools are the last that get a wave each (24,000 with up to 256 Gaussians);
# beyond, they are dealt in chunks of 64, the last one partial
@pytest.mark.parametrize("n,K", [(10_000, 63), (10_000, 64), (256, 6000), (256, 6001), (257, 2003), (12_345, 61)])
def test_dealt_pools(n, K):
    _check(scenes.make_object_scene(n, 1), K, 1, f"object-{n}x{K}")


def test_dealt_pools_of_a_dense_scene():
    sc = scenes.make_cube_cloud(12_000, 0)
    sc["log_scale"] += np.float32(1.0)
    sc["opacity"] *= np.float32(0.1)
    _check(sc, 64, 0, "dense-12000x64", sample=64)


def test_dealt_pools_of_rays_in_all_directions():
    """Hemispheres about random normals: the lanes of a dealt wave take new rays while
    others still walk."""
    sc = scenes.make_cube_cloud(12_000, 0)
    sc["log_scale"] += np.float32(1.0)
    sc["opacity"] *= np.float32(0.1)
    _check(sc, 64, 1, "dense-12000x64", sample=64)
