"""LBVH build at the sizes where its route changes, bit for bit against the
oracle's keys, order and tree (and the box checks of the build tests): the
one-block sort and its item counts, the packed inputs, the sort's tile sizes,
and trees whose ranges are long, far from their node, or all of one key."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_16043_amd import Gaussians, _lib, build_bvh, refit_bvh
from workloads import scenes

from test_gpu_build import _build, check_build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2047, 4096, 4097, 8192, 8193, 131_072, 131_073, 262_145, 786_433])
def test_build_sizes_where_the_sort_changes(n):
    check_build(scenes.make_cube_cloud(n, 0), f"cube-{n}")


@pytest.mark.parametrize("n", [(1 << 21) + 1, (1 << 22) + 1])
def test_sort_of_larger_tiles(n):
    """Keys and order only (4 and 8 items per thread)."""
    rng = np.random.default_rng(n)
    sc = scenes.make_cube_cloud(1000, 0)
    sc = {k: np.resize(v, (n,) + v.shape[1:]) for k, v in sc.items()}
    sc["mean"] = rng.uniform(-1.0, 1.0, (n, 3)).astype(np.float32)
    sc["mean"][::7] = sc["mean"][3]   # one key many times over: the order among them is the index
    _, _, A = _build(sc)
    _, _, keys = oracle.morton63(sc["mean"])
    order = oracle.sort_keys(keys)
    assert np.array_equal(A["perm"].astype(np.int64), order)
    assert np.array_equal(A["keys"], keys[order])


@pytest.mark.parametrize("n", [3000, 9000])
def test_build_all_equal_and_comb(n):
    sc = scenes.make_cube_cloud(n, 0)
    sc["mean"][:] = sc["mean"][17]
    check_build(sc, f"all-equal-{n}")
    # clusters at halving distances from a corner: every level of the tree splits
    # off one cluster, and most nodes reach to the far end
    sc = scenes.make_cube_cloud(n, 0)
    level = np.arange(n) % 20
    sc["mean"] = (sc["mean"] * np.float32(2.0) ** (-2 - level)[:, None] * np.float32(0.25)
                  + np.float32(2.0) ** (-level)[:, None]).astype(np.float32)
    check_build(sc, f"comb-{n}")


def _sections(A):
    return {k: v for k, v in A.items() if k != "header"}


@pytest.mark.parametrize("n", [100, 131_073, 262_145, 300_001])
def test_no_normals_is_the_normal_0_0_1(n):
    """Without normals (read directly, or above 2^18 Gaussians through the packed
    records) every section holds what it holds with all normals (0, 0, 1), after a
    build and after a refit to moved Gaussians, in a workspace sized for more."""
    rng = np.random.default_rng(n)
    sc = scenes.make_cube_cloud(n, 0)
    ws = torch.empty(int(_lib.load().rv_build_workspace_bytes(n + 5000)), dtype=torch.uint8, device="cuda")
    moved = (sc["mean"] + rng.normal(0.0, 0.05, sc["mean"].shape)).astype(np.float32)
    up = np.tile(np.array([0.0, 0.0, 1.0], np.float32), (n, 1))
    got = []
    for normal in (None, up):
        def gaussians(mean):
            return Gaussians(torch.from_numpy(mean), *(torch.from_numpy(sc[k]) for k in ("quat", "log_scale", "opacity")),
                             None if normal is None else torch.from_numpy(normal))
        bvh = build_bvh(gaussians(sc["mean"]), ws)
        built = bvh.arrays()
        got.append((built, refit_bvh(bvh, gaussians(moved), ws).arrays()))
    for a, b in zip(*got):
        assert np.array_equal(a["header"][:13].view(np.uint32), b["header"][:13].view(np.uint32))
        for k, v in _sections(a).items():
            assert np.array_equal(v.view(np.uint32), b[k].view(np.uint32)), k
    assert not np.array_equal(got[0][0]["leaf_boxes"], got[0][1]["leaf_boxes"])
