"""Sizes of the build's workspace (host-side queries, no GPU)."""
import os

import pytest

from paper_2311_16043_amd import _lib


@pytest.fixture(scope="module")
def build_bytes():
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2311_16043_amd import build
        build.build(verbose=False)
    return _lib.load().rv_build_workspace_bytes


def test_a_workspace_for_many_gaussians_holds_fewer(build_bytes):
    """A caller keeps one workspace, sized for its largest scene."""
    sizes = {int(1.001 ** k) for k in range(1, 20_800)}
    for edge in (1024, 2048, 4096, 8192, 1 << 17, 1 << 18, 3 << 18, 1 << 20, 1 << 22, 1 << 26, 1 << 27, 1 << 30):
        sizes |= set(range(edge - 4000, edge + 4000, 7)) | {edge - 1, edge, edge + 1}
    largest = 0
    for n in sorted(s for s in sizes if 1 <= s <= 1 << 30):
        need = build_bytes(n)
        assert need >= largest, n
        largest = need


@pytest.mark.parametrize("n", [20_000, 1 << 18, (1 << 18) + 1, 300_000, 1_200_000, 3_000_000, 1 << 26, 1 << 28, 1 << 30])
def test_workspace_per_gaussian(build_bytes, n):
    """43.4 bytes (topology 16, node boxes 24, boxes of 8, 64 and 512 leaves 3.4), with the
    inputs packed 83.4 (64 in the place of 24); the sort's arrays lie where the topology goes."""
    packed = (1 << 18) < n <= (1 << 26)
    assert build_bytes(n) <= (83.5 if packed else 43.5) * n + (1 << 14)
