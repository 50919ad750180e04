"""Workspace sizes grow with the work: a workspace made for a program's largest
call holds every smaller one."""
import os

import pytest

from paper_2603_00839_amd import rtg


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(rtg.LIB_PATH):
        from paper_2603_00839_amd import build_lib
        build_lib.build()
    return rtg.load_library()


@pytest.mark.parametrize("I1,I2", [(8, 3), (48, 48), (64, 64), (128, 128), (200, 37), (512, 512)])
def test_network_workspace_grows_with_the_batch(lib, I1, I2):
    sizes = [lib.rtg_cnn_workspace_bytes(n, I1, I2) for n in range(1, 100)]
    assert sizes[0] > 0 and sizes == sorted(sizes)


@pytest.mark.parametrize("N", [1, 3, 8, 32, 43])
def test_network_workspace_grows_with_the_image(lib, N):
    for other in (5, 48, 128, 131):
        sizes = [lib.rtg_cnn_workspace_bytes(N, n, other) for n in range(1, 300)]
        assert sizes[0] > 0 and sizes == sorted(sizes)
        sizes = [lib.rtg_cnn_workspace_bytes(N, other, n) for n in range(1, 300)]
        assert sizes[0] > 0 and sizes == sorted(sizes)
