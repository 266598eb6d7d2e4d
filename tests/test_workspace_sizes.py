"""Workspace sizes (host only): a buffer that a program once sized stays large enough."""
import os

import pytest

# (nz, ny, nx), levels, precision, n_ortho and the bytes that solves were given before their
# set-up tables and the coarse levels' mode tables changed
GIVEN = [((32, 32, 32), 6, "NPS_FP64", 2, 20470784), ((32, 32, 32), 6, "NPS_MIXED_BF16", 2, 11034112),
         ((128, 128, 128), 6, "NPS_FP64", 2, 224603648), ((128, 128, 128), 6, "NPS_MIXED_BF16", 2, 130507008),
         ((256, 256, 256), 6, "NPS_FP64", 2, 1676234240), ((2, 2, 2), 2, "NPS_FP32", 0, 1055488),
         ((2, 108, 172), 2, "NPS_MIXED_FP16", 2, 3698688), ((375936, 332, 4), 3, "NPS_MIXED_FP16", 1, 25913050112),
         ((4, 4, 65536), 3, "NPS_FP32", 0, 38325760), ((64, 96, 160), 5, "NPS_MIXED_FP16", 4, 77458432)]


@pytest.mark.parametrize("shape,levels,precision,n_ortho,given", GIVEN)
def test_solve_workspace_does_not_grow(repo_root, shape, levels, precision, n_ortho, given):
    if not os.path.exists(os.path.join(repo_root, "paper_2310_00177_amd", "libnps.so")):
        pytest.skip("libnps.so not built")
    from paper_2310_00177_amd import _lib
    need = _lib.nps_workspace_bytes(_lib.nps_dims(*shape), levels, getattr(_lib, precision), n_ortho)
    assert 0 < need <= given
