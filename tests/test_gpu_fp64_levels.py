"""FP64 network evaluations whose levels past the first also form their kernels on the
matrix cores (more than 32768 cells), against the oracle at the bound of the other FP64
parity tests, 1e-12.  Random labels make nearly every window general."""
import numpy as np
import pytest
import torch

import nps_inputs as gi
from oracle import network as onet

pytestmark = pytest.mark.gpu

nps = pytest.importorskip("paper_2310_00177_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def blob(levels, seed):
    rng = np.random.default_rng(seed)
    p = gi.xavier_params(levels, seed)
    for name, _, off, size in gi.blob_layout(levels):
        if name.endswith("B"):
            p[off:off + size] = 0.1 * rng.standard_normal(size)
    return p


# level 2 of 34 x 36 x 52 cells, its tiles cut along every axis, as the coarsest level and
# with a level below; grids of two planes (waves share their rows: level 1 of two planes,
# level 2 of one) and of four (level 2 of two planes, pooled), rows and columns cut
@pytest.mark.parametrize("shape,levels", [((68, 72, 104), 2), ((68, 72, 104), 3), ((2, 518, 254), 2),
                                          ((4, 292, 460), 3)])
def test_coarse_levels_match_oracle(shape, levels):
    rng = np.random.default_rng(sum(shape) + levels)
    lab = rng.choice(3, size=shape, p=(0.5, 0.3, 0.2)).astype(np.uint8)
    r = rng.standard_normal(shape)
    params = blob(levels, 4)
    got = nps.apply_precond(nps.Net(params, levels), torch.from_numpy(lab).cuda(),
                            torch.from_numpy(r).cuda()).cpu().numpy()
    ref = onet.Network(params, levels, lab).apply(r)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < 1e-12
    assert np.abs(got - ref).max() < 1e-12 * np.abs(ref).max()


def test_iterates_on_two_planes():
    """The level-1 kernels of a solve on two planes (their dots, the masked output) against the oracle's iterates."""
    from oracle import npsdo as onpsdo
    shape = (2, 130, 132)
    lab = np.zeros(shape, dtype=np.uint8)
    lab[:, :20] = gi.AIR
    lab[:, 60:70, 30:50] = gi.SOLID
    b = gi.gen_rhs(lab, seed=3)
    params = gi.multilevel_params(2)
    ref = onpsdo.solve(lab, b, onet.Network(params, 2, lab).apply, max_iter=5, fixed_iters=True)
    x, info = nps.solve(nps.Net(params, 2), torch.from_numpy(lab).cuda(), torch.from_numpy(b).cuda(), max_iter=5,
                        fixed_iters=True, precision=nps.FP64)
    assert info.iterations == 5
    assert np.linalg.norm(x.cpu().numpy() - ref.x) <= 1e-9 * np.linalg.norm(ref.x)
