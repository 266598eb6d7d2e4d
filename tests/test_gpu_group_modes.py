"""The kernel choice on a coarser level of the mixed modes (GPU): a wave's 16 x 4 cells of a
plane take the constant kernel in float where all their windows are pure cells of one
label, and kernels from the bf16-rounded weights otherwise.  The choice is part of the
results, so it is checked against both kernels formed on the CPU in double."""
import numpy as np
import pytest
import torch

import nps_inputs as gi
from oracle import network as onet

pytestmark = pytest.mark.gpu

nps = pytest.importorskip("paper_2310_00177_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def bf16(a):
    return torch.from_numpy(a).float().bfloat16().double().numpy()


def test_four_rows_choose_together():
    """Air rows every eight level-2 rows in half of the width: waves whose first two rows agree and whose
    last does not (pure, pure, pure, mixed), waves that start mixed, and whole pure and mixed waves."""
    shape, L = (64, 64, 160), 2
    lab2 = np.zeros(tuple(n // 2 for n in shape), dtype=np.uint8)   # (32, 32, 80): kernels formed on matrix cores
    lab2[:, 4::8, :32] = gi.AIR
    lab = lab2.repeat(2, 0).repeat(2, 1).repeat(2, 2)
    rng = np.random.default_rng(5)
    params = np.zeros(gi.param_count(L))
    W = B = None
    for name, lvl, off, size in gi.blob_layout(L):
        if (name, lvl) in (("c1B", 1), ("c2B", 1)):
            params[off + 13] = 1.0                                # level 1: the identity
        elif (name, lvl) == ("c1W", 2):
            params[off:off + size] = W = rng.uniform(-0.1, 0.1, size)
        elif (name, lvl) == ("c1B", 2):
            params[off:off + size] = B = 0.1 * rng.standard_normal(size)
        elif name == "a2B":
            params[off] = 1.0                                     # y = Interp(CConv(Pool(r)))
    r = np.where(lab == gi.FLUID, rng.standard_normal(shape), 0.0).astype(np.float32).astype(np.float64)
    y = nps.apply_precond(nps.Net(params, L), torch.from_numpy(lab).cuda(), torch.from_numpy(r).float().cuda(),
                          nps.MIXED_BF16).cpu().double().numpy()
    # the two kernels of level 2: exact, and from the count form (air and fluid relative to solid) in bf16
    W = W.reshape(27, 3, 27)
    C, D = bf16(B + W[:, 2].sum(1)), bf16((W[:, :2] - W[:, 2:]) / 8.0) * 8.0
    Wr = np.concatenate([D, np.zeros_like(W[:, 2:])], axis=1)
    img, r2 = onet.image(lab2), onet.pool(r)
    K = onet.cconv_kernels(img, W.reshape(27, 3, 3, 3, 3), B)
    exact = onet.cconv_apply(K, r2)
    rounded = onet.cconv_apply(onet.cconv_kernels(img, Wr.reshape(27, 3, 3, 3, 3), C), r2)
    bound = onet.cconv_apply(np.abs(K), np.abs(r2))
    pad = np.pad(lab2, 1, constant_values=gi.SOLID)
    windows = np.stack([pad[a:a + 32, b:b + 32, c:c + 80] for a in range(3) for b in range(3) for c in range(3)])
    pure = (windows == windows[0]).all(0)
    wave = pure.reshape(32, 8, 4, 5, 16).all(axis=(2, 4))         # 16 x 4 cells of a plane
    assert wave.any() and not wave.all() and (pure.reshape(32, 8, 4, 5, 16).any(axis=(2, 4)) & ~wave).any()
    wave = wave.repeat(4, axis=1).repeat(16, axis=2)
    x2 = np.where(wave, exact, rounded)
    # fp32 sums of 27 products, an interpolation and a combination
    tol = 64 * 2.0 ** -24 * onet.interpolate(bound)
    fluid = lab == gi.FLUID
    assert (np.abs(y - onet.interpolate(x2)) <= tol)[fluid].all()
    # ... which tells the two kernels apart
    assert np.median((np.abs(exact - rounded) / (64 * 2.0 ** -24 * bound))[~wave & pure]) > 8
