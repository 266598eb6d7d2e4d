"""Parameter gradient and adjoint on grids where their kernels' tiles end (GPU):
16 x 4 x 4 tiles cut along every axis, levels of a few cells, counts beyond 256
(two bf16 pieces, levels 4 and up), a grid without fluid in most tiles, and
batches whose systems add to the same sums.  Bars: those of the training parity
tests (FP64 1e-9, FP32 1e-6, bf16 leg 6e-3; adjoint 1e-12 and 1e-5)."""
import numpy as np
import pytest
import torch

import nps_inputs as gi
from oracle import gradient as og
from oracle import network as onet

pytestmark = pytest.mark.gpu

nps = pytest.importorskip("paper_2310_00177_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

BARS = {"FP64": 1e-9, "FP32": 1e-6, "MIXED_BF16": 6e-3}
# one tile; cut tiles; 6 levels down to one cell; a long thin grid with 5 levels
GRIDS = [((4, 4, 16), 2), ((6, 10, 18), 2), ((32, 32, 32), 6), ((16, 48, 80), 5)]


def rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def scene(shape, seed, fluid=0.6):
    rng = np.random.default_rng(seed)
    lab = rng.choice(3, size=shape, p=(fluid, 0.9 - fluid, 0.1)).astype(np.uint8)
    lab[shape[0] // 2:, :, shape[2] // 2:] = gi.AIR   # tiles without fluid
    b = rng.standard_normal(shape) * (lab == gi.FLUID)
    return lab, b / np.linalg.norm(b)


def blob(levels, seed):
    p = gi.xavier_params(levels, seed)
    rng = np.random.default_rng(seed + 1)
    for name, _, off, size in gi.blob_layout(levels):
        if name.endswith("B"):
            p[off:off + size] = rng.uniform(-0.5, 0.5, size)
    return p


@pytest.mark.parametrize("shape,levels", GRIDS)
@pytest.mark.parametrize("precision", list(BARS))
def test_batch_gradient_matches_oracle(shape, levels, precision):
    params, p = blob(levels, 5), getattr(nps, precision)
    systems = [scene(shape, s) for s in (1, 2)]
    labels = torch.from_numpy(np.stack([s[0] for s in systems])).cuda()
    b = torch.from_numpy(np.stack([s[1] for s in systems])).to(nps.vector_dtype(p)).cuda()
    ref_loss, ref = og.batch_loss_and_grad(params, levels, [s[0] for s in systems], [s[1] for s in systems])
    net, ws = nps.Net(params, levels), nps.train_workspace(shape, levels, p)
    ws.fill_(255)   # what the workspace held does not matter
    grad = torch.zeros(gi.param_count(levels), dtype=torch.float64, device="cuda")
    loss = nps.train_step(net, labels, b, grad, ws, precision=p)
    assert loss == pytest.approx(ref_loss, rel=10 * BARS[precision])
    assert rel(grad.cpu().numpy(), ref) <= BARS[precision]
    # the gradient is added to what the buffer holds, and a repeated step gives the same bits
    once = grad.clone()
    again = torch.zeros_like(grad)
    nps.train_step(net, labels, b, again, ws, precision=p)
    assert torch.equal(again, once)
    nps.train_step(net, labels, b, grad, ws, precision=p)
    assert torch.allclose(grad, 2 * once, rtol=1e-12, atol=0)


@pytest.mark.parametrize("shape,levels", GRIDS)
@pytest.mark.parametrize("precision,bar", [("FP64", 1e-12), ("FP32", 1e-5)])
def test_adjoint_matches_oracle(shape, levels, precision, bar):
    params = blob(levels, 9)
    lab, _ = scene(shape, 3)
    g = np.random.default_rng(4).standard_normal(shape)
    ref = og.transpose_apply(onet.Network(params, levels, lab), g)
    dt = torch.float64 if precision == "FP64" else torch.float32
    got = nps.apply_precond_transpose(nps.Net(params, levels), torch.from_numpy(lab).cuda(),
                                      torch.from_numpy(g).to(dt).cuda()).cpu().double().numpy()
    assert rel(got, ref) <= bar


# Level 1 without stored kernels (float, more than 32768 cells): 2-plane items with
# rows not of four cells, 4-plane items (from 1024 on) with a last chunk of 2 planes
# and a last footprint of 4 columns, whole footprints.
LARGE = [(34, 38, 70), (70, 62, 260), (64, 64, 256)]


@pytest.mark.parametrize("shape", LARGE)
def test_float_gradient_and_adjoint_match_fp64_on_large_grids(shape):
    """Against the FP64 path (matched to the oracle elsewhere), with the oracle tests' bars; boxes
    of fluid give groups of every kind."""
    rng = np.random.default_rng(sum(shape))
    lab = np.zeros(shape, dtype=np.uint8)
    lab[3 * shape[0] // 4:] = gi.AIR
    for i in range(10):
        lo = [int(rng.integers(0, n)) for n in shape]
        lab[tuple(slice(a, a + int(rng.integers(1, max(2, n // 4)))) for a, n in zip(lo, shape))] = 1 + i % 2
    labels = torch.from_numpy(lab).cuda()
    gen = torch.Generator(device="cuda").manual_seed(1)
    b = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64) * (labels == gi.FLUID)
    net, n = nps.Net(blob(2, 3), 2), gi.param_count(2)
    grads = {}
    for p in BARS:
        prec = getattr(nps, p)
        grad = torch.zeros(n, dtype=torch.float64, device="cuda")
        bt = b.to(nps.vector_dtype(prec))
        nps.train_step(net, labels[None], bt[None], grad, nps.train_workspace(shape, 2, prec), precision=prec)
        grads[p] = grad.cpu().numpy()
    for p in ("FP32", "MIXED_BF16"):
        assert rel(grads[p], grads["FP64"]) <= BARS[p], p
    ref = nps.apply_precond_transpose(net, labels, b)
    got = nps.apply_precond_transpose(net, labels, b.float())
    assert float(torch.linalg.norm(got - ref) / torch.linalg.norm(ref)) <= 1e-5
    # rows that cannot be read four cells at once give the same bits
    buf = torch.empty(b.numel() + 1, dtype=torch.float32, device="cuda")
    off = buf[1:].view(shape)
    off.copy_(b)
    assert torch.equal(nps.apply_precond_transpose(net, labels, off), got)


@pytest.mark.parametrize("precision", ["FP32", "MIXED_BF16"])
def test_symmetric_iterates_on_a_large_level_1(precision):
    """The float symmetric variant (three-piece kernels in both sweeps) follows the FP64 iterates at
    the bar of the other float iterate tests, 1e-4."""
    shape = (40, 32, 48)
    lab, b = scene(shape, 11)
    net = nps.Net(gi.multilevel_params(4), 4)
    labels, bt = torch.from_numpy(lab).cuda(), torch.from_numpy(b).cuda()
    kw = dict(max_iter=4, fixed_iters=True, symmetric=True)
    ref, _ = nps.solve(net, labels, bt, precision=nps.FP64, **kw)
    got, _ = nps.solve(net, labels, bt, precision=getattr(nps, precision), **kw)
    assert float(torch.linalg.norm(got - ref) / torch.linalg.norm(ref)) < 1e-4


@pytest.mark.parametrize("precision", list(BARS))
def test_gradient_on_a_thin_grid_matches_oracle(precision):
    """A large level 1 whose work items are a sixteenth full keeps its kernels in float too."""
    shape, levels = (132, 128, 4), 3
    params, p = blob(levels, 6), getattr(nps, precision)
    lab, b = scene(shape, 5)
    ref_loss, ref = og.batch_loss_and_grad(params, levels, [lab], [b])
    ws = nps.train_workspace(shape, levels, p)
    ws.fill_(255)
    grad = torch.zeros(gi.param_count(levels), dtype=torch.float64, device="cuda")
    loss = nps.train_step(nps.Net(params, levels), torch.from_numpy(lab[None]).cuda(),
                          torch.from_numpy(b[None]).to(nps.vector_dtype(p)).cuda(), grad, ws, precision=p)
    assert loss == pytest.approx(ref_loss, rel=10 * BARS[precision])
    assert rel(grad.cpu().numpy(), ref) <= BARS[precision]
