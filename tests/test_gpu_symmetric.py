"""GPU parity of the symmetric variant (appendix on symmetry): the adjoint
P^T, the asymmetry measure S, and solves preconditioned with P^T o P, against
the FP64 oracle through the C ABI.
"""
import numpy as np
import pytest
import torch

import nps_inputs as gi
from oracle import gradient as og
from oracle import laplacian as lap
from oracle import network as onet
from oracle import npsdo as onpsdo
from oracle import pcg as opcg

pytestmark = pytest.mark.gpu

nps = pytest.importorskip("paper_2310_00177_amd")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t if dtype is None else t.to(dtype)).cuda()


def rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def params_with_biases(L, seed):
    p = gi.xavier_params(L, seed)
    rng = np.random.default_rng(seed + 1)
    for name, _l, off, size in gi.blob_layout(L):
        if name.endswith("B"):
            p[off:off + size] = rng.uniform(-0.5, 0.5, size)
    return p


CASES = {
    "grad16": (gi.scene_gradcheck(), 5),
    "multi64": (gi.SceneSpec((64, 64, 96), 8, (3.0, 10.0), 2, ("flat", 32, 56)), 6),
}


@pytest.mark.parametrize("name", ["grad16", "multi64"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_transpose_matches_oracle(name, dtype):
    spec, L = CASES[name]
    lab = gi.gen_labels(spec, seed=3)
    params = params_with_biases(L, 7)
    g = np.random.default_rng(5).standard_normal(lab.shape)
    print(f"transpose {name} {dtype}", flush=True)
    y = nps.apply_precond_transpose(nps.Net(params, L), dev(lab), dev(g, dtype)).cpu().double().numpy()
    ref = og.transpose_apply(onet.Network(params, L, lab), g)
    assert rel(y, ref) <= (1e-12 if dtype == torch.float64 else 1e-5), rel(y, ref)
    assert np.all(y[lab != gi.FLUID] == 0)


def test_transpose_is_the_adjoint_of_the_gpu_network():
    spec, L = CASES["grad16"]
    lab = gi.gen_labels(spec, seed=4)
    net = nps.Net(params_with_biases(L, 9), L)
    rng = np.random.default_rng(6)
    x, y = rng.standard_normal(lab.shape), rng.standard_normal(lab.shape)
    labels = dev(lab)
    px = nps.apply_precond(net, labels, dev(x)).cpu().numpy()
    pty = nps.apply_precond_transpose(net, labels, dev(y)).cpu().numpy()
    assert float(np.sum(y * px)) == pytest.approx(float(np.sum(pty * x)), rel=1e-12)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_asymmetry_matches_oracle(precision):
    spec, L = CASES["grad16"]
    lab = gi.gen_labels(spec, seed=5)
    params = params_with_biases(L, 11)
    rng = np.random.default_rng(7)
    x, y = rng.standard_normal(lab.shape), rng.standard_normal(lab.shape)
    p = nps.FP64 if precision == "fp64" else nps.FP32
    dt = torch.float64 if precision == "fp64" else torch.float32
    s = nps.asymmetry(nps.Net(params, L), dev(lab), dev(x, dt), dev(y, dt), precision=p)
    ref = onet.asymmetry(onet.Network(params, L, lab), x, y)
    assert ref > 1e-3
    assert s == pytest.approx(ref, rel=1e-9 if precision == "fp64" else 1e-3)


def c1(seed):
    lab = gi.gen_labels(gi.scene_c1(), seed=seed)
    return lab, gi.gen_rhs(lab, seed=seed + 1)


@pytest.mark.parametrize("method", ["npsdo", "pcg"])
def test_symmetric_fixed_iterations_fp64_match_oracle(method):
    lab, b = c1(2)
    params = gi.multilevel_params(6)
    P = onet.Network(params, 6, lab)
    Ps = lambda v: og.transpose_apply(P, P.apply(v))  # noqa: E731
    net = nps.Net(params, 6)
    m = nps.NPSDO if method == "npsdo" else nps.PCG
    for k in (1, 2, 5):
        print(f"symmetric {method} fixed-iter k={k}", flush=True)
        if method == "npsdo":
            ref = onpsdo.solve(lab, b, Ps, max_iter=k, fixed_iters=True)
        else:
            ref = opcg.solve(lab, b, Ps, max_iter=k, fixed_iters=True)
        x, info = nps.solve(net, dev(lab), dev(b), max_iter=k, fixed_iters=True, precision=nps.FP64, method=m,
                            symmetric=True)
        assert info.iterations == k and info.status == 0
        assert rel(x.cpu().numpy(), ref.x) <= 1e-9, (k, rel(x.cpu().numpy(), ref.x))


@pytest.mark.parametrize("precision", ["fp32", "mixed_bf16"])
def test_symmetric_solve_reaches_tolerance(precision):
    lab, b = c1(1)
    p = {"fp32": nps.FP32, "mixed_bf16": nps.MIXED_BF16}[precision]
    print(f"symmetric solve {precision}", flush=True)
    x, info = nps.solve(nps.Net(gi.multilevel_params(6), 6), dev(lab), dev(b), tol=1e-6, max_iter=800, precision=p,
                        symmetric=True)
    assert info.status == 0, info
    assert lap.rel_residual(lab, b, x.cpu().numpy()) < 1e-6
    # The FP64 oracle takes 227 iterations (P alone: 31).  P^T o P squares the
    # conditioning, so float rounding in its two network passes costs
    # iterations (measured: 363 in FP32); the FP64 path matches the oracle
    # iterate by iterate above.
    assert 150 <= info.iterations <= 2 * 227, info.iterations


@pytest.mark.parametrize("shape,L", [((16, 16, 16), 5), ((32, 40, 48), 3)])   # stored kernels at level 1; not in float
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shift", [0, 5, -5])
def test_transpose_output_may_overlap_its_input(shape, L, dtype, shift):
    """y on top of g, and starting 5 elements past or before it: the bits of separate buffers."""
    rng = np.random.default_rng(8)
    labels = dev(rng.choice(3, size=shape, p=(0.6, 0.2, 0.2)).astype(np.uint8))
    net, n = nps.Net(params_with_biases(L, 12), L), int(np.prod(shape))
    g = dev(rng.standard_normal(shape), dtype)
    prec = nps.FP64 if dtype == torch.float64 else nps.FP32
    ws = nps.train_workspace(shape, L, prec)
    ref = nps.apply_precond_transpose(net, labels, g, ws=ws)
    for _ in range(3):
        buf = torch.zeros(n + 16, dtype=dtype, device="cuda")
        src, out = buf[8:8 + n], buf[8 + shift:8 + shift + n]
        src.copy_(g.view(-1))
        wp, wb = nps._ws_args(ws)
        rc = nps._lib.nps_apply_precond_transpose(net.handle, labels.data_ptr(), nps._dims(shape), src.data_ptr(),
                                                  out.data_ptr(), prec, wp, wb, nps._stream())
        torch.cuda.synchronize()
        assert rc == 0 and torch.equal(out.view(shape), ref)


# thin grids whose level 1 keeps its kernels in float (work items an eighth and a sixteenth
# full), and a half-full one (P^T forms them, the symmetric variant keeps them)
THIN = [((128, 66, 8), 2), ((132, 128, 4), 3), ((34, 70, 66), 2)]


@pytest.mark.parametrize("shape,L", THIN)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_transpose_on_thin_grids(shape, L, dtype):
    rng = np.random.default_rng(sum(shape))
    lab = rng.choice(3, size=shape, p=(0.6, 0.2, 0.2)).astype(np.uint8)
    g, params = rng.standard_normal(shape), params_with_biases(L, 13)
    y = nps.apply_precond_transpose(nps.Net(params, L), dev(lab), dev(g, dtype)).cpu().double().numpy()
    ref = og.transpose_apply(onet.Network(params, L, lab), g)
    assert rel(y, ref) <= (1e-12 if dtype == torch.float64 else 1e-5), rel(y, ref)
    assert np.all(y[lab != gi.FLUID] == 0)


@pytest.mark.parametrize("shape,L", THIN)
def test_symmetric_iterates_on_thin_grids(shape, L):
    """Float iterates of the symmetric variant against FP64's (1e-4, the bar of the other ragged-grid iterates)."""
    lab = np.zeros(shape, dtype=np.uint8)
    lab[3 * shape[0] // 4:] = gi.AIR
    lab[5:9, 3:7] = gi.SOLID
    b = gi.gen_rhs(lab, seed=4)
    net = nps.Net(gi.multilevel_params(L), L)
    kw = dict(max_iter=4, fixed_iters=True, symmetric=True)
    ref, _ = nps.solve(net, dev(lab), dev(b), precision=nps.FP64, **kw)
    for p in (nps.FP32, nps.MIXED_BF16):
        x, info = nps.solve(net, dev(lab), dev(b), precision=p, **kw)
        assert info.iterations == 4
        assert rel(x.cpu().numpy(), ref.cpu().numpy()) < 1e-4
