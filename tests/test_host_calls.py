"""What the library's host code does, on the CPU: the calls run against a stand-in for
the HIP runtime (fake_hip.cpp), whose kernels do not run and whose queries return what
the test says.  Each test is a child process, so that the stand-in never meets torch."""
import json
import os
import shutil
import subprocess
import sys

import pytest

PRELUDE = r"""
import ctypes, importlib.util, json, sys
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # ahead of the library: its calls bind to it
fake.fake_launched.restype = ctypes.c_char_p
fake.fake_state.argtypes = [ctypes.c_double] + [ctypes.c_int] * 3
spec = importlib.util.spec_from_file_location("_lib", sys.argv[2])
lib = importlib.util.module_from_spec(spec)
spec.loader.exec_module(lib)
SUCCESS, NOT_READY, FAILED = 0, 600, 719   # hipSuccess, hipErrorNotReady, hipErrorLaunchFailure
keep = []

def device(nbytes):
    b = np.zeros(nbytes + 256, dtype=np.uint8)
    keep.append(b)
    return (b.ctypes.data + 255) & ~255

def network(levels):
    p = np.zeros(lib.nps_param_count(levels))
    rc, net = lib.nps_net_create(p.ctypes.data, p.size, levels, device(lib.nps_net_bytes(levels)),
                                 lib.nps_net_bytes(levels), 0)
    assert rc == 0
    return net

def launched():
    out = [line.rsplit(" ", 2) for line in fake.fake_launched().decode().splitlines()]
    fake.fake_forget()
    return [(n, int(x), int(y)) for n, x, y in out]
"""


@pytest.fixture(scope="module")
def call(repo_root, tmp_path_factory):
    lib = os.path.join(repo_root, "paper_2310_00177_amd", "libnps.so")
    if not os.path.exists(lib):
        pytest.skip("libnps.so not built")
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(repo_root, "paper_2310_00177_amd", "csrc"),
                    os.path.join(repo_root, "tests", "fake_hip.cpp"), "-o", so], check=True)

    def run(body, **args):
        script = PRELUDE + "args = json.loads(sys.argv[3])\n" + body
        res = subprocess.run([sys.executable, "-c", script, so, os.path.join(repo_root, "paper_2310_00177_amd", "_lib.py"),
                              json.dumps(args)], capture_output=True, text=True, timeout=110)
        assert res.returncode == 0, res.stderr[-2000:]
        return json.loads(res.stdout.splitlines()[-1])

    return run


@pytest.mark.parametrize("phase", ["validating", "running", "finishing"])
def test_server_reports_a_failed_stream(call, phase):
    """Pending work keeps a step at NPS_OK; a failed stream ends it with NPS_EDEVICE in every phase."""
    rcs = call(r"""
phase = args["phase"]
rc, srv = lib.nps_server_create(network(2), 64 << 20, 1)
assert rc == 0
fake.fake_state(1.0, 8, 0, 0)
lab, b = np.zeros((4, 4, 4), dtype=np.uint8), np.ones((4, 4, 4))
o = lib.nps_opts(1e-6, 0 if phase == "finishing" else 100, 2, lib.NPS_FP32, 0, 0, 0)
rc, rid = lib.nps_server_submit(srv, lab.ctypes.data, lib.nps_dims(4, 4, 4), b.ctypes.data, o)
assert rc == 0
step = lambda n: [lib.nps_server_step(srv)[0] for _ in range(n)]
seen = []
fake.fake_query(0, NOT_READY if phase == "validating" else SUCCESS)
seen += step(2)          # admitted (and validated)
if phase != "validating":
    seen += step(1)      # bodies are out (finishing: the result's copy)
fake.fake_query(0, NOT_READY)
fake.fake_query(1, NOT_READY)
seen += step(4096)
fake.fake_query(0, FAILED)
fake.fake_query(1, FAILED)
failed = step(4096)      # the running phase looks at its stream once in 1024 steps
print(json.dumps([sorted(set(seen)), sorted(set(failed)), lib.nps_server_poll(srv, rid, 0, lib.nps_info())[0]]))
""", phase=phase)
    seen, failed, poll = rcs
    assert seen == [0]
    assert -8 in failed and set(failed) <= {0, -8}
    assert poll == 2


ADJOINT = r"""
def adjoint(kind, dims):
    '''Whether the call forms level 1's kernels in its adjoint (k_adj_l1m) instead of storing them.'''
    d, net = lib.nps_dims(*dims), network(2)
    ws, n = device(1 << 16), 1 << 62      # no kernel runs: nothing touches the workspace
    fake.fake_forget()
    if kind == "transpose":
        rc = lib.nps_apply_precond_transpose(net, 1 << 40, d, 2 << 40, 3 << 40, lib.NPS_FP32, ws, n, 0)
    elif kind == "train":
        rc, _ = lib.nps_train_step(net, 1 << 40, d, 1, 2 << 40, 3 << 40, lib.NPS_FP32, ws, n, 0)
    else:
        fake.fake_state(1.0, 8, 0, 0)
        o = lib.nps_opts(1e-6, 1, 2, lib.NPS_FP32, 0, 0, 1)
        rc = lib.nps_solve(net, 1 << 40, d, 2 << 40, 3 << 40, o, lib.nps_info(), ws, n, 0)
    assert rc >= 0, (kind, dims, rc, lib.nps_last_error())
    return any("k_adj_l1m" in name for name, _, _ in launched())
"""


def test_adjoint_stores_level_1_where_work_items_are_mostly_empty(call):
    """Thin grids and footprints that are half empty: the symmetric variant and P^T ran up to four times
    slower there than with stored kernels."""
    got = call(ADJOINT + r"""
print(json.dumps([[adjoint(k, d) for k in ("symmetric", "transpose", "train")] for d in args["dims"]]))
""", dims=[(512, 512, 4), (1024, 512, 8), (66, 66, 66), (512, 512, 32), (128, 128, 128), (256, 256, 256)])
    assert got == [[False, False, False], [False, False, True], [False, True, True], [False, True, True],
                   [True, True, True], [True, True, True]]


def test_launches_stay_within_the_axis_limit(call):
    """Grids a few cells wide and up to 10^8 long, which the calls accept, launch fewer than 2^32 threads along an axis."""
    got = call(r"""
most = {}
for dims in args["dims"]:
    d, net = lib.nps_dims(*dims), network(2)
    ws, n = device(1 << 16), 1 << 62
    fake.fake_state(1.0, 8, 0, 0)
    for p in (lib.NPS_FP64, lib.NPS_FP32):
        rcs = [lib.nps_apply_precond_transpose(net, 1 << 40, d, 2 << 40, 3 << 40, p, ws, n, 0),
               lib.nps_train_step(net, 1 << 40, d, 1, 2 << 40, 3 << 40, p, ws, n, 0)[0],
               lib.nps_solve(net, 1 << 40, d, 2 << 40, 3 << 40, lib.nps_opts(1e-6, 1, 2, p, 0, 0, 1), lib.nps_info(), ws, n, 0)]
        if p == lib.NPS_FP64 or min(dims) == 24:   # in float the item kernels take fewer than 2^24 work items
            rcs += [lib.nps_apply_precond(net, 1 << 40, d, 2 << 40, 3 << 40, p, ws, n, 0),
                    lib.nps_solve(net, 1 << 40, d, 2 << 40, 3 << 40, lib.nps_opts(1e-6, 1, 2, p, 0, 0, 0), lib.nps_info(), ws, n, 0)]
        assert min(rcs) >= 0, (dims, p, rcs, lib.nps_last_error())
        for name, x, y in launched():
            most[name] = max(most.get(name, 0), x, 256 * y)
print(json.dumps(most))
""", dims=[(140000000, 2, 2), (2, 140000000, 2), (2, 2, 140000000), (60000000, 4, 4), (24, 24, 1600000),
         (1600000, 24, 24)])
    assert any("k_pyramid" in name for name in got) and any("k_march_modes" in name for name in got)
    assert {name: t for name, t in got.items() if t >= 2 ** 32} == {}


@pytest.mark.parametrize("what", ["b = 0", "bad label", "no fluid", "not finite"])
@pytest.mark.parametrize("entry", ["solve", "server"])
def test_no_set_up_without_a_solve(call, what, entry):
    """A solve that ends at its validation launches the validation, and the result's copy where there is one."""
    got = call(r"""
state = {"b = 0": (0.0, 8, 0, 0), "bad label": (1.0, 8, 1, 0), "no fluid": (1.0, 0, 0, 0), "not finite": (1.0, 8, 0, 1)}[args["what"]]
fake.fake_state(*state)
net, d, o = network(2), lib.nps_dims(64, 64, 64), lib.nps_opts(1e-6, 100, 2, lib.NPS_MIXED_BF16, 0, 0, 0)
fake.fake_forget()
if args["entry"] == "solve":
    rc = lib.nps_solve(net, 1 << 40, d, 2 << 40, 3 << 40, o, lib.nps_info(), device(1 << 16), 1 << 62, 0)
else:
    rc, srv = lib.nps_server_create(net, 64 << 20, 1)
    lab, b = np.zeros((64, 64, 64), dtype=np.uint8), np.ones((64, 64, 64))
    _, rid = lib.nps_server_submit(srv, lab.ctypes.data, d, b.ctypes.data, o)
    for _ in range(8):
        assert lib.nps_server_step(srv)[0] == 0
    rc = lib.nps_server_poll(srv, rid, b.ctypes.data, lib.nps_info())[0]
print(json.dumps([rc, [name for name, _, _ in launched()]]))
""", what=what, entry=entry)
    rc, names = got
    assert rc == {"b = 0": 0, "bad label": -3, "no fluid": -4, "not finite": -5}[what]
    kept = ["k_validate", "k_live_list"] + (["k_finalize"] if what == "b = 0" else [])
    assert len(names) == len(kept) and all(k in n for k, n in zip(kept, names)), names
