"""lsh_build, whose levels' interpolation matrices are formed beside the next
level's row ID: the same factor bit for bit as lsh_plan_create +
lsh_factor_create over depths, uncompressed top levels, pivoting rules and
precisions, and for builds that run at the same time on two threads."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


CASES = [(8, 4, 4, 1e-4, 0, "fp32"), (16, 4, 4, 1e-5, 0, "fp64"), (40, 5, 6, 1e-4, 1, "fp32"),
         (112, 7, 4, 1e-6, 2, "fp64"), (160, 5, 4, 1e-4, 0, "fp32"), (64, 8, 10, 1e-9, 0, "fp64")]


@pytest.mark.parametrize("n,leaf,order,tol,fl,prec", CASES)
@pytest.mark.parametrize("rowid", ["block", "panel"])
def test_build_equals_separate_calls(n, leaf, order, tol, fl, prec, rowid, monkeypatch):
    import torch
    from paper_2007_12718_amd import lsh
    monkeypatch.setenv("LSH_ROWID", rowid)
    rng = np.random.default_rng(n)
    b = cuda(synth.bumps(n, rng))
    x = cuda(rng.standard_normal((2, n, n)) + 1j * rng.standard_normal((2, n, n)))
    o = dict(op_order=4, leaf=leaf, tol=tol, proxy_width=3, prec=prec, hbs_order=order, full_levels=fl)
    P = lsh.Plan(n, 0.5 * n, **o)
    y = lsh.Factor(P, b).apply_precond(x)
    for _ in range(2):
        P2, F2 = lsh.build(n, 0.5 * n, b, **o)
        assert P2.ranks() == P.ranks() and P2.lowrank_ranks() == P.lowrank_ranks()
        assert torch.equal(F2.apply_precond(x), y)


def test_builds_on_two_threads():
    import torch
    from paper_2007_12718_amd import lsh
    out, ref, err = {}, {}, []

    def one(i, n, leaf, prec):
        try:
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                rng = np.random.default_rng(i)
                b = cuda(synth.bumps(n, rng))
                x = cuda(rng.standard_normal((1, n, n)) + 0j)
                res = []
                for _ in range(3):
                    P, F = lsh.build(n, 0.5 * n, b, op_order=4, leaf=leaf, tol=1e-4, proxy_width=2, prec=prec)
                    res.append(F.apply_precond(x))
                    st.synchronize()
                    F.close()
                    P.close()
                out[i] = res
        except Exception as e:  # (reported by the main thread)
            err.append(e)

    todo = [(0, 96, 6, "fp32"), (1, 128, 8, "fp64")]
    for t in todo:
        one(*t)
    ref.update({i: v[0] for i, v in out.items()})
    out.clear()
    ths = [threading.Thread(target=one, args=t) for t in todo]
    for t in ths:
        t.start()
    for t in ths:
        t.join()
    assert not err, err
    for i, v in out.items():
        assert all(torch.equal(y, ref[i]) for y in v)


def test_a_level_just_below_its_bound():
    """1510 to 1536 candidates under a bound of 1544: their row ID takes more partial sums than one of 1544 rows."""
    import torch
    from paper_2007_12718_amd import lsh
    n = 384
    rng = np.random.default_rng(n)
    b = cuda(synth.bumps(n, rng))
    x = cuda(rng.standard_normal((1, n, n)) + 1j * rng.standard_normal((1, n, n)))
    o = dict(op_order=4, leaf=6, tol=1e-4, proxy_width=1, prec="fp32")
    P = lsh.Plan(n, 0.6 * n, **o)
    assert 1510 <= 2 * P.ranks()[1][2] <= 1536
    y = lsh.Factor(P, b).apply_precond(x)
    P2, F2 = lsh.build(n, 0.6 * n, b, **o)
    assert P2.ranks() == P.ranks()
    assert torch.equal(F2.apply_precond(x), y)


STARVED = r"""
import resource, sys, threading
import numpy as np
import torch
import synth
from paper_2007_12718_amd import lsh

b = torch.from_numpy(synth.bumps(64, np.random.default_rng(0))).cuda()
o = dict(op_order=4, leaf=8, tol=1e-4, proxy_width=2, prec="fp32")
P, F = lsh.build(64, 30.0, b, **o)
x = torch.ones((1, 64, 64), dtype=torch.complex128, device="cuda")
y = F.apply_precond(x)
torch.cuda.synchronize()
soft, hard = resource.getrlimit(resource.RLIMIT_NPROC)
resource.setrlimit(resource.RLIMIT_NPROC, (0, hard))
try:
    threading.Thread(target=int).start()
    print("THREADS ARE NOT LIMITED HERE", flush=True)
    sys.exit(0)
except RuntimeError:
    pass
try:
    lsh.build(64, 30.0, b, **o)
    print("BUILT", flush=True)
except lsh.LshError as e:
    print("REPORTED", e.code, flush=True)
resource.setrlimit(resource.RLIMIT_NPROC, (soft, hard))
P2, F2 = lsh.build(64, 30.0, b, **o)
assert torch.equal(F2.apply_precond(x), y)
print("BUILT AFTERWARDS", flush=True)
"""


def test_a_build_without_threads_is_an_error():
    """A process that may start no thread gets an error code from lsh_build, and builds again once it may."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", STARVED], cwd=root, capture_output=True, text=True, timeout=100)
    if "NOT LIMITED" in r.stdout:
        pytest.skip("this user's threads are not limited")
    assert r.returncode == 0 and "REPORTED -4" in r.stdout and "BUILT AFTERWARDS" in r.stdout, (r.stdout, r.stderr)
