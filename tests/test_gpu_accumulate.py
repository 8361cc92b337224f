"""Accumulates of axes whose g is no power of two in registers (k_ASR, k_AHR), and axes with lam = 1, whose
accumulate is the identity and left out: against the FP64 oracle, forward, adjoint, partial term ranges."""

import json
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.join(os.path.dirname(__file__), ".."))

import oracle
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.fixture(scope="module")
def fx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1602_03395_amd as m
    return m


def check(fx, shape, lam, dtype, seed):
    tol = 1e-12 if dtype == torch.complex128 else 1e-5
    npdt = np.complex128 if dtype == torch.complex128 else np.complex64
    dx, t = tuple(0.9 + 0.1 * j for j in range(len(shape))), 7.0
    a, abar = oracle.default_offsets(shape, dx, lam)
    abar = abar + 0.23 * np.asarray(dx)
    f = workloads.random_field(shape, seed).astype(npdt)
    y = workloads.random_field(shape, seed + 50).astype(npdt)
    plan = fx.Plan(shape, dx, 1.0, t, lam, list(a), list(abar), dtype)
    x = torch.from_numpy(f).cuda()
    out, rho = plan.expand(x)
    _, rho_only = plan.expand(x, want_psi=False)
    g = plan.expand_adjoint(torch.from_numpy(y).cuda())
    acc = torch.from_numpy(f).cuda()  # accumulates onto a field that is not zero
    n = plan.num_terms()
    cuts = sorted({0, n // 3, (2 * n) // 3 + 1 if n > 2 else n, n})
    for b, e in zip(cuts[:-1], cuts[1:]):
        plan.expand_range(x, acc, b, e, accumulate=True)
    torch.cuda.synchronize()
    ref = oracle.expand(f.astype(np.complex128), dx, 1.0, t, lam, a, abar)
    refh = oracle.expand_adjoint(y.astype(np.complex128), dx, 1.0, t, lam, a, abar)
    assert rel(out.cpu().numpy().astype(np.complex128), ref) <= tol
    assert rel(acc.cpu().numpy().astype(np.complex128), ref + f) <= tol
    for r in (rho, rho_only):
        assert rel(r.cpu().numpy().astype(np.float64), oracle.density(ref)) <= tol
    assert rel(g.cpu().numpy().astype(np.complex128), refh) <= tol
    return json.loads(plan.describe())


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("g", [3, 5, 6, 7, 9, 10, 12, 15])
def test_register_accumulate_of_any_g(fx, g, dtype):
    # along the contiguous axis (S = 1) and a strided one; 2 g + 1 terms leave a partial block
    for shape, lam in (((5, 4 * g), (2, g)), ((4 * g, 6), (3 * g, 5))):
        print("accumulate g", g, shape, lam, dtype, flush=True)
        d = check(fx, shape, lam, dtype, 9000 + g)
        assert any(p["kernel"] == "k_AHR" and p["M"] == 4 * g for p in d["adjoint_passes"]), d


IDENTITY = [((24, 20), (1, 4)), ((24, 20), (4, 1)), ((24, 20), (1, 1)), ((40,), (1,)), ((12, 10, 16), (1, 3, 1)),
            ((12, 10, 16), (2, 1, 1)), ((12, 10, 16), (1, 1, 4)), ((12, 10, 16), (8, 8, 1)), ((1, 30), (3, 1))]


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("case", range(len(IDENTITY)))
def test_unmagnified_axes(fx, case, dtype):
    shape, lam = IDENTITY[case]
    print("lam = 1", shape, lam, dtype, flush=True)
    d = check(fx, shape, lam, dtype, 9100 + case)
    for p in d["passes"] + d["adjoint_passes"]:
        assert not (p["kind"] in ("A", "AH") and p["lam"] == 1), d


def test_unmagnified_axis_with_a_spectrum_keeps_its_accumulate(fx):
    # a tabulated spectrum may give the term q = 0 a phase, which the accumulate carries
    shape, lam, dx, t = (18, 20), (3, 1), (1.0, 0.8), 5.0
    f = workloads.random_field(shape, 9200)
    spec = [0.3 + t * 0.5 * fx.fine_wavenumbers(m, l, d) ** 2 for m, l, d in zip(shape, lam, dx)]
    out, _ = fx.expand(torch.from_numpy(f).cuda(), dx, 1.0, t, lam, spectrum=spec)
    torch.cuda.synchronize()
    ref = oracle.expand(f, dx, 1.0, t, lam) * np.exp(-0.6j)
    assert rel(out.cpu().numpy(), ref) <= 1e-12
