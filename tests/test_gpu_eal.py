"""The lane-per-line kernels against the FP64 oracle: EA (k_EAL) and its adjoint (k_EAHL) for every compiled
(P, g), whole and partial term ranges (a range starts at any residue of the term index), a last tile with
few lines, several slices; E (k_EL) for every compiled P with powers of two and other g."""

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


# (P, g, lam) with gcd(lam, P g) = g
PG = [(2, 8, 24), (3, 8, 40), (4, 8, 40), (6, 8, 40), (8, 8, 40), (12, 8, 8), (16, 8, 40), (4, 4, 12), (6, 4, 20),
      (8, 4, 20), (12, 4, 28), (16, 4, 12), (8, 2, 50), (12, 2, 10), (16, 2, 6), (32, 2, 50), (32, 4, 20)]
PG32 = PG + [(64, 4, 20)]
CASES = [(torch.complex128, c) for c in PG] + [(torch.complex64, c) for c in PG32]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_eal_matches_oracle(fx, case):
    dtype, (P, g, lam0) = CASES[case]
    shape, lam = (P * g, 131, 127), (lam0, 1, 1)  # 16637 lines: the last tile has 61
    print("eal", dtype, shape, lam, flush=True)
    dx, t = (0.9, 1.0, 1.1), 13.0
    a, abar = oracle.default_offsets(shape, dx, lam)
    abar = abar + 0.41 * np.asarray(dx)
    npdt = np.complex128 if dtype == torch.complex128 else np.complex64
    f = workloads.random_field(shape, 8000 + case).astype(npdt)
    plan = fx.Plan(shape, dx, 1.0, t, lam, list(a), list(abar), dtype)
    passes = json.loads(plan.describe())["passes"]
    assert any(p["kind"] == "EA" and p["kernel"] == "k_EAL" for p in passes), passes
    adj = json.loads(plan.describe())["adjoint_passes"]
    assert any(p["kind"] == "EAH" and p["kernel"] == "k_EAHL" for p in adj), adj
    x = torch.from_numpy(f).cuda()
    out, rho = plan.expand(x)
    y = workloads.random_field(shape, 8050 + case).astype(npdt)
    gy = plan.expand_adjoint(torch.from_numpy(y).cuda())
    acc = torch.zeros_like(x)
    cuts = [0, 1, lam0 // 2 + 1, lam0]
    for b, e in zip(cuts[:-1], cuts[1:]):
        plan.expand_range(x, acc, b, e, accumulate=True)
    torch.cuda.synchronize()
    ref = oracle.expand(f.astype(np.complex128), dx, 1.0, t, lam, a, abar)
    tol = 1e-12 if dtype == torch.complex128 else 1e-5
    assert rel(out.cpu().numpy().astype(np.complex128), ref) <= tol
    assert rel(acc.cpu().numpy().astype(np.complex128), ref) <= tol
    assert rel(rho.cpu().numpy().astype(np.float64), oracle.density(ref)) <= tol
    refh = oracle.expand_adjoint(y.astype(np.complex128), dx, 1.0, t, lam, a, abar)
    assert rel(gy.cpu().numpy().astype(np.complex128), refh) <= tol


EL_CASES = [(2, 8, 24), (3, 5, 10), (4, 3, 9), (5, 9, 18), (6, 8, 40), (7, 4, 12), (8, 9, 9), (9, 2, 4), (10, 6, 12),
            (12, 8, 8), (15, 2, 14), (16, 4, 12), (32, 2, 10)]


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("case", range(len(EL_CASES)))
def test_el_matches_oracle(fx, case, dtype):
    P, g, lam1 = EL_CASES[case]
    shape, lam = (5, P * g, 821), (3, lam1, 1)  # strided E along the middle axis: 4105 lines
    print("el", dtype, shape, lam, flush=True)
    dx, t = (0.9, 1.0, 1.1), 13.0
    a, abar = oracle.default_offsets(shape, dx, lam)
    abar = abar + 0.29 * np.asarray(dx)
    npdt = np.complex128 if dtype == torch.complex128 else np.complex64
    f = workloads.random_field(shape, 8200 + case).astype(npdt)
    plan = fx.Plan(shape, dx, 1.0, t, lam, list(a), list(abar), dtype)
    passes = json.loads(plan.describe())["passes"]
    if not (dtype == torch.complex128 and P == 32):
        assert any(p["kind"] == "E" and p["axis"] == 1 and p["kernel"] == "k_EL" for p in passes), passes
    x = torch.from_numpy(f).cuda()
    out, rho = plan.expand(x)
    acc = torch.zeros_like(x)
    cuts = [0, 4, 3 * lam1 // 2, 3 * lam1]
    for b, e in zip(cuts[:-1], cuts[1:]):
        plan.expand_range(x, acc, b, e, accumulate=True)
    torch.cuda.synchronize()
    ref = oracle.expand(f.astype(np.complex128), dx, 1.0, t, lam, a, abar)
    tol = 1e-12 if dtype == torch.complex128 else 1e-5
    assert rel(out.cpu().numpy().astype(np.complex128), ref) <= tol
    assert rel(acc.cpu().numpy().astype(np.complex128), ref) <= tol
    assert rel(rho.cpu().numpy().astype(np.float64), oracle.density(ref)) <= tol


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_eal_several_slices(fx, dtype):
    # the slices of the other axes' terms share tiles: S = 96 is not a multiple of 64
    shape, lam, dx, t = (32, 24, 40), (40, 8, 10), (1.0, 1.0, 1.0), 20.0
    print("eal slices", dtype, shape, lam, flush=True)
    npdt = np.complex128 if dtype == torch.complex128 else np.complex64
    f = workloads.random_field(shape, 8100).astype(npdt)
    plan = fx.Plan(shape, dx, 1.0, t, lam, dtype=dtype)
    out, rho = plan.expand(torch.from_numpy(f).cuda())
    many, _ = plan.expand_many(torch.from_numpy(np.stack([f] * 9)).cuda())
    torch.cuda.synchronize()
    desc = json.loads(plan.describe())
    assert desc["slices"] > 1 and any(p["kernel"] == "k_EAL" for p in desc["passes"]), desc
    ref = oracle.expand(f.astype(np.complex128), dx, 1.0, t, lam)
    tol = 1e-12 if dtype == torch.complex128 else 1e-5
    assert rel(rho.cpu().numpy().astype(np.float64), oracle.density(ref)) <= tol
    for i in (0, 8):
        assert rel(many[i].cpu().numpy().astype(np.complex128), ref) <= tol
