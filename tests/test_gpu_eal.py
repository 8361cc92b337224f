"""The lane-per-line EA kernel (k_EAL) against the FP64 oracle: every compiled (P, g), whole and partial
term ranges (a range starts at any residue of the term index), a last tile with few lines, several
slices, and an odd magnification."""

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
      (8, 4, 20), (12, 4, 28), (16, 4, 12), (8, 2, 50), (12, 2, 10), (16, 2, 6)]
PG32 = PG + [(32, 2, 50), (32, 4, 20)]
CASES = [(torch.complex128, c) for c in PG if c != (16, 8, 40)] + [(torch.complex64, c) for c in PG32]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_eal_matches_oracle(fx, case):
    dtype, (P, g, lam0) = CASES[case]
    shape, lam = (P * g, 91, 91), (lam0, 1, 1)  # 8281 lines: the last tile has 25
    print("eal", dtype, shape, lam, flush=True)
    dx, t = (0.9, 1.0, 1.1), 13.0
    a, abar = oracle.default_offsets(shape, dx, lam)
    abar = abar + 0.41 * np.asarray(dx)
    npdt = np.complex128 if dtype == torch.complex128 else np.complex64
    f = workloads.random_field(shape, 8000 + case).astype(npdt)
    plan = fx.Plan(shape, dx, 1.0, t, lam, list(a), list(abar), dtype)
    passes = json.loads(plan.describe())["passes"]
    assert any(p["kind"] == "EA" and p["kernel"] == "k_EAL" for p in passes), passes
    x = torch.from_numpy(f).cuda()
    out, rho = plan.expand(x)
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
