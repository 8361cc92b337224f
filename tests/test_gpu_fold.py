"""The folded line kernels (k_EF, k_EAF, k_EHF) against the FP64 oracle: every radix class, one and
several transform stages, contiguous and strided lines, partial tiles, stacks, partial term ranges
and a blocked outer index."""

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


CASES = [
    # shape, lam
    ((125,), (4,)),              # one line, P = 125 = 25 5
    ((11, 13), (5, 3)),          # prime pruned lengths, one stage
    ((143, 5), (2, 7)),          # P = 143 = 13 11 strided, P = 5
    ((98, 30), (6, 9)),          # P = 49 strided, P = 10 with g = 3
    ((3, 360), (2, 7)),          # P = 360 = 20 18
    ((2, 500, 3), (3, 15, 2)),   # g = 5, P = 100, S = 3 (a tile wider than the lines)
    ((7, 1080), (1, 1)),         # three stages, one term
    ((5, 1024), (2, 5)),         # radix 16
    ((72, 33), (9, 4)),          # one stage with g = 9, strided; 33 = 11 3
    ((26, 28), (4, 3)),          # radices 13 and 14
    ((225, 4), (30, 3)),         # g = 15, P = 15
    ((17, 35), (3, 10)),         # 17: no plan (the runtime transforms), beside a folded axis
    ((4, 60, 25), (3, 7, 6)),    # fused EA over the first axis, g = 1 strided
    ((45, 20, 50), (6, 3, 4)),   # fused EA with g = 3
    ((12, 2400), (5, 2)),        # long FP64 rows
]


def _names(plan):
    d = json.loads(plan.describe())
    return {p["kernel"] for p in d["passes"]}, {p["kernel"] for p in d["adjoint_passes"]}


@pytest.mark.parametrize("case", range(len(CASES)))
def test_fold_matches_oracle(fx, case):
    shape, lam = CASES[case]
    print("fold", shape, lam, flush=True)
    dx, t = tuple(0.8 + 0.1 * j for j in range(len(shape))), 11.0
    a, abar = oracle.default_offsets(shape, dx, lam)
    abar = abar + 0.37 * np.asarray(dx)
    f = workloads.random_field(shape, 7000 + case)
    y = workloads.random_field(shape, 7100 + case)
    ref = oracle.expand(f, dx, 1.0, t, lam, a, abar)
    refh = oracle.expand_adjoint(y, dx, 1.0, t, lam, a, abar)
    plan = fx.Plan(shape, dx, 1.0, t, lam, list(a), list(abar), torch.complex128)
    assert set.union(*_names(plan)) & {"k_EF", "k_EAF", "k_EHF"}, plan.describe()
    out, rho = plan.expand(torch.from_numpy(f).cuda())
    g = plan.expand_adjoint(torch.from_numpy(y).cuda())
    torch.cuda.synchronize()
    assert rel(out.cpu().numpy(), ref) <= 1e-12
    assert rel(rho.cpu().numpy(), oracle.density(ref)) <= 1e-12
    assert rel(g.cpu().numpy(), refh) <= 1e-12
    f32, y32 = f.astype(np.complex64), y.astype(np.complex64)
    plan = fx.Plan(shape, dx, 1.0, t, lam, list(a), list(abar), torch.complex64)
    _, rho = plan.expand(torch.from_numpy(f32).cuda())
    g = plan.expand_adjoint(torch.from_numpy(y32).cuda())
    torch.cuda.synchronize()
    ref = oracle.expand(f32.astype(np.complex128), dx, 1.0, t, lam, a, abar)
    refh = oracle.expand_adjoint(y32.astype(np.complex128), dx, 1.0, t, lam, a, abar)
    assert rel(rho.cpu().numpy().astype(np.float64), oracle.density(ref)) <= 1e-5
    assert rel(g.cpu().numpy().astype(np.complex128), refh) <= 1e-5


@pytest.mark.parametrize("shape,lam,count", [((60,), (7,), 33), ((40, 36), (6, 5), 5), ((20, 90), (3, 4), 3)])
def test_fold_stacks_equal_single_fields(fx, shape, lam, count):
    # contiguous lines of all slices share tiles: the rows of a stack cross field boundaries
    print("fold stack", shape, lam, count, flush=True)
    dx = (1.0,) * len(shape)
    f = np.stack([workloads.random_field(shape, 7200 + i) for i in range(count)])
    plan = fx.Plan(shape, dx, 1.0, 9.0, lam)
    out, rho = plan.expand_many(torch.from_numpy(f).cuda())
    g = plan.density_adjoint_many(out, rho)
    torch.cuda.synchronize()
    for i in (0, 1, count - 1):
        ref = oracle.expand(f[i], dx, 1.0, 9.0, lam)
        up = 2.0 * oracle.density(ref) * ref
        assert rel(out[i].cpu().numpy(), ref) <= 1e-12
        assert rel(g[i].cpu().numpy(), oracle.expand_adjoint(up, dx, 1.0, 9.0, lam)) <= 1e-12


def test_fold_blocked_and_ranges(fx, monkeypatch):
    # blocks of the outer index and ranges of the term index start at q > 0 and accumulate
    shape, lam, dx, t = (42, 45, 50), (4, 6, 9), (1.0, 1.0, 1.0), 8.0
    print("fold blocked", shape, lam, flush=True)
    f = workloads.random_field(shape, 7300)
    y = workloads.random_field(shape, 7301)
    ref = oracle.expand(f, dx, 1.0, t, lam)
    monkeypatch.setenv("FX_WORKSPACE_MB", "8")
    plan = fx.Plan(shape, dx, 1.0, t, lam)
    assert json.loads(plan.describe())["outer_block"] < 9
    out, _ = plan.expand(torch.from_numpy(f).cuda())
    g = plan.expand_adjoint(torch.from_numpy(y).cuda())
    acc = torch.zeros(shape, dtype=torch.complex128, device="cuda")
    cuts = [0, 1, 7, 50, 121, 216]
    for b, e in zip(cuts[:-1], cuts[1:]):
        plan.expand_range(torch.from_numpy(f).cuda(), acc, b, e, accumulate=True)
    torch.cuda.synchronize()
    assert rel(out.cpu().numpy(), ref) <= 1e-12
    assert rel(acc.cpu().numpy(), ref) <= 1e-12
    assert rel(g.cpu().numpy(), oracle.expand_adjoint(y, dx, 1.0, t, lam)) <= 1e-12
