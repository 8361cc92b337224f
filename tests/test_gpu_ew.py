"""E of contiguous lines with the rows in registers (k_EW, pruned length 256, 8 and more subsequences) against the
folded kernels in FP64, which the oracle pins (its own matrix of such a line takes minutes): terms that fill the
workgroups' rounds of 16 rows and that do not, ranges of terms that start late, several slices."""

import json
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.join(os.path.dirname(__file__), ".."))

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


def plan_without(fx, monkeypatch, *args, **kw):
    monkeypatch.setenv("FX_EW", "0")
    plan = fx.Plan(*args, **kw)
    monkeypatch.delenv("FX_EW")
    return plan


# (points, lam, lines): g = 8 with whole and partial rounds of 16 terms, g = 16 (refused in FP64)
CASES = [(2048, 40, 130), (2048, 24, 190), (2048, 16 * 5 + 8, 50), (4096, 16, 260)]


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_ew_stack_of_lines(fx, monkeypatch, case, dtype):
    M, lam, count = CASES[case]
    if M == 4096 and dtype == torch.complex128:
        pytest.skip("a line of this length is refused in FP64")
    print("ew stack", dtype, M, lam, count, flush=True)
    npdt = np.complex128 if dtype == torch.complex128 else np.complex64
    f = np.stack([workloads.random_field((M,), 8400 + i).astype(npdt) for i in range(count)])
    x = torch.from_numpy(f).cuda()
    args = ((M,), (1.0,), 1.0, 90.0, (lam,))
    out, rho = fx.Plan(*args, dtype=dtype).expand_many(x)
    refdt = torch.complex64 if M == 4096 else torch.complex128
    ref, rref = plan_without(fx, monkeypatch, *args, dtype=refdt).expand_many(x.to(refdt))
    torch.cuda.synchronize()
    tol = 1e-12 if dtype == torch.complex128 else 1e-5
    assert rel(out.cpu().numpy().astype(np.complex128), ref.cpu().numpy()) <= tol
    assert rel(rho.cpu().numpy().astype(np.float64), rref.cpu().numpy()) <= tol


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_ew_ranges_and_slices(fx, monkeypatch, dtype):
    # a plane with E along its contiguous axis: ranges of terms that start late, two fields
    shape, lam = (300, 2048), (1, 24)
    print("ew plane", dtype, shape, lam, flush=True)
    npdt = np.complex128 if dtype == torch.complex128 else np.complex64
    f = np.stack([workloads.random_field(shape, 8300 + i).astype(npdt) for i in range(2)])
    x = torch.from_numpy(f).cuda()
    args = (shape, (0.9, 1.1), 1.0, 13.0, lam)
    plan = fx.Plan(*args, dtype=dtype)
    passes = json.loads(plan.describe())["passes"]
    assert any(p["kind"] == "E" and p["kernel"] == "k_EW" for p in passes), passes
    out, rho = plan.expand(x[1])
    acc = torch.zeros_like(x[1])
    for b, e in ((0, 1), (1, 24)):
        plan.expand_range(x[1], acc, b, e, accumulate=True)
    pair, _ = plan.expand_many(x)
    ref, rref = plan_without(fx, monkeypatch, *args, dtype=torch.complex128).expand(x[1].to(torch.complex128))
    torch.cuda.synchronize()
    ref = ref.cpu().numpy()
    tol = 1e-12 if dtype == torch.complex128 else 1e-5
    for y in (out, acc, pair[1]):
        assert rel(y.cpu().numpy().astype(np.complex128), ref) <= tol
    assert rel(rho.cpu().numpy().astype(np.float64), rref.cpu().numpy()) <= tol
