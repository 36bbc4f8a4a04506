"""Calls that run as one workgroup per matrix: orders at both sides of every 16-row block, both orientations, sketch widths of one
and two rounds of column blocks, every root order, against the oracle (fp32 results: 1e-5 relative, equal iteration counts).
"""
import numpy as np
import pytest
import torch

from oracle import prism_ref as O
from paper_2601_22137_amd import workloads as W

pytestmark = pytest.mark.gpu
SEED = W.SKETCH_SEED


@pytest.fixture(scope="module")
def prism():
    from paper_2601_22137_amd import prism as P
    P.lib()
    return P


@pytest.mark.parametrize("m,n,degree,sketch", [
    (1, 1, 5, 8), (16, 1, 5, 8), (20, 15, 5, 8), (17, 16, 3, 16), (64, 17, 5, 17), (31, 40, 5, 8), (33, 32, 5, 40), (64, 33, 5, 8), (48, 64, 3, 20),
    (64, 49, 5, 64), (63, 50, 5, 16), (7, 64, 5, 32)])
def test_polar(prism, m, n, degree, sketch):
    rng = np.random.default_rng(100 * m + n)
    s, l = min(m, n), max(m, n)
    u, v = np.linalg.qr(rng.standard_normal((l, s)))[0], np.linalg.qr(rng.standard_normal((s, s)))[0]
    x = (u * 10.0 ** (-rng.random(s))) @ v.T
    A = (x if m >= n else x.T).astype(np.float32)
    X = torch.from_numpy(np.ascontiguousarray(np.stack([A, np.zeros_like(A), 3.0 * A]))).cuda()
    r = prism.polar(X, degree, 40, sketch, SEED, 1e-5).read()
    Y = X.cpu().numpy()
    ref, oinfo = O.polar(A, degree, 40, sketch, SEED, 1e-5)
    assert int(r[0]["iters"]) == int(r[2]["iters"]) == oinfo["iters"] and int(r[0]["status"]) == 0
    assert int(r[1]["status"]) == prism.INFO_ZERO and not Y[1].any()
    for b in (0, 2):
        assert np.linalg.norm(Y[b] - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,p,sketch", [(1, 2, 8), (10, 4, 16), (16, 3, 32), (17, 1, 8), (32, 4, 16), (33, 2, 20), (48, 4, 32), (49, 3, 16), (64, 4, 8), (64, 1, 32)])
def test_inverse_root(prism, n, p, sketch):
    rng = np.random.default_rng(n + p)
    w = rng.standard_normal((n, 2 * n))
    A = (w @ w.T / (2 * n) + 1e-2 * np.eye(n)).astype(np.float32)
    bad = A.copy()
    bad[0, 0] = np.nan
    X = torch.from_numpy(np.stack([A, bad, A])).cuda()
    r = prism.inv_root(X, p, 40, sketch, SEED, 1e-5).read()
    Y = X.cpu().numpy()
    ref, oinfo = O.inv_root(A, p, 40, sketch, SEED, 1e-5)
    assert int(r[0]["iters"]) == oinfo["iters"] and int(r[0]["status"]) == 0
    assert int(r[1]["status"]) == prism.INFO_NONFINITE and np.array_equal(Y[1], bad, equal_nan=True)
    assert np.array_equal(Y[0], Y[2])
    assert np.linalg.norm(Y[0] - ref) <= 1e-5 * np.linalg.norm(ref)
    # a fixed budget with a first update at the upper end, no fit behind it
    X = torch.from_numpy(A[None].copy()).cuda()
    r = prism.inv_root(X, p, 3, 0, SEED, 0.0, warm_iters=1).read()
    ref, oinfo = O.inv_root(A, p, 3, 0, SEED, 0.0)
    assert int(r[0]["iters"]) == 3 and np.linalg.norm(X.cpu().numpy()[0] - ref) <= 1e-5 * np.linalg.norm(ref)


def test_profile_kinds_of_the_combined_launches(prism):
    """A launch that does the work of several steps is booked as itself, not as one of the products in it."""
    bf16 = torch.from_numpy(W.c2_muon_group(1, batch=1).view(np.int16)).cuda().view(torch.bfloat16)
    spd = {n: torch.from_numpy(W.c4_shampoo_spd(n=n, batch=1)).cuda() for n in (48, 200)}
    calls = [("fit_square", 5, ("bf16_polyq", "chain"), lambda: prism.polar(bf16.clone(), 5, 5, 16, SEED, 0.0, flags=prism.FLAG_BF16_PLAIN_ITERATE)),
             ("flow", 1, ("f32_apply", "f32_store", "f64_mnext"), lambda: prism.inv_root(spd[200].clone(), 4, 40, 16, SEED, 1e-5)),
             ("small_root", 1, ("f32_apply", "f32_store", "f64_mnext"), lambda: prism.inv_root(spd[48].clone(), 4, 40, 16, SEED, 1e-5))]
    for kind, count, others, call in calls:
        prism.profile_enable(True)
        try:
            call()
            torch.cuda.synchronize()
            prof = prism.profile_collect()
        finally:
            prism.profile_enable(False)
        assert prof[kind][1] == count and prof[kind][0] > 0.0
        assert not any(prof[k][1] for k in others)
