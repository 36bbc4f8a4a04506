"""All iterations of an fp32 call in one launch: the results of a launch per step, bit for bit, and the oracle's, at the edges of
its variants (orders with and without a remainder in the slab ring, fewer slabs than it has places, both tile sizes, 16 to 64 sketch
columns, no sketch, more iterations than the ring of arrays has sets), for every function that takes it.

A caller's workspace that is too small for the ring of arrays gets the launches.  The products sum in the same order on
both ways; the residual is summed by tile, whose size differs: relative error of fp32 partial sums, 1e-6.
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


def _spd(n, batch, seed):
    rng = np.random.default_rng(seed)
    w = rng.standard_normal((batch, n, 2 * n))
    return (w @ w.transpose(0, 2, 1) / (2 * n) + 1e-3 * np.eye(n)).astype(np.float32)


def _both(prism, call, fn, A, degree, sketch, p=0):
    """Outputs and reports on the library's workspace and on one 256 bytes too small for the ring."""
    need = prism.workspace_bytes(fn, A.shape[0], A.shape[1], A.shape[2], prism.F32, degree, sketch, p)
    res = []
    for ws in (None, torch.empty(need - 256, dtype=torch.uint8, device="cuda")):
        x = torch.from_numpy(A.copy()).cuda()
        out = call(x, ws)
        info = out[1] if isinstance(out, tuple) else out
        res.append(([x.cpu().numpy()] + ([out[0].cpu().numpy()] if isinstance(out, tuple) else []), info.read()))
    (xs, r), (ys, q) = res
    for x, y in zip(xs, ys):
        assert np.array_equal(x, y)
    assert np.array_equal(r["iters"], q["iters"]) and np.array_equal(r["status"], q["status"]) and np.array_equal(r["alpha"], q["alpha"])
    assert np.allclose(r["residual"], q["residual"], rtol=1e-6, atol=1e-6)   # atol: 1 - G at rounding level
    return xs, r


@pytest.mark.parametrize("batch,m,n,degree,sketch,tol,iters,warm", [
    (1, 100, 70, 5, 8, 1e-5, 40, 0), (3, 500, 299, 5, 8, 1e-5, 40, 0), (2, 180, 400, 3, 16, 1e-5, 40, 2), (1, 900, 600, 5, 32, 1e-5, 40, 0),
    (2, 300, 200, 5, 40, 1e-5, 40, 0), (2, 256, 128, 5, 0, 1e-5, 40, 0), (1, 512, 512, 5, 16, 0.0, 12, 3), (4, 300, 190, 5, 16, 1e-5, 0, 0), (2, 300, 190, 3, 16, 0.0, 1, 0),
    (2, 300, 60, 5, 8, 1e-5, 40, 0), (1, 33, 200, 3, 16, 1e-5, 40, 0), (3, 65, 20, 5, 32, 1e-5, 40, 0)])
def test_polar(prism, batch, m, n, degree, sketch, tol, iters, warm):
    rng = np.random.default_rng(m + n)
    A = (rng.standard_normal((batch, m, n)) * 10.0 ** (-rng.random((batch, 1, n)))).astype(np.float32)
    if batch > 2:
        A[1] = 0.0   # reported, never touched, while the others go on
    xs, r = _both(prism, lambda x, ws: prism.polar(x, degree, iters, sketch, SEED, tol, warm_iters=warm, workspace=ws), prism.FN_POLAR, A, degree, sketch)
    if batch > 2:
        assert not xs[0][1].any()
    ref, oinfo = O.polar(A[0], degree, iters, sketch, SEED, tol, alpha_schedule=[1.45 if degree == 5 else 1.0] * warm)
    assert int(r[0]["iters"]) == oinfo["iters"]
    if iters > 1:
        assert np.linalg.norm(xs[0][0] - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("batch,n,p,sketch,tol,iters", [
    (2, 100, 4, 16, 1e-5, 40), (1, 144, 3, 16, 1e-5, 40), (9, 256, 2, 32, 1e-5, 40), (2, 577, 4, 16, 1e-5, 40), (1, 768, 4, 32, 1e-5, 40),
    (3, 300, 4, 64, 1e-5, 40), (2, 400, 4, 0, 1e-5, 60), (5, 200, 3, 8, 0.0, 11), (2, 60, 4, 40, 1e-5, 40), (1, 64, 2, 64, 1e-5, 40), (3, 17, 3, 33, 1e-5, 40)])
def test_inverse_root(prism, batch, n, p, sketch, tol, iters):
    A = np.repeat(W.c4_shampoo_spd(n=n, batch=1), batch, axis=0)
    xs, r = _both(prism, lambda x, ws: prism.inv_root(x, p, iters, sketch, SEED, tol, workspace=ws), prism.FN_INV_ROOT, A, 3, sketch, p)
    assert all(np.array_equal(xs[0][0], xs[0][b]) for b in range(1, batch))
    ref, oinfo = O.inv_root(A[0], p, iters, sketch, SEED, tol)
    assert int(r[0]["iters"]) == oinfo["iters"]
    assert np.linalg.norm(xs[0][0] - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("batch,n,degree,sketch,iters", [(1, 130, 5, 16, 40), (2, 500, 3, 16, 40), (4, 256, 5, 32, 40), (1, 700, 5, 16, 40), (2, 350, 5, 50, 40),
                                                         (1, 64, 5, 16, 40), (3, 50, 3, 32, 40), (2, 20, 5, 40, 40)])
def test_square_root_sign_and_inverse(prism, batch, n, degree, sketch, iters):
    A = _spd(n, batch, n)
    xs, r = _both(prism, lambda x, ws: prism.sqrt(x, degree, iters, sketch, SEED, 1e-5, workspace=ws), prism.FN_SQRT, A, degree, sketch)
    w, v = np.linalg.eigh(A[0].astype(np.float64))
    root, inv = (v * np.sqrt(w)) @ v.T, (v / np.sqrt(w)) @ v.T
    assert np.linalg.norm(xs[0][0] - root) <= 1e-5 * np.linalg.norm(root) and np.linalg.norm(xs[1][0] - inv) <= 1e-5 * np.linalg.norm(inv)
    B = W.sign_indefinite(n=n, batch=batch)
    xs, r = _both(prism, lambda x, ws: prism.sign(x, degree, iters, sketch, SEED, 1e-5, workspace=ws), prism.FN_SIGN, B, degree, sketch)
    ref, oinfo = O.sign(B[0], degree, iters, sketch, SEED, 1e-5)
    assert int(r[0]["iters"]) == oinfo["iters"] and np.linalg.norm(xs[0][0] - ref) <= 1e-4 * np.linalg.norm(ref)
    rng = np.random.default_rng(n)
    Cm = (A + 0.2 * rng.standard_normal(A.shape) / np.sqrt(n)).astype(np.float32)   # not symmetric
    xs, r = _both(prism, lambda x, ws: prism.inverse(x, iters, sketch, SEED, 1e-5, workspace=ws), prism.FN_INVERSE, Cm, 5, sketch)
    ref, oinfo = O.inverse(Cm[0], iters, sketch, SEED, 1e-5)
    assert int(r[0]["status"]) == oinfo["status"]
    if oinfo["status"] == 0:
        assert np.linalg.norm(xs[0][0] - ref) <= 1e-4 * np.linalg.norm(ref)


def test_coefficient_schedule(prism):
    """A caller's coefficients and the fit behind them, past one turn of the ring."""
    A = W.sign_indefinite(n=300, batch=2)
    sched = [1.2, 0.9, 1.0]
    xs, r = _both(prism, lambda x, ws: prism.sign(x, 5, 20, 16, SEED, 1e-5, alpha_schedule=sched, workspace=ws), prism.FN_SIGN, A, 5, 16)
    ref, oinfo = O.sign(A[0], 5, 20, 16, SEED, 1e-5, alpha_schedule=sched)
    assert np.allclose(r[0]["alpha"][:3], sched) and int(r[0]["iters"]) == oinfo["iters"]
    assert np.linalg.norm(xs[0][0] - ref) <= 1e-4 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,batch", [(256, 16), (320, 12)])
def test_both_sides_of_the_largest_batch(prism, n, batch):
    """With one matrix more there is no workgroup left for every row block of a fit, and the call takes a launch per step: the same bits
    for the others, and iteration counts."""
    A = np.concatenate([W.sign_indefinite(n=n, batch=2), W.sign_indefinite(n=n, batch=1, data_seed=77)])
    A = np.tile(A, (batch // 3 + 2, 1, 1))
    res = []
    for count in (batch, batch + 1):
        x = torch.from_numpy(A[:count].copy()).cuda()
        r = prism.sign(x, 5, 40, 16, SEED, 1e-5).read()
        res.append((x[:batch].cpu().numpy(), r[:batch]))
    (x, r), (y, q) = res
    assert np.array_equal(x, y) and np.array_equal(r["iters"], q["iters"]) and np.array_equal(r["alpha"], q["alpha"])
    ref, oinfo = O.sign(A[0], 5, 40, 16, SEED, 1e-5)
    assert int(r[0]["iters"]) == oinfo["iters"] and np.linalg.norm(x[0] - ref) <= 1e-4 * np.linalg.norm(ref)
