"""fp32 products from three bf16 planes per operand: every function that takes them, at orders on both sides of the padding rule and
batches that get each of the tiles (64 x 64, 128 x 128, 128 x 256), in whole and in partial rounds, in numbers that eight XCDs share evenly and not, against the oracle and against the products of
fp32 operands (what a workspace too small for the planes gets).

Bars: 5e-7 for a single product against 64 bits; calls 1e-5 against the oracle, as for every fp32 path; the two ways differ by their rounding, a few 1e-7 per product, and by a stop
that rounding decides (at most half the tolerance)."""
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


def _operands(kind, batch, m, k, n, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    a, b = (torch.randn(batch, *s, generator=g, device="cuda") for s in ((m, k), (k, n)))
    if kind == "positive":
        a, b = a.abs(), b.abs()
    elif kind == "identity":                  # iterates close to their limit
        a, b = (torch.eye(*x.shape[1:], device="cuda") + 0.01 * x for x in (a, b))
    elif kind == "decades":                   # six of them, along k
        a = a * torch.logspace(-3, 3, k, device="cuda")[None, None, :]
    elif kind == "one":                       # one term per sum, all mantissas
        a, b = (torch.zeros_like(x).scatter_(2, torch.arange(x.shape[1], device="cuda").remainder(x.shape[2])[None, :, None].expand(batch, -1, 1),
                                             1.0 + torch.rand(batch, x.shape[1], 1, generator=g, device="cuda")) for x in (a, b))
    return a, b


# M, K, N, batch: every tile (64 x 64 in one round and in launches of no multiple of 128, 128 x 128, 128 x 256), K of the shortest ring, of partial
# windows of 256 and of whole ones, tile counts that are no multiple of eight
@pytest.mark.parametrize("kind", ["gauss", "positive", "identity", "decades", "one"])
@pytest.mark.parametrize("m,k,n,batch", [(64, 96, 64, 1), (192, 128, 320, 3), (448, 448, 448, 10), (576, 288, 64, 2), (1024, 1056, 1024, 1), (1024, 1024, 1024, 4), (1152, 96, 1152, 3),
                                         (1024, 512, 1280, 9), (1024, 4128, 1024, 8)])
def test_single_product_against_64_bits(prism, kind, m, k, n, batch):
    """Three planes hold an fp32 number exactly, and the three products of planes that are left out are at most 2^-24 of a term together (2^-25 for either m l, 2^-34 for l l;
    rms 2^-27.6), so that a product is as close as fp32 accumulation in windows of 256 makes it: 3e-7.  With the least of the six missing Gaussian operands would be at 2.5e-6."""
    a, b = _operands(kind, batch, m, k, n, m + k + n)
    c = torch.randn(batch, m, n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)) * 0.125
    out = prism.gemm_f32_planes(a, b, c)
    err = ref2 = 0.0
    for i in range(batch):
        ref = c[i].double() + a[i].double() @ b[i].double()
        err += float(((out[i].double() - ref) ** 2).sum())
        ref2 += float((ref ** 2).sum())
    assert np.sqrt(err / ref2) <= 5e-7, np.sqrt(err / ref2)


@pytest.mark.parametrize("kind", ["gauss", "positive", "decades"])
@pytest.mark.parametrize("m,k,batch", [(64, 96, 1), (192, 320, 3), (448, 672, 9), (1024, 1056, 1), (1024, 1536, 7), (1152, 1184, 8)])
def test_gram_product_against_64_bits(prism, kind, m, k, batch):
    """I - A^T A with A stored [K][M]: whole 64 x 64 blocks below the diagonal are the mirror image of those above, to the bit; within a block on the diagonal the two
    halves are computed each for itself (see gemm_split.hip) and agree to rounding (1e-8 of the norm)."""
    at, _ = _operands(kind, batch, k, m, 8, m + k)
    if kind == "decades":                     # along the columns here: the sums keep their range
        at = at / torch.logspace(-3, 3, m, device="cuda")[None, None, :]
    at = at.contiguous()
    out = prism.gemm_f32_planes(at, at)
    ref = torch.eye(m, device="cuda", dtype=torch.float64) - torch.stack([x.double().t().contiguous() @ x.double() for x in at])
    assert float((out.double() - ref).norm() / ref.norm()) <= 5e-7
    blocks = out.view(batch, m // 64, 64, m // 64, 64)
    mirror = out.transpose(1, 2).contiguous().view(batch, m // 64, 64, m // 64, 64)
    diag = torch.eye(m // 64, dtype=torch.bool, device="cuda")[None, :, None, :, None]
    assert bool(((blocks == mirror) | diag).all())
    assert float((out - out.transpose(1, 2)).double().norm() / ref.norm()) <= 5e-8


def test_products_of_planes_that_are_refused(prism):
    a = torch.zeros(1, 64, 96, device="cuda")
    lib = prism.lib()
    call = lambda m, n, k, km: lib.prism_gemm_f32_planes(a.data_ptr(), a.data_ptr(), a.data_ptr(), 1, m, n, k, km, None)
    assert [call(*x) for x in ((32, 64, 96, 0), (64, 96, 96, 0), (64, 64, 64, 0), (64, 64, 100, 0), (64, 64, 96, 2), (64, 128, 96, 1))] == [prism.EINVAL] * 6


def _rel(x, ref):
    return np.linalg.norm(np.asarray(x, dtype=np.float64) - ref) / np.linalg.norm(ref)


def _spd(n, batch):
    rng = np.random.default_rng(n)
    out = np.empty((batch, n, n), np.float32)
    w = rng.standard_normal((n, 2 * n))
    a = w @ w.T / (2 * n)
    for b in range(batch):   # one spectrum shifted: cheap, and no two matrices are the same
        out[b] = a + (0.02 + 0.01 * b) * np.eye(n)
    return out


def _general(n, batch):
    rng = np.random.default_rng(n)
    return (rng.standard_normal((batch, n, n)) / np.sqrt(n) * 0.3 + np.eye(n)).astype(np.float32)


def _both(prism, call, fn, A, degree, sketch, p=0):
    """Outputs and report from planes, and outputs from fp32 operands (a workspace 256 bytes short of the planes)."""
    need = prism.workspace_bytes(fn, A.shape[0], A.shape[1], A.shape[2], prism.F32, degree, sketch, p)
    res = []
    for ws in (None, torch.empty(need - 256, dtype=torch.uint8, device="cuda")):
        x = torch.from_numpy(A.copy()).cuda()
        out = call(x, ws)
        info = out[1] if isinstance(out, tuple) else out
        res.append(([x.cpu().numpy()] + ([out[0].cpu().numpy()] if isinstance(out, tuple) else []), info.read()))
    (xs, r), (ys, q) = res
    assert np.array_equal(r["status"], q["status"]) and np.abs(r["iters"] - q["iters"]).max() <= 1
    for x, y in zip(xs, ys):
        assert not np.array_equal(x, y)      # the planes were taken
        assert _rel(x, y.astype(np.float64)) <= 1e-5
    return xs, r


def _same(info, oinfo):
    assert info["iters"] == oinfo["iters"] and info["status"] == oinfo["status"], (info["residual"][:info["iters"] + 1], oinfo["residual"])


@pytest.mark.parametrize("n,batch,degree", [(384, 24, 5), (440, 10, 5), (450, 20, 3), (800, 1, 5), (1000, 1, 5), (1000, 4, 3), (1000, 8, 5), (1025, 1, 5)])
def test_sign(prism, n, batch, degree):
    A = W.sign_indefinite(n=n, batch=1, decades=1.5).repeat(batch, 0)
    A *= np.linspace(1.0, 2.0, batch, dtype=np.float32)[:, None, None]
    xs, r = _both(prism, lambda x, ws: prism.sign(x, degree, 40, 16, SEED, 1e-5, workspace=ws), prism.FN_SIGN, A, degree, 16)
    for b in (0, batch - 1):
        ref, oinfo = O.sign(A[b], degree, 40, 16, SEED, 1e-5)
        assert _rel(xs[0][b], ref) <= 1e-5
        _same(r[b], oinfo)


@pytest.mark.parametrize("n,batch,degree", [(470, 24, 5), (570, 5, 3), (800, 1, 3), (1000, 2, 5), (1024, 5, 5)])
def test_sqrt(prism, n, batch, degree):
    A = _spd(n, batch)
    xs, r = _both(prism, lambda x, ws: prism.sqrt(x, degree, 40, 16, SEED, 1e-5, workspace=ws), prism.FN_SQRT, A, degree, 16)
    for b in (0, batch - 1):
        s, inv, oinfo = O.sqrt(A[b], degree, 40, 16, SEED, 1e-5)
        assert _rel(xs[0][b], s) <= 1e-5 and _rel(xs[1][b], inv) <= 1e-5
        _same(r[b], oinfo)


@pytest.mark.parametrize("n,batch,p", [(1000, 1, 4), (832, 1, 2), (1024, 3, 3), (1000, 2, 2), (1024, 1, 5), (1000, 1, 8)])
def test_inverse_root(prism, n, batch, p):
    A = W.c4_shampoo_spd(n=n, batch=batch)
    if n == 832:   # padding to whole tiles of 128 would cost more than it gains: fp32 operands, whatever the workspace
        assert prism.workspace_bytes(prism.FN_INV_ROOT, 1, n, n, prism.F32, 3, 16, p) < prism.workspace_bytes(prism.FN_INV_ROOT, 1, 833, 833, prism.F32, 3, 16, p)
        return
    xs, r = _both(prism, lambda x, ws: prism.inv_root(x, p, 40, 16, SEED, 1e-5, workspace=ws), prism.FN_INV_ROOT, A, 3, 16, p)
    ref, oinfo = O.inv_root(A[-1], p, 40, 16, SEED, 1e-5)
    assert _rel(xs[0][-1], ref) <= 1e-5
    _same(r[-1], oinfo)


@pytest.mark.parametrize("n,batch", [(500, 20), (900, 1), (1000, 4)])
def test_inverse(prism, n, batch):
    A = _general(n, batch)
    xs, r = _both(prism, lambda x, ws: prism.inverse(x, 40, 16, SEED, 1e-5, workspace=ws), prism.FN_INVERSE, A, 5, 16)
    ref, oinfo = O.inverse(A[-1], 40, 16, SEED, 1e-5)
    assert _rel(xs[0][-1], ref) <= 1e-5
    _same(r[-1], oinfo)


@pytest.mark.parametrize("batch,m,n,degree", [(20, 700, 500, 5), (2, 700, 1200, 3), (1, 1500, 1000, 5), (4, 1000, 1000, 5), (1, 5000, 800, 5)])
def test_polar(prism, batch, m, n, degree):
    rng = np.random.default_rng(m + n)
    A = (rng.standard_normal((batch, m, n)) * (10.0 ** (-rng.random((batch, 1, n))) if m > n else 1.0)).astype(np.float32)
    if m == n:
        A += 2.0 * np.sqrt(n) * np.eye(n, dtype=np.float32)
    if batch > 2:
        A[1] = 0.0   # reported, never touched, while the others go on
    xs, r = _both(prism, lambda x, ws: prism.polar(x, degree, 40, 16, SEED, 1e-5, workspace=ws), prism.FN_POLAR, A, degree, 16)
    ref, oinfo = O.polar(A[-1], degree, 40, 16, SEED, 1e-5)
    assert _rel(xs[0][-1], ref) <= 1e-5
    _same(r[-1], oinfo)
    if batch > 2:
        assert r[1]["status"] == prism.INFO_ZERO and not xs[0][1].any()


def test_a_wild_schedule_diverges_at_the_oracles_iteration(prism):
    """Products that leave the range of fp32 end in infinities or NaN, and the matrix is stopped as it is with fp32 operands."""
    A = _spd(1000, 1)
    sched = [30.0] * 20
    x = torch.from_numpy(A.copy()).cuda()
    _, info = prism.sqrt(x, 5, 20, 8, SEED, 1e-5, alpha_schedule=sched)
    rec = info.read()[0]
    *_, oinfo = O.sqrt(A[0], 5, 20, 8, SEED, 1e-5, alpha_schedule=sched)
    assert rec["status"] == prism.INFO_DIVERGED == oinfo["status"] and rec["iters"] == oinfo["iters"]


def test_largest_finite_entries_do_not_round_to_infinity(prism):
    """A norm that only just is finite in 32 bits."""
    A = _spd(1000, 1)
    A *= np.float32(3.3e38) / np.abs(A).max()
    x = torch.from_numpy(A.copy()).cuda()
    _, info = prism.sqrt(x, 5, 40, 16, SEED, 1e-5)
    s, _, oinfo = O.sqrt(A[0], 5, 40, 16, SEED, 1e-5)
    assert _rel(x.cpu().numpy()[0], s) <= 1e-5
    _same(info.read()[0], oinfo)
