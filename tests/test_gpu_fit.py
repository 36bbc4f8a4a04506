"""The one-launch fit (sketch chain, moments, coefficient) against the fp64 oracle: the coefficients of the first
updates (at the upper end of their interval) and of the later ones, which the fit decides, at both sides of every limit
of its variants (order 64, which inverse roots up to p = 4 spend in one workgroup, 512, 1024, 2048; 16 and 32 rows per
workgroup; sketches of 16, 32 and 64 columns; the longest chain), and equal bits for equal matrices whatever their place
in a batch.

The chain is carried out in fp32 from the matrix R that the iteration itself has (relative error of a coefficient: a few
n * 2^-24 of partial sums that average out, measured below 1e-6); R of the second update carries the rounding of
the first.  bf16 polar factors fit from the bf16 R with the exact diagonal: 2e-2 as in the parity tests.
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


@pytest.mark.parametrize("n,batch,sketch,p", [
    (40, 3, 16, 4), (64, 2, 8, 1), (33, 2, 32, 2), (64, 300, 16, 3), (7, 1, 16, 4), (64, 5, 40, 4), (50, 2, 16, 5), (65, 2, 16, 4), (130, 2, 32, 2), (512, 1, 16, 4), (512, 17, 8, 4), (513, 1, 16, 4),
    (300, 1, 16, 8), (1000, 1, 32, 4), (1024, 9, 16, 4), (1024, 1, 64, 4), (1025, 1, 16, 4), (2048, 1, 32, 2)])
def test_inverse_root_coefficients(prism, n, batch, sketch, p):
    A = W.c4_shampoo_spd(n=n, batch=1)
    x = torch.from_numpy(np.repeat(A, batch, axis=0)).cuda()
    rec = prism.inv_root(x, p, 2, sketch, SEED, 0.0).read()
    ref, oinfo = O.inv_root(A[0], p, 2, sketch, SEED, 0.0)
    assert np.abs(rec[0]["alpha"][:2] - np.array(oinfo["alpha"][:2])).max() <= 1e-5
    out = x.cpu().numpy()
    assert np.linalg.norm(out[0] - ref) <= 1e-5 * np.linalg.norm(ref)
    assert all(np.array_equal(out[0], out[b]) for b in range(1, batch))
    assert all(np.array_equal(rec[0]["alpha"][:2], rec[b]["alpha"][:2]) for b in range(1, batch))


@pytest.mark.parametrize("n,batch,sketch", [(128, 2, 16), (512, 20, 32), (768, 1, 16), (768, 12, 16), (1024, 1, 32), (1280, 1, 16)])
def test_bf16_polar_coefficients(prism, n, batch, sketch):
    A = W.c3_polar_large(n=n, batch=1, sigma_decades=2.0)
    bits = W.to_bf16_bits(A) if A.dtype != np.uint16 else A
    x = torch.from_numpy(np.repeat(bits, batch, axis=0).view(np.int16)).cuda().view(torch.bfloat16)
    rec = prism.polar(x, 5, 2, sketch, SEED, 0.0).read()
    _, oinfo = O.polar(W.from_bf16_bits(bits)[0], 5, 2, sketch, SEED, 0.0)
    assert np.abs(rec[0]["alpha"][:2] - np.array(oinfo["alpha"][:2])).max() <= 2e-2
    out = x.view(torch.int16).cpu().numpy()
    assert all(np.array_equal(out[0], out[b]) for b in range(1, batch))


@pytest.mark.parametrize("degree", [3, 5])
def test_sign_coefficients_many_matrices(prism, degree):
    """More clusters than fit the chip at a time (2000 matrices of 8 workgroups)."""
    A = W.sign_indefinite(n=128, batch=2)
    x = torch.from_numpy(np.tile(A, (1000, 1, 1))).cuda()
    rec = prism.sign(x, degree, 3, 16, SEED, 0.0).read()
    out = x.cpu().numpy()
    for b in range(2):
        ref, oinfo = O.sign(A[b], degree, 3, 16, SEED, 0.0)
        assert np.abs(rec[b]["alpha"][:3] - np.array(oinfo["alpha"][:3])).max() <= 1e-4
        assert np.linalg.norm(out[b] - ref) <= 1e-4 * np.linalg.norm(ref)
        assert np.array_equal(out[b::2], np.broadcast_to(out[b], out[b::2].shape))


@pytest.mark.parametrize("n,batch,sketch", [(65, 3, 16), (300, 2, 16), (512, 20, 32), (500, 17, 8), (1000, 1, 32), (1024, 9, 16),
                                            (600, 2, 64), (1024, 1, 40), (1100, 2, 16), (2048, 1, 32)])
def test_rows_computed_for_a_missing_partner_fp32(prism, n, batch, sketch):
    """A workgroup does not depend on the others of its matrix being resident: with the wait cut to nothing every one
    computes what it finds missing itself, with the same bits.  (Enough updates, here and below, for coefficients inside
    their interval.)"""
    A = W.c4_shampoo_spd(n=n, batch=batch)
    recs, outs = [], []
    for flags in (0, prism.FLAG_FIT_NO_WAIT):
        x = torch.from_numpy(A.copy()).cuda()
        recs.append(prism.inv_root(x, 2, 10, sketch, SEED, 0.0, flags=flags).read())
        outs.append(x.cpu().numpy())
    assert np.array_equal(recs[0]["alpha"], recs[1]["alpha"]) and np.array_equal(recs[0]["residual"], recs[1]["residual"])
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("n,batch,sketch", [(128, 2, 16), (500, 20, 32), (768, 1, 16), (768, 12, 16), (1024, 1, 32), (1280, 1, 16), (1300, 2, 32)])
@pytest.mark.parametrize("plain", [False, True])
def test_rows_computed_for_a_missing_partner_bf16(prism, n, batch, sketch, plain):
    A = W.c3_polar_large(n=n, batch=batch, sigma_decades=2.0)
    base = prism.FLAG_BF16_PLAIN_ITERATE if plain else 0
    recs, outs = [], []
    for flags in (base, base | prism.FLAG_FIT_NO_WAIT):
        x = torch.from_numpy(A.view(np.int16)).cuda().view(torch.bfloat16)
        recs.append(prism.polar(x, 5, 9, sketch, SEED, 0.0, flags=flags).read())
        outs.append(x.view(torch.int16).cpu().numpy())
    assert np.array_equal(recs[0]["alpha"], recs[1]["alpha"]) and np.array_equal(recs[0]["residual"], recs[1]["residual"])
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("m,n,sketch", [(128, 100, 16), (300, 257, 32), (640, 640, 16), (1024, 1000, 32)])
def test_square_beside_the_fit_bf16(prism, m, n, sketch):
    """Q is formed by the launch that fits its coefficient: matrices that stop at different iterations, one that never starts."""
    A = W.c3_polar_large(n=max(m, n), batch=2, sigma_decades=1.0)[:, :, :n]
    bits = np.ascontiguousarray(np.concatenate([A, np.zeros_like(A[:1]), A[1:]]))
    x = torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)
    r = prism.polar(x, 5, 20, sketch, SEED, 2e-2).read()
    out = x.view(torch.int16).cpu().numpy().view(np.uint16)
    assert int(r[2]["status"]) == prism.INFO_ZERO and not out[2].any() and np.array_equal(out[1], out[3])
    for b in (0, 1):
        ref, oinfo = O.polar(W.from_bf16_bits(bits)[b], 5, 20, sketch, SEED, 2e-2)
        assert abs(int(r[b]["iters"]) - oinfo["iters"]) <= (0 if oinfo["residual"][-1] < 1.8e-2 else 1)
        assert np.linalg.norm(W.from_bf16_bits(out)[b] - ref) <= 2e-2 * np.linalg.norm(ref)


@pytest.mark.parametrize("batch,m,n,sketch", [(1, 768, 3072, 16), (2, 128, 100, 16), (3, 300, 257, 32), (2, 640, 640, 16), (16, 768, 768, 16), (2, 1024, 1000, 32)])
def test_square_beside_the_fit_bits(prism, batch, m, n, sketch):
    """The coefficients that a call reports, given to another one: that one forms Q in a launch of its own, and the bits are the same.
    (Plain iterate: with the split one the fit also decides when its low half is left out.)"""
    rng = np.random.default_rng(m + n)
    A = (rng.standard_normal((batch, m, n)) * np.exp(rng.standard_normal((batch, m, 1)))).astype(np.float32)
    x = torch.from_numpy(A).cuda().to(torch.bfloat16)
    plain = prism.FLAG_BF16_PLAIN_ITERATE
    for b in range(batch):               # a schedule holds for all matrices of a call
        x[b] = x[0]
    y = x.clone()
    r = prism.polar(x, 5, 6, sketch, SEED, 0.0, flags=plain).read()
    alpha = r[0]["alpha"][:6]
    assert all(np.array_equal(r[b]["alpha"][:6], alpha) for b in range(batch)) and len(set(alpha)) > 2
    q = prism.polar(y, 5, 6, sketch, SEED, 0.0, flags=plain, alpha_schedule=alpha).read()
    assert np.array_equal(q["residual"][:, :6], r["residual"][:, :6])
    assert torch.equal(x.view(torch.int16), y.view(torch.int16))


@pytest.mark.parametrize("n,p", [(40, 4), (100, 4), (300, 2), (512, 3), (1000, 5)])
def test_inverse_root_alone_and_in_a_batch(prism, n, p):
    """One matrix, where the update of X shares a launch with the first square, and a batch, where it does not: the same bits,
    and the mirrored half of X bit for bit outside the 64 x 64 blocks on the diagonal."""
    A = torch.from_numpy(W.c4_shampoo_spd(n=n, batch=1)).cuda()
    x, y = A.clone(), A.repeat(41 if n < 1000 else 3, 1, 1)
    prism.inv_root(x, p, 30, 16, SEED, 1e-5)
    prism.inv_root(y, p, 30, 16, SEED, 1e-5)
    assert torch.equal(x[0], y[0]) and torch.equal(x[0], y[-1])
    d = x[0] - x[0].T
    for i in range(0, n, 64):
        d[i:i + 64, i:i + 64] = 0
    assert not d.any()
    assert float((x[0] - x[0].T).norm()) <= 2e-6 * float(x[0].norm())   # on the diagonal to rounding: 30 updates of 2^-24


def _inside(alpha, residual, lo, hi):
    """Updates whose coefficient the fit decides and rounding does not: inside its interval, the residual still large."""
    return [k for k in range(len(alpha)) if lo * 1.001 < alpha[k] < hi * 0.999 and residual[k] > 0.05]


# The coefficient follows R: an error of some sqrt(256) 2^-24 = 1e-6 of its entries (sums in fp32, partial sums of 256) is
# at most 20 times larger against a residual of 0.05: 2e-5.  Measured: below 1e-6, sign 5e-6.
@pytest.mark.parametrize("n,batch,sketch,p", [
    (40, 3, 16, 4), (64, 2, 8, 1), (33, 2, 32, 2), (64, 300, 16, 3), (64, 5, 40, 4), (50, 2, 16, 5), (65, 2, 16, 4), (130, 2, 32, 2), (512, 1, 16, 4),
    (512, 17, 8, 4), (513, 1, 16, 4), (300, 1, 16, 8), (1000, 1, 32, 4), (1024, 9, 16, 4), (1024, 1, 64, 4), (1025, 1, 16, 4), (2048, 1, 32, 2)])
def test_inverse_root_coefficients_inside_their_interval(prism, n, batch, sketch, p):
    A = W.c4_shampoo_spd(n=n, batch=1)
    x = torch.from_numpy(np.repeat(A, batch, axis=0)).cuda()
    rec = prism.inv_root(x, p, 9, sketch, SEED, 0.0).read()
    _, oinfo = O.inv_root(A[0], p, 9, sketch, SEED, 0.0)
    alpha = np.array(oinfo["alpha"][:9])
    ks = _inside(alpha, oinfo["residual"], 1.0 / p, 2.0 / p)
    assert ks
    for b in (0, batch - 1):
        assert np.abs(rec[b]["alpha"][ks] - alpha[ks]).max() <= 2e-5 * 2.0 / p


@pytest.mark.parametrize("n,batch,sketch", [(128, 2, 16), (512, 20, 32), (768, 1, 16), (768, 12, 16), (1024, 1, 32), (1280, 1, 16)])
def test_bf16_polar_coefficients_inside_their_interval(prism, n, batch, sketch):
    """The bf16 iterate is known to 2^-9 of its entries, 2e-3, which is what the coefficients were seen to be off; four
    times that."""
    bits = W.c3_polar_large(n=n, batch=1, sigma_decades=2.0)
    x = torch.from_numpy(np.repeat(bits, batch, axis=0).view(np.int16)).cuda().view(torch.bfloat16)
    rec = prism.polar(x, 5, 8, sketch, SEED, 0.0).read()
    _, oinfo = O.polar(W.from_bf16_bits(bits)[0], 5, 8, sketch, SEED, 0.0)
    alpha = np.array(oinfo["alpha"][:8])
    ks = _inside(alpha, oinfo["residual"], 0.375, 1.45)
    assert ks
    for b in (0, batch - 1):
        assert np.abs(rec[b]["alpha"][ks] - alpha[ks]).max() <= 8e-3


@pytest.mark.parametrize("degree,updates", [(3, 13), (5, 9)])
def test_sign_coefficients_inside_their_interval(prism, degree, updates):
    A = W.sign_indefinite(n=128, batch=2)
    x = torch.from_numpy(np.tile(A, (1000, 1, 1))).cuda()
    rec = prism.sign(x, degree, updates, 16, SEED, 0.0).read()
    for b in range(2):
        _, oinfo = O.sign(A[b], degree, updates, 16, SEED, 0.0)
        alpha = np.array(oinfo["alpha"][:updates])
        ks = _inside(alpha, oinfo["residual"], *((0.5, 1.0) if degree == 3 else (0.375, 1.45)))
        assert ks
        for i in (b, b + 1998):
            assert np.abs(rec[i]["alpha"][ks] - alpha[ks]).max() <= 2e-5


@pytest.mark.parametrize("n,copies,degree,updates", [(400, 100, 5, 10), (512, 60, 3, 13)])
def test_sign_coefficients_more_clusters_than_fit_the_chip(prism, n, copies, degree, updates):
    """Orders at which the fit takes a batch of any size in one launch, 14 to 16 workgroups of 32 rows per matrix."""
    A = W.sign_indefinite(n=n, batch=2)
    x = torch.from_numpy(np.tile(A, (copies, 1, 1))).cuda()
    rec = prism.sign(x, degree, updates, 16, SEED, 0.0).read()
    for b in range(2):
        _, oinfo = O.sign(A[b], degree, updates, 16, SEED, 0.0)
        alpha = np.array(oinfo["alpha"][:updates])
        ks = _inside(alpha, oinfo["residual"], *((0.5, 1.0) if degree == 3 else (0.375, 1.45)))
        assert ks
        assert np.abs(rec[b]["alpha"][ks] - alpha[ks]).max() <= 2e-5
        assert all(np.array_equal(rec[b]["alpha"], rec[i]["alpha"]) for i in range(b, 2 * copies, 2))
        assert bool((x[b::2] == x[b]).all())
