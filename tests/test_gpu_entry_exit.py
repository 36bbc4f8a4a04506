"""Copy-in, copy-out and the split Gram product of the bf16 polar factor at the edges of their tiles: sides that no
vector width divides, arrays that start anywhere, wide matrices (transposed on the way), single long matrices whose
K loop is cut into parts.  Against the exact polar factor (SVD in fp64): Gaussian matrices with sides in a ratio of 1.5
and more are converged after eight updates, so the bf16 bar of 2e-2 holds for it as for the oracle.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def prism():
    from paper_2601_22137_amd import prism as P
    P.lib()
    return P


@pytest.mark.parametrize("m,n,batch", [(513, 200, 2), (200, 513, 2), (777, 136, 3), (1025, 129, 2), (129, 1025, 2), (71, 8, 2), (8, 71, 1),
                                       (1536, 256, 1), (3000, 300, 1), (301, 3001, 1), (9000, 130, 3)])
@pytest.mark.parametrize("offset", [0, 3])
@pytest.mark.parametrize("plain", [False, True])
def test_polar_bf16_any_shape_any_start(prism, m, n, batch, offset, plain):
    torch.manual_seed(m * 10007 + n)
    buf = torch.zeros(batch * m * n + 24, device="cuda", dtype=torch.bfloat16)
    x = buf[offset:offset + batch * m * n].view(batch, m, n)
    x.copy_(torch.randn(batch, m, n, device="cuda"))
    a = x.float().cpu().numpy().astype(np.float64)
    prism.polar(x, 5, 8, 16, 7, 0.0, flags=prism.FLAG_BF16_PLAIN_ITERATE if plain else 0)
    got = x.float().cpu().numpy().astype(np.float64)
    for b in range(batch):
        u, _, vh = np.linalg.svd(a[b], full_matrices=False)
        ref = u @ vh
        assert np.linalg.norm(got[b] - ref) <= 2e-2 * np.linalg.norm(ref)
    assert not buf[:offset].any() and not buf[offset + batch * m * n:].any()   # nothing written outside


def test_split_gram_product_fits_in_less_scratch(prism):
    """A workspace without room for the partial products: the one-pass product, same result to rounding."""
    m, n = 3072, 256
    torch.manual_seed(5)
    a = torch.randn(1, m, n, device="cuda").to(torch.bfloat16)
    x, y = a.clone(), a.clone()
    prism.polar(x, 5, 5, 16, 7, 0.0)
    size = lambda batch: prism.workspace_bytes(prism.FN_POLAR, batch, m, n, prism.BF16, 5, 16)
    one_pass = size(8) - 7 * ((size(16) - size(8)) // 8) + 65536     # batches of such matrices are not split
    assert one_pass < size(1)
    ws = torch.empty(one_pass, device="cuda", dtype=torch.uint8)
    prism.polar(y, 5, 5, 16, 7, 0.0, workspace=ws)
    assert torch.linalg.norm(x.double() - y.double()) <= 1e-2 * torch.linalg.norm(x.double())


@pytest.mark.parametrize("m,n,batch", [(9001, 300, 1), (8065, 70, 3), (130, 12011, 2)])
def test_polar_fp32_split_gram_product_of_any_length(prism, m, n, batch):
    """fp32: lengths that no number of parts divides.  Converged to 1e-6; the sums over 10^4 rows, in parts of 10^3 and those in
    chunks of 256, keep the error near 2^-24 sqrt(256): the fp32 bar of 1e-5."""
    torch.manual_seed(m + n)
    x = torch.randn(batch, m, n, device="cuda")
    a = x.cpu().numpy().astype(np.float64)
    prism.polar(x, 5, 30, 16, 7, 1e-6)
    got = x.cpu().numpy().astype(np.float64)
    for b in range(batch):
        u, _, vh = np.linalg.svd(a[b], full_matrices=False)
        assert np.linalg.norm(got[b] - u @ vh) <= 1e-5 * np.sqrt(min(m, n))


def test_norm_does_not_depend_on_the_address(prism):
    """The Frobenius norm is added up in an order that follows from the shape alone.  Without an update a call returns the
    scaled input; a norm that differs in its last fp64 bits shows in one of some 10^8 entries, so there are 10^9 here."""
    b, m, n = 48, 1000, 999
    for seed in range(6):
        torch.manual_seed(seed)
        a = torch.randn(b, m, n, device="cuda")
        buf = torch.empty(a.numel() + 8, device="cuda")
        first = None
        for offset in (0, 1, 2, 3):
            x = buf[offset:offset + a.numel()].view_as(a)
            x.copy_(a)
            prism.polar(x, 5, 0, 8, 7, 0.0)
            bits = x.view(torch.int32)
            if first is None:
                first = bits.clone()
            assert torch.equal(bits, first), (seed, offset)
