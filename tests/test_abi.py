"""The C-ABI library loads and exports every function include/prism.h declares; host-only
argument checks (no GPU needed: prism_workspace_bytes computes on the host)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2601_22137_amd import build, prism
    if not os.path.exists(prism.LIB_PATH):
        build.build(verbose=False)
    return prism.lib()


def _declared():
    text = open(os.path.join(ROOT, "include", "prism.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(prism_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_function_is_exported(lib):
    from paper_2601_22137_amd import prism
    names = _declared()
    assert len(names) >= 12
    for name in names:
        assert hasattr(lib, name), name
    assert sorted(prism.EXPORTS) == names


def test_workspace_query_and_argument_checks(lib):
    from paper_2601_22137_amd import prism as P
    out = ctypes.c_size_t(0)
    q = lambda *a: lib.prism_workspace_bytes(*a, ctypes.byref(out))
    assert q(P.FN_POLAR, 8, 4096, 4096, P.BF16, 5, 32, 0) == P.OK
    per_matrix = 4096 * 4096
    # six bf16 copies of the iterate (hi/lo/gram layout, double buffered) + R (fp32, bf16) + Q (bf16)
    assert 8 * per_matrix * (4 * 2 + 4 + 2 + 2) <= out.value <= 8 * per_matrix * 21
    assert q(P.FN_POLAR, 1, 64, 32, P.F32, 5, 8, 0) == P.OK and out.value > 0
    assert q(P.FN_POLAR, 0, 64, 32, P.F32, 5, 8, 0) == P.OK and out.value == 0      # an empty batch needs nothing
    assert q(P.FN_POLAR, 0, 64, 32, P.F32, 4, 8, 0) == P.EINVAL                     # ... but its arguments are checked
    assert q(P.FN_POLAR, -1, 64, 32, P.F32, 5, 8, 0) == P.EINVAL
    # size limits: 65535 matrices per call, 2^31 - 1 entries per matrix after rounding up to tiles
    assert q(P.FN_POLAR, 65535, 64, 32, P.F32, 5, 8, 0) == P.OK
    assert q(P.FN_POLAR, 65536, 64, 32, P.F32, 5, 8, 0) == P.EUNSUPPORTED
    assert q(P.FN_POLAR, 1, 4_190_000, 500, P.F32, 5, 8, 0) == P.OK
    assert q(P.FN_POLAR, 1, 4_194_400, 500, P.F32, 5, 8, 0) == P.EUNSUPPORTED
    assert q(P.FN_POLAR, 1, 129, 16_000_000, P.BF16, 5, 8, 0) == P.EUNSUPPORTED      # 256 x 16,000,000 once padded
    assert q(P.FN_POLAR, 1, 64, 32, P.F32, 4, 8, 0) == P.EINVAL
    assert q(P.FN_POLAR, 1, 64, 32, P.F32, 5, 65, 0) == P.EINVAL
    assert q(P.FN_POLAR, 1, 64, 32, 7, 5, 8, 0) == P.EINVAL
    assert q(P.FN_SQRT, 1, 64, 32, P.F32, 5, 8, 0) == P.EINVAL          # square root needs m == n
    assert q(P.FN_SQRT, 1, 64, 64, P.BF16, 5, 8, 0) == P.EUNSUPPORTED
    assert q(P.FN_INV_ROOT, 1, 64, 64, P.F32, 3, 8, 0) == P.EINVAL       # root order missing
    assert q(P.FN_INV_ROOT, 1, 64, 64, P.F32, 5, 8, 4) == P.EINVAL       # the update is linear in R
    assert q(P.FN_INV_ROOT, 1, 64, 64, P.F32, 3, 8, 9) == P.EINVAL
    assert q(P.FN_INV_ROOT, 32, 1024, 1024, P.F32, 3, 16, 4) == P.OK
    assert lib.prism_workspace_bytes(P.FN_POLAR, 1, 8, 8, P.F32, 5, 8, 0, None) == P.EINVAL


def test_info_layout_matches_header():
    from paper_2601_22137_amd import prism as P
    assert P.INFO_DTYPE.itemsize == 4 + 4 + 4 * 65 + 4 * 64


def test_profile_arrays_sized_by_the_header_macro_are_accepted(lib):
    """A C caller sizes its arrays with PRISM_PROFILE_KINDS: collect must take exactly that count
    (nothing recorded: no device call is made) and refuse a shorter one."""
    from paper_2601_22137_amd import prism as P
    text = open(os.path.join(ROOT, "include", "prism.h")).read()
    kinds = int(re.search(r"#define\s+PRISM_PROFILE_KINDS\s+(\d+)", text).group(1))
    assert kinds == len(P.PROFILE_KINDS)
    ms = (ctypes.c_double * kinds)()
    cnt = (ctypes.c_longlong * kinds)()
    assert lib.prism_profile_collect(ms, cnt, kinds) == P.OK
    assert lib.prism_profile_collect(ms, cnt, kinds - 1) == P.EINVAL


@pytest.mark.parametrize("m,n", [(8_388_000, 256), (16_777_000, 128), (256, 8_388_000), (4_194_000, 512)])
def test_parts_of_a_gram_product_do_not_add_to_the_size_limit(lib, m, n):
    """A single long matrix close to 2^31 - 1 entries: cutting its Gram product into parts of equal length must not pad it
    past the limit, which counts the sides rounded up to tiles only."""
    from paper_2601_22137_amd import prism as P
    out = ctypes.c_size_t(0)
    assert lib.prism_workspace_bytes(P.FN_POLAR, 1, m, n, P.BF16, 5, 8, 0, ctypes.byref(out)) == P.OK


@pytest.mark.parametrize("m,n,parts", [(58241, 484, 32), (484, 58241, 32), (8065, 300, 7), (65473, 1000, 32), (20000, 200, 19), (9000, 700, 8)])
def test_fp32_gram_product_of_a_tall_matrix_keeps_its_parts(lib, m, n, parts):
    """Whatever the length: the scratch of a single matrix holds at least `parts` partial products of 64-padded order (batches
    of more than eight have none)."""
    from paper_2601_22137_amd import prism as P
    out = ctypes.c_size_t(0)

    def size(batch):
        assert lib.prism_workspace_bytes(P.FN_POLAR, batch, m, n, P.F32, 5, 8, 0, ctypes.byref(out)) == P.OK
        return out.value
    per_matrix = (size(40) - size(20)) // 20
    common = size(20) - 20 * per_matrix
    order = (min(m, n) + 63) // 64 * 64
    assert size(1) - common - per_matrix >= parts * order * order * 4


@pytest.mark.parametrize("batch,m,n,dtype,degree,sketch", [(94, 116, 1, 1, 3, 32), (44, 67, 458, 0, 5, 32), (35, 811, 66, 0, 3, 8), (104, 81, 138, 0, 3, 32)])
def test_largest_batches_of_the_static_entry_point(lib, batch, m, n, dtype, degree, sketch):
    """Batches that leave less than half a matrix of the static array unused: what the fit keeps beside the iterates must
    not take that."""
    from paper_2601_22137_amd import prism as P
    assert P.workspace_bytes(P.FN_POLAR, batch, m, n, dtype, degree, sketch) <= P.STATIC_SCRATCH_BYTES


def test_full_launches_of_order_384_keep_fp32_operands(lib):
    """Up to 1536 tiles of 64 x 64 the products come from planes, which take scratch; from there on they do not."""
    from paper_2601_22137_amd import prism as P
    size = lambda batch: P.workspace_bytes(P.FN_SQRT, batch, 384, 384, P.F32, 5, 16)
    assert size(42) / 42 > 1.5 * size(43) / 43
