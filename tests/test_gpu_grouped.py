"""The grouped call (one library call over groups of different shapes, internal fork / join
streams): every group must come out exactly as from its own single-group call, and against the
oracle to the usual bars; the optimizer-side helpers are thin wrappers around it."""
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


def _rel(x, ref):
    return np.linalg.norm(np.asarray(x, dtype=np.float64) - ref) / np.linalg.norm(ref)


def _bf16(bits):
    return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)


def test_grouped_polar_equals_single_calls_and_oracle(prism):
    """Muon-shaped groups at a quarter of the size (192x192, 192x768, 768x192, 192x576), six groups
    so that internal streams are reused, twice in a row."""
    bits = [W.c2_muon_group(i % 4, batch=3 + i, scale=4, data_seed=1002 + 10 * (i // 4)) for i in range(6)]
    single = []
    for b in bits:
        x = _bf16(b.copy())
        prism.polar(x, 5, 5, 16, SEED, 0.0, flags=prism.FLAG_BF16_PLAIN_ITERATE)
        single.append(x)
    for rep in range(3):   # the last one with every kernel on the caller's stream
        xs = [_bf16(b.copy()) for b in bits]
        flags = prism.FLAG_BF16_PLAIN_ITERATE | (prism.FLAG_SINGLE_STREAM if rep == 2 else 0)
        _, infos = prism.run_grouped(prism.FN_POLAR, xs, 5, 5, 16, SEED, 0.0, flags=flags)
        torch.cuda.synchronize()
        for g, (x, ref) in enumerate(zip(xs, single)):
            assert torch.equal(x.view(torch.int16), ref.view(torch.int16)), g
            rec = infos[g].read()
            assert np.all(rec["iters"] == 5)
    out0 = W.from_bf16_bits(xs[1][0].view(torch.int16).cpu().numpy().view(np.uint16))
    ref, _ = O.polar(W.from_bf16_bits(bits[1][0]), 5, 5, 16, SEED, 0.0)
    assert _rel(out0, ref) <= 2e-2


def test_grouped_polar_in_parts_on_internal_streams(prism):
    """Batches that are multiples of four: the one launch sequence over all shapes is issued per
    quarter of every group on internal streams (split iterate here, and a tolerance, so that the
    per-matrix stop flags matter).  Same bits as the single calls, reports in the caller's arrays."""
    bits = [W.c2_muon_group(i, batch=8, scale=4, data_seed=1500 + i) for i in range(4)]
    single, single_info = [], []
    for b in bits:
        x = _bf16(b.copy())
        single_info.append(prism.polar(x, 5, 30, 16, SEED, 2e-2).read())
        single.append(x)
    xs = [_bf16(b.copy()) for b in bits]
    _, infos = prism.run_grouped(prism.FN_POLAR, xs, 5, 30, 16, SEED, 2e-2)
    torch.cuda.synchronize()
    for g in range(4):
        assert torch.equal(xs[g].view(torch.int16), single[g].view(torch.int16)), g
        rec = infos[g].read()
        assert np.array_equal(rec["iters"], single_info[g]["iters"]) and np.array_equal(rec["alpha"], single_info[g]["alpha"])
        assert np.array_equal(rec["status"], single_info[g]["status"])
    out0 = W.from_bf16_bits(xs[2][5].view(torch.int16).cpu().numpy().view(np.uint16))
    ref, oinfo = O.polar(W.from_bf16_bits(bits[2][5]), 5, 30, 16, SEED, 2e-2)
    assert _rel(out0, ref) <= 2e-2 and infos[2].read()[5]["iters"] == oinfo["iters"]


def test_grouped_fp32_polar_with_small_and_general_groups(prism):
    """fp32 groups to tolerance: three whose padded iterate is 64 x 64 (they run in the one-workgroup
    kernel) beside one that takes the general path; same bits as the single calls, oracle parity."""
    shapes = [(5, 64, 32), (3, 200, 72), (2, 40, 24), (4, 48, 64)]
    As = [np.concatenate([W.c1_polar_small(m=m, n=n, data_seed=2100 + 10 * g + i) for i in range(b)])
          for g, (b, m, n) in enumerate(shapes)]
    single = []
    for A in As:
        x = torch.from_numpy(A.copy()).cuda()
        prism.polar(x, 5, 30, 8, SEED, 1e-6)
        single.append(x)
    xs = [torch.from_numpy(A.copy()).cuda() for A in As]
    _, infos = prism.run_grouped(prism.FN_POLAR, xs, 5, 30, 8, SEED, 1e-6)
    torch.cuda.synchronize()
    for g, (x, ref) in enumerate(zip(xs, single)):
        assert torch.equal(x, ref), g
        rec = infos[g].read()
        want, oinfo = O.polar(As[g][0], 5, 30, 8, SEED, 1e-6)
        assert _rel(x[0].cpu().numpy(), want) <= 1e-5
        assert rec[0]["iters"] == oinfo["iters"] and rec[0]["status"] == prism.INFO_CONVERGED


def test_grouped_call_replays_from_a_hip_graph(prism):
    """The fork onto the internal streams and the join back are event waits, so a grouped call
    captures from the caller's stream like a single one: every replay, with eager work and
    synchronisations in between, must give the bits of the eager call."""
    bits = [W.c2_muon_group(i, batch=4, scale=4) for i in range(4)]
    src = [_bf16(b.copy()) for b in bits]
    eager = [t.clone() for t in src]
    _, h = prism.run_grouped(prism.FN_POLAR, eager, 5, 5, 16, SEED, 0.0, flags=prism.FLAG_BF16_PLAIN_ITERATE)
    torch.cuda.synchronize()
    alpha_eager = [r.read()["alpha"].copy() for r in h]
    xs = [t.clone() for t in src]
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        prism.run_grouped(prism.FN_POLAR, xs, 5, 5, 16, SEED, 0.0, flags=prism.FLAG_BF16_PLAIN_ITERATE)   # warm-up
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            _, handles = prism.run_grouped(prism.FN_POLAR, xs, 5, 5, 16, SEED, 0.0, flags=prism.FLAG_BF16_PLAIN_ITERATE)
        for _ in range(3):
            for x, s0 in zip(xs, src):
                x.copy_(s0)                                      # eager work between the replays
            graph.replay()
            side.synchronize()
            for g in range(4):
                assert torch.equal(xs[g].view(torch.int16), eager[g].view(torch.int16)), g
                assert np.array_equal(handles[g].read()["alpha"], alpha_eager[g])


def test_grouped_inverse_root_and_sqrt(prism):
    A1, A2 = W.c4_shampoo_spd(n=128, batch=2), W.c4_shampoo_spd(n=200, batch=3, data_seed=77)
    xs = [torch.from_numpy(A1.copy()).cuda(), torch.from_numpy(A2.copy()).cuda()]
    _, infos = prism.run_grouped(prism.FN_INV_ROOT, xs, 3, 40, 16, SEED, 1e-5, root_p=4)
    for A, x, h in zip((A1, A2), xs, infos):
        rec = h.read()
        for i in range(A.shape[0]):
            ref, oinfo = O.inv_root(A[i], 4, 40, 16, SEED, 1e-5)
            assert _rel(x[i].cpu().numpy(), ref) <= 1e-5
            assert rec[i]["iters"] == oinfo["iters"]
    S1, S2 = W.c5_wishart_spd(n=128, batch=2), W.c5_wishart_spd(n=192, batch=1, data_seed=5)
    xs = [torch.from_numpy(S1.copy()).cuda(), torch.from_numpy(S2.copy()).cuda()]
    invs, infos = prism.run_grouped(prism.FN_SQRT_NEWTON, xs, 3, 30, 1, SEED, 1e-5)
    for S, x, inv in zip((S1, S2), xs, invs):
        rx, ry, _ = O.sqrt_db_newton(S[0], 30, 1e-5)
        assert _rel(x[0].cpu().numpy(), rx) <= 1e-5 and _rel(inv[0].cpu().numpy(), ry) <= 1e-5


def test_grouped_argument_errors(prism):
    x = torch.zeros((1, 16, 16), dtype=torch.float32, device="cuda")
    with pytest.raises(prism.PrismError):
        prism.run_grouped(prism.FN_POLAR, [x, torch.zeros((1, 8, 8), dtype=torch.float32, device="cuda")], 4, 3, 0, SEED, 0.0)


def test_optimizer_helpers(prism):
    from paper_2601_22137_amd import optim
    rng = np.random.default_rng(3)
    shapes = [(96, 64), (64, 96), (96, 64), (128, 128), (64, 96)]
    grads = [torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda() for s in shapes]
    outs = optim.muon_orthogonalize(grads, degree=5, iters=8, sketch_dim=8)
    for g, o in zip(grads, outs):
        assert o.shape == g.shape
        ref, _ = O.polar(g.cpu().numpy(), 5, 8, 8, SEED, 0.0)
        assert _rel(o.cpu().numpy(), ref) <= 1e-5
    stats = [torch.from_numpy(W.c4_shampoo_spd(n=n, batch=1, data_seed=90 + n)[0]).cuda() for n in (64, 128, 64)]
    roots, iters = optim.shampoo_inverse_roots(stats, root_p=4)
    for s, r, it in zip(stats, roots, iters):
        ref, oinfo = O.inv_root(s.cpu().numpy(), 4, 40, 16, SEED, 1e-5)
        assert _rel(r.cpu().numpy(), ref) <= 1e-5 and it == oinfo["iters"]


def test_shared_gpu_flag_is_a_scheduling_hint(prism):
    """PRISM_FLAG_SHARED_GPU changes tile sizes only: at a size where it does (Gram dimension 768,
    a multiple of 256) a single call with the flag gives the bits of the grouped call, and both stay
    within the rounding of the unflagged call."""
    bits = [W.c2_muon_group(0, batch=2), W.c2_muon_group(3, batch=2)]
    plain = prism.FLAG_BF16_PLAIN_ITERATE
    xs = [_bf16(b.copy()) for b in bits]
    prism.run_grouped(prism.FN_POLAR, xs, 5, 5, 16, SEED, 0.0, flags=plain)
    torch.cuda.synchronize()
    for g, b in enumerate(bits):
        hinted = _bf16(b.copy())
        prism.polar(hinted, 5, 5, 16, SEED, 0.0, flags=plain | prism.FLAG_SHARED_GPU)
        assert torch.equal(hinted.view(torch.int16), xs[g].view(torch.int16))
        unhinted = _bf16(b.copy())
        prism.polar(unhinted, 5, 5, 16, SEED, 0.0, flags=plain)
        d = (unhinted.float() - hinted.float()).norm() / hinted.float().norm()
        assert float(d) <= 2e-2


def test_calls_from_two_host_threads(prism):
    """Two host threads, each with a stream of its own, issue calls of different shapes at the same
    time (ctypes releases the GIL during a call): workspaces are per stream and the shared state of
    the library is locked, so both get the bits of the same calls made one after the other."""
    import threading
    jobs = [(np.concatenate([W.c1_polar_small(m=200, n=72, data_seed=2500 + i) for i in range(3)]), 5),
            (np.concatenate([W.c1_polar_small(m=64, n=32, data_seed=2600 + i) for i in range(6)]), 3)]
    want = []
    for A, deg in jobs:
        x = torch.from_numpy(A.copy()).cuda()
        prism.polar(x, deg, 30, 8, SEED, 1e-6)
        want.append(x)
    torch.cuda.synchronize()
    got, errors = [None, None], []

    def work(j):
        try:
            A, deg = jobs[j]
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                for _ in range(20):
                    x = torch.from_numpy(A.copy()).cuda()
                    prism.polar(x, deg, 30, 8, SEED, 1e-6)
                st.synchronize()
            got[j] = x
        except Exception as e:          # noqa: BLE001 - reported by the assertion below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(j,)) for j in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for j in range(2):
        assert torch.equal(got[j], want[j]), j


def _ways(prism, run, grouped, make, ws_bytes):
    """The same matrices through a plain call (run as two halves), on one stream, in a caller's workspace and as a group beside
    another one: outputs (as integers) and reports."""
    res = []
    for kind in ("plain", "single", "workspace", "grouped"):
        x = make()
        if kind == "grouped":
            rec = grouped(x)
        elif kind == "workspace":
            rec = run(x, 0, torch.empty(ws_bytes, dtype=torch.uint8, device="cuda"))
        else:
            rec = run(x, prism.FLAG_SINGLE_STREAM if kind == "single" else 0, None)
        torch.cuda.synchronize()
        res.append((kind, x.view(torch.int16 if x.dtype == torch.bfloat16 else torch.int32).cpu(), rec.read()))
    return res


@pytest.mark.parametrize("n,batch,sketch", [(2048, 8, 32), (1536, 8, 16), (1300, 12, 32), (1100, 16, 16)])
def test_same_bits_however_a_batch_is_enqueued_bf16(prism, n, batch, sketch):
    torch.manual_seed(n)
    a = torch.randn(batch, n, n, device="cuda").to(torch.bfloat16)
    other = torch.randn(batch, 2 * n, n, device="cuda").to(torch.bfloat16)
    res = _ways(prism, lambda x, flags, ws: prism.polar(x, 5, 9, sketch, SEED, 0.0, flags=flags, workspace=ws),
                lambda x: prism.run_grouped(prism.FN_POLAR, [x, other.clone()], 5, 9, sketch, SEED, 0.0)[1][0], a.clone,
                prism.workspace_bytes(prism.FN_POLAR, batch, n, n, prism.BF16, 5, sketch))
    for kind, out, rec in res[1:]:
        assert torch.equal(out, res[0][1]), kind
        assert np.array_equal(rec["alpha"], res[0][2]["alpha"]), kind


@pytest.mark.parametrize("n,batch,sketch", [(2048, 8, 16), (1024, 8, 16), (1024, 16, 8), (1500, 10, 32)])
def test_same_bits_however_a_batch_is_enqueued_fp32(prism, n, batch, sketch):
    """Residuals too: their partial sums follow the tiles of the product.  (Updates enough for coefficients inside their
    interval, here and above: at its end all kernels agree.)"""
    torch.manual_seed(n)
    a = torch.randn(batch, n, n, device="cuda")
    a = a @ a.transpose(1, 2).contiguous() / n + 0.01 * torch.eye(n, device="cuda")
    other = torch.eye(64, device="cuda").repeat(1, 1, 1)
    for fn, call, args in ((prism.FN_SIGN, lambda x, f, ws: prism.sign(x, 5, 12, sketch, SEED, 0.0, flags=f, workspace=ws), (5, 12, sketch)),
                           (prism.FN_INV_ROOT, lambda x, f, ws: prism.inv_root(x, 2, 8, sketch, SEED, 0.0, flags=f, workspace=ws), (3, 8, sketch))):
        p = 2 if fn == prism.FN_INV_ROOT else 0
        res = _ways(prism, call, lambda x: prism.run_grouped(fn, [x, other.clone()], *args, SEED, 0.0, root_p=p)[1][0], a.clone,
                    prism.workspace_bytes(fn, batch, n, n, prism.F32, args[0], sketch, p))
        for kind, out, rec in res[1:]:
            assert torch.equal(out, res[0][1]), (fn, kind)
            assert rec.tobytes() == res[0][2].tobytes(), (fn, kind)


@pytest.mark.parametrize("w", [128, 200, 256, 512, 640])
def test_grouped_layer_with_split_gram_products(prism, w):
    """One layer: the long shapes cut their Gram product into parts, the square one goes with them as one part.  Bits of the
    single calls."""
    torch.manual_seed(w)
    src = [torch.randn(1, m, n, device="cuda").to(torch.bfloat16) for m, n in ((w, w), (w, 4 * w), (4 * w, w), (w, 9 * w), (12 * w, w))]
    for flags in (0, prism.FLAG_BF16_PLAIN_ITERATE):
        xs, ys = [t.clone() for t in src], [t.clone() for t in src]
        infos = prism.run_grouped(prism.FN_POLAR, xs, 5, 8, 16, SEED, 0.0, flags=flags)[1]
        for g, y in enumerate(ys):
            rec = prism.polar(y, 5, 8, 16, SEED, 0.0, flags=flags).read()
            assert torch.equal(xs[g].view(torch.int16), y.view(torch.int16)), (flags, g)
            assert np.array_equal(rec["alpha"], infos[g].read()["alpha"]), (flags, g)


@pytest.mark.parametrize("w,counts", [(768, (24, 8, 4)), (600, (25, 3, 30)), (1024, (3, 17, 2)), (1024, (20, 24))])
@pytest.mark.parametrize("plain", [False, True])
def test_grouped_shapes_on_both_sides_of_the_fused_fit(prism, w, counts, plain):
    """Shapes in unequal numbers: the fit of the few runs in one launch, that of the many in chain kernels, moments and solve.
    Bits of the single calls, reports in place."""
    flags = prism.FLAG_BF16_PLAIN_ITERATE if plain else 0
    torch.manual_seed(w + sum(counts))
    src = [torch.randn(b, m, n, device="cuda").to(torch.bfloat16) for b, (m, n) in zip(counts, ((w, w), (w, 2 * w), (2 * w, w)))]
    for tol, iters in ((0.0, 9), (1e-2, 20)):
        xs, ys = [t.clone() for t in src], [t.clone() for t in src]
        infos = prism.run_grouped(prism.FN_POLAR, xs, 5, iters, 16, SEED, tol, flags=flags)[1]
        for g, y in enumerate(ys):
            rec, got = prism.polar(y, 5, iters, 16, SEED, tol, flags=flags).read(), infos[g].read()
            assert torch.equal(xs[g].view(torch.int16), y.view(torch.int16)), (tol, g)
            assert np.array_equal(rec["alpha"], got["alpha"]) and np.array_equal(rec["iters"], got["iters"]), (tol, g)


@pytest.mark.parametrize("shapes,odd", [([(64, 96)], False), ([(128, 128), (128, 512), (512, 128)], False), ([(768, 768), (768, 3072)] * 16, False),
                                        ([(128, 132), (300, 128)], False), ([(256, 256), (256, 512)], True), ([(32, 64)] * 90 + [(64, 32)] * 90, False)])
def test_sources_where_they_are(prism, shapes, odd):
    """A list of matrices read from their own addresses: the bits of the stacked call, inputs untouched; a zero and a non-finite matrix
    come back as they are.  odd: addresses that no vector load takes."""
    rng = np.random.default_rng(len(shapes))
    mats = []
    for i, (m, n) in enumerate(shapes):
        buf = torch.from_numpy(rng.standard_normal(m * n + 1).astype(np.float32)).cuda().to(torch.bfloat16)
        mats.append((buf[1:] if odd and i == 0 else buf[:-1]).view(m, n))
    mats[-1].zero_()
    if len(mats) > 2:
        mats[1][0, 0] = float("inf")
    before = [t.clone() for t in mats]
    groups = {}
    for t in mats:
        groups.setdefault(tuple(t.shape), []).append(t)
    stacked = [torch.stack(ts) for ts in groups.values()]
    plain = prism.FLAG_BF16_PLAIN_ITERATE
    _, ref = prism.run_grouped(prism.FN_POLAR, stacked, 5, 5, 16, SEED, 0.0, flags=plain)
    out = [torch.full_like(s, 7.0) for s in stacked]
    _, got = prism.run_grouped(prism.FN_POLAR, out, 5, 5, 16, SEED, 0.0, flags=plain, sources=list(groups.values()))
    for s, o, a, b in zip(stacked, out, ref, got):
        assert torch.equal(s.view(torch.int16), o.view(torch.int16))
        assert np.array_equal(a.read()["status"], b.read()["status"])
    for t, b in zip(mats, before):
        assert torch.equal(t.view(torch.int16), b.view(torch.int16))


def test_calls_in_parts_from_other_streams(prism):
    """Grouped calls in quarters, mixed groups, and a batch that the library halves, from streams that never made such a call: nothing is
    allocated, calls that follow each other on different streams without a wait keep out of each other's workspaces, and the
    first call on a stream may be the captured one."""
    plain = prism.FLAG_BF16_PLAIN_ITERATE
    quarters = [_bf16(W.c2_muon_group(i, batch=8, scale=4)) for i in range(4)]
    mixed = [torch.from_numpy(W.c4_shampoo_spd(n=n, batch=1, data_seed=n)).cuda() for n in (40, 130, 200, 300, 80)]
    halves = [_bf16(np.repeat(W.c3_polar_large(n=1024, batch=1, sigma_decades=1.0), 8, axis=0))]
    kinds = [(quarters, lambda xs: prism.run_grouped(prism.FN_POLAR, xs, 5, 5, 16, SEED, 0.0, flags=plain)),
             (mixed, lambda xs: prism.run_grouped(prism.FN_INV_ROOT, xs, 3, 40, 16, SEED, 1e-5, root_p=4)),
             (halves, lambda xs: prism.polar(xs[0], 5, 5, 16, SEED, 0.0))]
    for src, call in kinds:
        want = [t.clone() for t in src]
        call(want)
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in range(3)]
        got = [[t.clone() for t in src] for _ in streams]
        call([t.clone() for t in src])              # torch's allocator has the reports' memory
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        for s, xs in zip(streams, got):
            with torch.cuda.stream(s):
                call(xs)
        torch.cuda.synchronize()
        assert free - torch.cuda.mem_get_info()[0] < (16 << 20)     # (torch: a segment of 2 MiB per stream for the reports)
        for xs in got:
            for x, w in zip(xs, want):
                assert torch.equal(x.view(torch.int16), w.view(torch.int16))
        side, graph, xs = torch.cuda.Stream(), torch.cuda.CUDAGraph(), [t.clone() for t in src]
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            call(xs)
        for _ in range(3):
            with torch.cuda.stream(side):
                for x, t in zip(xs, src):
                    x.copy_(t)
                graph.replay()
                side.synchronize()
            call([t.clone() for t in src])          # eager work between the replays
            torch.cuda.synchronize()
            for x, w in zip(xs, want):
                assert torch.equal(x.view(torch.int16), w.view(torch.int16))


def test_sources_of_a_refused_call_are_not_copied(prism):
    """The results' arrays of a call that is refused, for its arguments or for one of its groups, keep what they hold."""
    src = [torch.full((40, 30), 2.0, device="cuda"), torch.full((50, 50), 3.0, device="cuda")]
    out = [torch.full((1, 40, 30), 7.0, device="cuda"), torch.full((1, 50, 50), 7.0, device="cuda")]
    sources = [[t] for t in src]
    for fn, args, kw in [(prism.FN_POLAR, (5, 65, 8, SEED, 1e-5), {}), (prism.FN_POLAR, (5, 10, 8, SEED, float("nan")), {}),
                         (prism.FN_POLAR, (5, 10, 8, SEED, 1e-5), {"warm_iters": -1}), (prism.FN_POLAR, (4, 10, 8, SEED, 1e-5), {}),
                         (prism.FN_INV_ROOT, (3, 10, 8, SEED, 1e-5), {"root_p": 2})]:
        for order in ((0, 1), (1, 0)):              # inverse root: the second or the first group is not square
            with pytest.raises(prism.PrismError):
                prism.run_grouped(fn, [out[i] for i in order], *args, sources=[sources[i] for i in order], **kw)
            torch.cuda.synchronize()
            assert bool((out[0] == 7.0).all()) and bool((out[1] == 7.0).all())


def test_negative_views_among_the_gradients(prism):
    """A tensor whose values are those in memory with the other sign (a lazy negation) is not read where it is."""
    from paper_2601_22137_amd import optim
    rng = np.random.default_rng(11)
    grads = [torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda().to(torch.bfloat16) for s in ((96, 64), (64, 96), (96, 64))]
    want = optim.muon_orthogonalize([grads[0], -grads[1], grads[2]])
    got = optim.muon_orthogonalize([grads[0], torch._neg_view(grads[1]), grads[2]])
    for w, o in zip(want, got):
        assert torch.equal(w, o)
