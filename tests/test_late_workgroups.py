"""Launches in which one workgroup ends the iteration of a matrix while others of that matrix may only be starting: more
workgroups than the chip holds, and the same call on several streams.

Whether the matrix is done has to be one decision per workgroup.  A wave that looked for itself could leave, and the waves that saw
an older value would go on without what the first one writes for them (the number of their step): the first test reads the sources
for that, so that no kernel has to be run to show it.
"""
import os
import re

import numpy as np
import pytest
import torch

from paper_2601_22137_amd import workloads as W

SEED = W.SKETCH_SEED
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_22137_amd", "csrc")


def _body(name, start):
    """The text of the function that begins with `start`, comments taken out."""
    text = open(os.path.join(CSRC, name)).read()
    assert text.count(start) == 1
    text = text[text.index(start):]
    depth, at = 0, text.index("{")
    for i in range(at, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return re.sub(r"//[^\n]*", "", text[:i + 1])
    raise AssertionError("unbalanced braces")


@pytest.mark.parametrize("name,start", [("fit_device.h", "void fit_and_tiles("), ("flow.hip", "void flow_kernel(")])
def test_done_is_read_by_one_thread(name, start):
    body = _body(name, start)
    assert not re.search(r"if \([^;{]*\bdone\s*\)\s*return", body)
    assert re.search(r"if \(t == 0\) \{[^}]*\bdone\b", body)      # thread 0 looks


@pytest.fixture(scope="module")
def prism():
    from paper_2601_22137_amd import prism as P
    P.lib()
    return P


def _on_streams(call, x, streams=3, rounds=3):
    """call(copy of x) alone, then on several streams at once: the same bits and reports."""
    want = x.clone()
    ref = call(want).read()
    ss = [torch.cuda.Stream() for _ in range(streams)]
    for _ in range(rounds):
        got = [x.clone() for _ in ss]
        torch.cuda.synchronize()
        infos = []
        for s, y in zip(ss, got):
            with torch.cuda.stream(s):
                infos.append(call(y))
        torch.cuda.synchronize()
        for y, info in zip(got, infos):
            rec = info.read()
            assert torch.equal(y.view(torch.int16), want.view(torch.int16))
            assert np.array_equal(rec["iters"], ref["iters"]) and np.array_equal(rec["alpha"], ref["alpha"])
    return ref


@pytest.mark.gpu
@pytest.mark.parametrize("n,batch", [(768, 16), (512, 30)])
def test_square_beside_the_fit(prism, n, batch):
    """Fit and R^2 in one launch: 720 and 780 workgroups on 512 places, matrices that stop at different iterations."""
    A = np.concatenate([W.c3_polar_large(n=n, batch=1, sigma_decades=d) for d in (0.5, 1.0, 2.0)])
    x = torch.from_numpy(np.tile(A, ((batch + 2) // 3, 1, 1))[:batch].copy().view(np.int16)).cuda().view(torch.bfloat16)
    rec = _on_streams(lambda y: prism.polar(y, 5, 20, 16, SEED, 2e-2), x)
    assert len(set(rec["iters"])) > 1 and (rec["status"] == prism.INFO_CONVERGED).all()


@pytest.mark.gpu
@pytest.mark.parametrize("n,batch", [(256, 16), (320, 6), (576, 3)])
def test_all_iterations_in_one_launch(prism, n, batch):
    """Three calls at once of about one workgroup per CU each, matrices that stop at different iterations and one that never starts."""
    rng = np.random.default_rng(n)
    A = rng.standard_normal((batch, n, n))
    A = (A + A.transpose(0, 2, 1)) / 2.0
    for b in range(batch):                          # condition numbers from 1 to 100
        w, v = np.linalg.eigh(A[b])
        A[b] = (v * (np.where(w < 0.0, -1.0, 1.0) * 10.0 ** (-2.0 * b / batch * rng.random(n)))) @ v.T
    A = A.astype(np.float32)
    A[batch - 1] = 0.0
    rec = _on_streams(lambda y: prism.sign(y, 5, 40, 16, SEED, 1e-5), torch.from_numpy(A).cuda())
    assert len(set(rec["iters"][:-1])) > 1 and (rec["status"][:-1] == prism.INFO_CONVERGED).all()
    assert rec["status"][-1] == prism.INFO_ZERO
