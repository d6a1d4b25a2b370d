"""Solves of small systems in one launch (pcg_small.hpp) where the launch does not end as planned: the
library goes on with the launches of the fused form, and status, iterations, residuals and x equal
those of that form (AFSAI_OPT_PCG_FORM = 2) bit for bit.

What the launch meets is set from the host (AFSAI_OPT_PCG_ONE_LAUNCH); every kernel ends by itself.
"""
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def af():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    import paper_2010_14175_amd as af

    af.lib()
    return af


PAUSE = 64  # solves that take the ordinary launches after blocks that did not meet


@pytest.fixture(autouse=True)
def _one_launch_again(af):
    """Every test starts where small systems are tried in one launch."""
    A = synth.lap7(1, 1, 1)
    dA = af.DeviceCSR.from_host(A)
    P = af.setup(dA, 1, 1, 1e-2)
    for _ in range(PAUSE + 1):
        with _Forms(af) as forms:
            af.pcg_solve(dA, P, _vec([1.0]))
        if forms.one_launch:
            break
    assert forms() == (1, 0, 0, 0)


def _vec(x):
    import torch

    return torch.from_numpy(np.ascontiguousarray(x, np.float64)).cuda()


def _solve(af, dA, P, b, x0=None, options=(), **kw):
    """(status, iterations, converged, residuals, bits of x) under the options given."""
    try:
        for o, v in options:
            af.set_option(o, v)
        x, i = af.pcg_solve(dA, P, b, x=None if x0 is None else x0.clone(), **kw)
    finally:
        for o, _ in options:
            af.set_option(o, 0)
    return i.status, i.iters, i.converged, i.relres, i.true_relres, x.cpu().numpy().view(np.int64)


class _Forms:
    """What the solves inside the block added to the counts of the forms."""

    def __init__(self, af):
        self.af = af

    def __enter__(self):
        self.before = self.af.pcg_form_counts()
        return self

    def __exit__(self, *a):
        now = self.af.pcg_form_counts()
        self.one_launch, self.unmet, self.fused, self.separate = (
            now[k] - self.before[k] for k in ("one_launch", "unmet", "fused", "separate"))

    def __call__(self):
        return self.one_launch, self.unmet, self.fused, self.separate


def _same(p, q):
    assert p[:5] == q[:5], (p[:5], q[:5])
    np.testing.assert_array_equal(p[5], q[5])


@pytest.mark.parametrize("sides", [(5, 4, 3), (13, 13, 13)])
def test_no_block_on_the_xcd(af, sides):
    """A launch of which no block runs on its XCD writes no result: the record of an earlier solve, which
    the cached host block still holds, is not taken for one."""
    A = synth.lap7(*sides)
    dA = af.DeviceCSR.from_host(A)
    P = af.setup(dA, 5, 1, 1e-2)
    b1, b2 = (_vec(synth.uniform(5 + k, 1, A.n, -1.0, 1.0)) for k in range(2))
    x0 = _vec(synth.uniform(9, 2, A.n))
    want = _solve(af, dA, P, b2, x0, [(af.OPT_PCG_FORM, 2)], rtol=1e-8)
    _solve(af, dA, P, b1, rtol=1e-8)
    with _Forms(af) as forms:
        got = _solve(af, dA, P, b2, x0, [(af.OPT_PCG_ONE_LAUNCH, 3)], rtol=1e-8)
    _same(got, want)
    assert forms() == (1, 1, 1, 0)


@pytest.mark.parametrize("make,kmax,g,want", [
    (lambda: synth.lap7(1, 1, 1), 1, 0, (1, 0, 0, 0)), (lambda: synth.lap7(320, 1, 1), 2, 0, (1, 0, 0, 0)),
    (lambda: synth.lap7(20, 20, 20), 5, 1, (1, 0, 0, 0)), (lambda: synth.lap7(16, 32, 16), 0, 0, (1, 0, 0, 0)),
    (lambda: synth.lap7(25, 25, 26), 5, 0, (1, 0, 0, 0)), (lambda: synth.lap7(26, 26, 26), 5, 0, (0, 0, 1, 0)),
    (lambda: synth.lap7(20, 20, 41), 5, 0, (0, 0, 1, 0)), (lambda: synth.elast27(24, 1.0, 2), 10, 0, (0, 0, 1, 0)),
    (lambda: synth.lap7(99, 100, 101), 5, 0, (0, 0, 0, 1))])
def test_form_of_a_solve(af, make, kmax, g, want):
    """Which form the automatic choice takes on both sides of its limits (one launch up to 16,384 rows of 7
    entries, fused products up to 7 M entries; whole slices, as other layouts order A's rows by length
    and take separate updates), a solve at a time; the option takes the others."""
    A = make()
    dA = af.DeviceCSR.from_host(A)
    P = af.setup(dA, kmax, 1, 1e-2, g_prec=g)
    b = _vec(synth.uniform(5, 1, A.n, -1.0, 1.0))
    with _Forms(af) as forms:
        auto = _solve(af, dA, P, b, rtol=1e-8)
    assert forms() == want
    for form, other in ((1, (0, 0, 0, 1)), (2, (0, 0, 1, 0))):
        with _Forms(af) as forms:
            got = _solve(af, dA, P, b, options=[(af.OPT_PCG_FORM, form)], rtol=1e-8)
        assert forms() == other
        assert got[1] == auto[1]
        np.testing.assert_array_equal(got[5], auto[5])


def test_continued_launch_form(af):
    """A solve of more iterations than a launch takes stays in its form, launch after launch."""
    A = synth.lap7(3000, 1, 1, (1.0, 1e-9, 1e-9))
    dA = af.DeviceCSR.from_host(A)
    P = af.setup(dA, 0, 1, 1e-2)
    b = _vec(synth.uniform(5, 1, A.n))
    with _Forms(af) as forms:
        got = _solve(af, dA, P, b, rtol=1e-10)
    assert forms() == (1, 0, 0, 0) and got[1] > 1024
    _same(got, _solve(af, dA, P, b, options=[(af.OPT_PCG_FORM, 2)], rtol=1e-10))


@pytest.mark.parametrize("sides", [(1, 1, 1), (13, 13, 13), (25, 25, 26)])
def test_blocks_that_do_not_meet(af, sides):
    """A block that never comes to the first barrier (as when other solves hold its place): the others give
    up within milliseconds and the solve runs with the ordinary launches from the given x0."""
    A = synth.lap7(*sides)
    dA = af.DeviceCSR.from_host(A)
    P = af.setup(dA, 5, 1, 1e-2)
    b = _vec(synth.uniform(5, 1, A.n, -1.0, 1.0))
    x0 = _vec(synth.uniform(9, 2, A.n))
    want = _solve(af, dA, P, b, x0, [(af.OPT_PCG_FORM, 2)], rtol=1e-8)
    t0 = time.monotonic()
    with _Forms(af) as forms:
        got = _solve(af, dA, P, b, x0, [(af.OPT_PCG_ONE_LAUNCH, 1)], rtol=1e-8)
    assert time.monotonic() - t0 < 2.0
    assert forms() == (1, 1, 1, 0)
    _same(got, want)


def test_pause_after_blocks_that_did_not_meet(af):
    """Blocks that did not meet once: the next solves do not try, the one after them does."""
    A = synth.lap7(5, 4, 3)
    dA = af.DeviceCSR.from_host(A)
    P = af.setup(dA, 5, 1, 1e-2)
    b = _vec(synth.uniform(5, 1, A.n, -1.0, 1.0))
    want = _solve(af, dA, P, b, options=[(af.OPT_PCG_FORM, 2)], rtol=1e-8)
    _solve(af, dA, P, b, options=[(af.OPT_PCG_ONE_LAUNCH, 1)], rtol=1e-8)
    for k in range(PAUSE + 1):
        with _Forms(af) as forms:
            got = _solve(af, dA, P, b, rtol=1e-8)
        assert forms() == ((1, 0, 0, 0) if k == PAUSE else (0, 0, 1, 0)), k
        _same(got, want)


def test_places_on_the_xcds(af):
    """24 solves from as many threads, on streams of their own, each in flight for milliseconds because an
    arrival is missing: two go to each of the 8 XCDs at most, the others take the ordinary launches."""
    import threading

    import torch

    A = synth.lap7(13, 13, 13)
    dA = af.DeviceCSR.from_host(A)
    b = _vec(synth.uniform(5, 1, A.n, -1.0, 1.0))
    Ps = [af.setup(dA, 5, 1, 1e-2) for _ in range(24)]
    want = _solve(af, dA, Ps[0], b, options=[(af.OPT_PCG_FORM, 2)], rtol=1e-8)
    streams = [torch.cuda.Stream() for _ in Ps]
    xs = [torch.zeros_like(b) for _ in Ps]
    torch.cuda.synchronize()
    out, gate = [None] * len(Ps), threading.Barrier(len(Ps))

    def work(k):
        gate.wait()
        _, i = af.pcg_solve(dA, Ps[k], b, x=xs[k], rtol=1e-8, stream=streams[k])
        out[k] = (i.status, i.iters, i.converged, i.relres, i.true_relres)

    try:
        af.set_option(af.OPT_PCG_ONE_LAUNCH, 1)
        with _Forms(af) as forms:
            ts = [threading.Thread(target=work, args=(k,)) for k in range(len(Ps))]
            for t in ts:
                t.start()
            for t in ts:
                t.join()
    finally:
        af.set_option(af.OPT_PCG_ONE_LAUNCH, 0)
    torch.cuda.synchronize()
    assert 1 <= forms.one_launch <= 16 and forms.unmet == forms.one_launch and forms.fused == len(Ps)
    for k in range(len(Ps)):
        _same(out[k] + (xs[k].cpu().numpy().view(np.int64),), want)


@pytest.mark.parametrize("meets,maxit", [(2, None), (2, 1030), (2, 1025), (4, None)])
def test_blocks_that_do_not_meet_again(af, meets, maxit):
    """A block missing in the second launch of a solve, or coming when the others have given up (it must not
    pass the barrier and step its part of x): the launches of the fused form go on from iteration 1,024, to the
    end or to a maxit just behind it."""
    A = synth.lap7(3000, 1, 1, (1.0, 1e-9, 1e-9))
    dA = af.DeviceCSR.from_host(A)
    P = af.setup(dA, 0, 1, 1e-2)
    b = _vec(synth.uniform(5, 1, A.n))
    x0 = _vec(synth.uniform(9, 2, A.n))
    want = _solve(af, dA, P, b, x0, [(af.OPT_PCG_FORM, 2)], rtol=1e-10, maxit=maxit)
    assert want[1] > 1024
    with _Forms(af) as forms:
        got = _solve(af, dA, P, b, x0, [(af.OPT_PCG_ONE_LAUNCH, meets)], rtol=1e-10, maxit=maxit)
    assert forms() == (1, 1, 1, 0)
    _same(got, want)
