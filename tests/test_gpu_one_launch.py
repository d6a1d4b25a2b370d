"""Solves of small systems in one launch (pcg_small.hpp) where the launch does not end as planned: the
library goes on with the launches of the fused form, and status, iterations, residuals and x equal
those of that form (AFSAI_OPT_PCG_FORM = 2) bit for bit.

What the launch meets is set from the host (AFSAI_OPT_PCG_ONE_LAUNCH); every kernel ends by itself.
"""
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
    _same(_solve(af, dA, P, b2, x0, [(af.OPT_PCG_ONE_LAUNCH, 3)], rtol=1e-8), want)
