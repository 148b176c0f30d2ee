"""Greeks from an initial variance so small that the variance of the first log-price increment is subnormal in
FP32.  The hardware's square root of a subnormal is 0, so the step's derivative there is 0 too, not the
reciprocal root's infinity: every Greek is finite, and all but d/dv0 (which FP64 still resolves, near 1e17)
meet FP64 forward mode at the bar of paths that mix the variance step's branches, 1e-3 of each Greek's
scale max(|g|, per-path deviation).  Steps of both signs of the guard: v0 from the subnormals to 1e-36.  (A
path's own d/dv0 is near 1e19 at the normal end, where its FP32 square, and so that one standard error,
overflows with any form of the derivative: it is not asked for.)"""
import math

import numpy as np
import pytest

import oracle
from paper_2402_12111_amd import workloads as W

pytestmark = pytest.mark.gpu

NAMES = ("S0", "v0", "theta", "r", "kappa", "xi", "rho")
REST = [i for i, name in enumerate(NAMES) if name != "v0"]
V0 = [1e-45, 1e-40, 1e-38, 1e-37, 1e-36]


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2402_12111_amd import simr
    simr.library()
    return simr


@pytest.mark.parametrize("v0", V0)
@pytest.mark.parametrize("scheme", [0, 2, 3])
def test_european(S, v0, scheme):
    o = W.option(v0=v0, xi=0.5, paths=6001, steps=20, seed=19)
    gr = S.greeks(o, scheme=scheme)
    ext = S.greeks_ext(o, scheme=scheme)
    _, _, g, gse = oracle.greeks(oracle.Option(**o, scheme=scheme))
    assert np.isfinite(gr.grads).all() and np.isfinite(np.array(gr.grad_se)[REST]).all(), gr.grads
    assert np.isfinite(ext.grads).all() and np.isfinite(np.array(ext.grad_se)[REST]).all(), ext.grads
    tol = 1e-3 * np.maximum(np.abs(g), gse * math.sqrt(o["paths"]))
    d = np.abs(np.array(gr.grads) - g)
    assert (d[REST] <= tol[REST]).all(), (d / tol, gr.grads, g)


@pytest.mark.parametrize("scheme", [0, 2, 3])
def test_american_alone_and_in_a_batch(S, scheme):
    opts = [W.option(v0=v0, xi=0.5, K=105.0, payoff=W.AMER_PUT, paths=4099, steps=17, seed=20, stream=i)
            for i, v0 in enumerate(V0)]
    batch = S.greeks_batch(opts, scheme)
    for o, b in zip(opts, batch):
        assert np.isfinite(b.grads).all() and np.isfinite(np.array(b.grad_se)[REST]).all(), (o["v0"], b.grads)
        one = S.greeks(o, scheme)
        np.testing.assert_array_equal([one.price, one.std_err] + one.grads + one.grad_se,
                                      [b.price, b.std_err] + b.grads + b.grad_se)
