"""Greeks where each branch of the reversed variance step takes nearly every step, and where they mix: vol of
vol 0.05 (psi near 1e-4, b^2 near 1e4), 0.3 with a low variance (some steps past psi = 1.5), 1.0 (most
past it, with many exact zeros of V), for both QE schemes, against FP64 forward mode on the same paths.

The bar is the one of the European Greeks, 1e-4 of each Greek's scale max(|g|, per-path deviation), and 1e-3
where FP32 and FP64 can put steps in different branches; the vol-of-vol Greek adds what the forward pass's own
rounding gives: d x / d xi holds rho / xi^2 times the sum of V - E[V], E's rounding and the hardware
roots shift V by up to 2^-23 a step, each times S0 and the largest mean variance."""
import math

import numpy as np
import pytest

import oracle
from paper_2402_12111_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2402_12111_amd import simr
    simr.library()
    return simr


CASES = [
    (dict(xi=0.05, kappa=2.0, theta=0.04, v0=0.05, rho=-0.7), 1e-4),
    (dict(xi=0.3, kappa=1.0, theta=0.02, v0=0.005, rho=-0.5), 1e-3),
    (dict(xi=1.0, kappa=0.8, theta=0.03, v0=0.02, rho=-0.8), 1e-3),
]


@pytest.mark.parametrize("payoff", [0, 1])
@pytest.mark.parametrize("scheme", [0, 2])
@pytest.mark.parametrize("kw,rel", CASES)
def test_each_branch_of_the_reversed_step(S, kw, rel, scheme, payoff):
    o = W.option(K=100.0, payoff=payoff, paths=30001, steps=40, T=1.0, seed=12, **kw)
    gr = S.greeks(o, scheme=scheme)
    p, _, g, gse = oracle.greeks(oracle.Option(**o, scheme=scheme))
    tol = rel * np.maximum(np.abs(g), gse * math.sqrt(o["paths"]))
    vmax = max(kw["theta"], kw["v0"])
    extra = abs(kw["rho"]) / kw["xi"] ** 2 * o["steps"] * o["S0"] * vmax * 2.0 ** -23
    d = np.abs(np.array(gr.grads) - g)
    tol[S.GREEK_NAMES.index("xi")] += extra
    assert (d <= tol).all(), (d / tol, gr.grads, g)
