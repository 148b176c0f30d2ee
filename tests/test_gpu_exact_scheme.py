"""The Broadie-Kaya step, whose waves share the frequencies of their 64 paths' integrated-variance
laws, against the oracle on the same uniforms at the edges of that sharing: waves with 1 to 63
paths past the last one, a single path pair, laws of few and of the most frequencies (small and
large xi), the deterministic law (xi = 0), paths that start at v = 0 and |rho| = 1.  The bounds are
those of the FP32 state between steps: rounding of x and v once per step."""
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


@pytest.mark.parametrize("kw", [dict(paths=2, steps=1), dict(paths=65, steps=2), dict(paths=257, steps=3),
                                dict(paths=191, steps=2, xi=0.1), dict(paths=130, steps=1, xi=0.8),
                                dict(paths=130, steps=3, xi=0.0), dict(paths=64, steps=2, v0=0.0, rho=-1.0)])
def test_paths_match_the_oracle(S, kw):
    o = W.option(seed=17, **kw)
    x, v, _ = S.debug_paths(o, 4)
    rx, rv, _ = oracle.simulate(oracle.Option(**o, scheme=4))
    assert np.median(np.abs(x - rx)) < 1e-6 and np.abs(x - rx).max() < 1e-4, kw
    assert np.abs(v - rv).max() < 1e-5, kw


@pytest.mark.parametrize("n", [1, 3])
def test_write_out_of_ragged_paths(S, n):
    """American options (the write-out kernels, one option or three in a launch): the exercise
    policy valued on the oracle's paths."""
    opts = [W.option(K=110.0, payoff=W.AMER_PUT, paths=p, steps=2, seed=3, stream=i)
            for i, p in enumerate((700, 1025, 2000)[:n])]
    for o, g in zip(opts, S.price_batch(opts, 4)):
        one, tau, _ = S.debug_lsm(o, 4)
        assert (g.price, g.std_err) == (one.price, one.std_err)
        value = oracle.stopped_values(oracle.Option(**o, scheme=4), tau).mean()
        assert abs(g.price - max(value, 10.0)) <= 1e-4 * o["S0"]
