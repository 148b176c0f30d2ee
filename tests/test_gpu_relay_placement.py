"""An option whose blocks the plan puts on one XCD, and whose check at run time finds them elsewhere (launch mode 5
makes it find that): it exchanges through memory instead, with the same bits as blocks of 1024 threads
(mode 4), alone and among options that share its launch, on 6 functions and on 10.  A single block never
looks spread; 2, 25 and the most blocks of one poller do."""
import numpy as np
import pytest

from paper_2402_12111_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2402_12111_amd import simr
    simr.library()
    yield simr
    simr.set_lsm_launch(0)


def in_modes(S, call):
    """The results in mode 5, in mode 4 and, after them, in the default mode."""
    out = []
    for mode in (5, 4, 0):
        S.set_lsm_launch(mode)
        try:
            out.append(call())
        finally:
            S.set_lsm_launch(0)
    return out


@pytest.mark.parametrize("paths,steps", [(900, 4), (1025, 2), (25000, 9), (32768, 7), (65536, 5)])
def test_single_option(S, paths, steps):
    o = W.option(K=110.0, payoff=W.AMER_PUT, paths=paths, steps=steps, seed=31)
    (g, tau, beta), *others = in_modes(S, lambda: S.debug_lsm(o))
    for g1, tau1, beta1 in others:
        assert g == g1 and np.array_equal(tau, tau1) and np.array_equal(beta, beta1)


@pytest.mark.parametrize("n,paths", [(3, 25000), (20, 25000), (30, 25000), (9, 65536)])
def test_options_sharing_launches(S, n, paths):
    opts = [W.option(K=(110.0, 95.0)[i % 2], payoff=W.AMER_PUT, paths=paths - i, steps=(9, 3, 6)[i % 3], seed=32,
                     stream=i) for i in range(n)]
    far, other, near = in_modes(S, lambda: S.price_batch(opts))
    assert far == other == near


@pytest.mark.parametrize("paths,steps", [(1025, 3), (25000, 6), (32768, 5)])
def test_basket(S, paths, steps):
    b = W.basket(3, seed=4, moneyness=1.1, payoff=W.AMER_PUT, paths=paths, steps=steps)
    (g, tau, beta), *others = in_modes(S, lambda: S.debug_basket_lsm(b))
    for g1, tau1, beta1 in others:
        assert g == g1 and np.array_equal(tau, tau1) and np.array_equal(beta, beta1)
