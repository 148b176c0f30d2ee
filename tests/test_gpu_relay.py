"""The layouts of the cooperative induction give the same bits: those with a wave for the exchange (an
option's blocks on one XCD, or spread over them) against blocks of 1024 threads (launch mode 4),
through prices, exercise indices and FP64 coefficients.  Sizes: one block and one path more or
less, the most blocks of each shape, one option more than the XCDs take, so that near and spread
options share a launch; 1 to 3 steps, where the exchange has no, one and both of its buffers in
use, and dates without a regression (deep out of the money)."""
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


def both(S, call):
    """(result in the default mode, result in mode 4)."""
    out = []
    for mode in (0, 4):
        S.set_lsm_launch(mode)
        try:
            out.append(call())
        finally:
            S.set_lsm_launch(0)
    return out


@pytest.mark.parametrize("paths,steps,K", [(2, 3, 110.0), (1023, 9, 110.0), (1025, 1, 110.0), (1025, 2, 110.0),
                                           (25000, 3, 110.0), (32769, 9, 60.0), (65536, 12, 110.0),
                                           (65537, 7, 110.0), (131072, 9, 90.0), (131073, 5, 110.0),
                                           (262144, 6, 110.0)])
def test_single_option(S, paths, steps, K):
    o = W.option(K=K, payoff=W.AMER_PUT, paths=paths, steps=steps, seed=19)
    (g, tau, beta), (g4, tau4, beta4) = both(S, lambda: S.debug_lsm(o))
    assert g == g4 and np.array_equal(tau, tau4) and np.array_equal(beta, beta4)


@pytest.mark.parametrize("n,paths", [(8, 32768), (9, 32768), (17, 25000), (20, 25000), (30, 25000), (41, 25000),
                                     (9, 65536), (9, 131072), (5, 200000)])
def test_options_sharing_launches(S, n, paths):
    opts = [W.option(K=(110.0, 95.0, 60.0)[i % 3], payoff=(W.AMER_PUT, W.AMER_CALL)[i % 2], paths=paths - i,
                     steps=(11, 2, 8)[i % 3], seed=23, stream=i) for i in range(n)]
    got, want = both(S, lambda: S.price_batch(opts))
    assert got == want


@pytest.mark.parametrize("paths,steps", [(2, 2), (1024, 3), (1025, 1), (25000, 8), (32768, 6), (32769, 6)])
def test_basket(S, paths, steps):
    b = W.basket(3, seed=4, moneyness=1.1, payoff=W.AMER_PUT, paths=paths, steps=steps)
    (g, tau, beta), (g4, tau4, beta4) = both(S, lambda: S.debug_basket_lsm(b))
    assert g == g4 and np.array_equal(tau, tau4) and np.array_equal(beta, beta4)
