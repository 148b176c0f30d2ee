"""Which basket kernel runs, by assets, paths and steps (on 256 CUs), and that each is right there: one path per lane
from 524,288 paths on, or fewer with few steps, and for American baskets of more than 8 assets from 131,072;
one or two assets per lane otherwise, the basket summed in asset order from 131,072 paths on and for up to
8 assets.  Prices, Greeks and exercise policies against the oracle; terminal values of the two kernels on
both sides of each limit bit for bit."""
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


def b0(b):
    return float(np.dot(b["w"], b["S0"]))


def check_greeks(S, b):
    """Deltas and cross-gammas: pathwise FP32 rounding of about 1e-6 of the sample's scale."""
    g = S.basket_greeks(b)
    price, _, delta, delta_se, gamma, gamma_se = oracle.basket_greeks(oracle.Basket(**b))
    scale = np.sqrt(b["paths"])
    assert abs(g.price - price) <= 1e-4 * b0(b)
    assert np.all(np.abs(np.array(g.delta) - delta) <= 1e-4 * np.maximum(np.abs(delta), scale * delta_se))
    assert np.all(np.abs(np.array(g.gamma) - gamma) <= 1e-4 * np.maximum(np.abs(gamma), scale * gamma_se))


@pytest.mark.parametrize("d", [4, 8, 12, 20])
def test_greeks_one_path_per_lane(S, d):
    check_greeks(S, W.basket(d, seed=d, paths=1 << 19, steps=2))


@pytest.mark.parametrize("d", [12, 20])
def test_greeks_of_many_assets_summed_in_asset_order(S, d):
    check_greeks(S, W.basket(d, seed=d, paths=140000, steps=12))


@pytest.mark.parametrize("d", [12, 20])
def test_write_out_of_many_assets_one_path_per_lane(S, d):
    b = W.basket(d, seed=d, moneyness=1.1, payoff=W.AMER_PUT, paths=140000, steps=4)
    g, tau, _ = S.debug_basket_lsm(b)
    value = oracle.basket_stopped_values(oracle.Basket(**b), tau).mean()
    assert abs(g.price - max(value, 0.1 * b0(b))) <= 1e-4 * b0(b)


@pytest.mark.parametrize("d,paths,steps", [(5, 70000, (1, 5, 6)), (5, 140000, (11, 12)), (20, 140000, (11, 12)),
                                           (19, 140000, (17, 18)), (16, 270000, (24, 25)), (9, 270000, (84, 85)),
                                           (12, 1 << 19, (16,))])
def test_terminal_values_on_both_sides_of_each_limit(S, d, paths, steps):
    """As few as 300 paths run one or two assets per lane whatever the steps; the payoffs differ by the order of the
    basket sum only: d FP32 additions."""
    for n in steps:
        b = W.basket(d, paths=paths, steps=n)
        x, v, p = S.debug_basket_paths(b)
        xs, vs, ps = S.debug_basket_paths(dict(b, paths=300))
        assert np.array_equal(x[:300], xs) and np.array_equal(v[:300], vs), n
        np.testing.assert_allclose(p[:300], ps, rtol=0, atol=d * 2.0 ** -23 * b0(b))
        assert abs(S.basket_price(b).price - p.astype(np.float64).mean()) <= 1e-6 * b0(b)


@pytest.mark.parametrize("d,paths,steps", [(5, 70000, (2, 3)), (12, 140000, (5, 6)), (20, 140000, (11, 12)),
                                           (9, 270000, (17, 18)), (20, 270000, (11, 12))])
def test_greeks_on_both_sides_of_each_limit(S, d, paths, steps):
    for n in steps:
        check_greeks(S, W.basket(d, seed=d, paths=paths, steps=n))
