"""American options whose spills, Gram sums, factors and adjoints run in one launch over all of
them (three or more options in a pass) against single calls, bit for bit: the blocks of every
launch are assigned to options by a search over 64 options at a time, so the list is longer
than that, and its sizes are the edges of the launches -- 2 paths, one date, paths just below and
above a block (256), a Gram chunk (4,096) and an adjoint block, steps in no order."""
import random

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
    return simr


def options(n):
    r = random.Random(5)
    paths = [2, 255, 256, 257, 4095, 4096, 4097, 8191, 25000]
    steps = [1, 2, 3, 17, 40]
    return [W.option(K=r.choice((90.0, 110.0, 60.0)), payoff=r.choice((W.AMER_PUT, W.AMER_CALL)), T=r.choice((0.25, 1.0)),
                     xi=r.choice((0.3, 0.8)), paths=paths[i % len(paths)], steps=r.choice(steps), seed=11, stream=i)
            for i in range(n)]


@pytest.mark.parametrize("n,scheme", [(3, 0), (67, 0), (5, 1), (5, 2), (5, 3)])
def test_options_together_equal_single_calls(S, n, scheme):
    opts = options(n)
    for o, g in zip(opts, S.price_batch(opts, scheme)):
        assert g == S.price(o, scheme), o
    for o, g in zip(opts, S.greeks_batch(opts, scheme)):
        assert g == S.greeks(o, scheme), o


@pytest.mark.parametrize("ck", [8, 32])
def test_greeks_together_at_other_checkpoint_intervals(S, ck):
    """The adjoint block follows the path count and the interval: 131,072 paths take a larger block
    than 4,097, so the group's adjoints go in runs of one block size."""
    opts = [dict(o, paths=p) for o, p in zip(options(5), (4097, 131072, 131072, 257, 262144))]
    for o, g in zip(opts, S.greeks_batch(opts, 0, ck)):
        assert g == S.greeks(o, 0, ck), o
