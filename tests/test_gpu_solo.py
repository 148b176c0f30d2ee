"""One small European option (variates drawn by waves of their own) against the batch kernel, bit for bit:
the same paths and the same order of the sums, at the edges of its chunks of 8 steps, of a
wave and of a tile, for every tile shape and scheme that has the kernel, and on both entry points."""
import ctypes

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


def bits(r):
    return r.price, r.std_err


@pytest.mark.parametrize("tile", [(128, 1), (128, 4), (256, 1), (256, 2)])
@pytest.mark.parametrize("scheme", [0, 1, 2, 3])
def test_equals_the_batch_kernel(S, scheme, tile):
    S.price(W.option(paths=64, steps=1), scheme)  # tunes the scheme, so its tile can be put back
    old = S.get_tile()
    try:
        S.set_tile(*tile)
        for paths, steps in ((2, 1), (64, 7), (65, 8), (1023, 9), (1025, 16), (5000, 17), (131072, 3), (131073, 3)):
            o = W.option(K=101.0, payoff=steps % 2, paths=paths, steps=steps, seed=paths)
            want = bits(S.price_batch([o, o], scheme)[1])
            assert bits(S.price(o, scheme)) == want, (paths, steps)
            assert bits(S.price_noalloc(o, scheme)) == want, (paths, steps)
    finally:
        S.set_tile(*old)


@pytest.mark.parametrize("ck", [16, 32])
@pytest.mark.parametrize("scheme", [0, 1, 2, 3])
def test_greeks_on_its_checkpoints(S, scheme, ck):
    """The Greeks' price is the call's alone, and their values do not depend on where the checkpoints
    lie but for the order of the sums (1e-5 of each Greek's scale; a wrong checkpoint is off by its size)."""
    S.price(W.option(paths=64, steps=1), scheme)
    old = S.get_tile()
    try:
        S.set_tile(256, 1)
        for paths, steps in ((2, 1), (65, 8), (1023, 9), (1025, 32), (5000, 65), (98304, 17), (98305, 17)):
            o = W.option(K=101.0, payoff=1, paths=paths, steps=steps, seed=paths)
            g = S.greeks(o, scheme, checkpoint_every=ck)
            h = S.greeks(o, scheme, checkpoint_every=8)
            assert bits(g) == bits(S.price(o, scheme)), (paths, steps)
            for a, b, se in zip(g.grads, h.grads, h.grad_se):
                assert abs(a - b) <= 1e-5 * max(abs(b), se * paths ** 0.5), (paths, steps, a, b)
    finally:
        S.set_tile(*old)


def test_on_a_stream_with_new_constants_each_call(S):
    """On a stream of its own the small option is launched, not replayed: options of one shape and other
    constants give the default stream's results."""
    import torch
    opts = [W.option(K=95.0 + k, xi=0.2 + 0.1 * k, paths=3000, steps=19, seed=k) for k in range(4)]
    want = [bits(S.price(o)) for o in opts]
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        assert [bits(S.price(o)) for o in opts] == want
        assert [bits(S.price(o)) for o in reversed(opts)] == want[::-1]
    st.synchronize()


def test_profiling_records_price_and_not_the_allocation_free_call(S):
    """While profiling, a small price records its kernel; the allocation-free call creates no events."""
    L, ctx = S.library(), S.context()
    L.simr_profile_enable.argtypes = [ctypes.c_void_p, ctypes.c_int]
    L.simr_profile_read.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.POINTER(ctypes.c_double),
                                    ctypes.POINTER(ctypes.c_int64)]
    L.simr_profile_reset.argtypes = [ctypes.c_void_p]
    o = W.option(paths=3000, steps=9)
    want = bits(S.price(o))

    def launches():
        ms, n = ctypes.c_double(), ctypes.c_int64()
        assert L.simr_profile_read(ctx, 0, ctypes.byref(ms), ctypes.byref(n)) == 0
        return n.value

    L.simr_profile_reset(ctx)
    L.simr_profile_enable(ctx, 1)
    try:
        assert bits(S.price_noalloc(o)) == want and launches() == 0
        assert bits(S.price(o)) == want and launches() == 1
    finally:
        L.simr_profile_enable(ctx, 0)
        L.simr_profile_reset(ctx)
