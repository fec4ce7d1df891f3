"""CPU checks of the block shape that the resident-input convolution kernel takes for a call: the bounds its index arithmetic counts on hold
for every call it accepts, however large."""
import ctypes as C
import random

import pytest

NCU = 256


@pytest.fixture(scope="module")
def plan():
    import paper_2510_02822_amd as fq
    L = fq.load()
    L.flexiq_debug_halo_plan.argtypes = [C.POINTER(C.c_int64), C.POINTER(C.c_int64)]

    def ask(B, H, W, stride, pad, N, ch, R, out_bytes=1):
        out = (C.c_int64 * 5)()
        rc = L.flexiq_debug_halo_plan((C.c_int64 * 10)(B, H, W, stride, pad, N, ch, R, out_bytes, NCU), out)
        assert rc >= 0
        return (rc, *out) if rc else None
    yield ask
    fq.debug_force_halo(-1)


def _pixels(B, H, W, stride, pad, R):
    return B * ((H + 2 * pad - R) // stride + 1) * ((W + 2 * pad - R) // stride + 1)


def _lds_bytes(P, B, H, W, stride, pad, ch, R):
    """Bytes of the input rows under P consecutive output pixels, from the worst of all beginnings (counted, not derived)."""
    Ho, Wo = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    st = stride if R == 3 else 1
    VH, Wv = (Ho - 1) * st + R, (Wo - 1) * st + R
    row = lambda m: m // Wo // Ho * VH + m // Wo % Ho * st
    M = B * Ho * Wo
    rows = max(row(min(m + P, M) - 1) - row(m) + R for m in range(0, min(M, Ho * Wo), 1))
    return rows * st * -(-Wv // st) * (ch + 16)


@pytest.mark.parametrize("call", [
    (2 ** 31 - 200, 1, 1, 2, 0, 16, 32, 1),         # row indices beyond what any kernel takes
    (2 ** 31 - 500, 1, 1, 2, 0, 256, 64, 1),
    (12000, 60, 60, 2, 0, 16384, 32, 1),            # many column blocks times many tiles: the block index divided by 8 per column block
    (300000, 7, 7, 1, 1, 8192, 32, 3)])
def test_beyond_the_index_arithmetic(plan, call):
    # (every forced shape, so that it is not the cost model that keeps the call within the bounds)
    import paper_2510_02822_amd as fq
    for shape in range(1, 14):
        fq.debug_force_halo(shape)
        got = plan(*call)
        fq.debug_force_halo(-1)
        if got:
            _, P, BN, tiles, ncb, lds = got
            assert tiles * P < 2 ** 31 and tiles * ncb * 8 * ncb < 2 ** 32, (call, got)


def test_accepted_calls_are_in_bounds(plan):
    rng = random.Random(1)
    log = lambda lo, hi: int(lo * (hi / lo) ** rng.random())
    taken = 0
    for _ in range(3000):
        R = rng.choice((1, 3))
        stride, pad = rng.choice((1, 2)), rng.choice((0, 1, 2))
        B, H, W, N, ch = log(1, 1 << 20), log(3, 400), log(3, 400), log(1, 9000), 32 * log(1, 33)
        got = plan(B, H, W, stride, pad, N, ch, R, rng.choice((1, 4, 9)))
        if not got:
            continue
        taken += 1
        _, P, BN, tiles, ncb, lds = got
        M = _pixels(B, H, W, stride, pad, R)
        assert tiles == -(-M // P) and ncb == -(-N // BN) and ncb * BN <= -(-N // 256) * 256
        assert tiles * P < 2 ** 31 and tiles * ncb * 8 * ncb < 2 ** 32 and lds <= 160 * 1024
        assert lds >= 3072 + _lds_bytes(P, min(B, 40), H, W, stride, pad, ch, R), (B, H, W, stride, pad, N, ch, R, got)
    assert taken > 1000


def test_strides_and_filters_that_are_left_alone(plan):
    assert plan(4, 14, 14, 1, 1, 64, 64, 3)
    assert not plan(4, 14, 14, 3, 1, 64, 64, 3)     # strides 1 and 2 only
    assert not plan(4, 14, 14, 3, 0, 64, 64, 1)
    assert not plan(4, 14, 14, 1, 2, 64, 64, 5)     # 3x3 and 1x1 filters only
    assert not plan(4, 14, 14, 2, 1, 64, 544, 3)    # strided: an even number of pixels per copy, up to 512 channels
