"""GPU parity of the FP6 linear kernel whose weights are resident in registers against the CPU oracle, through flexiq_mixed_gemm_fp6: int32
sums, int8 codes and the consumer's FP6 codes bit for bit."""
import numpy as np
import pytest

import workloads
from helpers import both_layers, check_y, requant_fp32_sequence

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import oracle
    import paper_2510_02822_amd as fq
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fq.load()
    oracle.build()
    fq.debug_force_few_rows(0)
    fq.debug_force_tile_splitk(0)
    fq.debug_force_wreg6(1)
    yield torch, oracle, fq, torch.device("cuda:0")
    for hook in (fq.debug_force_few_rows, fq.debug_force_tile_splitk, fq.debug_force_wreg6):
        hook(-1)


def _positions(fq, hl, torch, Xd, dynamic):
    if dynamic:
        fq.flexiq_dynamic_positions(hl, Xd)
    assert fq.flexiq_fp6_channels(hl) == hl.C, "the case is meant to be on the FP6 path as a whole"


# (M, C, N, gs): every number of K-steps held (4, 8, 12, 16, 20), full and short of one to three; one row, tiles in either half of a
# block of 64 rows, ragged last tiles; blocks of one to four tiles, with 16 and 20 K-steps of more than the ring has slots (the ring in use
# beyond its slots with every number of K-steps: test_many_tiles_per_block); several column blocks, ragged ones, N not a multiple of 16 and of 4,
# more column blocks than an XCD's band
CASES = [(1, 256, 64, 64), (33, 64, 40, 32), (200, 192, 300, 32), (1000, 512, 2048, 64), (700, 320, 515, 32), (97, 448, 6144, 64), (2100, 768, 2049, 64),
         (450, 576, 4112, 32), (3300, 1024, 16384, 64), (830, 832, 16400, 32), (161, 960, 64, 64), (6500, 1280, 4160, 64), (65, 1088, 8200, 32), (4200, 1216, 4864, 64)]


@pytest.mark.parametrize("M,C,N,gs", CASES)
def test_sums_and_codes(env, M, C, N, gs):
    torch, oracle, fq, dev = env
    case = workloads.make_linear("wreg6", 22, M + C + N, M, C, N, gs)
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    Xd = torch.from_numpy(Xq).to(dev)
    fq.flexiq_set_ratio(hl, 1.0)
    _positions(fq, hl, torch, Xd, False)
    x6, xlow = fq.flexiq_lower_fp6(hl, Xd)
    rows = np.unique(np.concatenate([np.arange(min(M, 40)), np.arange(max(0, M - 40), M), np.linspace(0, M - 1, 24).astype(int)]))
    ref = oracle.forward_gemm(ol, np.ascontiguousarray(Xq[rows]), 1.0)
    so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9) or 1.0
    out = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, acc=True, y=True, q=True, out_scale=so)
    assert fq.debug_force_wreg6(0) == 1
    want = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, acc=True, y=True, q=True, out_scale=so)   # the tiled kernel: every row
    assert fq.debug_force_wreg6(1) == 0
    assert (out["acc"].cpu().numpy()[rows] == ref).all()
    check_y(out["y"].cpu().numpy()[rows], ref, ol)
    assert (out["q"].cpu().numpy()[rows] == requant_fp32_sequence(ref, ol, so)).all()
    for kind in ("acc", "y", "q"):   # ... and the builds that write one output
        only = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, out_scale=so, **{kind: True})[kind]
        assert fq.debug_force_wreg6(1) == 1 and torch.equal(only, want[kind]) and torch.equal(out[kind], want[kind]), kind


# A consumer at several ratios: all its channels as FP6 codes, some with the others lowered or as they are, none; its positions calibrated or found
@pytest.mark.parametrize("M,C,N,gs2", [(1, 256, 64, 32), (95, 448, 320, 32), (2500, 768, 3072, 64), (700, 1216, 1216, 64), (1290, 1024, 4096, 32)])
def test_codes_for_a_consumer(env, M, C, N, gs2):
    torch, oracle, fq, dev = env
    first = workloads.make_linear("wreg6a", 22, M + N, M, C, N, 64)
    second = workloads.make_linear("wreg6b", 22, M + N + 1, 64, N, 64, gs2)
    x_scale = oracle.absmax_scale(first.Xcal)
    o2, h2, _ = both_layers(second)
    hl = fq.flexiq_quantize_pack(first.W, np.abs(first.Xcal).max(0), x_scale, 64, bias=first.bias, out_perm=o2.perm)
    X = torch.from_numpy(np.ascontiguousarray(oracle.quantize(first.X, x_scale)[:, hl.info()["perm"]])).to(dev)
    fq.flexiq_set_ratio(hl, 1.0)
    for dynamic, r2 in ((False, 1.0), (False, 0.6), (True, 0.3), (True, 1.0), (False, 0.0)):
        k4 = fq.flexiq_set_ratio(h2, r2)
        _positions(fq, hl, torch, X, dynamic)
        x6, xlow = fq.flexiq_lower_fp6(hl, X)
        so = float(fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, y=True)["y"].abs().max()) / 127
        plain = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, q=True, out_scale=so)["q"]
        k6 = fq.flexiq_fp6_channels(h2)
        x6o = torch.zeros(fq.flexiq_fp6_bytes(h2, M), dtype=torch.uint8, device=dev)
        got = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, q=True, out_scale=so, lower_for=h2, x6_out=x6o)["q"]
        assert fq.debug_force_wreg6(1) == 1
        # the definition: the packer's FP6 codes of the plain rows, and the consumer's other 4-bit channels clamped and cleared
        want6 = torch.zeros_like(x6o)
        fq.flexiq_lower_fp6(h2, plain, x6=want6)
        assert torch.equal(x6o, want6), (dynamic, r2)
        sh = torch.from_numpy(np.repeat(fq.flexiq_layer_positions(h2).astype(np.int32), gs2)[:k4]).to(dev)
        low = plain.to(torch.int32)
        low[:, :k4] = ((low[:, :k4] >> sh).clamp(-8, 7)) << sh
        assert torch.equal(got[:, k6:].to(torch.int32), low[:, k6:]), (dynamic, r2)
        rows = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, q=True, out_scale=so, lower_for=h2)["q"]
        assert fq.debug_force_wreg6(1) == 1 and torch.equal(rows.to(torch.int32), low), (dynamic, r2)


def _ring(C):
    """LDS slots for row tiles: six while six of them and the tables fit."""
    held = -(-C // 256) * 4
    stage = 1024 * 8 * -(-(3 * held // 2) // 8)
    return min(6, (160 * 1024 - 2 * 256 * 4) // stage)


def _rows_for(torch, C, N, ragged):
    """Rows that give every block more than twice as many tiles as the ring has slots, and some blocks one more."""
    groups = torch.cuda.get_device_properties(0).multi_processor_count // -(-N // 256)
    M = 32 * ((2 * _ring(C) + 1) * groups + 1) - ragged
    tiles = -(-M // 32)
    assert groups > 1 and tiles // groups > 2 * _ring(C) and tiles % groups == 1
    return M


# Every number of K-steps held, full and short of one and of three: blocks of more than twice as many tiles as the ring has slots, so that every slot
# is filled again with rows that are multiplied, and the sums of a tile leave beside the next one many times, some blocks one tile ahead of others
@pytest.mark.parametrize("C", [256, 192, 64, 512, 448, 320, 768, 704, 576, 1024, 960, 832, 1280, 1216, 1088])
def test_many_tiles_per_block(env, C):
    torch, oracle, fq, dev = env
    N = 64 * torch.cuda.get_device_properties(0).multi_processor_count + 16   # a last column block of 16 columns
    M = _rows_for(torch, C, N, 11)
    case = workloads.make_linear("wreg6ring", 22, C, M, C, N, 32)
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    Xd = torch.from_numpy(Xq).to(dev)
    rows = np.r_[0, 31, 32, 32 * _ring(C) + 3, M // 2, M - 33, M - 1]
    fq.flexiq_set_ratio(hl, 1.0)
    _positions(fq, hl, torch, Xd, False)
    x6, xlow = fq.flexiq_lower_fp6(hl, Xd)
    ref = oracle.forward_gemm(ol, np.ascontiguousarray(Xq[rows]), 1.0)
    so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9)
    fq.debug_force_wreg6(0)   # the tiled kernel: every row
    want = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, acc=True, y=True, q=True, out_scale=so)
    assert fq.debug_force_wreg6(1) == 0
    assert (want["acc"].cpu().numpy()[rows] == ref).all() and (want["q"].cpu().numpy()[rows] == requant_fp32_sequence(ref, ol, so)).all()
    for kinds in ("q", "y", ("acc", "y", "q")):
        got = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, out_scale=so, **{k: True for k in kinds})
        assert fq.debug_force_wreg6(1) == 1
        for k in kinds:
            assert torch.equal(got[k], want[k]), (k, len(kinds))


# the same for the builds that write a consumer's FP6 codes and lowered rows (of at most 159 channel groups: fewer columns, more rows)
@pytest.mark.parametrize("C", [256, 64, 512, 320, 768, 576, 1024, 832, 1280, 1088])
def test_many_tiles_per_block_for_a_consumer(env, C):
    torch, oracle, fq, dev = env
    N = 5120
    M = _rows_for(torch, C, N, 5)
    first = workloads.make_linear("wreg6ring1", 22, C, M, C, N, 64)
    second = workloads.make_linear("wreg6ring2", 22, C + 1, 64, N, 64, 32)
    x_scale = oracle.absmax_scale(first.Xcal)
    W2, amax2, scale2 = second.W.reshape(64, N), np.abs(second.Xcal).max(0), float(np.abs(second.Xcal).max() / 127)
    h2 = fq.flexiq_quantize_pack(W2, amax2, scale2, 64)
    hl = fq.flexiq_quantize_pack(first.W, np.abs(first.Xcal).max(0), x_scale, 64, bias=first.bias, out_perm=h2.info()["perm"])
    X = torch.from_numpy(np.ascontiguousarray(oracle.quantize(first.X, x_scale)[:, hl.info()["perm"]])).to(dev)
    fq.flexiq_set_ratio(hl, 1.0)
    _positions(fq, hl, torch, X, False)
    x6, xlow = fq.flexiq_lower_fp6(hl, X)
    so = float(fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, y=True)["y"].abs().max()) / 127
    plain = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, q=True, out_scale=so)["q"]
    assert fq.debug_force_wreg6(1) == 1
    for r2 in (1.0, 0.4):
        k4 = fq.flexiq_set_ratio(h2, r2)
        k6 = fq.flexiq_fp6_channels(h2)
        assert 0 < k6 <= k4
        x6o = torch.zeros(fq.flexiq_fp6_bytes(h2, M), dtype=torch.uint8, device=dev)
        got = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, q=True, out_scale=so, lower_for=h2, x6_out=x6o)["q"]
        assert fq.debug_force_wreg6(1) == 1
        rows = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, q=True, out_scale=so, lower_for=h2)["q"]
        assert fq.debug_force_wreg6(0) == 1
        t6 = torch.zeros_like(x6o)
        tiled = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, q=True, out_scale=so, lower_for=h2, x6_out=t6)["q"]
        assert fq.debug_force_wreg6(1) == 0
        assert torch.equal(x6o, t6) and torch.equal(got[:, k6:], tiled[:, k6:]), r2
        # ... and from the definition: the packer's FP6 codes of the plain rows, the consumer's 4-bit channels clamped and cleared
        want6 = torch.zeros_like(x6o)
        fq.flexiq_lower_fp6(h2, plain, x6=want6)
        sh = torch.from_numpy(np.repeat(fq.flexiq_layer_positions(h2).astype(np.int32), 64)[:k4]).to(dev)
        low = plain.to(torch.int32)
        low[:, :k4] = ((low[:, :k4] >> sh).clamp(-8, 7)) << sh
        assert torch.equal(x6o, want6) and torch.equal(rows.to(torch.int32), low), r2


# Which calls it gets: every channel as FP6 and 256 to 1280 of them; (M, C, N, r, taken: by this kernel, else by the tiled one)
@pytest.mark.parametrize("M,C,N,r,taken", [(3000, 1024, 1024, 1.0, True), (3000, 1024, 1024, 0.5, False), (3000, 1344, 1024, 1.0, False), (6000, 192, 1024, 1.0, False),
                                           (6000, 256, 1024, 1.0, True)])
def test_route(env, M, C, N, r, taken):
    torch, oracle, fq, dev = env
    hooks = (fq.debug_force_few_rows, fq.debug_force_tile_splitk, fq.debug_force_wreg6)
    case = workloads.make_linear("wreg6r", 22, M + C, M, C, N, 64)
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    fq.flexiq_set_ratio(hl, r)
    x6, xlow = fq.flexiq_lower_fp6(hl, torch.from_numpy(Xq).to(dev))
    for hook in hooks:
        hook(-1)
    try:
        acc = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, acc=True)["acc"]
        assert fq.debug_force_wreg6(-1) == int(taken)
    finally:
        for hook, mode in zip(hooks, (0, 0, 1)):
            hook(mode)
    pick = np.r_[0:40, M - 1]
    assert (acc.cpu().numpy()[pick] == oracle.forward_gemm(ol, Xq[pick], r)).all()


# ... and where it is ahead of the tiled kernel: by how many tiles a block walks, how much of the grid is used, rows of whole quads, columns, and whether
# the output fits the last-level cache
@pytest.mark.parametrize("M,C,N,outputs", [
    (1576, 320, 2048, {"q": True, "y": True, "yq": True, "acc": True}),               # two tiles per block, a used share of 0.77
    (1576, 320, 1536, {"q": False, "y": True, "yq": False, "acc": False}),            # ... of 0.58
    (3152, 768, 515, {"q": False, "y": False, "acc": False}),                         # ... of 0.39, rows that leave element by element
    (1576, 320, 33000, {"q": False, "y": True, "yq": True}),                          # half of the chip idle, int8 rows of 8 bytes
    (1576, 320, 36864, {"q": True, "y": True}),                                       # ... of 16 bytes
    (197, 512, 51200, {"q": True, "y": True}), (197, 512, 65536, {"q": False, "y": False}),   # 200 and 256 column blocks of seven tiles
    (4200, 256, 16384, {"q": True, "y": False, "acc": False, "yq": True}),            # 275 MB of fp32
    (3900, 256, 16384, {"y": True, "acc": True})])                                    # 256 MB
def test_route_by_outputs(env, M, C, N, outputs):
    torch, oracle, fq, dev = env
    hooks = (fq.debug_force_few_rows, fq.debug_force_tile_splitk, fq.debug_force_wreg6)
    rng = np.random.default_rng(M + N)
    hl = fq.flexiq_quantize_pack(rng.standard_normal((N, C), dtype=np.float32) * 0.02, np.exp(rng.standard_normal(C)).astype(np.float32), 0.05, 64)
    fq.flexiq_set_ratio(hl, 1.0)
    gen = torch.Generator(device=dev)
    gen.manual_seed(N)
    x6, xlow = fq.flexiq_lower_fp6(hl, torch.randint(-128, 128, (M, C), dtype=torch.int8, device=dev, generator=gen))
    _positions(fq, hl, torch, xlow, False)
    for name, taken in outputs.items():
        kw = {k: True for k in (("y", "q") if name == "yq" else (name,))}
        for hook in hooks:
            hook(-1)
        try:
            got = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, out_scale=0.5, **kw)
            assert fq.debug_force_wreg6(-1) == int(taken), (name, taken)
        finally:
            for hook, mode in zip(hooks, (0, 0, 0 if taken else 1)):
                hook(mode)
        want = fq.flexiq_mixed_gemm_fp6(hl, xlow, x6, out_scale=0.5, **kw)   # the other kernel
        assert fq.debug_force_wreg6(1) == int(not taken)
        assert all(torch.equal(got[k], want[k]) for k in kw), name
