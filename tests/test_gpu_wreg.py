"""GPU parity of the linear kernel whose weights are resident in registers against the CPU oracle, through flexiq_mixed_gemm: int32
sums and int8 codes bit for bit."""
import numpy as np
import pytest

import workloads
from helpers import both_layers, check_q, check_y, requant_fp32_sequence

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
    fq.debug_force_halo(0)
    fq.debug_force_wreg(1)
    yield torch, oracle, fq, torch.device("cuda:0")
    for hook in (fq.debug_force_few_rows, fq.debug_force_tile_splitk, fq.debug_force_halo, fq.debug_force_wreg):
        hook(-1)


# (M, C, N, gs): every number of units held (16, 24, 32, 40), full, short of one unit and of seven, odd; one tile, ragged last tiles,
# blocks of one to three tiles (the loop and its last rounds; the ring in use beyond its slots: test_many_tiles_per_block), several
# column blocks with a ragged last one, more column blocks than compute units' share of row groups, N not a multiple of 32, of 16 and of 4
CASES = [(1, 512, 256, 64), (31, 288, 40, 32), (33, 480, 300, 32), (1000, 768, 3072, 64), (1025, 544, 2816, 32), (700, 736, 4100, 32),
         (2100, 1024, 2049, 64), (450, 992, 6144, 32), (830, 800, 6160, 32), (97, 1280, 16384, 64), (300, 1248, 10000, 32), (161, 1056, 16400, 32),
         (193, 320, 20000, 64)]


@pytest.mark.parametrize("M,C,N,gs", CASES)
def test_sums_and_codes(env, M, C, N, gs):
    torch, oracle, fq, dev = env
    case = workloads.make_linear("wreg", 22, M + C + N, M, C, N, gs)
    case.X *= 2.0   # some values saturate under the calibrated positions
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    Xd = torch.from_numpy(Xq).to(dev)
    rows = np.unique(np.concatenate([np.arange(min(M, 40)), np.arange(max(0, M - 40), M), np.linspace(0, M - 1, 24).astype(int)]))
    for r in sorted({0.0, gs / C, 0.5, 1.0}):
        fq.flexiq_set_ratio(hl, r)
        ref = oracle.forward_gemm(ol, np.ascontiguousarray(Xq[rows]), r)
        so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9) or 1.0
        codes = requant_fp32_sequence(ref, ol, so)
        out = fq.flexiq_mixed_gemm(hl, Xd, acc=True, y=True, q=True, out_scale=so)
        assert fq.debug_force_wreg(1) == 1
        assert (out["acc"].cpu().numpy()[rows] == ref).all(), r
        check_y(out["y"].cpu().numpy()[rows], ref, ol)
        assert (out["q"].cpu().numpy()[rows] == codes).all(), r
        check_q(codes, ref, ol, so)
        for kind in ("q", "y"):   # builds that write one output
            only = fq.flexiq_mixed_gemm(hl, Xd, out_scale=so, **{kind: True})[kind]
            assert fq.debug_force_wreg(1) == 1 and (only == out[kind]).all().item(), (r, kind)


def _tiles_per_block(torch, M, N):
    """Row tiles of the fullest and of the emptiest block, as the launcher deals them out."""
    cols, tiles = -(-N // 256), -(-M // 32)
    groups = max(1, min(tiles, torch.cuda.get_device_properties(0).multi_processor_count // cols))
    return -(-tiles // groups), tiles // groups


def _ring(C):
    """LDS slots for row tiles: four while four of them and the tables fit, else three."""
    held = -(-(C // 32) // 8) * 8
    return 4 if held * 1024 * 4 + 3 * 256 * 4 <= 160 * 1024 else 3


# Every number of units held, full (each piece of a tile copied by every wave) and not, by one unit and by seven: blocks of more than twice as
# many tiles as the ring has slots, so that every slot is filled again with rows that are multiplied, some blocks one tile ahead of others
@pytest.mark.parametrize("C,gs", [(512, 64), (480, 32), (288, 32), (768, 32), (544, 32), (736, 32), (1024, 64), (992, 32), (800, 32), (1280, 32), (1248, 32), (1056, 32)])
def test_many_tiles_per_block(env, C, gs):
    torch, oracle, fq, dev = env
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    N = 64 * cus + 16   # three groups of blocks on 256 compute units, and a last column block of 16 columns
    slots = _ring(C)
    M = 32 * ((2 * slots + 1) * (cus // -(-N // 256)) + 1) - 11
    most, least = _tiles_per_block(torch, M, N)
    assert least > 2 * slots and most == least + 1
    case = workloads.make_linear("wregring", 22, C, M, C, N, gs)
    case.X *= 2.0
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    Xd = torch.from_numpy(Xq).to(dev)
    rows = np.r_[0, 31, 32, 32 * slots + 3, M // 2, M - 33, M - 1]
    for r in sorted({0.0, gs / C, 0.5, 1.0}):
        fq.flexiq_set_ratio(hl, r)
        ref = oracle.forward_gemm(ol, np.ascontiguousarray(Xq[rows]), r)
        so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9)
        fq.debug_force_wreg(0)   # the tiled kernel: every row
        want = fq.flexiq_mixed_gemm(hl, Xd, acc=True, y=True, q=True, out_scale=so)
        assert 0 <= fq.debug_last_launch()["tile"] < fq.debug_force_tile(-1)
        assert (want["acc"].cpu().numpy()[rows] == ref).all() and (want["q"].cpu().numpy()[rows] == requant_fp32_sequence(ref, ol, so)).all()
        fq.debug_force_wreg(1)
        for kinds in ("q", "y", ("acc", "y", "q")):
            got = fq.flexiq_mixed_gemm(hl, Xd, out_scale=so, **{k: True for k in kinds})
            assert fq.debug_force_wreg(1) == 1
            for k in kinds:
                assert torch.equal(got[k], want[k]), (r, k, len(kinds))


# the same for the builds that lower for a consumer (of at most 159 channel groups: fewer columns, more rows)
@pytest.mark.parametrize("C", [512, 288, 768, 544, 1024, 992, 1280, 1056])
def test_many_tiles_per_block_lowered_for_a_consumer(env, C):
    torch, oracle, fq, dev = env
    N, slots = 5120, _ring(C)
    M = 32 * ((2 * slots + 1) * (torch.cuda.get_device_properties(0).multi_processor_count // (N // 256)) + 1) - 5
    assert _tiles_per_block(torch, M, N)[1] > 2 * slots
    first = workloads.make_linear("wregring1", 22, C, M, C, N, 32)
    second = workloads.make_linear("wregring2", 22, C + 1, 64, N, 64, 64)
    x_scale = oracle.absmax_scale(first.Xcal)
    o2, h2, _ = both_layers(second)
    hl = fq.flexiq_quantize_pack(first.W, np.abs(first.Xcal).max(0), x_scale, 32, bias=first.bias, out_perm=o2.perm)
    X = torch.from_numpy(np.ascontiguousarray(oracle.quantize(first.X, x_scale)[:, hl.info()["perm"]])).to(dev)
    for r1, r2 in ((0.0, 0.5), (0.5, 1.0), (1.0, 0.25)):
        fq.flexiq_set_ratio(hl, r1)
        k4 = fq.flexiq_set_ratio(h2, r2)
        so = float(fq.flexiq_mixed_gemm(hl, X[:64].contiguous(), y=True)["y"].abs().max()) / 127
        plain = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=so)["q"]
        assert fq.debug_force_wreg(0) == 1
        want = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=so, lower_for=h2)["q"]
        assert 0 <= fq.debug_last_launch()["tile"] < fq.debug_force_tile(-1)
        fq.debug_force_wreg(1)
        got = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=so, lower_for=h2)["q"]
        assert fq.debug_force_wreg(1) == 1 and torch.equal(got, want)
        # ... and from the definition: the codes of the consumer's 4-bit channels clamped and cleared at its positions
        sh = torch.from_numpy(np.repeat(o2.a_shift.astype(np.int32), 64)[:k4]).to(dev)
        low = plain.to(torch.int32)
        low[:, :k4] = ((low[:, :k4] >> sh).clamp(-8, 7)) << sh
        assert torch.equal(got.to(torch.int32), low) and not torch.equal(got, plain)


@pytest.mark.parametrize("M,C,N", [(2500, 768, 1024), (700, 1248, 512)])
def test_lowered_for_a_consumer_and_positions_found_at_run_time(env, M, C, N):
    torch, oracle, fq, dev = env
    first = workloads.make_linear("wreg1", 22, 1, M, C, N, 32)
    second = workloads.make_linear("wreg2", 22, 2, 64, N, 64, 32)
    x_scale = oracle.absmax_scale(first.Xcal)
    o2, h2, x2 = both_layers(second)
    hl = fq.flexiq_quantize_pack(first.W, np.abs(first.Xcal).max(0), x_scale, 32, bias=first.bias, out_perm=o2.perm)
    X = torch.from_numpy(np.ascontiguousarray(oracle.quantize(first.X, x_scale)[:, hl.info()["perm"]])).to(dev)
    for r1, r2 in ((0.0, 0.5), (0.5, 1.0), (1.0, 0.25)):
        fq.flexiq_set_ratio(hl, r1)
        fq.flexiq_set_ratio(h2, r2)
        fq.flexiq_dynamic_positions(hl, X)
        so = float(fq.flexiq_mixed_gemm(hl, X, y=True)["y"].abs().max()) / 127
        plain = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=so)["q"]
        assert fq.debug_force_wreg(0) == 1
        assert (plain == fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=so)["q"]).all().item()
        want = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=so, lower_for=h2)["q"]
        fq.debug_force_wreg(1)
        got = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=so, lower_for=h2)["q"]
        assert fq.debug_force_wreg(1) == 1 and (got == want).all().item() and (got != plain).any().item()
        fq.flexiq_input_prelowered(h2, True)
        pre = fq.flexiq_mixed_gemm(h2, got, acc=True)["acc"]
        fq.flexiq_input_prelowered(h2, False)
        assert (pre == fq.flexiq_mixed_gemm(h2, plain, acc=True)["acc"]).all().item()


# Calls whose blocks would walk several tiles and leave much of the grid unused go to the tiled kernel: (M, C, N, outputs, taken).  Shares of
# 0.39 and 0.91 with whole quads; 0.61 with two outputs, ragged and not; 0.53 and 0.85 with one ragged output; 0.55 with two; one tile per
# block and 0.53; many tiles and shares of 0.48 and 0.24, ragged 0.45 and 0.17
@pytest.mark.parametrize("M,C,N,outs,taken", [(3018, 384, 540, "q", False), (1320, 1024, 2880, "q", True), (4000, 384, 639, "qy", False), (4000, 384, 640, "qy", True),
                                              (6054, 512, 547, "y", False), (11400, 736, 1409, "y", True), (505, 384, 4597, "qy", False), (1000, 1280, 1101, "qy", True),
                                              (100352, 512, 128, "q", True), (60000, 512, 64, "q", False), (60000, 512, 123, "y", True), (60000, 512, 45, "y", False)])
def test_route_by_the_used_share_of_the_grid(env, M, C, N, outs, taken):
    torch, oracle, fq, dev = env
    case = workloads.make_linear("wregshare", 22, M + N, M, C, N, 32)
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    fq.flexiq_set_ratio(hl, 0.5)
    hooks = (fq.debug_force_few_rows, fq.debug_force_tile_splitk, fq.debug_force_halo, fq.debug_force_wreg)
    for hook in hooks:
        hook(-1)
    try:
        out = fq.flexiq_mixed_gemm(hl, torch.from_numpy(Xq).to(dev), out_scale=0.5, **{o: True for o in outs})
        tile = fq.debug_last_launch()["tile"]
        assert tile == -6 if taken else 0 <= tile < fq.debug_force_tile(-1), tile
    finally:
        for hook, mode in zip(hooks, (0, 0, 0, 1)):
            hook(mode)
    pick = np.r_[0:min(M, 40), M - 1]
    ref = oracle.forward_gemm(ol, Xq[pick], 0.5)
    if "q" in outs:
        assert (out["q"].cpu().numpy()[pick] == requant_fp32_sequence(ref, ol, 0.5)).all()
    if "y" in outs:
        check_y(out["y"].cpu().numpy()[pick], ref, ol)


# fp32 rows beyond the last-level cache leave at once where the number of units asks for it (build 2), the others between the matrix instructions of
# the next tile (1): below and above 240 MB with all units of 24 and 32 held, below and above 400 MB with 16, 20 of 24 and 28 of 32; ragged rows and columns
@pytest.mark.parametrize("M,C,N,r,build", [(12607, 768, 4756, 0.0, 1), (12607, 768, 4860, 0.0, 2), (12607, 1024, 4860, 0.5, 2), (12607, 512, 7924, 0.5, 1),
                                           (12607, 512, 7940, 0.5, 2), (12607, 640, 7940, 0.0, 2), (12607, 384, 7940, 1.0, 2), (12607, 896, 7940, 0.0, 1)])
def test_fp32_rows_beyond_the_cache(env, M, C, N, r, build):
    torch, oracle, fq, dev = env
    rng = np.random.default_rng(C + N)
    hl = fq.flexiq_quantize_pack(rng.standard_normal((N, C), dtype=np.float32) * 0.02, np.exp(rng.standard_normal(C)).astype(np.float32), 0.05, 32,
                                 bias=rng.standard_normal(N).astype(np.float32))
    fq.flexiq_set_ratio(hl, r)
    gen = torch.Generator(device=dev)
    gen.manual_seed(N)
    X = torch.randint(-128, 128, (M, C), dtype=torch.int8, device=dev, generator=gen)
    got = fq.flexiq_mixed_gemm(hl, X, y=True)["y"]
    assert fq.debug_force_wreg(0) == build
    want = fq.flexiq_mixed_gemm(hl, X, y=True)["y"]   # the tiled kernel
    assert fq.debug_force_wreg(1) == 0
    assert torch.equal(got, want)
