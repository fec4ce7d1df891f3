"""GPU parity of the convolution kernel whose input tile is resident in LDS (3x3 filters at stride 1 or 2 and any padding, strided or
padded 1x1 filters) against the CPU oracle, through flexiq_mixed_conv_implicit: int32 sums and int8 codes bit for bit."""
import numpy as np
import pytest

import helpers
import workloads
from helpers import both_layers, check_q, check_y, requant_fp32_sequence

pytestmark = pytest.mark.gpu
SHAPES = 13   # block shapes of the kernel's table


@pytest.fixture(scope="module")
def env():
    import torch
    import oracle
    import paper_2510_02822_amd as fq
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fq.load()
    oracle.build()
    yield torch, oracle, fq, torch.device("cuda:0")
    fq.debug_force_halo(-1)


# (B, H, W, C, N, R, stride, pad, gs): tiles that begin inside an image row and span several images, one pixel, one column, an
# odd number of units, runs of 16 / 10 / 2 / 1 LDS pixels per wave, strided rows of odd and even length, no and double
# padding, N below, above and not a multiple of 32, and not of 16 (no whole 16-byte pieces of an output row)
CASES = [(1, 7, 7, 256, 64, 3, 1, 1, 32), (9, 5, 4, 64, 48, 3, 1, 1, 32), (3, 13, 11, 96, 80, 3, 1, 1, 32), (2, 9, 30, 32, 200, 3, 1, 1, 32),
         (1, 1, 1, 64, 32, 3, 1, 1, 64), (2, 10, 12, 128, 33, 3, 1, 0, 64), (2, 6, 7, 160, 72, 3, 1, 2, 32), (3, 13, 10, 96, 64, 3, 2, 1, 32),
         (2, 8, 9, 512, 64, 3, 2, 1, 64), (4, 9, 9, 64, 96, 3, 2, 0, 32), (5, 11, 8, 128, 144, 1, 2, 0, 32), (2, 7, 9, 1024, 64, 1, 2, 0, 64),
         (2, 5, 6, 320, 40, 1, 1, 1, 32), (1, 40, 3, 64, 520, 3, 1, 1, 32), (1, 3, 40, 544, 32, 3, 1, 1, 32)]


@pytest.mark.parametrize("B,H,W,C,N,R,stride,pad,gs", CASES)
def test_all_block_shapes(env, B, H, W, C, N, R, stride, pad, gs):
    torch, oracle, fq, dev = env
    case = workloads.make_conv("halo", 21, 7 * B + H + W + C + N, B, H, W, C, N, R, R, stride, pad, gs)
    case.X *= 2.0   # some pixels saturate under the calibrated positions
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[..., ol.perm])
    Xd = torch.from_numpy(Xq).to(dev)
    ran = set()
    for r in sorted({0.0, gs / C, 0.5, 1.0}):
        fq.flexiq_set_ratio(hl, r)
        ref = oracle.forward_conv(ol, Xq, stride, pad, r)
        so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9) or 1.0
        codes = requant_fp32_sequence(ref, ol, so)
        for k in range(1, SHAPES + 1):
            fq.debug_force_halo(k)
            out = fq.flexiq_mixed_conv_implicit(hl, Xd, stride, pad, acc=True, y=True, q=True, out_scale=so)
            if fq.debug_force_halo(k) != k:
                continue   # (the tile of that shape does not fit LDS, or more shares of the reduction than units)
            ran.add(k)
            assert (out["acc"].cpu().numpy() == ref).all(), (r, k)
            check_y(out["y"].cpu().numpy(), ref, ol)
            assert (out["q"].cpu().numpy() == codes).all(), (r, k)
            only_q = fq.flexiq_mixed_conv_implicit(hl, Xd, stride, pad, q=True, out_scale=so)["q"]
            assert fq.debug_force_halo(k) == k and (only_q.cpu().numpy() == codes).all(), (r, k)
        check_q(codes, ref, ol, so)
    fq.debug_force_halo(-1)
    assert len(ran) >= 3
    fq.flexiq_mixed_conv_implicit(hl, Xd, stride, pad, acc=True)
    assert fq.debug_force_halo(-1) in ran   # the automatic route


@pytest.mark.parametrize("R,stride,pad", [(3, 3, 1), (1, 3, 0), (3, 4, 2)])
def test_larger_strides_stay_with_the_tiled_kernel(env, R, stride, pad):
    torch, oracle, fq, dev = env
    case = workloads.make_conv("halostride", 21, R + stride, 2, 13, 11, 64, 48, R, R, stride, pad, 32)
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[..., ol.perm])
    fq.flexiq_set_ratio(hl, 0.5)
    for k in (-1, 1):
        fq.debug_force_halo(k)
        got = fq.flexiq_mixed_conv_implicit(hl, torch.from_numpy(Xq).to(dev), stride, pad, acc=True)["acc"].cpu().numpy()
        assert 0 <= fq.debug_last_launch()["tile"] < fq.debug_force_tile(-1) and fq.debug_force_halo(-1) == 0
        assert (got == oracle.forward_conv(ol, Xq, stride, pad, 0.5)).all()


def test_positions_found_at_run_time_and_lowered_input(env):
    torch, oracle, fq, dev = env
    B, H, W, C, N, gs = 6, 14, 14, 128, 96, 32
    case = workloads.make_conv("halodyn", 21, 5, B, H, W, C, N, 3, 3, 1, 1, gs)
    case.X *= 3.0
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[..., ol.perm])
    Xd = torch.from_numpy(Xq).to(dev)
    G4 = fq.flexiq_set_ratio(hl, 0.75) // gs
    fq.flexiq_dynamic_positions(hl, Xd.reshape(-1, C))
    dyn = oracle.dynamic_act_shifts(Xq.reshape(-1, C), gs, G4, ol.a_shift)
    got = fq.flexiq_mixed_conv_implicit(hl, Xd, 1, 1, acc=True)["acc"].cpu().numpy()
    assert fq.debug_force_halo(-1) > 0
    assert (got == oracle.mixed_conv(Xq, ol.Wq.reshape(N, 3, 3, C), 1, 1, gs, G4, dyn, ol.w_shift)).all()
    fq.flexiq_static_positions(hl)
    sh = np.repeat(ol.a_shift.astype(np.int32), gs)[None, None, None, :]
    Xl = (np.clip(Xq.astype(np.int32) >> sh, -8, 7) << sh).astype(np.int8)
    Xl[..., G4 * gs:] = Xq[..., G4 * gs:]
    fq.flexiq_input_prelowered(hl, True)
    got = fq.flexiq_mixed_conv_implicit(hl, torch.from_numpy(Xl).to(dev), 1, 1, acc=True)["acc"].cpu().numpy()
    assert fq.debug_force_halo(-1) > 0
    assert (got == oracle.forward_conv(ol, Xq, 1, 1, 0.75)).all()


# (M, K, N, gs): one row, a tile and one row more, runs of 16 / 5 / 2 / 1 rows per wave, odd units, rows beyond M in the last tile,
# N not a multiple of 4, 16 or 32
@pytest.mark.parametrize("M,K,N,gs", [(1, 64, 64, 32), (33, 96, 48, 32), (129, 192, 90, 64), (100, 448, 200, 64), (257, 1024, 64, 32),
                                      (70, 544, 37, 32), (300, 320, 264, 64)])
def test_linear_calls_on_all_block_shapes(env, M, K, N, gs):
    torch, oracle, fq, dev = env
    case = workloads.make_linear("halolin", 22, M + K + N, M, K, N, gs, outlier_frac=0.02)
    case.X *= 2.0
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    Xd = torch.from_numpy(Xq).to(dev)
    fq.debug_force_stream(0)
    fq.debug_force_few_rows(0)
    fq.debug_force_tile_splitk(0)
    ran = set()
    try:
        for r in (0.0, 0.5, 1.0):
            fq.flexiq_set_ratio(hl, r)
            ref = oracle.forward_gemm(ol, Xq, r)
            so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9) or 1.0
            codes = requant_fp32_sequence(ref, ol, so)
            for k in range(1, SHAPES + 1):
                fq.debug_force_halo(k)
                out = fq.flexiq_mixed_gemm(hl, Xd, acc=True, y=True)
                if fq.debug_force_halo(k) != k:
                    continue
                ran.add(k)
                assert (out["acc"].cpu().numpy() == ref).all(), (r, k)
                check_y(out["y"].cpu().numpy(), ref, ol)
                assert (fq.flexiq_mixed_gemm(hl, Xd, q=True, out_scale=so)["q"].cpu().numpy() == codes).all(), (r, k)
    finally:
        fq.debug_force_halo(-1)
        fq.debug_force_stream(-1)
        fq.debug_force_few_rows(-1)
        fq.debug_force_tile_splitk(-1)
    assert len(ran) >= 3


def test_linear_route(env):
    """A mid-size call with a short reduction goes to this kernel by itself, one with many rows to another."""
    torch, oracle, fq, dev = env
    case = workloads.make_linear("haloroute", 22, 1, 1000, 512, 1024, 32)
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    fq.flexiq_set_ratio(hl, 0.5)
    Xd = torch.from_numpy(Xq).to(dev)
    n_tiled = fq.debug_force_tile(-1)
    got = fq.flexiq_mixed_gemm(hl, Xd, acc=True)["acc"].cpu().numpy()
    assert fq.debug_last_launch()["tile"] >= n_tiled
    assert (got == oracle.forward_gemm(ol, Xq, 0.5)).all()
    many = fq.flexiq_mixed_gemm(hl, Xd.repeat(16, 1), acc=True)["acc"]
    assert fq.debug_last_launch()["tile"] < n_tiled
    assert bool((many.view(16, 1000, 1024) == torch.from_numpy(got).to(dev)).all())


@pytest.mark.parametrize("k", range(1, SHAPES + 1))
def test_lowers_for_the_consumer(env, k):
    """flexiq_out.lower_for on every block shape: int8 rows in the consumer's channel order, its 4-bit channels lowered."""
    torch, oracle, fq, dev = env
    B, H, W, C, N1, gs2 = 2, 15, 13, 256, 192, 64
    c1 = workloads.make_conv("halolow1", 21, 11, B, H, W, C, N1, 3, 3, 2, 1, 32)
    xs1, am1 = helpers.calib(c1)
    o1 = oracle.prepare_layer(c1.W, am1, xs1, 32, bias=c1.bias)
    Xq = np.ascontiguousarray(oracle.quantize(c1.X, xs1)[..., o1.perm])
    ref = oracle.forward_conv(o1, Xq, 2, 1, 0.5)
    y = oracle.dequant_f64(ref, xs1, o1.w_scale, c1.bias)
    so = float(np.abs(y).max() / 127 * 0.9)
    c2 = workloads.make_conv("halolow2", 21, 12, B, H, W, N1, 64, 1, 1, 1, 0, gs2)
    am2 = np.abs(y).reshape(-1, N1).max(0).astype(np.float32) * np.float32(0.5)   # (half the range: some codes saturate)
    hl2 = fq.flexiq_quantize_pack(c2.W, am2, so, gs2)
    info = hl2.info()
    hl1 = fq.flexiq_quantize_pack(c1.W, am1, xs1, 32, bias=c1.bias, out_perm=info["perm"])
    fq.flexiq_set_ratio(hl1, 0.5)
    plain = requant_fp32_sequence(ref, o1, so)[..., info["perm"]].astype(np.int32)
    fq.debug_force_halo(k)
    for r2 in (0.0, 0.34, 1.0):
        k4 = fq.flexiq_set_ratio(hl2, r2)
        got = fq.flexiq_mixed_conv_implicit(hl1, torch.from_numpy(Xq).to(dev), 2, 1, q=True, out_scale=so, lower_for=hl2)["q"].cpu().numpy()
        assert fq.debug_force_halo(k) == k
        sh = np.repeat(info["a_shift"].astype(np.int32), gs2)
        want = plain.copy()
        want[..., :k4] = (np.clip(plain[..., :k4] >> sh[:k4], -8, 7) << sh[:k4])
        assert (got == want).all(), (k, r2)
    fq.debug_force_halo(-1)
