"""GPU parity of the packed 4-bit activation path: the stand-alone packer, the GEMM that reads packed codes, and a producer
that writes them for its consumer, against the CPU oracle (int32 accumulators, codes and bytes bit for bit)."""
import numpy as np
import pytest

import workloads
from helpers import both_layers, calib, check_q, check_y, requant_fp32_sequence

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import oracle
    import paper_2510_02822_amd as fq
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fq.load()
    oracle.build()
    return torch, oracle, fq, torch.device("cuda:0")


def _dev(torch, a, dev):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def decode_packed4(x4, k4p):
    """The documented layout, written out: the sixteen channels 16 p .. 16 p + 15 of a row are the eight bytes at 8 p; in
    dword e byte b holds channel 16 p + 8 e + b in its low half and channel 16 p + 8 e + 4 + b in its high half."""
    rows = x4.shape[0]
    out = np.zeros((rows, k4p), np.int32)
    for c in range(k4p):
        p, e, hi, b = c // 16, (c % 16) // 8, (c % 8) // 4, c % 4
        byte = x4[:, 8 * p + 4 * e + b].astype(np.int32)
        nib = (byte >> 4) & 15 if hi else byte & 15
        out[:, c] = np.where(nib >= 8, nib - 16, nib)
    return out


def _lowered_codes(oracle, Xq, gs, shifts, k):
    sh = np.repeat(np.asarray(shifts, np.int32), gs)[None, :k]
    L = np.clip(Xq[:, :k].astype(np.int32) >> sh, -8, 7)
    # spot-check the vectorised form against the oracle's scalar definition
    for i in (0, Xq.shape[0] - 1):
        for j in range(0, k, 7):
            assert L[i, j] == oracle.bitlower(int(Xq[i, j]), int(sh[0, j]))
    return L


@pytest.mark.parametrize("M,K,N,gs", [(64, 256, 256, 32), (301, 192, 72, 32), (77, 512, 64, 64), (1000, 160, 40, 32)])
def test_packer_and_gemm(env, M, K, N, gs):
    torch, oracle, fq, dev = env
    case = workloads.make_linear("p4", 11, M + K + N, M, K, N, gs, outlier_frac=0.02)
    ol, hl, x_scale = both_layers(case)
    Xq = oracle.quantize(case.X, x_scale)[:, ol.perm]
    Xd = _dev(torch, Xq, dev)
    G = K // gs
    for r in (1.0, 0.75, 0.5, 1.0 / G, 0.0):
        k4 = fq.flexiq_set_ratio(hl, r)
        k4p = fq.flexiq_packed4_channels(hl)
        assert k4p == (k4 // 64) * 64
        assert fq.flexiq_packed4_bytes(hl, M) == M * K // 2
        x4 = torch.full((M, K // 2), 0xA5, dtype=torch.uint8, device=dev)
        fq.flexiq_lower_packed4(hl, Xd, x4)
        torch.cuda.synchronize()
        x4h = x4.cpu().numpy()
        if k4p:
            assert (decode_packed4(x4h, k4p) == _lowered_codes(oracle, Xq, gs, ol.a_shift, k4p)).all(), r
        assert (x4h[:, k4p // 2:] == 0xA5).all()          # nothing written beyond the packed channels
        # the packed columns of X are not read: poison them
        Xp = Xq.copy()
        Xp[:, :k4p] = 77
        ref = oracle.forward_gemm(ol, Xq, r)
        so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9) or 1.0
        out = fq.flexiq_mixed_gemm_packed4(hl, _dev(torch, Xp, dev), x4, acc=True, y=True, q=True, out_scale=so)
        torch.cuda.synchronize()
        assert (out["acc"].cpu().numpy() == ref).all(), r
        check_q(out["q"].cpu().numpy(), ref, ol, so)
        assert (out["q"].cpu().numpy() == requant_fp32_sequence(ref, ol, so)).all()


def test_every_tile_shape_and_block_count(env):
    torch, oracle, fq, dev = env
    case = workloads.make_linear("p4tiles", 11, 5, 700, 320, 136, 32, outlier_frac=0.02)
    ol, hl, x_scale = both_layers(case)
    Xq = oracle.quantize(case.X, x_scale)[:, ol.perm]
    Xd = _dev(torch, Xq, dev)
    n = fq.debug_force_tile(-1)
    try:
        for r in (1.0, 0.5):
            k4 = fq.flexiq_set_ratio(hl, r)
            x4 = fq.flexiq_lower_packed4(hl, Xd)
            ref = oracle.forward_gemm(ol, Xq, r)
            for t in range(n):
                fq.debug_force_tile(t)
                for nb in (0, 1, 3):
                    fq.debug_max_blocks(nb)
                    got = fq.flexiq_mixed_gemm_packed4(hl, Xd, x4, acc=True)["acc"].cpu().numpy()
                    assert (got == ref).all(), (r, t, nb)
    finally:
        fq.debug_force_tile(-1)
        fq.debug_max_blocks(0)


@pytest.mark.parametrize("M,K,N,gs", [(1000, 64, 64, 32), (777, 64, 256, 32), (2000, 128, 528, 64), (513, 256, 80, 32),
                                      (300, 256, 128, 64), (4099, 128, 48, 32), (1, 256, 32, 32), (1500, 256, 272, 32)])
def test_row_streaming_kernel_reads_packed_codes(env, M, K, N, gs, kernel=2):
    """Layers with 64, 128 or 256 channels: the row-streaming kernel whose waves walk groups of 32 rows fetches the packed
    codes (half the bytes) and expands them in registers after the fragment read.  int8 rows (its only output in that build) against the oracle's accumulators requantised, for ratios that
    leave X pieces and packed pieces in one copy instruction, a trailing 4-bit group of 32 that is lowered from X, all
    packed, none packed; saturating inputs; rows that do not fill the last tile; several column blocks."""
    torch, oracle, fq, dev = env
    case = workloads.make_linear("p4st", 11, 3 * M + K + N, M, K, N, gs, outlier_frac=0.02)
    case.X *= 2.0   # some values saturate under the calibrated positions
    ol, hl, x_scale = both_layers(case)
    Xq = oracle.quantize(case.X, x_scale)[:, ol.perm]
    Xd = _dev(torch, Xq, dev)
    G = K // gs
    fq.debug_force_stream(kernel)
    try:
        for r in sorted({1.0, (G - 1) / G, 0.5, 1.0 / G, 0.0}):
            k4 = fq.flexiq_set_ratio(hl, r)
            k4p = fq.flexiq_packed4_channels(hl)
            x4 = fq.flexiq_lower_packed4(hl, Xd)
            Xp = Xq.copy()
            Xp[:, :k4p] = 77          # the packed columns of X are not read
            ref = oracle.forward_gemm(ol, Xq, r)
            so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.7) or 1.0
            got = fq.flexiq_mixed_gemm_packed4(hl, _dev(torch, Xp, dev), x4, q=True, out_scale=so)["q"].cpu().numpy()
            assert fq.debug_last_launch()["tile"] == -2 and fq.debug_force_stream(kernel) == kernel, (r, k4, k4p)   # ran on that kernel
            check_q(got, ref, ol, so)
            assert (got == requant_fp32_sequence(ref, ol, so)).all(), (r, k4, k4p)
    finally:
        fq.debug_force_stream(-1)


def test_run_time_positions_and_saturating_inputs(env):
    torch, oracle, fq, dev = env
    M, K, N, gs = 500, 256, 48, 32
    case = workloads.make_linear("p4dyn", 11, 9, M, K, N, gs, outlier_frac=0.02)
    case.X *= 4.0   # well above the calibrated ranges: the static positions saturate, the run-time ones do not
    ol, hl, x_scale = both_layers(case)
    Xq = oracle.quantize(case.X, x_scale)[:, ol.perm]
    Xd = _dev(torch, Xq, dev)
    k4 = fq.flexiq_set_ratio(hl, 0.75)
    G4 = k4 // gs
    x4 = fq.flexiq_lower_packed4(hl, Xd)
    got = fq.flexiq_mixed_gemm_packed4(hl, Xd, x4, acc=True)["acc"].cpu().numpy()
    assert (got == oracle.forward_gemm(ol, Xq, 0.75)).all()
    fq.flexiq_dynamic_positions(hl, Xd)
    dyn = oracle.dynamic_act_shifts(Xq, gs, G4, ol.a_shift)
    x4 = fq.flexiq_lower_packed4(hl, Xd)
    assert (decode_packed4(x4.cpu().numpy(), (k4 // 64) * 64) == _lowered_codes(oracle, Xq, gs, dyn, (k4 // 64) * 64)).all()
    got = fq.flexiq_mixed_gemm_packed4(hl, Xd, x4, acc=True)["acc"].cpu().numpy()
    assert (got == oracle.mixed_gemm(Xq, ol.Wq.reshape(N, K), gs, G4, dyn, ol.w_shift)).all()
    fq.flexiq_static_positions(hl)


def test_producer_packs_for_consumer(env):
    """fc1 writes fc2's leading channels as packed codes (flexiq_out.x4) and the rest of its int8 output lowered; fc2 reads
    both.  Intermediate tensor and fc2's accumulators equal the oracle's chain, for every tile shape of the producer."""
    torch, oracle, fq, dev = env
    M, K1, N1, N2, gs = 300, 192, 256, 96, 32
    c1 = workloads.make_linear("chain1", 8, 201, M, K1, N1, gs, outlier_frac=0.02)
    c2 = workloads.make_linear("chain2", 8, 202, M, N1, N2, gs, outlier_frac=0.02)
    xs1, am1 = calib(c1)
    o1 = oracle.prepare_layer(c1.W, am1, xs1, gs, bias=c1.bias)
    Xq = oracle.quantize(c1.X, xs1)[:, o1.perm]
    acc1 = oracle.forward_gemm(o1, Xq, 0.5)
    y1 = oracle.dequant_f64(acc1, xs1, o1.w_scale, o1.bias)
    s_mid = float(np.abs(y1).max() / 127.0)
    q1 = requant_fp32_sequence(acc1, o1, s_mid)
    check_q(q1, acc1, o1, s_mid)
    am2 = np.abs(q1).max(0).astype(np.float32) * np.float32(s_mid)
    o2 = oracle.prepare_layer(c2.W, am2, s_mid, gs, bias=c2.bias)
    X2 = np.ascontiguousarray(q1[:, o2.perm])
    h2 = fq.flexiq_quantize_pack(c2.W, am2, s_mid, gs, bias=c2.bias)
    h1 = fq.flexiq_quantize_pack(c1.W, am1, xs1, gs, bias=c1.bias, out_perm=o2.perm)
    fq.flexiq_set_ratio(h1, 0.5)
    Xd = _dev(torch, Xq, dev)
    n_tiles = fq.debug_force_tile(-1)
    try:
        for r2 in (1.0, 0.75, 0.375, 0.0):
            k4 = fq.flexiq_set_ratio(h2, r2)
            k4p = fq.flexiq_packed4_channels(h2)
            sh = np.repeat(o2.a_shift.astype(np.int32), gs)[None, :]
            want_mid = X2.astype(np.int32).copy()
            want_mid[:, :k4] = np.clip(want_mid[:, :k4] >> sh[:, :k4], -8, 7) << sh[:, :k4]
            want_codes = _lowered_codes(oracle, X2, gs, o2.a_shift, k4p) if k4p else None
            for t in (range(n_tiles) if r2 == 0.75 else (-1,)):
                fq.debug_force_tile(t)
                x4 = torch.full((M, N1 // 2), 0x5A, dtype=torch.uint8, device=dev)
                qbuf = {"q": torch.full((M, N1), 99, dtype=torch.int8, device=dev)}
                fq.flexiq_mixed_gemm(h1, Xd, q=True, out_scale=s_mid, bufs=qbuf, lower_for=h2, x4_out=x4)
                torch.cuda.synchronize()
                mid = qbuf["q"].cpu().numpy().astype(np.int32)
                assert (mid[:, k4p:] == want_mid[:, k4p:]).all(), (r2, t)
                assert (mid[:, :k4p] == 99).all(), (r2, t)          # q is left alone where the codes went to x4
                if k4p:
                    assert (decode_packed4(x4.cpu().numpy(), k4p) == want_codes).all(), (r2, t)
            fq.debug_force_tile(-1)
            got = fq.flexiq_mixed_gemm_packed4(h2, qbuf["q"], x4, acc=True)["acc"].cpu().numpy()
            assert (got == oracle.forward_gemm(o2, X2, r2)).all(), r2
    finally:
        fq.debug_force_tile(-1)
    with pytest.raises(fq.FlexiqError):   # packed output needs the consumer
        fq.flexiq_mixed_gemm(h1, Xd, q=True, out_scale=s_mid, x4_out=x4)


@pytest.mark.parametrize("K,N,gs", [(256, 256, 32), (1024, 72, 64), (192, 8200, 32)])
def test_few_row_dot_kernel_reads_packed_codes(env, K, N, gs):
    # calls of a few rows: the dot-product kernel takes the producer's packed codes as they are (no clamp, no packing in
    # the kernel); rows 1 and 2 by the automatic route, 3 and 4 forced, with one and with four column groups per block
    torch, oracle, fq, dev = env
    case = workloads.make_linear("p4few", 11, 900 + K + N, 4, K, N, gs, outlier_frac=0.02)
    case.X *= 2.0
    ol, hl, x_scale = both_layers(case)
    Xq = oracle.quantize(case.X, x_scale)[:, ol.perm]
    G = K // gs
    try:
        for r in sorted({1.0, 0.5, 1.0 / G, 0.0}):
            k4 = fq.flexiq_set_ratio(hl, r)
            k4p = fq.flexiq_packed4_channels(hl)
            ref = oracle.forward_gemm(ol, Xq, r)
            so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9) or 1.0
            for M, mode in ((1, -1), (2, -1), (3, 2), (4, 2), (2, 14), (4, 14)):
                Xd = _dev(torch, Xq[:M], dev)
                x4 = fq.flexiq_lower_packed4(hl, Xd)
                Xp = Xq[:M].copy()
                Xp[:, :k4p] = 77                      # the packed columns of X are not read
                fq.debug_force_few_rows(mode)
                out = fq.flexiq_mixed_gemm_packed4(hl, _dev(torch, Xp, dev), x4, acc=True, q=True, out_scale=so)
                torch.cuda.synchronize()
                if k4p:   # (no packed channel at this ratio: an ordinary call)
                    assert fq.debug_force_few_rows(mode) == 2 and fq.debug_last_launch()["tile"] == -4, (M, mode, r)
                assert (out["acc"].cpu().numpy() == ref[:M]).all(), (M, mode, r)
                check_q(out["q"].cpu().numpy(), ref[:M], ol, so)
        # more rows than the dot-product kernel takes: the tiled kernel reads the packed codes
        fq.debug_force_few_rows(-1)
        fq.flexiq_set_ratio(hl, 1.0)
        Xd = _dev(torch, np.ascontiguousarray(np.repeat(Xq, 3, axis=0)), dev)
        out = fq.flexiq_mixed_gemm_packed4(hl, Xd, fq.flexiq_lower_packed4(hl, Xd), acc=True)
        assert 0 <= fq.debug_last_launch()["tile"] < fq.debug_force_tile(-1)
        assert (out["acc"].cpu().numpy() == np.repeat(oracle.forward_gemm(ol, Xq, 1.0), 3, axis=0)).all()
    finally:
        fq.debug_force_few_rows(-1)


@pytest.mark.parametrize("M,K,N,gs", [(17, 768, 96, 32), (33, 1056, 300, 32), (130, 1472, 257, 64), (200, 384, 64, 64)])
def test_tile_per_block_kernel_reads_packed_codes(env, M, K, N, gs):
    """Every tile of the kernel whose waves split the reduction: K-steps of packed codes before none, some and all of the others, a trailing 4-bit group
    of 32 lowered from X, an odd number of units, rows and columns that do not fill the last tile."""
    torch, oracle, fq, dev = env
    case = workloads.make_linear("p4tile", 11, M + K + N, M, K, N, gs, outlier_frac=0.02)
    case.X *= 2.0   # some values saturate under the calibrated positions
    ol, hl, x_scale = both_layers(case)
    Xq = oracle.quantize(case.X, x_scale)[:, ol.perm]
    try:
        for r in sorted({1.0, 0.5, 3 * gs / K, 0.0}):
            fq.flexiq_set_ratio(hl, r)
            k4p = fq.flexiq_packed4_channels(hl)
            ref = oracle.forward_gemm(ol, Xq, r)
            so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9) or 1.0
            x4 = fq.flexiq_lower_packed4(hl, _dev(torch, Xq, dev))
            Xp = Xq.copy()
            Xp[:, :k4p] = 77   # the packed columns of X are not read
            for shape in (1, 2, 3, 4):   # the automatic tile and the three
                fq.debug_force_tile_splitk(shape)
                out = fq.flexiq_mixed_gemm_packed4(hl, _dev(torch, Xp, dev), x4, acc=True, y=True, q=True, out_scale=so)
                assert fq.debug_last_launch()["tile"] == -5
                assert (out["acc"].cpu().numpy() == ref).all(), (r, shape)
                check_y(out["y"].cpu().numpy(), ref, ol)
                assert (out["q"].cpu().numpy() == requant_fp32_sequence(ref, ol, so)).all(), (r, shape)
    finally:
        fq.debug_force_tile_splitk(-1)


@pytest.mark.parametrize("M", [1, 9, 50, 150, 300])
@pytest.mark.parametrize("pre", [False, True])
def test_tile_per_block_kernel_packs_for_a_consumer(env, M, pre):
    """Codes, the int8 columns beside them and what is left alone equal the tiled kernel's, by the automatic route and for every tile; a consumer whose
    activations arrive lowered takes no codes."""
    torch, oracle, fq, dev = env
    K, N = 800, 416
    first = workloads.make_linear("p4out1", 11, M, M, K, N, 32)
    second = workloads.make_linear("p4out2", 11, M + 1, 64, N, 64, 32)
    x_scale = oracle.absmax_scale(first.Xcal)
    o2, h2, _ = both_layers(second)
    hl = fq.flexiq_quantize_pack(first.W, np.abs(first.Xcal).max(0), x_scale, 32, bias=first.bias, out_perm=o2.perm)
    X = _dev(torch, oracle.quantize(first.X, x_scale)[:, hl.info()["perm"]], dev)
    fq.flexiq_input_prelowered(h2, pre)
    def call():
        x4 = torch.full((M, N // 2), 0x5A, dtype=torch.uint8, device=dev)
        q = torch.full((M, N), 99, dtype=torch.int8, device=dev)
        out = fq.flexiq_mixed_gemm(hl, X, q=True, y=True, out_scale=0.5, bufs={"q": q}, lower_for=h2, x4_out=x4)
        return x4, q, out["y"]
    try:
        for r1, r2 in ((0.0, 1.0), (0.5, 0.5), (1.0, 0.0)):
            fq.flexiq_set_ratio(hl, r1)
            fq.flexiq_set_ratio(h2, r2)
            fq.debug_force_tile_splitk(0)
            want = call()
            assert 0 <= fq.debug_last_launch()["tile"] < fq.debug_force_tile(-1)
            for shape in (-1, 2, 3, 4):
                fq.debug_force_tile_splitk(shape)
                got = call()
                assert fq.debug_last_launch()["tile"] == -5, (r1, r2, shape)
                for g, w in zip(got, want):
                    assert torch.equal(g, w), (r1, r2, shape)
    finally:
        fq.debug_force_tile_splitk(-1)
