"""GPU parity of the linear kernel that takes its activations chunk by chunk (long reductions) against the CPU oracle, through
flexiq_mixed_gemm: int32 sums and int8 codes bit for bit."""
import numpy as np
import pytest

import workloads
from helpers import both_layers, check_q, check_y, requant_fp32_sequence

pytestmark = pytest.mark.gpu

# rows (in fragments of 32) and shares of the reduction of the block shapes, in the order of the launcher's table
SHAPES = [(2, 1), (3, 1), (4, 1), (5, 1), (6, 1), (7, 1), (8, 1), (1, 2), (2, 2), (3, 2), (4, 2), (5, 2), (1, 4), (2, 4), (3, 4)]


@pytest.fixture(scope="module")
def env():
    import torch
    import oracle
    import paper_2510_02822_amd as fq
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    fq.load()
    oracle.build()
    others = (fq.debug_force_few_rows, fq.debug_force_tile_splitk, fq.debug_force_stream)   # (offered a call first)
    for hook in others:
        hook(0)
    yield torch, oracle, fq, torch.device("cuda:0")
    for hook in others + (fq.debug_force_chunk,):
        hook(-1)


# (C, N, gs): the ring of chunks not full (one unit; less than a chunk of every shape), one unit beyond one, two and three chunks of some, many; a
# single column block, a ragged last one, N not a multiple of 32, of 16 and of 4
LAYERS = [(32, 64, 32), (352, 300, 32), (544, 257, 32), (1056, 272, 32), (1664, 640, 64)]


@pytest.mark.parametrize("C,N,gs", LAYERS)
def test_every_shape(env, C, N, gs):
    torch, oracle, fq, dev = env
    case = workloads.make_linear("chunk", 23, C + N, 32 * 8 * 9 + 5, C, N, gs)
    case.X *= 2.0   # some values saturate under the calibrated positions
    ol, hl, x_scale = both_layers(case)
    Xq = np.ascontiguousarray(oracle.quantize(case.X, x_scale)[:, ol.perm])
    for r in sorted({0.0, gs / C, 0.5, 1.0}):
        fq.flexiq_set_ratio(hl, r)
        ref = oracle.forward_gemm(ol, Xq, r)
        so = float(np.abs(oracle.dequant_f64(ref, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9) or 1.0
        codes = requant_fp32_sequence(ref, ol, so)
        check_q(codes, ref, ol, so)
        for k, (fr, wk) in enumerate(SHAPES, 1):
            # one row, a full tile, one row beyond it, nine tiles (a band of eight and a rest) with a ragged last one
            for M in (1, 32 * fr, 32 * fr + 1, 32 * fr * 8 + 5):
                Xd = torch.from_numpy(Xq[:M]).to(dev)
                fq.debug_force_chunk(k)
                out = fq.flexiq_mixed_gemm(hl, Xd, acc=True, y=True, q=True, out_scale=so)
                assert fq.debug_force_chunk(k) == k and fq.debug_last_launch()["tile"] == -7
                assert (out["acc"].cpu().numpy() == ref[:M]).all(), (r, k, M)
                assert (out["q"].cpu().numpy() == codes[:M]).all(), (r, k, M)
                check_y(out["y"].cpu().numpy(), ref[:M], ol)
                for kind in ("q", "y"):   # builds that write one output
                    only = fq.flexiq_mixed_gemm(hl, Xd, out_scale=so, **{kind: True})[kind]
                    assert torch.equal(only, out[kind]), (r, k, M, kind)


@pytest.mark.parametrize("C,N", [(2400, 512), (1312, 1040)])
def test_lowered_for_a_consumer_prelowered_and_positions_found_at_run_time(env, C, N):
    torch, oracle, fq, dev = env
    M = 777
    first = workloads.make_linear("chunk1", 23, C, M, C, N, 32)
    gs2 = 64 if N % 64 == 0 else 0
    x_scale = oracle.absmax_scale(first.Xcal)
    if gs2:
        second = workloads.make_linear("chunk2", 23, C + 1, 64, N, 64, gs2)
        o2, h2, _ = both_layers(second)
    hl = fq.flexiq_quantize_pack(first.W, np.abs(first.Xcal).max(0), x_scale, 32, bias=first.bias, out_perm=o2.perm if gs2 else None)
    X = torch.from_numpy(np.ascontiguousarray(oracle.quantize(first.X, x_scale)[:, hl.info()["perm"]])).to(dev)
    for r1, r2 in ((0.0, 0.5), (0.5, 1.0), (1.0, 0.25)):
        fq.flexiq_set_ratio(hl, r1)
        fq.flexiq_dynamic_positions(hl, X)
        so = 1.0
        for k in range(1, len(SHAPES) + 1):
            calls = [dict(q=True), dict(y=True), dict(acc=True)]
            if gs2:
                fq.flexiq_set_ratio(h2, r2)
                calls.append(dict(q=True, lower_for=h2))
            for pre in (False, True):   # (codes that arrive unlowered under that flag: whatever the bytes are, both kernels multiply the same)
                fq.flexiq_input_prelowered(hl, pre)
                for call in calls:
                    fq.debug_force_chunk(0)
                    want = fq.flexiq_mixed_gemm(hl, X, out_scale=so, **call)
                    assert fq.debug_force_chunk(k) == 0
                    got = fq.flexiq_mixed_gemm(hl, X, out_scale=so, **call)
                    assert fq.debug_force_chunk(k) == k
                    for name in set(call) - {"lower_for"}:
                        assert torch.equal(got[name], want[name]), (r1, k, pre, call.keys())
            fq.flexiq_input_prelowered(hl, False)
    fq.debug_force_chunk(-1)


@pytest.mark.parametrize("C,N,gs2", [(1376, 1056, 32), (992, 352, 32), (1344, 320, 64)])
def test_lowered_for_a_consumer_whose_channels_end_inside_a_block(env, C, N, gs2):
    """Columns that end 32 (or 64) into the last block of every width, 4-bit channels of the consumer that end inside a block, groups of 32 and 64."""
    torch, oracle, fq, dev = env
    M = 300
    first = workloads.make_linear("chunk3", 23, C, M, C, N, 32, outlier_frac=0.02)
    second = workloads.make_linear("chunk4", 23, C + 1, 64, N, 64, gs2)
    x_scale = oracle.absmax_scale(first.Xcal)
    amax = np.abs(first.Xcal).max(0)
    o2, h2, _ = both_layers(second)
    ol = oracle.prepare_layer(first.W, amax, x_scale, 32, bias=first.bias)
    hl = fq.flexiq_quantize_pack(first.W, amax, x_scale, 32, bias=first.bias, out_perm=o2.perm)
    Xq = np.ascontiguousarray(oracle.quantize(first.X, x_scale)[:, ol.perm])
    X = torch.from_numpy(Xq).to(dev)
    for r1, r2 in ((0.0, 0.5), (0.5, 1.0), (1.0, 3 * gs2 / N)):
        fq.flexiq_set_ratio(hl, r1)
        k4 = fq.flexiq_set_ratio(h2, r2)
        acc = oracle.forward_gemm(ol, Xq, r1)
        so = float(np.abs(oracle.dequant_f64(acc, x_scale, ol.w_scale, ol.bias)).max() / 127 * 0.9)
        want = requant_fp32_sequence(acc, ol, so)[:, o2.perm].astype(np.int32)
        for c in range(k4):   # (Section 4.1: cut to four bits at the position and put back there)
            s = int(o2.a_shift[c // gs2])
            want[:, c] = np.clip(want[:, c] >> s, -8, 7) << s
        for k in range(1, len(SHAPES) + 1):
            fq.debug_force_chunk(k)
            got = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=so, lower_for=h2)["q"]
            assert fq.debug_force_chunk(k) == k
            assert (got.cpu().numpy() == want).all(), (r1, r2, k)
    fq.debug_force_chunk(-1)


# Calls of more than 1280 channels whose blocks are one round go to this kernel, in every form it accepts, and from 576 channels on those that would be one
# short round of the kernel with a resident input tile; no other of at most 1280
def test_route(env):
    torch, oracle, fq, dev = env
    for hook in (fq.debug_force_few_rows, fq.debug_force_tile_splitk, fq.debug_force_stream):
        hook(-1)
    gen = np.random.default_rng(5)
    for C, M, taken in ((1280, 3000, False), (1312, 3000, True), (1024, 1500, True), (1024, 9000, False), (576, 1500, True), (544, 1500, False)):
        nx = fq.flexiq_quantize_pack(0.02 * gen.standard_normal((64, 768), dtype=np.float32), np.ones(768, np.float32), 0.03, 32)
        hl = fq.flexiq_quantize_pack(0.02 * gen.standard_normal((768, C), dtype=np.float32), np.ones(C, np.float32), 0.03, 32, out_perm=nx.info()["perm"])
        X = torch.randint(-128, 128, (M, C), dtype=torch.int8, device=dev)
        for r in (0.0, 0.5):
            fq.flexiq_set_ratio(hl, r)
            fq.flexiq_set_ratio(nx, 0.5)
            for call in (dict(q=True), dict(y=True), dict(acc=True, q=True))[: 3 if C > 1280 else 1]:   # (whether a round is short depends on what is written)
                fq.debug_force_chunk(-1)
                got = fq.flexiq_mixed_gemm(hl, X, out_scale=1.0, **call)
                assert (fq.debug_last_launch()["tile"] == -7) == taken
                fq.debug_force_chunk(0)
                want = fq.flexiq_mixed_gemm(hl, X, out_scale=1.0, **call)
                for name in call:
                    assert torch.equal(got[name], want[name])
            fq.debug_force_chunk(-1)
            want = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=1.0)["q"]
            fq.flexiq_dynamic_positions(nx, want)
            positions = fq.flexiq_layer_positions(nx)
            fq.flexiq_static_positions(nx)
            got = fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=1.0, scan_for=nx)["q"]   # (a scan for the consumer follows as a kernel of its own)
            assert (fq.debug_last_launch()["tile"] == -7) == (C > 1280) and torch.equal(got, want)
            assert (np.asarray(fq.flexiq_layer_positions(nx)) == np.asarray(positions)).all()


# What bounds a call decides: not where the weights of a wide layer cross once per row tile, nor where most of a tall block's columns are padding
@pytest.mark.parametrize("M,C,N,r,out,taken", [
    (140, 1920, 11696, 0.0, "q", True), (450, 2176, 8096, 0.0, "q", False), (204, 4480, 8864, 0.0, "q", False), (695, 3200, 10976, 0.0, "q", False),
    (695, 3200, 10976, 1.0, "q", True), (414, 4992, 7712, 0.0, "y", False), (17, 3392, 7408, 0.5, "q", True), (51125, 1600, 80, 0.25, "q", False),
    (20000, 1344, 64, 0.5, "q", True), (1314, 1728, 5968, 0.25, "q", False),
    (22799, 768, 64, 1.0, "q", False), (19097, 768, 32, 0.5, "q", False), (14170, 640, 48, 0.5, "q", True), (23447, 704, 128, 1.0, "q", True),
    (32371, 2176, 64, 0.5, "q", True)])   # (506 blocks: one round only if two of them share a compute unit)
def test_route_by_what_bounds_the_call(env, M, C, N, r, out, taken):
    torch, oracle, fq, dev = env
    for hook in (fq.debug_force_few_rows, fq.debug_force_tile_splitk, fq.debug_force_stream, fq.debug_force_chunk):
        hook(-1)
    hl = fq.flexiq_quantize_pack(0.02 * np.random.default_rng(6).standard_normal((N, C), dtype=np.float32), np.ones(C, np.float32), 0.03, 32)
    fq.flexiq_set_ratio(hl, r)
    X = torch.randint(-128, 128, (M, C), dtype=torch.int8, device=dev)
    got = fq.flexiq_mixed_gemm(hl, X, out_scale=1.0, **{out: True})[out]
    tile = fq.debug_last_launch()["tile"]
    fq.debug_force_chunk(0)
    want = fq.flexiq_mixed_gemm(hl, X, out_scale=1.0, **{out: True})[out]
    fq.debug_force_chunk(-1)
    assert torch.equal(got, want)
    assert (tile == -7) == taken
