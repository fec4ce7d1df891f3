"""GPU parity of the scan for run-time extraction positions at the edges of its block layout: a lone row, rows that are not a multiple of a
thread's trip, one group and all groups, more than 64 groups in a block, more than 256 pieces of 16 channels (several columns of blocks), through both
entry points, against the oracle (whole numbers)."""
import ctypes

import numpy as np
import pytest

import workloads
from helpers import both_layers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,C,gs", [(1, 64, 64), (1, 768, 32), (77, 5088, 32), (515, 4160, 64), (1576, 96, 32), (4099, 320, 64), (16385, 64, 32)])
def test_scan_edges(M, C, gs):
    import torch
    import oracle
    import paper_2510_02822_amd as fq
    fq.load()
    oracle.build()
    case = workloads.make_linear("scan", 12, M + C, 8, C, 16, gs, outlier_frac=0.02)
    ol, hl, x_scale = both_layers(case)
    rng = np.random.default_rng(M + C)
    # a small value everywhere, one larger one in every group and a few at the first and the last row
    X = rng.integers(-3, 4, (M, C), dtype=np.int64).astype(np.int8)
    for g in range(C // gs):
        X[rng.integers(M), g * gs + rng.integers(gs)] = rng.integers(-128, 128)
    X[0, rng.integers(C)] = -128
    X[M - 1, C - 1] = 127
    Xd = torch.from_numpy(X).to("cuda")
    G = C // gs
    for r in (1.0, 1.0 / G, 0.5, 0.0):
        g4 = fq.flexiq_set_ratio(hl, r) // gs
        want = oracle.dynamic_act_shifts(X, gs, g4, ol.a_shift)
        for _ in range(2):   # (the second call finds the scan words as the first one left them)
            fq.flexiq_dynamic_positions(hl, Xd)
            assert np.array_equal(fq.flexiq_layer_positions(hl)[:G], want[:G]), (M, C, gs, r)
        for _ in range(2):   # the scan whose words are shared by all blocks and layers
            fq.flexiq_static_positions(hl)
            fq.flexiq_dynamic_positions_static(hl, Xd)
            assert np.array_equal(fq.flexiq_layer_positions(hl)[:G], want[:G]), (M, C, gs, r)


def _runtime():
    """The HIP runtime that this process runs on."""
    paths = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}
    assert len(paths) == 1, paths
    lib = ctypes.CDLL(paths.pop())
    return lib.hipSetDevice, lib.hipGetLastError


@pytest.mark.parametrize("M,C", [(3, 1024), (200, 1024), (600, 1600), (200, 128)])
def test_a_scan_reports_only_its_own_errors(M, C):
    """An error that another call of the thread has left behind (here: a device that does not exist) is neither reported by a product that scans
    for its consumer, on whichever kernels it runs, nor by the scan alone, nor taken away."""
    import torch
    import paper_2510_02822_amd as fq
    fq.load()
    gen = np.random.default_rng(7)
    N = 512
    nx = fq.flexiq_quantize_pack(0.02 * gen.standard_normal((64, N), dtype=np.float32), np.ones(N, np.float32), 0.03, 32)
    hl = fq.flexiq_quantize_pack(0.02 * gen.standard_normal((N, C), dtype=np.float32), np.ones(C, np.float32), 0.03, 32, out_perm=nx.info()["perm"])
    fq.flexiq_set_ratio(nx, 1.0)
    X = torch.randint(-128, 128, (M, C), dtype=torch.int8, device="cuda")
    q = torch.empty(M, N, dtype=torch.int8, device="cuda")
    def product():
        fq.flexiq_mixed_gemm(hl, X, q=True, out_scale=1.0, bufs={"q": q}, scan_for=nx)
    product()
    torch.cuda.synchronize()
    set_device, last_error = _runtime()
    for call in (product, lambda: fq.flexiq_dynamic_positions(nx, q), lambda: fq.flexiq_dynamic_positions_static(nx, q)):
        last_error()
        assert set_device(1 << 20) != 0
        try:
            call()
        finally:
            left = last_error()
        assert left != 0
    torch.cuda.synchronize()


def _chain(M, K, N, seed):
    """Two layers of which the first one writes in the second one's channel order, the first one's activations, and what the oracle makes of them."""
    import oracle
    import paper_2510_02822_amd as fq
    from helpers import calib
    oracle.build()
    c1 = workloads.make_linear("scanp", seed, 401 + M + K, M, K, N, 32, outlier_frac=0.02)
    c2 = workloads.make_linear("scanc", seed, 402 + M + K, 8, N, 48, 32, outlier_frac=0.02)
    xs, am1 = calib(c1)
    o1 = oracle.prepare_layer(c1.W, am1, xs, 32, bias=c1.bias)
    Xq = np.ascontiguousarray(oracle.quantize(c1.X, xs)[:, o1.perm])
    fq.load()
    return c1, c2, o1, xs, am1, Xq


# rows, channels in and out; the kernel of the product (index of the last launch, None: the tiled one, which scans in its own epilogue)
@pytest.mark.parametrize("M,K,N,kernel,packed", [
    (1, 768, 256, -4, False), (9, 1024, 128, -4, False), (64, 416, 320, -4, False), (64, 64, 1024, -4, False),        # few rows: a scan behind them
    (1, 1024, 128, -4, True), (59, 64, 160, None, False), (1, 320, 160, None, False), (33, 192, 320, None, False),    # ... a short reduction: not
    (40, 768, 288, -5, False), (200, 1024, 160, -5, False), (40, 832, 96, -5, True), (200, 384, 160, -5, True),       # a tile per block
    (700, 1344, 1536, -7, False), (9, 768, 128, None, True)])                                                         # chunk by chunk; codes of few rows
def test_scan_of_a_product(M, K, N, kernel, packed):
    import torch
    import oracle
    import paper_2510_02822_amd as fq
    from helpers import requant_fp32_sequence
    from paper_2510_02822_amd import binding
    c1, c2, o1, xs, am1, Xq = _chain(M, K, N, 14)
    acc = oracle.forward_gemm(o1, Xq, 0.5)
    s_mid = float(np.abs(oracle.dequant_f64(acc, xs, o1.w_scale, o1.bias)).max() / 127.0) * 3.0
    q1 = requant_fp32_sequence(acc, o1, s_mid)
    am2 = np.full(N, 127.0 * s_mid, np.float32)   # calibrated too wide: what the scan finds differs
    o2 = oracle.prepare_layer(c2.W, am2, s_mid, 32, bias=c2.bias)
    X2 = np.ascontiguousarray(q1[:, o2.perm])
    h2 = fq.flexiq_quantize_pack(c2.W, am2, s_mid, 32, bias=c2.bias)
    h1 = fq.flexiq_quantize_pack(c1.W, am1, xs, 32, bias=c1.bias, out_perm=o2.perm)
    fq.flexiq_set_ratio(h1, 0.5)
    X, small = torch.from_numpy(Xq).to("cuda"), torch.from_numpy((Xq // 8).astype(np.int8)).to("cuda")

    def product(x, scale):
        if packed:   # (the C entry point: Python's passes no scan_for)
            q, x4 = torch.empty((M, N), dtype=torch.int8, device="cuda"), fq.flexiq_lower_packed4(h1, x)
            out = binding._Out(q=q.data_ptr(), out_scale=scale, scan_for=h2._h)
            stream = torch.cuda.current_stream().cuda_stream
            assert fq.load().flexiq_mixed_gemm_packed4(h1._h, x.data_ptr(), x4.data_ptr(), M, ctypes.byref(out), stream) == 0
            return q
        return fq.flexiq_mixed_gemm(h1, x, q=True, out_scale=scale, scan_for=h2)["q"]

    differs = False
    for r2 in (1.0, 0.25, 0.0, 0.75):
        fq.flexiq_set_ratio(h2, r2)
        want = oracle.dynamic_act_shifts(X2, 32, oracle.groups_for_ratio(r2, o2.G), o2.a_shift)
        differs |= bool((want != o2.a_shift).any())
        for before in ("calibrated", "scanned"):
            if before == "calibrated":
                fq.flexiq_static_positions(h2)
            else:
                product(small, 4.0 * s_mid)   # (other positions, and scan words that have to be clean again)
            q = product(X, s_mid)
            tile = fq.debug_last_launch()["tile"]
            assert tile == kernel or (kernel is None and 0 <= tile < fq.debug_force_tile(-1)), tile
            assert (q.cpu().numpy() == X2).all(), (r2, before)
            assert (fq.flexiq_layer_positions(h2) == want).all(), (r2, before)
    assert differs


@pytest.mark.parametrize("M,K,N", [(2, 1024, 128), (40, 768, 128), (700, 1344, 1536)])
def test_scan_behind_a_product_in_a_graph(M, K, N):
    """Product and scan captured once and replayed on changing activations, with eager calls and synchronisations in between: every replay leaves the
    positions of its own data."""
    import torch
    import oracle
    import paper_2510_02822_amd as fq
    c1, c2, o1, xs, am1, Xq = _chain(M, K, N, 15)
    s_mid = float(np.abs(oracle.dequant_f64(oracle.forward_gemm(o1, Xq, 0.5), xs, o1.w_scale, o1.bias)).max() / 127.0)
    am2 = np.full(N, 127.0 * s_mid, np.float32)
    h2 = fq.flexiq_quantize_pack(c2.W, am2, s_mid, 32, bias=c2.bias)
    h1 = fq.flexiq_quantize_pack(c1.W, am1, xs, 32, bias=c1.bias, out_perm=h2.info()["perm"])
    fq.flexiq_set_ratio(h1, 0.5)
    fq.flexiq_set_ratio(h2, 1.0)
    x = torch.from_numpy(Xq).to("cuda")
    bufs, other = {"q": torch.empty((M, N), dtype=torch.int8, device="cuda")}, torch.empty((M, N), dtype=torch.int8, device="cuda")
    ends = {"acc": torch.empty((M, 48), dtype=torch.int32, device="cuda")}

    def chain():
        fq.flexiq_mixed_gemm(h1, x, q=True, out_scale=s_mid, bufs=bufs, scan_for=h2)
        fq.flexiq_mixed_gemm(h2, bufs["q"], acc=True, bufs=ends)

    chain()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        chain()
    a_shift = h2.info()["a_shift"]
    for div in (1, 3, 9, 2, 1):
        now = (Xq.astype(np.int32) // div).astype(np.int8)
        x.copy_(torch.from_numpy(now))
        fq.flexiq_mixed_gemm(h1, torch.zeros_like(x), q=True, out_scale=s_mid, bufs={"q": other}, scan_for=h2)   # (an eager scan of other data)
        g.replay()
        torch.cuda.synchronize()
        q = bufs["q"].cpu().numpy()
        want = oracle.dynamic_act_shifts(q, 32, N // 32, a_shift)
        assert (fq.flexiq_layer_positions(h2) == want).all(), div
        eager = fq.flexiq_mixed_gemm(h1, x, q=True, out_scale=s_mid, scan_for=h2)["q"]
        assert (eager.cpu().numpy() == q).all(), div
        assert torch.equal(fq.flexiq_mixed_gemm(h2, eager, acc=True)["acc"], ends["acc"]), div
