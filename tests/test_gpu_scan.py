"""GPU parity of the scan for run-time extraction positions at the edges of its block layout: a lone row, rows that are not a multiple of a
thread's trip, one group and all groups, more than 64 groups in a block, more than 256 pieces of 16 channels (several columns of blocks), through both
entry points, against the oracle (whole numbers)."""
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
    import ctypes
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
