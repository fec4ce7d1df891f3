"""The native calls of the binding (csrc/calls.cpp) against the functions of binding.py that they stand for.  On the CPU: what they are as objects,
and the refusal of what is no layer, no GPU tensor or no argument list of theirs.  On the GPU: the same results, the same refusals of GPU tensors that
do not fit a live layer, and the stream."""
import copy
import inspect
import pickle
import weakref

import numpy as np
import pytest

import workloads
from helpers import both_layers

CALLS = ["flexiq_mixed_gemm", "flexiq_mixed_gemm_fp6", "flexiq_mixed_gemm_packed4", "flexiq_mixed_conv_implicit", "flexiq_lower_fp6", "flexiq_lower_packed4",
         "flexiq_quantize_act", "flexiq_permute_channels", "flexiq_dynamic_positions"]


@pytest.mark.parametrize("name", CALLS)
def test_calls_are_native_and_keep_their_signature(name):
    import paper_2510_02822_amd as fq
    f = getattr(fq, name)
    assert fq.binding._calls is not None and type(f).__name__ == "Call" and f.__name__ == name and f.__doc__ == f.__wrapped__.__doc__
    assert str(inspect.signature(f)) == str(inspect.signature(f.__wrapped__))


@pytest.mark.parametrize("name", CALLS)
def test_calls_are_used_like_functions(name):
    import paper_2510_02822_amd as fq
    f = getattr(fq, name)
    assert copy.deepcopy({"call": f})["call"] is f and copy.copy(f) is f and weakref.ref(f)() is f
    for protocol in range(pickle.HIGHEST_PROTOCOL + 1):
        assert pickle.loads(pickle.dumps(f, protocol)) is f
    assert inspect.isfunction(f) and inspect.isroutine(f) and callable(f)
    for attribute in ("__defaults__", "__kwdefaults__", "__code__", "__closure__", "__globals__"):
        assert getattr(f, attribute) is getattr(f.__wrapped__, attribute)
    with pytest.raises(AttributeError):
        f.no_such_attribute
    holder = type("Holder", (), {"call": f})
    bound = holder().call
    assert holder.call is f and inspect.ismethod(bound) and bound.__func__ is f
    with pytest.raises((AttributeError, AssertionError)):   # (the holder stands for the first argument)
        bound(*[None] * (len(inspect.signature(f).parameters) - 1 - len(f.__defaults__ or ())))


def test_sizes_of_a_layer_are_ordinary_attributes():
    import paper_2510_02822_amd as fq
    layer = fq.Layer(0, 4, 64, 3, 1, 32)
    assert {k: vars(layer)[k] for k in ("N", "C", "R", "S", "group_size")} == {"N": 4, "C": 64, "R": 3, "S": 1, "group_size": 32}
    for value in (np.int64(8), 8.0, None, 1 << 70):
        layer.N = value
        assert layer.N is value
    del layer.C
    assert not hasattr(layer, "C")


def test_what_a_native_call_does_not_serve():
    import torch
    import paper_2510_02822_amd as fq
    fq.load()
    freed = fq.Layer(0, 4, 64, 1, 1, 32)
    x = torch.zeros(2, 64, dtype=torch.int8)   # not on a GPU
    bad = [(fq.flexiq_mixed_gemm, (freed, x), {}, AssertionError), (fq.flexiq_mixed_gemm, (), {}, TypeError), (fq.flexiq_mixed_gemm, (freed, x), {"Q": True}, TypeError),
           (fq.flexiq_mixed_gemm, (freed, x), {"X": x}, TypeError), (fq.flexiq_mixed_gemm, (freed, "x"), {}, AttributeError), (fq.flexiq_mixed_gemm, (freed,) * 12, {}, TypeError),
           (fq.flexiq_mixed_gemm_fp6, (freed, x), {}, TypeError), (fq.flexiq_mixed_conv_implicit, (freed, x, 0, 0), {}, AssertionError),
           (fq.flexiq_quantize_act, (torch.zeros(3), 1.0), {}, AssertionError), (fq.flexiq_permute_channels, (freed, x), {}, AssertionError),
           (fq.flexiq_dynamic_positions, (freed, x), {}, AssertionError), (fq.flexiq_lower_fp6, (freed, x), {}, AssertionError), (fq.flexiq_lower_packed4, (freed, x), {}, AssertionError)]
    for f, args, kw, error in bad:
        for g in (f, f.__wrapped__):
            with pytest.raises(error):
                g(*args, **kw)


@pytest.mark.gpu
def test_same_results_as_the_functions_they_stand_for():
    import torch
    import paper_2510_02822_amd as fq
    dev = torch.device("cuda:0")
    first, second, cv = (workloads.make_linear("calls", 31, 1, 70, 128, 256, 32), workloads.make_linear("calls2", 31, 2, 70, 256, 64, 32),
                         workloads.make_conv("calls3", 31, 3, 2, 9, 7, 64, 64, 3, 3, 2, 1, 32))
    _, h2, _ = both_layers(second)
    x_scale = float(np.abs(first.Xcal).max() / 127)
    h1 = fq.flexiq_quantize_pack(first.W, np.abs(first.Xcal).max(0), x_scale, 32, bias=first.bias, out_perm=h2.info()["perm"])
    _, hc, sc = both_layers(cv)
    for h in (h1, h2, hc):
        fq.flexiq_set_ratio(h, 0.75)
    xf = torch.from_numpy(first.X).to(dev)
    native = {n: getattr(fq, n) for n in CALLS}
    plain = {n: getattr(fq, n).__wrapped__ for n in CALLS}

    def run(f):
        got = []
        q = f["flexiq_quantize_act"](xf, x_scale)
        own = torch.empty_like(q)
        assert f["flexiq_quantize_act"](xf, scale=x_scale, out=own) is own and torch.equal(own, q)
        x = f["flexiq_permute_channels"](h1, q)
        x6, xlow = f["flexiq_lower_fp6"](h1, x)
        mine = torch.zeros_like(x6)
        a, b = f["flexiq_lower_fp6"](h1, x, x6=mine, need_xlow=True)
        assert a is mine and b is not x and torch.equal(b, xlow)
        with pytest.raises(fq.FlexiqError):   # (a 4-bit group of 32 is left over: its channels have to be lowered somewhere)
            f["flexiq_lower_fp6"](h1, x, need_xlow=False)
        x4 = f["flexiq_lower_packed4"](h1, x)
        got += [q, x, xlow, x4[:, :32]]   # (of 96 4-bit channels 64 are packed)
        for kw in ({"acc": True}, {"y": True, "q": True, "out_scale": 0.25}, {"q": True, "out_scale": 0.25, "lower_for": h2},
                   {"q": True, "out_scale": np.float32(0.5)}, {"acc": 1, "out_scale": 2}):   # (the last two: not served natively)
            got += list(f["flexiq_mixed_gemm"](h1, x, **kw).values())
            got += list(f["flexiq_mixed_gemm_fp6"](h1, xlow, x6, **kw).values())
            got += list(f["flexiq_mixed_gemm_packed4"](h1, x, x4, **kw).values())
        bufs = {"y": torch.zeros(70, 256, device=dev)}
        out = f["flexiq_mixed_gemm"](h1, x, False, True, bufs=bufs, out_scale=1.0)
        assert list(out) == ["acc", "y", "q"] and out["y"] is bufs["y"] and out["acc"] is None and out["q"] is None
        got.append(out["y"])
        n6 = torch.zeros(fq.flexiq_fp6_bytes(h2, 70), dtype=torch.uint8, device=dev)
        n4 = torch.zeros(70, 128, dtype=torch.uint8, device=dev)
        f["flexiq_mixed_gemm_fp6"](h1, xlow, x6, q=True, out_scale=0.25, lower_for=h2, x6_out=n6)
        f["flexiq_mixed_gemm"](h1, x, q=True, out_scale=0.25, lower_for=h2, x4_out=n4)
        f["flexiq_mixed_gemm"](h1, x, q=True, out_scale=0.25, scan_for=h2)
        fq.flexiq_static_positions(h2)
        xc = torch.from_numpy(np.ascontiguousarray(np.clip(np.rint(cv.X / sc), -127, 127).astype(np.int8))).to(dev)
        got += [n6, n4] + list(f["flexiq_mixed_conv_implicit"](hc, xc, 2, 1, q=True, y=True, out_scale=0.25).values())
        assert f["flexiq_dynamic_positions"](h1, x) is None
        got.append(torch.from_numpy(fq.flexiq_layer_positions(h1).astype(np.int32)))
        fq.flexiq_static_positions(h1)
        for bad in ({"q": True, "out_scale": -1.0}, {}, {"q": True, "lower_for": hc}):   # refused by the library
            with pytest.raises(fq.FlexiqError):
                f["flexiq_mixed_gemm"](h1, x, **bad)
        other = torch.cuda.Stream()
        other.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(other):
            z = f["flexiq_mixed_gemm"](h1, x, acc=True)["acc"]
        torch.cuda.current_stream().wait_stream(other)
        return got + [z]

    for a, b in zip(run(native), run(plain)):
        assert (a is None and b is None) or (a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and torch.equal(a, b))


def _live(fq, workloads):
    """A linear layer of 128 channels, one that reads its 256 outputs, and a convolution, all at 3/4 of the channels at 4 bits."""
    first, second, cv = (workloads.make_linear("calls", 31, 1, 70, 128, 256, 32), workloads.make_linear("calls2", 31, 2, 70, 256, 64, 32),
                         workloads.make_conv("calls3", 31, 3, 2, 9, 7, 64, 64, 3, 3, 2, 1, 32))
    layers = [both_layers(c)[1] for c in (first, second, cv)]
    for h in layers:
        fq.flexiq_set_ratio(h, 0.75)
    return layers


@pytest.mark.gpu
def test_tensors_that_do_not_fit_a_live_layer():
    """What the native checks let through would go to a kernel: type, contiguity, the number of dimensions and the channels."""
    import torch
    import paper_2510_02822_amd as fq
    dev = torch.device("cuda:0")
    h, _, hc = _live(fq, workloads)
    rows = torch.zeros(70, 128, dtype=torch.int8, device=dev)
    image = torch.zeros(2, 9, 7, 64, dtype=torch.int8, device=dev)
    x6 = torch.zeros(fq.flexiq_fp6_bytes(h, 70), dtype=torch.uint8, device=dev)
    x4 = torch.zeros(70, 64, dtype=torch.uint8, device=dev)
    bad_rows = [rows.to(torch.uint8), rows.to(torch.int32), rows.t().contiguous().t(), torch.zeros(70, 256, dtype=torch.int8, device=dev)[:, ::2], rows[:, :64].contiguous(),
                torch.zeros(70, 256, dtype=torch.int8, device=dev), rows[0], rows.view(7, 10, 128), rows.cpu()]
    bad_images = [image.to(torch.uint8), image.permute(0, 3, 1, 2), image[:, :, :, :32].contiguous(), torch.zeros(2, 9, 7, 96, dtype=torch.int8, device=dev), image[0], image[None], image.cpu()]
    calls = [(fq.flexiq_mixed_gemm, lambda x: (h, x, True), bad_rows), (fq.flexiq_mixed_gemm_fp6, lambda x: (h, x, x6, True), bad_rows),
             (fq.flexiq_mixed_gemm_packed4, lambda x: (h, x, x4, True), bad_rows), (fq.flexiq_lower_fp6, lambda x: (h, x), bad_rows),
             (fq.flexiq_lower_packed4, lambda x: (h, x), bad_rows), (fq.flexiq_mixed_conv_implicit, lambda x: (hc, x, 2, 1, True), bad_images),
             (fq.flexiq_dynamic_positions, lambda x: (h, x), bad_rows[:6] + bad_rows[8:]),   # (any number of dimensions)
             (fq.flexiq_permute_channels, lambda x: (h, x), bad_rows[:4] + bad_rows[8:]),    # (... and whole rows of its own)
             (fq.flexiq_quantize_act, lambda x: (x, 0.5), [rows, rows.half(), rows.double(), torch.zeros(70, 128, device=dev).t(), torch.zeros(70, 128)])]
    for f, arguments, bad in calls:
        for x in bad:
            for g in (f, f.__wrapped__):
                with pytest.raises(AssertionError):
                    g(*arguments(x))
    assert fq.flexiq_dynamic_positions(h, rows.view(7, 10, 128)) is None   # what is accepted: sizes that are no plain integers too
    fq.flexiq_static_positions(h)
    want = fq.flexiq_mixed_gemm(h, rows, True)["acc"]
    vars(h)["N"] = 512   # (more than it has: the output is as large as the attribute says at the time of the call)
    assert fq.flexiq_mixed_gemm(h, rows, True)["acc"].shape == fq.flexiq_mixed_gemm.__wrapped__(h, rows, True)["acc"].shape == (70, 512)
    h.N, h.C = np.int64(256), np.int64(128)
    assert torch.equal(fq.flexiq_mixed_gemm(h, rows, True)["acc"], want)


@pytest.mark.gpu
def test_calls_go_to_the_current_stream():
    """Captured on a stream of their own: work on any other stream would not be in the graph, whose replays write every output again."""
    import torch
    import paper_2510_02822_amd as fq
    dev = torch.device("cuda:0")
    h, _, hc = _live(fq, workloads)
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    x = torch.randint(-128, 128, (70, 128), dtype=torch.int8, device=dev, generator=gen)
    small = torch.randint(-2, 3, (70, 128), dtype=torch.int8, device=dev, generator=gen)
    image = torch.randint(-128, 128, (2, 9, 7, 64), dtype=torch.int8, device=dev, generator=gen)
    xf = torch.randn(70, 128, device=dev, generator=gen)
    x6, xlow = fq.flexiq_lower_fp6(h, x)
    x4 = fq.flexiq_lower_packed4(h, x)
    own = torch.zeros_like(x6)   # (rows of the last 64 and K-steps that the packer does not write stay zero)
    calls = [lambda: [fq.flexiq_mixed_gemm(h, x, acc=True)["acc"]], lambda: [fq.flexiq_mixed_gemm_fp6(h, xlow, x6, y=True)["y"]],
             lambda: [fq.flexiq_mixed_gemm_packed4(h, x, x4, q=True, out_scale=0.5)["q"]], lambda: [fq.flexiq_mixed_conv_implicit(hc, image, 2, 1, acc=True)["acc"]],
             lambda: list(fq.flexiq_lower_fp6(h, x, x6=own, need_xlow=True)), lambda: [fq.flexiq_lower_packed4(h, x)[:, :32]], lambda: [fq.flexiq_quantize_act(xf, 0.02)],
             lambda: [fq.flexiq_permute_channels(h, x)]]
    for call in calls:
        want = [o.clone() for o in call()]
        assert all(o.any().item() for o in want)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            outs = call()
        for _ in range(3):
            for o in outs:
                o.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(o, w) for o, w in zip(outs, want))
    fq.flexiq_dynamic_positions(h, x)
    want = fq.flexiq_layer_positions(h).copy()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fq.flexiq_dynamic_positions(h, x)
    for _ in range(3):
        fq.flexiq_dynamic_positions(h, small)
        assert not np.array_equal(fq.flexiq_layer_positions(h), want)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(fq.flexiq_layer_positions(h), want)
