"""The binding's native call: what it takes gives the same bits as the library's C entry point, and what it does not take is treated as before."""
import ctypes

import numpy as np
import pytest

import paper_1802_06905_amd as cc
from paper_1802_06905_amd import binding

pytestmark = pytest.mark.gpu

CONV = cc.Problem(4, 8, 6, 5, 7, 3, 3, 1, 1)
POOL = cc.Problem(4, 8, 8, 5, 7, 3, 3, 1, 1)


def operands(torch, kind):
    gen = torch.Generator(device="cuda").manual_seed(5)
    make = lambda *shape: torch.randn(*shape, generator=gen, device="cuda").to(kind)  # noqa: E731
    return make(7, 9, 8, 4), make(6, 3, 3, 8), torch.full((6, 7, 5, 4), float("nan"), device="cuda"), torch.full((8, 7, 5, 4), float("nan"), device="cuda")


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("where", ["current", "null", "side", "handle"])
def test_native_call_runs_on_the_stream_it_is_given(dtype, where):
    import torch
    image, filt, out, pooled = operands(torch, torch.float32 if dtype == 0 else torch.bfloat16)
    ref, ref_pool = torch.empty_like(out), torch.empty_like(pooled)
    assert binding._lib.cacnn_conv_forward(ctypes.byref(CONV), dtype, image.data_ptr(), filt.data_ptr(), ref.data_ptr(), 0) == 0
    assert binding._lib.cacnn_pool_forward(ctypes.byref(POOL), dtype, 1, image.data_ptr(), ref_pool.data_ptr(), 0) == 0
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    stream = {"current": None, "null": 0, "side": side, "handle": side.cuda_stream}[where]
    assert binding._native is not None
    cc.cacnn_conv_forward(CONV, dtype, image, filt, out, stream=stream)
    cc.cacnn_pool_forward(POOL, dtype, cc.CACNN_POOL_MAX, image, pooled, stream=stream)
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and torch.equal(pooled, ref_pool)


def test_current_stream_is_the_one_that_a_graph_captures():
    import torch
    image, filt, out, _ = operands(torch, torch.float32)
    cc.cacnn_conv_forward(CONV, 0, image, filt, out)
    torch.cuda.synchronize()
    eager, graph, side = out.clone(), torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        cc.cacnn_conv_forward(CONV, 0, image, filt, out)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)


def test_other_operands_are_treated_as_before():
    import torch
    image, filt, out, pooled = operands(torch, torch.float32)
    want = out.clone()
    cc.cacnn_conv_forward(CONV, 0, image, filt, want)
    # a plain sequence, an integer type of another kind, raw addresses
    for args in ((tuple(getattr(CONV, n) for n, _ in cc.Problem._fields_), 0, image, filt), (CONV, np.int64(0), image, filt),
                 (CONV, 0, image.data_ptr(), filt.data_ptr())):
        out.fill_(float("nan"))
        cc.cacnn_conv_forward(*args, out)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    # a parameter is a tensor, too
    out.fill_(float("nan"))
    cc.cacnn_conv_forward(CONV, 0, image, torch.nn.Parameter(filt), out)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    for bad in ((image, filt, out[1:]), (image[1:], filt, out), (image, filt[1:], out), (image.half(), filt.half(), out), (image, filt, out.int()),
                (image.transpose(0, 1), filt, out), (image.cpu(), filt, out), (image, filt, out.double())):
        with pytest.raises(ValueError):
            cc.cacnn_conv_forward(CONV, 0, *bad)
    with pytest.raises(ValueError):
        cc.cacnn_pool_forward(POOL, 0, 1, image, pooled[1:])
    with pytest.raises(cc.CacnnError):
        cc.cacnn_conv_forward(CONV, 7, image, filt, out)
    with pytest.raises(cc.CacnnError):
        cc.cacnn_pool_forward(POOL, 0, 9, image, pooled)
    with pytest.raises(cc.CacnnError):
        cc.cacnn_conv_forward(cc.Problem(4, 8, 6, 5, 7, 3, 3, 0, 1), 0, image, filt, out)
