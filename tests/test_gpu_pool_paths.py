"""GPU parity of the pooling kernels where a call's sizes choose between them: images per thread (1, 2, 4, 8 by what divides B and by
the pointers' alignment), windows compiled in and batches of any other, and Images beyond a buffer descriptor's 2 GiB."""
import numpy as np
import pytest

import cacnn_inputs as ci
from oracle import conv as oconv
from oracle import pool as opool
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_1802_06905_amd as cc
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return cc, torch


# B: 1, 2, 4 and 8 images per thread (fp32: at most 4), whole cache lines; R x S: the compiled windows, one element, batches of 8, 4
# and 1 with and without remainders, a window of one row and one column
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B", [1, 3, 6, 20, 8, 64])
def test_images_per_thread_and_windows(env, dtype, B):
    cc, torch = env
    for R, S, sw, sh in [(3, 3, 2, 2), (3, 3, 1, 1), (2, 2, 2, 2), (1, 1, 1, 1), (2, 3, 1, 2), (1, 4, 1, 1), (8, 1, 1, 1), (5, 5, 2, 1), (7, 7, 7, 7)]:
        cfg = ci.custom("pool", B, 5, 5, 4, 3, R, S, sw, sh, dtype=dtype, dist="uniform", seed=60 + B)
        img, flt = ci.make_inputs(cfg)
        for misalign in (0, 1, 2):
            d_img, _ = gu.upload(cfg, img, flt, torch, misalign=misalign)
            for mode, name in ((1, "max"), (0, "avg")):
                print(f"[pool] {dtype} {cfg.dims} {name} misalign {misalign}", flush=True)
                out = torch.full((int(np.prod(cfg.out_shape)),), float("nan"), device="cuda:0")
                cc.cacnn_pool_forward(cfg.dims, gu.dtype_code(cfg), mode, d_img, out)
                torch.cuda.synchronize()
                got = out.cpu().numpy().reshape(cfg.out_shape).astype(np.float64)
                ref = opool.pool_fp64(oconv.Problem(*cfg.dims), img, name)
                if name == "max":
                    assert np.array_equal(got, ref)
                else:
                    # R*S roundings of partial sums of values below 1 in size, and that of the division
                    assert np.max(np.abs(got - ref)) <= (R * S + 1) * 2.0 ** -24


# rows of whole cache lines: 4 images per thread, and 8 where the thread count at 4 would pass the limit of the kernel's divisions
@pytest.mark.parametrize("C", [7000, 30000])
def test_streamed_output_at_the_thread_limit(env, C):
    cc, torch = env
    dims = (32, C, C, 1, 1, 2, 2, 1, 1)
    img = torch.empty(2, 2, C, 32, device="cuda:0", dtype=torch.bfloat16).uniform_(-1, 1)
    out = torch.full((C, 1, 1, 32), float("nan"), device="cuda:0")
    print(f"[pool] thread limit {dims}", flush=True)
    cc.cacnn_pool_forward(dims, 1, 1, img, out)
    ref = img.amax(dim=(0, 1)).float().view(C, 1, 1, 32)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


def test_image_beyond_two_gib(env):
    """Windows that do not overlap, so that the reference is a reshape: 2.2 GB of fp32 and of bf16."""
    cc, torch = env
    for dtype, tt, B in ((0, torch.float32, 256), (1, torch.bfloat16, 512)):
        dims = (B, 16, 16, 52, 52, 7, 7, 7, 7)
        img = torch.empty(364, 364, 16, B, device="cuda:0", dtype=tt).uniform_(-1, 1)
        assert img.numel() * img.element_size() > 2 ** 31
        out = torch.full((16, 52, 52, B), float("nan"), device="cuda:0")
        print(f"[pool] beyond 2 GiB {dims} {tt}", flush=True)
        cc.cacnn_pool_forward(dims, dtype, 1, img, out)
        ref = img.view(52, 7, 52, 7, 16, B).amax(dim=(1, 3)).permute(2, 1, 0, 3).float()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        del img, out, ref
