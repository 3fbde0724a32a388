"""GPU parity of the fp32 stem kernel whose two sets of waves work on two tiles half a tile apart, against the fp64 oracle: one to seven tiles
per workgroup, of which the sets get different numbers, and tiles that overhang Out in every direction."""
import numpy as np
import pytest

import cacnn_inputs as ci
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# B, K, W, H: workgroups with one tile, with none or one, with one or two, two or three, three or four, six or seven; K below and at a tile (above
# it another kernel runs); odd extents and batches that fill a tile in part
SHAPES = [(32, 64, 2, 2), (32, 64, 30, 32), (32, 64, 32, 36), (64, 64, 34, 34), (32, 33, 59, 57), (36, 64, 41, 43), (4, 5, 3, 1), (64, 64, 56, 58), (32, 65, 9, 8)]


@pytest.mark.parametrize("b,k,w,h", SHAPES)
def test_stem_on_sizes_around_whole_rounds(b, k, w, h):
    import torch
    import paper_1802_06905_amd as cc
    cfg = ci.custom("stem", b, 3, k, w, h, 7, 7, 2, 2, dtype="f32", dist="normal", seed=w + h)
    img, flt = ci.make_inputs(cfg)
    d_img, d_flt = gu.upload(cfg, img, flt, torch)
    n, guard = int(np.prod(cfg.out_shape)), 64
    words = torch.full((n + 2 * guard,), -7.0, dtype=torch.float32, device="cuda:0")
    out = words[guard:guard + n]
    plan = cc.cacnn_tile_plan(cfg.dims, 0)
    plan.variant = [i for i in range(cc.cacnn_variant_count()) if cc.cacnn_variant_name(i).startswith("f32 fxsd ")][0]
    plan.b_c, plan.b_r, plan.b_s = 3, 7, 7
    ref, ab = gu.oracle_full(cfg, img, flt)
    for _ in range(3):
        out.fill_(float("nan"))
        cc.cacnn_conv_forward_with_plan(cfg.dims, 0, plan, d_img, d_flt, out)
        torch.cuda.synchronize()
        assert bool((words[:guard] == -7.0).all()) and bool((words[guard + n:] == -7.0).all())
        # one rounding of 2^-24 for a product and one for its addition, relative to the sum of absolute products
        assert gu.rel_err(out.cpu().numpy().reshape(cfg.out_shape), ref, ab) <= 2 * 147 * 2.0 ** -24
