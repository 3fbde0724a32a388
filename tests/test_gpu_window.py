"""GPU parity of the bf16 kernels that keep a tile's window in LDS (csrc/cacnn_window.hip) against the fp64 oracle, every tile shape on the
sizes where its indexing can go wrong."""
import ctypes

import numpy as np
import pytest

import cacnn_inputs as ci
from tests import gpu_util as gu
from tests.test_gpu_flat import GUARD, check, env  # noqa: F401

pytestmark = pytest.mark.gpu


def shapes_of(lib):
    """(index, images of a tile, its positions) of every window kernel"""
    for i in range(lib.cacnn_internal_window_count()):
        x = (ctypes.c_int32 * 5)()
        assert lib.cacnn_internal_window_info(i, x) == 0
        yield i, x[4], x[3] * x[1] * 32 // x[4]


def run(env, cfg, img, flt, index, tw, bufs, misalign_filter=0, out_offset=0):  # noqa: F811
    cc, torch, lib = env
    lib.cacnn_internal_window_forward.argtypes = [ctypes.POINTER(cc.Problem)] + [ctypes.c_int] * 3 + [ctypes.c_void_p] * 4
    d_img = gu.upload(cfg, img, flt, torch)[0]
    d_flt = gu.upload(cfg, img, flt, torch, misalign=misalign_filter)[1]
    n, first = int(np.prod(cfg.out_shape)), GUARD + out_offset
    words = torch.full((first + n + GUARD,), -7.0, dtype=torch.float32, device="cuda:0")
    out = words[first:first + n]
    out.fill_(float("nan"))
    rc = lib.cacnn_internal_window_forward(ctypes.byref(cc.Problem(*cfg.dims)), index, tw, bufs, d_img.data_ptr(), d_flt.data_ptr(),
                                           out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((words[:first] == -7.0).all()) and bool((words[first + n:] == -7.0).all()), (cfg.dims, index, tw, bufs)
    return rc, out.cpu().numpy().reshape(cfg.out_shape)


# C, K, W, H, R, S, sw, sh: filter columns of one chunk, of one and a row, of several with a masked one; one r and many; an odd and an even
# number of chunks; K below, at and beyond a tile; outputs smaller than a tile in either direction and not a multiple of it; strides, also
# beyond the filter's extent; 1 x 1
SHAPES = [(8, 5, 3, 2, 1, 1, 1, 1), (1, 33, 17, 9, 3, 9, 1, 2), (3, 32, 9, 11, 7, 7, 2, 2), (4, 64, 33, 3, 2, 2, 1, 1), (1, 40, 2, 35, 11, 11, 4, 4),
          (5, 70, 6, 7, 1, 3, 3, 4), (16, 31, 5, 5, 3, 3, 1, 1)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_every_window_tile_on_edge_shapes(env, shape):  # noqa: F811
    lib, ran = env[2], 0
    for index, images, positions in shapes_of(lib):
        # a tile's images, a tile and part of one, fewer than a tile
        for B in sorted({images, images + 8, 8}):
            cfg = ci.custom("window", B, *shape, dtype="bf16", dist="normal", seed=80 + B)
            img, flt = ci.make_inputs(cfg)
            ref, ab = gu.oracle_full(cfg, img, flt)
            tw = positions
            while tw >= 1:
                for bufs in (1, 2):
                    print(f"[window] kernel {index} {cfg.dims} tw {tw} bufs {bufs}", flush=True)
                    rc, out = run(env, cfg, img, flt, index, tw, bufs, misalign_filter=bufs - 1, out_offset=tw % 3)
                    if rc == 3:         # the box is too large
                        continue
                    assert rc == 0
                    check(cfg, out, ref, ab, f"kernel {index} tw {tw} bufs {bufs}")
                    ran += 1
                tw //= 2
    assert ran > 0


def test_many_tiles_per_workgroup(env):  # noqa: F811
    """Workgroups that walk several position tiles, with two boxes in turn, and the last round partly filled; Out in whole lines and not."""
    lib = env[2]
    for index, images, positions in shapes_of(lib):
        cfg = ci.custom("window", images, 3, 33, 75, 128 // images * 9 + 1, 3, 3, 1, 1, dtype="bf16", dist="normal", seed=7)
        img, flt = ci.make_inputs(cfg)
        ref, ab = gu.oracle_full(cfg, img, flt)
        for bufs in (1, 2):
            print(f"[window] kernel {index} {cfg.dims} bufs {bufs}", flush=True)
            for out_offset in (0, 1):
                rc, out = run(env, cfg, img, flt, index, max(1, positions // 8), bufs, out_offset=out_offset)
                assert rc == 0
                check(cfg, out, ref, ab, f"kernel {index} bufs {bufs}")


def test_values_that_are_not_finite_stay_where_they_belong(env):  # noqa: F811
    """A NaN or an infinity of the Image reaches the outputs whose window holds it and no other, one of the Filter its output channel."""
    cc, torch, lib = env
    dims = (16, 3, 40, 20, 37, 7, 7, 2, 2)
    cfg = ci.custom("window", *dims, dtype="bf16", dist="normal", seed=4)
    img, flt = ci.make_inputs(cfg)
    img, flt = img.copy(), flt.copy()
    img[9, 20, 1, 5] = np.nan
    img[30, 3, 2, 0] = np.inf
    flt[7, 3, 2, 1] = np.inf
    hit = np.zeros(cfg.out_shape, dtype=bool)
    for x, y, b in ((9, 20, 5), (30, 3, 0)):
        for h in range(cfg.H):
            for w in range(cfg.W):
                if 0 <= x - 2 * w < 7 and 0 <= y - 2 * h < 7:
                    hit[:, h, w, b] = True
    hit[7] = True
    for index, images, positions in shapes_of(lib):
        if images > 16:
            continue
        for tw in (positions, positions // 4, 1):
            for bufs in (1, 2):
                rc, out = run(env, cfg, img, flt, index, tw, bufs)
                assert rc == 0
                assert np.array_equal(~np.isfinite(out), hit), (index, tw, bufs)


def test_window_kernels_refuse_what_they_cannot_hold(env):  # noqa: F811
    cc, torch, lib = env
    for index, images, positions in shapes_of(lib):
        for dims in ((images + 4, 3, 8, 4, 4, 3, 3, 1, 1), (images, 2, 8, 4, 4, 3, 3, 1, 1), (images, 512, 8, 40, 40, 3, 3, 1, 1)):
            cfg = ci.custom("window", *dims, dtype="bf16", dist="normal", seed=1)
            img, flt = ci.make_inputs(cfg)
            assert run(env, cfg, img, flt, index, positions, 1)[0] == 3
