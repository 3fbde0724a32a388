"""GPU parity of the kernels with flattened positions (csrc/cacnn_flat.hip) against the fp64 oracle: every compiled one on the
sizes where its indexing can go wrong, whatever the library would choose for such a call."""
import ctypes

import numpy as np
import pytest

import cacnn_inputs as ci
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_1802_06905_amd as cc
    from paper_1802_06905_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib = binding._lib
    lib.cacnn_internal_flat_forward.argtypes = [ctypes.POINTER(cc.Problem), ctypes.c_int, ctypes.c_int] + [ctypes.c_void_p] * 4
    lib.cacnn_internal_flat_info.argtypes = [ctypes.c_int, ctypes.POINTER(ctypes.c_int32)]
    return cc, torch, lib


def kernels(lib, dtype):
    """(index, images per group, whether that has to be all images, whether it stages in LDS) of every flattened kernel of the dtype"""
    for i in range(lib.cacnn_internal_flat_count()):
        x = (ctypes.c_int32 * 8)()
        assert lib.cacnn_internal_flat_info(i, x) == 0
        if x[0] == (0 if dtype == "f32" else 1):
            yield i, abs(x[3]), x[3] < 0, x[7] > 0


GUARD = 96      # words before and behind Out that a call must leave alone


def run(env, cfg, img, flt, index, misalign=0, out_offset=0):
    cc, torch, lib = env
    d_img, d_flt = gu.upload(cfg, img, flt, torch, misalign=misalign)
    n, first = int(np.prod(cfg.out_shape)), GUARD + out_offset
    words = torch.full((first + n + GUARD,), -7.0, dtype=torch.float32, device="cuda:0")
    out = words[first:first + n]
    out.fill_(float("nan"))
    prob = cc.Problem(*cfg.dims)
    rc = lib.cacnn_internal_flat_forward(ctypes.byref(prob), gu.dtype_code(cfg), index, d_img.data_ptr(), d_flt.data_ptr(),
                                         out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((words[:first] == -7.0).all()) and bool((words[first + n:] == -7.0).all()), (cfg.dims, index)
    return rc, out.cpu().numpy().reshape(cfg.out_shape)


def check(cfg, out, ref, ab, what):
    """The products of bf16 or fp32 inputs enter a sum of fp32 additions: at most one rounding of 2^-24 per product (fp32
    products are rounded as well: twice that), relative to the sum of absolute products."""
    tol = 2 * cfg.C * cfg.R * cfg.S * 2.0 ** -24
    e = gu.rel_err(out, ref, ab)
    assert e <= tol, f"{cfg.dims} {cfg.dtype} {what}: {e:.3e} > {tol:.3e}"


# C, K, W, H, R, S, sw, sh: a filter row (S*C contraction indices) shorter than, equal to, one more than and not a multiple of a
# 16-byte chunk; odd and even numbers of chunks, fewer chunks than waves; K and the positions beyond and below a tile; strides, also
# above the filter's extent; a Filter larger than the Image (the other tile order); one, two, several whole and partly filled LDS stages
SHAPES = [(3, 5, 3, 2, 2, 1, 1, 1), (1, 33, 4, 5, 3, 3, 2, 1), (8, 32, 1, 1, 1, 1, 1, 1), (9, 40, 5, 3, 1, 1, 1, 2), (5, 7, 6, 4, 3, 3, 1, 1),
          (16, 64, 3, 3, 3, 3, 2, 2), (7, 31, 2, 9, 4, 5, 3, 1), (50, 97, 2, 1, 2, 2, 1, 1), (4, 16, 11, 13, 1, 2, 2, 3), (24, 130, 9, 7, 1, 3, 1, 1),
          (131, 20, 2, 3, 1, 3, 1, 1), (64, 72, 3, 2, 3, 3, 1, 1)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_every_flat_kernel_on_edge_shapes(env, dtype, shape):
    lib, ran = env[2], 0
    cases = {}
    for index, images, exactly, lds in kernels(lib, dtype):
        # as many images as a group holds, one more, an odd number beyond a half-wave's lanes
        for B in ((images,) if exactly else (images, images + 1, 37)):
            if B not in cases:
                cfg = ci.custom("flat", B, *shape, dtype=dtype, dist="normal", seed=40 + B)
                img, flt = ci.make_inputs(cfg)
                cases[B] = (cfg, img, flt) + gu.oracle_full(cfg, img, flt)
            cfg, img, flt, ref, ab = cases[B]
            print(f"[flat] kernel {index} {dtype} {cfg.dims}", flush=True)
            for misalign in (0, 1):
                rc, out = run(env, cfg, img, flt, index, misalign)
                if rc == 3:     # a filter row shorter than a chunk
                    assert (exactly or lds) and shape[0] * shape[5] < (4 if dtype == "f32" else 8)
                    continue
                assert rc == 0
                check(cfg, out, ref, ab, f"kernel {index} misalign {misalign}")
                ran += 1
    assert ran > 0


# filter rows of 1 to 7 contraction indices, and of one whole chunk: the waves that share a tile have no step, one, two or several,
# the last of an odd number of columns fills half of one
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c,r,s", [(1, 1, 1), (1, 2, 2), (3, 1, 1), (1, 8, 3), (2, 11, 1), (5, 9, 1), (7, 17, 1), (1, 5, 7), (8, 1, 1), (4, 2, 2)])
def test_short_rows_and_single_steps(env, dtype, c, r, s):
    lib, ran = env[2], 0
    for index, images, exactly, lds in kernels(lib, dtype):
        if exactly or lds:
            continue
        for B in (images, 13):
            cfg = ci.custom("flat", B, c, 35, 7, 6, r, s, 2, 1, dtype=dtype, dist="normal", seed=70 + c)
            img, flt = ci.make_inputs(cfg)
            ref, ab = gu.oracle_full(cfg, img, flt)
            print(f"[flat] kernel {index} {dtype} {cfg.dims}", flush=True)
            for misalign in (0, 1):
                rc, out = run(env, cfg, img, flt, index, misalign)
                assert rc == 0
                check(cfg, out, ref, ab, f"kernel {index} misalign {misalign}")
                ran += 1
    assert ran > 0


# rows of Out that are whole cache lines, which the kernels that stage in LDS store past the L2 (where Out starts at a multiple of 64
# bytes: words 0 and 16 behind a line, not 1): one line in all, K beyond a tile, several tiles of positions with the last one partly filled
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(8, 5, 8, 4, 1, 1, 1, 1), (9, 65, 16, 10, 3, 3, 1, 1), (3, 33, 32, 33, 7, 7, 2, 2)], ids=lambda s: "x".join(map(str, s)))
def test_streamed_output_of_staged_kernels(env, dtype, shape):
    lib, ran = env[2], 0
    for index, images, exactly, lds in kernels(lib, dtype):
        if not lds or (exactly and images > 1):
            continue
        cfg = ci.custom("flat", images, *shape, dtype=dtype, dist="normal", seed=50 + images)
        img, flt = ci.make_inputs(cfg)
        ref, ab = gu.oracle_full(cfg, img, flt)
        print(f"[flat] kernel {index} {dtype} {cfg.dims}", flush=True)
        for out_offset in (0, 16, 1):
            rc, out = run(env, cfg, img, flt, index, out_offset=out_offset)
            assert rc == 0
            check(cfg, out, ref, ab, f"kernel {index} out {out_offset}")
        ran += 1
    assert ran > 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_flat_kernels_refuse_what_they_cannot_hold(env, dtype):
    cc, torch, lib = env
    for index, images, exactly, lds in kernels(lib, dtype):
        for B in (images - 1, images + 1) if exactly else (images - 1,):
            if B >= 1:
                cfg = ci.custom("flat", B, 16, 8, 2, 2, 1, 1, dtype=dtype, seed=3)
                rc, out = run(env, cfg, *ci.make_inputs(cfg), index)
                assert rc == 3 and np.isnan(out).all()
    cfg = ci.custom("flat", 1, 16, 8, 2, 2, 1, 1, dtype=dtype, seed=3)
    assert run(env, cfg, *ci.make_inputs(cfg), 10 ** 6)[0] == 3 and run(env, cfg, *ci.make_inputs(cfg), -1)[0] == 3


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c", [3, 11])
def test_nonfinite_inputs_stay_local_in_flat_kernels(env, dtype, c):
    """The last chunk of a filter row is moved back to end with the row, so that its first elements are multiplied by zero on both
    sides: an Inf or NaN in one of them, in the row behind it or in a neighbouring image must reach its own outputs only."""
    lib = env[2]
    for index, images, exactly, lds in kernels(lib, dtype):
        B = images if exactly else max(images, 2)
        dims = (B, c, 34, 4, 3, 2, 3 if exactly or lds else 1, 1, 2)
        cfg = ci.custom("flat_inf", *dims, dtype=dtype, dist="normal", seed=9)
        img0, flt = ci.make_inputs(cfg)
        _, _, K, W, H, R, S, sw, sh = dims
        for n, (x, y, ch, b) in enumerate([(0, 0, c - 1, 0), (1, 1, 0, B - 1), (2, 0, c // 2, B // 2), (img0.shape[0] - 1, img0.shape[1] - 1, c - 1, B - 1)]):
            img = img0.copy()
            img[x, y, ch, b] = np.inf if n % 2 == 0 else np.nan
            print(f"[flat] kernel {index} {dtype} {dims} non-finite at {(x, y, ch, b)}", flush=True)
            rc, out = run(env, cfg, img, flt, index)
            assert rc == 0
            want = np.zeros(cfg.out_shape, bool)
            for w in range(W):
                for h in range(H):
                    if 0 <= x - sw * w < R and 0 <= y - sh * h < S:
                        want[:, h, w, b] = True
            assert np.array_equal(~np.isfinite(out), want), (index, (x, y, ch, b))


def test_binding_refuses_short_device_tensors_and_uses_the_current_stream(env):
    """The binding leaves the length check of ordinary device tensors to the library: a buffer one element short is refused with the
    same error as before, before anything is enqueued, and a call without a stream goes to torch's current one."""
    cc, torch, _ = env
    cfg = ci.custom("binding", 4, 8, 8, 3, 3, 1, 1, dtype="f32", dist="normal", seed=5)
    img, flt = ci.make_inputs(cfg)
    d_img, d_flt = gu.upload(cfg, img, flt, torch)
    n = int(np.prod(cfg.out_shape))
    prob, out = cc.Problem(*cfg.dims), torch.full((n,), -7.0, device="cuda:0")
    for args in ((d_img[:-1], d_flt, out), (d_img, d_flt[:-1], out), (d_img, d_flt, out[:-1]), (d_img.to(torch.float16), d_flt, out)):
        with pytest.raises(ValueError):
            cc.cacnn_conv_forward(prob, 0, *args)
    pool = cc.Problem(4, 8, 8, 3, 3, 1, 1, 1, 1)
    with pytest.raises(ValueError):
        cc.cacnn_pool_forward(pool, 0, 1, d_img, out[:n - 1])
    torch.cuda.synchronize()
    assert bool((out == -7.0).all())
    side, first = torch.cuda.Stream(), torch.full((n,), float("nan"), device="cuda:0")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(2000000)                    # a millisecond of work that the call has to wait behind on its own stream
        cc.cacnn_conv_forward(prob, 0, d_img, d_flt, first)
        assert not side.query()
    side.synchronize()
    ref, ab = gu.oracle_full(cfg, img, flt)
    check(cfg, first.cpu().numpy().reshape(cfg.out_shape), ref, ab, "side stream")


# Image or Filter just below the 2 GiB that the 32-bit offsets reach: many images, one image, a long contraction
@pytest.mark.parametrize("dtype,dims", [("bf16", (32, 16, 5, 1446, 1446, 3, 3, 1, 1)), ("bf16", (1, 16, 3, 8188, 8190, 3, 1, 1, 1)),
                                        ("bf16", (2, 131071, 8191, 1, 1, 1, 1, 1, 1)), ("f32", (32, 16, 5, 1022, 1021, 3, 3, 1, 1)),
                                        ("f32", (1, 16, 3, 5790, 5790, 2, 2, 1, 1)), ("f32", (4, 65535, 8191, 1, 1, 1, 1, 1, 1))])
def test_operands_just_below_two_gib(env, dtype, dims):
    """Inputs of -1, 0 and 1, whose sums are exact: every output is written, and those at the corners and at drawn positions are right."""
    cc, torch, lib = env
    B, C, K, W, H, R, S, sw, sh = dims
    kind, esz = (torch.float32, 4) if dtype == "f32" else (torch.bfloat16, 2)
    img_shape, flt_shape = (sw * (W - 1) + R, sh * (H - 1) + S, C, B), (K, R, S, C)
    size = max(int(np.prod(img_shape, dtype=np.int64)), int(np.prod(flt_shape, dtype=np.int64))) * esz
    assert 0.99 * 2 ** 31 < size < 2 ** 31
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(12)
    img = torch.randint(-1, 2, img_shape, device="cuda:0", dtype=torch.int8, generator=gen).to(kind)
    flt = torch.randint(-1, 2, flt_shape, device="cuda:0", dtype=torch.int8, generator=gen).to(kind)
    words = torch.empty(K * H * W * B + 2 * GUARD, device="cuda:0")
    out = words[GUARD:-GUARD].view(K, H, W, B)
    rng = np.random.default_rng(3)
    at = sorted({(w, h) for w in (0, W // 2, W - 1) for h in (0, H // 2, H - 1)} | {(int(rng.integers(W)), int(rng.integers(H))) for _ in range(40)})
    windows = torch.stack([img[sw * w:sw * w + R, sh * h:sh * h + S].reshape(R * S * C, B) for w, h in at]).cpu().float()
    want = torch.matmul(flt.view(K, -1).cpu().float(), windows)                   # position, k, image; integers below 2^24
    prob, ran = cc.Problem(*dims), 0
    for index, images, exactly, lds in kernels(lib, dtype):
        if B < images or (exactly and B != images):
            continue
        words.fill_(-7.0)
        out.fill_(float("nan"))
        print(f"[flat] kernel {index} {dtype} {dims}", flush=True)
        rc = lib.cacnn_internal_flat_forward(ctypes.byref(prob), 0 if dtype == "f32" else 1, index, img.data_ptr(), flt.data_ptr(),
                                             out.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert rc == 0
        assert bool((words[:GUARD] == -7.0).all()) and bool((words[-GUARD:] == -7.0).all())
        assert not bool(torch.isnan(out).any())
        got = torch.stack([out[:, h, w] for w, h in at]).cpu()
        assert torch.equal(got, want), (index, dims)
        ran += 1
    assert ran >= 4
