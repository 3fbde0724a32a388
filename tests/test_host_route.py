"""Which kernel cacnn_conv_forward launches (host only: nothing is enqueued): the layers that stay on the variants with box tiles, those that
go to the kernels with flattened positions, and that a call that cannot be planned is still refused."""
import ctypes

import pytest

import cacnn_inputs as ci
import paper_1802_06905_amd as cc
from paper_1802_06905_amd import binding

F32, BF16 = cc.CACNN_F32, cc.CACNN_BF16_F32ACC


def routed(dims, dtype, image=0, filt=0):
    name, workgroups, threads = binding.routed_kernel(dims, dtype, image, filt)
    assert workgroups >= 1 and workgroups * threads < 2 ** 32       # what a launch can hold
    return name


@pytest.mark.parametrize("name", ["c2", "c3", "c4", "c5"])
def test_fixed_geometry_layers_run_their_planned_variant(name):
    cfg = ci.CONFIGS[name]
    dtype = F32 if cfg.dtype == "f32" else BF16
    assert routed(cfg.dims, dtype) == cc.cacnn_variant_name(cc.cacnn_tile_plan(cfg.dims, dtype).variant)
    # operands that are not 16-byte aligned rule out the kernels that need it, whichever of the two it is
    for image, filt in ((4, 0), (0, 8), (4, 4)):
        assert " flat " in routed(cfg.dims, dtype, image, filt)
    assert " flat " not in routed(cfg.dims, dtype)                  # (and nothing of that is remembered for aligned ones)


# one image, images that 16-byte items do not divide, channels that they do not divide, few tiles
@pytest.mark.parametrize("dtype,dims", [(F32, (1, 3, 8, 16, 16, 3, 3, 1, 1)), (F32, (5, 30, 50, 27, 19, 5, 5, 1, 1)),
                                        (BF16, (1, 128, 128, 28, 28, 3, 3, 1, 1)), (BF16, (16, 3, 64, 112, 112, 7, 7, 2, 2)),
                                        (BF16, (3, 367, 237, 15, 15, 3, 3, 1, 1)), (BF16, (64, 30, 64, 14, 14, 3, 3, 1, 1)),
                                        (F32, (64, 1, 48, 28, 28, 3, 3, 1, 1)), (BF16, (8, 512, 512, 7, 7, 1, 1, 1, 1))])
def test_small_and_ragged_layers_run_flattened(dtype, dims):
    assert " flat " in routed(dims, dtype)


# filter rows shorter than 16 bytes: one large fp32 image is the case where box tiles are faster (up to 1.5 times)
@pytest.mark.parametrize("C,R,S", [(1, 1, 1), (3, 1, 1), (1, 3, 3), (2, 7, 1)])
def test_one_large_image_with_short_filter_rows(C, R, S):
    for K in (1, 40):
        assert " flat " not in routed((1, C, K, 1000, 1000, R, S, 1, 1), F32)
        assert " flat " not in routed((1, C, K, 250, 400, R, S, 1, 1), F32)
        assert " flat " in routed((1, C, K, 250, 399, R, S, 1, 1), F32)
        assert " flat " in routed((2, C, K, 1000, 1000, R, S, 1, 1), F32)
        assert " flat " in routed((1, C, K, 12, 10000, R, S, 1, 1), F32) and " flat " in routed((1, C, K, 10000, 12, R, S, 1, 1), F32)
        assert " flat " in routed((1, C, K, 1000, 1000, R, S, 1, 1), BF16)
    assert " flat " in routed((1, 4, 40, 1000, 1000, 1, 1, 1, 1), F32)


# windows that overlap in a bf16 Image of hundreds of MB stay on the fixed-geometry kernels (up to 1.7 times faster there); in fp32, in a
# smaller Image and without overlap the flattened kernels are faster
def test_large_bf16_images_with_overlapping_windows():
    for dims in ((16, 888, 24, 126, 126, 3, 3, 1, 1), (16, 1360, 3, 127, 127, 3, 3, 1, 1), (32, 152, 1, 151, 107, 1, 7, 1, 1), (64, 200, 8, 279, 279, 1, 7, 1, 1)):
        assert routed(dims, BF16) == cc.cacnn_variant_name(cc.cacnn_tile_plan(dims, BF16).variant)
    for dtype, dims in ((F32, (32, 256, 3, 76, 76, 3, 3, 1, 1)), (BF16, (8, 464, 76, 97, 97, 3, 3, 1, 1)), (BF16, (40, 56, 2, 345, 345, 1, 1, 1, 1))):
        assert " fx" in cc.cacnn_variant_name(cc.cacnn_tile_plan(dims, dtype).variant) and " flat " in routed(dims, dtype)


@pytest.mark.parametrize("dtype,dims", [(F32, (128, 9, 8, 700, 700, 3, 3, 1, 1)), (BF16, (250, 9, 8, 700, 700, 3, 3, 1, 1))])
def test_an_image_of_two_gib_stays_on_box_tiles(dtype, dims):
    problem = cc.Problem(*dims)
    assert problem.IW * problem.IH * problem.C * problem.B * (4 if dtype == F32 else 2) >= 2 ** 31
    assert routed(dims, dtype) == cc.cacnn_variant_name(cc.cacnn_tile_plan(dims, dtype).variant)
    below = (dims[0] // 2,) + dims[1:]
    assert " flat " in routed(below, dtype)


@pytest.mark.parametrize("dims", [(1, 1, 1, 24000, 24000, 1, 1, 1, 1), (1, 1, 1, 20000, 20000, 1, 8, 1, 1)])
def test_flattened_kernels_decline_launches_of_2_32_threads(dims):
    """They have one workgroup per tile: with small tiles and an Out of 2^28 words and more the threads of a launch would not fit 32 bits."""
    lib = binding._lib
    lib.cacnn_internal_flat_us.restype = ctypes.c_double
    lib.cacnn_internal_flat_us.argtypes = [ctypes.POINTER(cc.Problem), ctypes.c_int, ctypes.c_int]
    problem, taken, declined = cc.Problem(*dims), 0, 0
    for i in range(lib.cacnn_internal_flat_count()):
        x = (ctypes.c_int32 * 8)()
        assert lib.cacnn_internal_flat_info(i, x) == 0
        dtype, mb, ng, im, wm, wn, wk, nch = x
        if dtype != BF16 or im not in (1, -1) or (nch and dims[1] * dims[6] < 8):
            continue
        tiles = -(-dims[3] * dims[4] // (32 * ng * wn))                # (one output channel, one image)
        fits = tiles * 64 * wm * wn * wk < 2 ** 32
        assert (lib.cacnn_internal_flat_us(ctypes.byref(problem), BF16, i) > 0) == fits
        taken, declined = taken + fits, declined + (not fits)
    assert taken and declined
    routed(dims, BF16)


@pytest.mark.parametrize("dtype,dims", [(BF16, (1, 1, 1, 30000, 30000, 1, 1, 1, 1)), (BF16, (1, 1, 1, 16384, 2 ** 15, 1, 8, 1, 1))])
def test_a_tile_list_beyond_the_index_range_is_refused(dtype, dims):
    with pytest.raises(cc.CacnnError):
        binding.routed_kernel(dims, dtype)


def test_arguments_out_of_range_are_refused():
    for dims, dtype in (((1, 3, 8, 16, 16, 3, 3, 1, 1), 2), ((1, 0, 8, 16, 16, 3, 3, 1, 1), F32), ((2 ** 31, 3, 8, 16, 16, 3, 3, 1, 1), F32)):
        with pytest.raises(cc.CacnnError):
            binding.routed_kernel(dims, dtype)


def test_the_launch_cache_is_safe_with_several_threads():
    """More problems than the cache holds, from eight threads at once (ctypes lets go of the interpreter's lock in a call): every answer is the
    one that a single thread gets."""
    import threading
    problems = [((b, c, 24, 9, 7, 3, 3, 1, 1), dtype) for b in (1, 3, 8, 32, 64) for c in (1, 3, 8, 16, 24, 32, 48, 64, 65, 100) for dtype in (F32, BF16)]
    want = [binding.routed_kernel(*p) for p in problems]
    wrong = []

    def work(first):
        for i in range(2 * len(problems)):
            n = (first * 13 + i * 7) % len(problems)
            if binding.routed_kernel(*problems[n]) != want[n]:
                wrong.append(problems[n])

    threads = [threading.Thread(target=work, args=(t,)) for t in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(set(want)) > 5 and not wrong


def pool_images(dims, dtype, image=0, out=0):
    lib = binding._lib
    lib.cacnn_internal_pool_images.argtypes = [ctypes.POINTER(cc.Problem), ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    return lib.cacnn_internal_pool_images(ctypes.byref(cc.Problem(*dims)), dtype, image, out)


def test_images_per_thread_of_a_pooling_call():
    """One 16-byte load's images, fewer where B or an address asks for it; bf16 rows of whole cache lines: half as many, but for windows whose
    overlap has the loads set the pace."""
    def at(B, R, S, sw, sh, dtype, image=0, out=0):
        return pool_images((B, 40, 40, 20, 20, R, S, sw, sh), dtype, image, out)
    for B, bf16, f32 in ((1, 1, 1), (3, 1, 1), (6, 2, 2), (20, 4, 4), (8, 8, 4)):
        assert (at(B, 3, 3, 1, 1, BF16), at(B, 3, 3, 1, 1, F32)) == (bf16, f32)
    assert [at(8, 3, 3, 1, 1, BF16, image) for image in (2, 4, 8, 16)] == [1, 2, 4, 8] and at(8, 3, 3, 1, 1, BF16, 0, 4) == 1
    for R, S, sw, sh in ((2, 2, 2, 2), (2, 2, 1, 1), (3, 3, 2, 2), (7, 7, 7, 7), (1, 1, 1, 1), (3, 1, 1, 1)):
        assert at(64, R, S, sw, sh, BF16) == 4 and at(64, R, S, sw, sh, F32) == 4
    for R, S, sw, sh in ((3, 3, 1, 1), (7, 7, 1, 1), (7, 8, 1, 2), (7, 7, 2, 2), (7, 1, 1, 1), (5, 5, 1, 1)):
        assert at(64, R, S, sw, sh, BF16) == 8 and at(64, R, S, sw, sh, F32) == 4
    # (4 images per thread only where the kernel's divisions hold as many threads)
    assert pool_images((32, 7000, 7000, 1, 1, 2, 2, 1, 1), BF16) == 4 and pool_images((32, 30000, 30000, 1, 1, 2, 2, 1, 1), BF16) == 8
    assert pool_images((64, 40, 39, 20, 20, 2, 2, 2, 2), BF16) == 0


# Workgroups share a tile's contraction where few tiles have a long one; their sums and tiles fit the scratch memory, and where the tiles
# fill the device or the contraction is short nothing is divided.
def test_long_contractions_of_few_tiles_are_divided():
    for dtype, dims in ((F32, (1, 784, 64, 3, 12, 3, 3, 1, 1)), (BF16, (72, 976, 16, 5, 5, 3, 3, 2, 2)), (BF16, (3, 859, 480, 42, 5, 3, 3, 2, 2))):
        name, parts, workgroups = binding.routed_split(dims, dtype)
        assert " flat " in name and not name.endswith(" c0") and parts >= 2 and workgroups % parts == 0
        m, n, i, w, _ = name.split()[2:]
        wm, wn, _ = (int(x) for x in w[1:].split("x"))
        words = wm * int(m[1:]) * 32 * wn * int(n[1:]) * 32 * max(1, -int(i[1:]))
        assert workgroups * words <= 2 ** 21 and workgroups // parts <= 4096
    for dtype, dims in ((F32, (1, 3, 8, 16, 16, 3, 3, 1, 1)), (BF16, (1, 128, 128, 28, 28, 3, 3, 1, 1)), (BF16, (16, 3, 64, 112, 112, 7, 7, 2, 2)),
                        (F32, (64, 64, 64, 56, 56, 1, 1, 1, 1)), (F32, (7, 1, 8, 5, 5, 1, 1, 1, 1))):
        assert binding.routed_split(dims, dtype) is None


# A tile's window in LDS: first layers of few channels with whole rows of images, where the time before the first product is small beside the
# rest; not for other batches, Images that 16-byte loads cannot read, or a last round of tiles that is mostly empty.
def test_first_layers_keep_their_window_in_lds():
    for dims in ((16, 3, 64, 112, 112, 7, 7, 2, 2), (32, 3, 64, 112, 112, 7, 7, 2, 2), (256, 3, 16, 98, 98, 5, 5, 1, 1)):
        assert " flat window " in routed(dims, BF16)
        assert " flat window " not in routed(dims, BF16, image=8) and " flat " in routed(dims, BF16, image=8)
        assert " flat window " in routed(dims, BF16, filt=2)
        assert " flat window " not in routed(dims, F32)
    for dims in ((8, 3, 64, 56, 56, 7, 7, 2, 2), (40, 3, 64, 112, 112, 7, 7, 2, 2), (16, 2, 64, 112, 112, 7, 3, 2, 2), (64, 3, 59, 33, 72, 5, 5, 1, 1)):
        assert " flat window " not in routed(dims, BF16) and " flat " in routed(dims, BF16)


# Layers whose plan is a fixed-geometry variant and that measurements give to the flattened kernels, and some that they leave where they are
def test_short_launches_of_fixed_geometry_variants_run_flattened():
    for dtype, dims in ((F32, (256, 32, 498, 81, 3, 1, 1, 1, 1)), (F32, (128, 512, 64, 15, 15, 1, 1, 2, 2)), (BF16, (256, 32, 16, 36, 43, 1, 1, 1, 1)),
                        (BF16, (8, 88, 96, 77, 77, 1, 1, 2, 2))):
        assert " fx" in cc.cacnn_variant_name(cc.cacnn_tile_plan(dims, dtype).variant) and " flat " in routed(dims, dtype)
    for dtype, dims in ((F32, (8, 64, 64, 56, 56, 3, 3, 1, 1)), (BF16, (64, 64, 256, 56, 56, 1, 1, 1, 1)), (BF16, (32, 128, 256, 28, 28, 3, 3, 2, 2)),
                        (BF16, (128, 400, 224, 26, 5, 3, 3, 1, 1)), (BF16, (32, 96, 206, 42, 42, 3, 3, 1, 1)), (F32, (8, 320, 496, 37, 7, 3, 3, 1, 1))):
        assert routed(dims, dtype) == cc.cacnn_variant_name(cc.cacnn_tile_plan(dims, dtype).variant)


# The corrected comparison of the two estimates knows no largest size: what a layer of 240 MB or 7 GFLOP is given to, a larger one is as well
@pytest.mark.parametrize("dtype,dims,sizes", [(F32, (256, 32, 498, 0, 3, 1, 1, 1, 1), (81, 155, 170)),
                                              (F32, (256, 32, 498, 81, 0, 1, 1, 1, 1), (3, 5, 6, 7, 9)),
                                              (F32, (128, 512, 64, 0, 0, 1, 1, 2, 2), (26, 30, 32, 38, 44)),
                                              (F32, (128, 512, 64, 0, 15, 1, 1, 2, 2), (40, 60, 70, 80)),
                                              (F32, (64, 52, 0, 5, 54, 7, 1, 1, 1), (400, 1216, 1600)),
                                              (BF16, (256, 24, 2, 0, 0, 1, 1, 1, 1), (90, 120, 145, 200)), (BF16, (56, 56, 7, 0, 0, 1, 1, 1, 1), (100, 179, 250))])
def test_a_larger_layer_stays_on_the_kernel_of_the_smaller_one(dtype, dims, sizes):
    for n in sizes:
        grown = tuple(n if d == 0 else d for d in dims)
        assert " fx" in cc.cacnn_variant_name(cc.cacnn_tile_plan(grown, dtype).variant) and " flat " in routed(grown, dtype), grown
