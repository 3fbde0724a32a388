"""GPU parity of the flattened kernels whose workgroups share a tile's contraction, against the fp64 oracle: every staged kernel, parts of
equal and of unequal length, and the calls of cacnn_conv_forward that are routed to them."""
import ctypes
import threading

import numpy as np
import pytest

import cacnn_inputs as ci
from tests import gpu_util as gu
from tests.test_gpu_flat import GUARD, check, env, kernels  # noqa: F401

pytestmark = pytest.mark.gpu


def split(env, cfg, img, flt, index, parts, misalign=0, out_offset=0):  # noqa: F811
    cc, torch, lib = env
    lib.cacnn_internal_split_forward.argtypes = [ctypes.POINTER(cc.Problem), ctypes.c_int, ctypes.c_int, ctypes.c_int] + [ctypes.c_void_p] * 3
    d_img, d_flt = gu.upload(cfg, img, flt, torch, misalign=misalign)
    n, first = int(np.prod(cfg.out_shape)), GUARD + out_offset
    words = torch.full((first + n + GUARD,), -7.0, dtype=torch.float32, device="cuda:0")
    out = words[first:first + n]
    out.fill_(float("nan"))
    torch.cuda.synchronize()
    rc = lib.cacnn_internal_split_forward(ctypes.byref(cc.Problem(*cfg.dims)), gu.dtype_code(cfg), index, parts, d_img.data_ptr(),
                                          d_flt.data_ptr(), out.data_ptr())
    torch.cuda.synchronize()
    assert bool((words[:first] == -7.0).all()) and bool((words[first + n:] == -7.0).all()), (cfg.dims, index)
    return rc, out.cpu().numpy().reshape(cfg.out_shape)


# C, K, W, H, R, S, sw, sh with contractions of two to some fifty stages: filter rows that are and are not whole chunks, K and positions
# beyond and below a tile, one tile and several
SHAPES = [(131, 20, 2, 3, 1, 3, 1, 1), (70, 33, 3, 2, 3, 3, 1, 1), (64, 130, 5, 7, 3, 3, 2, 2), (601, 5, 3, 1, 2, 1, 1, 2)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_every_staged_kernel_in_parts(env, dtype, shape):  # noqa: F811
    lib, ran, cases = env[2], 0, {}
    for index, images, exactly, lds in kernels(lib, dtype):
        if not lds:
            continue
        for B in ((images,) if exactly else (images, 37)):
            if B not in cases:
                cfg = ci.custom("split", B, *shape, dtype=dtype, dist="normal", seed=60 + B)
                img, flt = ci.make_inputs(cfg)
                cases[B] = (cfg, img, flt) + gu.oracle_full(cfg, img, flt)
            cfg, img, flt, ref, ab = cases[B]
            print(f"[split] kernel {index} {dtype} {cfg.dims}", flush=True)
            for parts in (2, 3, 7, 64):      # (64: one stage a part)
                rc, out = split(env, cfg, img, flt, index, parts, misalign=parts % 2, out_offset=parts % 5)
                if rc == 3:                  # a contraction of one stage
                    continue
                assert rc == 0
                check(cfg, out, ref, ab, f"kernel {index} parts {parts}")
                again = split(env, cfg, img, flt, index, parts, misalign=parts % 2, out_offset=parts % 5)[1]
                assert np.array_equal(out, again), "the sums are added in a fixed order"
                ran += 1
    assert ran > 0


# routed calls: the null stream runs the divided kernel, another stream and a graph the undivided one, and all agree
@pytest.mark.parametrize("dtype,dims", [("f32", (4, 200, 40, 6, 5, 3, 3, 1, 1)), ("bf16", (24, 700, 19, 5, 5, 3, 3, 1, 1)), ("bf16", (3, 400, 70, 9, 5, 3, 3, 2, 2))])
def test_streams_graphs_and_threads(env, dtype, dims):  # noqa: F811
    cc, torch, _ = env
    from paper_1802_06905_amd import binding
    cfg = ci.custom("split", *dims, dtype=dtype, dist="normal", seed=3)
    img, flt = ci.make_inputs(cfg)
    ref, ab = gu.oracle_full(cfg, img, flt)
    dt = gu.dtype_code(cfg)
    assert binding.routed_split(cfg.dims, dt) is not None
    d_img, d_flt = gu.upload(cfg, img, flt, torch)
    n = int(np.prod(cfg.out_shape))
    outs = [torch.full((n,), float("nan"), dtype=torch.float32, device="cuda:0") for _ in range(8)]
    host = lambda t: t.cpu().numpy().reshape(cfg.out_shape)  # noqa: E731
    for _ in range(3):
        cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, outs[0])
        torch.cuda.synchronize()
        check(cfg, host(outs[0]), ref, ab, "null stream")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(3):
            cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, outs[1])
    torch.cuda.synchronize()
    check(cfg, host(outs[1]), ref, ab, "side stream")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, outs[2])
    for _ in range(3):
        outs[2].fill_(float("nan"))
        graph.replay()
        cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, outs[3])     # beside a replay on the null stream
        torch.cuda.synchronize()
        assert np.array_equal(host(outs[2]), host(outs[1])) and np.array_equal(host(outs[3]), host(outs[0]))

    def work(out):
        torch.cuda.set_device(0)
        for _ in range(50):
            cc.cacnn_conv_forward(cfg.dims, dt, d_img, d_flt, out, stream=0)

    threads = [threading.Thread(target=work, args=(o,)) for o in outs[4:]]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert all(np.array_equal(host(o), host(outs[0])) for o in outs[4:])


def test_non_finite_values_stay_where_they_belong(env):  # noqa: F811
    """An infinity in one channel's Filter reaches that channel alone, through whichever part it lies in."""
    cc, torch, _ = env
    dims = (4, 200, 40, 6, 5, 3, 3, 1, 1)
    cfg = ci.custom("split", *dims, dtype="f32", dist="normal", seed=9)
    img, flt = ci.make_inputs(cfg)
    flt = flt.copy()
    flt[7, 2, 1, 150] = np.inf
    d_img, d_flt = gu.upload(cfg, img, flt, torch)
    out = torch.zeros(int(np.prod(cfg.out_shape)), dtype=torch.float32, device="cuda:0")
    cc.cacnn_conv_forward(cfg.dims, 0, d_img, d_flt, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(cfg.out_shape)
    assert not np.isfinite(got[7]).any() and np.isfinite(np.delete(got, 7, axis=0)).all()


def test_different_problems_one_behind_the_other(env):  # noqa: F811
    """Launches of different problems without a wait between them use the same scratch memory and counters, with other numbers of tiles, of parts and
    of sums: each gives the bits that it gives alone."""
    cc, torch, _ = env
    from paper_1802_06905_amd import binding
    problems = [("f32", (4, 200, 40, 6, 5, 3, 3, 1, 1)), ("bf16", (24, 700, 19, 5, 5, 3, 3, 1, 1)), ("bf16", (3, 400, 70, 9, 5, 3, 3, 2, 2)), ("f32", (1, 784, 64, 3, 12, 3, 3, 1, 1)),
                ("bf16", (72, 976, 16, 5, 5, 3, 3, 2, 2)), ("bf16", (3, 859, 480, 42, 5, 3, 3, 2, 2))]
    calls, kinds = [], set()
    for dtype, dims in problems:
        cfg = ci.custom("split", *dims, dtype=dtype, dist="normal", seed=12)
        img, flt = ci.make_inputs(cfg)
        _, parts, workgroups = binding.routed_split(dims, gu.dtype_code(cfg))
        kinds.add((parts, workgroups // parts))
        alone = torch.full((int(np.prod(cfg.out_shape)),), float("nan"), dtype=torch.float32, device="cuda:0")
        calls.append((cfg, *gu.upload(cfg, img, flt, torch), alone))
        cc.cacnn_conv_forward(dims, gu.dtype_code(cfg), *calls[-1][1:], stream=0)
        torch.cuda.synchronize()
        check(cfg, alone.cpu().numpy().reshape(cfg.out_shape), *gu.oracle_full(cfg, img, flt), "alone")
    assert len(kinds) == len(problems)
    order = np.random.default_rng(2).integers(0, len(calls), 120)
    outs = [torch.full_like(calls[i][3], float("nan")) for i in order]
    torch.cuda.synchronize()
    for i, out in zip(order, outs):
        cfg, d_img, d_flt, _ = calls[i]
        cc.cacnn_conv_forward(cfg.dims, gu.dtype_code(cfg), d_img, d_flt, out, stream=0)
    torch.cuda.synchronize()
    for n, (i, out) in enumerate(zip(order, outs)):
        assert torch.equal(out, calls[i][3]), (n, calls[i][0].dims)
