"""What the library hands to the runtime, with a stand-in for the runtime (tests/hip_stand_in.cpp): nothing runs, no GPU is needed."""
import os
import subprocess
import sys

import pytest

import paper_1802_06905_amd as cc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (in a process of its own: the stand-in has to be there before the library looks for the runtime)
PRELUDE = r'''
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
hip.stand_in_launches.restype = ctypes.c_char_p
hip.stand_in_cost.argtypes = [ctypes.c_char_p, ctypes.c_double]
lib.cacnn_variant_name.restype = ctypes.c_char_p
V, I = ctypes.c_void_p, ctypes.c_int
IMAGE, FILTER, OUT = 1 << 20, 2 << 20, 3 << 20       # addresses that nothing reads
def problem(*dims): return ctypes.byref((ctypes.c_int64 * 9)(*dims))
def kernels(): return hip.stand_in_launches().decode().split()
def forward(dims, dtype, stream=0, image=IMAGE):
    assert lib.cacnn_conv_forward(problem(*dims), I(dtype), V(image), V(FILTER), V(OUT), V(stream)) == 0
    return kernels()
def tune(dims, dtype, stream=0, image=IMAGE):
    assert lib.cacnn_tune(problem(*dims), I(dtype), V(image), V(FILTER), V(OUT), V(stream), V(0)) == 0
    return kernels()
'''


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    stand_in = str(tmp_path_factory.mktemp("stand_in") / "hip_stand_in.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-o", stand_in, os.path.join(ROOT, "tests", "hip_stand_in.cpp"), "-ldl"], check=True)

    def program(body):
        p = subprocess.run([sys.executable, "-c", PRELUDE + body, stand_in, cc.library_path()], capture_output=True, text=True, timeout=120)
        assert p.returncode == 0, p.stdout + p.stderr
        return p.stdout
    return program


def test_tuning_times_the_window_kernels(run):
    """A first bf16 layer that runs on a window kernel untuned stays on one when it is tuned and they are the fastest, on every stream; an Image that
    16-byte loads cannot read is not tried on them."""
    run(r'''
stem = (16, 3, 64, 112, 112, 7, 7, 2, 2)
hip.stand_in_cost(b"conv_window", 1.0)
hip.stand_in_cost(b"conv_", 2.0)
assert "conv_window" in forward(stem, 1)[0]
untuned = forward(stem, 1)
for stream in (0, 4096):
    timed = tune(stem, 1, stream)
    assert set(untuned) <= set(timed) and any("conv_flat" in k for k in timed)
    for where in (0, 4096):
        assert "conv_window" in forward(stem, 1, where)[0]
assert not any("conv_window" in k for k in tune(stem, 1, 0, IMAGE + 8)) and "conv_window" not in forward(stem, 1, 0, IMAGE + 8)[0]
assert not any("conv_window" in k for k in tune(stem, 0))
''')


def test_tuning_leaves_a_window_kernel_for_a_faster_one(run):
    run(r'''
stem = (16, 3, 64, 112, 112, 7, 7, 2, 2)
hip.stand_in_cost(b"conv_flat_lds", 1.0)
hip.stand_in_cost(b"conv_", 2.0)
assert any("conv_window" in k for k in tune(stem, 1, 4096))
assert "conv_flat_lds" in forward(stem, 1, 4096)[0]
''')


def test_tuning_on_another_stream_leaves_the_null_stream_its_divided_kernel(run):
    """Workgroups share a contraction on the null stream alone, and a problem has one entry for all streams: what that stream ran, by estimate or by
    its own tuning, is what it runs after a tuning elsewhere, which cannot time it."""
    run(r'''
deep = (1, 784, 64, 3, 12, 3, 3, 1, 1)
hip.stand_in_cost(b"conv_", 1.0)
divided = forward(deep, 0)
assert "FlatSplitArgs" in divided[0] and "FlatSplitArgs" not in forward(deep, 0, 4096)[0]
assert not any("FlatSplitArgs" in k for k in tune(deep, 0, 4096))
assert forward(deep, 0) == divided and "FlatSplitArgs" not in forward(deep, 0, 4096)[0]
''')
    run(r'''
deep = (1, 784, 64, 3, 12, 3, 3, 1, 1)
hip.stand_in_cost(b"FlatSplitArgs", 2.0)
hip.stand_in_cost(b"conv_", 1.0)
assert any("FlatSplitArgs" in k for k in tune(deep, 0))
for stream in (0, 4096):
    assert "FlatSplitArgs" not in forward(deep, 0)[0]
    tune(deep, 0, 4096)
''')


def test_every_device_gets_the_lds_that_a_kernel_needs(run):
    """A kernel's LDS limit is a setting of one device: each variant, and the divided, flattened and window kernels, launch on a second one as well."""
    out = run(r'''
shapes = [(32, 3, 64, 112, 112, 7, 7, 2, 2), (32, 3, 65, 9, 8, 7, 7, 2, 2), (36, 3, 64, 41, 43, 7, 7, 2, 2), (64, 64, 64, 14, 14, 3, 3, 1, 1), (64, 40, 70, 13, 9, 3, 3, 1, 1),
          (64, 64, 64, 14, 14, 1, 1, 1, 1), (64, 64, 64, 14, 14, 1, 1, 2, 2), (64, 64, 64, 14, 14, 3, 3, 2, 2), (32, 72, 64, 14, 14, 5, 5, 1, 1), (8, 5, 9, 6, 7, 3, 3, 1, 1)]
plan = (ctypes.c_char * 4096)()
ran = set()
for i in range(lib.cacnn_variant_count()):
    dtype = int(lib.cacnn_variant_name(i).startswith(b"bf16"))
    for dims in shapes:
        if lib.cacnn_plan_variant(problem(*dims), I(dtype), I(i), plan, V(0), V(0)) == 0:
            for device in (0, 1):
                hip.stand_in_device(device)
                assert lib.cacnn_conv_forward_with_plan(problem(*dims), I(dtype), plan, V(IMAGE), V(FILTER), V(OUT), V(0)) == 0, (device, lib.cacnn_variant_name(i), dims)
                ran.update(kernels())
for dims, dtype in (((1, 784, 64, 3, 12, 3, 3, 1, 1), 0), ((72, 976, 16, 5, 5, 3, 3, 2, 2), 1), ((16, 3, 64, 112, 112, 7, 7, 2, 2), 1), ((128, 3, 32, 89, 89, 5, 5, 2, 2), 1)):
    for device in (2, 3):
        hip.stand_in_device(device)
        for stream in (0, 4096):
            ran.update(forward(dims, dtype, stream))
print("\n".join(ran))
''')
    for part in ("conv_f32_stem_pair", "conv_f32_stem_direct", "conv_f32_direct16", "conv_bf16_direct", "FlatSplitArgs", "conv_window"):
        assert part in out


def test_the_stem_kernel_takes_no_planes_beyond_31_bits_of_offset(run):
    """One k-tile (K <= 64) runs on the pair of sets, more on the kernel with staging waves; an Image of which ten planes reach 2^31 bytes is given to neither."""
    run(r'''
plan = (ctypes.c_char * 4096)()
variant = [i for i in range(lib.cacnn_variant_count()) if lib.cacnn_variant_name(i).startswith(b"f32 fxsd ")][0]
for B, K, H in ((8192, 8, 1089), (8192, 65, 1089), (8192, 8, 1090), (8192, 64, 100), (32, 65, 9), (32, 64, 9), (8180, 7, 1092), (8180, 70, 1091)):
    dims = problem(B, 3, K, 2, H, 7, 7, 2, 2)
    status = lib.cacnn_plan_variant(dims, I(0), I(variant), plan, V(0), V(0))
    assert status == (0 if 10 * 4 * 3 * B * (2 * H + 5) < 2 ** 31 else 3), (B, K, H)
    if status == 0:
        assert lib.cacnn_conv_forward_with_plan(dims, I(0), plan, V(IMAGE), V(FILTER), V(OUT), V(0)) == 0
        assert [("stem_pair" if K <= 64 else "stem_direct") in k for k in kernels()] == [True], (B, K, H)
    assert lib.cacnn_plan_variant(problem(32, 3, K, 2, 9, 7, 7, 2, 2), I(0), I(variant), plan, V(0), V(0)) == 0
    if status:
        assert lib.cacnn_conv_forward_with_plan(dims, I(0), plan, V(IMAGE), V(FILTER), V(OUT), V(0)) == 3 and not kernels()
''')
