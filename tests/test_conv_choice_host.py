"""Which kernel a convolution gets, asked of the library on the CPU: ``native/record_conv_launches.cpp`` replaces the
launchers of the built library with ones that print what they were called with."""

import os
import shutil
import subprocess

import pytest

import bench
import test_gpu_layers
from paper_2109_01611_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if not hipcc:
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("choice") / "record")
    lib = os.path.dirname(build.LIB)
    subprocess.run([hipcc, "-O1", "-std=c++17", "-w", "-x", "hip", "--cuda-host-only", "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC, os.path.join(HERE, "native", "record_conv_launches.cpp"), "-x", "none", "-o", exe,
                    "-L", lib, "-lgpulet", "-Wl,-rpath," + lib], check=True, timeout=300)

    def ask(requests):
        """[(CUs, [(N, C, H, W, K, R, S, stride, pad, stored channels), ...]), ...] -> per request [(kernel, tile, layers), ...]"""
        text = "\n".join("%d %d %s" % (cu, len(layers), " ".join(str(v) for l in layers for v in l)) for cu, layers in requests)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=120, check=True).stdout
        done = [[]]
        for line in out.splitlines():
            if line == "end":
                done.append([])
            else:
                kernel, tile, *layers = line.split()
                done[-1].append((kernel, int(tile), layers))
        assert len(done) == len(requests) + 1
        return done[:-1]
    return ask


def inception(N, H, reduce3, K3, reduce5, K5, C, K1):
    """The three independent convolutions of an inception block that share a launch (both reduce layers in one tensor)."""
    both = reduce3 + reduce5
    return [(N, reduce3, H, H, K3, 3, 3, 1, 1, both), (N, reduce5, H, H, K5, 5, 5, 1, 2, both), (N, C, H, H, K1, 1, 1, 1, 0, C)]


# CUs, layers, the tile that measured fastest or within 2 % of it (us with it and with the tile in brackets)
GROUPS = [
    (192, inception(32, 14, 96, 208, 16, 48, 480, 64), 1),     # 12.0 (128x128: 12.6): hardly more tiles than CUs
    (192, inception(32, 14, 128, 256, 24, 64, 512, 64), 1),    # 14.3 (128x128: 14.8)
    (256, inception(32, 28, 128, 192, 32, 96, 256, 64), 1),    # 28.7 (128x128: 30.4): two shallower members
    (256, inception(32, 14, 112, 224, 24, 64, 512, 64), 0),    # 12.0 (128x64: 13.0)
    (64, inception(1, 14, 128, 256, 24, 64, 512, 64), 14),     # 7.1 (64x64: 7.6): one round of small tiles
    (64, inception(1, 7, 192, 384, 48, 128, 832, 128), 14),    # 7.5 (64x64: 10.2)
]


@pytest.mark.parametrize("case", GROUPS, ids=lambda c: "%d-%s" % (c[0], "x".join(map(str, c[1][0][:5]))))
def test_tile_of_a_launch_group(launches, case):
    cu, layers, tile = case
    for order in (layers, layers[::-1]):
        (kernel, got, members), = launches([(cu, order)])[0]
        assert (kernel, got) == ("group", tile)
        depth = {"%dx%dx%dx%dx%d" % l[:5]: l[1] * l[5] * l[6] for l in layers}
        assert [depth[m] for m in members] == sorted(depth.values(), reverse=True)      # deepest member first


def test_the_small_patch_cases_reach_every_patch_tile(launches):
    # the layers of the GPU parity tests, on a whole GPU: 1, 2 = 64x32 with a long and a short patch, 3, 4 = 64x16, 5 = 128x32
    want = {(1, 128, 7, 7, 40): 4, (1, 64, 14, 14, 24): 4, (3, 64, 7, 7, 72): 4, (2, 64, 14, 14, 72): 3, (9, 128, 7, 7, 72): 3,
            (5, 256, 14, 14, 264): 1, (1, 64, 28, 28, 520): 2, (1, 192, 5, 3, 8): 4, (8, 64, 14, 14, 520): 5, (40, 128, 7, 7, 392): 5}
    assert set(test_gpu_layers.SMALL_PATCH_CASES) <= set(want)
    got = launches([(256, [c + (3, 3, 1, 1, c[1])]) for c in want])
    assert [g[0][:2] for g in got] == [("patch", v) for v in want.values()]


def test_the_benchmark_names_the_kernel_it_times(launches):
    # variant 0 is the 128x64 patch tile; its mangled name is in the library
    assert launches([(256, [(32, 256, 14, 14, 256, 3, 3, 1, 1, 256)])])[0] == [("patch", 0, ["32x256x14x14x256"])]
    name, args = bench.BENCH_KERNEL.rstrip(">").split("<")
    mangled = "%d%sI%sE" % (len(name), name, "".join("Lb%dE" % (a == "true") if a in ("true", "false") else "Li%sE" % a
                                                        for a in args.split(",")))
    with open(build.LIB, "rb") as fh:
        assert mangled.encode() in fh.read()
