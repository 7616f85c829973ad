"""Which launches a forward pass makes, asked of the library on the CPU: ``native/record_model_launches.cpp`` replaces the
launchers of the built library with ones that print what they were called for."""

import os
import shutil
import subprocess

import pytest

from paper_2109_01611_amd import build, gpulet

HERE = os.path.dirname(os.path.abspath(__file__))
INPUT, OUTPUT, WORKSPACE = 0x10000000, 0x80000000, 0x100000000


@pytest.fixture(scope="session")
def model_launches(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if not hipcc:
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("launches") / "record")
    lib = os.path.dirname(build.LIB)
    subprocess.run([hipcc, "-O1", "-std=c++17", "-w", "-x", "hip", "--cuda-host-only", "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC, os.path.join(HERE, "native", "record_model_launches.cpp"), "-x", "none", "-o", exe,
                    "-L", lib, "-lgpulet", "-Wl,-rpath," + lib], check=True, timeout=300)

    def ask(cu, batch, in_shape, layers, split_k=1, in_at=INPUT, out_at=OUTPUT, n_bufs=None, in_buf=0, out_buf=1):
        """``layers``: dicts of ``gpulet_layer`` fields (a missing ``bias`` means one is there) -> [(kernel, layers run), ...]"""
        rows = []
        for l in layers:
            f = dict(res_buf=-1, K=0, R=0, S=0, stride=0, pad=0, relu=0, mode=0, out_fp32=0, group_next=0, bias=1)
            f.update(l)
            rows.append(" ".join(str(int(f[n])) for n in ("op", "in_buf", "out_buf", "res_buf", "C", "K", "R", "S", "stride", "pad",
                                                             "relu", "mode", "out_fp32", "group_next", "bias")))
        text = "%d %d %d %x %x %d %d %d %d %d %d %d\n%s\n" % (
            (cu, batch, split_k, in_at, out_at, len(layers), n_bufs or len(layers) + 1) + tuple(in_shape) + (in_buf, out_buf, "\n".join(rows)))
        out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=120, check=True).stdout.split("\n")
        assert out[-2:] == ["end", ""]
        return [(k, int(n)) for k, n in (line.split() for line in out[:-2])]
    return ask


def straight(*layers):
    """Layers one behind the other, each with a buffer of its own: ("conv", C, K, k, stride, pad), ("dw", C, stride),
    ("max", C, k, stride, pad), ("fc", In, Out)."""
    out = []
    for i, l in enumerate(layers):
        f = dict(in_buf=0 if i == 0 else i + 1, out_buf=1 if i + 1 == len(layers) else i + 2, C=l[1], relu=1)
        if l[0] == "conv":
            f.update(op=gpulet.OP_CONV, K=l[2], R=l[3], S=l[3], stride=l[4], pad=l[5])
        elif l[0] == "dw":
            f.update(op=gpulet.OP_DWCONV, R=3, S=3, stride=l[2], pad=1)
        elif l[0] == "max":
            f.update(op=gpulet.OP_POOL, R=l[2], stride=l[3], pad=l[4], mode=gpulet.POOL_MAX)
        else:
            f.update(op=gpulet.OP_FC, K=l[2])
        out.append(f)
    return out
