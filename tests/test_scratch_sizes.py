"""Scratch memory is sized once: a context created for, or used on, a larger
field allocates nothing in calls on smaller ones, also where the smaller
field has more groups of the Huffman encoder.  Host code against the stand-in
runtime of tests/hipstub, without a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = os.path.join(ROOT, "tests", "hipstub")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_smaller_fields_allocate_nothing(tmp_path):
    if not os.path.exists(HIPCC) or shutil.which("g++") is None:
        pytest.skip("hipcc or g++ not available")
    flags = ["--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-Wno-unused-value", "-Wno-unused-result"]
    # the stub's own count of groups makes room for the driver's, which
    # follows the encoder's rule
    srcs = {"api": (os.path.join(ROOT, "paper_2509_20563_amd", "csrc", "fz_api.hip"), []),
            "stub": (os.path.join(STUB, "hip_stub.cpp"), ["-Dencode_groups=stub_encode_groups"]),
            "drv": (os.path.join(STUB, "scratch_sizes.cpp"), [])}
    objs = []
    for name, (src, extra) in srcs.items():
        obj = str(tmp_path / f"{name}.o")
        r = subprocess.run([HIPCC, *flags, *extra, "-c", src, "-o", obj], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        objs.append(obj)
    exe = str(tmp_path / "scratch_sizes")
    r = subprocess.run(["g++", "-Wl,--wrap=hipMalloc", *objs, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout[-2000:])
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
