"""The library's host code on a HIP runtime without a GPU (fake_hip.cpp): fixtures `host` and `hip`."""
import ctypes as C
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2501_10054_amd import build as B
from paper_2501_10054_amd import tardis as T

HERE = os.path.dirname(os.path.abspath(__file__))
GIB = 1 << 30


@pytest.fixture(scope="session")
def host(tmp_path_factory):
    tmp = str(tmp_path_factory.mktemp("host"))
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    flags = ["--offload-arch=gfx950", "-O1", "-fPIC", "-std=c++17", "-Wno-unused-function", "--offload-host-only"]
    obj = lambda s: os.path.join(tmp, os.path.basename(s) + ".o")
    sources = [os.path.join(B.CSRC, s) for s in B.SOURCES]
    compile_ = lambda s: subprocess.run([hipcc, *flags, "-c", s, "-o", obj(s)], check=True, capture_output=True)
    with ThreadPoolExecutor(8) as ex:
        list(ex.map(compile_, sources))
    undefined = subprocess.run(["nm", "-u", *map(obj, sources)], check=True, capture_output=True, text=True).stdout
    stub = os.path.join(tmp, "code.c")                # (the device code, which nothing here loads)
    with open(stub, "w") as f:
        f.writelines(f"char {name}[8];\n" for name in sorted(set(re.findall(r"__hip_fatbin\w+", undefined))))
    out = os.path.join(tmp, "libhost.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["gcc", "-fPIC", "-c", stub, "-o", stub + ".o"], check=True)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include", "-w",
                    os.path.join(HERE, "fake_hip.cpp"), *map(obj, sources), stub + ".o", "-Wl,-Bsymbolic", "-o", out], check=True)
    return Host(out)


class Host:
    def __init__(self, path):
        self.lib = C.CDLL(path)
        self.lib.fake_used.restype = C.c_size_t
        self.lib.fake_events.restype = self.lib.fake_launches.restype = C.c_char_p
        self.lib.fake_reset.argtypes = [C.c_size_t]
        self.lib.tardis_fold.argtypes = [C.POINTER(T.tardis_ffn_desc), C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p,
                                         C.POINTER(T.tardis_fold_opts), C.c_void_p, C.POINTER(C.c_void_p)]
        self.lib.tardis_destroy.argtypes = [C.c_void_p]
        for name in ("tardis_ffn_forward_batched", "tardis_dense_forward"):
            getattr(self.lib, name).argtypes = [C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p]

    def fold(self, d=512, h=2048, max_batch=1, deterministic=0, dtype=T.BF16, bits=8):
        """status, handle"""
        at = lambda k: C.c_void_p((1 << 38) + (k << 30))       # (never read: nothing runs)
        desc = T.tardis_ffn_desc(d, h, dtype, 0, at(0), None, at(1), None)
        opts = T.tardis_fold_opts(bits, dtype, max_batch, deterministic, 0.0)
        out = C.c_void_p()
        return self.lib.tardis_fold(desc, at(2), at(3), at(4), at(5), opts, None, out), out

    def events(self):
        return self.lib.fake_events().decode().split()

    def launches(self):
        return self.lib.fake_launches().decode().split()


@pytest.fixture
def hip(host):
    host.lib.fake_reset(288 * GIB)
    yield host
    host.lib.fake_reset(288 * GIB)
    assert host.lib.tardis_release_memory() == T.OK
    assert host.lib.fake_used() == 0
