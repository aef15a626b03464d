"""The library's host side (csrc/api.cpp) on the CPU, against the model of the
HIP runtime in host_runtime.cpp: `host` is the Python binding loaded on it."""
import ctypes
import os
import shutil
import subprocess
from types import SimpleNamespace

import pytest
import torch

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2310_08770_amd", "csrc")
ROCM = "/opt/rocm/include"


@pytest.fixture(scope="session")
def host_lib(tmp_path_factory):
    if not (shutil.which("g++") and os.path.exists(ROCM)):
        pytest.skip("needs g++ and the HIP headers")
    d = tmp_path_factory.mktemp("host")
    cmd = ["g++", "-std=c++17", "-O0", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}"]
    srcs = {"api.o": os.path.join(CSRC, "api.cpp"), "runtime.o": os.path.join(HERE, "host_runtime.cpp")}
    jobs = [subprocess.Popen([*cmd, "-c", s, "-o", str(d / o)]) for o, s in srcs.items()]
    assert [j.wait() for j in jobs] == [0, 0]
    # (-Bsymbolic: the model's functions, not those of a runtime already loaded)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *[str(d / o) for o in srcs], "-o", str(d / "libhost.so")],
                   check=True)
    return str(d / "libhost.so")


@pytest.fixture
def host(host_lib, monkeypatch):
    """Tracker over the model: track() takes CPU tensors and stream numbers."""
    from paper_2310_08770_amd import ccpt
    monkeypatch.setattr(ccpt, "LIB_PATH", host_lib)
    monkeypatch.setattr(ccpt, "_lib", None)
    L = ccpt.lib()
    L.host_limit.argtypes = [ctypes.c_size_t]
    L.host_live.restype = ctypes.c_size_t
    made = []

    def tracker(**kw):
        tr = ccpt.Tracker(device=0, **kw)
        tr.device = torch.device("cpu")
        made.append(tr)
        return tr

    def launches():
        """(ny, nx, count, fused_min, pairs_ok) of the correlation launches since the last call"""
        buf = (ctypes.c_int * (5 * 4096))()
        n = L.host_log(buf, 4096)
        return [tuple(buf[5 * i:5 * i + 5]) for i in range(n)]

    L.host_limit(2**63)
    L.host_last_error_clear()
    launches()
    yield SimpleNamespace(tracker=tracker, launches=launches, limit=L.host_limit, live=L.host_live, asked=L.host_asked, refuse=L.host_refuse, lib=L,
                          no_tables=L.host_no_tables)
    L.host_limit(2**63)
    L.host_refuse(0)
    for tr in made:
        tr.close()
