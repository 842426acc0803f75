"""Which launches a call makes: the library's host side on the CPU, with the
launches written down instead of made."""
import ctypes
import json
import os
import shutil
import subprocess

import pytest

from paper_2511_02742_amd import build, hough

HERE = os.path.dirname(os.path.abspath(__file__))
FAKE = ctypes.c_void_p(4096)   # a device pointer: never read here


class Library:
    def __init__(self, path):
        self.lib = lib = ctypes.CDLL(path)
        for name in ("hough_create", "hough_destroy", "hough_find", "hough_find_noalloc", "hough_graph_create",
                     "hough_graph_destroy", "hough_config_default"):
            real = getattr(hough.load_library(), name)
            getattr(lib, name).argtypes, getattr(lib, name).restype = real.argtypes, real.restype
        lib.launches.restype = ctypes.c_char_p
        lib.set_memory.argtypes = [ctypes.c_size_t]

    def log(self):
        return [json.loads(x) for x in self.lib.launches().decode().splitlines()]

    def create(self, **cfg):
        c = hough.HoughConfig()
        self.lib.hough_config_default(ctypes.byref(c))
        for k, v in cfg.items():
            setattr(c, k, v)
        h = ctypes.c_void_p()
        return self.lib.hough_create(ctypes.byref(c), 0, ctypes.byref(h)), h

    def calls(self, events, hits, noalloc=False, **cfg):
        """The launches of one find call in a new context: a list of dicts."""
        st, h = self.create(**cfg)
        assert st == 0, (st, cfg)
        self.log()
        fn = self.lib.hough_find_noalloc if noalloc else self.lib.hough_find
        st = fn(h, None, events, hits, FAKE, FAKE, FAKE, FAKE, hits, FAKE, hits, FAKE)
        assert st == 0, (st, cfg)
        got = [x for x in self.log() if "launch" in x]
        self.lib.hough_destroy(h)
        return got


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    so = tmp_path_factory.mktemp("host") / "host.so"
    subprocess.check_call([gxx, "-std=c++20", "-O1", "-w", "-fPIC", "-shared", "-I", os.path.join(HERE, "native", "host"),
                           "-I", build.INCLUDE, "-I", build.CSRC, "-x", "c++", os.path.join(build.CSRC, "hough_host.hip"),
                           os.path.join(HERE, "native", "launches.cpp"), "-o", str(so)])
    return Library(str(so))


@pytest.mark.parametrize("n_rho", [1024, 1200, 2048, 2400, 3000, 4096, 4704, 5000])
@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_a_split_sweep_does_not_refuse_a_grid(host, n_rho, threads):
    """Rows too long for the finder's row-stream path switch a configured split
    sweep off; whether the split's own row buffers fit does not matter then."""
    st, h = host.create(n_rho=n_rho, sweep_groups=2, sweep_threads=threads)
    assert st == 0
    host.lib.hough_destroy(h)
