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
        self.limit = {}   # dynamic LDS that a kernel's launches may ask for, as it was set last

    def log(self):
        got = [json.loads(x) for x in self.lib.launches().decode().splitlines()]
        self.limit.update({(x["limit"], x["threads"]): x["bytes"] for x in got if "limit" in x})
        return got

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


NMS, ARGMAX = 1, 0


# The dense shape's rule at its edges: (configuration, events, hits, most hits of
# an event in it, or None where the call enqueues the context's shape alone).
DENSE = [
    ({}, 767, 767 * 27, None),
    ({}, 768, 768 * 27, 352),                         # small events: 352 hits, whatever the mean
    ({}, 768, 768 * 136, 387),                        # else 1.9 times what a workgroup takes on average
    ({}, 768, 768 * 137, None),                       # hits times rows
    ({}, 1024, 1024 * 137, 520),                      # from 1024 events on whatever they hold,
    ({}, 1024, 1024 * 600, 2280),
    ({}, 1024, 1024 * 1100, 2560),                    # up to the shape's list of hits
    ({}, 1024, 1024 * 2560, 2560),
    ({}, 1024, 1024 * 2560 + 1, None),                # some event has more
    ({}, 1023, 1023 * 137, None),
    ({"n_theta": 1025}, 1024, 1024 * 137, None),
    ({"n_theta": 1025}, 1024, 1024 * 100, None),
    ({"rho_min": -300.0, "rho_max": 300.0}, 1024, 1024 * 137, None),   # azimuths to 351 degrees leave the grid
    ({"rho_min": -360.0, "rho_max": 360.0}, 1024, 1024 * 137, 520),
    ({"rho_min": -300.0, "rho_max": 300.0, "phi_unit": 1}, 1024, 1024 * 137, 520),
    ({"n_rho": 999}, 3071, 3071 * 27, None),
    ({"n_rho": 999}, 3072, 3072 * 27, 352),
    ({"n_rho": 1000, "n_theta": 180}, 768, 768 * 320, 912),
    ({"n_rho": 1000, "n_theta": 180}, 768, 768 * 321, None),
    ({"n_rho": 1000, "n_theta": 180}, 768, 768 * 27, 512),     # on few rows events of up to 512 hits are small
    ({"n_rho": 1000, "n_theta": 511}, 768, 768 * 27, 512),
    ({"n_rho": 1000, "n_theta": 512}, 768, 768 * 27, 352),
    ({"n_rho": 1000, "n_theta": 180}, 4096, 4096 * 400, 1536),
    ({"n_rho": 1000, "n_theta": 180, "peak_mode": ARGMAX}, 768, 768 * 27, 1536),
    ({"n_rho": 1000, "n_theta": 180, "peak_mode": ARGMAX}, 4096, 4096 * 321, None),
    ({"wg_threads": 1024}, 4096, 4096 * 110, None),
    ({"tile_rows": 14}, 4096, 4096 * 110, None),
    ({"sweep_groups": 1}, 4096, 4096 * 110, None),
    ({"nms_radius": 3}, 4096, 4096 * 110, 1672),
    ({"nms_radius": 3, "min_votes": 5}, 4096, 4096 * 110, None),       # wide windows from T = 6 on,
    ({"nms_radius": 1, "min_votes": 2}, 4096, 4096 * 110, 1672),
    ({"peak_mode": ARGMAX, "min_votes": 4}, 1024, 1024 * 110, 2560),   # the largest bin from T = 4
    ({"peak_mode": ARGMAX, "min_votes": 3}, 1024, 1024 * 110, None),
    ({"n_rho": 1000, "n_theta": 180, "peak_mode": 2}, 4096, 4096 * 110, None),
]


@pytest.mark.parametrize("cfg,events,hits,most", DENSE)
def test_dense_shape(host, cfg, events, hits, most):
    """A call that may take the dense shape enqueues it and, for the choice made on
    the device, the context's own; every other call the context's alone."""
    got = host.calls(events, hits, **cfg)
    kinds = [x["launch"] for x in got]
    if most is None:
        assert kinds[-2] in ("find", "find_cf") and "order_pick" not in kinds and "picked" not in kinds
        return
    assert kinds == ["order_pick", "picked", "list", "compact"]
    order, dense, rest, compact = got
    assert order["hits"] == most and dense["defer"] == 0 and order["events"] == dense["events"] == events
    assert compact["ordered"] == 1
    # two workgroups per CU, a slot for each; the other shape is the context's own
    assert dense["threads"] == 512 and dense["lds"] <= (160 << 10) // 2 - 2048 and rest["threads"] == 1024 and rest["groups"] == 256
    assert dense["slots"] == min(events, 512)
    # no event that the choice lets in outgrows the shape's list
    assert most <= 512 + min(dense["hs_cap"] // 64 * 64, 56 * 64)


def test_dense_shape_needs_its_workspace(host):
    """Without memory for the dense shape's slots, and in the fixed scratch, a call
    takes the context's own shape; a captured one has its own workspace."""
    try:
        host.lib.set_memory(200 << 20)   # the slots of one workgroup per CU are 128 MiB, of two 256
        assert [x["launch"] for x in host.calls(1024, 1024 * 110)] == ["order", "find", "compact"]
    finally:
        host.lib.set_memory(1 << 40)
    assert [x["launch"] for x in host.calls(1024, 1024 * 110, noalloc=True)] == ["order", "find", "compact"]
    st, h = host.create()
    g = ctypes.c_void_p()
    host.log()
    n = 1024 * 110
    assert host.lib.hough_graph_create(h, 1024, n, FAKE, FAKE, FAKE, FAKE, n, FAKE, n, FAKE, ctypes.byref(g)) == 0
    assert [x["launch"] for x in host.log()] == ["order_pick", "picked", "list", "compact"]
    host.lib.hough_graph_destroy(g)
    host.lib.hough_destroy(h)


@pytest.mark.parametrize("cfg,threads", [({}, 512), ({"min_votes": 2}, 512), ({"min_votes": 1}, 1024), ({"sweep_groups": 2}, 1024),
                                         ({"rho_min": -350.0, "rho_max": 350.0}, 1024), ({"rho_min": -360.0, "rho_max": 360.0}, 512),
                                         ({"peak_mode": ARGMAX, "min_votes": 2, "n_theta": 205}, 1024),
                                         ({"peak_mode": ARGMAX, "min_votes": 2, "n_theta": 204}, 512),
                                         ({"peak_mode": ARGMAX, "min_votes": 3, "n_theta": 1025}, 1024),
                                         ({"peak_mode": ARGMAX, "min_votes": 3, "n_theta": 1024}, 512),
                                         ({"peak_mode": ARGMAX, "min_votes": 4, "n_theta": 1025}, 512),
                                         ({"nms_radius": 2, "min_votes": 2, "n_theta": 1025}, 512),
                                         ({"nms_radius": 3, "min_votes": 2, "n_theta": 256}, 1024),
                                         ({"nms_radius": 3, "min_votes": 3, "n_theta": 1025}, 1024),
                                         ({"nms_radius": 3, "min_votes": 3, "n_theta": 1024}, 512),
                                         ({"nms_radius": 3, "min_votes": 4, "n_theta": 1025}, 512)])
def test_long_rows_that_would_be_tiled_anyway(host, cfg, threads):
    """Where nearly every event would outgrow the lists or leaves the grid, long
    rows keep sixteen waves, as with a configured split sweep."""
    got = [x for x in host.calls(64, 9000, n_rho=2048, **cfg) if x["launch"] in ("find", "picked")]
    assert [x["threads"] for x in got] == [threads]


# Long rows: (rho bins, threads of the shape that streams them, hits its list holds)
LONG = [(1160, 512, 2560), (2048, 512, 4096), (2304, 512, 4096), (2400, 256, 2560), (4096, 256, 4096)]


@pytest.mark.parametrize("n_rho,threads,most", LONG)
@pytest.mark.parametrize("mode", [NMS, ARGMAX])
def test_large_events_on_long_rows(host, n_rho, threads, most, mode):
    """An event that the shape for long rows would sweep tile by tile (it outgrows
    its list, say) is faster swept so by sixteen waves: alone the host sends it there, a
    call enqueues both shapes, and the first leaves such events to the second."""
    def of(events, hits, **kw):
        return [x for x in host.calls(events, hits, n_rho=n_rho, peak_mode=mode, **kw) if x["launch"] not in ("sweep", "band")]
    # alone past the list's size: the host knows
    assert [(x["launch"], x["threads"], x["stream_ok"]) for x in of(1, most + 1)] == [("find", 1024, 0)]
    for n, hits in ((1, most), (2, 300), (4, most + 1), (64, 9000), (300, 90000)):
        for noalloc in (False, True):
            got = of(n, hits, noalloc=noalloc)
            assert [x["launch"] for x in got] == ["order_pick", "picked", "list"] + (["compact"] if n > 1 else [])
            assert got[0]["hits"] == 2**63 - 1 and got[1]["defer"] == 1 and got[1]["threads"] == threads
            assert got[1]["hs_cap"] // 64 * 64 >= most - 512
            assert got[2]["threads"] == 1024 and got[2]["stream_ok"] == 0 and got[2]["split"] == 0
            assert n == 1 or got[3]["ordered"] == (1 if n > 256 else 0)
    # where the second list does not fit the fixed scratch, the tiled shape takes the call
    assert [(x["launch"], x.get("threads")) for x in of(64, 1 << 20, noalloc=True)][-2] in (("list", 1024), ("find", 1024))
    # configured shapes are what they were
    assert [x["threads"] for x in of(1, most + 1, wg_threads=256) + of(2, most + 1, wg_threads=512)[:1]] == [256, 512]


@pytest.mark.parametrize("events", [1, 2, 64, 300])
@pytest.mark.parametrize("noalloc", [False, True])
def test_few_votes_on_long_rows(host, events, noalloc):
    """A call of few votes in all has no second launch: that would cost it more than
    an event of it that is swept tile by tile; an event alone that outgrows the list
    still has the sixteen waves."""
    def of(hits, n_theta):
        return [(x["launch"], x["threads"]) for x in host.calls(events, hits, n_rho=2048, n_theta=n_theta, noalloc=noalloc)
                if x["launch"] in ("find", "picked", "list")]
    for n_theta in (32, 64):
        hits = 65536 // n_theta
        assert of(hits, n_theta) == [("find", 512)]
        assert of(hits + 1, n_theta) == [("picked", 512), ("list", 1024)]
    hits = 65536 // 14
    assert of(hits, 14) == [("find", 1024 if events == 1 else 512)]


@pytest.mark.parametrize("n_rho", [1024, 1160, 2048, 4096])
@pytest.mark.parametrize("events", [1, 2, 8, 9])
def test_scratch_limit_of_the_call_without_allocation(host, n_rho, events):
    """The fixed scratch takes the calls it took when long rows had the tiled
    shape: what the other shape adds to the workspace is left out where it does
    not fit."""
    def fits(hits, **kw):
        st, h = host.create(n_rho=n_rho, **kw)
        r = host.lib.hough_find_noalloc(h, None, events, hits, FAKE, FAKE, FAKE, FAKE, hits, FAKE, hits, FAKE)
        host.lib.hough_destroy(h)
        return r == 0
    def most(**kw):
        lo, hi = 1, 1 << 24
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if fits(mid, **kw) else (lo, mid)
        return lo
    tiled = dict(wg_threads=1024) if n_rho > 1152 else {}
    assert most() >= most(**tiled)


def test_a_context_leaves_the_other_contexts_their_lds(host):
    """The dynamic LDS that a kernel may ask for is one setting per process: making
    a context never takes from it what another's launches ask for."""
    configs = [dict(wg_threads=512), dict(), dict(n_rho=2048), dict(wg_threads=512, tile_rows=14), dict(n_rho=512, tile_rows=16),
               dict(n_theta=180, n_rho=1000, peak_mode=2), dict(n_theta=90, n_rho=500, peak_mode=2), dict(n_rho=3000),
               dict(n_rho=1000, n_theta=180, peak_mode=ARGMAX), dict(wg_threads=256, tile_rows=6), dict(sweep_groups=2), dict()]
    live = []
    for cfg in configs:
        st, h = host.create(**cfg)
        assert st == 0
        host.log()
        live.append((cfg, h))
        for c, other in live:
            for events, hits in ((1, 300), (4, 1200), (300, 9000), (2048, 50000), (2, 9000)):
                assert host.lib.hough_find(other, None, events, hits, FAKE, FAKE, FAKE, FAKE, hits, FAKE, hits, FAKE) == 0
                for x in host.log():
                    kernel = {"find": "find", "picked": "find", "list": "find", "find_cf": "cf"}.get(x.get("launch"))
                    if kernel:
                        assert x["lds"] <= host.limit[kernel, x["threads"]], (c, "after", cfg, x, host.limit)
    for _, h in live:
        host.lib.hough_destroy(h)


@pytest.mark.parametrize("cfg,slots", [({"wg_threads": 256, "tile_rows": 6}, 768), ({"wg_threads": 256, "tile_rows": 6, "peak_mode": ARGMAX}, 1024),
                                       ({"wg_threads": 256, "peak_mode": ARGMAX}, 512), ({}, 512)])
def test_a_slot_for_every_workgroup(host, cfg, slots):
    """As many large-event slots as the most workgroups that any kernel taking them
    has resident at once (here one more per CU than the finder, for 256 threads of
    the largest-bin search)."""
    find = [x for x in host.calls(4096, 4096 * 400, n_rho=1000, **cfg) if x["launch"] in ("find", "picked")][0]
    assert find["slots"] == slots


@pytest.mark.parametrize("n_theta", [1, 2, 5, 7, 8, 13, 14, 15, 16, 30, 64, 180, 1024, 1025])
@pytest.mark.parametrize("mode", [NMS, ARGMAX])
def test_every_grid_has_its_launches(host, n_theta, mode):
    """Over grids from one row to many, of short rows to the longest: no call is
    enqueued with a shape that no kernel has, nor with more LDS than there is."""
    for n_rho in (5, 64, 500, 512, 900, 999, 1000, 1024, 1025, 1152, 1153, 1500, 2048, 2304, 2305, 3000, 4096, 4704, 4705, 9000):
        for extra in ({}, {"nms_radius": 2}, {"wg_threads": 256}, {"wg_threads": 512}, {"sweep_groups": 2, "sweep_threads": 512}):
            cfg = dict(n_theta=n_theta, n_rho=n_rho, peak_mode=mode, rho_min=-750.0, rho_max=750.0, **extra)
            st, h = host.create(**cfg)
            if st != 0:   # rows that no LDS tile holds, by the configured threads or a wide window
                assert n_rho >= 4096
                continue
            host.log()
            for events, hits in ((1, 55), (1, 5000), (2, 300), (9, 9000), (64, 9000), (300, 30000), (768, 20000), (1100, 60000),
                                 (4096, 100000), (4096, 2000000)):
                for fn in (host.lib.hough_find, host.lib.hough_find_noalloc):
                    r = fn(h, None, events, hits, FAKE, FAKE, FAKE, FAKE, hits, FAKE, hits, FAKE)
                    assert r in (0, -2 if fn is host.lib.hough_find_noalloc else 0), (cfg, events, hits, r)
                    for x in host.log():
                        if x.get("launch") in ("find", "picked", "list"):
                            assert x["lds"] + 2048 <= 160 << 10 and x["threads"] in (256, 512, 1024)
            host.lib.hough_destroy(h)
