"""What a tile workspace has to zero between calls (tile_state.h), on the CPU:
every short sequence of calls -- level 2 pushed or gathered, calls that fail on
the way, a new width, a race that fits plans without running tiles -- against
what the arrays hold."""
import ctypes
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("tile") / "libtile.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall",
                    "-I", os.path.join(ROOT, "paper_1910_13874_amd", "csrc"),
                    os.path.join(ROOT, "tests", "tile_state_shim.cpp"), "-o", out], check=True)
    L = ctypes.CDLL(out)
    L.ts_new.restype = ctypes.c_void_p
    for name in ("ts_free", "ts_zero", "ts_copy_replaced", "ts_begin", "ts_end"):
        getattr(L, name).argtypes = [ctypes.c_void_p] + [ctypes.c_int] * (name in ("ts_begin", "ts_end"))
    L.ts_fit.argtypes = [ctypes.c_void_p, ctypes.c_ulong, ctypes.c_int]
    return L


class Arrays:
    """counts: level 1 (and the worklist length); level2; copy: level 1's
    16-bit copy.  True: zero."""

    def __init__(self):
        self.counts = self.level2 = self.copy = False
        self.bytes = 0

    def fit(self, fill, nbytes, gathered):
        if nbytes != self.bytes:
            self.counts = self.level2 = False  # another layout
        self.bytes = nbytes
        if fill & 1:
            self.counts = self.level2 = True
        if fill & 2:
            self.level2 = True
        if fill & 4:
            self.copy = True
        assert self.counts
        assert gathered or self.level2
        assert not gathered or self.copy

    def ran(self, gathered, ok):
        if not ok:
            self.counts = self.level2 = False
            self.copy = self.copy and not gathered
        elif gathered:
            self.level2 = False


# gathered, then: the call succeeds, fails, or only fits (a width race)
OPS = [(g, how) for g in (0, 1) for how in ("ok", "fails", "fits")] + [(0, "wide"), (1, "wide")]


def test_every_short_sequence(lib):
    for seq in itertools.product(OPS, repeat=5):
        p, a = lib.ts_new(), Arrays()
        for gathered, how in seq:
            nbytes = 200 if how == "wide" else 100
            if how == "wide" and gathered:  # the copy's array grows
                lib.ts_copy_replaced(p)
                a.copy = False
            a.fit(lib.ts_fit(p, nbytes, gathered), nbytes, gathered)
            if how == "fits":
                continue
            lib.ts_begin(p, gathered)
            assert not lib.ts_zero(p)
            a.ran(gathered, how != "fails")
            if how != "fails":
                lib.ts_end(p, gathered)
                assert lib.ts_zero(p)
        lib.ts_free(p)


def test_steady_calls_zero_nothing(lib):
    """Repeated calls of one kind fill nothing; changing kinds fills level 2
    once after gathered tiles and the copy once before the first."""
    p = lib.ts_new()
    fills = []
    for gathered in (0, 0, 1, 1, 0, 0, 1, 0):
        fills.append(lib.ts_fit(p, 100, gathered))
        lib.ts_begin(p, gathered)
        lib.ts_end(p, gathered)
    assert fills == [1, 0, 4, 0, 2, 0, 0, 2]
    lib.ts_free(p)
