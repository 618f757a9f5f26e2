"""Rules of the fill that are plain arithmetic on sizes (csrc/ckpt_rules.h), compiled with g++ and checked over their whole
range.  CPU only."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_02599_amd", "csrc")
SHIM = """
#include "ckpt_rules.h"
extern "C" int ask() { return ckpt_rules::kAsk; }
extern "C" int spread_split(int x, int slice, int KS, int nq) { return ckpt_rules::spread_split(x, slice, KS, nq); }
extern "C" int rows_pass(int tiles, int pitch, int B) { return ckpt_rules::rows_pass(tiles, pitch, B); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = tmp_path_factory.mktemp("rules")
    (out / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                           str(out / "shim.cpp"), "-o", str(out / "librules.so")])
    return ctypes.CDLL(str(out / "librules.so"))


@pytest.mark.parametrize("KS", [1, 2, 4])
def test_slices_fetch_the_bounds_of_different_splits(rules, KS):
    """Tiles of block diagonal D = 2 .. 31 have 8 (D - 1) + 1 middle splits.  Every place lies in the tile; the slices share
    no place but the one on their border; and together they reach as many splits as they have lanes, or all."""
    for nq in range(9, 8 * 30 + 2, 8):
        asking = nq > rules.ask()
        got = [[rules.spread_split(x, s, KS, nq) for x in range(12 if asking and s == 0 else 0, 16)] for s in range(KS)]
        flat = [k for g in got for k in g]
        assert min(flat) >= 0 and max(flat) < nq, (KS, nq)
        sharing = got[1:] if asking else got
        for a, b in zip(sharing, sharing[1:]):
            assert max(a) <= min(b), (KS, nq, a, b)
        if sharing:
            lanes = 16 * len(sharing)
            assert len({k for g in sharing for k in g}) == min(nq, lanes), (KS, nq)
        if asking:
            assert len(set(got[0])) == 4


@pytest.mark.parametrize("tiles,pitch,B,passing", [
    (10, 2112, 64, 1), (22, 4160, 8, 1), (30, 1024, 16, 1), (4, 1024, 98, 1), (29, 1 << 16, 1 << 20, 1),
    (4, 1024, 97, 0), (22, 4160, 4, 0), (6, 1088, 40, 0), (10, 2112, 8, 0), (1, 64, 2, 0)])
def test_rows_pass_through_the_caches_by_their_size(rules, tiles, pitch, B, passing):
    """128 MB of rows in one diagonal: 64 x 96 stages, 8 x 192 and the smallest batch that is split unasked are above it,
    batches of the sizes that only a caller splits below."""
    assert rules.rows_pass(tiles, pitch, B) == passing
