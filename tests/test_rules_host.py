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
extern "C" int asked_split(int x, int number, int qlo, int nq) { return ckpt_rules::asked_split(x, number, qlo, nq); }
extern "C" int operand_chunks(int reach) { return ckpt_rules::operand_chunks(reach); }
extern "C" int sample_chunks(int reach) { return ckpt_rules::sample_chunks(reach); }
extern "C" int left_below(int kk) { return ckpt_rules::left_below(kk); }
extern "C" int left_above(int kk) { return ckpt_rules::left_above(kk); }
extern "C" int right_below(int kk, int shift) { return ckpt_rules::right_below(kk, shift); }
extern "C" int right_above(int kk, int shift) { return ckpt_rules::right_above(kk, shift); }
extern "C" int far_offset() { return ckpt_rules::kFar; }
extern "C" int flow_pays(int nblk, int chunks, long long B, int samples) { return ckpt_rules::flow_pays(nblk, chunks, B, samples); }
extern "C" int chain_stages() { return ckpt_rules::kChainStages; }
extern "C" int chain_row(int L, int q) { return ckpt_rules::chain_row(L, q); }
extern "C" long long chain_lds(int L, int pitch) { return ckpt_rules::chain_lds(L, pitch); }
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


def test_asked_neighbours_give_a_split_of_the_tile(rules):
    """Whatever byte stands in the table, the place lies in the tile.  Lanes 0 .. 7 ask cells (qlo, j) and lanes 8 .. 11 cells
    (i, j0 - 1) above them; split q has the number q + 1, C_all of row i the number i + 1, an infeasible cell 0.  A split of the
    tile is taken, C_all of row qlo is split qlo, and in all other cases a lane has its own place of twelve."""
    for I, nq in [(0, 41), (3, 41), (0, 49), (7, 57), (20, 81), (0, 241)]:
        qlo = 8 * (I + 1)
        qhi = qlo + nq - 1  # = j0
        place = [x * nq // 12 for x in range(12)]
        assert len(set(place)) == 12 and place[0] == 0 and place[-1] < nq
        for x in range(12):
            assert all(0 <= rules.asked_split(x, n, qlo, nq) < nq for n in range(256))
            assert rules.asked_split(x, 0, qlo, nq) == place[x]
            for i in [qlo] if x < 8 else range(8 * I, qlo):
                assert rules.asked_split(x, i + 1, qlo, nq) == (0 if i == qlo else place[x]), (I, nq, x, i, "C_all")
                for q in range(i + 1, qhi + x + 1 if x < 8 else qhi):
                    want = q - qlo if qlo <= q <= qhi else place[x]
                    assert rules.asked_split(x, q + 1, qlo, nq) == want, (I, nq, x, i, q)


@pytest.mark.parametrize("tiles,pitch,B,passing", [
    (10, 2112, 64, 1), (22, 4160, 8, 1), (30, 1024, 16, 1), (4, 1024, 98, 1), (29, 1 << 16, 1 << 20, 1),
    (4, 1024, 97, 0), (22, 4160, 4, 0), (6, 1088, 40, 0), (10, 2112, 8, 0), (1, 64, 2, 0)])
def test_rows_pass_through_the_caches_by_their_size(rules, tiles, pitch, B, passing):
    """128 MB of rows in one diagonal: 64 x 96 stages, 8 x 192 and the smallest batch that is split unasked are above it,
    batches of the sizes that only a caller splits below."""
    assert rules.rows_pass(tiles, pitch, B) == passing


def test_whatever_a_work_group_reads_of_other_tiles_has_been_waited_for(rules):
    """Every shift up to the chain's largest one, every sub-chunk of a band: the lowest column of an operand and of a sample lie in
    chunks that are waited for, no chunk is waited for in vain, nothing is read above the band, and a sample stands on
    the right side of the columns that it bounds."""
    band = 12
    m0, first, last = 64 * band, 4 * band, 4 * band + 3
    column = lambda k: 16 * k + 15
    for reach in range(500):
        operands, samples = 64 * (band - rules.operand_chunks(reach)), 64 * (band - rules.sample_chunks(reach))
        assert operands <= m0 - reach and (reach == 0 or operands > m0 - reach - 64)
        lowest = m0
        for shift in {0, reach, *range(max(0, reach - 80), reach)}:
            for kk in range(first, last + 1):
                assert column(rules.left_below(kk)) == 16 * kk - 1 and column(rules.left_above(kk)) == 16 * kk + 15
                below, above = column(rules.right_below(kk, shift)), column(rules.right_above(kk, shift))
                assert below <= 16 * kk - shift < below + 17 and above - 16 < 16 * kk + 15 - shift <= above, (kk, shift)
                assert operands <= above <= m0 + 63, (reach, shift, kk)
                lowest = min(lowest, below, column(rules.left_below(kk)))
        assert samples <= lowest < samples + 64, (reach, lowest)


def test_differences_with_the_far_offset_are_32_bit_numbers_beyond_every_row(rules):
    """In the widest table that the one launch takes: a missing column less any shift, any column less the shift that reads
    nothing, and the one less the other."""
    widest = max(chunks for nblk in range(1, 33) for samples in (0, 1) for chunks in range(1, 4096)
                 if rules.flow_pays(nblk, chunks, ctypes.c_longlong(1), samples))
    assert widest == 1125
    far, row = rules.far_offset(), 4 * 64 * widest  # bytes of a row; columns and shifts lie in 0 .. row
    for column in (-far, 0, row - 4):
        for shift in (0, row, far):
            assert -2**31 <= column - shift < 2**31 and -2**31 <= shift - column < 2**31, (column, shift)
            if column < 0 or shift == far:
                assert column - shift <= -row - 16, (column, shift)
    assert far - row >= row  # cells that do not exist, from the bands below


def test_rows_of_a_short_chain_in_lds(rules):
    """Cells (q, j), 1 <= q <= j < L, one row each in the order of the table and no other; where a row begins is never
    below the first one nor beyond the end, also for the row below the last (read by nobody)."""
    rules.chain_lds.restype = ctypes.c_longlong
    for L in range(1, rules.chain_stages() + 1):
        rows = rules.chain_lds(L, 64) // (4 * 64)
        assert [rules.chain_row(L, q) + j - q for q in range(1, L) for j in range(q, L)] == list(range(rows)), L
        assert all(0 <= rules.chain_row(L, q) <= rows for q in range(1, L + 1)), L
