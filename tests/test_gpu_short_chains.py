"""Chains of up to thirteen stages, a work-group each with the table in LDS, against the oracle and against the kernels of
longer chains (every schedule asked for with list_split is made of those)."""
import pytest

from gpu_util import assert_tables_equal
from workloads import random_chain_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amd():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2302_02599_amd as amd
    amd.load_library()
    return amd


@pytest.mark.parametrize("L,M,B,size_hi", [
    (1, 0, 1, 1), (1, 1023, 2, 9), (2, 63, 3, 5), (3, 64, 2, 100), (5, 300, 4, 0), (7, 130, 2, 40),  # no shift at all; shifts beyond the budget
    (8, 1023, 3, 300), (8, 1024, 2, 300),  # the widest table with a thread a column, and the next one
    (9, 64, 2, 13), (10, 700, 3, 90), (12, 447, 5, 2), (13, 511, 300, 30),  # more work-groups than compute units
    (13, 512, 2, 30), (14, 300, 2, 30),  # beyond LDS; longer
])
def test_short_chains(amd, oracle_mod, L, M, B, size_hi):
    import torch
    batch = random_chain_batch(L, M, B, 4100 + L, size_hi=size_hi, time_hi=900, overheads=True, own_wdelta=True, zero_sizes=size_hi == 0)
    print(f"case {batch.name}", flush=True)
    sol = amd.solve(batch)
    assert_tables_equal(oracle_mod, batch, sol, nthreads=4)
    apart = amd.solve(batch, list_split=1)
    assert torch.equal(sol.cost[..., :M + 1], apart.cost[..., :M + 1]) and torch.equal(sol.arg[..., :M + 1], apart.arg[..., :M + 1])


@pytest.mark.parametrize("L", [1, 8, 13])
def test_times_up_to_the_largest_and_flags(amd, L):
    import torch
    batch = random_chain_batch(L, 90, 4, 4200 + L, size_hi=9, time_hi=900)
    batch.wabar[:] = batch.wa[:, 1:] + 1
    batch.uf[1], batch.ub[1] = (1 << 30) // (L + 1), (1 << 30) - 1   # sums close below 2^30
    batch.uf[2, L - 1] = -5
    batch.wa[3, L] = (1 << 28) + 1
    batch.wabar[3, L - 1] = (1 << 28) + 1
    sol, apart = amd.solve(batch, check=False), amd.solve(batch, check=False, list_split=1)
    flags = [amd.ckpt_check_inputs(s.workspace, s.L, s.M, s.B).tolist() for s in (sol, apart)]
    assert flags[0] == flags[1] and flags[0][0] == 0 and flags[0][2] & 1 and flags[0][3] & 4
    assert torch.equal(sol.cost[:2, :, :91], apart.cost[:2, :, :91]) and torch.equal(sol.arg[:2, :, :91], apart.arg[:2, :, :91])


@pytest.mark.parametrize("L", [2, 7, 8, 9, 13])
def test_forward_times_that_add_up_to_the_sentinel(amd, oracle_mod, L):
    """2^30 is flagged, one less is not and its table is the oracle's."""
    import torch
    batch = random_chain_batch(L, 90, 3, 4300 + L, size_hi=9, time_hi=900)
    for b, total in ((0, (1 << 30) - 1), (1, 1 << 30)):
        batch.uf[b] = total // L
        batch.uf[b, L // 2] += total - L * (total // L)
        assert int(batch.uf[b].sum(dtype="int64")) == total
    sol, apart = amd.solve(batch, check=False), amd.solve(batch, check=False, list_split=1)
    for s in (sol, apart):
        assert amd.ckpt_check_inputs(s.workspace, s.L, s.M, s.B).tolist() == [0, 2, 0]
        assert_tables_equal(oracle_mod, batch, s, chains=[0, 2])


def test_first_solve_of_a_process_inside_a_capture():
    """A table of more LDS than a kernel has by default, captured without ckpt_init by a process that has solved nothing:
    what the kernel has to be allowed is no work for a stream.  Every replay gives the tables of the eager solve."""
    import os
    import subprocess
    import sys
    code = r'''
import numpy as np, torch, sys
sys.path.insert(0, %r)
import paper_2302_02599_amd as amd
from workloads import random_chain_batch
batch = random_chain_batch(13, 500, 20, 4400, size_hi=60, time_hi=900)
L, M, B = batch.L, batch.M, batch.B
ins = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (batch.uf, batch.ub, batch.wa, batch.wabar)]
cost = torch.empty((B, amd.ckpt_table_rows(L), amd.ckpt_row_pitch(M)), dtype=torch.int32, device="cuda")
arg = torch.empty(cost.shape, dtype=torch.uint8, device="cuda")
ws = torch.empty(amd.ckpt_workspace_bytes(L, M, B), dtype=torch.uint8, device="cuda")
side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
torch.cuda.synchronize()
with torch.cuda.graph(graph, stream=side):
    amd.ckpt_solve_batched(*ins, L, M, B, cost, arg, ws)
same = []
for _ in range(3):
    cost.fill_(-1), arg.fill_(99)
    graph.replay()
    torch.cuda.synchronize()
    ref = amd.solve(batch, list_split=1)
    same.append(torch.equal(cost[..., :M + 1], ref.cost[..., :M + 1]) and torch.equal(arg[..., :M + 1], ref.arg[..., :M + 1]))
print("RESULT", amd.load_library().ckpt_kernel_name_of(3, L, M, B), same)
''' % os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert "RESULT b'chain_kernel' [True, True, True]" in out.stdout, out.stdout[-2000:] + out.stderr[-2000:]
