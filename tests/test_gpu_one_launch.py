"""The kernel that fills small batches in one launch, against the oracle and against the kernels that take two launches a
block diagonal (every schedule asked for with list_split is made of those)."""
import numpy as np
import pytest

from gpu_util import assert_tables_equal
from paper_2302_02599_amd.binding import Solution
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
    (1, 0, 1, 1), (8, 63, 3, 9), (8, 64, 2, 30),   # one tile; one chunk and the first column of a second
    (9, 130, 2, 40), (16, 191, 5, 50),             # two blocks, one and eight columns in the last
    (17, 200, 2, 13), (24, 320, 3, 61),            # nine splits between the blocks; shifts that end inside four columns
    (25, 1000, 2, 333), (31, 449, 4, 0),           # first splits that do not wait for the last diagonal; no shift at all
    (41, 3000, 2, 2900),                           # shifts over more than 32 chunks, tiles below their frontier
    (90, 70, 2, 6),                                # a list of splits longer than a wave
    (254, 65, 1, 3),                               # the longest chain
    (64, 1100, 8, 90), (65, 1919, 5, 700),         # splits dropped by bounds; sizes of a third of the budget
    (88, 300, 39, 0), (200, 1300, 1, 60),          # no shift at all; lists of more splits than two waves have lanes
    (37, 1500, 29, 100),                           # five blocks, the shortest chains with bounds
])
def test_every_tile_in_one_launch(amd, oracle_mod, L, M, B, size_hi):
    import torch
    batch = random_chain_batch(L, M, B, 2100 + L, size_hi=size_hi, time_hi=900, overheads=True, own_wdelta=True, zero_sizes=size_hi == 0)
    print(f"case {batch.name}", flush=True)
    sol = amd.solve(batch)
    assert_tables_equal(oracle_mod, batch, sol, nthreads=4)
    apart = amd.solve(batch, list_split=1)
    for _ in range(3):  # into memory that held finished cells before
        again = amd.solve(batch, groups=1)
        torch.cuda.synchronize()
        assert torch.equal(again.cost[..., :M + 1], apart.cost[..., :M + 1]) and torch.equal(again.arg[..., :M + 1], apart.arg[..., :M + 1])


@pytest.mark.parametrize("L,M,B", [(8, 500, 28), (8, 500, 29), (16, 500, 75), (16, 500, 76), (20, 600, 66), (20, 600, 67),
                                   (32, 500, 109), (32, 500, 110), (32, 2000, 27), (32, 2000, 28),
                                   (56, 700, 58), (56, 700, 59), (96, 800, 44), (96, 800, 45)])
def test_both_sides_of_the_rule(amd, L, M, B):
    import torch
    batch = random_chain_batch(L, M, B, 2300 + L + B, size_hi=M // 20, time_hi=900)
    sol, apart = amd.solve(batch), amd.solve(batch, list_split=2)
    assert torch.equal(sol.cost[..., :M + 1], apart.cost[..., :M + 1]) and torch.equal(sol.arg[..., :M + 1], apart.arg[..., :M + 1])


@pytest.mark.parametrize("largest", [0, 50, 63, 64, 128])
def test_samples_below_the_lowest_operand(amd, oracle_mod, largest):
    """Splits dropped by bounds where a sample lies in the chunk below that of the lowest operand: no shift at all, but
    overheads, so that cells become feasible in different columns; and largest shifts at the edge of a chunk.  Into tables and a workspace
    that hold a solve of much smaller costs: whatever is read too early is too low."""
    import torch
    L, M, B = 66, 1100, 5  # nine blocks, 18 chunks
    batch = random_chain_batch(L, M, B, 2500 + largest, size_hi=60 if largest else 500, time_hi=100000, overheads=True, own_wdelta=True)
    batch.wa[:] = np.random.default_rng(2600 + largest).choice([0, 1, largest // 2, largest], size=batch.wa.shape)
    batch.wa[:, 1:-1:5] = largest
    batch.wabar[:] = batch.wa[:, 1:]
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in batch.dense()]
    cost = torch.empty((B, amd.ckpt_table_rows(L), amd.ckpt_row_pitch(M)), dtype=torch.int32, device="cuda")
    arg = torch.empty(cost.shape, dtype=torch.uint8, device="cuda")
    ws = torch.empty(amd.ckpt_workspace_bytes(L, M, B), dtype=torch.uint8, device="cuda")

    def fill(uf, ub):
        amd.ckpt_solve_batched(uf, ub, *dev[2:4], L, M, B, cost, arg, ws, wdelta=dev[4], of=dev[5], ob=dev[6])
        assert amd.ckpt_check_inputs(ws, L, M, B).tolist() == [0] * B

    print(f"case {batch.name}", flush=True)
    for _ in range(3):
        fill(torch.ones_like(dev[0]), torch.ones_like(dev[1]))
        fill(*dev[:2])
        assert_tables_equal(oracle_mod, batch, Solution(L, M, B, cost, arg, ws), nthreads=4)
