"""The kernel that a profiled solve names is the one that ran, and the cells that it counts are those of the table."""
import numpy as np
import pytest

import paper_2302_02599_amd as amd
from workloads import random_chain_batch

SHAPES = [(8, 64, 1, "chain_kernel"), (13, 500, 4, "chain_kernel"),
          (14, 500, 4, "flow_kernel"), (24, 512, 1, "flow_kernel"), (53, 777, 5, "flow_kernel"), (66, 1100, 5, "flow_kernel"),
          (16, 500, 76, "tile_rows_kernel"), (20, 600, 67, "tile_rows_kernel"), (96, 800, 45, "tile_rows_kernel")]


@pytest.mark.parametrize("L,M,B,rows", SHAPES)
def test_name_of_the_kernel_that_fills_a_batch(L, M, B, rows):
    lib = amd.load_library()
    names = [lib.ckpt_kernel_name_of(k, L, M, B) for k in range(5)]
    assert names == [b"precompute_kernel", b"frontier_kernel", b"gemm_kernel", rows.encode(), None]
    assert lib.ckpt_kernel_name_of(3, 0, M, B) == lib.ckpt_kernel_name(3) == b"tile_rows_kernel"


@pytest.mark.gpu
@pytest.mark.parametrize("L,M,B,rows", SHAPES)
def test_profiled_solve(L, M, B, rows):
    """One launch, without a precomputation or behind it, or two a diagonal; and 320 bytes for every cell and 64 columns, by whichever
    kernel it is stored (a row finished by the block product counts there; what it hands over counts again)."""
    import torch
    batch = random_chain_batch(L, M, B, 4700 + L, size_hi=M // 20, time_hi=900)
    print(f"case {batch.name}", flush=True)
    sol = amd.solve(batch)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    cost, arg = torch.empty_like(sol.cost), torch.empty_like(sol.arg)
    kinds = amd.ckpt_solve_profiled(up(batch.uf), up(batch.ub), up(batch.wa), up(batch.wabar), L, M, B, cost, arg, sol.workspace,
                                    count_bytes=True)
    assert torch.equal(cost[..., :M + 1], sol.cost[..., :M + 1]) and torch.equal(arg[..., :M + 1], sol.arg[..., :M + 1])
    launches = {name: v[1] for name, v in kinds.items()}
    blocks = -(-L // 8)
    one = rows != "tile_rows_kernel"
    assert launches == {"precompute_kernel": int(rows != "chain_kernel"), "frontier_kernel": launches["frontier_kernel"],
                        "gemm_kernel": 0 if one else max(0, blocks - 2), rows: 1 if one else blocks}
    cells = 320 * amd.ckpt_table_elems(L, M, B) // 64
    if one:
        assert kinds[rows][3] == cells and (kinds[rows][2] == 0) == (rows == "chain_kernel" or blocks == 1)
    else:
        assert kinds[rows][3] + kinds["gemm_kernel"][3] >= cells
