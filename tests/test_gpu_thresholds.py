"""The threshold tables and per-chain scalars, written by work-groups of a few rows: lengths at the edges of a wave, of a
work-group's rows and of its waves, few chains and (sixteen rows a work-group) many, against the oracle."""
import dataclasses

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


@pytest.mark.parametrize("L", [1, 3, 4, 5, 16, 17, 63, 64, 65, 128, 129, 254])
@pytest.mark.parametrize("many", [False, True])
def test_rows_and_chains(amd, oracle_mod, L, many):
    import torch
    B = 1024 // ((L + 3) // 4) + 1 if many else 2
    batch = random_chain_batch(L, 20, B, 3100 + L, size_hi=7, time_hi=900, overheads=True, own_wdelta=True)
    print(f"case {batch.name}", flush=True)
    sol = amd.solve(batch)
    if L <= 65 or not many:
        assert_tables_equal(oracle_mod, batch, sol, nthreads=4)
    else:  # the same chains a few at a time
        for b in (0, B - 1):
            arrays = {k: getattr(batch, k)[b:b + 1] for k in ("uf", "ub", "wa", "wabar", "wdelta", "of", "ob")}
            one = amd.solve(dataclasses.replace(batch, B=1, **arrays))
            assert torch.equal(sol.cost[b, :, :21], one.cost[0, :, :21]) and torch.equal(sol.arg[b, :, :21], one.arg[0, :, :21])


@pytest.mark.parametrize("where", ["first", "wave", "last"])
@pytest.mark.parametrize("field,value,bit", [("uf", -1, 1), ("wdelta", -1, 1), ("ub", 1 << 30, 2), ("ob", (1 << 28) + 1, 4), ("wabar", 0, 8)])
def test_input_flags_of_any_stage(amd, where, field, value, bit):
    L = 200
    batch = random_chain_batch(L, 20, 3, 77, size_hi=7, time_hi=900, overheads=True, own_wdelta=True)
    batch.wa[:] = abs(batch.wa) + 1
    batch.wabar[:] = batch.wa[:, 1:] + 1
    at = {"first": 0, "wave": 64, "last": getattr(batch, field).shape[1] - 1}[where]
    getattr(batch, field)[1, at] = value
    sol = amd.solve(batch, check=False)
    assert amd.ckpt_check_inputs(sol.workspace, sol.L, sol.M, sol.B).tolist() == [0, bit, 0]
