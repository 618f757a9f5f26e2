"""Sizes that the binding checks tensors against follow the numbers of the call, whatever type these have.  CPU only: tables that
are not given are refused by the library, behind the binding's own checks."""
import numpy as np
import pytest
import torch

import paper_2302_02599_amd as amd
from paper_2302_02599_amd import binding


def test_sizes_of_a_number_that_changes_in_place():
    L, M, B = torch.tensor(8), np.array(64), torch.tensor(1)
    for stages, chains in [(8, 1), (100, 1), (8, 3), (254, 2)]:
        L.fill_(stages), B.fill_(chains)
        assert binding._sizes(L, M, B) == (amd.ckpt_table_elems(stages, 64, chains), amd.ckpt_workspace_bytes(stages, 64, chains))
        assert binding._walk_bytes(L, B) == amd.ckpt_schedule_workspace_bytes(stages, chains)
        assert binding._sizes(stages, 64, chains) == binding._sizes(L, M, B)


@pytest.mark.parametrize("number", [int, np.int64, np.int32, np.array, torch.tensor])
def test_numbers_of_any_integer_type_are_taken(number):
    with pytest.raises(amd.CkptError, match="bad argument"):
        amd.ckpt_select_plan(None, number(8), number(64), number(1), None, None, stream=0)
    with pytest.raises(amd.CkptError, match="bad argument"):
        amd.ckpt_schedule_batched(None, None, None, number(8), number(64), number(1), None, None, 10, None, None, stream=0)
