"""What a handle keeps of device memory after its state was read does not grow with the model."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [False, True], ids=["handle", "batch"])
def test_ordered_messages_are_given_back(batch):
    import torch
    m, L, rng = 1 << 21, 8, np.random.default_rng(4)  # 134 MB of messages
    edges = rng.permutation(2 * m).astype(np.int32).reshape(m, 2)
    un, pw = rng.random((2 * m, L), dtype=np.float32), rng.random((m, L, L), dtype=np.float32)
    print("CASE", m, L, batch, flush=True)
    with (M.Batch([W.Model(2 * m, L, edges, un, pw)]) if batch else M.Solver(2 * m, L, edges, un, pw)) as s:
        free = torch.cuda.mem_get_info()[0]
        for _ in range(2):
            U, phi = s.get_state(0)[:2] if batch else s.get_state()
        kept = free - torch.cuda.mem_get_info()[0]
    assert np.array_equal(U, un) and not phi.any()
    assert kept <= 4 * m + (32 << 20)  # (the list of slots, and what the runtime took)
