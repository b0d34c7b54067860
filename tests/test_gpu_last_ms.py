"""The time that an FP32 handle reports after an adjoint forward is that of its FP32 run,
also where the FP64 run beside it in the launch takes much longer."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("every", [40, 15])
def test_time_of_the_fp32_run(every):
    model = W.uniform(100, 64, seed=1)  # an FP64 update of 64 labels takes half as long again as an FP32 one
    own = {}
    for dtype in (np.float32, np.float64):
        with M.Solver.from_model(model.astype(dtype)) as s:
            s.iterate(40)
            s.iterate(40)
            own[dtype] = s.last_iterate_ms()
    with M.Solver.from_model(model) as s:
        s.adjoint_forward(40, every)
        s.adjoint_forward(40, every)
        ms = s.last_iterate_ms()
    print("CASE", every, "FP32", own[np.float32], "FP64", own[np.float64], "forward", ms, flush=True)
    assert 0.5 * own[np.float32] <= ms <= 0.5 * (own[np.float32] + own[np.float64])
