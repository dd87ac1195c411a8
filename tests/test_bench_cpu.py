"""bench.py's side measurements leave the headline's output alone."""
import pytest

import bench


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("agree", [True, False])
def test_one_call_line_keeps_the_plans_output(accumulate, agree):
    """the one-call products write a C of their own; what is left in the plan's,
    which the oracle checks afterwards, is what the plan's step wrote"""
    import torch
    Cd = torch.full((5, 3), 2.0, dtype=torch.float64).t().contiguous().t()
    writes = []

    def product(C):
        writes.append(C.data_ptr())
        C.copy_(C + 1.5 if accumulate else torch.full_like(C, 1.5))

    def plan_step():
        v = 1.5 if agree else 1.75
        Cd.copy_(Cd + v if accumulate else torch.full_like(Cd, v))
    line = bench.one_call_line(product, plan_step, Cd, lambda: None, 4, accumulate, 1e9)
    assert len(writes) == 2 + 4 + 1 and Cd.data_ptr() not in writes
    assert torch.all(Cd == (2.0 if accumulate else 0.0) + (1.5 if agree else 1.75))
    assert line["same_bits_as_plan"] is agree
    assert line["ms_per_call"] > 0 and line["tflops"] >= 0
