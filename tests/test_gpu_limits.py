"""Calls at the edges of what the entry points take: they are refused or answered as
their plain definition is, whatever form the library gives them."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# A noise variance beyond the float32 range: a mixed fit stores its windows in float32, so
# the pivots are infinite, no likelihood exists and the call is refused (block None: no
# factor failed).  In float64 the same holds beyond the float64 range.
@pytest.mark.parametrize("precision,log_sn2", [("mixed", 89.0), ("mixed", 100.0), ("mixed", 708.0), ("mixed", 800.0),
                                               ("fp64", 709.9), ("fp64", 800.0)])
@pytest.mark.parametrize("B", [0, 2])
def test_variance_beyond_the_storage_type_is_refused(lib, precision, log_sn2, B):
    p = synth.make_random(seed=7, n=600, d=3, M=5, s=40, n_u=5, B=B, uneven=(60, 180), sn2=0.05)
    p.log_hyp = p.log_hyp.copy()
    p.log_hyp[-1] = log_sn2
    problem = lib.LmlProblem.from_problem(p, precision=precision)
    for call in (lambda: lib.fit_problem(p, precision=precision).free(), lambda: problem(p.log_hyp, grad=False),
                 lambda: problem(p.log_hyp, grad=True)):
        with pytest.raises(lib.LmaError) as e:
            call()
        assert e.value.status == lib.LMA_E_NOT_PD and e.value.block is None


# 2^30 points (a launch holds fewer than 2^32 threads) and one more: every count and label
def test_bounded_assignment_of_two_to_the_thirty_points(lib):
    import torch
    n = 2 ** 30 + 1
    P = torch.rand((n, 1), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    C = torch.tensor([[0.25], [0.75]], dtype=torch.float64, device="cuda")
    label, count, rounds = lib.bounded_assign(P, C, 0, n)
    nearer = (P[:, 0] - 0.25) ** 2 <= (P[:, 0] - 0.75) ** 2   # ties to the lower index
    assert rounds == 1 and bool(torch.equal(label == 0, nearer))
    assert count.tolist() == [int(nearer.sum()), n - int(nearer.sum())]
    del P, label, nearer
    lib.release_cache()
    torch.cuda.empty_cache()
