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
