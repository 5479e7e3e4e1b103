"""Planner options that no plan takes are refused at every size, also where the
state would stay in one workgroup's LDS."""
import pytest

import synth
from paper_2504_17881_amd import prx as P


@pytest.mark.parametrize("dtype", [P.PRX_C64, P.PRX_C128])
@pytest.mark.parametrize("n", [3, 4, 10, 13, 14, 15, 20])
@pytest.mark.parametrize("opts", [dict(max_fuse=4097), dict(max_fuse=-1), dict(max_virtual=11),
                                  dict(span_max=6)])
def test_bad_options_are_refused(n, dtype, opts):
    s = P.prx_sched_from_rotations(n, *synth.random_pauli_rotations(n, 20, seed=n))
    with pytest.raises(P.PrxError):
        P.prx_plan_destroy(P.prx_plan_create(s, n, dtype, 0, 20, P.PRX_FUSED, opts))
    P.prx_plan_destroy(P.prx_plan_create(s, n, dtype, 0, 20, P.PRX_FUSED, dict(max_fuse=4096)))
    P.prx_sched_destroy(s)
