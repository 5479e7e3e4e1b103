"""complex64 plans that stay in LDS hand the norm to their last chunk, whatever
the number of their passes: short plans executed one after another stay at
norm 1."""
import pytest

import synth
from paper_2504_17881_amd import prx as P
from gpu_util import to_dev, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M,runs", [(4, 30, 1), (6, 100, 2000), (10, 100, 2000), (11, 60, 1),
                                      (12, 100, 500), (14, 300, 200)])
def test_norm_of_repeated_plans(n, M, runs):
    x, z, phi = synth.random_pauli_rotations(n, M, seed=31 + n)
    x[-5:] = [1, 2, 4, 8, 1]   # few rotations in the last chunk
    phi = phi / 8
    s = P.prx_sched_from_rotations(n, x, z, phi)
    pl = P.prx_plan_create(s, n, P.PRX_C64, 0, M, P.PRX_FUSED)
    info = P.prx_plan_get_info(pl)
    last = P.prx_plan_pass(pl, info["passes"] - 1)
    assert last["B"] == n and last["chunk_count"] > 1
    r = P.prx_plan_chunk(pl, last["chunk_begin"] + last["chunk_count"] - 1)["rot_count"]
    ws = workspace(info["workspace_bytes"])
    P.prx_plan_upload(pl, ws)
    psi = to_dev(1.5 * synth.gaussian_state(n, 1), P.PRX_C64)
    print(f"[norm n={n} M={M}] {runs} executions, {info['passes']} passes", flush=True)
    for _ in range(runs):
        P.prx_plan_execute(pl, psi, ws)
    red = workspace(P.prx_reduce_workspace_bytes(n))
    norm = P.prx_norm2(psi, n, P.PRX_C64, red) ** 0.5
    # what follows the hand-off: the last chunk's rotations, two FP32
    # coefficients each and two roundings per component, its factors and scale
    assert abs(norm - 1.0) <= (4 * r + 4) * 2.0 ** -24, norm - 1.0
    P.prx_plan_destroy(pl)
    P.prx_sched_destroy(s)
