"""A batch's graph, whose samples in LDS run beside the rounds of the others,
against the eager execution: the same bits on every replay, with eager work
and changed states between the replays."""
import pytest
import torch

import synth
from paper_2504_17881_amd import prx as P
from gpu_util import basis_state, dev, to_dev, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,ns,max_grid", [
    (P.PRX_C64, [14, 15, 6, 16, 13], 0),
    (P.PRX_C64, [20, 9, 14], 3),
    (P.PRX_C64, [7, 14, 12], 0),                     # no rounds
    (P.PRX_C64, [15, 16], 0),                        # no samples in LDS
    (P.PRX_C64, [6 + i % 10 for i in range(300)], 0),  # samples in LDS by size
    (P.PRX_C128, [13, 14, 11, 16, 6], 0),
])
def test_graph_equals_eager(dtype, ns, max_grid):
    scheds, starts = [], []
    for i, n in enumerate(ns):
        x, z, phi = synth.random_pauli_rotations(n, 60, seed=900 + i)
        scheds.append(P.prx_sched_from_rotations(n, x, z, phi))
        starts.append(to_dev(synth.gaussian_state(n, i), dtype))
    psis = [t.clone() for t in starts]
    b = P.prx_batch_create(ns, scheds, dtype, [synth.basis_index(n) for n in ns])
    P.prx_batch_set_max_grid(b, max_grid)
    ws = workspace(P.prx_batch_workspace_bytes(b))
    ov = torch.zeros(2 * len(ns), dtype=torch.float64, device=dev())
    P.prx_batch_upload(b, psis, ws)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = P.prx_batch_graph(b, ws, ov, st)
    print(f"[batch graph S={len(ns)} n {min(ns)}..{max(ns)} dtype={dtype}]", flush=True)
    for rep in range(4):
        for t, p in zip(starts, psis):
            t.mul_(-1.0 if rep else 1.0)
            p.copy_(t)
        ov.zero_()
        P.prx_batch_execute(b, ws, ov)
        torch.cuda.synchronize()
        ref, ref_ov = [p.clone() for p in psis], ov.clone()
        for t, p in zip(starts, psis):
            p.copy_(t)
        ov.zero_()
        torch.cuda.synchronize()
        P.prx_graph_launch(g, st)
        st.synchronize()
        assert torch.equal(ov, ref_ov), rep
        for i, (p, r) in enumerate(zip(psis, ref)):
            assert torch.equal(torch.view_as_real(p), torch.view_as_real(r)), (rep, i, ns[i])
    P.prx_graph_destroy(g)
    P.prx_batch_destroy(b)
    for s in scheds:
        P.prx_sched_destroy(s)
