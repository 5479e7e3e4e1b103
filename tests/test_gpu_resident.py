"""Plans whose state stays in one workgroup's LDS (4 to 14 qubits at
complex64, 4 to 13 at complex128): one launch for all passes, against the
oracle.  complex128 at 1e-12; complex64 at 8 * 2^-24 * sqrt(M) + 1e-6 (a few
ulps per rotation, random walk), from a state of norm 3 where the plan has
several passes, so that every in-kernel renormalisation counts."""
import math

import numpy as np
import pytest
import torch

import synth
from oracle import statevector as sv
from paper_2504_17881_amd import prx as P
from gpu_util import apply, rel_err, to_dev, to_host, workspace

pytestmark = pytest.mark.gpu


def _rotations(n, M, seed):
    """Random strings with diagonal runs and angles up to pi."""
    x, z, phi = synth.random_pauli_rotations(n, M, seed=seed)
    x[::7] = 0
    z[::7] |= np.uint64(1)
    return x, z, phi


@pytest.mark.parametrize("dtype", [P.PRX_C128, P.PRX_C64])
@pytest.mark.parametrize("n,M", [(4, 300), (5, 150), (6, 40), (9, 300), (10, 700), (11, 1),
                                 (11, 260), (12, 500), (13, 400), (14, 300)])
def test_resident_plans(n, M, dtype):
    x, z, phi = _rotations(n, M, 900 + n)
    s = P.prx_sched_from_rotations(n, x, z, phi)
    pl = P.prx_plan_create(s, n, dtype, 0, M, P.PRX_FUSED)
    info = P.prx_plan_get_info(pl)
    passes = [P.prx_plan_pass(pl, i) for i in range(info["passes"])]
    if n <= (14 if dtype == P.PRX_C64 else 13):
        assert all(p["kind"] == 2 and p["B"] == n and p["grid_blocks"] == 1 for p in passes)
        assert info["passes"] == -(-info["kernel_rotations"] // 128)
    several = dtype == P.PRX_C64 and len(passes) > 1
    psi0 = synth.gaussian_state(n, 2)
    ref = sv.c_apply_rotations(psi0, x, z, phi)
    start = to_dev((3.0 if several else 1.0) * psi0, dtype)
    print(f"[resident n={n} M={M} dtype={dtype}] {len(passes)} passes", flush=True)
    got = start.clone()
    apply(got, n, dtype, s, P.PRX_FUSED)
    tol = 1e-12 if dtype == P.PRX_C128 else 8 * 2.0 ** -24 * math.sqrt(info["kernel_rotations"]) + 1e-6
    assert rel_err(to_host(got), ref) <= tol
    # pass by pass (the timed form) and replayed as a graph: the same bits
    ws = workspace(info["workspace_bytes"])
    P.prx_plan_upload(pl, ws)
    timed = start.clone()
    ms, _ = P.prx_plan_execute_timed(pl, timed, ws)
    assert torch.equal(timed, got) and (ms > 0).all()
    stream = torch.cuda.Stream()
    psi = start.clone()
    torch.cuda.synchronize()
    g = P.prx_plan_graph(pl, psi, ws, stream)
    for _ in range(3):
        psi.copy_(start)
        torch.cuda.synchronize()
        P.prx_graph_launch(g, stream)
        stream.synchronize()
        assert torch.equal(psi, got)
    P.prx_graph_destroy(g)
    P.prx_plan_destroy(pl)
    P.prx_sched_destroy(s)


@pytest.mark.parametrize("n,dtype", [(14, P.PRX_C64), (13, P.PRX_C128), (12, P.PRX_C128)])
def test_few_frames_go_to_tile_passes(n, dtype):
    """Rotations that all fit one or two tile frames: the largest resident
    sizes take tile passes of several workgroups instead."""
    M = 240
    x, z, phi = synth.random_pauli_rotations(n, M, seed=n)
    x &= np.uint64(0x3ff)
    phi = phi / 4
    s = P.prx_sched_from_rotations(n, x, z, phi)
    pl = P.prx_plan_create(s, n, dtype, 0, M, P.PRX_FUSED)
    assert all(P.prx_plan_pass(pl, i)["B"] < n for i in range(P.prx_plan_get_info(pl)["passes"]))
    P.prx_plan_destroy(pl)
    psi0 = synth.gaussian_state(n, 2)
    got = to_dev(psi0, dtype)
    print(f"[few frames n={n} dtype={dtype}]", flush=True)
    apply(got, n, dtype, s, P.PRX_FUSED)
    tol = 1e-12 if dtype == P.PRX_C128 else 8 * 2.0 ** -24 * math.sqrt(M) + 1e-6
    assert rel_err(to_host(got), sv.c_apply_rotations(psi0, x, z, phi)) <= tol
    P.prx_sched_destroy(s)
