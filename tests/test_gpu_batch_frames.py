"""Batches with more resident samples than one launch takes, and tile samples
in frames of every size that a batch chooses, against the oracle: complex128
at 1e-12, complex64 at 8 * 2^-24 * sqrt(N) + 1e-6."""
import math

import numpy as np
import pytest
import torch

import synth
from oracle import statevector as sv
from paper_2504_17881_amd import prx as P
from gpu_util import basis_state, dev, rel_err, to_dev, to_host, workspace

pytestmark = pytest.mark.gpu


def _run(ns, M, dtype, seed, max_grid=0):
    """Random strings with diagonal ones among them, Gaussian states."""
    rots, scheds, starts = [], [], []
    for i, n in enumerate(ns):
        x, z, phi = synth.random_pauli_rotations(n, M, seed=seed + i)
        x[::5] = 0
        z[::5] |= np.uint64(1)
        rots.append((x, z, phi))
        scheds.append(P.prx_sched_from_rotations(n, x, z, phi))
        starts.append(to_dev(synth.gaussian_state(n, i), dtype) if n < 20
                      else basis_state(n, 5, dtype))
    basis = [synth.basis_index(n) for n in ns]
    psis = [t.clone() for t in starts]
    b = P.prx_batch_create(ns, scheds, dtype, basis)
    P.prx_batch_set_max_grid(b, max_grid)
    ws = workspace(P.prx_batch_workspace_bytes(b))
    ovd = torch.zeros(2 * len(ns), dtype=torch.float64, device=dev())
    P.prx_batch_upload(b, psis, ws)
    print(f"[batch frames S={len(ns)} n {min(ns)}..{max(ns)} dtype={dtype}]", flush=True)
    P.prx_batch_execute(b, ws, ovd)
    P.prx_batch_check(b, ws)
    ov = ovd.cpu().numpy()
    P.prx_batch_destroy(b)
    for s in scheds:
        P.prx_sched_destroy(s)
    return rots, starts, psis, basis, ov


def _check(ns, M, dtype, got):
    rots, starts, psis, basis, ov = got
    tol = 1e-12 if dtype == P.PRX_C128 else 8 * 2.0 ** -24 * math.sqrt(3 * M) + 1e-6
    for i, n in enumerate(ns):
        ref = sv.c_apply_rotations(to_host(starts[i]), *rots[i])
        out = to_host(psis[i])
        assert rel_err(out, ref) <= tol, (i, n)
        assert ov[2 * i] == out[basis[i]].real and ov[2 * i + 1] == out[basis[i]].imag


@pytest.mark.parametrize("dtype", [P.PRX_C64, P.PRX_C128])
@pytest.mark.parametrize("max_grid", [0, 7])
def test_more_residents_than_one_launch(dtype, max_grid):
    top = 14 if dtype == P.PRX_C64 else 13
    ns = [6 + i % (top - 5) for i in range(270)]
    _check(ns, 40, dtype, _run(ns, 40, dtype, 3000, max_grid))


@pytest.mark.parametrize("dtype,ns,max_grid", [
    (P.PRX_C64, [15, 14, 17, 15], 0),           # 12-qubit frames
    (P.PRX_C64, [22, 15, 21, 9, 22], 0),        # 13
    (P.PRX_C64, [24, 25, 13, 24], 0),           # 14: 4096 items over the resident workgroups
    (P.PRX_C64, [24, 24], 5),
    (P.PRX_C128, [14, 15, 13, 14], 0),          # 11
    (P.PRX_C128, [19, 14, 18, 8], 0),           # 12
    (P.PRX_C128, [19, 14, 18], 3),
])
def test_tile_samples_of_every_frame_size(dtype, ns, max_grid):
    M = 24
    _check(ns, M, dtype, _run(ns, M, dtype, 4000, max_grid))


def test_more_tile_samples_than_lanes():
    """More passes in a round than a wave has lanes."""
    ns = [15 + i % 2 for i in range(150)]
    _check(ns, 20, P.PRX_C64, _run(ns, 20, P.PRX_C64, 5000))
