"""The complex64 renormalisation hand-off between passes: summed by the next
pass (up to 512 partials), by one workgroup, or by two launches, and the
changes from one form to another within a plan.

The input has norm 3, so only a plan whose hand-offs all carry the right norm
ends at the oracle's state of norm 1; relative 2-norm error at most
8 * 2^-24 * sqrt(M) + 1e-6 (a few ulps per rotation, random walk)."""
import math

import numpy as np
import pytest

import synth
from oracle import statevector as sv
from paper_2504_17881_amd import prx as P
from gpu_util import apply, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M,opts", [
    (16, 200, dict(tile_qubits=12, max_virtual=4)),              # 16 partials
    (20, 120, dict(tile_qubits=12)),                             # 256: four loads per lane
    (21, 120, dict(tile_qubits=12)),                             # 512: the longest direct sum
    (18, 120, dict(tile_qubits=12)),                             # 64: one load per lane
    (22, 60, dict(tile_qubits=12)),                              # 1024: one workgroup
    (17, 200, dict(tile_qubits=10, max_grid=100)),               # capped grid, ragged count
    (20, 120, dict(tile_qubits=14, max_virtual=10)),             # persistent workgroups
    (18, 300, dict(tile_qubits=13, max_virtual=3, span_max=4)),  # spans and tiles mixed
    (20, 200, dict(tile_qubits=14, max_virtual=2, span_max=1)),  # 2^11 and 2^6 partials mixed
    (25, 24, dict(tile_qubits=10, max_virtual=6)),               # 2^15: two launches
    (16, 200, dict(tile_qubits=12, renorm_every=3)),
])
def test_hand_off_forms(n, M, opts):
    x, z, phi = synth.random_pauli_rotations(n, M, seed=500 + n)
    phi = phi / 8
    # few distinct X masks in a row, so that spans and tiles both occur
    x[::3] &= np.uint64(0xff)
    psi0 = synth.gaussian_state(n, 3)
    ref = sv.c_apply_rotations(psi0, x, z, phi)
    s = P.prx_sched_from_rotations(n, x, z, phi)
    pl = P.prx_plan_create(s, n, P.PRX_C64, 0, M, P.PRX_FUSED, opts)
    passes = [P.prx_plan_pass(pl, i) for i in range(P.prx_plan_get_info(pl)["passes"])]
    P.prx_plan_destroy(pl)
    assert sum(p["norm_out"] for p in passes) >= 2
    print(f"[renorm n={n} opts={opts}] blocks {sorted({p['grid_blocks'] for p in passes})}",
          flush=True)
    t = to_dev(3.0 * psi0, P.PRX_C64)
    apply(t, n, P.PRX_C64, s, P.PRX_FUSED, opts=opts)
    P.prx_sched_destroy(s)
    assert rel_err(to_host(t), ref) <= 8 * 2.0 ** -24 * math.sqrt(M) + 1e-6
