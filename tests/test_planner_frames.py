"""Frames of fused plans just above the tile size: a frame's XOR masks may
span more than n - B of the index bits above the low ones (host interpreter
against the oracle), and the default frame sizes by state size."""
import numpy as np
import pytest

import synth
from oracle import statevector as sv
from paper_2504_17881_amd import prx as P
from plan_interp import run_plan


@pytest.mark.parametrize("n,dtype,opts", [
    (13, P.PRX_C64, dict(tile_qubits=12)),
    (14, P.PRX_C128, None),
    (14, P.PRX_C128, dict(tile_qubits=13, max_virtual=9)),
    (15, P.PRX_C64, dict(tile_qubits=14, max_virtual=10)),
    (15, P.PRX_C64, None),
    (14, P.PRX_C64, dict(tile_qubits=10, chunk_rank=3, max_virtual=6)),
    (15, P.PRX_C128, dict(commuting=1)),
])
def test_wide_frames_match_oracle(n, dtype, opts):
    M = 150
    x, z, phi = synth.random_pauli_rotations(n, M, seed=70 + n)
    x[::7] = 0
    z[::7] |= np.uint64(1)
    s = P.prx_sched_from_rotations(n, x, z, phi)
    pl = P.prx_plan_create(s, n, dtype, 0, M, P.PRX_FUSED, opts)
    info = P.prx_plan_get_info(pl)
    tiles = [p for p in (P.prx_plan_pass(pl, i) for i in range(info["passes"])) if p["kind"] == 2]
    assert max(p["g"] for p in tiles) > n - info["tile_qubits"]
    assert all(p["b"] >= 4 and p["b"] + p["g"] == p["B"] for p in tiles)
    psi0 = synth.gaussian_state(n, 3)
    err = np.linalg.norm(run_plan(pl, psi0, n) - sv.c_apply_rotations(psi0, x, z, phi))
    # records hold FP32 coefficients at complex64: 2^-24 each, random signs
    assert err <= (1e-11 if dtype == P.PRX_C128 else 8 * 2.0 ** -24 * M ** 0.5)
    P.prx_plan_destroy(pl)
    P.prx_sched_destroy(s)


@pytest.mark.parametrize("dtype,sizes", [
    (P.PRX_C64, {15: 12, 18: 12, 19: 13, 22: 13, 23: 14, 34: 14}),
    (P.PRX_C128, {14: 11, 18: 11, 19: 12, 33: 12}),
])
def test_default_frame_sizes(dtype, sizes):
    for n, B in sizes.items():
        x, z, phi = synth.random_pauli_rotations(n, 140, seed=n)
        s = P.prx_sched_from_rotations(n, x, z, phi)
        pl = P.prx_plan_create(s, n, dtype, 0, 140, P.PRX_FUSED)
        assert P.prx_plan_get_info(pl)["tile_qubits"] == B
        P.prx_plan_destroy(pl)
        # named frames keep their defaults
        pl = P.prx_plan_create(s, n, dtype, 0, 140, P.PRX_FUSED, dict(max_virtual=3))
        assert P.prx_plan_get_info(pl)["tile_qubits"] == (12 if dtype == P.PRX_C64 else 11)
        P.prx_plan_destroy(pl)
        P.prx_sched_destroy(s)


@pytest.mark.parametrize("n", [19, 22, 23, 28])
def test_narrow_frames_where_wide_ones_save_no_pass(n):
    # one high X mask: one pass in frames of any size
    M = 60
    x, z, phi = synth.random_pauli_rotations(n, M, seed=n)
    x = (x & np.uint64(0x7f)) | np.uint64(1 << (n - 1))
    s = P.prx_sched_from_rotations(n, x, z, phi / 8)
    pl = P.prx_plan_create(s, n, P.PRX_C64, 0, M, P.PRX_FUSED)
    info = P.prx_plan_get_info(pl)
    assert info["tile_qubits"] == 12 and info["passes"] == 1
    P.prx_plan_destroy(pl)
    P.prx_sched_destroy(s)


@pytest.mark.parametrize("dirs", [5, 6, 7])
@pytest.mark.parametrize("n,dtype,B", [(14, P.PRX_C64, 12), (13, P.PRX_C128, 11),
                                       (12, P.PRX_C128, 11)])
def test_plans_too_slow_in_lds_take_the_frames_they_were_compared_with(n, dtype, B, dirs):
    """A state that one workgroup's LDS holds takes tile passes where few of
    them do; those are the frames of B - 4 masks that the rule counted, not
    frames of n - B."""
    M = 480
    x, z, phi = synth.random_pauli_rotations(n, M, seed=n + dirs)
    x &= np.uint64(((1 << dirs) - 1) << (n - dirs) | 15)
    s = P.prx_sched_from_rotations(n, x, z, phi / 8)
    named = P.prx_plan_create(s, n, dtype, 0, M, P.PRX_FUSED,
                              dict(tile_qubits=B, max_virtual=B - 4))
    fewest = P.prx_plan_get_info(named)["passes"]
    P.prx_plan_destroy(named)
    assert fewest == 4
    pl = P.prx_plan_create(s, n, dtype, 0, M, P.PRX_FUSED)
    info = P.prx_plan_get_info(pl)
    assert info["tile_qubits"] == B and info["passes"] == fewest
    P.prx_plan_destroy(pl)
    P.prx_sched_destroy(s)
