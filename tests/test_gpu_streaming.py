"""States above 256 MiB, whose plain sweeps (and, from 1 GiB, scaling) use
non-temporal accesses, and plain sweeps beside fused passes, which follow theirs: against a
plain torch form of the rotation in complex128 (itself against the oracle).
complex128 at 1e-13, complex64 at 8 * 2^-24 * sqrt(M) + 1e-6."""
import math

import numpy as np
import pytest
import torch

import synth
from oracle import statevector as sv
from paper_2504_17881_amd import prx as P
from gpu_util import apply, dev, rel_err, tdtype, to_dev, to_host, workspace

pytestmark = pytest.mark.gpu


def _rotate(psi, n, x, z, phi):
    """exp(i phi P) psi with P = i^|x&z| X^x Z^z, in complex128."""
    k = torch.arange(1 << n, device=dev()) ^ int(x)
    s = k & int(z)
    for sh in (32, 16, 8, 4, 2, 1):
        s ^= s >> sh
    sign = (1 - 2 * (s & 1)).to(torch.float64)
    w = 1j * math.sin(phi) * 1j ** bin(int(x) & int(z)).count("1")
    return math.cos(phi) * psi + w * sign * psi[k]


def _strings(n, M, seed):
    x, z, phi = synth.random_pauli_rotations(n, M, seed=seed)
    x[1::3] = 0
    z[1::3] |= np.uint64(1)
    return x, z, phi


def test_reference():
    n, M = 10, 12
    x, z, phi = _strings(n, M, 5)
    psi = synth.gaussian_state(n, 1)
    t = to_dev(psi, P.PRX_C128)
    for r in zip(x, z, phi):
        t = _rotate(t, n, *r)
    assert rel_err(to_host(t), sv.c_apply_rotations(psi, x, z, phi)) <= 1e-13


@pytest.mark.parametrize("dtype,n", [(P.PRX_C64, 25), (P.PRX_C64, 27), (P.PRX_C128, 25)])
def test_plain_and_scale(dtype, n):
    M = 3
    x, z, phi = _strings(n, M, 70 + n)
    g = torch.Generator(device=dev()).manual_seed(n)
    psi = torch.randn(1 << n, dtype=tdtype(dtype), device=dev(), generator=g)
    ref = psi.to(torch.complex128)
    for r in zip(x, z, phi):
        ref = _rotate(ref, n, *r)
    s = P.prx_sched_from_rotations(n, x, z, phi)
    print(f"[streaming plain n={n} dtype={dtype}]", flush=True)
    apply(psi, n, dtype, s, P.PRX_PLAIN)
    P.prx_sched_destroy(s)
    tol = 1e-13 if dtype == P.PRX_C128 else 8 * 2.0 ** -24 * math.sqrt(M) + 1e-6
    norm = float(torch.linalg.vector_norm(ref))
    assert float(torch.linalg.vector_norm(psi.to(torch.complex128) - ref)) <= tol * norm
    P.prx_renormalize(psi, n, dtype, workspace(P.prx_reduce_workspace_bytes(n)))
    assert float(torch.linalg.vector_norm(psi.to(torch.complex128) - ref / norm)) <= tol


@pytest.mark.parametrize("dtype,n", [(P.PRX_C64, 16), (P.PRX_C128, 16), (P.PRX_C64, 22)])
def test_plain_beside_fused(dtype, n):
    # one diagonal-free string with a fresh high X mask between tile runs
    M = 9
    x, z, phi = synth.random_pauli_rotations(n, M, seed=n)
    phi = phi / 8  # one piece each
    x &= np.uint64(0x3f)
    x[4] = np.uint64((1 << n) - 64)
    opts = dict(tile_qubits=10, max_virtual=-1, span_max=1)
    s = P.prx_sched_from_rotations(n, x, z, phi)
    pl = P.prx_plan_create(s, n, dtype, 0, M, P.PRX_FUSED, opts)
    info = P.prx_plan_get_info(pl)
    P.prx_plan_destroy(pl)
    print(f"[streaming beside fused n={n} dtype={dtype}] {info}", flush=True)
    assert info["plain_passes"] >= 1 and info["tile_passes"] >= 1
    psi = synth.gaussian_state(n, 2)
    t = to_dev(psi, dtype)
    apply(t, n, dtype, s, P.PRX_FUSED, opts=opts)
    P.prx_sched_destroy(s)
    tol = 1e-12 if dtype == P.PRX_C128 else 8 * 2.0 ** -24 * math.sqrt(M) + 1e-6
    assert rel_err(to_host(t), sv.c_apply_rotations(psi, x, z, phi)) <= tol
