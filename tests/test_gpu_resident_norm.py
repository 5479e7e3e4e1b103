"""complex64 plans that stay in LDS hand the norm to their last chunk, whatever
the number of their passes: short plans executed one after another stay at
norm 1, and their error stays near that of plain FP32."""
import numpy as np
import pytest

import synth
from paper_2504_17881_amd import prx as P
from gpu_util import to_dev, to_host, workspace

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


@pytest.mark.parametrize("every", [1, 2, 3])
@pytest.mark.parametrize("M", [3, 128, 131, 259])
def test_timed_form_with_a_last_pass_of_one_chunk(M, every):
    n = 8
    x, z, phi = synth.random_pauli_rotations(n, M, seed=5)
    s = P.prx_sched_from_rotations(n, x, z, phi / 8)
    pl = P.prx_plan_create(s, n, P.PRX_C64, 0, M, P.PRX_FUSED, dict(renorm_every=every))
    ws = workspace(P.prx_plan_get_info(pl)["workspace_bytes"])
    P.prx_plan_upload(pl, ws)
    a = to_dev(1.5 * synth.gaussian_state(n, 1), P.PRX_C64)
    b = a.clone()
    print(f"[timed M={M} every={every}]", flush=True)
    P.prx_plan_execute(pl, a, ws)
    P.prx_plan_execute_timed(pl, b, ws)
    assert np.array_equal(to_host(a), to_host(b))
    P.prx_plan_destroy(pl)
    P.prx_sched_destroy(s)


def _plain_fp32(n, x, z, phi, psi, ends, fp32):
    """psi + tau sigma psi' rotation by rotation, the cosines at the ends of the
    chunks; in FP32 every result is rounded once.  Normalised at the end."""
    k, cosines = np.arange(1 << n), 1.0
    rnd = (lambda a: a.astype(np.complex64).astype(np.complex128)) if fp32 else (lambda a: a)
    for j, (xr, zr, p) in enumerate(zip(x.astype(int), z.astype(int), phi)):
        kp = k ^ xr
        par = kp & zr
        for sh in (8, 4, 2, 1):
            par ^= par >> sh
        tau = np.float32(np.tan(p)) if fp32 else np.tan(p)
        phase = 1j ** ((bin(xr & zr).count("1") + 1) & 3)
        psi = rnd(psi + float(tau) * phase * (1 - 2 * (par & 1)) * psi[kp])
        cosines *= np.cos(p)
        if j + 1 in ends:
            psi = rnd(psi * float(np.float32(cosines) if fp32 else cosines))
            cosines = 1.0
    return psi / np.linalg.norm(psi)


@pytest.mark.parametrize("n", [6, 8, 10])
def test_error_beside_plain_fp32(n):
    """A phase-estimation round of small angles, whose chunk factors are all near
    1 and recur in every step, over 30 seeds.  A plain FP32 evaluation rounds a
    coefficient per rotation and a factor per chunk; the in-place pairs round two
    coefficients and a factor per label: at most 3/4 more variance is allowed."""
    err = plain = 0.0
    for seed in range(30):
        x, z, h = synth.jw_hamiltonian(n, 24, 700 + seed)
        ham = P.prx_ham_create(n, x, z, h / np.sum(np.abs(h)))
        s = P.prx_sched_partial(ham, 10, 0.8, 8, 6, seed)
        _, x, z, phi = (np.array(v) for v in P.prx_sched_view(s))
        pl = P.prx_plan_create(s, n, P.PRX_C64, 0, len(x), P.PRX_FUSED)
        info = P.prx_plan_get_info(pl)
        last = P.prx_plan_pass(pl, info["passes"] - 1)
        chunks = [P.prx_plan_chunk(pl, c) for c in
                  range(last["chunk_begin"] + last["chunk_count"])]
        ends = {c["rot_begin"] + c["rot_count"] for c in chunks}
        assert info["kernel_rotations"] == len(x)
        ws = workspace(info["workspace_bytes"])
        P.prx_plan_upload(pl, ws)
        psi = to_dev(synth.gaussian_state(n, seed), P.PRX_C64)
        psi0 = to_host(psi)
        P.prx_plan_execute(pl, psi, ws)
        ref = _plain_fp32(n, x, z, phi, psi0, ends, False)
        err += np.linalg.norm(to_host(psi) - ref) ** 2
        plain += np.linalg.norm(_plain_fp32(n, x, z, phi, psi0, ends, True) - ref) ** 2
        P.prx_plan_destroy(pl)
        P.prx_sched_destroy(s)
        P.prx_ham_destroy(ham)
    print(f"[beside plain FP32 n={n}] variance {err / plain:.2f}", flush=True)
    assert err <= 1.75 * plain
