"""prx_workspace_bytes of a schedule is enough for the plan of any part of it:
an application may be resumed from any rotation index, and the frames of a
part follow from the part's own rotations."""
import numpy as np
import pytest

import synth
from paper_2504_17881_amd import prx as P


def _sorted_terms(n, L, steps):
    x, z, h = synth.jw_hamiltonian(n, L, 3)
    o = np.tile(np.lexsort((z, x)), steps)
    return x[o], z[o], 0.3 * h[o]


def _random_then_one_mask(n, a, b):
    x, z, phi = synth.random_pauli_rotations(n, a + b, seed=n)
    x[a:] = (x[a:] & np.uint64(0x7f)) | np.uint64(1 << (n - 1))
    return x, z, phi / 4


def _check(n, dtype, rots, parts, kernel=P.PRX_FUSED):
    s = P.prx_sched_from_rotations(n, *rots)
    have = P.prx_workspace_bytes(n, dtype, s, kernel)
    for a, b in parts:
        pl = P.prx_plan_create(s, n, dtype, a, b, kernel)
        need = P.prx_plan_get_info(pl)["workspace_bytes"]
        P.prx_plan_destroy(pl)
        assert need <= have, (a, b, need, have)
    P.prx_sched_destroy(s)


@pytest.mark.parametrize("kernel", [P.PRX_PLAIN, P.PRX_FUSED, P.PRX_AUTO])
@pytest.mark.parametrize("n", [2, 4, 9, 12, 13, 14, 15, 19, 22, 24, 26, 28, 30])
@pytest.mark.parametrize("dtype", [P.PRX_C64, P.PRX_C128])
def test_prefixes_suffixes_and_inner_parts_fit(n, dtype, kernel):
    lists = [_random_then_one_mask(n, 60, 90),
             synth.random_pauli_rotations(n, 40, seed=n)]
    if n >= 4:
        lists.append(_sorted_terms(n, min(150, 2 * n * n), 2))
    for rots in lists:
        M = len(rots[0])
        rng = np.random.default_rng(n)
        inner = [sorted(int(v) for v in rng.integers(0, M + 1, 2)) for _ in range(20)]
        step = max(1, M // 20)
        cuts = list(range(0, M + 1, step))
        _check(n, dtype, rots, [(0, c) for c in cuts] + [(c, M) for c in cuts] + inner, kernel)


def test_equal_masks_longer_than_a_pass():
    """Spans of rank 1 leave the most norm partials."""
    n, M = 24, 400
    x = np.full(M, 1 << (n - 1), dtype=np.uint64)
    z = np.arange(M, dtype=np.uint64)
    _check(n, P.PRX_C64, (x, z, np.full(M, 0.1)), [(0, M), (7, 300)])


def test_masks_that_make_each_other_up():
    """A chunk of two rotations each: the most chunk records a list takes."""
    M = 3000
    x = np.array([16, 32, 48] * (M // 3), dtype=np.uint64)
    for n, dtype in ((10, P.PRX_C64), (14, P.PRX_C64), (24, P.PRX_C64), (12, P.PRX_C128),
                     (18, P.PRX_C128)):
        z = np.arange(M, dtype=np.uint64) % np.uint64(1 << n)
        _check(n, dtype, (x, z, np.full(M, 0.1)), [(0, M), (1, M), (2, M - 5)])


@pytest.mark.parametrize("n", [16, 20, 24, 28])
def test_tuned_shapes_fit(n):
    """The tile shapes that the autotuner times with a workspace of this size."""
    rots = _sorted_terms(n, 200, 1)
    s = P.prx_sched_from_rotations(n, *rots)
    have = P.prx_workspace_bytes(n, P.PRX_C64, s, P.PRX_FUSED)
    for B in (12, 13, 14):
        pl = P.prx_plan_create(s, n, P.PRX_C64, 0, 200, P.PRX_FUSED,
                               dict(tile_qubits=B, chunk_rank=4, max_virtual=B - 4, max_fuse=128,
                                    span_max=4))
        assert P.prx_plan_get_info(pl)["workspace_bytes"] <= have
        P.prx_plan_destroy(pl)
    P.prx_sched_destroy(s)
