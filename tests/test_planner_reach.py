"""The planner's furthest passes, found in one sweep over the rotations: the
number of passes against every segmentation into spans and frames, and a cost
that does not grow with the length of a pass."""
import time

import numpy as np
import pytest

import synth
from paper_2504_17881_amd import prx as P


def _rank(vs):
    rows = []
    for v in vs:
        for r in rows:
            v = min(v, v ^ r)
        if v:
            rows.append(v)
    return len(rows)


def _frame(xs, B, G):
    return any(_rank([x >> (B - g) for x in xs]) <= g for g in range(G + 1))


def _span(xs, m):
    basis = []
    for x in xs:
        if x == 0 or x in basis:
            continue
        if len(basis) == m or _rank(basis + [x]) == len(basis):
            return False
        basis.append(x)
    return len(xs) <= 64


def _reach(x, B, G, m, max_fuse):
    """End of the longest pass from every position (a prefix of a pass is one)."""
    M, end = len(x), []
    for q in range(M):
        e = q + 1
        while e < M and e - q < max_fuse and (_frame(x[q:e + 1], B, G) or _span(x[q:e + 1], m)):
            e += 1
        end.append(e)
    return end


@pytest.mark.parametrize("seed", range(4))
@pytest.mark.parametrize("dirs,max_fuse", [(3, 128), (9, 128), (9, 11)])
def test_fewest_passes(seed, dirs, max_fuse):
    n, M, B, G, m = 17, 90, 12, 3, 3
    rng = np.random.default_rng(seed)
    pool = [int(v) for v in rng.integers(1, 1 << n, dirs)]
    x = []
    for _ in range(M):
        a, b = rng.integers(0, dirs, 2)
        x.append(0 if rng.random() < 0.1 else pool[a] ^ (pool[b] if rng.random() < 0.3 else 0))
    end = _reach(x, B, G, m, max_fuse)
    # fewest jumps over the line: a pass may end anywhere in its reach
    fewest, far, stop = 0, 0, 0
    for p in range(M):
        far = max(far, end[p])
        if p == stop:
            fewest, stop = fewest + 1, far
    z = rng.integers(0, 1 << n, M)
    s = P.prx_sched_from_rotations(n, np.array(x, dtype=np.uint64), z.astype(np.uint64),
                                   np.full(M, 0.1))
    pl = P.prx_plan_create(s, n, P.PRX_C64, 0, M, P.PRX_FUSED,
                           dict(tile_qubits=B, chunk_rank=4, max_virtual=G, span_max=m,
                                max_fuse=max_fuse))
    assert P.prx_plan_get_info(pl)["passes"] == fewest
    P.prx_plan_destroy(pl)
    P.prx_sched_destroy(s)


def test_planning_cost_does_not_grow_with_the_pass():
    n, M = 20, 4000
    x, z, phi = synth.random_pauli_rotations(n, M, seed=1)
    x &= np.uint64(0x3f << (n - 6))
    s = P.prx_sched_from_rotations(n, x, z, phi / 8)

    def seconds(max_fuse):
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            P.prx_plan_destroy(P.prx_plan_create(s, n, P.PRX_C64, 0, M, P.PRX_FUSED,
                                                 dict(max_fuse=max_fuse)))
            best = min(best, time.perf_counter() - t)
        return best

    # (from every position anew: 30 times as long)
    assert seconds(2048) <= 4 * seconds(32)
    P.prx_sched_destroy(s)
