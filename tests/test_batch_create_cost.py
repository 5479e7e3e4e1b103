"""A batch plans every sample once: creating it takes no longer for samples
whose passes prx_batch_get_info counts in another frame than they run in."""
import time

import synth
from paper_2504_17881_amd import prx as P


def _create_seconds(n, scheds):
    t = time.perf_counter()
    b = P.prx_batch_create([n] * len(scheds), scheds, P.PRX_C64, [0] * len(scheds))
    t = time.perf_counter() - t
    P.prx_batch_destroy(b)
    return t


def test_samples_are_planned_once():
    S, M = 12, 1500
    scheds = {n: [P.prx_sched_from_rotations(n, *synth.random_pauli_rotations(n, M, seed=i))
                  for i in range(S)] for n in (11, 13)}
    best = {n: min(_create_seconds(n, s) for _ in range(5)) for n, s in scheds.items()}
    # (a narrow plan of the same list takes longer than the resident one)
    assert best[13] <= 1.5 * best[11], best
    for s in scheds[11] + scheds[13]:
        P.prx_sched_destroy(s)
