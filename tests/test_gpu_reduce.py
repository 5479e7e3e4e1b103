"""Reductions at the edges of their launch shapes (one block up to 13 qubits,
the last ragged grid, the full one), with cancellation, and from several
threads and streams at once."""
import math
import threading

import numpy as np
import pytest
import torch

from paper_2504_17881_amd import prx as P
from gpu_util import dev, tdtype, workspace

pytestmark = pytest.mark.gpu


def _states(n, dtype, seed):
    """Dyadic values with large terms that cancel exactly: exact FP64 sums."""
    rng = np.random.default_rng(seed)
    N = 1 << n
    a = (rng.integers(-512, 513, N) + 1j * rng.integers(-512, 513, N)) / 64.0
    b = (rng.integers(-512, 513, N) + 1j * rng.integers(-512, 513, N)) / 64.0
    if N >= 4:
        a[0] = a[1] = 2.0 ** 11
        b[0], b[1] = 2.0 ** 11 + 0j, -(2.0 ** 11) + 0j
    return a, b


@pytest.mark.parametrize("dtype", [P.PRX_C64, P.PRX_C128])
@pytest.mark.parametrize("n", [1, 2, 5, 12, 13, 14, 15, 20, 22, 23])
def test_exact_sums(n, dtype):
    """Every product and sum of these values is exact in FP64, so the results
    equal the integer arithmetic whatever the order."""
    a, b = _states(n, dtype, n)
    ia = (a * 64).real.astype(np.int64), (a * 64).imag.astype(np.int64)
    ib = (b * 64).real.astype(np.int64), (b * 64).imag.astype(np.int64)
    re = int(np.sum(ia[0] * ib[0] + ia[1] * ib[1]))
    im = int(np.sum(ia[0] * ib[1] - ia[1] * ib[0]))
    nn = int(np.sum(ia[0] ** 2 + ia[1] ** 2))
    ta = torch.from_numpy(a).to(dev(), tdtype(dtype))
    tb = torch.from_numpy(b).to(dev(), tdtype(dtype))
    ws = workspace(P.prx_reduce_workspace_bytes(n))
    print(f"[reduce n={n} dtype={dtype}]", flush=True)
    assert P.prx_overlap(ta, tb, n, dtype, ws) == complex(re / 4096.0, im / 4096.0)
    assert P.prx_norm2(ta, n, dtype, ws) == nn / 4096.0
    P.prx_renormalize(ta, n, dtype, ws)
    want = torch.from_numpy(a).to(dev(), tdtype(dtype))
    scale = 1.0 / math.sqrt(nn / 4096.0)
    want = torch.view_as_complex(torch.view_as_real(want) *
                                 (np.float32(scale).item() if dtype == P.PRX_C64 else scale))
    assert torch.equal(ta, want)


def test_threads_and_streams():
    """More threads than result slots, each on its own stream and workspace."""
    n = 14
    T = 70
    states = [torch.randn(1 << n, dtype=torch.complex128, device=dev()) for _ in range(T)]
    want = [float(torch.view_as_real(t).square().sum()) for t in states]
    ws = [workspace(P.prx_reduce_workspace_bytes(n)) for _ in range(T)]
    streams = [torch.cuda.Stream() for _ in range(8)]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        for _ in range(5):
            v = P.prx_norm2(states[i], n, P.PRX_C128, ws[i], stream=streams[i % 8])
            if abs(v - want[i]) > 1e-11 * want[i]:
                bad.append((i, v, want[i]))
    th = [threading.Thread(target=work, args=(i,)) for i in range(T)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad
