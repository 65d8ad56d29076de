"""GPU: the several-channel fp32 forward's running offsets against the fp64
oracle.  Keys come in order of decreasing distance, so that a row's largest
exponent grows from about -60 to 0 over the key steps and the offset is raised
many times.  The pass rule is the fp32 tier's, 1e-5 of sum_n Phi |v| per
element for exponents of order one, plus what the expanded square adds here:
its three fp32 numbers (score with the key's half norm, the product with tau',
the query's half norm) are of the size of tau (|q|^2 + |k|^2), up to 168 for
the queries next to the farthest keys, and each is rounded by 2^-24 of it, so
3 * 2^-24 * 168 = 3e-5 of each term.
"""
import numpy as np
import pytest

import oracle
import parity
from paper_2609_04910_amd import gauss_sum as gs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,C,N", [(3, 2, 2049), (16, 40, 1500), (40, 17, 3000), (100, 3, 1000), (200, 70, 700)])
def test_offsets_raised_many_times(D, C, N):
    import torch
    rng = np.random.default_rng(D + C)
    u = rng.standard_normal((N, D))
    k = (u / np.linalg.norm(u, axis=1, keepdims=True) * np.linspace(9.0, 0.1, N)[:, None]).astype(np.float32)
    q = (0.05 * rng.standard_normal((100, D))).astype(np.float32)
    q[::10] = k[:10] * 1.02          # rows next to the farthest keys
    v = rng.standard_normal((N, C)).astype(np.float32)
    out = gs.gauss_sum_fwd(*(torch.from_numpy(x).cuda() for x in (q, k, v)), 1.0).cpu().numpy()
    ref, scale = oracle.fwd(q, k, v, 1.0, threads=parity.oracle_threads())
    size = (q.astype(np.float64) ** 2).sum(1).max() + (k.astype(np.float64) ** 2).sum(1).max()
    tol = 1e-5 + 3 * 2.0 ** -24 * size
    print(parity.compare("f32 D=%d C=%d" % (D, C), out, ref, scale, tol), flush=True)
