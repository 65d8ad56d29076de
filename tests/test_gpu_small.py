"""GPU: the one-launch kernel of small problems at the edges of its tiles and of
its dispatch, against the fp64 oracle (pass rule of tests/parity.py): single
rows and columns, ragged sizes that end inside a 16-byte load, every chunk
count of D and C, running offsets and scales that are raised late, batches.
"""
import numpy as np
import pytest

import parity
from paper_2609_04910_amd import gauss_sum as gs
from paper_2609_04910_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("qk", ["f16", "bf16"])
@pytest.mark.parametrize("M,N,D,C", [
    (1, 1, 1, 1), (17, 31, 1, 1), (16, 257, 3, 1), (33, 1000, 32, 1), (100, 129, 33, 1), (65, 513, 100, 1),
    (15, 33, 7, 2), (40, 600, 31, 16), (64, 512, 64, 32), (50, 300, 65, 17), (30, 270, 128, 31),
    (70, 290, 5, 33), (35, 261, 40, 64), (19, 100, 97, 50),
    (2048, 2048, 50, 1),        # at the limits of the dispatch
    (2049, 2100, 100, 1),
])
def test_small_matches_oracle(M, N, D, C, qk):
    w = parity.random_workload(M * 7 + N + D + C, M, N, D, C, qk=qk, vdt="f16" if N % 2 else "f32")
    rows = None if M * N * D < 1 << 26 else np.arange(0, M, 61)
    print(parity.check_workload(w, rows=rows, key_rows=rows), flush=True)


@pytest.mark.parametrize("C", [1, 3])
def test_offsets_and_scales_raised_late(C):
    # keys in order of decreasing distance and increasing value magnitude, so
    # that the running offset and the running scale move in many steps; kernel
    # values from 2^-60 up to about one
    w = parity.random_workload(3 + C, 48, 2000, 16, C, tau=1.0)
    r = np.linspace(3.0, 0.2, 2000)[:, None]
    u = w.k.astype(np.float32)
    k = (u / np.linalg.norm(u, axis=1, keepdims=True) * r * 3.0).astype(np.float16)
    q = (0.2 * w.q.astype(np.float32)).astype(np.float16)
    w.k = w.k_values = k
    w.q = w.q_values = q
    w.v = (w.v * np.exp2(np.linspace(-20, 6, 2000))[:, None]).astype(np.float32)
    print(parity.check_workload(w), flush=True)


@pytest.mark.parametrize("D,qk", [(1, "f16"), (10, "bf16"), (32, "f16"), (45, "f16"), (64, "bf16")])
def test_small_svgd(D, qk):
    import torch
    N = 333
    w = parity.random_workload(D, N, N, D, D, qk=qk, same=True)
    x, sc = parity.to_torch(w.q), parity.to_torch(w.v)
    got = gs.gauss_sum_svgd(x, sc, float(w.tau)).cpu().numpy()
    torch.cuda.synchronize()
    import oracle
    th = parity.oracle_threads()
    xv, one = w.q_values, np.ones((N, 1), np.float32)
    s, a = oracle.fwd(xv, xv, w.v, float(w.tau), threads=th)
    d, b = oracle.dq(xv, xv, one, one, float(w.tau), threads=th)
    parity.compare("svgd D=%d" % D, got, s - d, a + b, parity.TOL[qk])


def test_small_batch_equals_single_calls():
    # a batch whose problems together still count as small takes the same
    # kernel: bitwise the single calls
    import torch
    rng = np.random.default_rng(2)
    q, k = (torch.from_numpy(rng.standard_normal((3, 130, 20)).astype(np.float16)).cuda() for _ in range(2))
    v, g = (torch.from_numpy(rng.standard_normal((3, 130, 4)).astype(np.float32)).cuda() for _ in range(2))
    out = gs.gauss_sum_fwd_bwd_batched(q, k, v, 0.05, g)
    for b in range(3):
        one = gs.gauss_sum_fwd_bwd(q[b], k[b], v[b], 0.05, g[b])
        for x, y in zip(out, one):
            assert torch.equal(x[b], y)
