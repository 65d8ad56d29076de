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
    (2048, 2048, 50, 1),        # many workgroups (the dispatch's limits: below)
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


def _bf16(x):
    return wl._store_points(x.astype(np.float32), "bf16")


@pytest.mark.parametrize("C", [1, 3, 40])
@pytest.mark.parametrize("what", ["v", "v_most", "dout", "keys", "queries"])
def test_blocks_of_tiny_numbers(what, C):
    # scales come from single key steps and from 16 rows: steps and rows of
    # subnormal (or, for bf16 points, nearly subnormal) numbers with zeros among
    # them, beside ordinary ones
    w = parity.random_workload(5, 300, 1000, 8, C, qk="bf16" if what in ("keys", "queries") else "f16", tau=0.3)
    if what in ("v", "v_most"):
        w.v[:64 if what == "v" else 700] *= np.float32(1e-39)
        w.v[5:9] = 0.0
    elif what == "dout":
        w.g[16:48] *= np.float32(1e-39)
        w.g[20] = 0.0
    elif what == "keys":
        kv = w.k_values.copy()
        kv[:300] *= np.float32(1e-36)
        w.k, w.k_values = _bf16(kv)
    else:
        qv = w.q_values.copy()
        qv[:100] *= np.float32(1e-38)
        w.q, w.q_values = _bf16(qv)
    print(parity.check_workload(w), flush=True)


@pytest.mark.parametrize("N", [1000, 13000])
@pytest.mark.parametrize("C", [1, 3, 70])
def test_subnormal_arrays(C, N):
    # nothing but subnormal values, through the small and the prepared path:
    # sums stay finite and, with upstream gradients of 2^100, the gradients are
    # ordinary numbers (twice the usual bound: the values' own 2^-20, the copies'
    # fp16 numbers near 2^-3 and fp32 sums near 2^-126 round a little more)
    w = parity.random_workload(6, 200, N, 8, C, tau=0.3)
    w.v = (np.sign(w.v) * (1.0 + np.abs(w.v)) * 1e-39).astype(np.float32)
    w.g = np.sign(w.g) * np.float32(2.0 ** 100)
    for fused in (False, True):
        got = parity.run(w, ("fwd", "dq", "dk", "dv"), fused=fused)
        assert np.all(np.isfinite(got["fwd"]))
        for p in ("dq", "dk", "dv"):
            ref, scale = parity.oracle_ref(w, p)
            print(parity.compare("%s fused=%s" % (p, fused), got[p], ref, scale, 4e-3), flush=True)


@pytest.mark.parametrize("qk", ["f16", "bf16"])
@pytest.mark.parametrize("C", [1, 3, 40])
@pytest.mark.parametrize("size", [2e8, 8e9, 1e12])
def test_far_from_the_origin_stays_finite(size, C, qk):
    # tau |x|^2 far beyond the stated domain: exponents round by whole units and
    # more, so results mean nothing, but no fp16 number may overflow
    w = parity.random_workload(3, 200, 1000, 8, C, tau=size / 4e4)
    q, k = w.q_values.astype(np.float32), w.k_values.astype(np.float32)
    q[:, 0] += 200.0
    k[:, 0] += 200.0
    w.q, w.q_values = wl._store_points(q, qk)
    w.k, w.k_values = wl._store_points(k, qk)
    got = parity.run(w, ("fwd", "dq", "dk", "dv"), fused=True)
    for p in ("fwd", "dq", "dk", "dv"):
        assert np.all(np.isfinite(got[p])), p
    import torch
    phi = gs.gauss_sum_svgd(parity.to_torch(w.k), parity.to_torch(np.repeat(w.v[:, :1], 8, 1)), float(w.tau))
    assert torch.isfinite(phi).all()


# The dispatch's limits: the longest chains of key steps that the kernel takes
# and one step more, for sixteen and for eight waves, and the most rounds of
# workgroups; both sides against the oracle.
@pytest.mark.parametrize("M,N,D,C,want,path", [
    (2048, 8192, 20, 1, "fwd", "small"),        # 256 steps: 16 a wave
    (2048, 8193, 20, 1, "fwd", "prepared"),     # 17
    (2100, 6656, 50, 1, "fwd", "small"),        # 13 of sixteen waves
    (2100, 6657, 50, 1, "fwd", "prepared"),
    (2100, 4864, 20, 20, "fwd", "small"),       # 152 steps: 19 of eight waves
    (2100, 4865, 20, 20, "fwd", "prepared"),
    (4096, 4096, 20, 1, "fwd", "small"),        # one round of 256 workgroups
    (4112, 4096, 20, 1, "fwd", "prepared"),     # a second one
    (2048, 2048, 100, 20, "fwd", "small"),      # 8192 tiles
    (2048, 2049, 100, 20, "fwd", "prepared"),
    (4096, 4096, 20, 1, "dq", "small"),
    (4097, 4096, 20, 1, "dq", "prepared"),
    (4000, 4096, 50, 1, "dq", "small"),
])
def test_limits_of_the_dispatch(M, N, D, C, want, path):
    w = parity.random_workload(M + N, M, N, D, C)
    rows, routes = np.arange(0, M, 29), []
    got = parity.run(w, (want,), routes=routes)
    assert routes == [path]
    ref, scale = parity.oracle_ref(w, want, rows=rows)
    print(parity.compare(want, got[want][rows], ref, scale, parity.TOL["f16"]), flush=True)
