"""GPU: the prepared path (k_prep, k_row_check, k_fwd, k_dq, combines) at D <= 128
and C <= 64, where calls of a few hundred or thousand points go to the one-launch
kernel: the cases of the other GPU tests that name a kernel or a range mode of
the prepared path, with more keys than that kernel ever takes (12288).  Every
case asserts its route.  Reference: the fp64 oracle on sampled rows (pass rule
of tests/parity.py).
"""
import numpy as np
import pytest

import oracle
import parity
from paper_2609_04910_amd import gauss_sum as gs
from paper_2609_04910_amd import workloads as wl

pytestmark = pytest.mark.gpu

MANY = 12500  # keys


def check(w, passes=("fwd", "dq", "dk", "dv"), rows=None, key_rows=None, **kw):
    key_rows = np.arange(0, w.N, 97) if key_rows is None else key_rows
    print(parity.check_workload(w, passes, rows=rows, key_rows=key_rows, path="prepared", **kw), flush=True)


# every instance of k_fwd and k_dq at D <= 128: (D, C) per chunk count of D and
# per class of C (single channel, one to sixteen, 17 - 32, 33 - 64 channels)
@pytest.mark.parametrize("qk", ["f16", "bf16"])
@pytest.mark.parametrize("D,C", [(1, 1), (32, 1), (17, 2), (31, 16), (20, 17), (32, 32), (9, 33), (32, 64),
                                 (33, 1), (64, 1), (50, 5), (64, 16), (40, 30), (64, 33), (45, 64),
                                 (65, 1), (128, 1), (100, 9), (128, 16), (90, 32), (128, 50), (70, 64)])
def test_instances(D, C, qk):
    M = 260 + D  # ragged query tiles
    w = parity.random_workload(D * 7 + C, M, MANY + D, D, C, qk=qk, vdt="f16" if C % 2 else "f32")
    check(w, rows=np.arange(0, M, 5))


@pytest.mark.parametrize("D,C", [(16, 3), (16, 1), (48, 20), (100, 1), (100, 9)])
def test_range_levels_plain_shifted_exact(D, C):
    # query blocks at growing distance from a key cloud: largest kernel values
    # of a row about 2^-4 (plain), 2^-14 and 2^-19 (shifted by 2^15) and 2^-30
    # (running or exact row maxima)
    rng = np.random.default_rng(5 + D)
    B, tau = 128, np.float32(1.0)
    k32 = (0.3 * rng.standard_normal((MANY, D))).astype(np.float32)
    targets = (-4.0, -14.0, -19.0, -30.0)
    c = float(tau) * np.log2(np.e) / 2.0
    blocks = []
    for L in targets:
        u = rng.standard_normal((B, D))
        u /= np.linalg.norm(u, axis=1, keepdims=True)
        lo, hi = np.zeros(B), np.full(B, 40.0)  # radius with nearest-key log2 Phi of L, by bisection
        for _ in range(30):
            r = 0.5 * (lo + hi)
            x = u * r[:, None]
            d2 = (x ** 2).sum(1)[:, None] + (k32 ** 2).sum(1)[None] - 2.0 * x @ k32.T.astype(np.float64)
            near = -c * d2.min(1) > L
            lo, hi = np.where(near, r, lo), np.where(near, hi, r)
        blocks.append((u * lo[:, None]).astype(np.float32))
    q = np.concatenate(blocks).astype(np.float16)
    k = k32.astype(np.float16)
    q64, k64 = q.astype(np.float64), k.astype(np.float64)
    L = -c * ((q64 ** 2).sum(1)[:, None] + (k64 ** 2).sum(1)[None] - 2.0 * q64 @ k64.T).min(1)
    if D <= 64:  # (a cloud in many dimensions has rows that no key is near to)
        assert np.all(L[:B] > -8)
    assert np.all(L[B:3 * B] < -8) and np.all(L[B:3 * B] > -23) and np.all(L[3 * B:] < -23)
    v = rng.standard_normal((MANY, C)).astype(np.float32)
    g = rng.standard_normal((4 * B, C)).astype(np.float32)
    w = wl.Workload("range_levels", 4 * B, MANY, D, C, tau, "f16", q, k, v, g, ("fwd", "dq", "dk", "dv"), False, q, k)
    check(w, rows=np.arange(0, 4 * B, 5))


@pytest.mark.parametrize("D,C", [(32, 4), (32, 1), (20, 20), (64, 4), (128, 4), (128, 40)])
def test_online_offsets_rescale(D, C):
    # keys in order of decreasing distance: the largest kernel value of a row
    # grows from about 2^-400 to 2^-30 over its key steps, so that the forward's
    # running offsets are raised many times
    rng = np.random.default_rng(17 + D)
    M, tau = 300, np.float32(1.0)
    c = float(tau) * np.log2(np.e) / 2.0
    centre = rng.standard_normal(D)
    q = (centre + 0.05 * rng.standard_normal((M, D))).astype(np.float16)
    u = rng.standard_normal((MANY, D))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    k = (centre + u * np.sqrt(np.linspace(400.0, 30.0, MANY) / c)[:, None]).astype(np.float16)
    q64, k64 = q.astype(np.float64), k.astype(np.float64)
    L = -c * ((q64 ** 2).sum(1)[:, None] + (k64 ** 2).sum(1)[None] - 2.0 * q64 @ k64.T)
    assert np.all(L.max(axis=1) < -23) and np.all(L[:, :500].max(axis=1) < L.max(axis=1) - 60)
    v = rng.standard_normal((MANY, C)).astype(np.float32)
    w = wl.Workload("online_rescale", M, MANY, D, C, tau, "f16", q, k, v, None, ("fwd",), False, q, k)
    check(w, ("fwd",), rows=np.arange(0, M, 3))


@pytest.mark.parametrize("qk,D,C", [("f16", 48, 8), ("bf16", 30, 1), ("f16", 100, 33)])
def test_deterministic_and_unaligned_rows(qk, D, C):
    # two calls agree bit for bit, and so does one with points, values and
    # gradients at odd element offsets (other loads, same numbers)
    import torch
    w = parity.random_workload(6 + D, 300, MANY, D, C, qk=qk)
    q, k, v, g = parity.gpu_inputs(w, alias=False)

    def off(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)
    res = []
    for a in ((q, k, v, g), (q, k, v, g), tuple(off(t) for t in (q, k, v, g))):
        out = []
        size = gs.gauss_sum_fwd_bwd_workspace_size(300, MANY, D, C, gs._dtype_code(q.dtype))
        assert parity.route(lambda ws: out.extend(gs.gauss_sum_fwd_bwd(*a[:3], float(w.tau), a[3], workspace=ws)),
                            size) == "prepared"
        res.append(out)
    for other in res[1:]:
        for x, y in zip(res[0], other):
            assert torch.equal(x, y)


@pytest.mark.parametrize("D,C,qk,off", [(16, 3, "f16", 64.0), (64, 1, "f16", 16.0), (64, 5, "f16", 48.0),
                                        (32, 4, "bf16", 24.0), (128, 16, "f16", 24.0)])
def test_translated_clouds(D, C, qk, off):
    w = parity.random_workload(11, 300, MANY, D, C, qk=qk)
    w.q, w.q_values = wl._store_points(w.q_values.astype(np.float32) + np.float32(off), qk)
    w.k, w.k_values = wl._store_points(w.k_values.astype(np.float32) + np.float32(off), qk)
    check(w, rows=np.arange(0, 300, 3))


@pytest.mark.parametrize("tiny", [1e-5, 1e-7])
def test_bf16_points_with_a_tiny_coordinate(tiny):
    w = parity.random_workload(11, 300, MANY, 16, 4, qk="bf16")
    for name in ("q", "k"):
        x = getattr(w, name + "_values").astype(np.float32).copy()
        x[:, -1] *= np.float32(tiny)
        bits, vals = wl._store_points(x, "bf16")
        setattr(w, name, bits)
        setattr(w, name + "_values", vals)
    check(w, rows=np.arange(0, 300, 3))


def test_rows_of_one_dominating_key():
    # kernel values near 1e-15 and steep: a row's terms other than its largest
    # vanish.  The gradients are differences of two fp32 sums, so where that
    # key's coordinate nearly equals the row's, 2^-20 of the dominating term is
    # allowed beside the usual bound.
    w = parity.random_workload(21, 150, MANY, 8, 4, spread=3.0, tau=3.0)
    routes = []
    got = parity.run(w, ("fwd", "dq"), fused=True, routes=routes)
    assert routes == ["prepared"]
    tol = parity.TOL["f16"]
    ref, scale = parity.oracle_ref(w, "fwd")
    print(parity.compare("fwd", got["fwd"], ref, scale, tol))
    ref, scale = parity.oracle_ref(w, "dq")
    size = np.abs(w.q_values.astype(np.float64)).max() * scale.max(axis=1, keepdims=True)
    print(parity.compare("dq", got["dq"], ref, scale + 2.0 ** -20 / tol * size, tol))


@pytest.mark.parametrize("N,D,qk,vdt", [(4500, 17, "f16", "f32"), (4600, 32, "bf16", "f32"), (4500, 64, "f16", "f16"),
                                        (4500, 128, "f16", "f32")])
def test_mmd_flow(N, D, qk, vdt):
    rng = np.random.default_rng(N + D)
    x = rng.standard_normal((N, D)).astype(np.float32)
    x[N // 2:] += 0.5
    v = (np.where(np.arange(N) < N // 2, 1.0, -1.0) / N * np.exp(rng.standard_normal(N)))[:, None]
    v = (v * 64).astype(np.float16) if vdt == "f16" else v.astype(np.float32)
    xs, xv = wl._store_points(x, qk)
    tau, out = 1.0 / D, []
    xt, vt = parity.to_torch(xs), parity.to_torch(v)
    size = gs.gauss_sum_mmd_flow_workspace_size(N, D, gs._dtype_code(xt.dtype), gs._dtype_code(vt.dtype))
    assert parity.route(lambda ws: out.extend(gs.gauss_sum_mmd_flow(xt, vt, tau, want=(True, True, False),
                                                                    workspace=ws)), size) == "prepared"
    _, _, mmd2 = gs.gauss_sum_mmd_flow(xt, vt, tau)
    rows, th = np.arange(0, N, 23), parity.oracle_threads()
    t32 = float(np.float32(tau))
    ref, scale = oracle.fwd(xv, xv, v, t32, rows=rows, threads=th)
    s = out[0].cpu().numpy()
    parity.compare("flow s", s[rows], ref, scale, parity.TOL[qk])
    ref, scale = oracle.dq(xv, xv, v, np.ones((N, 1), np.float32), t32, rows=rows, threads=th)
    parity.compare("flow field", out[1].cpu().numpy()[rows], ref, scale, parity.TOL[qk])
    total = float((v.astype(np.float64) * s.astype(np.float64)).sum())
    assert abs(float(mmd2) - total) <= 1e-12 * float(np.abs(v.astype(np.float64) * s).sum())


@pytest.mark.parametrize("N,D,qk,sdt", [(3700, 17, "f16", "f32"), (3700, 32, "bf16", "f32"), (3000, 50, "bf16", "f16"),
                                        (3000, 64, "f16", "f32")])
def test_svgd(N, D, qk, sdt):
    w = parity.random_workload(N + D, N, N, D, D, qk=qk, vdt=sdt, same=True)
    x, score, out = parity.to_torch(w.q), parity.to_torch(w.v), []
    size = gs.gauss_sum_svgd_workspace_size(N, D, gs._dtype_code(x.dtype), gs._dtype_code(score.dtype))
    assert parity.route(lambda ws: out.append(gs.gauss_sum_svgd(x, score, float(w.tau), workspace=ws)),
                        size) == "prepared"
    rows, th, one = np.arange(0, N, 23), parity.oracle_threads(), np.ones((N, 1), np.float32)
    s, a = oracle.fwd(w.q_values, w.q_values, w.v, float(w.tau), rows=rows, threads=th)
    d, b = oracle.dq(w.q_values, w.q_values, one, one, float(w.tau), rows=rows, threads=th)
    parity.compare("svgd", out[0].cpu().numpy()[rows], s - d, a + b, parity.TOL[qk])


@pytest.mark.parametrize("B,M,D,C", [(3, 200, 32, 1), (2, 130, 20, 3), (3, 97, 24, 40), (3, 200, 64, 1), (2, 150, 50, 3),
                                     (2, 100, 40, 50), (3, 120, 100, 1), (2, 100, 128, 5), (2, 90, 80, 40)])
def test_batches(B, M, D, C):
    # the instances for several problems per launch: all problems in one group,
    # two, and one (bitwise the single calls)
    import torch
    rng = np.random.default_rng(D + C)
    q = (rng.standard_normal((B, M, D)) / np.sqrt(D)).astype(np.float16)
    k = (rng.standard_normal((B, MANY, D)) / np.sqrt(D)).astype(np.float16)
    v = rng.standard_normal((B, MANY, C)).astype(np.float32)
    g = rng.standard_normal((B, M, C)).astype(np.float32)
    tq, tk, tv, tg = (parity.to_torch(a) for a in (q, k, v, g))
    rows, keys, th = np.arange(0, M, 7), np.arange(0, MANY, 411), parity.oracle_threads()
    refs = [(oracle.fwd(q[b], k[b], v[b], 1.0, rows=rows, threads=th),
             oracle.dq(q[b], k[b], v[b], g[b], 1.0, rows=rows, threads=th),
             oracle.dk(q[b], k[b], v[b], g[b], 1.0, rows=keys, threads=th),
             oracle.dv(q[b], k[b], v[b], g[b], 1.0, rows=keys, threads=th)) for b in range(B)]
    for group in range(1, B + 1):
        out, size = [], gs.gauss_sum_fwd_bwd_batched_workspace_size(M, MANY, D, C, group)
        assert parity.route(lambda ws: out.extend(gs.gauss_sum_fwd_bwd_batched(tq, tk, tv, 1.0, tg, workspace=ws)),
                            size) == "prepared"
        sums = gs.gauss_sum_fwd_batched(tq, tk, tv, 1.0, group=group)
        for b in range(B):
            for name, got, (ref, scale), r in zip(("fwd", "dq", "dk", "dv"), out, refs[b], (rows, rows, keys, keys)):
                parity.compare("%s[%d] group %d" % (name, b, group), got[b].cpu().numpy()[r], ref, scale,
                               parity.TOL["f16"])
            parity.compare("sum[%d]" % b, sums[b].cpu().numpy()[rows], *refs[b][0], parity.TOL["f16"])
            if group == 1:
                for got, one in zip(out, gs.gauss_sum_fwd_bwd(tq[b], tk[b], tv[b], 1.0, tg[b])):
                    assert torch.equal(got[b], one)
                assert torch.equal(sums[b], gs.gauss_sum_fwd(tq[b], tk[b], tv[b], 1.0))


@pytest.mark.parametrize("M,D,C", [(300, 16, 1), (300, 64, 1), (200, 40, 12), (200, 100, 40)])
def test_graph_replays_match_eager(M, D, C):
    # replays of a captured sum and gradients, with eager calls of the library
    # on other inputs between them, equal the eager results bit for bit
    import torch
    w, w2 = (parity.random_workload(s, M, MANY, D, C) for s in (1, 2))
    q, k, v, g = parity.gpu_inputs(w, alias=False)
    other = parity.gpu_inputs(w2, alias=False)
    tau = float(w.tau)
    size = gs.gauss_sum_fwd_bwd_workspace_size(M, MANY, D, C)
    ws = torch.full((size,), parity.SENTINEL, dtype=torch.uint8, device="cuda")
    out = torch.empty((M, C), dtype=torch.float32, device="cuda")

    def call():
        return gs.gauss_sum_fwd_bwd(q, k, v, tau, g, out=out, workspace=ws)
    eager = [t.clone() for t in call()]
    torch.cuda.synchronize()
    assert not bool((ws == parity.SENTINEL).all())  # the prepared path
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = call()
    for rep in range(3):
        for t in captured:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in zip(captured, eager):
            assert torch.equal(got, ref), rep
        gs.gauss_sum_fwd_bwd(*other[:3], tau, other[3])
        torch.cuda.synchronize()
