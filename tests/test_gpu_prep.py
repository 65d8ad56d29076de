"""GPU: the one-launch preparation at the edges of its dispatch, against the
fp64 oracle: arrays just within and just beyond what every workgroup reduces
itself (16384 elements), odd row lengths (no 16-byte row loads), and enough
items that a thread takes several.  The pass rule is that of tests/parity.py.
(Of test_preparation_edges the last three shapes go to the one-launch kernel, and
with gradients the first two take their maxima in a launch of their own; the
cases after it assert their route.)
"""
import numpy as np
import pytest

import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,D,C,qk", [
    (70, 16384, 3, 1, "f16"),    # maxima taken inline
    (70, 16385, 3, 1, "f16"),    # maxima in a launch of their own, a few partials
    (1, 1, 1, 1, "f16"),
    (513, 512, 33, 17, "bf16"),  # bf16: the points' maxima too
    (300, 4097, 24, 5, "bf16"),
])
def test_preparation_edges(M, N, D, C, qk):
    w = parity.random_workload(M + N, M, N, D, C, qk=qk, vdt="f16" if C > 1 else "f32")
    print(parity.check_workload(w), flush=True)


def test_several_items_per_thread():
    w = parity.random_workload(5, 40, 200003, 136, 3)
    rows = np.array([0, 1, 77777, 131071, 131072, 200002])
    print(parity.check_workload(w, key_rows=rows), flush=True)


def elements(w, grads):
    """Elements of the arrays whose maxima a call's preparation takes (bf16: the
    points of a gradient too)."""
    n = w.N * w.C
    if grads:
        n += w.M * w.C
        if w.qk_dtype == "bf16":
            n += w.M * w.D + w.N * w.D
    return n


# shapes that the one-launch kernel never takes (C > 64, or D > 128), the
# gradient call's arrays just within and just beyond 16384 elements
@pytest.mark.parametrize("M,N,D,C,qk,inline", [
    (100, 152, 20, 65, "f16", True),       # 16380
    (100, 153, 20, 65, "f16", False),      # 16445
    (60, 132, 20, 65, "bf16", True),       # 16320: values, dout and both point sets
    (60, 133, 20, 65, "bf16", False),      # 16405
    (90, 31, 130, 5, "bf16", True),        # 16335, D > 128
    (90, 32, 130, 5, "bf16", False),       # 16470
    (7000, 9384, 130, 1, "f16", True),     # 16384, single channel
    (7000, 9385, 130, 1, "f16", False),
])
def test_maxima_inline_or_in_a_launch_with_gradients(M, N, D, C, qk, inline):
    w = parity.random_workload(M + N, M, N, D, C, qk=qk, vdt="f16" if C > 1 else "f32")
    assert (elements(w, True) <= 16384) == inline
    rows = np.arange(0, M, max(1, M // 60))
    print(parity.check_workload(w, rows=rows, key_rows=np.arange(0, N, max(1, N // 60)), path="prepared"), flush=True)


def test_maxima_of_a_batch_beyond_the_workgroups_that_repeat_them():
    # 40 small problems: few elements each, but more than 1024 workgroups in the
    # launch, so the maxima get a launch of their own; the largest magnitudes
    # differ by problem
    import oracle
    from paper_2609_04910_amd import gauss_sum as gs
    rng = np.random.default_rng(4)
    B, M, N, D, C = 40, 60, 70, 140, 3
    q, k = (rng.standard_normal((B, n, D)).astype(np.float16) for n in (M, N))
    v = (rng.standard_normal((B, N, C)) * np.exp2(np.arange(B) - 20.0)[:, None, None]).astype(np.float32)
    g = (rng.standard_normal((B, M, C)) * np.exp2(10.0 - np.arange(B))[:, None, None]).astype(np.float32)
    out, size = [], gs.gauss_sum_fwd_bwd_batched_workspace_size(M, N, D, C, B)
    t = [parity.to_torch(a) for a in (q, k, v, g)]
    assert parity.route(lambda ws: out.extend(gs.gauss_sum_fwd_bwd_batched(*t[:3], 1.0 / D, t[3], workspace=ws)),
                        size) == "prepared"
    tau = float(np.float32(1.0 / D))
    for b in range(0, B, 3):
        for got, fn in zip(out, ("fwd", "dq", "dk", "dv")):
            args = (q[b], k[b], v[b]) + (() if fn == "fwd" else (g[b],))
            ref, scale = getattr(oracle, fn)(*args, tau, threads=parity.oracle_threads())
            parity.compare("%s[%d]" % (fn, b), got[b].cpu().numpy(), ref, scale, parity.TOL["f16"])
