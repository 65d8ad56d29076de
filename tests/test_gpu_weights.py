"""GPU: single-channel gradients and flows with unequal weights against the
fp64 oracle (pass rule of tests/parity.py).  A row whose near neighbours carry
small weights needs kernel values that keep their precision relative to the
largest Phi |v| of that row, not relative to the largest |v| of all keys.
"""
import numpy as np
import pytest

import oracle
import parity
from paper_2609_04910_amd import gauss_sum as gs
from paper_2609_04910_amd import workloads as wl

pytestmark = pytest.mark.gpu


def log_normal(w, sigma, seed=0):
    """Replaces the values of w by signed log-normal weights."""
    rng = np.random.default_rng(seed)
    w.v = (np.sign(w.v) * np.exp(sigma * rng.standard_normal((w.N, 1)))).astype(np.float32)
    return w


@pytest.mark.parametrize("sigma", [3.0, 4.0])
@pytest.mark.parametrize("M,N,D,qk", [(1000, 1000, 8, "f16"), (333, 1100, 40, "bf16"), (200, 700, 100, "f16")])
def test_small_log_normal_weights(M, N, D, qk, sigma):
    w = log_normal(parity.random_workload(D, M, N, D, 1, qk=qk, tau=32.0 / D), sigma)
    print(parity.check_workload(w), flush=True)


def check_clusters(w):
    """Pass rule of tests/parity.py with one more term for the gradients: they
    are differences of two fp32 sums, sum P k_d and q_d sum P, each of size up
    to max|k_d| sum |P| and rounded by 2^-24 of that a few times.  Where one
    term dominates a row and its k_d - q_d nearly vanishes, that exceeds the
    rounding of the terms."""
    tol = parity.TOL[w.qk_dtype]
    for fused in (False, True):
        got = parity.run(w, ("fwd", "dq", "dk", "dv"), fused=fused)
        for p in ("fwd", "dq", "dk", "dv"):
            ref, scale = parity.oracle_ref(w, p)
            if p in ("dq", "dk"):
                _, own = parity.oracle_ref(w, "fwd" if p == "dq" else "dv")  # sum_n Phi |v_n|, sum_m Phi |g_m|
                size = np.abs(w.g if p == "dq" else w.v).astype(np.float64) * own
                pts = np.abs(w.q_values.astype(np.float64)).max() + np.abs(w.k_values.astype(np.float64)).max()
                scale = scale + 2.0 ** -22 / tol * float(w.tau) * pts * size
            print(p, parity.compare("%s fused=%s" % (p, fused), got[p], ref, scale, tol), flush=True)


@pytest.mark.parametrize("sigma", [3.0, 4.0])
def test_small_clusters_log_normal_weights(sigma):
    w = wl.make("mixture_d32", seed=1, M=1500, N=1500, tau=10.0)
    w.C, w.v = 1, w.v[:, :1].copy()
    w.g = np.random.default_rng(1).standard_normal((1500, 1)).astype(np.float32)
    check_clusters(log_normal(w, sigma))


@pytest.mark.parametrize("sigma", [3.0, 4.0])
def test_small_flow_log_normal_weights(sigma):
    import torch
    w = log_normal(parity.random_workload(7, 1000, 1000, 8, 1, tau=4.0, same=True), sigma)
    s, _, mmd2 = gs.gauss_sum_mmd_flow(parity.to_torch(w.q), parity.to_torch(w.v), float(w.tau))
    torch.cuda.synchronize()
    ref, scale = oracle.fwd(w.q_values, w.q_values, w.v, float(w.tau), threads=parity.oracle_threads())
    print(parity.compare("flow s", s.cpu().numpy(), ref, scale, parity.TOL["f16"]))
    m, a = float((w.v * ref).sum()), float((np.abs(w.v) * scale).sum())
    assert abs(float(mmd2) - m) <= parity.TOL["f16"] * a


def test_small_values_of_every_magnitude():
    # weights across the whole range of fp32, subnormal ones and zeros among
    # them, growing and falling over the keys, with rows next to each kind
    rng = np.random.default_rng(11)
    w = parity.random_workload(11, 64, 1500, 12, 1, tau=1.0)
    e = np.linspace(-145.0, 120.0, 750)
    mag = np.exp2(np.concatenate([e, e[::-1]]))
    mag[::37] = 0.0
    w.v = (mag[:, None] * rng.choice([-1.0, 1.0], (1500, 1))).astype(np.float32)
    w.g = (w.g * 2.0 ** -20).astype(np.float32)
    print(parity.check_workload(w), flush=True)
