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


def cluster_weights(D, C, e, M=700, N=13000, tau=1.0, qk="f16", seed=3):
    """32 clusters whose keys weigh from 1 down to 2^-e; more keys than the
    one-launch kernel takes (12288 at most)."""
    rng = np.random.default_rng(seed)
    centres = 2.0 * rng.standard_normal((32, D))
    lk, lq = rng.integers(0, 32, N), rng.integers(0, 32, M)
    w = parity.random_workload(seed, M, N, D, C, qk=qk, tau=tau)
    w.k, w.k_values = wl._store_points((centres[lk] + 0.3 * rng.standard_normal((N, D))).astype(np.float32), qk)
    w.q, w.q_values = wl._store_points((centres[lq] + 0.3 * rng.standard_normal((M, D))).astype(np.float32), qk)
    w.v = (rng.standard_normal((N, C)) * np.exp2(-e * lk / 31.0)[:, None]).astype(np.float32)
    return w


@pytest.mark.parametrize("D,tau,e,qk", [(32, 1.0, 12, "f16"), (48, 0.7, 12, "f16"), (100, 0.3, 12, "bf16"),
                                        (200, 0.15, 12, "f16")])
def test_cluster_weights_one_channel(D, tau, e, qk):
    # waves whose 64 sampled keys miss a row's cluster, while 1024 would not
    print(parity.check_workload(cluster_weights(D, 1, e, tau=tau, qk=qk), ("dq", "dk", "dv")), flush=True)


def test_few_rows_beyond_the_bound_at_wide_weights():
    # cluster weights down to 2^-24: rows whose 64 sampled keys hold their
    # cluster have no offset, and beyond 2^-14 the products are subnormal, so
    # a few rows of such waves miss the bound; every other row keeps it
    w = cluster_weights(32, 1, 24, M=4096)
    got = parity.run(w, ("fwd", "dq"), fused=True)
    for p in ("fwd", "dq"):
        ref, scale = parity.oracle_ref(w, p)
        over = (np.abs(got[p] - ref) > parity.TOL["f16"] * scale).any(1)
        print(p, int(over.sum()), flush=True)
        assert over.mean() < 0.05


@pytest.mark.parametrize("D,C,tau,qk", [(32, 4, 1.0, "f16"), (32, 4, 1.0, "bf16"), (32, 32, 1.0, "f16"),
                                        (64, 20, 0.5, "f16"), (48, 60, 0.7, "f16"), (100, 40, 0.3, "bf16"),
                                        (100, 128, 0.3, "f16"), (40, 256, 0.8, "f16")])
def test_cluster_weights_several_channels(D, C, tau, qk):
    # values fall to 2^-12 of the largest: a row's products Phi <g, v> are then
    # small against the largest possible one whatever its Phi are
    print(parity.check_workload(cluster_weights(D, C, 12, M=500, tau=tau, qk=qk)), flush=True)


@pytest.mark.parametrize("C", [2, 32, 33, 64, 65, 128, 129, 256])
def test_largest_products(C):
    # every value and upstream gradient at the largest magnitude, kernel values
    # next to 1: the products are as large as the scales allow
    w = parity.random_workload(C, 600, 13000, 40, C, spread=1e-2)
    w.v = np.full((13000, C), 1.9990234375, np.float16)
    w.g = np.full((600, C), -3.998046875, np.float16)
    got = parity.run(w, ("dq", "dk"))
    for p in ("dq", "dk"):
        rows = np.arange(0, 600 if p == "dq" else 13000, 41)
        ref, scale = parity.oracle_ref(w, p, rows=rows)
        print(parity.compare("%s C=%d" % (p, C), got[p][rows], ref, scale, parity.TOL["f16"]), flush=True)
