"""GPU: gradients of clustered points against the fp64 oracle (pass rule of
tests/parity.py): waves whose coarse key sample misses a row's own cluster,
with the whole sample reaching it (tau = 1: unshifted kernel values) or not
(tau = 10: exact row maxima), and rows far from every key.
"""
import numpy as np
import pytest

import parity
from paper_2609_04910_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau", wl.MIXTURE_TAUS)
def test_mixture_gradients(tau):
    w = wl.make("mixture_d32", seed=4, M=4700, N=4501, tau=tau)
    rows, keys = np.arange(0, 4700, 23), np.arange(0, 4501, 23)
    print(parity.check_workload(w, ("fwd", "dq", "dk", "dv"), rows=rows, key_rows=keys), flush=True)


@pytest.mark.parametrize("D,C,qk", [(40, 1, "f16"), (100, 5, "f16"), (150, 5, "f16"), (60, 20, "bf16")])
def test_two_far_clusters_and_outliers(D, C, qk):
    # a tight cluster of one key in 200 (missed by 64 sampled keys), which the
    # queries of every wave include, and a few outlying queries
    w = parity.random_workload(D, 4200, 4100, D, C, qk=qk, tau=2.0 / D)
    far = np.zeros(D, np.float32)
    far[0] = 6.0 * np.sqrt(D) / 2

    def move(x, sel):
        y = x.astype(np.float32) if qk == "f16" else (x.astype(np.uint32) << 16).view(np.float32)
        y = y.copy()
        y[sel] = 0.5 * y[sel] + far
        return wl._store_points(y, qk)
    w.q, w.q_values = move(w.q, np.arange(0, 4200, 64))
    w.k, w.k_values = move(w.k, np.arange(7, 4100, 200))
    rows, keys = np.arange(0, 4200, 32), np.arange(7, 4100, 50)
    print(parity.check_workload(w, rows=rows, key_rows=keys), flush=True)
