"""GPU: the one-launch preparation at the edges of its dispatch, against the
fp64 oracle: arrays just within and just beyond what every workgroup reduces
itself (16384 elements), odd row lengths (no 16-byte row loads), and enough
items that a thread takes several.  The pass rule is that of tests/parity.py.
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
