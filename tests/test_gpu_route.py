"""GPU: which calls the one-launch kernel takes.  It is meant for calls whose
time the prepared path's launches would dominate; shapes on which it measured
clearly slower than the prepared path (few rows against many keys, many rounds
of workgroups, one gradient of wide values, rows at odd 16-bit addresses) have
to take the prepared path, small and ordinary ones the one launch.
"""
import pytest

import parity
from paper_2609_04910_amd import gauss_sum as gs

pytestmark = pytest.mark.gpu


def _tensors(M, N, D, C, dtype, B=0, offset=0):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + D + C)
    lead = (B,) if B else ()

    def rand(*shape):
        n = 1
        for x in shape:
            n *= x
        flat = torch.empty(n + offset, dtype=dtype, device="cuda")
        flat[offset:] = torch.randn(n, generator=g, device="cuda").to(dtype)
        return flat[offset:].view(*shape)
    q, k = rand(*lead, M, D), rand(*lead, N, D)
    v = torch.randn(*lead, N, C, generator=g, device="cuda")
    return q, k, v, torch.randn(*lead, M, C, generator=g, device="cuda")


def _route(kind, M, N, D, C, bf16=False, B=0, offset=0):
    import torch
    dt, code = (torch.bfloat16, gs.GS_BF16) if bf16 else (torch.float16, gs.GS_F16)
    q, k, v, go = _tensors(M, N, D, C, dt, B, offset)
    n = max(B, 1)
    if kind == "sum":
        size = gs.gauss_sum_fwd_batched_workspace_size(M, N, D, C, n, code)
        fn = gs.gauss_sum_fwd_batched if B else gs.gauss_sum_fwd
        return parity.route(lambda ws: fn(q, k, v, 1.0, workspace=ws), size)
    if kind == "svgd":
        size = gs.gauss_sum_svgd_workspace_size(N, D, code)
        return parity.route(lambda ws: gs.gauss_sum_svgd(k, v, 1.0, workspace=ws), size)
    if kind == "flow":
        size = gs.gauss_sum_mmd_flow_workspace_size(N, D, code)
        return parity.route(lambda ws: gs.gauss_sum_mmd_flow(k, v, 1.0, want=(True, True, False), workspace=ws), size)
    if kind == "dq":
        size = gs.gauss_sum_bwd_workspace_size(M, N, D, C, code, want_dk=False, want_dv=False)
        return parity.route(lambda ws: gs.gauss_sum_bwd(q, k, v, 1.0, go, want=(True, False, False), workspace=ws),
                            size)
    size = gs.gauss_sum_fwd_bwd_batched_workspace_size(M, N, D, C, n, code)
    fn = gs.gauss_sum_fwd_bwd_batched if B else gs.gauss_sum_fwd_bwd
    return parity.route(lambda ws: fn(q, k, v, 1.0, go, workspace=ws), size)


# us per call, one launch against prepared
@pytest.mark.parametrize("kind,M,N,D,C", [
    ("sum", 16384, 1024, 50, 1),      # 28.3 / 21.0
    ("sum", 605, 9692, 50, 1),        # 34.1 / 25.5
    ("sum", 302, 4846, 100, 20),      # 42.4 / 27.4
    ("sum", 4293, 4293, 20, 50),      # 58.2 / 44.2
    ("sum", 2500, 2500, 65, 1),       # 68.5 / 24.2
    ("sum", 2500, 2500, 63, 1),       # 37.4 / 22.1
    ("dq", 750, 12000, 20, 1),        # 43.9 / 26.4
    ("dq", 3000, 3000, 20, 50),       # 1.19 times
    ("dq", 1500, 1500, 100, 50),      # 1.26 times
    ("both", 2842, 2842, 65, 10),     # above 2
    ("both", 5028, 1386, 65, 64),     # 255 / 112
    ("flow", 2842, 2842, 65, 1),      # 80.0 / 48.9
    ("svgd", 2010, 2010, 33, 33),     # 35.8 / 27.4
])
def test_prepared_where_one_launch_is_slower(kind, M, N, D, C):
    assert _route(kind, M, N, D, C) == "prepared"


@pytest.mark.parametrize("kind,M,N,D,C", [
    ("sum", 4096, 4096, 16, 1), ("sum", 1, 1, 1, 1), ("sum", 2048, 2048, 100, 20), ("sum", 2000, 2000, 45, 3),
    ("dq", 1, 1, 128, 60), ("dq", 4000, 4000, 50, 1), ("both", 3001, 5003, 50, 10), ("both", 2048, 2048, 100, 60),
    ("both", 1000, 1000, 65, 1), ("flow", 1000, 1000, 3, 1), ("flow", 4000, 4000, 45, 1), ("svgd", 1500, 1500, 45, 45),
    ("svgd", 3500, 3500, 20, 20),
])
@pytest.mark.parametrize("bf16", [False, True])
def test_one_launch_where_it_is_faster(kind, M, N, D, C, bf16):
    if bf16 and D > 64 and C > 32:
        pytest.skip("no such instance: it would spill (prepared path)")
    assert _route(kind, M, N, D, C, bf16) == "small"


def test_wide_shapes_and_batches():
    assert _route("sum", 64, 64, 129, 1) == "prepared"     # D > 128
    assert _route("sum", 64, 64, 16, 65) == "prepared"     # C > 64
    assert _route("sum", 400, 400, 20, 1, B=16) == "small"
    assert _route("sum", 200, 200, 20, 1, B=2000) == "prepared"
    assert _route("both", 64, 64, 100, 50, bf16=True) == "prepared"


def test_base_addresses_count_as_row_alignment():
    # even D, but every row two bytes off a 4-byte word
    assert _route("sum", 2500, 2500, 100, 20) == "prepared"
    assert _route("sum", 2000, 2000, 100, 1) == "small"
    assert _route("sum", 2000, 2000, 100, 1, offset=1) == "prepared"
