"""The calls whose speed is tracked, over the range in which the library is used.

A case names one call (``call``), its sizes, data types and the kind of point
cloud.  The clouds are those of the library's own workloads: ``normal``
(N(0, I), tau = 1 / D), ``scaled`` (N(0, I / D), tau = 1), ``unit`` (rows of
norm one, tau = 4), ``mixture`` (32 clusters of width 0.3 around N(0, 4 I)
centres) and ``two`` (half N(0, I), half N(0.5, I), weights +-1/N).

Calls:
  fwd            gauss_sum_fwd
  step           GaussSum under autograd: the sum, then the gradients of q, k, v
  fwd_bwd        gauss_sum_fwd_bwd: the sum and dq, dk, dv for a known dout
  flow           gauss_sum_mmd_flow: witness values, flow field and MMD^2
  svgd           gauss_sum_svgd: one SVGD direction
  fwd_batched    gauss_sum_fwd_batched over B clouds
  grad_batched   gauss_sum_fwd_bwd_batched over B clouds
"""
import math

import torch

from paper_2609_04910_amd import gauss_sum as gs

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _case(call, M, N, D, C=1, B=1, points="f16", values="f32", cloud="normal", tau=0.0, name=None):
    case = dict(call=call, B=B, M=M, N=N, D=D, C=C, points=points, values=values, cloud=cloud, tau=tau)
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # a particle flow in the plane or in space with a thousand particles,
        # thousands of steps: latency and launches
        _case("flow", 1000, 1000, 3, values="f16", cloud="two", tau=0.5, name="flow_small"),
        # SVGD with an ordinary number of particles on a posterior of odd
        # dimension, scores in single precision
        _case("svgd", 1500, 1500, 45, C=45, name="svgd_small"),
        # one small dense sum (kernel regression, witness function), the
        # library's dense_d16 workload
        _case("fwd", 4096, 4096, 16, name="fwd_d16"),
        # a training step through autograd on a minibatch, ragged sizes
        _case("step", 3001, 5003, 50, C=10, name="step_ragged"),
        # the MMD flow of 65536 particles in D = 64, the mmd_flow workload
        _case("flow", 65536, 65536, 64, values="f16", cloud="two", tau=7.413e-3, name="flow_d64"),
        # the svgd workload: wide values, sum and all three gradients
        _case("fwd_bwd", 16384, 16384, 128, C=128, values="f16", name="grad_c128"),
        # density-like sums on clustered bf16 points with a narrow kernel: most
        # kernel values vanish (the mixture_d32 workload at tau = 10)
        _case("fwd", 131072, 131072, 32, C=4, points="bf16", cloud="mixture", tau=10.0, name="fwd_mixture"),
        # sum and gradients on the same clusters at tau = 1 (a flow or SVGD on a
        # multimodal target)
        _case("fwd_bwd", 32768, 32768, 32, C=4, points="bf16", cloud="mixture", tau=1.0, name="grad_mixture"),
        # many clouds at once (the D sweep of the paper's benchmark)
        _case("fwd_batched", 16384, 16384, 32, B=64, cloud="scaled", name="batch_d32"),
        # forward and backward of four clouds (the N sweep of the paper's benchmark)
        _case("grad_batched", 32768, 32768, 32, B=4, cloud="scaled", name="batch_grad_d32"),
        # the same layout in single precision with several channels
        _case("fwd_batched", 16384, 16384, 32, C=32, B=4, points="f32", cloud="scaled", name="batch_c32_f32"),
        # the largest: wide points, rectangular, sum and all gradients (the
        # rect_d256 workload at a quarter of its queries and an eighth of its keys)
        _case("fwd_bwd", 32768, 262144, 256, C=16, values="f16", cloud="unit", name="rect_d256"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["fwd", "fwd", "fwd_bwd", "fwd_bwd", "step", "flow", "svgd", "fwd_batched", "grad_batched"])
    points = rng.choice(["f16", "f16", "bf16"])
    values = rng.choice(["f32", "f16"])
    cloud = rng.choice(["normal", "scaled", "unit", "mixture"])
    D, C, B = _log_int(rng, 3, 256), rng.choice([1, 1, _log_int(rng, 2, 128)]), 1
    M, N = _log_int(rng, 500, 65536), _log_int(rng, 500, 65536)
    if call == "flow":
        points, values, cloud, C = "f16", "f16", "two", 1
        M = N = _log_int(rng, 500, 65536)
        D = _log_int(rng, 3, 64)
    elif call == "svgd":
        cloud = "normal"
        M = N = _log_int(rng, 500, 16384)
        D = C = _log_int(rng, 3, 128)
    elif call == "step":
        M, N = _log_int(rng, 500, 16384), _log_int(rng, 500, 16384)
    elif call in ("fwd_batched", "grad_batched"):
        cloud = "scaled"
        B = rng.randint(2, 64 if call == "fwd_batched" else 8)
        M = N = _log_int(rng, 500, 16384)
        D, C = _log_int(rng, 3, 64), rng.choice([1, 1, _log_int(rng, 2, 32)])
    if call in ("fwd", "fwd_batched") and rng.random() < 0.3:
        # single precision: separate clouds of moderate width
        points, values = "f32", "f32"
        cloud = rng.choice(["normal", "scaled"])
        M, N = min(M, 32768), min(N, 32768)
    tau = {"two": 1.0 / (2.0 * D), "mixture": rng.choice([0.1, 1.0, 10.0])}.get(cloud, 0.0)
    return _case(call, M, N, D, C=C, B=B, points=points, values=values, cloud=cloud, tau=tau)


def _tau(case):
    if case["tau"]:
        return float(case["tau"])
    return {"normal": 1.0 / case["D"], "scaled": 1.0, "unit": 4.0}[case["cloud"]]


def _inputs(case, seed):
    """(q, k, v, dout) on the GPU; k is q where the call takes one point set."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    B, M, N, D, C = (case[n] for n in "BMNDC")
    pdt, vdt = DTYPES[case["points"]], DTYPES[case["values"]]

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=torch.float32)

    centres = 2.0 * normal(32, D) if case["cloud"] == "mixture" else None

    def cloud(n):
        shape = (B, n, D) if "batched" in case["call"] else (n, D)
        x = normal(*shape)
        if case["cloud"] == "scaled":
            x *= D ** -0.5
        elif case["cloud"] == "unit":
            x /= x.norm(dim=-1, keepdim=True)
        elif case["cloud"] == "mixture":
            label = torch.randint(0, 32, shape[:-1], generator=gen, device=dev)
            x = centres[label] + 0.3 * x
        elif case["cloud"] == "two":
            x[n // 2:] += 0.5
        return x.to(pdt)

    q = cloud(M)
    if case["call"] == "flow":
        v = torch.full((N, 1), 1.0 / N, device=dev)
        v[N // 2:] *= -1.0
        return q, q, v.to(vdt), None
    if case["call"] == "svgd":
        score = -q.to(torch.float32) + 0.1 * normal(N, C)
        return q, q, score.to(vdt), None
    k = cloud(N)
    lead = (B,) if "batched" in case["call"] else ()
    v = normal(*lead, N, C).to(vdt)
    dout = normal(*lead, M, C) if case["call"] in ("step", "fwd_bwd", "grad_batched") else None
    return q, k, v, dout


def prepare(case, seed):
    q, k, v, dout = _inputs(case, seed)
    if case["call"] == "step":
        q, k, v = (x.requires_grad_(True) for x in (q, k, v))
    return dict(call=case["call"], q=q, k=k, v=v, dout=dout, tau=_tau(case))


def run(state):
    call, q, k, v, dout, tau = (state[n] for n in ("call", "q", "k", "v", "dout", "tau"))
    if call == "fwd":
        return gs.gauss_sum_fwd(q, k, v, tau)
    if call == "step":
        s = gs.GaussSum.apply(q, k, v, tau)
        return (s.detach(),) + torch.autograd.grad(s, (q, k, v), dout)
    if call == "fwd_bwd":
        return gs.gauss_sum_fwd_bwd(q, k, v, tau, dout)
    if call == "flow":
        return gs.gauss_sum_mmd_flow(q, v, tau)
    if call == "svgd":
        return gs.gauss_sum_svgd(q, v, tau)
    if call == "fwd_batched":
        return gs.gauss_sum_fwd_batched(q, k, v, tau)
    return gs.gauss_sum_fwd_bwd_batched(q, k, v, tau, dout)


def work(case):
    """Points, values and upstream gradients read once, outputs written once.
    Per pair: 2 D flops for the score, 2 C for the sum; the gradients add 2 C
    for the weight <dout, v>, 2 D each for dq and dk and 2 C for dv.  (A flow
    or SVGD direction is a sum and a query gradient with unit weights.)"""
    B, M, N, D, C = (case[n] for n in "BMNDC")
    call = case["call"]
    size = {"f32": 4, "f16": 2, "bf16": 2}
    pts, val = size[case["points"]], size[case["values"]]
    one_set = call in ("flow", "svgd")
    read = B * ((M + (0 if one_set else N)) * D * pts + N * C * val)
    if call in ("fwd", "fwd_batched"):
        return {"bytes": read + B * M * C * 4, "flops": B * M * N * (2 * D + 2 * C)}
    if call == "flow":
        return {"bytes": read + 4 * N * (D + 1) + 8, "flops": M * N * (4 * D + 2)}
    if call == "svgd":
        return {"bytes": read + 4 * N * D, "flops": M * N * (4 * D + 2 * C)}
    out = pts * (M + N) * D + val * N * C if call == "step" else 4 * ((M + N) * D + N * C)
    return {"bytes": read + B * (M * C * 4 + M * C * 4 + out), "flops": B * M * N * (6 * D + 6 * C)}


def tolerance(case):
    # Kernel values and weights are rounded to fp16 (2^-12 each, of terms whose
    # signed sum is smaller than they are); single precision carries 2^-22 of
    # the scores.  About four times the largest error against 64 bits that
    # calls of each kind show.
    if case["points"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 2e-3}


def _exact_one(q, k, v, dout, tau, want_grad):
    """(s, dq, dk, dv) of one problem in 64 bits, over blocks of query rows."""
    q, k, v = q.double(), k.double(), v.double()
    g = None if dout is None else dout.double()
    M, N = q.shape[0], k.shape[0]
    kk = (k * k).sum(1)
    s = torch.empty(M, v.shape[1], dtype=torch.float64, device=q.device)
    dq = torch.empty_like(q) if want_grad else None
    dk = torch.zeros_like(k) if want_grad else None
    dv = torch.zeros_like(v) if want_grad else None
    vt, kt = v.t().contiguous(), k.t().contiguous()
    rows = max(1, (1 << 28) // max(1, N))
    for a in range(0, M, rows):
        x = q[a:a + rows]
        d2 = (x @ kt).mul_(-2.0).add_(kk).add_((x * x).sum(1, keepdim=True)).clamp_(min=0.0)
        phi = d2.mul_(-0.5 * tau).exp_()
        s[a:a + rows] = phi @ v
        if want_grad:
            y = g[a:a + rows]
            dv += phi.t() @ y
            p = phi.mul_(y @ vt)
            dq[a:a + rows] = tau * (p @ k - x * p.sum(1, keepdim=True))
            dk += tau * (p.t() @ x - k * p.sum(0).unsqueeze(1))
    return s, dq, dk, dv


def exact(case, seed):
    q, k, v, dout = _inputs(case, seed)
    call = case["call"]
    # the library takes tau as a 32-bit number
    tau = float(torch.tensor(_tau(case), dtype=torch.float32))
    if call == "fwd":
        return _exact_one(q, k, v, None, tau, False)[0]
    if call in ("step", "fwd_bwd"):
        return _exact_one(q, k, v, dout, tau, True)
    if call == "flow":
        ones = torch.ones(q.shape[0], 1, dtype=torch.float64, device=q.device)
        s, field, _, _ = _exact_one(q, k, v, ones, tau, True)
        return s, field, (v.double() * s).sum()
    if call == "svgd":
        ones = torch.ones(q.shape[0], 1, dtype=torch.float64, device=q.device)
        s = _exact_one(q, k, v, None, tau, False)[0]
        return s - _exact_one(q, k, ones, ones, tau, True)[1]
    each = [_exact_one(q[b], k[b], v[b], None if dout is None else dout[b], tau, dout is not None)
            for b in range(q.shape[0])]
    if call == "fwd_batched":
        return torch.stack([e[0] for e in each])
    return tuple(torch.stack([e[i] for e in each]) for i in range(4))
