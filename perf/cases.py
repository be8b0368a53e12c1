"""The framework's work as a user's program asks for it, as cases that can be timed and checked.

Eight cases are the online path (one linear layer per call: a decode step of one to a few dozen rows, a short
ragged prompt, a long prefill batch; per-channel, integer per-group and real-valued per-group scales), four are the
offline stage that produces its weights (front-end and repack, adaptive smoothing, Hessian and compensation).
Layer sizes are those of this repository's benchmark and tests (4096 x 4096, 4096 x 11008, 5120 x 13824, 8192 x 28672,
11008 x 4096) or generic.  Value distributions: activations N(0,1) with 1 % of the channels scaled x20; int4 codes
as round-to-nearest gives them for normal weights; scales small and positive.
"""
import math

import torch

from paper_2406_09904_amd import binding as qqq

GROUP = 128


def _case(name, op, M, K, N, **more):
    return dict(name=name, op=op, M=M, K=K, N=N, **more)


def listed():
    return [
        # one token through the smallest attention projection: launches and latency are all there is
        _case("decode_pc_m1_k4096_n4096", "linear_pc", 1, 4096, 4096),
        # one token through a gate/up projection with group scales: an interactive session
        _case("decode_pg_m1_k4096_n11008", "linear_pg", 1, 4096, 11008, sg_max=15),
        # sixteen concurrent sessions on the largest layer: weight streaming
        _case("decode_pc_m16_k8192_n28672", "linear_pc", 16, 8192, 28672),
        # an odd number of sessions, group scales as the front-end emits them (up to 18, codes in [-7,7])
        _case("decode_pg_m37_k5120_n13824", "linear_pg", 37, 5120, 13824, sg_max=18),
        # a short prompt, or many sessions at once
        _case("prefill_pc_m200_k5120_n13824", "linear_pc", 200, 5120, 13824),
        # a prompt of ragged length with the paper's real-valued group scales
        _case("prefill_f16_m777_k4096_n11008", "linear_f16", 777, 4096, 11008),
        # a long prompt through a down projection with group scales
        _case("prefill_pg_m4096_k11008_n4096", "linear_pg", 4096, 11008, 4096, sg_max=15),
        # a long prompt through the largest layer
        _case("prefill_pc_m4096_k8192_n28672", "linear_pc", 4096, 8192, 28672),
        # round-to-nearest weights of a layer: group codes, scales and the device layout
        _case("weights_pg_k4096_n11008", "weights_pg", 0, 4096, 11008),
        # smoothing search of one layer on 512 calibration tokens, the default grid
        _case("smoothing_m512_k4096_n4096", "smoothing", 512, 4096, 4096, grid=20),
        # compensated weights of a square layer: Hessian of 2048 tokens, then the sweep
        _case("compensate_pc_m2048_k4096_n4096", "compensate_pc", 2048, 4096, 4096),
        # the same with group scales on a wider, shallower layer and a ragged token count
        _case("compensate_pg_m1111_k2048_n5632", "compensate_pg", 1111, 2048, 5632),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["linear_pc", "linear_pc", "linear_pg", "linear_pg", "linear_f16", "weights_pg", "smoothing",
                     "compensate_pc", "compensate_pg"])
    if op.startswith("linear"):
        K = 128 * _log_int(rng, 8, 86)            # 1024 .. 11008
        N = 16 * _log_int(rng, 64, 1792)          # 1024 .. 28672
        M = _log_int(rng, 1, 4096)
        while M * K * N > 4096 * 8192 * 28672:
            M = max(1, M // 2)
        more = dict(sg_max=rng.choice([15, 18])) if op == "linear_pg" else {}
    elif op == "weights_pg":
        K, N, M, more = 128 * _log_int(rng, 8, 86), 16 * _log_int(rng, 64, 1792), 0, {}
    elif op == "smoothing":
        K, N = 128 * _log_int(rng, 8, 32), 16 * _log_int(rng, 64, 256)
        M, more = _log_int(rng, 64, 512), dict(grid=rng.randint(8, 20))
    else:
        K, N = 128 * _log_int(rng, 8, 24), 16 * _log_int(rng, 64, 256)     # 1024 .. 3072 by 1024 .. 4096
        M, more = _log_int(rng, 300, 2048), {}
    return dict(op=op, M=M, K=K, N=N, **more)


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _activations(g, M, K):
    a = torch.randn((M, K), generator=g, device="cuda", dtype=torch.float32)
    ch = torch.randperm(K, generator=g, device="cuda")[:K // 100]
    a[:, ch] *= 20.0
    return a.to(torch.float16)


def _codes(g, N, K, sigma):
    """int4 codes in [-7,7] of normal weights, and the natural words that hold them."""
    c = torch.randn((N, K), generator=g, device="cuda", dtype=torch.float32).mul_(sigma).round_().clamp_(-7, 7)
    c = c.to(torch.int32)
    nat = torch.zeros((N, K // 8), dtype=torch.int32, device="cuda")
    for i in range(8):
        nat |= (c[:, i::8] & 15) << (4 * i)
    return c, nat


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device="cuda", dtype=torch.float32).mul_(hi - lo).add_(lo)


def _linear_inputs(case, seed):
    g = _gen(seed)
    M, K, N, op = case["M"], case["K"], case["N"], case["op"]
    a = _activations(g, M, K)
    codes, nat = _codes(g, N, K, 1.9 if op == "linear_pc" else 2.6)
    s_g = None
    if op == "linear_pc":
        s_w = _uniform(g, (N,), 0.005, 0.02).to(torch.float16)
    else:
        s_w = _uniform(g, (N,), 0.001, 0.005).to(torch.float16)
        if op == "linear_pg":
            s_g = torch.randint(1, case["sg_max"] + 1, (K // GROUP, N), generator=g, device="cuda").to(torch.int8)
        else:
            s_g = _uniform(g, (K // GROUP, N), 4.0, 15.5).to(torch.float16)
    return a, codes, nat, s_g, s_w


def _weights(g, N, K):
    """fp16 weights of a trained-looking layer: a sigma per output channel, a few heavy input channels."""
    sigma = torch.exp(_uniform(g, (N, 1), math.log(0.01), math.log(0.04)))
    w = torch.randn((N, K), generator=g, device="cuda", dtype=torch.float32) * sigma
    w[:, torch.randperm(K, generator=g, device="cuda")[:max(K // 1000, 1)]] *= 8.0
    return w.to(torch.float16)


def _offline_inputs(case, seed):
    g = _gen(seed)
    M, K, N, op = case["M"], case["K"], case["N"], case["op"]
    w = _weights(g, N, K)
    if op == "weights_pg":
        return None, w
    if op == "smoothing":
        return _activations(g, M, K), w
    # calibration activations are correlated across channels: a few common directions plus noise
    base = torch.randn((M, 64), generator=g, device="cuda", dtype=torch.float32)
    mix = torch.randn((64, K), generator=g, device="cuda", dtype=torch.float32)
    x = 0.15 * (base @ mix) + torch.randn((M, K), generator=g, device="cuda", dtype=torch.float32)
    return x.to(torch.float16), w


def prepare(case, seed):
    M, K, N, op = case["M"], case["K"], case["N"], case["op"]
    st = dict(case=case)
    if op.startswith("linear"):
        a, _, nat, s_g, s_w = _linear_inputs(case, seed)
        st.update(a=a, packed=qqq.qqq_pack_w4(nat, K), s_g=s_g, s_w=s_w)
        if op == "linear_f16":
            st["ws"] = qqq.new_workspace(M, N, K)
        else:
            st["ws"] = qqq.new_linear_workspace(M, N, K)
        if op == "linear_pg":
            st["sg"] = case["sg_max"] | (qqq.SG_SYMMETRIC_CODES if case["sg_max"] > 16 else 0)
    else:
        st["x"], st["w"] = _offline_inputs(case, seed)
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    op = st["case"]["op"]
    if op == "linear_pc":
        return qqq.qqq_linear_w4a8_perchannel(st["a"], st["packed"], st["s_w"], st["ws"])
    if op == "linear_pg":
        return qqq.qqq_linear_w4a8_pergroup(st["a"], st["packed"], st["s_g"], st["s_w"], st["ws"], sg_max=st["sg"])
    if op == "linear_f16":
        a_q, s_a = qqq.qqq_quant_act(st["a"])
        return qqq.qqq_gemm_w4a8_pergroup_f16scale(a_q, s_a, st["packed"], st["s_g"], st["s_w"], st["ws"])
    if op == "weights_pg":
        w_nat, s_star, s_int, s_wc, s_wg = qqq.qqq_quantize_w4_pergroup(st["w"])
        return [qqq.qqq_pack_w4(w_nat, st["case"]["K"]), s_star, s_int, s_wc, s_wg]
    if op == "smoothing":
        return qqq.qqq_adaptive_smoothing(st["x"], st["w"], st["case"]["grid"])
    H = qqq.qqq_hessian(st["x"])
    if op == "compensate_pc":
        return [H, *qqq.qqq_gptq_quantize_w4_perchannel(st["w"], H)]
    return [H, *qqq.qqq_gptq_quantize_w4_pergroup(st["w"], H)]


def work(case):
    M, K, N, op = case["M"], case["K"], case["N"], case["op"]
    G = K // GROUP
    if op.startswith("linear"):
        scales = {"linear_pc": 0, "linear_pg": G * N, "linear_f16": 2 * G * N}[op]
        return {"bytes": 2 * M * K + N * K // 2 + scales + 2 * N + 2 * M * N, "flops": 2 * M * N * K}
    if op == "weights_pg":
        return {"bytes": 2 * N * K + N * K // 2 + 5 * G * N + 2 * N, "flops": N * K}
    if op == "smoothing":
        # X W^T once and one product per grid point; both matrices in and out
        return {"bytes": 4 * M * K + 4 * N * K, "flops": 2 * M * N * K * (case["grid"] + 1)}
    # Hessian (one triangle), its factor, and every output channel's sweep over the channels still to come
    scales = 2 * N if op == "compensate_pc" else 5 * G * N + 2 * N
    return {"bytes": 2 * M * K + 8 * K * K + 2 * N * K + N * K // 2 + scales,
            "flops": M * K * K + K * K * K // 3 + N * K * K}


def tolerance(case):
    op = case["op"]
    if op.startswith("linear"):
        # integer sums are exact, the result is rounded once to fp16: 2.1e-4 over all binades; activations whose
        # code sits on a rounding tie move it far less than that
        return {"rel": 8e-4}
    if op == "weights_pg":
        return "exact"
    if op == "smoothing":
        # the losses: fp64 sums on a reference product accumulated in fp32 (3e-9 to 7e-9 from 64 bits; another order of
        # its sums as far again); all else is rounded where the interface says and so equal
        return {"rel": 3e-8}
    # H: fp64 sums of fp16 products, here even exact (0 from 64 bits).  Codes: decided by fp64 running weights; a quotient on a rounding tie may go either
    # way, and then the rest of that output channel follows (one row of N): four such rows
    return {"rel": 1e-14, "differ": 4.0 / case["N"]}


# ---------------------------------------------------------------- the same numbers in 64 bits

def _quantised_rows(a):
    """Per-token int8 codes (the interface states the fp32 steps) and scales, as float64."""
    a32 = a.to(torch.float32)
    s = a32.abs().amax(dim=1, keepdim=True) / torch.tensor(127.0, device=a.device)
    safe = torch.where(s == 0, torch.ones_like(s), s)
    q = torch.round(a32 / safe).clamp_(-127, 127)
    return q.to(torch.float64), s.to(torch.float64)


def _weight_quotient(w64, s64):
    """clamp(rne(fp32(w / s)), -7, 7); a zero scale gives 0."""
    safe = torch.where(s64 == 0, torch.ones_like(s64), s64)
    q = torch.round((w64 / safe).to(torch.float32)).clamp_(-7, 7).to(torch.float64)
    return torch.where(s64 == 0, torch.zeros_like(q), q)


def _block_scale(amax32):
    return (amax32 / torch.tensor(7.0, device=amax32.device)).to(torch.float16)


def _words(codes64):
    c = codes64.to(torch.int32)
    nat = torch.zeros((c.shape[0], c.shape[1] // 8), dtype=torch.int32, device=c.device)
    for i in range(8):
        nat |= (c[:, i::8] & 15) << (4 * i)
    return nat


def _group_tables(codes64, s_wg):
    """s*_Wg, its integer form and s_Wc from codes [N,K] and group scales [G,N]."""
    N, K = codes64.shape
    sg = s_wg.to(torch.float32)
    cmax = codes64.abs().reshape(N, K // GROUP, GROUP).amax(dim=2).to(torch.float32)
    s_wc = ((cmax * sg.t()).amax(dim=1) / torch.tensor(127.0, device=sg.device)).to(torch.float16)
    wc = s_wc.to(torch.float32)
    safe = torch.where(wc == 0, torch.ones_like(wc), wc)
    star = (sg / safe).to(torch.float16).clamp(max=18.203125)
    star = torch.where(wc == 0, torch.zeros_like(star), star)
    s_int = torch.round(star.to(torch.float32)).clamp(1, 18).to(torch.int8)
    return star, s_int, s_wc


def _exact_linear(case, seed):
    a, codes, _, s_g, s_w = _linear_inputs(case, seed)
    q, s_a = _quantised_rows(a)
    w = codes.to(torch.float64)
    if s_g is not None:
        w = torch.round(w * s_g.to(torch.float64).t().repeat_interleave(GROUP, dim=1))
        if case["op"] == "linear_pg":
            w.clamp_(-128, 127)
    return (q @ w.t()) * s_a * s_w.to(torch.float64)


def _exact_weights(case, seed):
    _, w = _offline_inputs(case, seed)
    N, K = w.shape
    blocks = w.to(torch.float32).reshape(N, K // GROUP, GROUP)
    s_wg = _block_scale(blocks.abs().amax(dim=2)).t().contiguous()
    codes = _weight_quotient(w.to(torch.float64), s_wg.to(torch.float64).t().repeat_interleave(GROUP, dim=1))
    star, s_int, s_wc = _group_tables(codes, s_wg)
    return [None, star, s_int, s_wc, s_wg]   # the device layout is the library's own


def _exact_smoothing(case, seed):
    x, w = _offline_inputs(case, seed)
    G = case["grid"]
    x32, w32 = x.to(torch.float32), w.to(torch.float32)
    amax = x32.abs().amax(dim=0)
    sigmas = (amax.max().to(torch.float64) * torch.arange(1, G + 1, device=x.device, dtype=torch.float64) / G).to(torch.float32)
    ref = x.to(torch.float64) @ w.to(torch.float64).t()

    def smoothed(sigma):
        s = torch.where(amax > sigma, amax / sigma, torch.ones_like(amax))
        return s, (x32 / s).to(torch.float16), (w32 * s).to(torch.float16)

    losses = torch.empty(G, dtype=torch.float64, device=x.device)
    for i in range(G):
        _, xs, ws = smoothed(sigmas[i])
        q, s_a = _quantised_rows(xs)
        s_w = _block_scale(ws.to(torch.float32).abs().amax(dim=1)).to(torch.float64)[:, None]
        codes = _weight_quotient(ws.to(torch.float64), s_w)
        losses[i] = ((q @ codes.t()) * s_a * s_w.t() - ref).square().sum()
    best = torch.argmin(losses)
    s, xs, ws = smoothed(sigmas[best])
    return {"xs": xs, "ws": ws, "s": s, "sigmas": sigmas, "losses": losses, "best": best.to(torch.int32).reshape(1)}


def _exact_compensation(case, seed):
    x, w = _offline_inputs(case, seed)
    N, K = w.shape
    x64 = x.to(torch.float64)
    H = 2.0 * (x64.t() @ x64)
    A = H + 0.01 * H.diagonal().mean() * torch.eye(K, dtype=torch.float64, device=x.device)
    # H^-1 = U^T U: row i of U over its diagonal is row i of the inverse for the channels still free
    U = torch.linalg.cholesky(torch.cholesky_inverse(torch.linalg.cholesky(A)), upper=True)
    U = U / U.diagonal()[:, None]
    W = w.to(torch.float64)
    codes = torch.zeros_like(W)
    grouped = case["op"] == "compensate_pg"
    if not grouped:
        s_w = _block_scale(w.to(torch.float32).abs().amax(dim=1))
        s = s_w.to(torch.float64)
    tables = []
    for b in range(0, K, GROUP):
        if grouped:
            tables.append(_block_scale(W[:, b:b + GROUP].abs().amax(dim=1).to(torch.float32)))
            s = tables[-1].to(torch.float64)
        err = torch.empty((N, GROUP), dtype=torch.float64, device=x.device)
        block = W[:, b:b + GROUP].clone()
        for i in range(GROUP):
            q = _weight_quotient(block[:, i], s)
            codes[:, b + i] = q
            err[:, i] = block[:, i] - q * s
            block[:, i:] -= err[:, i, None] * U[b + i, b + i:b + GROUP]
        W[:, b + GROUP:] -= err @ U[b:b + GROUP, b + GROUP:]
    if not grouped:
        return [H, _words(codes), s_w]
    s_wg = torch.stack(tables)
    star, s_int, s_wc = _group_tables(codes, s_wg)
    return [H, _words(codes), s_wg, star, s_int, s_wc]


def exact(case, seed):
    op = case["op"]
    if op.startswith("linear"):
        return _exact_linear(case, seed)
    if op == "weights_pg":
        return _exact_weights(case, seed)
    if op == "smoothing":
        return _exact_smoothing(case, seed)
    return _exact_compensation(case, seed)
