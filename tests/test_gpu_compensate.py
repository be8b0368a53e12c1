"""The compensation sweep at the edges of its blocks (64 channels a factorisation block, 128 a sweep block, 512 a sweep, 16 output
channels a workgroup, 64 x 64 update tiles) against the CPU oracle, which forms and eliminates the inverse Hessian.

Bar: scales bit for bit and codes identical; both sides decide a code by a quotient good to far better than 1e-9, so
one may differ only at a rounding tie (then the rest of that output channel follows): none on these seeds.
"""
import numpy as np
import pytest
import torch

from oracle import qqq_calib_oracle as cal
from oracle import qqq_oracle as orc
from paper_2406_09904_amd import binding as qqq
from paper_2406_09904_amd import synth
from tests.util import f16_bits, to_dev

pytestmark = pytest.mark.gpu


def layer(M, K, N, seed):
    g = synth.rng(seed)
    r = min(16, K)
    x = (g.standard_normal((M, r)) @ g.standard_normal((r, K)) * 0.5 + 0.5 * g.standard_normal((M, K))).astype(np.float16)
    x[:, K // 3] = 0                                     # a channel that never fires
    return x.view(np.uint16), synth.weights_fp16(N, K, seed + 1).view(np.uint16)


def dev16(bits):
    return to_dev(np.ascontiguousarray(bits).view(np.uint16), torch)


@pytest.mark.parametrize("K,N", [(8, 1), (64, 31), (72, 33), (128, 32), (200, 65), (328, 130), (576, 70), (1160, 40)])
def test_per_channel_sweep_at_block_edges(K, N):
    x, w = layer(2 * K + 10, K, N, 400 + K + N)
    H = cal.hessian(x)
    codes, s_bits, _ = cal.gptq_quantize(w, H, 0.01)
    w_nat, s_w = qqq.qqq_gptq_quantize_w4_perchannel(dev16(w), torch.from_numpy(H).cuda(), 0.01)
    torch.cuda.synchronize()
    assert np.array_equal(f16_bits(s_w), s_bits)
    assert np.array_equal(orc.w8_perchannel(w_nat.cpu().numpy().view(np.uint32), K), codes)


@pytest.mark.parametrize("M,K,shift", [(1, 1, 0), (3, 31, 0), (65, 72, 0), (64, 72, 4), (33, 2056, 0), (31, 2051, 0)])
def test_hessian_tiles(M, K, shift):
    """32- and 64-wide tiles, whole and element-wise rows (odd K, or a base that is not 16-byte aligned), ragged edges.
    Every product of two fp16 is exact in fp64 and these sums stay below 53 bits: equal bit for bit, both halves."""
    x = synth.activations_fp16(M, K, 600 + M + K, "normal", 0.02, 10.0)
    buf = torch.zeros(M * K + 8, dtype=torch.float16, device="cuda")
    d_x = buf[shift:shift + M * K].view(M, K)
    d_x.copy_(torch.from_numpy(x))
    H = qqq.qqq_hessian(d_x).cpu().numpy()
    assert np.array_equal(H, cal.hessian(x.view(np.uint16)))


@pytest.mark.parametrize("K,N", [(128, 1), (256, 33), (640, 97), (1152, 20)])
def test_per_group_sweep_at_block_edges(K, N):
    x, w = layer(2 * K + 10, K, N, 500 + K + N)
    H = cal.hessian(x)
    codes, s_wg, _ = cal.gptq_quantize_pergroup(w, H, 128, 0.01)
    star, s_int, s_wc = cal.pergroup_scales_from_codes(codes, s_wg, 128)
    got = qqq.qqq_gptq_quantize_w4_pergroup(dev16(w), torch.from_numpy(H).cuda(), 0.01)
    torch.cuda.synchronize()
    w_nat, g_wg, g_star, g_int, g_wc = got
    assert np.array_equal(orc.w8_perchannel(w_nat.cpu().numpy().view(np.uint32), K), codes)
    assert np.array_equal(f16_bits(g_wg), s_wg) and np.array_equal(f16_bits(g_star), star)
    assert np.array_equal(f16_bits(g_wc), s_wc) and np.array_equal(g_int.cpu().numpy(), s_int)


def test_factorisation_larger_than_its_launches_carry():
    """K = 6528: the first blocks of the factorisation owe the columns before them more update tiles than the launches of
    the next blocks take along.  Against a 64-bit torch sweep by the explicit inverse; the bar as above."""
    K, N = 6528, 24
    g = torch.Generator(device="cuda").manual_seed(77)
    x = torch.randn((1500, 48), generator=g, device="cuda") @ torch.randn((48, K), generator=g, device="cuda") * 0.2
    x = (x + torch.randn(x.shape, generator=g, device="cuda")).to(torch.float16).to(torch.float64)
    H = 2.0 * (x.t().contiguous() @ x)
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.03).to(torch.float16)
    w_nat, s_w = qqq.qqq_gptq_quantize_w4_perchannel(w, H, 0.01)
    damped = H + 0.01 * H.diagonal().mean() * torch.eye(K, dtype=torch.float64, device="cuda")
    U = torch.linalg.cholesky(torch.cholesky_inverse(torch.linalg.cholesky(damped)), upper=True)
    U = U / U.diagonal()[:, None]
    run, s = w.to(torch.float64), s_w.to(torch.float64)
    codes = torch.zeros_like(run)
    for i in range(K):
        codes[:, i] = torch.round((run[:, i] / s).to(torch.float32)).clamp_(-7, 7)
        run[:, i + 1:] -= (run[:, i] - codes[:, i] * s)[:, None] * U[i, i + 1:]
    got = orc.w8_perchannel(w_nat.cpu().numpy().view(np.uint32), K)
    assert np.array_equal(got, codes.cpu().numpy().astype(got.dtype))


# ---- weights and Hessians that hold infinities or NaN: the output channel's codes are 0 from the first quotient that is no
# ---- number on, its later group scales 0, a NaN does not count for a group's maximum; other output channels are as without
INF, NAN = 0x7C00, 0x7E00


def codes_of(w_nat, K):
    return orc.w8_perchannel(w_nat.cpu().numpy().view(np.uint32), K)


@pytest.mark.parametrize("K,N,at", [(72, 20, 40), (200, 40, 70), (1160, 33, 700)])
def test_per_channel_weights_that_are_no_numbers(K, N, at):
    x, w = layer(2 * K + 10, K, N, 900 + K)
    H = cal.hessian(x)
    codes, s_bits, _ = cal.gptq_quantize(w, H, 0.01)
    for row, k, bits in ((3, at, INF), (5, at + 1, NAN), (7, 0, INF | 0x8000), (9, K - 1, INF)):
        w[row, k] = bits                 # an infinite or NaN scale: every quotient of the row is NaN
        codes[row] = 0
    w_nat, s_w = qqq.qqq_gptq_quantize_w4_perchannel(dev16(w), torch.from_numpy(H).cuda(), 0.01)
    assert np.array_equal(codes_of(w_nat, K), codes)
    good = [n for n in range(N) if n not in (3, 5, 7, 9)]
    assert np.array_equal(f16_bits(s_w)[good], s_bits[good])
    assert not np.isfinite(f16_bits(s_w)[[3, 5, 7, 9]].view(np.float16)).any()


def test_per_group_weights_that_are_no_numbers():
    K, N = 640, 20
    x, w = layer(2 * K + 10, K, N, 950)
    places = ((2, 200, INF), (4, 300, NAN), (6, 10, NAN), (8, 130, INF | 0x8000), (11, 639, NAN))
    for row, k, _ in places:
        w[row, k] = 0
    H = cal.hessian(x)
    codes, s_wg, _ = cal.gptq_quantize_pergroup(w, H, 128, 0.01)
    for row, k, bits in places:
        w[row, k] = bits
        g = k // 128
        s_wg[g + 1:, row] = 0
        if bits == NAN:                  # the channels before it keep their codes
            codes[row, k:] = 0
        else:                            # the group's scale is infinite
            codes[row, 128 * g:] = 0
            s_wg[g, row] = INF
    got = qqq.qqq_gptq_quantize_w4_pergroup(dev16(w), torch.from_numpy(H).cuda(), 0.01)
    assert np.array_equal(codes_of(got[0], K), codes)
    assert np.array_equal(f16_bits(got[1]), s_wg)


@pytest.mark.parametrize("percdamp", [0.01, 0.0])
@pytest.mark.parametrize("K,at,value", [(72, 0, np.inf), (384, 60, np.inf), (384, 383, np.nan), (640, 300, np.nan)])
def test_hessian_of_activations_that_are_no_numbers(K, at, value, percdamp):
    """Only the first channel, which nothing moves, has a code; the first group's scale is that of the weights."""
    N = 20
    x, w = layer(2 * K + 10, K, N, 970 + K)
    x = x.copy()
    x[5, at] = np.array([value], np.float16).view(np.uint16)[0]
    with np.errstate(invalid="ignore"):
        H = torch.from_numpy(cal.hessian(x)).cuda()
    s_bits = cal.channel_scales(w)
    codes = np.zeros((N, K), np.int8)
    codes[:, 0] = cal.rtn_codes(w[:, 0].view(np.float16), s_bits.view(np.float16))
    w_nat, s_w = qqq.qqq_gptq_quantize_w4_perchannel(dev16(w), H, percdamp)
    assert np.array_equal(codes_of(w_nat, K), codes) and np.array_equal(f16_bits(s_w), s_bits)
    if K % 128 == 0:
        s_wg = np.zeros((K // 128, N), np.uint16)
        s_wg[0] = cal.channel_scales(np.ascontiguousarray(w[:, :128]))
        codes[:, 0] = cal.rtn_codes(w[:, 0].view(np.float16), s_wg[0].view(np.float16))
        got = qqq.qqq_gptq_quantize_w4_pergroup(dev16(w), H, percdamp)
        assert np.array_equal(codes_of(got[0], K), codes) and np.array_equal(f16_bits(got[1]), s_wg)


@pytest.mark.parametrize("M,K,edge", [(128, 968, None), (193, 1032, 127.4375), (130, 1160, 127.5), (150, 1032, np.inf), (129, 968, np.nan),
                                      (257, 1160, None), (200, 1288, 32640.0), (194, 1032, np.inf), (321, 1160, np.nan)])
def test_hessian_from_digits(M, K, edge):
    """The int8 products: sums of whole numbers, so every element is the exact sum rounded once.  Values over fp16's whole range
    below 127.5, subnormal ones among them.  Where one value of one channel is larger, its tiles are compared with fp64 products: from 32640 on
    they are made of those.  (Shapes of up to two stages of tokens, and few of K = 968, are computed in fp64 throughout.)"""
    rng = np.random.default_rng(M + K)
    x = (rng.standard_normal((M, K)) * np.exp2(rng.integers(-22, 5, K))).astype(np.float16)
    x[rng.integers(0, M, 50), rng.integers(0, K, 50)] = np.float16(2.0 ** -24)
    at = K - 3
    if edge is not None:
        x[M - 1 if M % 2 else 0, at] = edge   # seen by the last stage or by the first
        x[0, 5] = -edge if np.isfinite(edge) and edge < 127.5 else x[0, 5]
    H = qqq.qqq_hessian(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(H.view(np.int64), H.T.copy().view(np.int64))
    x64 = x.astype(np.float64)
    exact = np.ones((K, K), bool)
    if edge is not None and not edge < 127.5:
        lo = at // 64 * 64   # the 64 x 64 tiles with the channel in their rows or columns
        exact[lo:lo + 64, :] = exact[:, lo:lo + 64] = False
        with np.errstate(invalid="ignore"):
            want = 2.0 * (x64.T @ x64)
        got, ref = H[~exact], want[~exact]
        assert np.array_equal(np.isfinite(got), np.isfinite(ref))
        ok = np.isfinite(ref)
        scale = np.sqrt(np.outer(np.diag(want), np.diag(want)))[~exact][ok]
        assert (np.abs(got[ok] - ref[ok]) <= 2.0 ** -52 * M * scale).all()   # M fp64 roundings of partial sums below that product
        x64[:, at] = 0.0
    m = (x64 * 2.0 ** 24).astype(np.int64)
    hi, lo = m >> 12, m & 0xFFF
    s = (hi.T @ hi).astype(object) * 2 ** 24 + (hi.T @ lo + lo.T @ hi).astype(object) * 2 ** 12 + (lo.T @ lo).astype(object)
    want = s.astype(np.float64) * 2.0 ** -47   # int -> float rounds once, half to even
    assert np.array_equal(H[exact], want[exact])


def exact_hessian(x):
    """2 X^T X of finite fp16 values in whole numbers (multiples of 2^-48), rounded to fp64 once."""
    m = (x.astype(np.float64) * 2.0 ** 24).astype(np.int64)
    hi, lo = m >> 20, m & 0xFFFFF
    s = (hi.T @ hi).astype(object) * 2 ** 40 + (hi.T @ lo + lo.T @ hi).astype(object) * 2 ** 20 + (lo.T @ lo).astype(object)
    return s.astype(np.float64) * 2.0 ** -47


@pytest.mark.parametrize("M,K,kind", [(449, 1032, "everywhere"), (256, 1160, "channels"), (450, 1032, "last token"),
                                      (193, 1288, "one value"), (129, 2056, "bits"), (257, 1032, "bits"), (383, 1032, "middle")])
def test_hessian_from_five_digits(M, K, kind):
    """Values from 127.5 up to the last one below 32640: the sums go on with a fifth digit from where they stand, and stay exact."""
    rng = np.random.default_rng(M + K)
    x = (rng.standard_normal((M, K)) * np.exp2(rng.integers(-22, 5, K))).astype(np.float16)
    if kind == "everywhere":
        x = np.clip(x.astype(np.float32) * 2000, -32624, 32624).astype(np.float16)
    elif kind == "channels":
        x[:, 7], x[:, K // 2], x[:, K - 1] = 32624, -32624, x[:, K - 1] * np.float16(64) + np.float16(200)
    elif kind == "last token":
        x[M - 1, :] = rng.choice([-127.5, 127.5, 128, 999, -32624], K)
    elif kind == "one value":
        x[70, 100] = -127.5
    elif kind == "middle":
        x[130:200, :64] = -500.25
    else:   # every finite magnitude below 32640 alike, subnormal ones among them
        bits = rng.integers(0, 0x77F8, (M, K)).astype(np.uint16) | (rng.integers(0, 2, (M, K)) << 15).astype(np.uint16)
        x = bits.view(np.float16)
    H = qqq.qqq_hessian(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(H, exact_hessian(x))


@pytest.mark.parametrize("M", [16384, 16385])
@pytest.mark.parametrize("values", [[127.4375, -127.4375, 127.0, -2.0 ** -24], [32624.0, -32624.0, 127.5, 2.0 ** -24, -32512.0]])
def test_hessian_at_the_token_limit(M, values):
    """Channels that are constant at the ends of four and five digits, at the last token count of the int8 products' 32-bit sums and one past
    it (fp64 products).  Every partial sum has at most 22 + 15 bits, so both are exact."""
    K = 1032
    c = np.resize(np.array(values), K)
    x = torch.from_numpy(c.astype(np.float16)).cuda().repeat(M, 1)
    H = qqq.qqq_hessian(x).cpu().numpy()
    assert np.array_equal(H, 2.0 * M * np.outer(c, c))


@pytest.mark.parametrize("share", [0.01, 1.0])
def test_hessian_of_heavy_channels_is_no_slower_than_fp64(share):
    """Large values in one channel of a hundred, and in all: 16384 tokens on the int8 products against 16385 on the fp64 ones."""
    K = 1032
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((16385, K), generator=g, device="cuda").half()
    x[:, torch.randperm(K, generator=g, device="cuda")[:max(1, int(K * share))]] *= 200
    times = []
    for rows in (x[:16384], x):
        best = float("inf")
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(3):
                qqq.qqq_hessian(rows)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        times.append(best)
    assert times[0] < 1.1 * times[1], times


@pytest.mark.parametrize("K,N,shift", [(64, 17, 16), (520, 40, 48), (1032, 33, 0)])
def test_factorisation_on_a_workspace_in_use(K, N, shift):
    """The factorisation's flags and the lines that its workgroups share, on a workspace that begins anywhere and holds the last call's
    Hessian, factor and flags, then bytes that are no numbers: each call gives the oracle's codes."""
    need = int(qqq.lib().qqq_gptq_workspace_bytes(N, K))
    buf = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    ws = buf[shift:shift + need]
    for seed in (1, 2, 1):
        x, w = layer(2 * K + 10, K, N, 700 + K + seed)
        H = cal.hessian(x)
        codes, s_bits, _ = cal.gptq_quantize(w, H, 0.01)
        d_w, d_H = dev16(w), torch.from_numpy(H).cuda()
        w_nat = torch.empty((N, K // 8), dtype=torch.int32, device="cuda")
        s_w = torch.empty((N,), dtype=torch.float16, device="cuda")
        rc = qqq.lib().qqq_gptq_quantize_w4_perchannel(d_w.data_ptr(), d_H.data_ptr(), N, K, 0.01, w_nat.data_ptr(), s_w.data_ptr(),
                                                       ws.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
        assert rc == 0, qqq.lib().qqq_last_error()
        torch.cuda.synchronize()
        assert np.array_equal(f16_bits(s_w), s_bits) and np.array_equal(codes_of(w_nat, K), codes), seed
        assert (buf[:shift] == 0xFF).all() and (buf[shift + need:] == 0xFF).all()


@pytest.mark.parametrize("K,N", [(2176, 33), (1800, 1040)])
def test_updates_that_go_with_the_next_sweep(K, N):
    """More than three sweeps: the last columns receive a sweep's moves beside the next one, in one row of tiles and in several, a ragged last
    tile of columns among them.  Against a 64-bit torch sweep by the explicit inverse; the bar as above."""
    g = torch.Generator(device="cuda").manual_seed(78)
    x = torch.randn((900, 48), generator=g, device="cuda") @ torch.randn((48, K), generator=g, device="cuda") * 0.2
    x = (x + torch.randn(x.shape, generator=g, device="cuda")).to(torch.float16).to(torch.float64)
    H = 2.0 * (x.t().contiguous() @ x)
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.03).to(torch.float16)
    w_nat, s_w = qqq.qqq_gptq_quantize_w4_perchannel(w, H, 0.01)
    damped = H + 0.01 * H.diagonal().mean() * torch.eye(K, dtype=torch.float64, device="cuda")
    U = torch.linalg.cholesky(torch.cholesky_inverse(torch.linalg.cholesky(damped)), upper=True)
    U = U / U.diagonal()[:, None]
    run, s = w.to(torch.float64), s_w.to(torch.float64)
    codes = torch.zeros_like(run)
    for i in range(K):
        codes[:, i] = torch.round((run[:, i] / s).to(torch.float32)).clamp_(-7, 7)
        run[:, i + 1:] -= (run[:, i] - codes[:, i] * s)[:, None] * U[i, i + 1:]
    got = orc.w8_perchannel(w_nat.cpu().numpy().view(np.uint32), K)
    assert np.array_equal(got, codes.cpu().numpy().astype(got.dtype))


def _compensate(w, H):
    return qqq.qqq_gptq_quantize_w4_perchannel(w, H, 0.01)


@pytest.mark.parametrize("K,N,cus", [(200, 20, 8), (1032, 33, 8), (1288, 33, 16)])
def test_compensation_on_a_stream_confined_to_a_few_cus(K, N, cus):
    """The narrowest CU masks that a stream takes, a CU or two of each XCD: most of the factorisation's workgroups start when others are through."""
    import ctypes

    x, w = layer(2 * K + 10, K, N, 800 + K)
    d_w, H = dev16(w), torch.from_numpy(cal.hessian(x)).cuda()
    want = _compensate(d_w, H)
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so")
    handle, mask = ctypes.c_void_p(), (ctypes.c_uint32 * 8)((1 << cus) - 1)
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, mask) == 0
    with torch.cuda.stream(torch.cuda.ExternalStream(handle.value)):
        got = _compensate(d_w, H)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, got))
    hip.hipStreamDestroy(handle)


def test_compensation_captured_and_replayed():
    """Flags and tickets start anew in every replay, also with other inputs and eager calls in between."""
    K, N = 712, 48
    layers = []
    for seed in (5, 6):
        x, w = layer(2 * K + 10, K, N, 810 + seed)
        layers.append((dev16(w), torch.from_numpy(cal.hessian(x)).cuda()))
    want = [_compensate(*one) for one in layers]
    d_w, H = (t.clone() for t in layers[0])
    _compensate(d_w, H)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = _compensate(d_w, H)
    for i in (0, 1, 1, 0):
        d_w.copy_(layers[i][0])
        H.copy_(layers[i][1])
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(want[i], got)), i
        _compensate(*layers[1 - i])


@pytest.mark.parametrize("K,N", [(64, 17), (200, 20), (576, 48), (1032, 33), (1344, 16)])
@pytest.mark.parametrize("most", [1, 2, 3, 5])
def test_factorisation_by_a_few_workgroups(K, N, most):
    """One workgroup does all of it, two and more share it: the same bits."""
    x, w = layer(2 * K + 10, K, N, 820 + K)
    d_w, H = dev16(w), torch.from_numpy(cal.hessian(x)).cuda()
    want = _compensate(d_w, H)
    before = qqq.set_factor_workgroups(most)
    try:
        got = [_compensate(d_w, H) for _ in range(3)]
    finally:
        qqq.set_factor_workgroups(before)
    assert all(torch.equal(a, b) for one in got for a, b in zip(want, one))


def test_compensations_that_share_eight_cus():
    """Four calls at once on streams of the same eight CUs: none has its CUs to itself, each goes on with what it gets."""
    import ctypes

    K, N = 576, 24
    x, w = layer(2 * K + 10, K, N, 830)
    d_w, H = dev16(w), torch.from_numpy(cal.hessian(x)).cuda()
    want = _compensate(d_w, H)
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so")
    handles, got, mask = [], [], (ctypes.c_uint32 * 8)(0xFF)
    for _ in range(4):
        handles.append(ctypes.c_void_p())
        assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handles[-1]), 8, mask) == 0
    for _ in range(2):
        for handle in handles:
            with torch.cuda.stream(torch.cuda.ExternalStream(handle.value)):
                got.append(_compensate(d_w, H))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for one in got for a, b in zip(want, one))
    del got
    for handle in handles:
        hip.hipStreamDestroy(handle)
