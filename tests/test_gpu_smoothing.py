"""The smoothing search where its kernels change path: K at and past the rows kept in registers (4096 weights, 8192
activations), channel groups not divisible by the eight XCDs, more grid points than the workspace holds at a time, ragged token
counts, each of the four tiles of the loss product, and the search point by point; against the steps it stands for, one by one.

The smoothed tensors, thresholds and vectors are compared bit for bit.  A loss is an fp64 sum built on exact integers and
the fp32 reference product: from the steps' own integers, scales and reference product in another order it differs by
rounding of fp64 only, 1e-12 (and the search's own reference product is the one qqq_fp16_gemm_nt returns).
"""
import pytest
import torch

from paper_2406_09904_amd import binding as qqq
from paper_2406_09904_amd import synth

pytestmark = pytest.mark.gpu


BY_STEPS = " + loss"                                     # after the last point's GEMM


@pytest.mark.parametrize("M,K,N,G,route", [
    (1, 128, 16, 3, "loss tile=64x128 points=3"), (70, 4096, 144, 9, "loss tile=64x128 points=5 + loss tile=64x128 points=4"),
    (33, 4224, 272, 4, "loss tile=64x128 points=4"), (200, 8192, 128, 3, "loss tile=64x128 points=3"),
    (9, 8320, 1040, 9, "loss tile=64x128 points=5 + loss tile=64x128 points=4"), (87, 128, 2832, 23, "loss tile=128x128 points=23"),
    (300, 512, 2064, 9, "loss tile=128x256 points=9"), (300, 512, 4096, 21, "loss tile=128x256 points=21"),
    (700, 256, 2064, 40, "loss tile=128x128 points=25 + loss tile=128x128 points=15"),
    (500, 2944, 4080, 8, "loss tile=128x512 points=8"),
    (5, 512, 48, 3, "loss tile=64x128 points=3"), (5, 640, 48, 3, "loss tile=64x128 points=3"), (5, 1024, 48, 3, "loss tile=64x128 points=3"),
    (5, 1152, 144, 3, "loss tile=64x128 points=3"), (5, 2048, 48, 3, "loss tile=64x128 points=3"), (5, 2176, 48, 3, "loss tile=64x128 points=3"),
    (5, 2688, 48, 3, "loss tile=64x128 points=3"), (5, 3200, 48, 3, "loss tile=64x128 points=3"), (5, 3968, 48, 3, "loss tile=64x128 points=3"),
    (19, 8320, 48, 2, BY_STEPS), (3, 16384, 16, 9, BY_STEPS), (130, 12416, 64, 5, BY_STEPS), (40, 6144, 256, 1, BY_STEPS)])
def test_grid_points_equal_their_steps(M, K, N, G, route):
    x = torch.from_numpy(synth.activations_fp16(M, K, 700 + M, "normal", 4 / K, 40.0)).cuda()
    w = torch.from_numpy(synth.weights_fp16(N, K, 701 + M)).cuda()
    w[N // 2].zero_()                                    # a channel of zeros
    got = qqq.qqq_adaptive_smoothing(x, w, G)
    assert qqq.last_route().endswith(route), qqq.last_route()
    amax = qqq.qqq_channel_absmax(x)
    assert torch.equal(amax, x.float().abs().amax(dim=0))
    ref = qqq.qqq_fp16_gemm_nt(x, w).double()
    losses = []
    for g in range(G):
        xs, ws, _ = qqq.qqq_smooth_apply(x, w, amax, got["sigmas"][g:g + 1].clone())
        a_q, s_a = qqq.qqq_quant_act(xs)
        w_nat, s_w = qqq.qqq_quantize_w4_perchannel(ws)
        acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
        qqq.qqq_gemm_w4a8_perchannel(a_q, s_a, qqq.qqq_pack_w4(w_nat, K), s_w, qqq.new_workspace(M, N, K), acc_out=acc)
        losses.append((acc.double() * s_a.double()[:, None] * s_w.double()[None, :] - ref).square().sum())
    losses = torch.stack(losses)
    assert torch.allclose(got["losses"], losses, rtol=1e-12, atol=0.0)
    best = int(got["best"].item())
    assert best == int(torch.argmin(got["losses"]).item())
    xs, ws, s = qqq.qqq_smooth_apply(x, w, amax, got["sigmas"][best:best + 1].clone())
    assert torch.equal(got["xs"], xs) and torch.equal(got["ws"], ws) and torch.equal(got["s"], s)


@pytest.mark.parametrize("M,K,N,G,route", [
    (20, 128, 16, 9, "loss tile=64x128 points=9"), (20, 1024, 16, 9, "loss tile=64x128 points=5 + loss tile=64x128 points=4"),
    (70, 4096, 32, 17, " + loss tile=64x128 points=3 + loss tile=64x128 points=2"), (33, 4224, 16, 12, " + loss tile=64x128 points=3"),
    (500, 128, 16, 9, "loss tile=64x128 points=5 + loss tile=64x128 points=4"), (20, 128, 32, 16, "loss tile=64x128 points=16"),
    (20, 128, 32, 17, "loss tile=64x128 points=17")])
def test_more_points_than_the_smoothed_weights_have_room_for(M, K, N, G, route):
    """From more than N / 2 points on, smoothing vectors are made batch by batch in the workspace (the sixteen of N = 32 just fit)."""
    test_grid_points_equal_their_steps(M, K, N, G, route)


def _search(x, w, G, xs, ws):
    """The C entry point with the caller's outputs."""
    (M, K), N = x.shape, w.shape[0]
    s, sigmas = torch.empty(K, device="cuda"), torch.empty(G, device="cuda")
    losses, best = torch.empty(G, dtype=torch.float64, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
    work = torch.empty(int(qqq.lib().qqq_smoothing_workspace_bytes(M, N, K)), dtype=torch.uint8, device="cuda")
    rc = qqq.lib().qqq_adaptive_smoothing(x.data_ptr(), w.data_ptr(), M, N, K, G, xs.data_ptr(), ws.data_ptr(), s.data_ptr(), sigmas.data_ptr(),
                                          losses.data_ptr(), best.data_ptr(), work.data_ptr(), work.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0, qqq.lib().qqq_last_error()
    return s, sigmas, best, losses


@pytest.mark.parametrize("M,K,N,G", [(20, 256, 64, 9), (70, 4096, 144, 9), (300, 512, 2064, 9), (40, 6144, 256, 1)])
def test_search_in_place(M, K, N, G):
    """The smoothed layer may take the layer's own place: bit for bit what it is elsewhere (the losses but for the order of fp64 sums)."""
    x = torch.from_numpy(synth.activations_fp16(M, K, 730 + M, "normal", 4 / K, 40.0)).cuda()
    w = torch.from_numpy(synth.weights_fp16(N, K, 731 + M)).cuda()
    xs, ws = torch.empty_like(x), torch.empty_like(w)
    want = _search(x, w, G, xs, ws)
    got = _search(x, w, G, x, w)
    assert torch.equal(x, xs) and torch.equal(w, ws)
    assert all(torch.equal(a, b) for a, b in zip(want[:3], got[:3])) and torch.allclose(want[3], got[3], rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("M,K,N,G,at", [(20, 256, 64, 9, 0), (2100, 1024, 2064, 9, 1), (300, 512, 320, 5, 37), (40, 6144, 256, 1, 0)])
def test_search_with_the_smoothed_weights_in_the_activations_place(M, K, N, G, at):
    """Smoothed weights in the buffer of X, from its row `at` on: X is smoothed before they are written."""
    buf = torch.empty((max(M, at + N), K), dtype=torch.float16, device="cuda")
    x, ws = buf[:M], buf[at:at + N]
    x.copy_(torch.from_numpy(synth.activations_fp16(M, K, 735 + M, "normal", 4 / K, 40.0)))
    w = torch.from_numpy(synth.weights_fp16(N, K, 736 + M)).cuda()
    xs, want_xs, want_ws = torch.empty_like(x), torch.empty_like(x), torch.empty_like(w)
    want = _search(x, w, G, want_xs, want_ws)
    got = _search(x, w, G, xs, ws)
    assert torch.equal(xs, want_xs) and torch.equal(ws, want_ws)
    assert all(torch.equal(a, b) for a, b in zip(want[:3], got[:3])) and torch.allclose(want[3], got[3], rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("M,K,N,G,tile", [(20, 256, 144, 8, "64x128"), (87, 128, 2832, 23, "128x128"), (300, 512, 2064, 9, "128x256"),
                                          (500, 2944, 4080, 8, "128x512")])
def test_overflowing_points_lose(M, K, N, G, tile):
    """Points at which a weight overflows, in tiles with rows past M and channels past N: their loss is infinite, as its terms are, and a later,
    finite one wins.  (One heavy input channel, so that every row's code in it is not 0.)"""
    g = torch.Generator(device="cuda").manual_seed(740 + M)
    x = torch.randn((M, K), generator=g, device="cuda") * 0.05
    x[:, 7] = torch.rand(M, generator=g, device="cuda") + 7.0
    w = torch.randn((N, K), generator=g, device="cuda") * 0.02
    w[N // 3, 7] = 12000.0                               # 8 times that is past fp16's 65504
    x, w = x.to(torch.float16), w.to(torch.float16)
    got = qqq.qqq_adaptive_smoothing(x, w, G)
    assert "loss tile=%s" % tile in qqq.last_route(), qqq.last_route()
    amax, ref = qqq.qqq_channel_absmax(x), qqq.qqq_fp16_gemm_nt(x, w).double()
    losses = []
    for i in range(G):
        xs, ws, _ = qqq.qqq_smooth_apply(x, w, amax, got["sigmas"][i:i + 1].clone())
        a_q, s_a = qqq.qqq_quant_act(xs)
        w_nat, s_w = qqq.qqq_quantize_w4_perchannel(ws)
        acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
        qqq.qqq_gemm_w4a8_perchannel(a_q, s_a, qqq.qqq_pack_w4(w_nat, K), s_w, qqq.new_workspace(M, N, K), acc_out=acc)
        losses.append((acc.double() * s_a.double()[:, None] * s_w.double()[None, :] - ref).square().sum())
    losses = torch.stack(losses)
    assert torch.isinf(losses[0]) and torch.isfinite(losses[-1])
    assert torch.allclose(got["losses"], losses, rtol=1e-12, atol=0.0), (got["losses"], losses)
    assert int(got["best"].item()) == int(torch.argmin(losses).item())


@pytest.mark.parametrize("M,K,N,tile", [
    (1, 16, 1, "32x32"), (65, 48, 129, "32x32"), (64, 64, 128, "32x32"), (130, 80, 255, "32x32"), (257, 16, 9000, "32x32"),
    (33, 256, 7000, "32x32"), (33, 1040, 300, "64x128"), (65, 1296, 129, "64x128"), (64, 320, 128, "64x128"), (130, 336, 255, "64x128"),
    (17, 2064, 1, "64x128"), (1, 272, 1, "64x128"), (257, 80, 9000, "64x128")])
def test_reference_product_tiles(M, K, N, tile):
    """Ragged 64 x 128 tiles with K not divisible by a stage of 64, and the one-wave tiles of small problems:
    |error| <= K 2^-24 sum |x w| (fp32 sums in any order)."""
    x = torch.from_numpy(synth.activations_fp16(M, K, 800 + K, "normal", 0.02, 10.0)).cuda()
    w = torch.from_numpy(synth.weights_fp16(N, K, 801 + K)).cuda()
    y = qqq.qqq_fp16_gemm_nt(x, w).double()
    assert qqq.last_route() == "fp16 tile=" + tile
    bound = (x.double().abs() @ w.double().abs().t().contiguous()) * K * 2.0 ** -24
    assert bool(((y - x.double() @ w.double().t().contiguous()).abs() <= bound).all())
