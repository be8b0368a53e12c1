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
