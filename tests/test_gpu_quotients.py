"""The quantisers' quotients at their ties: rows whose largest magnitude is each of the finite fp16 values in turn and whose
other values lie as close to half a step as fp16 has them, against the CPU oracle (IEEE division), bit for bit."""
import numpy as np
import pytest
import torch

from oracle import qqq_oracle as orc
from paper_2406_09904_amd import binding as qqq

pytestmark = pytest.mark.gpu


def rows(levels, seed):
    """[31743, 128] fp16: the row's maximum, then values one or no fp16 step from (k + 1/2) max / levels, either sign."""
    rng = np.random.default_rng(seed)
    top = np.arange(1, 0x7C00, dtype=np.uint16)
    amax = top.view(np.float16).astype(np.float64)[:, None]
    k = rng.integers(0, levels, (top.size, 127)).astype(np.float64)
    near = ((k + 0.5) * amax / levels).astype(np.float16).view(np.uint16).astype(np.int32)
    near = np.clip(near + rng.integers(-1, 2, near.shape), 0, top[:, None].astype(np.int32)).astype(np.uint16)
    near |= (rng.integers(0, 2, near.shape) << 15).astype(np.uint16)
    return np.ascontiguousarray(np.concatenate([top[:, None], near], axis=1))


def dev(bits):
    return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.float16)


def test_activations():
    x = rows(127, 1)
    a_q, s_a = qqq.qqq_quant_act(dev(x))
    o_q, o_s = orc.quant_act(x)
    assert np.array_equal(s_a.cpu().numpy(), o_s)
    assert np.array_equal(a_q.cpu().numpy(), o_q)


@pytest.mark.parametrize("grouped", [False, True])
def test_weights(grouped):
    w = rows(7, 2)
    if grouped:
        w_nat, s_star, s_int, s_wc, s_wg = qqq.qqq_quantize_w4_pergroup(dev(w))
        o_nat, o_wg, o_star, o_int, o_wc = orc.quantize_w4_pergroup(w)
        for got, want in ((s_wg, o_wg), (s_wc, o_wc), (s_star, o_star)):
            assert np.array_equal(got.view(torch.int16).cpu().numpy().view(np.uint16), want)
        assert np.array_equal(s_int.cpu().numpy(), o_int)
    else:
        w_nat, s_w = qqq.qqq_quantize_w4_perchannel(dev(w))
        o_nat, o_s = orc.quantize_w4_perchannel(w)
        assert np.array_equal(s_w.view(torch.int16).cpu().numpy().view(np.uint16), o_s)
    assert np.array_equal(w_nat.cpu().numpy().view(np.uint32), o_nat)
