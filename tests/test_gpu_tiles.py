"""The 256 x 256 per-group and the 192 x 256 prefill tiles (their dequantised patches leave in two halves) on ragged
shapes against the CPU oracle: integers bit for bit, fp16 outputs within 1 ulp."""
import pytest

from paper_2406_09904_amd import binding as qqq
from tests.test_gpu_midsize import check, inputs, reference, run

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset():
    yield
    qqq.set_prefill_tuning(0)
    qqq.set_prefill_ksplit(0)
    qqq.set_group_mode_override(0)


@pytest.mark.parametrize("M,K,N,k_splits", [(256, 384, 256, 1), (300, 640, 784, 1), (513, 1408, 272, 2), (129, 128, 16, 1)])
@pytest.mark.parametrize("variant,hi,sg_max,knob", [("pg", 16, 16, 3), ("pgb", 16, 16, 5), ("pg", 127, 0, 0), ("real", 0, 0, 0)])
def test_256_row_tile(M, K, N, k_splits, variant, hi, sg_max, knob):
    a_q, s_a, w, s_w = inputs(M, K, N, M + K + N + 31)
    s_g, o_acc, o_y = reference(variant, a_q, s_a, w, s_w, K, N, 41, hi or 16)
    qqq.set_prefill_tuning(10)
    qqq.set_prefill_ksplit(k_splits)
    qqq.set_group_mode_override(knob)
    acc, y = run(variant, a_q, s_a, w, s_w, K, s_g=s_g, sg_max=sg_max)
    assert "tile=256x256" in qqq.last_route(), qqq.last_route()
    check(acc, y, o_acc, o_y)


@pytest.mark.parametrize("M,K,N,k_splits", [(192, 384, 256, 1), (197, 640, 784, 1), (400, 1408, 272, 2), (97, 128, 16, 1)])
@pytest.mark.parametrize("variant,hi,sg_max,knob", [("pc", 0, 0, 0), ("pg", 16, 16, 3), ("pgb", 16, 16, 5), ("pg", 127, 0, 0),
                                                    ("real", 0, 0, 0)])
def test_192_row_tile(M, K, N, k_splits, variant, hi, sg_max, knob):
    a_q, s_a, w, s_w = inputs(M, K, N, M + K + N + 37)
    s_g, o_acc, o_y = reference(variant, a_q, s_a, w, s_w, K, N, 43, hi or 16)
    qqq.set_prefill_tuning(12)
    qqq.set_prefill_ksplit(k_splits)
    qqq.set_group_mode_override(knob)
    acc, y = run(variant, a_q, s_a, w, s_w, K, s_g=s_g, sg_max=sg_max)
    assert "tile=192x256" in qqq.last_route(), qqq.last_route()
    check(acc, y, o_acc, o_y)


# tiles without their last 32 rows: as many rows as they have, one fewer, one tile and several, ragged columns, a K split
@pytest.mark.parametrize("tune,M,K,N,k_splits", [(12, 160, 384, 256, 1), (12, 777, 256, 272, 1), (12, 319, 1408, 784, 2), (10, 224, 384, 256, 1), (10, 447, 640, 272, 2),
                                                 (15, 96, 384, 256, 1), (15, 191, 640, 784, 1), (16, 96, 256, 144, 1), (16, 190, 640, 272, 2), (16, 33, 128, 16, 1)])
@pytest.mark.parametrize("variant,hi,sg_max,knob", [("pc", 0, 0, 0), ("pg", 16, 16, 3), ("pgb", 16, 16, 5), ("pg", 127, 0, 0), ("real", 0, 0, 0)])
def test_tiles_without_their_last_rows(tune, M, K, N, k_splits, variant, hi, sg_max, knob):
    if tune == 10 and variant == "pc":
        tune, M = 12, M * 5 // 7                         # (256 x 256 is for group scales)
    a_q, s_a, w, s_w = inputs(M, K, N, M + K + N + 53)
    s_g, o_acc, o_y = reference(variant, a_q, s_a, w, s_w, K, N, 47, hi or 16)
    qqq.set_kernel_override(2)
    qqq.set_prefill_tuning(tune)
    qqq.set_prefill_ksplit(k_splits)
    qqq.set_group_mode_override(knob)
    try:
        acc, y = run(variant, a_q, s_a, w, s_w, K, s_g=s_g, sg_max=sg_max)
    finally:
        qqq.set_kernel_override(0)
    assert "less 32 rows" in qqq.last_route(), qqq.last_route()
    check(acc, y, o_acc, o_y)
