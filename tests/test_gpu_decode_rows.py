"""The decode kernel's three-row-tile instances on ragged shapes against the CPU oracle: integers bit for bit, fp16
outputs within 1 ulp."""
import pytest

from paper_2406_09904_amd import binding as qqq
from tests.test_gpu_midsize import check, inputs, reference, run

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset():
    yield
    qqq.set_kernel_override(0)
    qqq.set_skinny_tuning(0, 0, 0, 0)


@pytest.mark.parametrize("M", [33, 48, 49])
@pytest.mark.parametrize("K,N,waves", [(640, 11008, 0), (384, 16448, 0), (2048, 11008, 4), (2048, 4096, 0), (1152, 272, 0)])
@pytest.mark.parametrize("variant,hi,sg_max", [("pc", 0, 0), ("pg", 16, 16), ("pg", 127, 0), ("real", 0, 0)])
def test_decode_three_row_tiles(M, K, N, waves, variant, hi, sg_max):
    """64-, 32- and 16-channel workgroups, eight and four waves (at most one and more than one workgroup per CU)."""
    a_q, s_a, w, s_w = inputs(M, K, N, M + K + N + 51)
    s_g, o_acc, o_y = reference(variant, a_q, s_a, w, s_w, K, N, 61, hi or 16)
    qqq.set_kernel_override(1)
    qqq.set_skinny_tuning(0, 0, waves, 0)
    acc, y = run(variant, a_q, s_a, w, s_w, K, s_g=s_g, sg_max=sg_max)
    assert ("mt=3" if M <= 48 else "mt=4") in qqq.last_route(), qqq.last_route()
    check(acc, y, o_acc, o_y)
