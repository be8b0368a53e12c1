"""17 to 64 rows with a workspace too small for the decode kernel: the prefill kernels need none, so the call runs there
whichever of the two the cost model ranks first; up to 16 rows it is refused.  Parity unpinned: sizes of this repository,
results against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2406_09904_amd import binding as qqq
from tests.test_gpu_midsize import inputs, reference
from tests.util import f16_bits, to_dev, ulp_distance

pytestmark = pytest.mark.gpu


def call(variant, args, s_g, ws, acc, **kw):
    if variant == "pc":
        return qqq.qqq_gemm_w4a8_perchannel(*args[:3], args[3], ws, acc_out=acc, **kw)
    if variant == "pg":
        return qqq.qqq_gemm_w4a8_pergroup(*args[:3], s_g, args[3], ws, sg_max=15, acc_out=acc, **kw)
    if variant == "pgany":
        return qqq.qqq_gemm_w4a8_pergroup(*args[:3], s_g, args[3], ws, acc_out=acc, **kw)
    return qqq.qqq_gemm_w4a8_pergroup_f16scale(*args[:3], s_g, args[3], ws, acc_out=acc, **kw)


@pytest.mark.parametrize("variant", ["pc", "pg", "pgany", "real"])
@pytest.mark.parametrize("M,K,N", [(17, 256, 64), (46, 1024, 10608), (64, 384, 1040)])
def test_small_workspace_is_no_reason_to_refuse(variant, M, K, N):
    a_q, s_a, w, s_w = inputs(M, K, N, M + K + N)
    s_g, o_acc, o_y = reference("pg" if variant == "pgany" else variant, a_q, s_a, w, s_w, K, N, 8,
                                127 if variant == "pgany" else 15)
    args = (to_dev(a_q, torch), to_dev(s_a, torch), qqq.qqq_pack_w4(to_dev(w, torch), K), to_dev(s_w.view(np.uint16), torch))
    d_sg = None if s_g is None else to_dev(s_g, torch)
    need = qqq.qqq_gemm_workspace_bytes(M, N, K)
    for nbytes in (16, need - 16, need):
        ws = torch.zeros((nbytes,), dtype=torch.uint8, device="cuda")
        acc = torch.full((M, N), -12345, dtype=torch.int32, device="cuda")
        y = call(variant, args, d_sg, ws, acc)
        if nbytes < need:
            route = qqq.last_route()
            assert "prefill persistent" in route or ("prefill" in route and "ksplit=1 " in route), (nbytes, route)
        torch.cuda.synchronize()
        assert np.array_equal(acc.cpu().numpy(), o_acc), (nbytes, qqq.last_route())
        assert ulp_distance(f16_bits(y), o_y).max() <= 1
    small = torch.zeros((16,), dtype=torch.uint8, device="cuda")
    few = (args[0][:16].contiguous(), args[1][:16].contiguous()) + args[2:]
    with pytest.raises(qqq.QQQError) as e:
        call(variant, few, d_sg, small, None)
    assert e.value.code == 3
    qqq.set_kernel_override(1)
    try:
        with pytest.raises(qqq.QQQError) as e:
            call(variant, args, d_sg, small, None)
        assert e.value.code == 3
    finally:
        qqq.set_kernel_override(0)
