"""Output columns past the last: whole row tiles whose last column block is partly or wholly empty, with one output to spare
behind every pixel or none, through every kernel family that shares the output stage.  Tolerances as in test_gpu_parity.py."""
import pytest

import plan_hooks as hooks
from oracle import direct_conv as oracle
from paper_1907_02129_amd import binding as icv
from paper_1907_02129_amd.workloads import ConvShape, make_tensors
from test_gpu_parity import check_against_oracle, run_fused_case, run_indirect

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", ["whole", "one_more"])
@pytest.mark.parametrize("K", [1, 31, 33, 65, 97, 130])
@pytest.mark.parametrize("kernel,dtype,C,k,plan", [
    ("gemm", "bf16", 64, 1, hooks.NO_SPLIT), ("gemm", "u8i8", 128, 1, hooks.NO_SPLIT), ("gemm", "f32", 32, 1, hooks.NO_SPLIT),
    ("patch", "bf16", 64, 3, icv.PLAN_WINDOW), ("freg", "u8i8", 64, 3, icv.PLAN_FILTER_REGS), ("freg", "bf16", 32, 3, icv.PLAN_FILTER_REGS),
    ("any", "bf16", 40, 1, hooks.NO_SPLIT), ("any", "f32", 20, 1, hooks.NO_SPLIT), ("lowc", "bf16", 4, 3, 0), ("gather", "bf16", 64, 3, icv.PLAN_GATHER)])
def test_columns_past_the_last(kernel, dtype, C, k, plan, K, rows):
    s = ConvShape(f"ragged_{kernel}_{dtype}_k{K}", 1, 16, 16 + (rows == "one_more"), C, K, k, k, PT=k // 2, PL=k // 2, PB=k // 2, PR=k // 2,
                  dtype=dtype, zero_point=77 if dtype == "u8i8" else 0, seed=900 + K)
    assert hooks.family(icv.plan_name(icv.make_params(s, plan=plan))) == kernel
    x, w = make_tensors(s)
    buf, _ = run_indirect(s, x, w, plan=plan)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    acc, mag = oracle.conv2d_abs(s, x, w) if dtype != "u8i8" else (oracle.conv2d_u8i8(s, x, w, s.zero_point), None)
    for stride in (0, K + 1):
        run_fused_case(s, x, w, acc, mag, True, True, plan=plan, out_pixel_stride=stride)
