"""The split-reduction kernel (small problems): both tiles, every way of reading rows (dense, 32-bit entries, block form), row
lengths around the 16-byte piece, one to many slices and stages, odd numbers of MFMA steps, ragged pixel and channel counts,
narrow and wide output, and the patch-matrix product.

Tolerances as in test_gpu_parity.py: exact for u8i8, the fp32 accumulation bound (any order) for the others."""
import numpy as np
import pytest
import torch

import icv_layout as layout
import plan_hooks as hooks
from oracle import direct_conv as oracle
from paper_1907_02129_amd import binding as icv
from paper_1907_02129_amd.workloads import ConvShape, make_tensors
from test_gpu_parity import check_against_oracle, run_fused_case, run_im2col, run_indirect

pytestmark = pytest.mark.gpu
TILE16, TILE32, WINDOW, NEVER = hooks.tile(8), hooks.tile(9), hooks.tile(10), hooks.tile(14)


def _shapes():
    out = []
    # (dtype, C, K): whole and ragged pieces; patches of fewer, as many and more stages than wavefronts
    for i, (dtype, C, K, k) in enumerate([("bf16", 512, 70, 3), ("bf16", 20, 16, 1), ("bf16", 24, 33, 3), ("bf16", 37, 17, 5), ("bf16", 64, 96, 3),
                                          ("bf16", 96, 15, 3), ("bf16", 224, 64, 2), ("u8i8", 512, 40, 3), ("u8i8", 17, 31, 3),
                                          ("u8i8", 48, 129, 1), ("u8i8", 64, 32, 5), ("u8i8", 100, 8, 3), ("f32", 64, 65, 3),
                                          ("f32", 4, 8, 3), ("f32", 33, 30, 3), ("f32", 256, 12, 1), ("f32", 48, 48, 2)]):
        zp = (0, 128, 77)[i % 3] if dtype == "u8i8" else 0
        pad = k // 2
        out.append(ConvShape(f"sp_{dtype}_c{C}_k{K}_{k}x{k}", 1 + i % 3, 9, 7 + i % 2, C, K, k, k, SY=1 + (i % 4 == 3), DX=1 + (i % 5 == 2),
                             PT=pad, PL=pad, PB=pad, PR=pad, dtype=dtype, zero_point=zp, seed=700 + i))
    # more tiles than the chip holds with all slices: fewer slices per tile
    out.append(ConvShape("sp_many", 4, 41, 43, 64, 40, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype="u8i8", zero_point=9, seed=730))
    out.append(ConvShape("sp_one_pixel", 1, 1, 1, 64, 5, 1, 1, seed=731))
    return out


@pytest.mark.parametrize("tile", [TILE16, TILE32], ids=["16x16", "32x32"])
@pytest.mark.parametrize("per_image", [0, icv.PLAN_PER_IMAGE], ids=["batch", "per_image"])
@pytest.mark.parametrize("s", _shapes(), ids=lambda s: s.name)
def test_split_reduction_matches_oracle(s, per_image, tile):
    print("conv", s.name, icv.plan_name(icv.make_params(s, plan=tile | per_image)), flush=True)
    x, w = make_tensors(s)
    buf, xd = run_indirect(s, x, w, plan=tile | per_image)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    if icv.im2col_bytes(buf.p):
        out2, _ = run_im2col(s, buf, xd)
        check_against_oracle(s, out2.cpu().numpy(), x, w)
    acc, mag = oracle.conv2d_abs(s, x, w) if s.dtype != "u8i8" else (oracle.conv2d_u8i8(s, x, w, s.zero_point), None)
    for stride in (0, s.K + 3):
        run_fused_case(s, x, w, acc, mag, True, True, plan=tile | per_image, out_pixel_stride=stride)


@pytest.mark.parametrize("dtype,C", [("bf16", 512), ("u8i8", 416), ("f32", 64), ("f32", 100)])
def test_small_problems_are_split_and_large_ones_are_not(dtype, C):
    """The library's own choice: same results as the plan it replaces, and no split at a batch that fills the chip (which the
    window kernel may take)."""
    s = ConvShape(f"sp_auto_{dtype}_{C}", 1, 7, 7, C, 96, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype=dtype, seed=740)
    print("conv", s.name, icv.plan_name(icv.make_params(s)), flush=True)
    assert hooks.family(icv.plan_name(icv.make_params(s))) == "split"
    assert "split" not in icv.plan_name(icv.make_params(s, plan=NEVER))
    x, w = make_tensors(s)
    buf, _ = run_indirect(s, x, w)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    buf, _ = run_indirect(s, x, w, plan=NEVER)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    big = s.with_(N=512)
    assert "split" not in icv.plan_name(icv.make_params(big))
    assert hooks.family(icv.plan_name(icv.make_params(big, plan=NEVER))) == {512: "patch", 416: "any", 64: "freg", 100: "any"}[C]
    if hooks.family(icv.plan_name(icv.make_params(big))) != "window":
        assert icv.plan_name(icv.make_params(big)) == icv.plan_name(icv.make_params(big, plan=NEVER))
        assert icv.packed_filter_bytes(icv.make_params(big)) == icv.packed_filter_bytes(icv.make_params(big, plan=NEVER))


@pytest.mark.parametrize("tile", [TILE16, TILE32], ids=["16x16", "32x32"])
def test_infinite_weights_stay_in_their_channel(tile):
    """An odd number of MFMA steps: what multiplies the missing half must be zeros, not another step's weights."""
    s = ConvShape("sp_inf", 1, 6, 5, 24, 40, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=741)      # 27 pieces, 14 steps
    x, w = make_tensors(s)
    clean = run_indirect(s, x, w, plan=tile)[0].output.clone()
    wd = icv.to_device(w).clone()
    wd[7] = float("inf")
    buf = icv.prepare(s, wd, plan=tile)
    icv.run(buf, icv.to_device(x))
    torch.cuda.synchronize()
    others = [k for k in range(s.K) if k != 7]
    assert torch.equal(buf.output[..., others], clean[..., others])
    assert not np.isfinite(buf.output[..., 7].cpu().numpy()).any()


def _window_shapes():
    mk = ConvShape
    out = []
    # fewer stages than wavefronts, as many, more; windows that cross images and rows; ragged K; strides and dilations
    for i, (dtype, n, h, w, C, K, r, s) in enumerate([
            ("bf16", 3, 7, 7, 512, 70, 3, 3), ("bf16", 2, 14, 13, 256, 64, 3, 3), ("bf16", 1, 9, 30, 64, 33, 5, 5), ("bf16", 2, 5, 6, 192, 130, 2, 2),
            ("u8i8", 5, 7, 7, 512, 40, 3, 3), ("u8i8", 2, 11, 17, 128, 65, 5, 5), ("u8i8", 1, 6, 5, 384, 8, 2, 3),
            ("f32", 2, 7, 9, 96, 31, 3, 3), ("f32", 1, 13, 12, 32, 64, 5, 5), ("f32", 3, 4, 4, 160, 20, 2, 2)]):
        zp = (0, 128, 77)[i % 3] if dtype == "u8i8" else 0
        for sy, dx, pad in ((1, 1, 1), (2, 2, 3)):
            out.append(mk(f"win_{dtype}_c{C}_{r}x{s}_s{sy}", n, h, w, C, K, r, s, SY=sy, SX=sy, DX=dx, PT=pad, PL=pad, PB=pad, PR=pad,
                          dtype=dtype, zero_point=zp, seed=750 + i))
    return out


@pytest.mark.parametrize("s", _window_shapes(), ids=lambda s: s.name)
def test_window_split_matches_oracle(s):
    p = icv.make_params(s, plan=WINDOW)
    name = icv.plan_name(p)
    print("conv", s.name, name, flush=True)
    x, w = make_tensors(s)
    buf, xd = run_indirect(s, x, w, plan=WINDOW)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    # (a window that does not fit LDS beside the entries stays with its own plan)
    fits = s.name != "win_bf16_c512_3x3_s2"
    assert (name.startswith("mfma_") and "64x64" in name and name.endswith("split")) == fits, name
    if fits:
        got, tail = layout.logical_indirection(p, buf.indirection, s.N * buf.Hout * buf.Wout)
        assert np.array_equal(got, oracle.indirection(s)) and np.all(tail == -1)
        out2, _ = run_im2col(s, buf, xd)
        check_against_oracle(s, out2.cpu().numpy(), x, w)
    acc, mag = oracle.conv2d_abs(s, x, w) if s.dtype != "u8i8" else (oracle.conv2d_u8i8(s, x, w, s.zero_point), None)
    for stride in (0, s.K + 3):
        run_fused_case(s, x, w, acc, mag, True, True, plan=WINDOW, out_pixel_stride=stride)


@pytest.mark.parametrize("s", [
    ConvShape("wide_bf16", 3, 53, 54, 416, 11, 3, 3, seed=770),
    ConvShape("wide_f32", 7, 29, 32, 256, 32, 3, 3, DY=2, DX=2, PT=2, PL=2, PB=2, PR=2, dtype="f32", seed=771),
    ConvShape("wide_u8", 1, 82, 82, 240, 32, 5, 5, dtype="u8i8", zero_point=77, seed=772),
], ids=lambda s: s.name)
def test_the_library_chooses_32x32_tiles_for_wide_rows(s):
    """Windows above 128 KB: rows gathered through 32-bit entries.  (Where the window is smaller the window kernel's 32 x 32 tile
    takes the problem, under a name of its own.)"""
    name = icv.plan_name(icv.make_params(s))
    print("conv", s.name, name, flush=True)
    assert name == {"bf16": "mfma_bf16_split_32x32", "f32": "mfma_f32_split_32x32", "u8i8": "mfma_i8_split_32x32"}[s.dtype]
    row = s.C * {"bf16": 2, "f32": 4, "u8i8": 1}[s.dtype]
    assert icv.tile_span_bound(icv.make_params(s), 32) * row > 128 * 1024
    x, w = make_tensors(s)
    buf, _ = run_indirect(s, x, w)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
