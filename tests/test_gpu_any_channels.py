"""Rows of any length and alignment on the tensor cores: every tile, row lengths around the 16-byte piece, ragged
pixel and channel counts, dense and gathered rows, the patch-matrix product, and what a row's neighbours hold.

Tolerances as in test_gpu_parity.py: exact for u8i8, the fp32 accumulation bound (any order) for the others."""
import numpy as np
import pytest
import torch

import plan_hooks as hooks
from oracle import direct_conv as oracle
from paper_1907_02129_amd import binding as icv
from paper_1907_02129_amd.workloads import ConvShape, make_tensors
from test_gpu_parity import check_against_oracle, run_fused_case, run_im2col, run_indirect

pytestmark = pytest.mark.gpu


DT = {"bf16": "bf16", "u8i8": "i8", "f32": "f32"}         # a plan name's type


def _shapes():
    out = []
    # channels: bytes per row below, at and above whole 16-byte pieces; K: one, two and more column blocks, ragged
    for i, (dtype, C, K) in enumerate([("bf16", 5, 33), ("bf16", 40, 24), ("bf16", 9, 65), ("bf16", 24, 130), ("bf16", 48, 192),
                                       ("bf16", 37, 8), ("bf16", 100, 64), ("u8i8", 7, 40), ("u8i8", 15, 20), ("u8i8", 17, 70),
                                       ("u8i8", 48, 129), ("u8i8", 96, 32), ("f32", 1, 9), ("f32", 3, 64), ("f32", 5, 31),
                                       ("f32", 8, 66), ("f32", 33, 140)]):
        zp = (0, 128, 77)[i % 3] if dtype == "u8i8" else 0
        out.append(ConvShape(f"any_{dtype}_c{C}_k{K}", 2, 13, 11, C, K, 3, 3, SY=1 + i % 2, PT=1, PL=1, PB=1, PR=1,
                             dtype=dtype, zero_point=zp, seed=600 + i))
    # enough row tiles for the 128-row tiles (K > 32: at least 512 workgroups of 128 rows)
    out.append(ConvShape("any_wide_128x128", 3, 150, 147, 12, 70, 1, 2, seed=630))
    out.append(ConvShape("any_wide_128x64", 3, 149, 148, 18, 64, 2, 1, dtype="u8i8", zero_point=5, seed=631))
    # 1x1: the input itself is the matrix
    out.append(ConvShape("any_1x1_bf16", 3, 9, 7, 40, 72, 1, 1, seed=632))
    out.append(ConvShape("any_1x1_u8", 2, 17, 5, 33, 48, 1, 1, dtype="u8i8", zero_point=200, seed=633))
    out.append(ConvShape("any_one_pixel", 1, 1, 1, 24, 8, 1, 1, seed=634))
    return out


@pytest.mark.parametrize("plan", [0, icv.PLAN_PER_IMAGE, icv.PLAN_GATHER, hooks.ANY], ids=["auto", "per_image", "gather", "any"])
@pytest.mark.parametrize("s", _shapes(), ids=lambda s: s.name)
def test_any_channel_count_matches_oracle(s, plan):
    name = icv.plan_name(icv.make_params(s, plan=plan))
    print("conv", s.name, name, flush=True)
    assert hooks.family(name) in (("any",) if plan == hooks.ANY else ("any", "split", "lowc", "window"))
    x, w = make_tensors(s)
    buf, xd = run_indirect(s, x, w, plan=plan)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    out2, _ = run_im2col(s, buf, xd)
    check_against_oracle(s, out2.cpu().numpy(), x, w)


@pytest.mark.parametrize("dtype,C", [("bf16", 20), ("f32", 7), ("bf16", 5)])
def test_a_row_never_sees_its_neighbours(dtype, C):
    """One pixel full of infinities and NaN, in a tensor whose pixels are further apart than C with NaN in between:
    exactly the outputs whose window holds that pixel are affected."""
    s = ConvShape("any_nan", 1, 9, 10, C, 36, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype=dtype, seed=640)
    x, w = make_tensors(s)
    buf, xd = run_indirect(s, x, w)
    clean = buf.output.clone()
    stride = C + 3
    wide = torch.full((1, 9, 10, stride), float("nan"), dtype=xd.dtype, device="cuda:0")
    wide[..., :C] = xd
    wide[0, 4, 5, :C] = float("inf")
    wide[0, 4, 5, 0] = float("nan")
    b2 = icv.prepare(s, icv.to_device(w), in_pixel_stride=stride)
    icv.run(b2, wide.contiguous())
    torch.cuda.synchronize()
    hit = np.zeros((9, 10), bool)
    hit[3:6, 4:7] = True
    got = b2.output[0].cpu().numpy()
    assert np.isnan(got[hit]).all()
    assert np.array_equal(got[~hit], clean[0].cpu().numpy()[~hit])


@pytest.mark.parametrize("s,tiles", [
    # (the number of images decides the tile, the buffers of one image serve all: blocks of 128 entries, tiles of 64 and 128 rows)
    (ConvShape("one_128x128", 1, 150, 147, 12, 70, 1, 2, seed=635), {1: "64x64", 3: "128x128"}),
    (ConvShape("one_128x64", 1, 149, 148, 18, 64, 2, 1, dtype="u8i8", zero_point=5, seed=636), {1: "64x64", 3: "128x64"}),
    (ConvShape("one_rows", 1, 64, 61, 96, 190, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=637), {1: "64x64", 5: "128x64", 14: "128x64"}),
    (ConvShape("one_f32", 1, 61, 67, 48, 136, 2, 2, dtype="f32", seed=638), {1: "64x64", 14: "128x64"}),
], ids=lambda v: v.name if hasattr(v, "name") else "")
def test_one_image_buffer_under_every_tile(s, tiles):
    """With the any-channel-count kernel itself, and with the library's choice among the kernels that read the buffer."""
    x1, w = make_tensors(s)
    for plan in (icv.PLAN_PER_IMAGE | hooks.ANY, icv.PLAN_PER_IMAGE):
        built = icv.prepare(s, icv.to_device(w), plan=plan)
        torch.cuda.synchronize()
        for n, tile in tiles.items():
            big = s.with_(N=n)
            x, _ = make_tensors(big)
            p = icv.make_params(big, plan=plan)
            print("conv", s.name, n, icv.plan_name(p), flush=True)
            if plan & hooks.ANY:
                assert icv.plan_name(p) == f"mfma_{DT[s.dtype]}_any_{tile}"
            else:
                assert hooks.family(icv.plan_name(p)) == ("window" if s.name == "one_rows" else "any")
            out = torch.full((n, built.Hout, built.Wout, s.K), -7, dtype=built.output.dtype, device="cuda:0")
            icv.conv2d_nhwc(p, icv.to_device(x), built.packed, built.indirection, built.zero_row, out)
            torch.cuda.synchronize()
            for i in sorted({0, n - 1}):
                check_against_oracle(s, out[i:i + 1].cpu().numpy(), x[i:i + 1], w)


@pytest.mark.parametrize("s,tile,per_image", [
    (ConvShape("lib_128x128", 34, 31, 31, 24, 256, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=641), "128x128", True),
    (ConvShape("lib_128x64", 51, 50, 50, 24, 64, 3, 3, seed=642), "128x64", True),
    (ConvShape("lib_128x128_u8", 40, 84, 84, 40, 96, 3, 3, SY=2, SX=2, PT=1, PL=1, PB=1, PR=1, dtype="u8i8", zero_point=7, seed=643), "128x128", False),
    (ConvShape("lib_128x64_f32", 39, 56, 56, 4, 64, 5, 5, PT=2, PL=2, PB=2, PR=2, dtype="f32", seed=644), "128x64", False),
], ids=lambda v: getattr(v, "name", ""))
def test_large_tiles_where_the_library_chooses_them(s, tile, per_image):
    """Rows of one to three pieces, whose window the window kernel does not take."""
    plan = icv.PLAN_PER_IMAGE if per_image else 0
    assert icv.plan_name(icv.make_params(s, plan=plan)) == f"mfma_{DT[s.dtype]}_any_{tile}"
    print("conv", s.name, flush=True)
    x, w = make_tensors(s)
    buf, _ = run_indirect(s, x, w, plan=plan)
    one = s.with_(N=1)
    for n in (0, s.N // 2, s.N - 1):
        check_against_oracle(one, buf.output[n:n + 1].cpu().numpy(), x[n:n + 1], w)


@pytest.mark.parametrize("plan", [0, icv.PLAN_PER_IMAGE, icv.PLAN_GATHER], ids=["auto", "per_image", "gather"])
@pytest.mark.parametrize("k", [(3, 3), (7, 7), (5, 4)], ids=["3x3", "7x7", "5x4"])
@pytest.mark.parametrize("dtype,C", [("bf16", 1), ("bf16", 2), ("bf16", 3), ("u8i8", 1), ("u8i8", 2), ("u8i8", 3), ("u8i8", 4),
                                     ("f32", 1), ("f32", 2), ("f32", 3)])
def test_first_layers_of_few_channels(dtype, C, k, plan):
    """Rows of one to twelve bytes, whole and ragged paddings of the flattened reduction, pixels packed and apart."""
    zp = 41 * C if dtype == "u8i8" else 0
    s = ConvShape(f"first_{dtype}_c{C}", 3, 23, 19, C, 40 + 30 * (C % 2), *k, SY=2, SX=1 + C % 2, PT=k[0] // 2, PL=k[1] // 2,
                  PB=1, PR=2, dtype=dtype, zero_point=zp, seed=650 + C)
    x, w = make_tensors(s)
    assert icv.plan_name(icv.make_params(s, plan=plan)).endswith("lowc_64x64")
    buf, xd = run_indirect(s, x, w, plan=plan)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    out2, _ = run_im2col(s, buf, xd)
    check_against_oracle(s, out2.cpu().numpy(), x, w)
    stride = C + 1
    apart = torch.full((3, 23, 19, stride), 9, dtype=torch.float32, device="cuda:0").to(xd.dtype)
    apart[..., :C] = xd
    b2 = icv.prepare(s, icv.to_device(w), plan=plan, in_pixel_stride=stride)
    icv.run(b2, apart)
    torch.cuda.synchronize()
    assert torch.equal(b2.output, buf.output)


@pytest.mark.parametrize("C,k", [(1, 1), (1, 3), (16, 1), (5, 3), (31, 3), (113, 3), (1024, 1), (1025, 1), (440, 5)])
def test_filter_sums_behind_the_packed_filter(C, k):
    """Filters of fewer, as many and more bytes than a lane's 16 and a wavefront's 1024, at any alignment, extreme weights."""
    s = ConvShape(f"sums_{C}_{k}", 1, 8, 8, C, 37, k, k, dtype="u8i8", zero_point=3, seed=645)
    _, w = make_tensors(s)
    w[0], w[1] = -128, 127
    p = icv.make_params(s)
    packed = torch.zeros(icv.packed_filter_bytes(p), dtype=torch.uint8, device="cuda:0")
    icv.pack_filter(p, icv.to_device(w), packed)
    sums = packed[-((s.K * 4 + 15) // 16 * 16):].cpu().numpy().view(np.int32)[:s.K]
    assert np.array_equal(sums, w.astype(np.int64).reshape(s.K, -1).sum(axis=1))


def _accumulators(s, x, w):
    return oracle.conv2d_abs(s, x, w) if s.dtype != "u8i8" else (oracle.conv2d_u8i8(s, x, w, s.zero_point), None)


@pytest.mark.parametrize("relu,narrow", [(True, True), (False, True), (True, False)], ids=["relu_narrow", "narrow", "relu"])
@pytest.mark.parametrize("K,hw", [(40, (23, 19)), (300, (23, 19)), (300, (31, 31)), (300, (3, 2)), (70, (130, 131))],
                         ids=["k40", "k300", "k300_two_blocks", "k300_one_tile", "many_tiles"])
@pytest.mark.parametrize("dtype,C", [("bf16", 1), ("bf16", 2), ("bf16", 3), ("u8i8", 1), ("u8i8", 2), ("u8i8", 3), ("u8i8", 4),
                                     ("f32", 1), ("f32", 2), ("f32", 3)])
def test_first_layers_of_few_channels_with_fused_output(dtype, C, K, hw, relu, narrow):
    """The output stage of every short row length: one and many column groups of a workgroup, one tile, more tiles than single
    teams take; padded output pixels, the whole-batch and the one-image buffer."""
    s = ConvShape(f"first_f_{dtype}_c{C}_k{K}", 2, *hw, C, K, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype=dtype,
                  zero_point=60 * C if dtype == "u8i8" else 0, seed=660 + C)
    x, w = make_tensors(s)
    assert hooks.family(icv.plan_name(icv.make_params(s))) == "lowc"
    acc, mag = _accumulators(s, x, w)
    for plan in (0, icv.PLAN_PER_IMAGE):
        run_fused_case(s, x, w, acc, mag, relu, narrow, plan=plan, out_pixel_stride=K + 3)


@pytest.mark.parametrize("k", [(1, 1), (3, 3)], ids=["1x1", "3x3"])
@pytest.mark.parametrize("dtype,C", [("bf16", 8), ("bf16", 16), ("u8i8", 16), ("u8i8", 32)])
def test_short_rows_of_16_and_32_bytes(dtype, C, k):
    """Compact entries and rows of whole pieces in the short-row kernel, which keeps them where the window kernel does not take
    them: bfloat16 pointwise layers by the library's choice, the others by the hook."""
    s = ConvShape(f"short_{dtype}_c{C}", 3, 23, 19, C, 70, *k, SY=2, PT=k[0] // 2, PL=k[1] // 2, PB=1, PR=2, dtype=dtype,
                  zero_point=3 * C if dtype == "u8i8" else 0, seed=655)
    x, w = make_tensors(s)
    acc, mag = _accumulators(s, x, w)
    for per_image in (0, icv.PLAN_PER_IMAGE):
        p = icv.make_params(s, plan=hooks.NO_SPLIT | per_image)
        print("conv", s.name, icv.plan_name(p), flush=True)
        assert hooks.family(icv.plan_name(p)) == "lowc" and icv.get_indirection_layout(p).entry_bytes == 2
        if dtype == "bf16" and k == (1, 1):
            assert icv.plan_name(icv.make_params(s, plan=per_image)) == icv.plan_name(p)
        buf, _ = run_indirect(s, x, w, plan=hooks.NO_SPLIT | per_image)
        check_against_oracle(s, buf.output.cpu().numpy(), x, w)
        run_fused_case(s, x, w, acc, mag, True, True, plan=hooks.NO_SPLIT | per_image, out_pixel_stride=73)


_FUSED = [
    # (shape, tile): every tile with whole rows and with a padded last piece, rows shorter than a piece, dense rows
    (ConvShape("fu_128x128_whole", 3, 150, 147, 24, 70, 1, 2, seed=681), "any_128x128"),
    (ConvShape("fu_128x128_tail", 3, 150, 147, 12, 70, 1, 2, seed=682), "any_128x128"),
    (ConvShape("fu_128x64_whole", 3, 149, 148, 48, 64, 2, 1, dtype="u8i8", zero_point=128, seed=683), "any_128x64"),
    (ConvShape("fu_128x64_tail", 3, 149, 148, 18, 64, 2, 1, dtype="u8i8", zero_point=5, seed=684), "any_128x64"),
    (ConvShape("fu_64x64_whole", 2, 13, 11, 48, 192, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=685), "any_64x64"),
    (ConvShape("fu_64x64_tail", 2, 13, 11, 37, 130, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=686), "any_64x64"),
    (ConvShape("fu_128x32_whole", 2, 13, 11, 40, 24, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=687), "any_128x32"),
    (ConvShape("fu_128x32_tail", 2, 13, 11, 37, 8, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=688), "any_128x32"),
    (ConvShape("fu_short", 2, 13, 11, 5, 16, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype="u8i8", zero_point=99, seed=689), "any_64x64"),
    (ConvShape("fu_1x1", 3, 9, 7, 40, 72, 1, 1, seed=690), "any_64x64"),
    (ConvShape("fu_1x1_u8", 2, 17, 5, 33, 48, 1, 1, dtype="u8i8", zero_point=200, seed=691), "any_64x64"),
    (ConvShape("fu_f32_64x64", 2, 13, 11, 33, 140, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype="f32", seed=692), "any_64x64"),
    (ConvShape("fu_f32_128x32", 2, 13, 11, 5, 31, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype="f32", seed=693), "any_128x32"),
]


@pytest.mark.parametrize("relu,narrow", [(True, True), (False, True), (True, False), (False, False)],
                         ids=["relu_narrow", "narrow", "relu", "bias"])
@pytest.mark.parametrize("s,tile", _FUSED, ids=lambda v: getattr(v, "name", ""))
def test_fused_output_of_every_tile(s, tile, relu, narrow):
    """Bias, ReLU and narrow output of the any-channel-count kernel itself (never the split-reduction kernel in its place), padded
    output pixels, with the whole-batch and the one-image buffer."""
    x, w = make_tensors(s)
    acc, mag = _accumulators(s, x, w)
    for plan in (hooks.NO_SPLIT, hooks.NO_SPLIT | icv.PLAN_PER_IMAGE):
        assert icv.plan_name(icv.make_params(s, plan=plan)) == f"mfma_{DT[s.dtype]}_{tile}"
        run_fused_case(s, x, w, acc, mag, relu, narrow, plan=plan, out_pixel_stride=s.K + 5)


@pytest.mark.parametrize("plan", [0, icv.PLAN_PER_IMAGE], ids=["auto", "per_image"])
@pytest.mark.parametrize("dtype,C,K", [("bf16", 96, 140), ("bf16", 96, 64), ("bf16", 160, 24), ("u8i8", 192, 70), ("f32", 48, 33)])
def test_aligned_rows_that_are_gathered_per_kernel_element(dtype, C, K, plan):
    """Rows of whole 64-byte units that no power of two fits: the any-channel-count kernel itself, whose larger tiles run on a
    large batch, and what the library chooses on that kernel's buffers."""
    s = ConvShape(f"rows_{dtype}_{C}", 5, 45, 47, C, K, 3, 3, SY=1 + (K == 24), PT=1, PL=1, PB=1, PR=1, dtype=dtype,
                  zero_point=11 if dtype == "u8i8" else 0, seed=670)
    name = icv.plan_name(icv.make_params(s, plan=plan))
    print("conv", s.name, name, flush=True)
    assert hooks.family(name) in ("any", "window")
    big = s.with_(N=40)
    tile = {("bf16", 96): "128x64", ("bf16", 160): "128x32", ("u8i8", 192): "128x128", ("f32", 48): "128x64"}[dtype, C]
    assert icv.plan_name(icv.make_params(s, plan=plan | hooks.ANY)) == f"mfma_{DT[dtype]}_any_" + ("128x32" if C == 160 else "64x64")
    assert icv.plan_name(icv.make_params(big, plan=plan | hooks.ANY)) == f"mfma_{DT[dtype]}_any_{tile}"
    assert hooks.family(icv.plan_name(icv.make_params(big, plan=plan))) == ("any" if dtype == "f32" else "window")
    xb, wb = make_tensors(big)
    one = s.with_(N=1)
    for hook in (0, hooks.ANY):
        bbuf, _ = run_indirect(big, xb, wb, plan=plan | hook)
        for n in (0, 17, 39):
            check_against_oracle(one, bbuf.output[n:n + 1].cpu().numpy(), xb[n:n + 1], wb)
    x, w = make_tensors(s)
    buf, _ = run_indirect(s, x, w, plan=plan | hooks.ANY)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    buf, xd = run_indirect(s, x, w, plan=plan)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    gathered, _ = run_indirect(s, x, w, plan=icv.PLAN_GATHER | plan)
    check_against_oracle(s, gathered.output.cpu().numpy(), x, w)
    out2, _ = run_im2col(s, buf, xd)
    check_against_oracle(s, out2.cpu().numpy(), x, w)
