"""The window kernel: every tile on every form of rows, entries and output it accepts, against the CPU oracle.

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

TILES = ["128x64", "64x64", "128x32", "32x32_r8", "64x128", "64x64_r4"]


def window(tile):
    return hooks.tile(11) | (tile + 2) << 12


def _shapes():
    mk, out = ConvShape, []
    # stages of four, three and two steps, rows of an odd number of pieces, of two pieces and of one; padded last pieces; reductions
    # with fewer stages than shares; ragged pixels and channels; strides, dilations, asymmetric padding; block-form entries (filter in registers)
    for i, (dtype, n, h, w, C, K, r, s, st, d, pad) in enumerate([
            ("bf16", 3, 13, 11, 64, 70, 3, 3, 1, 1, 1), ("bf16", 2, 13, 11, 48, 192, 3, 3, 1, 1, 1), ("bf16", 2, 17, 9, 96, 33, 3, 3, 2, 1, 1),
            ("bf16", 2, 12, 19, 40, 65, 3, 3, 1, 2, 2), ("bf16", 3, 10, 9, 16, 40, 5, 5, 1, 1, 2), ("bf16", 5, 9, 7, 8, 24, 3, 3, 1, 1, 1),
            ("bf16", 2, 13, 14, 37, 130, 3, 3, 1, 1, 1), ("bf16", 1, 14, 13, 160, 31, 5, 5, 2, 1, 2), ("bf16", 2, 8, 9, 416, 64, 3, 3, 1, 1, 1),
            ("bf16", 1, 1, 5, 32, 9, 2, 2, 1, 1, 1), ("bf16", 2, 23, 20, 128, 100, 3, 3, 1, 1, 1), ("bf16", 1, 40, 61, 96, 66, 3, 3, 1, 1, 0),
            ("u8i8", 3, 13, 11, 64, 70, 3, 3, 1, 1, 1), ("u8i8", 2, 13, 11, 48, 129, 3, 3, 2, 1, 1), ("u8i8", 2, 9, 14, 33, 64, 5, 5, 1, 1, 2),
            ("u8i8", 2, 12, 9, 16, 33, 3, 3, 1, 1, 1), ("u8i8", 1, 11, 12, 417, 40, 3, 3, 1, 1, 1), ("u8i8", 2, 10, 13, 256, 96, 3, 3, 1, 2, 2),
            ("u8i8", 3, 13, 9, 32, 48, 1, 1, 1, 1, 0), ("u8i8", 2, 11, 13, 16, 70, 1, 1, 2, 1, 1), ("u8i8", 2, 7, 9, 32, 33, 1, 2, 1, 1, 0),
            ("f32", 2, 13, 11, 16, 66, 3, 3, 1, 1, 1), ("f32", 2, 10, 12, 33, 40, 3, 3, 2, 1, 1), ("f32", 1, 9, 10, 4, 20, 4, 4, 1, 1, 2),
            ("f32", 1, 12, 13, 24, 31, 5, 5, 1, 1, 2)]):
        zp = (0, 128, 77)[i % 3] if dtype == "u8i8" else 0
        out.append(mk(f"win_{dtype}_c{C}_k{K}_{r}x{s}_s{st}_d{d}", n, h, w, C, K, r, s, SY=st, SX=st, DY=d, DX=d, PT=pad, PL=pad,
                      PB=pad - (pad > 1), PR=pad, dtype=dtype, zero_point=zp, seed=1000 + i))
    return out


@pytest.mark.parametrize("per_image", [0, icv.PLAN_PER_IMAGE], ids=["whole_batch", "per_image"])
@pytest.mark.parametrize("tile", range(len(TILES)), ids=TILES)
@pytest.mark.parametrize("s", _shapes(), ids=lambda s: s.name)
def test_window_matches_oracle(s, tile, per_image):
    plan = window(tile) | per_image
    name = icv.plan_name(icv.make_params(s, plan=plan))
    print("conv", s.name, name, flush=True)
    assert f"_window_{TILES[tile]}_" in name
    # block-form entries, or int32 ones where other kernels read the buffer too
    assert icv.get_indirection_layout(icv.make_params(s, plan=plan)).entry_bytes == (4 if per_image and "_any_" in name else 2)
    x, w = make_tensors(s)
    buf, xd = run_indirect(s, x, w, plan=plan)
    one = s.with_(N=1) if per_image else s          # what the buffer describes
    got, tail = layout.logical_indirection(buf.p, buf.indirection, one.N * buf.Hout * buf.Wout)
    assert np.array_equal(got, oracle.indirection(one)) and np.all(tail == -1)
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)
    if icv.im2col_bytes(buf.p):                     # the patch matrix by the same filter, through the kernel of the plan's buffers
        out2, _ = run_im2col(s, buf, xd)
        check_against_oracle(s, out2.cpu().numpy(), x, w)
    acc, mag = oracle.conv2d_abs(s, x, w) if s.dtype != "u8i8" else (oracle.conv2d_u8i8(s, x, w, s.zero_point), None)
    for stride in (0, s.K + 3):
        run_fused_case(s, x, w, acc, mag, True, True, plan=plan, out_pixel_stride=stride)


@pytest.mark.parametrize("s,pieces", [
    # the window of whole rows does not fit, whatever the tile: chunks of equal and of two sizes, in stages and step by step
    (ConvShape("chunks_even", 1, 30, 66, 512, 40, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=1030), 64),
    (ConvShape("chunks_uneven", 1, 25, 70, 352, 33, 3, 3, SY=2, SX=2, PT=1, PL=1, PB=1, PR=1, seed=1031), 44),
    (ConvShape("chunks_of_odd_steps", 1, 12, 180, 416, 40, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype="u8i8", zero_point=9, seed=1032), 26),
], ids=lambda v: getattr(v, "name", ""))
@pytest.mark.parametrize("tile", range(len(TILES)), ids=TILES)
def test_rows_in_chunks(s, pieces, tile):
    p = icv.make_params(s, plan=window(tile))
    assert f"_window_{TILES[tile]}_" in icv.plan_name(p)
    # window and zero row, rows an odd number of pieces apart, and the entries
    rows = int(TILES[tile].split("x")[0])
    assert (icv.tile_span_bound(p, rows) + 1) * (pieces | 1) * 16 + s.R * s.S * rows * 2 > 160 * 1024
    x, w = make_tensors(s)
    buf, _ = run_indirect(s, x, w, plan=window(tile))
    check_against_oracle(s, buf.output.cpu().numpy(), x, w)


@pytest.mark.parametrize("tile", range(len(TILES)), ids=TILES)
@pytest.mark.parametrize("dtype,C", [("bf16", 20), ("bf16", 48), ("f32", 7)])
def test_a_row_never_sees_its_neighbours(dtype, C, tile):
    """One pixel of infinities and NaN, in a tensor whose pixels are further apart than C with NaN in between, and one channel of
    infinite weights: exactly the outputs that hold them are affected."""
    s = ConvShape("win_nan", 1, 9, 10, C, 36, 3, 3, PT=1, PL=1, PB=1, PR=1, dtype=dtype, seed=1040)
    x, w = make_tensors(s)
    clean = run_indirect(s, x, w, plan=window(tile))[0].output.clone()
    xd, wd = icv.to_device(x), icv.to_device(w).clone()
    stride = C + 3
    wide = torch.full((1, 9, 10, stride), float("nan"), dtype=xd.dtype, device="cuda:0")
    wide[..., :C] = xd
    wide[0, 4, 5, :C] = float("inf")
    wide[0, 4, 5, 0] = float("nan")
    wd[7] = float("inf")
    buf = icv.prepare(s, wd, plan=window(tile), in_pixel_stride=stride)
    icv.run(buf, wide.contiguous())
    torch.cuda.synchronize()
    hit = np.zeros((9, 10), bool)
    hit[3:6, 4:7] = True
    others = [k for k in range(s.K) if k != 7]
    got = buf.output[0].cpu().numpy()
    assert np.isnan(got[hit]).all()
    assert np.array_equal(got[~hit][:, others], clean[0].cpu().numpy()[~hit][:, others])
    assert not np.isfinite(got[..., 7]).any()


@pytest.mark.parametrize("dtype,C,K,kernel,plans", [
    ("bf16", 256, 24, "any", (8,)), ("bf16", 16, 48, "any", (0, 8)), ("u8i8", 32, 256, "any", (0, 8)), ("u8i8", 128, 304, "freg", (0, 8)),
    ("bf16", 96, 40, "any", (0, 8)), ("f32", 64, 32, "any", (8,))])
def test_the_library_chooses_it(dtype, C, K, kernel, plans):
    """Where it is the library's own choice: a large batch, several of its images against the oracle; one image of it."""
    k = 5 if dtype == "f32" else 3
    s = ConvShape(f"win_auto_{dtype}_{C}", 48, 40, 39, C, K, k, k, PT=k // 2, PL=k // 2, PB=k // 2, PR=k // 2, dtype=dtype, seed=1050)
    one = s.with_(N=1)
    x, w = make_tensors(s)
    for plan in plans:                              # (8: icv.PLAN_PER_IMAGE)
        name = icv.plan_name(icv.make_params(s, plan=plan))
        print("conv", s.name, plan, name, flush=True)
        assert "_window_" in name and kernel in name
        buf, _ = run_indirect(s, x, w, plan=plan)
        for n in (0, 23, 47):
            check_against_oracle(one, buf.output[n:n + 1].cpu().numpy(), x[n:n + 1], w)


@pytest.mark.parametrize("tile", [0, 3], ids=[TILES[0], TILES[3]])
def test_graph_replays_match_eager(tile):
    """Captured once, replayed on new inputs with eager calls in between (LDS above the default limit: set on the first call)."""
    s = ConvShape("win_graph", 2, 24, 40, 160, 72, 3, 3, PT=1, PL=1, PB=1, PR=1, seed=1060)
    x, w = make_tensors(s)
    buf, xd = run_indirect(s, x, w, plan=window(tile))
    xd = xd.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        icv.run(buf, xd)
    for i in range(4):
        xi, _ = make_tensors(s.with_(seed=1061 + i))
        xd.copy_(icv.to_device(xi))
        torch.cuda.synchronize()
        buf.output.fill_(-7)
        icv.run(buf, xd)
        torch.cuda.synchronize()
        eager = buf.output.clone()
        buf.output.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(buf.output, eager)
