// Host side of the split-reduction kernel: which problems take it with which tile, and the launch.
#include "icv_igemm_split_kernel.h"

namespace icv {

static const int kSplitTileRows[] = {16, 32};

// As many wavefronts per tile as keep every tile resident at once: a compute unit holds the wavefronts of one workgroup with
// all slices, of two with half of them, and so on.
static int slices_for(int64_t tiles, int64_t cus, int stages)
{
    int slices = kSplitMaxSlices;
    while (slices > 2 && tiles * slices > cus * kSplitMaxSlices) slices /= 2;
    return slices < stages ? slices : stages;
}

// The plan's own kernel walks a tile's reduction serially: its time is a start and so much per 128 bytes of reduction, as
// long as its grid is a single round.  The split kernel's is a start, so much per 128 bytes of the longest slice and
// so much per further round of its (smaller) tiles.  All in microseconds, fitted to graph replays of 90 problems
// (7 x 7 to 90 x 80 pixels, batch 1 to 140, 16 to 512 channels, 1x1 to 5x5); the split kernel has to promise a tenth.
// Measured, own kernel -> split kernel: one 7 x 7 image, 512 to 512 channels, 3x3: bf16 19.6 -> 8.7, uint8 15.6 -> 7.5, fp32 90.5
// -> 15.8; batch 8 of it: 20.6 -> 12.2, 14.2 -> 9.5, 92.4 -> 37.4; one 14 x 14 image, 256 to 256: bf16 11.7 -> 6.9, fp32
// 47.0 -> 11.5; 2 x 45 x 75, 64 to 64, fp32: 17.4 -> 13.8.  Past one round of the own kernel's tiles it loses: batch 64
// of the first in bf16 takes 27.0 against 46.2.  With the window in LDS (icv_igemm_window_split.hip): batch 16 of the first
// 21.0 -> 12.6, batch 32 21.4 -> 13.0 (uint8 15.6 -> 9.7), batch 64 25.0 against 25.2; 41 x 41, 320 to 208, 5x5 48.4 -> 17.8.  The bfloat16 and uint8 filter-in-registers kernel stays ahead everywhere
// (5.4 against 6.7 on one 28 x 28 image, 128 to 128 channels).
int choose_split(const icv_conv_params* p, const Geometry& g, double* us)
{
    const bool f32 = p->dtype == ICV_F32;
    const int64_t cus = 256;                     // (not the device's: a plan must not depend on where it is made)
    const int64_t row_bytes = (int64_t)p->C * g.elem_bytes;
    const double stages = (double)((g.T * ((row_bytes + 15) / 16) + 7) / 8);
    const int64_t images = g.per_image ? p->N : 1, img_rows = g.per_image ? (int64_t)g.Hout * g.Wout : g.M;
    const bool rows = g.kind == PLAN_MFMA && !g.patch_rows && !g.gemm_on_input;      // goes to the any-channel-count kernel
    double start = 3.7, per_stage;
    if (g.kind == PLAN_MFMA_FREG) {
        // Not what the kernel takes (16 channels, 3x3: 6.2 us; 32: 8.4; 64: 13 to 15 with one row block per pass, 16 to 18 with two)
        // but what the split kernel's model below, 1 to 2.4 us short of the truth in fp32, is to be compared with.  Fitted to
        // 185 drawn problems: of those the split kernel then takes none is slower, and 497 of the 498 us to be gained are.
        // (3.7 + 0.7 a stage made 14 of them slower: 8 x 9 x 9, 32 to 512 channels, 3x3 8.4 -> 10.6; 4 x 33 x 20, 16 to 480,
        // stride 2, 6.4 -> 8.1.)
        if (!f32) return -1;
        start = g.freg_mb == 1 ? 1.8 : 1.0;
        per_stage = g.freg_mb == 1 ? 0.64 : 0.8;
    } else if (g.kind == PLAN_MFMA_ANY || rows) {
        start = 2.9;
        per_stage = f32 ? 0.7 : 0.42;
    } else {
        per_stage = f32 ? 0.61 : (p->dtype == ICV_U8I8 && g.patch_rows ? 0.3 : 0.22);
    }
    const int64_t own_mr = g.kind == PLAN_MFMA_ANY ? kAnyTiles[g.run_variant].MR : g.MR, own_nr = g.kind == PLAN_MFMA_ANY ? kAnyTiles[g.run_variant].NR : g.NR;
    const int64_t own_tiles = images * ((img_rows + own_mr - 1) / own_mr) * ((p->K + own_nr - 1) / own_nr);
    if (own_tiles > cus) {
        // More than one round: in bf16 and uint8 only what measured slow there, tiles of 64 x 64 (two of them share a
        // compute unit at 1.35 times the time of one).  fp32 is bound by the matrix cores, whose work the tile's area counts.
        const double area = (double)g.MR * g.NR / 4096.0;
        if (g.kind != PLAN_MFMA || (rows && !f32)) return -1;
        if (f32) per_stage *= area * (double)own_tiles / cus;
        else if (own_tiles <= 2 * cus && area == 1.0) per_stage *= 1.35;
        else return -1;
    }
    int best = -1;
    double best_time = 0.9 * (start + per_stage * stages);
    for (int tile = SPLIT_16; tile <= SPLIT_32; tile++) {
        const int64_t MR = kSplitTileRows[tile];
        const int64_t tiles = images * ((img_rows + MR - 1) / MR) * ((p->K + MR - 1) / MR);
        const int slices = slices_for(tiles, cus, (int)stages);
        const double longest = (double)(((int)stages + slices - 1) / slices) * slices;
        double t;
        if (tile == SPLIT_16) {
            const double more = tiles > cus ? (double)(tiles - cus) / cus : 0.0;
            t = 3.6 + (f32 ? 0.083 : 0.07) * longest + more * (0.25 + (f32 ? 0.08 : 0.047) * stages);
        } else {
            const double more = (double)((tiles + cus - 1) / cus - 1);
            t = 3.9 + (f32 ? 0.22 : 0.1) * longest + more * (0.35 + (f32 ? 0.21 : 0.09) * stages);
        }
        if (t < best_time) { best_time = t; best = tile; }
    }
    // the window in LDS: 64 x 64 tiles, one workgroup per compute unit
    if (g.kind == PLAN_MFMA && !g.per_image && g.T >= 4 && row_bytes % 128 == 0) {
        const int64_t span = tile_span_bound(p, g.Hout, g.Wout, 64);
        if (span < 65535 && window_split_lds_bytes(g.T, row_bytes, span) <= kLdsPerCu) {
            const int64_t tiles = ((g.M + 63) / 64) * ((p->K + 63) / 64);
            const double rounds = (double)((tiles + cus - 1) / cus);
            const double t = 1.2 + rounds * (4.0 + (f32 ? 0.6 : 0.1) * stages);
            if (t < best_time) { best_time = t; best = kChooseWindow; }
        }
    }
    *us = best_time;
    return best;
}

int launch_igemm_split(const icv_conv_params* p, const Geometry& g, const void* input, const void* packed,
                       const int32_t* ind, const void* zero_row, void* out, int a_mode, hipStream_t s)
{
    const int tile = g.split_tile;
    if (tile < SPLIT_16 || tile > SPLIT_32) return ICV_ERR_UNSUPPORTED;
    SplitArgs a{};      // every field starts at zero; the ones this call uses are set below
    a.a = (const uint8_t*)input;
    a.zero_row = (const uint8_t*)zero_row;
    a.w = (const uint8_t*)packed;
    a.out = out;
    a.row_bytes = p->C * g.elem_bytes;
    if (a.row_bytes < 16) return ICV_ERR_UNSUPPORTED;
    const int rows = a_mode != A_GATHERED ? SPLIT_DENSE : (g.kind == PLAN_MFMA_FREG ? SPLIT_BLOCK16 : SPLIT_INT32);
    if (rows == SPLIT_BLOCK16) {
        a.rec = (const int4*)ind;
        a.ent = (const uint16_t*)(a.rec + g.img_tiles);
    } else if (rows == SPLIT_INT32) {
        a.ind = ind;
    }
    a.stride_bytes = g.in_stride * g.elem_bytes;
    a.a_row_stride = a_mode == A_DENSE_WORKSPACE ? (int64_t)g.T * a.row_bytes : (int64_t)a.stride_bytes;
    a.a_rows = a_mode == A_DENSE_WORKSPACE ? patch_matrix_rows(g) : g.M;
    a.image_bytes = a_mode == A_GATHERED ? g.image_bytes : 0;
    const int64_t MR = kSplitTileRows[tile], NR = MR;
    const int64_t images = g.per_image ? p->N : 1, img_tiles = (g.img_rows + MR - 1) / MR, n_tiles = (p->K + NR - 1) / NR;
    const int64_t tiles = images * img_tiles * n_tiles;
    if (tiles >= (1ll << 31) - 8 || g.img_tiles >= (1ll << 31)) return ICV_ERR_UNSUPPORTED;
    a.img_tiles = (uint32_t)img_tiles;
    a.img_rows = (uint32_t)g.img_rows;
    while ((1 << a.block_shift) < g.MR) ++a.block_shift;
    if ((1 << a.block_shift) != g.MR || g.MR < 32) return ICV_ERR_UNSUPPORTED;
    a.total_tiles = (uint32_t)tiles;
    a.tiles_per_xcd = (uint32_t)((tiles + 7) / 8);
    a.K = p->K; a.T = g.T; a.out_stride = g.out_stride;
    a.P = (a.row_bytes + 15) / 16;
    a.step_taps = 8 / a.P;
    a.step_pieces = 8 % a.P;
    a.by_P = make_fast_div((uint32_t)a.P);
    a.n_steps = (g.T * a.P + 1) / 2;
    a.n_stages = (a.n_steps + 3) / 4;
    const bool tail = a.row_bytes % 16 != 0;
    a.tail_shift = tail ? 16 - a.row_bytes % 16 : 0;
    // The workgroups of an XCD share its L2: the larger operand is the one they should all read together
    const int64_t filter_bytes = (int64_t)p->K * g.T * a.row_bytes, input_bytes = (int64_t)p->N * p->Hin * p->Win * a.row_bytes;
    a.rows_inner = filter_bytes > input_bytes ? 1 : 0;
    a.inner = (uint32_t)(a.rows_inner ? images * img_tiles : n_tiles);
    a.by_inner = make_fast_div(a.inner);
    a.by_img_tiles = make_fast_div(a.img_tiles);
    a.slices = slices_for(tiles, device_cu_count(), a.n_stages);
    a.vector_out = a.out_stride % 4 == 0 ? 1 : 0;
    a.ep = g.ep;
    switch (p->dtype) {
    case ICV_BF16: return launch_split_bf16(a, tile, rows, tail, s);
    case ICV_U8I8: return launch_split_u8(a, tile, rows, tail, s);
    case ICV_F32: return launch_split_f32(a, tile, rows, tail, s);
    }
    return ICV_ERR_UNSUPPORTED;
}

}  // namespace icv
