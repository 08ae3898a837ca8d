// Host side of the window kernel: which problems run it with which tile, and the launch.
#include "icv_igemm_window_kernel.h"

namespace icv {

// MR x NR tile, split over WM x WN wavefronts times WS shares of the reduction (launch_window_instances has the instantiations)
struct WindowTile {
    int32_t MR, NR, waves, WS;
};
static const WindowTile kWindowTiles[] = {
    {128, 64, 4, 1}, {64, 64, 4, 1}, {128, 32, 4, 1}, {32, 32, 8, 8}, {64, 128, 4, 1}, {64, 64, 8, 4},
};

// Time in microseconds: constant, per MFMA step of a wavefront, per KB of window for the first round of tiles and, per further tile a
// compute unit gets, the same three; for rows of an odd number of pieces, whose steps need an address each, two more terms per step.
// Least squares of relative errors over 6000 drawn problems (7 to 96 pixels a side, batch 1 to 256, 16 to 512 channels, 8 to 512
// columns, 3x3 to 7x7), graph replays; rms error 8 to 12 %.
static const float kWindowTime[3][kNumWindowTiles][8] = {      // fp32, bfloat16, uint8
    {{5.284f, 0.256f, 0.021f, 0.932f, 0.339f, 0.005f, 0.076f, 0.0f},
     {4.400f, 0.145f, 0.024f, 0.645f, 0.170f, 0.002f, 0.082f, 0.001f},
     {4.500f, 0.145f, 0.022f, 0.490f, 0.168f, 0.016f, 0.088f, 0.006f},
     {5.138f, 0.264f, 0.022f, 1.377f, 0.316f, 0.010f, 0.250f, 0.093f},
     {5.128f, 0.256f, 0.021f, 0.836f, 0.314f, 0.0f, 0.065f, 0.013f},
     {6.137f, 0.489f, 0.020f, 3.659f, 0.680f, 0.013f, 0.170f, 0.059f}},
    {{5.324f, 0.060f, 0.017f, 0.907f, 0.058f, 0.021f, 0.056f, 0.017f},
     {4.602f, 0.040f, 0.018f, 0.523f, 0.036f, 0.016f, 0.052f, 0.008f},
     {4.701f, 0.042f, 0.018f, 0.509f, 0.033f, 0.022f, 0.051f, 0.014f},
     {5.120f, 0.056f, 0.011f, 1.456f, 0.071f, 0.011f, 0.084f, 0.028f},
     {5.127f, 0.059f, 0.017f, 0.802f, 0.059f, 0.014f, 0.055f, 0.008f},
     {5.885f, 0.092f, 0.014f, 3.637f, 0.127f, 0.021f, 0.071f, 0.072f}},
    {{6.018f, 0.059f, 0.013f, 0.964f, 0.057f, 0.020f, 0.059f, 0.019f},
     {5.112f, 0.042f, 0.012f, 0.685f, 0.036f, 0.012f, 0.049f, 0.013f},
     {5.265f, 0.041f, 0.014f, 0.689f, 0.033f, 0.020f, 0.051f, 0.019f},
     {5.631f, 0.053f, 0.009f, 1.474f, 0.076f, 0.007f, 0.071f, 0.089f},
     {5.738f, 0.057f, 0.012f, 0.856f, 0.060f, 0.009f, 0.058f, 0.009f},
     {6.554f, 0.098f, 0.009f, 2.534f, 0.109f, 0.008f, 0.070f, 0.103f}},
};
// The kernels it stands in for, the same way: constant, per 128 bytes of the reduction, per KB of window, and the three again per further
// tile.  Any-channel-count kernel by kAnyTiles, then the pixel-range kernel with 64 x 64, 128 x 64, 128 x 128 and 256 x 64 tiles; rms
// error 5 to 14 %.
static const float kOwnTime[3][8][6] = {
    {{3.631f, 3.724f, 0.0f, 0.0f, 1.850f, 0.0f},
     {3.507f, 2.131f, 0.0f, 0.324f, 0.961f, 0.0f},
     {3.136f, 0.801f, 0.0f, 0.0f, 0.688f, 0.0f},
     {2.757f, 1.029f, 0.0f, 0.0f, 0.726f, 0.0f},
     {5.998f, 0.636f, 0.015f, 0.0f, 0.854f, 0.0f},
     {5.751f, 1.299f, 0.0f, 0.0f, 1.518f, 0.0f},
     {9.880f, 1.810f, 0.025f, 0.0f, 0.0f, 1.162f},
     {6.040f, 1.934f, 0.017f, 0.0f, 0.0f, 1.526f}},
    {{7.422f, 0.626f, 0.0f, 0.641f, 0.581f, 0.0f},
     {6.546f, 0.400f, 0.0f, 0.438f, 0.442f, 0.0f},
     {3.862f, 0.360f, 0.0f, 0.700f, 0.189f, 0.0f},
     {3.710f, 0.501f, 0.0f, 0.321f, 0.428f, 0.0f},
     {5.132f, 0.284f, 0.005f, 0.350f, 0.031f, 0.043f},
     {5.646f, 0.439f, 0.005f, 0.784f, 0.120f, 0.039f},
     {7.322f, 0.468f, 0.025f, 0.0f, 0.467f, 0.016f},
     {7.308f, 0.434f, 0.010f, 0.069f, 0.470f, 0.009f}},
    {{5.390f, 0.946f, 0.0f, 1.959f, 0.537f, 0.0f},
     {5.413f, 0.585f, 0.0f, 1.863f, 0.317f, 0.0f},
     {3.779f, 0.428f, 0.0f, 0.727f, 0.227f, 0.0f},
     {4.466f, 0.510f, 0.0f, 0.398f, 0.405f, 0.0f},
     {4.725f, 0.420f, 0.006f, 3.668f, 0.0f, 0.0f},
     {5.704f, 0.476f, 0.008f, 0.0f, 0.250f, 0.035f},
     {8.543f, 0.508f, 0.023f, 2.688f, 0.450f, 0.005f},
     {5.928f, 0.522f, 0.017f, 3.140f, 0.475f, 0.0f}},
};
// Windows of more than 128 KB of whole rows are left to the other kernels: in pieces, or alone on a compute unit, they lost to the
// any-channel-count kernel by up to two thirds (stride 2 on 93 x 115 pixels of 317 channels).
static const int64_t kWindowPieces = 128 * 64;
static const int64_t kCus = 256;      // (not the device's: a plan must not depend on where it is made)

static int64_t tiles_of(const icv_conv_params* p, const Geometry& g, const WindowTile& t)
{
    const int64_t images = g.per_image ? p->N : 1, img_rows = g.per_image ? (int64_t)g.Hout * g.Wout : g.M;
    // (both are powers of two: a division of 64 bits is some 30 cycles, twelve of them for the six tiles)
    return images * ((img_rows + t.MR - 1) >> __builtin_ctz((unsigned)t.MR)) * ((p->K + t.NR - 1) >> __builtin_ctz((unsigned)t.NR));
}

static size_t window_lds_bytes(const WindowTile& t, int T, int64_t cap_rows, int chunk)
{
    const int64_t w = (cap_rows + 1) * (chunk | 1) * 16 + (int64_t)T * t.MR * 2;
    const int64_t parts = t.WS > 1 ? t.waves * 4096 : 0;
    return (size_t)(w > parts ? w : parts);
}

// MFMA steps of a stage for chunks of these many pieces; 0: an address per step
static int stage_steps(int P, int chunk)
{
    if (P % 2) return 0;
    const int last = P % chunk ? P % chunk : chunk;
    for (int u = 4; u >= 2; u--)
        if (chunk % (2 * u) == 0 && last % (2 * u) == 0) return u;
    return 0;
}

// Pieces of a row that are in LDS at a time, 0: the tile's window does not fit.  The window gets the whole LDS while no compute unit has
// a second tile, else what leaves room for another workgroup, of four wavefronts for two more (1 to 1.1 % above the best of 53, 80
// and 160 KB over the fitted problems).  Rows of an odd number of pieces are not cut (a step would straddle two chunks).
static int window_chunk(const WindowTile& t, int T, int P, int64_t cap_rows, int64_t tiles)
{
    const int64_t per_cu = (tiles + kCus - 1) / kCus, most = t.waves <= 4 ? 3 : 2;
    auto fits = [&](int c, size_t budget) { return window_lds_bytes(t, T, cap_rows, c) <= budget && (cap_rows + 1) * (c | 1) < 65536; };
    for (int64_t n = per_cu < most ? per_cu : most; n >= 1; n--) {
        const size_t budget = kLdsPerCu / (size_t)n / 1024 * 1024;
        if (fits(P, budget)) return P;
        if (P % 2) continue;
        int first = 0;
        for (int c = P - 2; c >= 4; c -= 2) {
            if (!fits(c, budget)) continue;
            if (!first) first = c;
            if (2 * c < first) break;
            if (stage_steps(P, c)) return c;
        }
        if (first >= 8 || (n == 1 && first)) return first;
    }
    return 0;
}

// Whether window_chunk finds any number of pieces for it: the whole row or, cut, the fewest (LDS use grows with them)
static bool window_fits_lds(const WindowTile& t, int T, int P, int64_t cap_rows)
{
    auto fits = [&](int c) { return window_lds_bytes(t, T, cap_rows, c) <= kLdsPerCu && (cap_rows + 1) * (c | 1) < 65536; };
    return cap_rows < 65536 && (fits(P) || (P % 2 == 0 && P >= 6 && fits(4)));
}

static bool window_takes(const Geometry& g, int64_t row_bytes)
{
    return row_bytes >= 16 && g.T * row_bytes < (1ll << 27);      // (32-bit offsets in a column block of the filter)
}

void window_times(const icv_conv_params* p, const Geometry& g, WindowTimes* times)
{
    for (int tile = 0; tile < kNumWindowTiles; tile++) times->us[tile] = kNoWindow;
    const int64_t row_bytes = (int64_t)p->C * g.elem_bytes;
    if (!window_takes(g, row_bytes)) return;
    const int P = (int)((row_bytes + 15) / 16);
    const double all_steps = (double)((g.T * P + 1) / 2);
    for (int64_t rows = 32; rows <= 128; rows *= 2) {
        const int64_t cap_rows = tile_span_bound(p, g.Hout, g.Wout, rows);
        if (cap_rows * P > kWindowPieces) return;      // (nor those of more rows)
        const double kb = (double)cap_rows * P / 64.0;
        for (int tile = 0; tile < kNumWindowTiles; tile++) {
            const WindowTile& t = kWindowTiles[tile];
            if (t.MR != rows || (t.NR > 32 && 2 * p->K <= t.NR) || !window_fits_lds(t, g.T, P, cap_rows)) continue;
            const float* k = kWindowTime[p->dtype][tile];
            const double steps = all_steps / t.WS, tiles = (double)tiles_of(p, g, t), more = tiles > kCus ? tiles / kCus - 1.0 : 0.0;
            double us = k[0] + k[1] * steps + k[2] * kb + more * (k[3] + k[4] * steps + k[5] * kb);
            if (P % 2) us += steps * (k[6] + more * k[7]);
            times->us[tile] = us;
        }
    }
}

int fastest_window(const WindowTimes& times, int64_t block_rows, double* us)
{
    int best = -1;
    for (int tile = 0; tile < kNumWindowTiles; tile++)
        if (kWindowTiles[tile].MR <= block_rows && times.us[tile] < kNoWindow && (best < 0 || times.us[tile] < *us)) {
            best = tile;
            *us = times.us[tile];
        }
    return best;
}

// What the plan's own kernel takes, modelled; 1e30: not one that is compared
double own_kernel_time(const icv_conv_params* p, const Geometry& g)
{
    const int64_t images = g.per_image ? p->N : 1, img_rows = g.per_image ? (int64_t)g.Hout * g.Wout : g.M;
    const int P = (p->C * g.elem_bytes + 15) / 16;
    if (g.kind == PLAN_MFMA_FREG) {
        // uint8 (an XOR per fragment that the window kernel does once per byte; in bfloat16 and fp32 level): row blocks in passes
        if (p->dtype != ICV_U8I8) return 0.0;
        const int64_t wn = g.freg_wn, groups = (p->K + 32 * wn - 1) / (32 * wn), ranges = kCus / groups > 1 ? kCus / groups : 1;
        const int64_t blocks = images * ((img_rows + 31) / 32), per = (blocks + ranges - 1) / ranges;
        const double passes = (double)((per + 4 / wn - 1) / (4 / wn)), steps = g.T * P / 2.0;
        return 3.31 + 0.0162 * steps + passes * (0.919 + 0.0271 * steps);
    }
    int at;
    int64_t mr, nr, span = 0;
    if (g.kind == PLAN_MFMA_ANY) {
        at = g.run_variant;
        if (at > 3) return 1e30;
        mr = kAnyTiles[at].MR; nr = kAnyTiles[at].NR;
    } else if (g.kind == PLAN_MFMA && g.patch_rows) {
        mr = kTileVariants[g.variant].MR; nr = kTileVariants[g.variant].NR;
        // 256 x 128 tiles, which need a grid of them that fills the chip, keep their problems: of 4000 drawn ones the window kernel was chosen
        // for 16 in bfloat16 by a fit with an rms error of 28 %, and took 1.14 times as long (0.89 to 1.26); by a better fit (12 %) for 15 in
        // uint8, 1.06 times as long
        if (mr == 256 && nr == 128) return 0.0;
        at = mr == 64 ? 4 : (mr == 128 ? (nr == 64 ? 5 : 6) : 7);
        span = tile_span_bound(p, g.Hout, g.Wout, mr);
    } else {
        return 1e30;
    }
    const float* k = kOwnTime[p->dtype][at];
    const double tiles = (double)(images * ((img_rows + mr - 1) / mr) * ((p->K + nr - 1) / nr)), more = tiles > kCus ? tiles / kCus - 1.0 : 0.0;
    const double stages = (double)((g.T * P + 7) / 8), kb = (double)span * P / 64.0;
    return k[0] + k[1] * stages + k[2] * kb + more * (k[3] + k[4] * stages + k[5] * kb);
}

bool window_tile_fits(const icv_conv_params* p, const Geometry& g, int tile, bool any_size)
{
    const int64_t row_bytes = (int64_t)p->C * g.elem_bytes, P = (row_bytes + 15) / 16;
    if (tile < 0 || tile >= kNumWindowTiles || !window_takes(g, row_bytes)) return false;
    const int64_t cap_rows = tile_span_bound(p, g.Hout, g.Wout, kWindowTiles[tile].MR);
    return window_fits_lds(kWindowTiles[tile], g.T, (int)P, cap_rows) && (any_size || cap_rows * P <= kWindowPieces);
}

int launch_igemm_window(const icv_conv_params* p, const Geometry& g, const void* input, const void* packed, const int32_t* ind, void* out,
                        hipStream_t s)
{
    if (g.win_tile < 0 || g.win_tile >= kNumWindowTiles) return ICV_ERR_UNSUPPORTED;
    const WindowTile& t = kWindowTiles[g.win_tile];
    WindowArgs a{};      // every field starts at zero; the ones this call uses are set below
    a.a = (const uint8_t*)input;
    a.w = (const uint8_t*)packed;
    a.out = out;
    if (g.block_entries) a.ent = (const uint16_t*)((const int4*)ind + g.img_tiles);
    else a.ind = ind;
    a.row_bytes = p->C * g.elem_bytes;
    a.stride_bytes = g.in_stride * g.elem_bytes;
    a.image_bytes = g.image_bytes;
    while ((1 << a.block_shift) < g.MR) ++a.block_shift;
    if (a.row_bytes < 16 || (1 << a.block_shift) != g.MR || (g.block_entries ? g.MR != 32 : g.MR % t.MR != 0)) return ICV_ERR_UNSUPPORTED;
    const int64_t images = g.per_image ? p->N : 1, img_tiles = (g.img_rows + t.MR - 1) / t.MR, n_tiles = (p->K + t.NR - 1) / t.NR;
    const int64_t tiles = images * img_tiles * n_tiles;
    if (tiles >= (1ll << 31) - 8 || g.img_tiles >= (1ll << 31)) return ICV_ERR_UNSUPPORTED;
    a.img_tiles = (uint32_t)img_tiles;
    a.img_rows = (uint32_t)g.img_rows;
    a.img_blocks = (uint32_t)g.img_tiles;
    a.total_tiles = (uint32_t)tiles;
    a.tiles_per_xcd = (uint32_t)((tiles + 7) / 8);
    a.col_blocks = (uint32_t)((p->K + 31) / 32);
    // The workgroups of an XCD share its L2: the larger operand is the one they should all read together
    const int64_t filter_bytes = (int64_t)p->K * g.T * a.row_bytes, input_bytes = (int64_t)p->N * p->Hin * p->Win * a.row_bytes;
    a.rows_inner = filter_bytes > input_bytes ? 1 : 0;
    a.inner = (uint32_t)(a.rows_inner ? images * img_tiles : n_tiles);
    a.by_inner = make_fast_div(a.inner);
    a.by_img_tiles = make_fast_div(a.img_tiles);
    a.by_stride = make_fast_div((uint32_t)a.stride_bytes);
    a.q = make_range_geom(p->Hin, p->Win, g.Hout, g.Wout, p->SY, p->SX, p->DY, p->DX, p->PT, p->PL, p->R, p->S);
    a.K = p->K; a.T = g.T; a.out_stride = g.out_stride;
    a.P = (a.row_bytes + 15) / 16;
    a.n_steps = (g.T * a.P + 1) / 2;
    a.tail_shift = a.row_bytes % 16 ? 16 - a.row_bytes % 16 : 0;
    const int64_t cap_rows = tile_span_bound(p, g.Hout, g.Wout, t.MR);
    a.chunk = cap_rows < 65536 ? window_chunk(t, g.T, a.P, cap_rows, tiles) : 0;
    if (a.chunk <= 0) return ICV_ERR_UNSUPPORTED;
    a.cap_rows = (int32_t)cap_rows;
    a.n_chunks = (a.P + a.chunk - 1) / a.chunk;
    a.last_chunk = a.P - (a.n_chunks - 1) * a.chunk;
    a.pitch = a.chunk | 1;
    a.by_chunk = make_fast_div((uint32_t)a.chunk);
    a.by_last_chunk = make_fast_div((uint32_t)a.last_chunk);
    a.ent_at = (a.cap_rows + 1) * a.pitch * 16;
    a.vector_out = a.out_stride % 4 == 0 ? 1 : 0;
    a.zero_fill = p->dtype == ICV_U8I8 ? (0x01010101u * (uint32_t)p->input_zero_point) ^ 0x80808080u : 0u;
    a.ep = g.ep;
    const size_t lds_bytes = window_lds_bytes(t, g.T, cap_rows, a.chunk);
    const int unroll = stage_steps(a.P, a.chunk);
    switch (p->dtype) {
    case ICV_BF16: return launch_window_bf16(a, g.win_tile, unroll, lds_bytes, !g.ep_plain, s);
    case ICV_U8I8: return launch_window_u8(a, g.win_tile, unroll, lds_bytes, !g.ep_plain, s);
    case ICV_F32: return launch_window_f32(a, g.win_tile, unroll, lds_bytes, !g.ep_plain, s);
    }
    return ICV_ERR_UNSUPPORTED;
}

}  // namespace icv
