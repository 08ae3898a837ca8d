// Host side of the any-channel-count kernel: which tile, and the launch.
#include "icv_igemm_any_kernel.h"

namespace icv {

const TileVariant kAnyTiles[] = {
    {128, 128, 1, 4, "128x128"},
    {128, 64, 2, 2, "128x64"},
    {64, 64, 2, 2, "64x64"},
    {128, 32, 4, 1, "128x32"},
    {32, 32, 1, 1, "split"},           // the split-reduction kernel alone
};

// Timed with all three tiles on 2300 drawn problems (7 to 96 pixels a side, batch 1 to 256, 16 to 512 channels, 33 to 1024
// columns, 1x1 to 5x5), the choice is on average 1.4 % (bf16), 1.9 % (uint8) and 0.8 % (fp32) above the best of the three; the
// worst, up to twice it, are 1x1 layers of one stage with more than two rounds of tiles.
int choose_any_tile(int64_t images, int64_t img_rows, int32_t K, int32_t row_bytes, int64_t patch_bytes, int32_t dtype, bool any_batch)
{
    if (row_bytes < 16) return 2;      // rows shorter than a piece: built for this tile only
    if (K <= 32) return 3;
    const bool f32 = dtype == ICV_F32, bf16 = dtype == ICV_BF16, short_patch = patch_bytes < 1000;
    auto tiles = [&](int v) {
        return images * ((img_rows + kAnyTiles[v].MR - 1) / kAnyTiles[v].MR) * ((K + kAnyTiles[v].NR - 1) / kAnyTiles[v].NR);
    };
    // 64 columns also where 128 would leave half of the last column tile empty.  192 columns, 128 x 64 against 128 x 128: 48
    // channels, 128 x 27 x 27: uint8 24.8 against 34.3 us, fp32 134.2 against 168.0, bf16 32.5 against 33.3; 96 channels, 16 x 56 x 56: bf16
    // 28.3 against 32.9.  In bf16 from 256 columns on the rows are read too often (288 columns, 29 x 46 x 30, 24 channels, 5x5: 39.9
    // against 30.3; of 14 drawn problems with 600 tiles or more 9 lose 3 to 16 %, 3 gain over 5), except where 128 x 128 is just past two per
    // compute unit (543 to 579 tiles: 0.87).  (A batch-independent layout has 128 columns there, and the kernel may run with 64.)
    bool half = K > 64 && K < 512 && K % 128 != 0 && K % 128 <= 64;
    if (bf16 && K >= 256) half = half && !any_batch && tiles(0) > 2 * 256 && tiles(0) < 600;
    const int wide = K <= 64 || half ? 1 : 0;
    if (any_batch) return wide;
    // 64 x 64 when the wider tile leaves most of the chip with a single workgroup or none: two and more per compute
    // unit are what hides this kernel's latencies.  fp32, bound by the matrix cores, wants two everywhere.  Measured with 128 x 128
    // against 64 x 64, bf16 (uint8): 392 tiles, 192 channels, 3x3: 30.9 against 44.5 us (20.5 against 25.5); 400 tiles, 384 channels: 58.2
    // against 88.0 (35.3 against 46.1); 294 tiles, 320 channels, 5x5: 117.9 against 117.3 (72.8 against 58.6); 281 tiles: 35.5
    // against 38.4 (27.4 against 23.6).  fp32, 392 tiles: 218.9 against 210.3; uint8, 344
    // tiles of a reduction of only 496: 16.2 against 12.9; fp32, 549 tiles of 128 x 64: 257.5 against 221.8.
    // In bf16 128 x 64 where a compute unit gets two of them at most but would get a fourth of 64 x 64: 42 of the drawn problems, 0.82
    // to 1.00 of the time of the other choice but for two (1.04, 1.07).
    if (bf16 && !short_patch && tiles(2) > 3 * 256 && tiles(1) <= 2 * 256) return 1;
    // (128 x 128 where it would get a fifth, 264 to 296 tiles: 0.87 to 0.99 with plain output, 0.93 to 1.14 with the fused one; not kept)
    int64_t fill;
    if (f32) fill = half ? 1024 : 512;
    else if (wide) fill = short_patch || K <= 64 || bf16 ? 512 : 336;
    else fill = patch_bytes < 600 ? 512 : (short_patch ? 400 : 336);      // (600 to 1000 bytes, 404 to 492 tiles: 0.70 to 0.97, twice 1.1)
    return tiles(wide) >= fill ? wide : 2;
}

int64_t any_packed_bytes(const Geometry& g, int32_t row_bytes)
{
    const int64_t P = (row_bytes + 15) / 16;
    return g.n_tiles * (g.NR / 32) * ((g.T * P + 1) / 2) * 1024;
}

int launch_igemm_any(const icv_conv_params* p, const Geometry& g, const void* input, const void* packed,
                     const int32_t* ind, const void* zero_row, void* out, int a_mode, hipStream_t s)
{
    AnyArgs a{};      // every field starts at zero; the ones this call uses are set below
    a.a = (const uint8_t*)input;
    a.zero_row = (const uint8_t*)zero_row;
    a.w = (const uint8_t*)packed;
    a.ind = a_mode == A_GATHERED ? ind : nullptr;
    a.out = out;
    a.row_bytes = p->C * g.elem_bytes;
    a.a_row_stride = a_mode == A_DENSE_WORKSPACE ? (int64_t)g.T * a.row_bytes : (int64_t)g.in_stride * g.elem_bytes;
    a.a_rows = a_mode == A_DENSE_WORKSPACE ? patch_matrix_rows(g) : g.M;
    a.image_bytes = a_mode == A_GATHERED ? g.image_bytes : 0;
    const TileVariant& tv = kAnyTiles[g.run_variant];
    if (a_mode == A_GATHERED && g.MR % tv.MR != 0) return ICV_ERR_UNSUPPORTED;
    while ((1 << a.block_shift) < g.MR) ++a.block_shift;
    const int64_t images = g.per_image ? p->N : 1, img_tiles = (g.img_rows + tv.MR - 1) / tv.MR, n_tiles = (p->K + tv.NR - 1) / tv.NR;
    const int64_t tiles = images * img_tiles * n_tiles;
    a.img_tiles = (uint32_t)img_tiles;
    a.img_rows = (uint32_t)g.img_rows;
    if (n_tiles * tv.NR > g.n_tiles * g.NR) return ICV_ERR_UNSUPPORTED;       // the packed filter has no more column blocks
    if (tiles >= (1ll << 31) - 8) return ICV_ERR_UNSUPPORTED;
    a.total_tiles = (uint32_t)tiles;
    a.tiles_per_xcd = (uint32_t)((tiles + 7) / 8);
    a.n_tiles = (uint32_t)n_tiles;
    a.by_n_tiles = make_fast_div(a.n_tiles);
    a.by_img_tiles = make_fast_div(a.img_tiles);
    a.K = p->K; a.T = g.T; a.out_stride = g.out_stride;
    a.P = (a.row_bytes + 15) / 16;
    a.n_pieces = g.T * a.P;
    a.step_taps = 8 / a.P;
    a.step_pieces = 8 % a.P;
    a.n_steps = (a.n_pieces + 1) / 2;
    a.n_stages = (a.n_steps + 3) / 4;
    const int tail = a.row_bytes % 16 == 0 ? ROWS_WHOLE : (a.row_bytes > 16 ? ROWS_TAIL : ROWS_SHORT);
    a.tail_shift = tail == ROWS_TAIL ? 16 - a.row_bytes % 16 : 0;
    a.ep = g.ep;
    switch (p->dtype) {
    case ICV_BF16: return launch_any_bf16(a, g.run_variant, tail, !g.ep_plain, s);
    case ICV_U8I8: return launch_any_u8(a, g.run_variant, tail, !g.ep_plain, s);
    case ICV_F32: return launch_any_f32(a, g.run_variant, tail, !g.ep_plain, s);
    }
    return ICV_ERR_UNSUPPORTED;
}

}  // namespace icv
