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

int choose_any_tile(int64_t M, int32_t K, int32_t row_bytes, int64_t patch_bytes, int32_t dtype, bool any_batch)
{
    if (row_bytes < 16) return 2;      // rows shorter than a piece: built for this tile only
    if (K <= 32) return 3;
    const bool f32 = dtype == ICV_F32;
    // 64 columns also where 128 would leave half of the last column tile empty.  192 columns, 128 x 64 against 128 x 128: 48
    // channels, 128 x 27 x 27: uint8 24.8 against 34.3 us, fp32 134.2 against 168.0, bf16 32.5 against 33.3; 96 channels, 16 x 56 x 56: bf16
    // 28.3 against 32.9.  In bf16 not for patches over 4 KB (100 channels, 5x5: 52.4 against 51.6) nor, at any batch, past 256
    // columns (320: 44.7 against 40.2), where the rows are read too often.
    bool half = K > 64 && K < 512 && K % 128 != 0 && K % 128 <= 64;
    if (dtype == ICV_BF16) half = half && (K < 256 ? patch_bytes < 4096 : !any_batch);
    const int wide = K <= 64 || half ? 1 : 0;
    // 64 x 64 when the wider tile leaves most of the chip with a single workgroup or none: two and more per compute
    // unit are what hides this kernel's latencies.  fp32, bound by the matrix cores, wants two everywhere.  Measured with 128 x 128
    // against 64 x 64, bf16 (uint8): 392 tiles, 192 channels, 3x3: 30.9 against 44.5 us (20.5 against 25.5); 400 tiles, 384 channels: 58.2
    // against 88.0 (35.3 against 46.1); 294 tiles, 320 channels, 5x5: 117.9 against 117.3 (72.8 against 58.6); 281 tiles: 35.5
    // against 38.4 (27.4 against 23.6).  fp32, 392 tiles: 218.9 against 210.3; uint8, 344
    // tiles of a reduction of only 496: 16.2 against 12.9; fp32, 549 tiles of 128 x 64: 257.5 against 221.8.  A batch-independent buffer's layout must not depend on N.
    const int64_t tiles = ((M + 127) / 128) * ((K + kAnyTiles[wide].NR - 1) / kAnyTiles[wide].NR);
    return any_batch || tiles >= (f32 && half ? 1024 : (f32 || K <= 64 || patch_bytes < 1000 ? 512 : 336)) ? wide : 2;
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
    a.img_tiles = (uint32_t)g.img_tiles;
    a.img_rows = (uint32_t)g.img_rows;
    const int64_t tiles = g.m_tiles * g.n_tiles;
    if (tiles >= (1ll << 31) - 8) return ICV_ERR_UNSUPPORTED;
    a.total_tiles = (uint32_t)tiles;
    a.tiles_per_xcd = (uint32_t)((tiles + 7) / 8);
    a.n_tiles = (uint32_t)g.n_tiles;
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
    const TileVariant& tv = kAnyTiles[g.variant];
    if (tv.MR != g.MR || tv.NR != g.NR) return ICV_ERR_UNSUPPORTED;
    switch (p->dtype) {
    case ICV_BF16: return launch_any_bf16(a, g.variant, tail, !g.ep_plain, s);
    case ICV_U8I8: return launch_any_u8(a, g.variant, tail, !g.ep_plain, s);
    case ICV_F32: return launch_any_f32(a, g.variant, tail, !g.ep_plain, s);
    }
    return ICV_ERR_UNSUPPORTED;
}

}  // namespace icv
