// Tensor-core Indirect GEMM for channel counts of any size: the pixel rows need no alignment and no round length.
//
// The kernels that copy rows straight into LDS move whole aligned 16-byte pieces and split rows into 64-byte stages; a
// row of 96 bytes (48 bfloat16 channels) or of 74 (37 of them) does not fit that.  Here a row is P = ceil(row / 16)
// pieces of 16 bytes, the last one padded with zeros, and the two nested loops of Listing 3 become one walk over the
// T*P pieces of an output pixel's patch, eight pieces (128 bytes, four MFMA steps) per stage:
//
//  * A goes through registers, where alignment and padding are free: a thread owns one piece column of the stage and
//    MR/32 rows, loads its 16 bytes from wherever the entry points (the hardware takes any address), shifts the last
//    piece of a row into place -- it is read as the row's LAST 16 bytes, so nothing beyond the row is ever touched --
//    and writes it to one of two LDS buffers.  The rows of stage s + 1 and the entries of stage s + 2 are in flight
//    while stage s is multiplied; one barrier per stage.
//  * B comes from global memory in operand order (the packed layout of the filter-in-registers kernel), one coalesced
//    1 KB read per fragment and wavefront, one stage ahead.  It never touches LDS: a B fragment serves four MFMAs with
//    128 x 128 tiles (32 bytes per clock of the 64 that L1 gives), two with 128 x 64, one with 64 x 64.
//
// Measured (one launch): 48 bfloat16 channels, 128 images of 27 x 27, 192 output channels, 3x3: 30.6 us, 506 TFLOP/s (128 x 64
// tiles; 33.3 with 128 x 128), where the vector ALUs took 2344 us; 416 uint8 channels, 2 x 78 x 78, 120 output channels:
// 19.3 us, 565 TOP/s.  What bounds the first is L1: per stage a workgroup brings 16 KB of rows and 16 KB of filter through
// it, the counters show 0.91 accesses a busy cycle (MFMA 24 % busy, LDS 24 %, no conflicts).  Both now run on the window kernel
// (icv_igemm_window_kernel.h: 25.4 and 15.8 us), which reads these buffers; what stays here are pointwise and other kernels of less
// than four elements, fp32, rows of one to three pieces, windows too large for LDS, and the patch-matrix product.
//
// Small workgroups (36 KB of LDS, four wavefronts, no persistence): two to four share a compute unit and hide each
// other's barriers, first loads and stores.  A block of entries may have more rows than the tile (the one-image buffer, laid
// out for the tile of a large batch, serves small ones with smaller tiles).
//
// uint8 activations: every A fragment is XORed with 0x80 (x -> x - 128 as a signed byte); the zero row holds the zero
// point; the filter is zero wherever a piece is padding.
#pragma once
#include "icv_mfma_common.h"
#include "icv_pixel_range.h"

namespace icv {

struct AnyArgs {
    const uint8_t* a;          // input tensor | patch matrix
    const uint8_t* zero_row;
    const uint8_t* w;          // packed filter [32-column block][MFMA step][lane][16 bytes]
    const int32_t* ind;        // [block][kernel element][block rows] byte offsets, negative = zero row; null: dense A
    void* out;
    int64_t a_row_stride;      // dense A: bytes between rows
    int64_t a_rows;            // dense A: rows that may be read (later ones re-read the last)
    int64_t image_bytes;       // batch-independent buffer: bytes between batch elements of the input (else 0)
    uint32_t img_tiles, img_rows;   // row tiles and output pixels per image (one image = the whole batch otherwise)
    uint32_t block_shift;      // log2 of the rows of a block of entries, no fewer than a tile's
    FastDiv by_n_tiles, by_img_tiles;
    uint32_t total_tiles, tiles_per_xcd, n_tiles;
    int32_t K, T, out_stride;
    int32_t row_bytes;         // C * element size
    int32_t P;                 // pieces per row
    int32_t n_pieces;          // T * P
    int32_t step_taps, step_pieces;   // 8 / P, 8 % P
    int32_t n_steps, n_stages; // MFMA steps of two pieces, stages of four steps
    int32_t tail_shift;        // bytes by which a row's last piece, read as the row's last 16 bytes, is shifted down
    EpilogueArgs ep;
};

__device__ inline bytes16_t load16_any(const uint8_t* p)      // 16 bytes from any address
{
    bytes16_t v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// length of a pixel row: whole pieces; a padded last piece; shorter than a piece
enum AnyTail : int { ROWS_WHOLE = 0, ROWS_TAIL = 1, ROWS_SHORT = 2 };

// WM x WN wavefronts
template <int DT, int MR, int NR, int WM, int WN, int TAIL, bool DENSE, bool FUSED>
__global__ __launch_bounds__(256, 2) void k_igemm_any(AnyArgs g)
{
    constexpr bool I8 = DT == ICV_U8I8;
    constexpr int MRW = MR / WM, MB = MRW / 32, NB = NR / WN / 32;
    constexpr int RPT = MR / 32;                 // rows per thread
    constexpr int PITCH = 144;                   // eight pieces and one of padding: fragment reads spread over the banks
    static_assert(WM * WN == 4 && MB >= 1 && NB >= 1, "four wavefronts");
    using acc_t = typename Acc<I8>::type;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * MR * PITCH];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    // XCD x (workgroups x, x + 8, ...) takes a contiguous run of tiles, column tiles innermost: neighbours share rows
    // and filter in its L2
    const uint32_t tile = (blockIdx.x & 7u) * g.tiles_per_xcd + (blockIdx.x >> 3);
    if (tile >= g.total_tiles) return;           // the whole workgroup, before any barrier
    const uint32_t mt = fast_div(tile, g.by_n_tiles), nt = tile - mt * g.n_tiles;
    const uint32_t img = fast_div(mt, g.by_img_tiles), t_img = mt - img * g.img_tiles;

    // ---- A: this thread's piece column and rows
    const int q = tid & 7, r0 = tid >> 3;
    const uint8_t* const a_img = g.a + (int64_t)img * g.image_bytes;
    const uint32_t row_img = t_img * MR, blk = row_img >> g.block_shift;
    // (uniform; a 64-bit address per lane costs the registers that keep four wavefronts of the 128 x 128 tile on a SIMD)
    const int32_t* const ent = DENSE ? nullptr : g.ind + (((int64_t)blk * g.T) << g.block_shift) + (row_img - (blk << g.block_shift));
    const uint8_t* base[RPT];                    // what the entries count from (dense A: the row)
#pragma unroll
    for (int i = 0; i < RPT; i++) {
        base[i] = a_img;
        if constexpr (DENSE) {
            int64_t m = (int64_t)img * g.img_rows + (int64_t)t_img * MR + r0 + 32 * i;
            if (m > g.a_rows - 1) m = g.a_rows - 1;
            base[i] = g.a + m * g.a_row_stride;
        }
    }
    // walk over the pieces q, q + 8, ...: kernel element and piece of its row
    int tap = q / g.P, piece = q - tap * g.P;
    auto advance = [&]() {
        tap += g.step_taps;
        piece += g.step_pieces;
        if (piece >= g.P) { piece -= g.P; ++tap; }
    };
    int32_t e[RPT];
    int e_tap = 0, e_piece = 0;                  // what e was read for (pieces past the last: tap >= T)
    auto read_entries = [&]() {
        e_tap = tap; e_piece = piece;
        const int t = tap < g.T ? tap : g.T - 1;
        if constexpr (DENSE) {
#pragma unroll
            for (int i = 0; i < RPT; i++) e[i] = t * g.row_bytes;
        } else {
            const uint32_t at = ((uint32_t)t << g.block_shift) + (uint32_t)r0;
#pragma unroll
            for (int i = 0; i < RPT; i++) e[i] = *(const int32_t*)((const uint8_t*)ent + at * 4u + 128 * i);
        }
        advance();
    };
    bytes16_t av[RPT];
    bool v_past = false, v_last = false;         // the pieces in av lie past the patch; are the last of their row
    auto read_rows = [&]() {
        v_past = e_tap >= g.T;
        v_last = TAIL == ROWS_TAIL && e_piece == g.P - 1;
        int o = e_piece * 16;
        if (TAIL == ROWS_TAIL && o > g.row_bytes - 16) o = g.row_bytes - 16;
#pragma unroll
        for (int i = 0; i < RPT; i++) {
            const uint8_t* src = e[i] < 0 ? g.zero_row : base[i] + (uint32_t)e[i];
            if constexpr (TAIL == ROWS_SHORT) {
                // byte by byte: nothing beyond the row may be read
                bytes16_t v = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int b = 0; b < 15; b++) {
                    const uint32_t x = src[b < g.row_bytes ? b : 0];
                    v[b >> 2] |= (b < g.row_bytes ? x : 0u) << (8 * (b & 3));
                }
                av[i] = v;
            } else {
                av[i] = load16_any(src + o);
            }
        }
    };
    auto to_lds = [&](int buf) {
        uint8_t* d = lds + buf * (MR * PITCH) + r0 * PITCH + q * 16;
#pragma unroll
        for (int i = 0; i < RPT; i++) {
            bytes16_t v = av[i];
            if constexpr (TAIL == ROWS_TAIL) {
                const bytes16_t s = shift_down(v, g.tail_shift);
                v = v_last ? s : v;
            }
            if (v_past) v = bytes16_t{0u, 0u, 0u, 0u};
            *(bytes16_t*)(d + i * 32 * PITCH) = v;
        }
    };

    // ---- B: this wavefront's column blocks
    const int wm = wave / WN, wn = wave % WN;
    const uint8_t* wp[NB];
#pragma unroll
    for (int j = 0; j < NB; j++)
        wp[j] = g.w + ((int64_t)(nt * (NR / 32) + wn * NB + j) * g.n_steps) * 1024 + lane * 16;
    uint4 b[4][NB];
    auto read_filter = [&](int stage, int ks) __attribute__((always_inline)) {
        int f = stage * 4 + ks;
        if (f > g.n_steps - 1) f = g.n_steps - 1;
#pragma unroll
        for (int j = 0; j < NB; j++) b[ks][j] = *(const uint4*)(wp[j] + (int64_t)f * 1024);
    };

    acc_t acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; i++)
#pragma unroll
        for (int j = 0; j < NB; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[i][j][r] = 0;

    const uint32_t frag = (uint32_t)(wm * MRW + lrow) * PITCH + lhalf * 16;
    auto multiply = [&](const uint8_t* A, int ks) __attribute__((always_inline)) {
        uint4 af[MB];
#pragma unroll
        for (int i = 0; i < MB; i++) af[i] = *(const uint4*)(A + i * 32 * PITCH + ks * 32);
#pragma unroll
        for (int i = 0; i < MB; i++)
#pragma unroll
            for (int j = 0; j < NB; j++) {
                if constexpr (DT == ICV_F32) acc[i][j] = mfma32_f32(af[i], b[ks][j], acc[i][j]);
                else acc[i][j] = mfma32<I8>(af[i], b[ks][j], acc[i][j]);
            }
    };
    // Three copies of the stage -- with everything that follows in flight, the last but one, the last -- so that no
    // load is conditional: a wait behind a conditional load would have to assume that it was not issued.
    auto run_stage = [&](int s, auto more_rows, auto more_entries) __attribute__((always_inline)) {
        constexpr bool ROWS = decltype(more_rows)::value, ENTRIES = decltype(more_entries)::value;
        to_lds(s & 1);
        if constexpr (ROWS) read_rows();
        if constexpr (ENTRIES) read_entries();
        // LDS only: the loads of the next stage stay in flight.  One barrier per stage is enough: a buffer is written
        // again two stages later, after the barrier that every wavefront reaches with its reads of it done.
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint8_t* A = lds + (s & 1) * (MR * PITCH) + frag;
        const int steps = g.n_steps - s * 4;                  // at least four unless this is the last stage
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
            if (ROWS || ks < steps) {
                multiply(A, ks);
                if constexpr (ROWS) read_filter(s + 1, ks);
            }
    };
    // (in the order in which the loop issues them, unconditionally, so that the loop's waits can be exact)
    read_entries();
    read_rows();
    read_entries();
#pragma unroll
    for (int ks = 0; ks < 4; ks++) read_filter(0, ks);
    int s = 0;
    for (; s + 2 < g.n_stages; s++) run_stage(s, std::true_type(), std::true_type());
    if (s + 1 < g.n_stages) run_stage(s++, std::true_type(), std::false_type());
    run_stage(s, std::false_type(), std::false_type());

    const int64_t img_row0 = (int64_t)img * g.img_rows;
    const int64_t m_base = img_row0 + (int64_t)t_img * MR + wm * MRW + 4 * lhalf;
    const int32_t n_base = (int32_t)nt * NR + wn * (NB * 32) + lrow;
    const bool whole_rows = (t_img + 1) * MR <= g.img_rows, whole = whole_rows && (int32_t)(nt + 1) * NR <= g.K;
    store_tile<FUSED, I8, MB, NB>(g.out, acc, img_row0 + g.img_rows, g.K, g.out_stride, m_base, n_base, whole, whole_rows, g.ep);
}

// Every instantiation of one dtype: one translation unit each, so that they compile side by side.
template <int DT, int MR, int NR, int WM, int WN, int TAIL>
static int launch_any_tile(const AnyArgs& a, bool fused, hipStream_t s)
{
    const dim3 grid(8u * a.tiles_per_xcd);
    const bool dense = a.ind == nullptr;
    if (dense && fused) hipLaunchKernelGGL((k_igemm_any<DT, MR, NR, WM, WN, TAIL, true, true>), grid, dim3(256), 0, s, a);
    else if (dense) hipLaunchKernelGGL((k_igemm_any<DT, MR, NR, WM, WN, TAIL, true, false>), grid, dim3(256), 0, s, a);
    else if (fused) hipLaunchKernelGGL((k_igemm_any<DT, MR, NR, WM, WN, TAIL, false, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_igemm_any<DT, MR, NR, WM, WN, TAIL, false, false>), grid, dim3(256), 0, s, a);
    ICV_HIP_CHECK(hipGetLastError());
    return ICV_OK;
}

template <int DT>
static int launch_any_instances(const AnyArgs& a, int variant, int tail, bool fused, hipStream_t s)
{
#define ICV_ANY_CASE(V, MR, NR, WM, WN, TAIL) \
    if (variant == V && tail == TAIL) return launch_any_tile<DT, MR, NR, WM, WN, TAIL>(a, fused, s);
    ICV_ANY_CASE(0, 128, 128, 1, 4, ROWS_WHOLE)
    ICV_ANY_CASE(0, 128, 128, 1, 4, ROWS_TAIL)
    ICV_ANY_CASE(1, 128, 64, 2, 2, ROWS_WHOLE)
    ICV_ANY_CASE(1, 128, 64, 2, 2, ROWS_TAIL)
    ICV_ANY_CASE(2, 64, 64, 2, 2, ROWS_WHOLE)
    ICV_ANY_CASE(2, 64, 64, 2, 2, ROWS_TAIL)
    ICV_ANY_CASE(2, 64, 64, 2, 2, ROWS_SHORT)
    ICV_ANY_CASE(3, 128, 32, 4, 1, ROWS_WHOLE)
    ICV_ANY_CASE(3, 128, 32, 4, 1, ROWS_TAIL)
#undef ICV_ANY_CASE
    return ICV_ERR_UNSUPPORTED;
}

int launch_any_bf16(const AnyArgs& a, int variant, int tail, bool fused, hipStream_t s);
int launch_any_u8(const AnyArgs& a, int variant, int tail, bool fused, hipStream_t s);
int launch_any_f32(const AnyArgs& a, int variant, int tail, bool fused, hipStream_t s);

}  // namespace icv
