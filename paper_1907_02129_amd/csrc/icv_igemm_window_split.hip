// Tensor-core Indirect GEMM for few output pixels and long reductions (7 x 7 to 28 x 28 maps of wide layers at small and
// medium batches): a tile's input window in LDS, its reduction split over the wavefronts of a workgroup.
//
// Such a layer gives every compute unit one 64 x 64 tile or none, and the pixel-range kernel then multiplies its hundred
// stages one after the other, a barrier each, with one multiplying wavefront per SIMD: 0.22 us per 128 bytes of
// reduction where the matrix cores need 0.05.  Here
//
//  * the window -- the tile's range of consecutive input pixels, whole rows -- and the tile's 16-bit entries are copied to
//    LDS at once; a single barrier follows.  The R*S kernel elements re-use the window as in the pixel-range kernel;
//  * each of eight wavefronts takes a contiguous run of the reduction's 128-byte stages for the whole tile: two wavefronts
//    per SIMD that hide each other's LDS reads, and no barrier until the partial tiles are summed;
//  * the filter comes from global memory in operand order, two stages ahead, and never enters LDS: a compute unit reads
//    its 64 columns once (590 KB for 512 channels, 3x3: 4.4 us of L1).
// That and the products (4.4 us) start when the whole window is there: 32 maps of 7 x 7, 512 to 512 channels take 14.3 us with
// L1 and the matrix cores busy 47 and 30 % of it.
//
// LDS rows are padded by a piece, which spreads the fragment reads of neighbouring rows over the banks.
#include "icv_mfma_common.h"
#include "icv_pixel_range.h"

namespace icv {

struct WindowSplitArgs {
    const uint8_t* a;          // input tensor
    const uint8_t* w;          // packed filter [32-column block][MFMA step][lane][16 bytes]
    const int4* ranges;        // per row tile {first byte offset, pixels}
    const uint16_t* rows;      // [row tile][kernel element][64]: pixel number in the range, cap_rows = the zero row
    void* out;
    uint32_t M;
    uint32_t total_tiles, tiles_per_xcd, inner;
    FastDiv by_inner;
    uint32_t rows_inner;       // 1: row tiles run fastest (the filter is the larger operand), 0: column tiles
    int32_t K, T, out_stride;
    int32_t stride_bytes;      // bytes between input pixels
    int32_t pieces;            // 16-byte pieces of an LDS row: the pixel's and one of padding
    FastDiv by_pieces;
    int32_t cap_rows;          // pixel rows reserved in LDS; the zero row follows them
    int32_t chunks;            // stages per kernel element: row bytes / 128
    FastDiv by_chunks;
    int32_t n_stages;
    int32_t ent_at;            // LDS offset of the entries
    int32_t vector_out;        // 1: four neighbouring outputs may be stored at once
    uint32_t zero_fill;        // four bytes of the zero row: zeros, or the zero point of uint8 activations
    EpilogueArgs ep;
};

constexpr int kWindowWaves = 8;

template <int DT>
__global__ __launch_bounds__(64 * kWindowWaves) void k_igemm_window_split(WindowSplitArgs g)
{
    constexpr bool I8 = DT == ICV_U8I8;
    constexpr int D = 2;                         // stages of filter in flight
    using acc_t = typename Acc<I8>::type;
    using out_acc_t = typename std::conditional<I8, int32_t, float>::type;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t tile = (blockIdx.x & 7u) * g.tiles_per_xcd + (blockIdx.x >> 3);
    if (tile >= g.total_tiles) return;           // the whole workgroup, before any barrier
    const uint32_t outer = fast_div(tile, g.by_inner), in = tile - outer * g.inner;
    const uint32_t mt = g.rows_inner ? in : outer, nt = g.rows_inner ? outer : in;
    const int pitch = g.pieces * 16;

    // ---- this wavefront's stages and the first of their filter fragments
    const int share = g.n_stages / kWindowWaves, extra = g.n_stages - share * kWindowWaves;
    const int s0 = wave * share + (wave < extra ? wave : extra);
    const int n = share + (wave < extra ? 1 : 0);

    // ---- window and entries -> LDS, every wavefront its 1 KB pieces
    {
        const int ent_bytes = g.T * 128;
        const uint16_t* const src = g.rows + (int64_t)mt * g.T * 64;
        for (int u = wave; u * 1024 < ent_bytes; u += kWindowWaves) {
            int o = u * 1024 + lane * 16;
            if (o > ent_bytes - 16) o = ent_bytes - 16;       // (the LDS reserved for them is whole KB)
            copy16_global_to_lds(src, (uint32_t)o, (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + g.ent_at + u * 1024)));
        }
        const int4 range = g.ranges[mt];
        const uint8_t* const first = g.a + __builtin_amdgcn_readfirstlane(range.x);
        int count = __builtin_amdgcn_readfirstlane(range.y);
        if (count > g.cap_rows) count = g.cap_rows;
        const uint32_t total = (uint32_t)count * (uint32_t)g.pieces;
        for (uint32_t u = wave; u * 64u < total; u += kWindowWaves) {
            uint32_t at = u * 64u + lane;
            if (at > total - 1) at = total - 1;                // (lands in the rows behind the last, which nothing reads)
            const uint32_t row = fast_div(at, g.by_pieces);
            uint32_t piece = at - row * (uint32_t)g.pieces;
            if (piece > (uint32_t)g.pieces - 2u) piece = (uint32_t)g.pieces - 2u;      // the padding repeats the last one
            copy16_global_to_lds(first, row * (uint32_t)g.stride_bytes + piece * 16u,
                                 (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + u * 1024)));
        }
    }
    const uint8_t* const wp = g.w + (int64_t)(nt * 2) * g.n_stages * 4096 + lane * 16;
    uint4 b[D][4][2];
    auto read_filter = [&](int d, int stage, bool used) __attribute__((always_inline)) {
        const uint8_t* p = wp + (int64_t)(used ? stage : 0) * 4096;
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
#pragma unroll
            for (int j = 0; j < 2; j++) b[d][ks][j] = *(const uint4*)(p + (int64_t)j * g.n_stages * 4096 + ks * 1024);
    };
#pragma unroll
    for (int d = 0; d < D; d++) read_filter(d, s0 + d, d < n);
    wait_vmcnt<0>();
    __syncthreads();
    // the zero row last: a copy's surplus lanes may have written there
    for (int i = tid; i < pitch / 4; i += 64 * kWindowWaves) *(uint32_t*)(lds + g.cap_rows * pitch + i * 4) = g.zero_fill;
    __syncthreads();

    acc_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[i][j][r] = 0;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const uint16_t* const ent = (const uint16_t*)(lds + g.ent_at) + lrow;
    int tap = (int)fast_div((uint32_t)s0, g.by_chunks), chunk = s0 - tap * g.chunks;
    if (tap > g.T - 1) tap = g.T - 1;            // (a wavefront without a stage)
    // stages past the last: the walk stops at the last kernel element, whose entries are there
    auto locate = [&](uint32_t (&at)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; i++) at[i] = (uint32_t)ent[tap * 64 + i * 32] * (uint32_t)pitch + (uint32_t)(chunk * 128 + lhalf * 16);
        if (++chunk == g.chunks) { chunk = 0; if (tap < g.T - 1) ++tap; }
    };
    uint32_t at[D][2];
#pragma unroll
    for (int d = 0; d < D; d++) locate(at[d]);
    for (int s = 0; s < n; s += D) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            if (s + d < n) {
#pragma unroll
                for (int ks = 0; ks < 4; ks++) {
                    uint4 af[2];
#pragma unroll
                    for (int i = 0; i < 2; i++) af[i] = *(const uint4*)(lds + at[d][i] + ks * 32);
#pragma unroll
                    for (int i = 0; i < 2; i++)
#pragma unroll
                        for (int j = 0; j < 2; j++) {
                            if constexpr (DT == ICV_F32) acc[i][j] = mfma32_f32(af[i], b[d][ks][j], acc[i][j]);
                            else acc[i][j] = mfma32<I8>(af[i], b[d][ks][j], acc[i][j]);
                        }
                }
            }
            __builtin_amdgcn_sched_barrier(0);                    // (registers: no load before its slot is free)
            locate(at[d]);
            read_filter(d, s0 + s + d + D, s + d + D < n);        // unconditional: the waits leave the younger loads in flight
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- sum the partial tiles, 32 rows at a time, in the window's place
    typedef typename FourOutputs<I8>::vec_t out4_t;
#pragma unroll
    for (int i = 0; i < 2; i++) {
        __syncthreads();                         // the window has been read; the sums of the rows before have been taken
        out_acc_t* part = (out_acc_t*)(lds + wave * 8192);       // [32][64]
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) part[(8 * (r >> 2) + 4 * lhalf + (r & 3)) * 64 + j * 32 + lrow] = acc[i][j][r];
        __syncthreads();
        const int v = tid;                       // 512 threads, 512 groups of four columns
        out4_t sum = *(const out4_t*)(lds + v * 16);
#pragma unroll
        for (int w = 1; w < kWindowWaves; w++) sum += *(const out4_t*)(lds + w * 8192 + v * 16);
        const int64_t row = (int64_t)mt * 64 + i * 32 + (v >> 4);
        const int32_t col = (int32_t)nt * 64 + (v & 15) * 4;
        if (row < (int64_t)g.M) store_four<I8>(g.out, row * g.out_stride + col, sum, col, g.K, g.vector_out, g.ep);
    }
}

// LDS: window rows and the zero row, at least what the partial tiles need; then the entries
static int64_t window_bytes(int64_t row_bytes, int64_t cap_rows)
{
    // whole KB: the last copy of the window may write to the end of its KB
    const int64_t w = ((cap_rows + 1) * (row_bytes + 16) + 1023) / 1024 * 1024 + 1024;
    return w > kWindowWaves * 8192 ? w : kWindowWaves * 8192;
}

size_t window_split_lds_bytes(int T, int64_t row_bytes, int64_t cap_rows)
{
    return (size_t)(window_bytes(row_bytes, cap_rows) + (T * 128 + 1023) / 1024 * 1024);
}

template <int DT>
static int launch_window(const WindowSplitArgs& a, size_t lds_bytes, hipStream_t s)
{
    auto kern = k_igemm_window_split<DT>;
    static bool raised[kMaxDevices] = {};      // one array per instantiation of this function template
    const int st = allow_full_lds((const void*)kern, raised);
    if (st != ICV_OK) return st;
    hipLaunchKernelGGL(kern, dim3(8u * a.tiles_per_xcd), dim3(64 * kWindowWaves), lds_bytes, s, a);
    ICV_HIP_CHECK(hipGetLastError());
    return ICV_OK;
}

int launch_igemm_window_split(const icv_conv_params* p, const Geometry& g, const void* input, const void* packed,
                              const int32_t* ind, void* out, hipStream_t s)
{
    const int64_t row_bytes = (int64_t)p->C * g.elem_bytes;
    if (g.MR != 64 || g.NR != 64 || row_bytes % 128 != 0 || g.patch_rows < 1 || g.zero_row_number != (uint32_t)g.patch_rows)
        return ICV_ERR_UNSUPPORTED;
    const size_t lds_bytes = window_split_lds_bytes(g.T, row_bytes, g.patch_rows);
    if (lds_bytes > kLdsPerCu || g.per_image) return ICV_ERR_UNSUPPORTED;
    WindowSplitArgs a{};      // every field starts at zero; the ones this call uses are set below
    a.a = (const uint8_t*)input;
    a.w = (const uint8_t*)packed;
    a.ranges = (const int4*)ind;
    a.rows = (const uint16_t*)(a.ranges + g.img_tiles);
    a.out = out;
    a.M = (uint32_t)g.M;
    const int64_t tiles = g.m_tiles * g.n_tiles;
    if (tiles >= (1ll << 31) - 8) return ICV_ERR_UNSUPPORTED;
    a.total_tiles = (uint32_t)tiles;
    a.tiles_per_xcd = (uint32_t)((tiles + 7) / 8);
    // The workgroups of an XCD share its L2: the larger operand is the one they should all read together
    a.rows_inner = (int64_t)p->K * g.T * row_bytes > (int64_t)p->N * p->Hin * p->Win * row_bytes ? 1 : 0;
    a.inner = (uint32_t)(a.rows_inner ? g.m_tiles : g.n_tiles);
    a.by_inner = make_fast_div(a.inner);
    a.K = p->K; a.T = g.T; a.out_stride = g.out_stride;
    a.stride_bytes = g.in_stride * g.elem_bytes;
    a.pieces = (int32_t)(row_bytes / 16) + 1;
    a.by_pieces = make_fast_div((uint32_t)a.pieces);
    a.cap_rows = g.patch_rows;
    a.chunks = (int32_t)(row_bytes / 128);
    a.by_chunks = make_fast_div((uint32_t)a.chunks);
    a.n_stages = g.T * a.chunks;
    a.ent_at = (int32_t)window_bytes(row_bytes, g.patch_rows);
    a.vector_out = a.out_stride % 4 == 0 ? 1 : 0;
    a.zero_fill = p->dtype == ICV_U8I8 ? 0x01010101u * (uint32_t)p->input_zero_point : 0u;
    a.ep = g.ep;
    switch (p->dtype) {
    case ICV_BF16: return launch_window<ICV_BF16>(a, lds_bytes, s);
    case ICV_U8I8: return launch_window<ICV_U8I8>(a, lds_bytes, s);
    case ICV_F32: return launch_window<ICV_F32>(a, lds_bytes, s);
    }
    return ICV_ERR_UNSUPPORTED;
}

}  // namespace icv
