// Tensor-core Indirect GEMM with a tile's input window in LDS and the filter straight from memory: rows of any length from 16
// bytes on, whose kernel elements re-read the same input pixels.
//
// The gathering kernels bring a row to the compute unit once per kernel element, 9 to 25 times: on 48 channels, 3x3, L1 was busy 91 % of
// their time.  Here
//
//  * the valid entries of a tile's output pixels name one short range of input pixels (icv_pixel_range.h, known before anything is
//    read).  Its rows -- as many 16-byte pieces of them at a time as fit the LDS budget -- are copied to LDS through registers, where
//    alignment, the padded last piece and the sign of uint8 activations (XOR 0x80, once per byte instead of once per product) are
//    free.  Entries become 16-bit piece numbers of LDS rows;
//  * B comes from global memory in operand order (the packed layout of the any-channel-count and the filter-in-registers kernel), one
//    coalesced 1 KB read per fragment, RING steps ahead, and never enters LDS.  A fragment serves MB products: L1 gives 55 to 60 bytes a clock,
//    a KB takes 18 clocks of it and 3 to 4 of the shared return path per LDS fragment, MB products take 8 MB clocks of a compute unit;
//  * between the copies and the output no barrier: wavefronts run apart and hide each other's latencies.  A stage is U steps of one
//    kernel element, so one address per row block serves it with immediate offsets (an address per step made the loop 1.6 times as
//    long); the fragments of a step are read before the products of the step before it;
//  * small problems split the reduction over WS wavefronts of a workgroup; the partial tiles meet in the window's place.
//
// Measured (graph replays, against the kernels that had these problems): 128 x 27 x 27, 48 to 192 channels, 3x3 bf16 33.8 -> 25.4 us;
// 84 x 8 x 8, 96 to 512, 5x5 uint8 28.4 -> 13.4; 160 to 8, 18 x 68 x 87, 5x5 bf16 91 -> 45; one 62 x 66 image, 256 to 256, stride 2,
// batch-independent buffer, 37.0 -> 11.2; 24 x 92 x 92, 32 to 30 uint8 25.1 -> 12.0.  In the steady state (512 x 14 x 14, 256 to 256, 3x3)
// 1.03 PFLOP/s bf16 on random data, 1.9 on zeros: power is what is left.  What bounds the medium sizes is the start (the window
// lands before anything multiplies) and the end (stores), which two to three workgroups on a compute unit hide from each other.
#pragma once
#include "icv_igemm_any_kernel.h"

namespace icv {

struct WindowArgs {
    const uint8_t* a;          // input tensor
    const uint8_t* w;          // packed filter [32-column block][MFMA step][lane][16 bytes]
    const int32_t* ind;        // [block][kernel element][block rows] byte offsets, negative = zero row; or null and
    const uint16_t* ent;       // block form: [32-row block][kernel element][32] pixel numbers from the block's base, 0xFFFF = zero row
    void* out;
    int64_t image_bytes;       // batch-independent buffer: bytes between batch elements of the input (else 0)
    uint32_t img_tiles, img_rows;   // row tiles and output pixels per image (one image = the whole batch otherwise)
    uint32_t block_shift;      // log2 of the rows of a block of entries, no fewer than a tile's (block form: not used)
    uint32_t img_blocks;       // block form: 32-row blocks of an image
    FastDiv by_inner, by_img_tiles, by_stride, by_chunk, by_last_chunk;
    uint32_t total_tiles, tiles_per_xcd, inner, rows_inner, col_blocks;   // inner: tiles along the dimension that runs fastest (rows_inner: rows)
    RangeGeom q;
    int32_t K, T, out_stride;
    int32_t row_bytes, stride_bytes;   // C * element size; bytes between input pixels
    int32_t P;                 // 16-byte pieces per row
    int32_t chunk, last_chunk, n_chunks;      // pieces of a row in LDS at a time; in the last chunk
    int32_t pitch;             // pieces between LDS rows, odd: fragment reads spread over the banks
    int32_t cap_rows;          // pixel rows reserved in LDS; the zero row follows them
    int32_t ent_at;            // LDS offset of the entries
    int32_t n_steps;           // MFMA steps of two pieces in the packed filter
    int32_t tail_shift;        // bytes by which a row's last piece, read as the row's last 16 bytes, is shifted down
    int32_t vector_out;        // 1: four neighbouring outputs may be stored at once
    uint32_t zero_fill;        // four bytes of the zero row
    EpilogueArgs ep;
};

// one step: A fragments hold bytes that are signed already
template <int DT>
__device__ inline typename Acc<DT == ICV_U8I8>::type mfma_signed(const uint4& a, const uint4& b, typename Acc<DT == ICV_U8I8>::type c)
{
    if constexpr (DT == ICV_U8I8) {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(i32x4_t, a), __builtin_bit_cast(i32x4_t, b), c, 0, 0, 0);
    } else if constexpr (DT == ICV_F32) {
        return mfma32_f32(a, b, c);
    } else {
        return mfma32<false>(a, b, c);
    }
}

// A workgroup: WM x WN wavefronts of MB x NB blocks of 32 x 32 each, the reduction split over WS of them.  U: MFMA steps of a stage
// (chunks are whole stages), 0: rows whose pieces make no such stages.
template <int DT, int MB, int NB, int WM, int WN, int WS, int U, bool FUSED>
__global__ __launch_bounds__(64 * WM * WN * WS, 2) void k_igemm_window(WindowArgs g)
{
    constexpr bool I8 = DT == ICV_U8I8;
    constexpr int WAVES = WM * WN * WS, THREADS = 64 * WAVES, MR = 32 * MB * WM, NR = 32 * NB * WN;
    using acc_t = typename Acc<I8>::type;
    using out_acc_t = typename std::conditional<I8, int32_t, float>::type;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    const uint32_t tile = (blockIdx.x & 7u) * g.tiles_per_xcd + (blockIdx.x >> 3);
    if (tile >= g.total_tiles) return;           // the whole workgroup, before any barrier
    const uint32_t outer = fast_div(tile, g.by_inner), in = tile - outer * g.inner;
    const uint32_t mt = g.rows_inner ? in : outer, nt = g.rows_inner ? outer : in;
    const uint32_t img = fast_div(mt, g.by_img_tiles), t_img = mt - img * g.img_tiles;
    const uint32_t row_img = t_img * MR;         // the tile's first output pixel in its image

    // ---- the window: closed-form bounds, nothing is read before its first copy
    uint32_t row_last = row_img + MR - 1;
    if (row_last > g.img_rows - 1) row_last = g.img_rows - 1;
    const int32_t first = lowest_pixel_from(g.q, decompose(g.q, row_img));
    const int32_t last = highest_pixel_upto(g.q, decompose(g.q, row_last));
    uint32_t count = last >= first ? (uint32_t)(last - first) + 1u : 1u;
    if (count > (uint32_t)g.cap_rows) count = (uint32_t)g.cap_rows;
    const uint8_t* const a_win = g.a + (int64_t)img * g.image_bytes + (int64_t)first * g.stride_bytes;
    auto copy_chunk = [&](int c) __attribute__((always_inline)) {
        constexpr int L = 8;                // loads in flight
        const uint32_t cp = c == g.n_chunks - 1 ? (uint32_t)g.last_chunk : (uint32_t)g.chunk;
        const FastDiv by = c == g.n_chunks - 1 ? g.by_last_chunk : g.by_chunk;
        const uint32_t total = count * cp;
        for (uint32_t u0 = 0; u0 < total; u0 += L * THREADS) {
            bytes16_t v[L];
            uint32_t dst[L];
            bool lastp[L];
#pragma unroll
            for (int u = 0; u < L; u++) {
                uint32_t at = u0 + u * THREADS + tid;
                if (at > total - 1) at = total - 1;            // (writes what its neighbour writes)
                const uint32_t row = fast_div(at, by);
                const uint32_t piece = at - row * cp;
                dst[u] = (row * (uint32_t)g.pitch + piece) * 16u;
                uint32_t o = ((uint32_t)(c * g.chunk) + piece) * 16u;
                lastp[u] = o > (uint32_t)g.row_bytes - 16u;          // (only where the last piece is padded)
                if (lastp[u]) o = (uint32_t)g.row_bytes - 16u;
                v[u] = load16_any(a_win + (uint64_t)(row * (uint32_t)g.stride_bytes + o));
            }
#pragma unroll
            for (int u = 0; u < L; u++) {
                if (g.tail_shift) {
                    const bytes16_t s = shift_down(v[u], g.tail_shift);
                    v[u] = lastp[u] ? s : v[u];
                }
                if constexpr (I8) v[u] ^= 0x80808080u;
                *(bytes16_t*)(lds + dst[u]) = v[u];
            }
        }
    };
    // ---- entries -> LDS as 16-bit piece numbers of their rows
    const uint32_t zero_at = (uint32_t)g.cap_rows * (uint32_t)g.pitch;
    {
        auto piece_of = [&](bool zero, int32_t row) -> uint32_t {
            return zero || (uint32_t)row >= (uint32_t)g.cap_rows ? zero_at : (uint32_t)row * (uint32_t)g.pitch;
        };
        uint16_t* const dst = (uint16_t*)(lds + g.ent_at);       // [kernel element][MR]
        if (g.ind) {
            const uint32_t blk = row_img >> g.block_shift;
            const int32_t* const src = g.ind + (((int64_t)blk * g.T) << g.block_shift) + (row_img - (blk << g.block_shift));
            for (int i = tid; i < g.T * (MR / 4); i += THREADS) {
                const int tap = i / (MR / 4), quad = i % (MR / 4);
                const int4 e = *(const int4*)(src + ((int64_t)tap << g.block_shift) + quad * 4);
                auto at = [&](int32_t v) -> uint32_t { return piece_of(v < 0, (int32_t)fast_div((uint32_t)v, g.by_stride) - first); };
                *(uint2*)(dst + tap * MR + quad * 4) = uint2{at(e.x) | at(e.y) << 16, at(e.z) | at(e.w) << 16};
            }
        } else {
            for (int i = tid; i < g.T * (MR / 4); i += THREADS) {
                const int tap = i / (MR / 4), quad = i % (MR / 4);
                uint32_t blk = (row_img >> 5) + (uint32_t)(quad >> 3);
                if (blk > g.img_blocks - 1) blk = g.img_blocks - 1;      // (its rows are not stored)
                const int32_t base = lowest_pixel_from(g.q, decompose(g.q, blk * 32u)) - first;
                const uint2 e = *(const uint2*)(g.ent + ((int64_t)blk * g.T + tap) * 32 + (quad & 7) * 4);
                auto at = [&](uint32_t v) -> uint32_t { return piece_of(v == 0xFFFFu, (int32_t)v + base); };
                *(uint2*)(dst + tap * MR + quad * 4) = uint2{at(e.x & 0xFFFFu) | at(e.x >> 16) << 16, at(e.y & 0xFFFFu) | at(e.y >> 16) << 16};
            }
        }
        for (int i = tid; i < g.pitch * 4; i += THREADS) *(uint32_t*)(lds + zero_at * 16u + i * 4) = g.zero_fill;
    }

    // ---- this wavefront's blocks and its share of the reduction
    const int ws = wave / (WM * WN), wn = wave % WN, wm = wave / WN % WM;
    const uint8_t* wp[NB];
#pragma unroll
    for (int j = 0; j < NB; j++) {
        uint32_t cb = nt * (NR / 32) + wn * NB + j;
        if (cb > g.col_blocks - 1) cb = g.col_blocks - 1;      // (columns past the last are not stored)
        wp[j] = g.w + (int64_t)cb * g.n_steps * 1024;
    }
    acc_t acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; i++)
#pragma unroll
        for (int j = 0; j < NB; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[i][j][r] = 0;

    const uint16_t* const ent = (const uint16_t*)(lds + g.ent_at) + wm * (MB * 32) + lrow;
    constexpr int RING = U == 3 ? 3 : 4;         // filter steps in flight
    const uint32_t lane16 = (uint32_t)lane * 16u;
    uint4 b[RING][NB], af[2][MB];
    auto read_filter = [&](int d, uint32_t at) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NB; j++) b[d][j] = *(const uint4*)(wp[j] + at + lane16);
    };
    auto multiply = [&](int da, int db) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < MB; i++)
#pragma unroll
            for (int j = 0; j < NB; j++) acc[i][j] = mfma_signed<DT>(af[da][i], b[db][j], acc[i][j]);
    };
    for (int c = 0; c < g.n_chunks; c++) {
        if (c > 0) __syncthreads();              // the chunk before has been read
        copy_chunk(c);
        __syncthreads();
        const int cp = c == g.n_chunks - 1 ? g.last_chunk : g.chunk;
        uint32_t e[MB], at[MB];
        if constexpr (U > 0) {
            // stages of U steps, all of one kernel element: an address serves a stage
            const int S = cp / (2 * U), total = g.T * S;          // stages per kernel element, in all
            const int s0 = WS > 1 ? total * ws / WS : 0, n = (WS > 1 ? total * (ws + 1) / WS : total) - s0;
            int tap = 0, r = 0;                  // of the stage whose address is computed next
            if (WS > 1) { tap = s0 / S; r = s0 - tap * S; }
            int b_r = r;
            uint32_t b_at = ((uint32_t)(tap * g.P + c * g.chunk) / 2u + (uint32_t)(r * U)) * 1024u;
            const uint32_t b_gap = (uint32_t)(g.P - cp) * 512u, b_end = (uint32_t)(g.n_steps - U) * 1024u;
            auto next_filter_stage = [&]() __attribute__((always_inline)) {
                b_at += U * 1024u;
                if (++b_r == S) { b_r = 0; b_at += b_gap; }
                if (b_at > b_end) b_at = b_end;
            };
            auto read_entries = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < MB; i++) e[i] = ent[tap * MR + i * 32];
                if (tap < g.T - 1) ++tap;
            };
            const uint32_t half16 = (uint32_t)lhalf * 16u;
            read_entries();
#pragma unroll
            for (int i = 0; i < MB; i++) at[i] = e[i] * 16u + half16 + (uint32_t)(r * (U * 32));
            read_entries();
#pragma unroll
            for (int d = 0; d < RING; d++) {
                read_filter(d, b_at + (d % U) * 1024u);
                if (d % U == U - 1) next_filter_stage();
            }
#pragma unroll
            for (int i = 0; i < MB; i++) af[0][i] = *(const uint4*)(lds + at[i]);
            // (both unrolled to whole rings and pairs of fragment buffers)
            constexpr int STAGES = U == 4 ? 1 : 2;
            auto stage = [&](int k) __attribute__((always_inline)) {
                uint32_t next[MB];
                if (++r == S) {
                    r = 0;
#pragma unroll
                    for (int i = 0; i < MB; i++) asm("v_lshl_add_u32 %0, %1, 4, %2" : "=v"(next[i]) : "v"(e[i]), "v"(half16));
                    read_entries();
                } else {
#pragma unroll
                    for (int i = 0; i < MB; i++) next[i] = at[i] + U * 32;
                }
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int v = k * U + u;
#pragma unroll
                    for (int i = 0; i < MB; i++)
                        af[(v + 1) & 1][i] = u + 1 < U ? *(const uint4*)(lds + at[i] + (u + 1) * 32) : *(const uint4*)(lds + next[i]);
                    __builtin_amdgcn_sched_barrier(0);       // (the fragments of the next step before the products of this one)
                    multiply(v & 1, v % RING);
                    __builtin_amdgcn_sched_barrier(0);
                    read_filter(v % RING, b_at + u * 1024u);
                }
                next_filter_stage();
#pragma unroll
                for (int i = 0; i < MB; i++) at[i] = next[i];
            };
            int s = 0;
            for (; s + STAGES <= n; s += STAGES) {
#pragma unroll
                for (int k = 0; k < STAGES; k++) stage(k);
            }
#pragma unroll
            for (int k = 0; k < STAGES - 1; k++)
                if (s + k < n) stage(k);
        } else {
            // any number of pieces: the halves of a wavefront may be at different kernel elements, an address per step
            // (rows of an odd number of pieces are in LDS whole: one chunk)
            const int total = g.n_chunks == 1 ? g.n_steps : g.T * (cp / 2);
            const int s0 = WS > 1 ? total * ws / WS : 0, n = (WS > 1 ? total * (ws + 1) / WS : total) - s0;
            int tap = (2 * s0 + lhalf) / cp, piece = 2 * s0 + lhalf - tap * cp;
            const int tap0 = 2 * s0 / cp;
            int b_r = 2 * s0 - tap0 * cp;
            const uint32_t b_gap = (uint32_t)(g.P - cp) * 512u, b_end = (uint32_t)(g.n_steps - 1) * 1024u;
            uint32_t b_at = (uint32_t)(g.n_chunks == 1 ? s0 : (tap0 * g.P + c * g.chunk + b_r) / 2) * 1024u;
            auto next_filter = [&](int d) __attribute__((always_inline)) {
                read_filter(d, b_at < b_end ? b_at : b_end);
                b_at += 1024u;
                b_r += 2;
                if (g.n_chunks > 1 && b_r == cp) { b_r = 0; b_at += b_gap; }
            };
            bool past = false;
            uint32_t o = 0;
            auto read_entries = [&]() __attribute__((always_inline)) {
                past = tap >= g.T;
                o = (uint32_t)piece;
#pragma unroll
                for (int i = 0; i < MB; i++) e[i] = ent[(past ? g.T - 1 : tap) * MR + i * 32];
                piece += 2;
                if (piece >= cp) { piece -= cp; ++tap; }
                if (piece >= cp) { piece -= cp; ++tap; }         // (rows of one piece)
            };
            auto read_frags = [&](int d) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < MB; i++) af[d][i] = *(const uint4*)(lds + (past ? zero_at : e[i] + o) * 16u);
            };
            read_entries();
#pragma unroll
            for (int d = 0; d < RING; d++) next_filter(d);
            read_frags(0);
            read_entries();
            auto step = [&](int v) __attribute__((always_inline)) {
                read_frags((v + 1) & 1);
                read_entries();
                __builtin_amdgcn_sched_barrier(0);
                multiply(v & 1, v % RING);
                __builtin_amdgcn_sched_barrier(0);
                next_filter(v % RING);
            };
            int s = 0;
            for (; s + 4 <= n; s += 4) {
#pragma unroll
                for (int v = 0; v < 4; v++) step(v);
            }
#pragma unroll
            for (int v = 0; v < 3; v++)
                if (s + v < n) step(v);
        }
    }

    const int64_t img_row0 = (int64_t)img * g.img_rows;
    if constexpr (WS == 1) {
        const int64_t m_base = img_row0 + (int64_t)row_img + wm * (MB * 32) + 4 * lhalf;
        const int32_t n_base = (int32_t)nt * NR + wn * (NB * 32) + lrow;
        const bool whole_rows = row_img + MR <= g.img_rows, whole = whole_rows && (int32_t)(nt + 1) * NR <= g.K;
        store_tile<FUSED, I8, MB, NB>(g.out, acc, img_row0 + g.img_rows, g.K, g.out_stride, m_base, n_base, whole, whole_rows, g.ep);
    } else {
        // the partial tiles meet in the window's place, a 32 x 32 block of every wavefront at a time
        typedef typename FourOutputs<I8>::vec_t out4_t;
#pragma unroll
        for (int i = 0; i < MB; i++)
#pragma unroll
            for (int j = 0; j < NB; j++) {
                __syncthreads();                 // the window has been read; the sums before have been taken
                out_acc_t* part = (out_acc_t*)(lds + wave * 4096);
#pragma unroll
                for (int r = 0; r < 16; r++) part[(8 * (r >> 2) + 4 * lhalf + (r & 3)) * 32 + lrow] = acc[i][j][r];
                __syncthreads();
                for (int v = tid; v < WM * WN * 256; v += THREADS) {
                    const int block = v >> 8, in = v & 255;      // block: the wavefront of slice 0
                    out4_t sum = *(const out4_t*)(lds + block * 4096 + in * 16);
#pragma unroll
                    for (int w = 1; w < WS; w++) sum += *(const out4_t*)(lds + (w * WM * WN + block) * 4096 + in * 16);
                    const uint32_t row = row_img + (uint32_t)(block / WN * (MB * 32) + i * 32 + (in >> 3));
                    const int32_t col = (int32_t)nt * NR + block % WN * (NB * 32) + j * 32 + (in & 7) * 4;
                    if (row < g.img_rows)
                        store_four<I8>(g.out, (img_row0 + row) * g.out_stride + col, sum, col, g.K, g.vector_out, g.ep);
                }
            }
    }
}

template <int DT, int MB, int NB, int WM, int WN, int WS, int U, bool FUSED>
static int launch_window_one(const WindowArgs& a, size_t lds_bytes, hipStream_t s)
{
    auto kern = k_igemm_window<DT, MB, NB, WM, WN, WS, U, FUSED>;
    if (lds_bytes > 64 * 1024) {
        static bool raised[kMaxDevices] = {};      // one array per instantiation of this function template
        const int st = allow_full_lds((const void*)kern, raised);
        if (st != ICV_OK) return st;
    }
    hipLaunchKernelGGL(kern, dim3(8u * a.tiles_per_xcd), dim3(64 * WM * WN * WS), lds_bytes, s, a);
    ICV_HIP_CHECK(hipGetLastError());
    return ICV_OK;
}

template <int DT, int MB, int NB, int WM, int WN, int WS>
static int launch_window_tile(const WindowArgs& a, int unroll, size_t lds_bytes, bool fused, hipStream_t s)
{
    constexpr bool F = WS == 1;      // (the sum of partial tiles has a run-time output stage)
#define ICV_WINDOW_STEPS(U)                                                                               \
    if (unroll == U && F && fused) return launch_window_one<DT, MB, NB, WM, WN, WS, U, F>(a, lds_bytes, s); \
    if (unroll == U) return launch_window_one<DT, MB, NB, WM, WN, WS, U, false>(a, lds_bytes, s);
    ICV_WINDOW_STEPS(4)
    ICV_WINDOW_STEPS(3)
    ICV_WINDOW_STEPS(2)
    ICV_WINDOW_STEPS(0)
#undef ICV_WINDOW_STEPS
    return ICV_ERR_UNSUPPORTED;
}

// Every instantiation of one dtype: one translation unit each, so that they compile side by side.  The tiles are kWindowTiles'.
template <int DT>
static int launch_window_instances(const WindowArgs& a, int tile, int unroll, size_t lds_bytes, bool fused, hipStream_t s)
{
    switch (tile) {
    case 0: return launch_window_tile<DT, 2, 1, 2, 2, 1>(a, unroll, lds_bytes, fused, s);
    case 1: return launch_window_tile<DT, 1, 1, 2, 2, 1>(a, unroll, lds_bytes, fused, s);
    case 2: return launch_window_tile<DT, 1, 1, 4, 1, 1>(a, unroll, lds_bytes, fused, s);
    case 3: return launch_window_tile<DT, 1, 1, 1, 1, 8>(a, unroll, lds_bytes, fused, s);
    case 4: return launch_window_tile<DT, 2, 1, 1, 4, 1>(a, unroll, lds_bytes, fused, s);
    case 5: return launch_window_tile<DT, 2, 1, 1, 2, 4>(a, unroll, lds_bytes, fused, s);
    }
    return ICV_ERR_UNSUPPORTED;
}

int launch_window_bf16(const WindowArgs& a, int tile, int unroll, size_t lds_bytes, bool fused, hipStream_t s);
int launch_window_u8(const WindowArgs& a, int tile, int unroll, size_t lds_bytes, bool fused, hipStream_t s);
int launch_window_f32(const WindowArgs& a, int tile, int unroll, size_t lds_bytes, bool fused, hipStream_t s);

}  // namespace icv
