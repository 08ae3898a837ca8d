// Tensor-core Indirect GEMM for problems too small to fill the chip: the reduction of one output tile is split over the
// wavefronts of a workgroup.
//
// A layer with few output pixels (one image at a time, the 7 x 7 maps at the end of a network) has fewer output tiles
// than the chip has compute units, and the other kernels walk the whole R*S*C reduction of a tile serially: what bounds
// them is the latency of that chain.  Here each of up to 16 wavefronts takes a contiguous run of the reduction's 128-byte
// stages for the whole tile and works on its own: a private piece of LDS, no barrier, its own loads D stages ahead.
// The partial tiles meet in LDS at the end, where all threads sum them and apply the output stage.
//
//  * A: a wavefront stages its rows through registers (coalesced 128-byte reads from any address, as in the
//    any-channel-count kernel) into its own LDS tile and reads the operand fragments back.  The instructions of one
//    wavefront reach LDS in order, so one buffer is enough.
//  * B comes from global memory in operand order, one coalesced read per fragment, as far ahead as the rows.
//  * Entries are read 2 D stages ahead, so that a row's address is there when its load is issued and the loads in flight
//    are never drained for one.
//
// The 32 x 32 tile runs as the window kernel's (rows in LDS once instead of once per kernel element: 83 x 8 x 12, 336 to 64
// channels, 5x5 30.2 -> 15.6 us) where its window fits; here remain pointwise layers and windows above 128 KB.
//
// Tiles: 16 x 16 (most workgroups: a wavefront's loads are what a small problem waits for) and 32 x 32 (each loaded byte
// multiplied twice as often).  64 x 64 was tried and taken out: it was ahead in one problem of ninety, by a fifth.  The rule
// that chooses, with what it measured, is at choose_split in the host file.
#pragma once
#include "icv_mfma_common.h"
#include "icv_pixel_range.h"

namespace icv {

struct SplitArgs {
    const uint8_t* a;          // input tensor | patch matrix
    const uint8_t* zero_row;
    const uint8_t* w;          // packed filter [32-column block][MFMA step][lane][16 bytes]
    const int32_t* ind;        // [block][kernel element][block rows] byte offsets, negative = zero row
    const int4* rec;           // block form: per 32-row block {base byte offset, ...}
    const uint16_t* ent;       // block form: [block][kernel element][32] pixel numbers from the base, 0xFFFF = zero row
    void* out;
    int64_t a_row_stride;      // dense A: bytes between rows
    int64_t a_rows;            // dense A: rows that may be read (later ones re-read the last)
    int64_t image_bytes;       // batch-independent buffer: bytes between batch elements of the input (else 0)
    uint32_t img_tiles, img_rows;    // tiles of this kernel and output pixels per image (one image = the whole batch otherwise)
    uint32_t block_shift;      // log2 of the rows of a block of entries
    FastDiv by_inner, by_img_tiles;
    uint32_t total_tiles, tiles_per_xcd, inner;   // inner: tiles along the dimension that runs fastest
    uint32_t rows_inner;       // 1: row tiles run fastest (the filter is the larger operand), 0: column tiles
    int32_t K, T, out_stride;
    int32_t row_bytes, stride_bytes;   // C * element size; bytes between input pixels
    int32_t P;                 // 16-byte pieces per row
    FastDiv by_P;
    int32_t step_taps, step_pieces;    // 8 / P, 8 % P
    int32_t n_steps, n_stages; // MFMA steps of 32 bytes, stages of 128
    int32_t tail_shift;        // bytes by which a row's last piece, read as the row's last 16 bytes, is shifted down
    int32_t slices;            // wavefronts of a workgroup, at most n_stages
    int32_t vector_out;        // 1: four neighbouring outputs may be stored at once
    EpilogueArgs ep;
};

enum SplitRows : int { SPLIT_DENSE = 0, SPLIT_INT32 = 1, SPLIT_BLOCK16 = 2 };

typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int DT, int BLK>
struct SplitAcc {
    using type = typename std::conditional<BLK == 32, typename Acc<DT == ICV_U8I8>::type,
                 typename std::conditional<DT == ICV_U8I8, i32x4_t, f32x4_t>::type>::type;
};

template <int DT, int BLK>
__device__ inline typename SplitAcc<DT, BLK>::type split_mfma(const uint4& a, const uint4& b, typename SplitAcc<DT, BLK>::type c)
{
    if constexpr (BLK == 32) {
        if constexpr (DT == ICV_F32) return mfma32_f32(a, b, c);
        else return mfma32<DT == ICV_U8I8>(a, b, c);
    } else if constexpr (DT == ICV_U8I8) {
        const i32x4_t av = {(int)(a.x ^ 0x80808080u), (int)(a.y ^ 0x80808080u), (int)(a.z ^ 0x80808080u), (int)(a.w ^ 0x80808080u)};
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(av, __builtin_bit_cast(i32x4_t, b), c, 0, 0, 0);
    } else if constexpr (DT == ICV_BF16) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    } else {
        // as mfma32_f32: product j pairs element j of the four lane groups of A with those of B
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.x), __builtin_bit_cast(float, b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.y), __builtin_bit_cast(float, b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.z), __builtin_bit_cast(float, b.z), c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.w), __builtin_bit_cast(float, b.w), c, 0, 0, 0);
    }
}

constexpr int kSplitPitch = 144;               // eight pieces and one of padding: fragment reads spread over the banks
constexpr int split_region_bytes(int BLK)      // LDS of a wavefront: its rows, later its partial tile (which is smaller)
{
    return BLK * kSplitPitch;
}

// A tile is BLK x BLK; D stages of rows are in flight per wavefront.
constexpr int kSplitMaxSlices = 16;
template <int DT, int BLK, int D, bool TAIL, int ROWS>
__global__ __launch_bounds__(64 * kSplitMaxSlices) void k_igemm_split(SplitArgs g)
{
    constexpr bool I8 = DT == ICV_U8I8;
    constexpr int RPT = BLK / 8;                 // rows per lane: lane -> piece lane % 8 of rows lane / 8, + 8, ...
    constexpr int KS = BLK == 32 ? 4 : 2;        // MFMA steps per stage (32 or 64 bytes of the reduction)
    constexpr int REGION = split_region_bytes(BLK);
    static_assert(BLK * BLK * 4 <= REGION, "the partial tile takes the place of the rows");
    using acc_t = typename SplitAcc<DT, BLK>::type;
    using out_acc_t = typename std::conditional<I8, int32_t, float>::type;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // XCD x (workgroups x, x + 8, ...) takes a contiguous run of tiles
    const uint32_t tile = (blockIdx.x & 7u) * g.tiles_per_xcd + (blockIdx.x >> 3);
    if (tile >= g.total_tiles) return;           // the whole workgroup, before any barrier
    const uint32_t outer = fast_div(tile, g.by_inner), in = tile - outer * g.inner;
    const uint32_t mt = g.rows_inner ? in : outer, nt = g.rows_inner ? outer : in;
    const uint32_t img = fast_div(mt, g.by_img_tiles), t_img = mt - img * g.img_tiles;

    // this wavefront's stages s0 .. s0 + n - 1
    const int share = g.n_stages / g.slices, extra = g.n_stages - share * g.slices;
    const int s0 = wave * share + (wave < extra ? wave : extra);
    const int n = share + (wave < extra ? 1 : 0);

    // ---- A
    const int q = lane & 7, r0 = lane >> 3;
    const uint8_t* const a_img = g.a + (int64_t)img * g.image_bytes;
    // (a block of entries is 32 rows or more, so the tile's rows share one)
    const uint8_t* base[ROWS == SPLIT_DENSE ? RPT : 1];
    const int32_t* ent32 = nullptr;
    const uint16_t* ent16 = nullptr;
    uint32_t first = 0;
    if constexpr (ROWS == SPLIT_DENSE) {
#pragma unroll
        for (int i = 0; i < RPT; i++) {
            int64_t m = (int64_t)img * g.img_rows + t_img * BLK + r0 + 8 * i;
            if (m > g.a_rows - 1) m = g.a_rows - 1;
            base[i] = g.a + m * g.a_row_stride;
        }
    } else {
        const uint32_t row = t_img * BLK, blk = row >> g.block_shift;      // in its image
        const int64_t at = (((int64_t)blk * g.T) << g.block_shift) + (row & ((1u << g.block_shift) - 1u)) + r0;
        if constexpr (ROWS == SPLIT_INT32) ent32 = g.ind + at;
        else { ent16 = g.ent + at; first = (uint32_t)g.rec[blk].x; }
    }
    // walk over the pieces (s0 * 8 + q), + 8, ...: kernel element and piece of its row
    int tap = (int)fast_div((uint32_t)(s0 * 8 + q), g.by_P), piece = s0 * 8 + q - tap * g.P;
    int32_t e[D][RPT];
    int e_off[D];                                // byte of the row; -1: the piece lies past the patch
    bool e_last[D];
    auto read_entries = [&](int d) __attribute__((always_inline)) {
        const bool past = tap >= g.T;
        const int t = past ? g.T - 1 : tap;
        e_last[d] = TAIL && piece == g.P - 1;
        int o = piece * 16;
        if (TAIL && o > g.row_bytes - 16) o = g.row_bytes - 16;
        e_off[d] = past ? -1 : o;
#pragma unroll
        for (int i = 0; i < RPT; i++) {
            if constexpr (ROWS == SPLIT_DENSE) {
                e[d][i] = t * g.row_bytes;
            } else if constexpr (ROWS == SPLIT_INT32) {
                e[d][i] = ent32[((int64_t)t << g.block_shift) + 8 * i];
            } else {
                e[d][i] = ent16[t * 32 + 8 * i];
            }
        }
        tap += g.step_taps;
        piece += g.step_pieces;
        if (piece >= g.P) { piece -= g.P; ++tap; }
    };
    bytes16_t av[D][RPT];
    bool v_past[D], v_last[D];
    auto read_rows = [&](int d, bool used) __attribute__((always_inline)) {
        v_past[d] = e_off[d] < 0;
        v_last[d] = e_last[d];
        const uint32_t o = e_off[d] < 0 ? 0u : (uint32_t)e_off[d];
#pragma unroll
        for (int i = 0; i < RPT; i++) {
            const uint8_t* src;
            if constexpr (ROWS == SPLIT_DENSE) {
                src = base[i] + (uint32_t)e[d][i];
            } else if constexpr (ROWS == SPLIT_INT32) {
                src = e[d][i] < 0 ? g.zero_row : a_img + (uint32_t)e[d][i];
            } else {
                src = e[d][i] == 0xFFFF ? g.zero_row : a_img + (first + (uint32_t)e[d][i] * (uint32_t)g.stride_bytes);
            }
            src = used ? src + o : g.w;
            __builtin_memcpy(&av[d][i], src, 16);             // 16 bytes from any address
        }
    };
    uint8_t* const mine = lds + wave * REGION;
    auto to_lds = [&](int d) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RPT; i++) {
            bytes16_t v = av[d][i];
            if constexpr (TAIL) {
                const bytes16_t s = shift_down(v, g.tail_shift);
                v = v_last[d] ? s : v;
            }
            if (v_past[d]) v = bytes16_t{0u, 0u, 0u, 0u};
            *(bytes16_t*)(mine + (r0 + 8 * i) * kSplitPitch + q * 16) = v;
        }
    };

    // ---- B.  Lanes of a 32 x 32 fragment: column lane % 32, bytes 16 * (lane / 32) of the 32-byte step.  A 16 x 16
    // fragment takes 16 of a 32-column block's columns and two steps: lane group lane / 16 holds step
    // lane / 32 of the two, half (lane / 16) % 2 of it.
    const uint8_t* const wp = BLK == 32
        ? g.w + (int64_t)nt * g.n_steps * 1024 + lane * 16
        : g.w + (int64_t)(nt >> 1) * g.n_steps * 1024 + (((lane >> 4) & 1) * 32 + (nt & 1) * 16 + (lane & 15)) * 16;
    uint4 b[D][KS];
    auto read_filter = [&](int d, int stage, bool used) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
            int f = BLK == 32 ? stage * 4 + ks : stage * 4 + 2 * ks + (lane >> 5);
            if (f > g.n_steps - 1) f = g.n_steps - 1;
            if (!used) f = 0;
            b[d][ks] = *(const uint4*)(wp + (int64_t)f * 1024);
        }
    };

    acc_t acc;
#pragma unroll
    for (int r = 0; r < BLK * BLK / 64; r++) acc[r] = 0;
    const uint8_t* const frag = mine + (BLK == 32 ? (lane & 31) * kSplitPitch + (lane >> 5) * 16
                                                  : (lane & 15) * kSplitPitch + (lane >> 4) * 16);
    auto multiply = [&](int d, int ks, bool half) __attribute__((always_inline)) {
        uint4 bf = b[d][ks];
        if (half && (lane >> 5)) bf = uint4{0u, 0u, 0u, 0u};
        acc = split_mfma<DT, BLK>(*(const uint4*)(frag + ks * (128 / KS)), bf, acc);
    };
    // (the fences keep the compiler from moving a lane's LDS accesses across other lanes'; the hardware runs one
    // wavefront's in order)
    auto stage_rows = [&](int d) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        to_lds(d);
        asm volatile("" ::: "memory");
    };

    // ---- the first D stages' rows, the entries of D more, then one loop.  No load is conditional, so that the waits
    // leave the younger ones in flight; those for stages past this wavefront's last read one address and are not used.
#pragma unroll
    for (int d = 0; d < D; d++) read_entries(d);
#pragma unroll
    for (int d = 0; d < D; d++) {
        read_rows(d, d < n);
        read_entries(d);
        read_filter(d, s0 + d, d < n);
    }
    for (int s = 0; s < n; s += D) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            const bool live = s + d < n, more = s + d + D < n;
            if (live) stage_rows(d);
            __builtin_amdgcn_sched_barrier(0);
            read_rows(d, more);
            read_entries(d);
            __builtin_amdgcn_sched_barrier(0);
            if (live) {
                const int steps = g.n_steps - (s0 + s + d) * 4;       // at least four unless this is the last stage
#pragma unroll
                for (int ks = 0; ks < KS; ks++)
                    if (ks * (4 / KS) < steps) {
                        // a pair of steps of which there is only the first: the second multiplies zeros
                        multiply(d, ks, BLK == 16 && 2 * ks + 1 >= steps);
                    }
            }
            __builtin_amdgcn_sched_barrier(0);                        // (registers: no load before its slot is free)
            read_filter(d, s0 + s + d + D, more);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- sum the partial tiles
    const int64_t row0 = (int64_t)img * g.img_rows + (int64_t)t_img * BLK;
    const int64_t m_end = (int64_t)(img + 1) * g.img_rows;
    const int threads = g.slices * 64;
    typedef typename FourOutputs<I8>::vec_t out4_t;
    {
        out_acc_t* part = (out_acc_t*)mine;      // [BLK][BLK]
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < BLK * BLK / 64; r++) {
            const int row = BLK == 32 ? 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3) : 4 * (lane >> 4) + r;
            part[row * BLK + (lane & (BLK - 1))] = acc[r];
        }
        __syncthreads();
        for (int v = tid; v < BLK * BLK / 4; v += threads) {
            out4_t sum = *(const out4_t*)(lds + v * 16);
#pragma unroll 4
            for (int w = 1; w < g.slices; w++) sum += *(const out4_t*)(lds + w * REGION + v * 16);
            const int64_t row = row0 + v / (BLK / 4);
            const int32_t col = (int32_t)nt * BLK + v % (BLK / 4) * 4;
            if (row >= m_end) continue;
            store_four<I8>(g.out, row * g.out_stride + col, sum, col, g.K, g.vector_out, g.ep);
        }
    }
}

// Every instantiation of one dtype: one translation unit each, so that they compile side by side.
enum SplitTile : int { SPLIT_16 = 0, SPLIT_32 = 1 };

template <int DT, int BLK, int D, bool TAIL, int ROWS>
static int launch_split_one(const SplitArgs& a, hipStream_t s)
{
    auto kern = k_igemm_split<DT, BLK, D, TAIL, ROWS>;
    const size_t lds_bytes = (size_t)a.slices * split_region_bytes(BLK);
    if (a.slices < 1 || a.slices > kSplitMaxSlices || a.slices > a.n_stages || lds_bytes > kLdsPerCu) return ICV_ERR_UNSUPPORTED;
    if (lds_bytes > 64 * 1024) {
        static bool raised[kMaxDevices] = {};      // one array per instantiation of this function template
        const int st = allow_full_lds((const void*)kern, raised);
        if (st != ICV_OK) return st;
    }
    hipLaunchKernelGGL(kern, dim3(8u * a.tiles_per_xcd), dim3(64 * a.slices), lds_bytes, s, a);
    ICV_HIP_CHECK(hipGetLastError());
    return ICV_OK;
}

template <int DT, int BLK, int D>
static int launch_split_tile(const SplitArgs& a, int rows, bool tail, hipStream_t s)
{
    if constexpr (BLK == 16) {      // (32 x 32 tiles of such a plan are the window kernel's)
        if (rows == SPLIT_BLOCK16) return tail ? ICV_ERR_UNSUPPORTED : launch_split_one<DT, BLK, D, false, SPLIT_BLOCK16>(a, s);
    }
    if (rows == SPLIT_BLOCK16) return ICV_ERR_UNSUPPORTED;
    if (rows == SPLIT_INT32)
        return tail ? launch_split_one<DT, BLK, D, true, SPLIT_INT32>(a, s)
                    : launch_split_one<DT, BLK, D, false, SPLIT_INT32>(a, s);
    return tail ? launch_split_one<DT, BLK, D, true, SPLIT_DENSE>(a, s)
                : launch_split_one<DT, BLK, D, false, SPLIT_DENSE>(a, s);
}

template <int DT>
static int launch_split_instances(const SplitArgs& a, int tile, int rows, bool tail, hipStream_t s)
{
    switch (tile) {
    case SPLIT_16: return launch_split_tile<DT, 16, 3>(a, rows, tail, s);
    case SPLIT_32: return launch_split_tile<DT, 32, 2>(a, rows, tail, s);
    }
    return ICV_ERR_UNSUPPORTED;
}

int launch_split_bf16(const SplitArgs& a, int tile, int rows, bool tail, hipStream_t s);
int launch_split_u8(const SplitArgs& a, int tile, int rows, bool tail, hipStream_t s);
int launch_split_f32(const SplitArgs& a, int tile, int rows, bool tail, hipStream_t s);

}  // namespace icv
