// Grouped expert GEMMs (the SwiGLU expert MLPs of the MoE layer, one GEMM pair per expert).
//
//   gate_up: for each expert e, the rows of x routed to e (gathered through row_token, never
//            materialised) times W_gate_up[e]^T, with SwiGLU fused in the epilogue:
//            H[r, c] = silu(g) * u, g = x_r . W_gate[e][c], u = x_r . W_up[e][c].
//   down:    Y[r, :] = H[r, :] W_down[e]^T for the rows r of expert e.
//
// Work list: expert e owns rows [offsets[e], offsets[e+1]) of the expert-major order and
// M-tiles [tile_off[e], tile_off[e+1]); both come from the dispatch scan, on the device, so
// the grid is launched with an upper bound of M-tiles and surplus blocks exit at once.
//
// Kernels (all fp32 accumulation; the launchers at the end pick one per problem):
//  - gemm_bf16_dma: the prefill kernel (gemm_tile_rows: at least 112 rows per expert).  Block tile
//    256 x 256 x 64, 4 waves of 128 x 128 on v_mfma_f32_32x32x16_bf16, operands copied
//    global -> LDS by global_load_lds_dwordx4 into a 5-unit ring; remainder rows of a few
//    experts (TilePlan) go to extra blocks of the same launch (weight-streaming tasks of
//    gemm_stream.h).  Described in detail above the kernel.
//  - gemm_bf16_mid: smaller problems.  Block tile 64 or 128 x 128 x 64, two blocks per CU,
//    operands copied global -> LDS likewise, the contraction started at a different k-tile in
//    each N-tile.  Described above the kernel.
//  - decode-sized batches use gemm_skinny.hip instead (weight streaming).
// fp32 path: gemm_f32, 64 x 64 x 32 tiles on the fp32 matrix instructions.
#include "gemm_stream.h"
#include "tilegrid.h"

namespace elb {

namespace {

// The expert e that owns item `item` of a numbering in which expert e's items are
// [per tile_off[e], per tile_off[e + 1]): every lane looks at one expert (N <= 64), so it takes
// one memory round trip instead of a binary search's six.  first: e's first item; tiles, row0,
// end: its M-tiles, first row and row past its last one.
__device__ __forceinline__ void find_expert(const int* __restrict__ tile_off,
                                            const int* __restrict__ offsets, int N, int item,
                                            int per, int& e, int& first, int& tiles, int& row0,
                                            int& end) {
    const int lane = threadIdx.x & 63;
    const int l = lane < N ? lane : N - 1;
    const int t0 = tile_off[l], t1 = tile_off[l + 1];
    const int r0 = offsets[l], r1 = offsets[l + 1];
    const uint64_t mine = __ballot(lane < N && t0 * per <= item && item < t1 * per);
    e = __builtin_ctzll(mine | (1ull << 63));
    first = __builtin_amdgcn_readlane(t0, e) * per;
    tiles = __builtin_amdgcn_readlane(t1, e) - __builtin_amdgcn_readlane(t0, e);
    row0 = __builtin_amdgcn_readlane(r0, e);
    end = __builtin_amdgcn_readlane(r1, e);
}

// M-tile `tile` (tile_rows rows): its expert e, first row, rows; tiles: e's tiles, last: the rows
// from its last tile on
__device__ __forceinline__ void find_tile(const int* __restrict__ tile_off,
                                          const int* __restrict__ offsets, int N, int tile,
                                          int tile_rows, int& e, int& row0, int& rows,
                                          int& tiles, int& last) {
    int first, end;
    find_expert(tile_off, offsets, N, tile, 1, e, first, tiles, row0, end);
    last = end - row0 - (tiles - 1) * tile_rows;
    row0 += (tile - first) * tile_rows;
    rows = end - row0 < tile_rows ? end - row0 : tile_rows;
}

// Block -> tile mapping.  Blocks are dispatched round-robin over the 8 XCDs (block b runs on
// XCD b % 8), and each XCD has its own L2.  Tiles are numbered expert-major, M-tile, then
// N-tile innermost, and XCD x takes the contiguous range [x * per, (x + 1) * per) of that
// order, so the blocks resident on one XCD at a time share their experts' weight tiles and
// gathered token rows through that XCD's L2.  The grid is an upper bound (a multiple of 8);
// surplus blocks exit.
__device__ __forceinline__ bool xcd_tile(int b, int total, int nt_count, int& mt, int& nt) {
    const int per = (total + 7) >> 3;
    const int s = b >> 3;
    const int L = (b & 7) * per + s;
    if (s >= per || L >= total) return false;
    mt = L / nt_count;
    nt = L - mt * nt_count;
    return true;
}

// silu(z) = z / (1 + e^-z), with a hardware reciprocal (the result is rounded to bf16 or
// compared at 1e-4 in fp32, far above its error)
__device__ __forceinline__ float silu(float z) {
    return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z));
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel for mid-sized batches (tens of rows per expert): 64 or 128 x 128 block tiles
//
// Here the expert weights still have to be streamed (at 60 rows per expert the MFMAs need a
// third of the time the weights take), but every weight meets too many token rows for the
// decode kernels, which read the rows straight from L2.  So both operands go through LDS
// (global_load_lds_dwordx4, 8 rows x 128 bytes per instruction, chunks XOR-swizzled as in the
// large-tile kernel), and everything else is arranged for the stream:
//  - 80 KB of LDS per block, two blocks per CU: one block's start, end and barriers fall into
//    the other's stream;
//  - three 64-deep weight units of 128 rows (16 KB), and two (128-row tiles) or three (64-row
//    tiles) token units: a unit is refilled as soon as the barrier shows that every wave has
//    read it, so weights are two k-tiles ahead;
//  - block (e, ntile) starts its contraction at k-tile ntile nk / nt_count and wraps around:
//    weight rows lie a multiple of 1 KB or more apart, and blocks that all walk the same
//    columns at the same time crowd onto part of the memory channels (gate/up at 60 rows per
//    expert, the former register-staged form of this kernel: 135 us in step, 107 us rotated).
//    Also with many M-tiles per expert, where it matters little (layer us, rotated / experts of
//    two tiles or more in step: 4096 tokens top-8, m = 1088, N = 64 611 / 624; d = 1024, m = 576,
//    N = 32 147 / 148; 8192 tokens top-2, d = 1024, m = 192, N = 8 67.5 / 66.5);
//  - the M-tiles of an expert that share a weight tile are neighbours on one XCD and start at
//    the same k-tile, so the second one finds most of the weights in L2.  Weights that only
//    one tile reads carry the non-temporal hint, shared ones do not (two tiles per expert, 152
//    rows: gate/up 213 us with the hint, 153 without; one tile, 60 rows: 96 and 102).
// A tile with at most 64 rows left takes the 64-row form (block-uniform): half the LDS traffic
// and MFMAs.  4 waves (2 x 2), v_mfma_f32_32x32x16_bf16 with the weights first, so a lane ends
// with 4 consecutive output columns of a token row; in gate/up the 128 weight rows are 64 gate
// and the matching 64 up rows, and each wave owns matching 32-column pairs.
// Measured against the register-staged double-buffered form it replaces (OLMoE-shaped layer,
// gate/up + down us): 256 tokens 130 + 56 -> 85 + 47, 512 tokens 135 + 63 -> 93 + 52 (5.8 and
// 5.1 TB/s of weights).
// ------------------------------------------------------------------------------------------
constexpr int BM = 128, BN = 128;

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// two floats -> two bf16 (round to nearest even) in one v_cvt_pk_bf16_f32
typedef __bf16 bf16x2_vt __attribute__((ext_vector_type(2)));
typedef float f32x2_vt __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const f32x2_vt v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_vt));
}

// MODE 0 = gate_up (+SwiGLU -> H), 1 = down (-> Y); TM x TN: the block tile, rows (token rows of
// the expert) x weight rows, WM: waves along the rows; rot: first k-tile of the block, < nk; nt:
// the weight copies carry the non-temporal hint; DMA: x and the weights are 16-byte aligned
template <int MODE, int TM, int TN, int WM, bool DMA = true>
__device__ __forceinline__ void gemm_mid_body(const bf16_t* __restrict__ A,
                                              const int* __restrict__ row_token,
                                              const bf16_t* __restrict__ B, int e, int row0,
                                              int rows, int ntile, int rot, int d, int m,
                                              bf16_t* __restrict__ C, char* sm, bool nt) {
    constexpr int TK = 64;
    constexpr int BU = TN * TK * 2, AU = TM * TK * 2;  // bytes of a weight / token unit
    constexpr int NB = 3, NA = (TM == TN) ? 2 : 3;     // units of each
    constexpr int IB = TN / 32, IA = TM / 32;          // copy instructions per wave and unit
    constexpr int WN = 4 / WM;
    constexpr int FM = TM / WM / 32, FN = TN / WN / 32;  // 32-row fragments per wave
    constexpr int OUTC = (MODE == 0) ? TN / 2 : TN;    // output columns of the block
    constexpr int WC = OUTC / WN;                      // output columns of a wave
    constexpr int PITCH = OUTC * 2 + 16;               // bytes per row of the staged output
    static_assert(NB * BU + NA * AU <= TN * 640 && TM * PITCH <= TN * 640, "LDS of the kernels");
    char* const smb = sm;
    char* const sma = sm + NB * BU;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / WN, wn = wid % WN;
    const int Kd = (MODE == 0) ? d : m;
    const int nk = Kd / TK;

    // copy sources: lane l of copy i fills physical chunk l & 7 of the unit's row
    // 8 (I wid + i) + (l >> 3) with that row's logical chunk (64-bit addresses)
    const char* a_src[IA];
    const char* b_src[IB];
#pragma unroll
    for (int i = 0; i < IA; ++i) {
        const int r = 8 * (IA * wid + i) + (lane >> 3);
        const int rr = r < rows ? r : rows - 1;  // rows past the tile's end: never stored
        const int64_t src = (MODE == 0) ? (int64_t)row_token[row0 + rr] * d
                                        : (int64_t)(row0 + rr) * m;
        a_src[i] = reinterpret_cast<const char*>(A + src) + swz8(r, lane & 7) * 16;
    }
#pragma unroll
    for (int i = 0; i < IB; ++i) {
        const int r = 8 * (IB * wid + i) + (lane >> 3);
        int brow;
        if (MODE == 0) {
            brow = (r < OUTC) ? ntile * OUTC + r : m + ntile * OUTC + (r - OUTC);
        } else {
            brow = ntile * TN + r;
            brow = brow < d ? brow : d - 1;  // columns past d: never stored
        }
        const int64_t src = ((int64_t)e * ((MODE == 0) ? 2 * m : d) + brow) * Kd;
        b_src[i] = reinterpret_cast<const char*>(B + src) + swz8(r, lane & 7) * 16;
    }
    const uint32_t lds_b = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(lds_void_t*)smb + (uint32_t)wid * (IB * 1024));
    const uint32_t lds_a = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(lds_void_t*)sma + (uint32_t)wid * (IA * 1024));
    // The copies are inline assembly: the compiler cannot tell which unit a copy writes, and
    // would otherwise wait for every copy in flight before each LDS read; waits are explicit.
    auto k_bytes = [&](int t) {  // byte offset of k-tile t of this block's rotated order
        const int kt = t + rot < nk ? t + rot : t + rot - nk;
        return (int64_t)kt * (TK * 2);
    };
    auto issue_a = [&](int t, int unit) {
        const int64_t kb = k_bytes(t);
#pragma unroll
        for (int i = 0; i < IA; ++i) {
            const uint32_t la = lds_a + unit * AU + i * 1024;
            const char* const va = a_src[i] + kb;
            if constexpr (!DMA) {
                copy16_any(sma + unit * AU + (wid * IA + i) * 1024 + lane * 16, va);
                continue;
            }
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                         :: "s"(la), "v"(va) : "memory", "m0");
        }
    };
    auto issue_b = [&](int t, int unit) {
        const int64_t kb = k_bytes(t);
#pragma unroll
        for (int i = 0; i < IB; ++i) {
            const uint32_t la = lds_b + unit * BU + i * 1024;
            const char* const va = b_src[i] + kb;
            if constexpr (!DMA) {
                copy16_any(smb + unit * BU + (wid * IB + i) * 1024 + lane * 16, va);
                continue;
            }
            if (nt)
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off nt"
                             :: "s"(la), "v"(va) : "memory", "m0");
            else
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                             :: "s"(la), "v"(va) : "memory", "m0");
        }
    };

    const int l32 = lane & 31, hi = lane >> 5;
    int a_row[FM], b_row[FN];  // gate/up: fragments 0 .. FN/2 - 1 gate, the rest matching up
#pragma unroll
    for (int i = 0; i < FM; ++i) a_row[i] = (wm * (TM / WM) + 32 * i + l32) * 128;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int up = (MODE == 0 && j >= FN / 2) ? 1 : 0;
        b_row[j] = (up * OUTC + WC * wn + 32 * (j - up * (FN / 2)) + l32) * 128;
    }
    int cofs[4];  // byte offset of the chunk this lane reads for k16-step kk
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) cofs[kk] = swz8(l32, 2 * kk + hi) * 16;

    f32x16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

    // Copies in flight: at the barrier that opens k-tile t every wave has read tile t - 1, whose
    // units then receive the weights of tile t + 2 and the token rows of tile t + 2 (three
    // token units) or t + 1 (two).  Copies complete in order, and what tile t + 1 needs is
    // issued before the weights of t + 2, so the wait that opens it may leave those IB (three
    // token units: IB + IA) copies in flight.
    constexpr int AHEAD_A = NA - 1;
    if (AHEAD_A == 2) {
        issue_a(0, 0);
        issue_b(0, 0);
        if (nk > 1) {
            issue_a(1, 1);
            issue_b(1, 1);
        }
    } else {
        issue_b(0, 0);
        issue_a(0, 0);
        if (nk > 1) issue_b(1, 1);
    }
    int ub = 0, ua = 0;  // units of tile t
    for (int t = 0; t < nk; ++t) {
        if (t + 1 < nk) ELB_WAIT_VMCNT(AHEAD_A == 2 ? IB + IA : IB);
        else ELB_WAIT_VMCNT(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const int ua_next = ua + AHEAD_A >= NA ? ua + AHEAD_A - NA : ua + AHEAD_A;
        const int ub_next = ub + 2 >= NB ? ub + 2 - NB : ub + 2;
        if (t + AHEAD_A < nk) issue_a(t + AHEAD_A, ua_next);
        if (t + 2 < nk) issue_b(t + 2, ub_next);
        const char* const pa = sma + ua * AU;
        const char* const pb = smb + ub * BU;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            bf16x8_t fa[FM], fb[FN];
#pragma unroll
            for (int j = 0; j < FN; ++j)
                fb[j] = *reinterpret_cast<const bf16x8_t*>(pb + b_row[j] + cofs[kk]);
#pragma unroll
            for (int i = 0; i < FM; ++i)
                fa[i] = *reinterpret_cast<const bf16x8_t*>(pa + a_row[i] + cofs[kk]);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i],
                                                                        acc[i][j], 0, 0, 0);
        }
        ua = ua + 1 == NA ? 0 : ua + 1;
        ub = ub + 1 == NB ? 0 : ub + 1;
    }

    // epilogue: bf16 rows staged in LDS (lane: token row l32, columns 8 g + 4 hi .. + 3 of each
    // 32-column fragment), then whole rows stored with 16-byte stores
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        char* const rowp = sm + (wm * (TM / WM) + 32 * i + l32) * PITCH + hi * 8;
#pragma unroll
        for (int j = 0; j < ((MODE == 0) ? FN / 2 : FN); ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float a0 = acc[i][j][4 * g + r];
                    v[r] = (MODE == 0) ? silu(a0) * acc[i][j + FN / 2][4 * g + r] : a0;
                }
                const int col = wn * WC + j * 32 + g * 8;
                const u32x2_t pk = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                *reinterpret_cast<u32x2_t*>(rowp + col * 2) = pk;
            }
    }
    __syncthreads();
    constexpr int CPR = OUTC * 2 / 16;  // 16-byte chunks per row
    constexpr int RPI = 256 / CPR;      // rows per pass of the block
    const int cc = tid % CPR, r0 = tid / CPR;
    const int ldc = (MODE == 0) ? m : d;
    const int col = ntile * OUTC + cc * 8;
    if (MODE == 1 && col >= d) return;
    bf16_t* const dst = C + (int64_t)row0 * ldc + col;
#pragma unroll
    for (int b = 0; b < TM / RPI; ++b) {
        const int r = r0 + b * RPI;
        if (r < rows)
            *reinterpret_cast<u32x4_t*>(dst + (int64_t)r * ldc) =
                *reinterpret_cast<const u32x4_t*>(sm + r * PITCH + cc * 16);
    }
}

template <int MODE, bool DMA>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_bf16_mid(
    const bf16_t* __restrict__ A, const int* __restrict__ row_token,
    const bf16_t* __restrict__ B, const int* __restrict__ offsets,
    const int* __restrict__ tile_off, int N, int d, int m, bf16_t* __restrict__ C) {
    __shared__ __attribute__((aligned(1024))) char sm[5 * 128 * 128];
    const int nt_count = (MODE == 0) ? m / 64 : (d + BN - 1) / BN;
    // block -> (expert, N-tile, M-tile innermost), XCD-contiguous (xcd_tile with one column)
    int L, unused;
    if (!xcd_tile(blockIdx.x, tile_off[N] * nt_count, 1, L, unused)) return;
    int e, first, tiles, row0, end;
    find_expert(tile_off, offsets, N, L, nt_count, e, first, tiles, row0, end);
    const int ntile = (L - first) / tiles;
    row0 += (L - first - ntile * tiles) * BM;
    const int left = end - row0;
    const int rot = (int)((int64_t)ntile * (((MODE == 0) ? d : m) / 64) / nt_count);
    if (left <= 64)
        gemm_mid_body<MODE, 64, BN, 2, DMA>(A, row_token, B, e, row0, left, ntile, rot, d, m, C,
                                            sm, tiles == 1);
    else
        gemm_mid_body<MODE, 128, BN, 2, DMA>(A, row_token, B, e, row0, left < BM ? left : BM,
                                             ntile, rot, d, m, C, sm, tiles == 1);
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel with LDS DMA: 256 x 256 block tile, k-tiles of 64, 4 waves (2 x 2) of
// 128 x 128, v_mfma_f32_32x32x16_bf16, one block per CU (the copy ring takes all 160 KB of LDS).
//
// Copies: global_load_lds_dwordx4 (no staging registers, no ds_write).  Each copy
// instruction moves 8 rows x 128 bytes, one whole cache line per row (full lines move more
// bytes per request than half lines).  While an expert has few M-tiles its weight copies can
// carry the non-temporal hint: each weight tile is read by one or two tiles, close together in
// time, and streaming it keeps the caches for the token rows and for the other GEMM's operands
// (measured with two tiles in step: down GEMM -8 %, gate/up unchanged); with more tiles, or tiles
// that do not keep step, it costs more than it saves (gemm_dma_body has the rule).
// The A half (token rows) and the B half (weight rows) of a k-tile
// are separate 32 KB units of a 5-unit ring; the B half, which usually misses to HBM, is
// issued two k-tiles ahead of its use and the A half one k-tile ahead.  LDS rows are
// unpadded (128 B) with their eight 16-byte chunks XOR-swizzled per row so that the 16
// lanes of one ds_read_b128 pass (16 consecutive rows, same logical chunk) hit distinct banks.
//
// MFMA operands are swapped (weights as the first operand): each accumulator tile is then the
// transpose of the output tile, so a lane holds 4 consecutive output columns of one token row
// per group of 4 registers.  The epilogue writes them (bf16, 8 bytes per lane) into a padded
// row-major tile in LDS and the block then stores whole rows with 16-byte coalesced stores.
// ------------------------------------------------------------------------------------------
constexpr int LBM = 256, LBN = 256;

// Remainder rows of the large-tile GEMM (TilePlan): for each expert e in tail_list, the
// 1..kTailRows rows past its last full M-tile, by extra blocks at the end of the grid, one per
// (listed expert, task) of gemm_stream.h.  The 4 waves split the contraction's 64-deep stages
// four ways; the partial tiles are summed in LDS in a fixed order and wave 0 stores them.
template <int MODE, int MT>
__device__ __forceinline__ void tail_task(const bf16_t* const (&wp)[SK_NF],
                                          const bf16_t* const (&xp)[2], int s0, int s1,
                                          int rows, int64_t out_row0, int out_ld, int out_col,
                                          bf16_t* __restrict__ C, char* lds) {
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    f32x4_t acc[MT][SK_NF];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int f = 0; f < SK_NF; ++f) acc[t][f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (s1 > s0) stream_mma<MT, 2>(wp, xp, s0, s1, acc);
    f32x4_t* r4 = reinterpret_cast<f32x4_t*>(lds);  // [wave][t][f][lane]
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int f = 0; f < SK_NF; ++f) r4[((w * MT + t) * SK_NF + f) * 64 + lane] = acc[t][f];
    __syncthreads();
    if (w != 0) return;  // no barrier follows
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int f = 0; f < SK_NF; ++f) {
            f32x4_t v = r4[(t * SK_NF + f) * 64 + lane];
#pragma unroll
            for (int ww = 1; ww < 4; ++ww) v += r4[((ww * MT + t) * SK_NF + f) * 64 + lane];
            acc[t][f] = v;
        }
    stream_store<MODE, MT>(acc, rows, out_row0, out_ld, out_col, C, lane);
}

template <int MODE>
__device__ __forceinline__ void tail_block(const bf16_t* __restrict__ A,
                                           const int* __restrict__ row_token,
                                           const bf16_t* __restrict__ B,
                                           const int* __restrict__ offsets,
                                           const int* __restrict__ tail_list, int task, int d,
                                           int m, int tile_rows, bf16_t* __restrict__ C,
                                           char* lds) {
    const int per_e = (MODE == 0) ? m / 32 : d / 64;
    const int i = task / per_e, c = task - i * per_e;
    if (i >= tail_list[0]) return;  // block-uniform, before any barrier
    const int e = tail_list[1 + i];
    const int ce = offsets[e + 1] - offsets[e];
    const int full = ce / tile_rows * tile_rows;
    const int rows = ce - full;  // 1..kTailRows (32) by the plan
    const int row0 = offsets[e] + full;
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int ns = ((MODE == 0) ? d : m) / 64;
    const int s0 = ns * w / 4, s1 = ns * (w + 1) / 4;
    const bf16_t* wp[SK_NF];
    const bf16_t* xp[2];
    stream_task<MODE, 2>(A, row_token, B, e, c, row0, rows, d, m, lane, wp, xp);
    const int out_ld = (MODE == 0) ? m : d;
    const int out_col = (MODE == 0) ? 32 * c : 64 * c;
    if (rows <= 16) tail_task<MODE, 1>(wp, xp, s0, s1, rows, row0, out_ld, out_col, C, lds);
    else tail_task<MODE, 2>(wp, xp, s0, s1, rows, row0, out_ld, out_col, C, lds);
}

// One 256 x 256 tile.  NTW: the weight copies carry the non-temporal hint (the kernel below picks
// it); ROT: the contraction starts at its k-tile rot (see the pipeline), else at 0.
template <int MODE, bool NTW, bool ROT>
__device__ __forceinline__ void gemm_dma_tile(const bf16_t* __restrict__ A,
                                              const int* __restrict__ row_token,
                                              const bf16_t* __restrict__ B, int e, int ntile,
                                              int row0, int rows, int rot, int d, int m,
                                              bf16_t* __restrict__ C, char* sm_bytes) {
    constexpr int TM = 256, TN = 256, TK = 64;
    constexpr int UNIT = TM * TK;  // elements of one ring unit: the A or the B half of a k-tile
    constexpr int NU = 5;          // units in the ring
    constexpr int OUTC = (MODE == 0) ? 128 : TN;  // output columns of the block
    constexpr int PITCH = OUTC * 2 + 16;          // bytes per row of the staged output tile
    static_assert(TM == TN && TM * PITCH <= NU * UNIT * 2, "staging tile exceeds LDS");
    bf16_t* const sm = reinterpret_cast<bf16_t*>(sm_bytes);
    const int Kd = (MODE == 0) ? d : m;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
    const int wm = wid >> 1, wn = wid & 1;

    // Copy sources: wave w copies rows [64w, 64w + 64) of each tile, 8 rows (1 KB) per
    // instruction; lane l fills physical chunk l & 7 of row 64w + 8i + (l >> 3), so it
    // fetches that row's logical chunk swz8(row, l & 7) (the XOR is its own inverse).
    // The copy instruction adds a 32-bit per-lane byte offset to a 64-bit scalar base, so the
    // bases are per block: the expert's weight matrix, and in the down GEMM the tile's first
    // H row.  The offsets then stay below one expert's weights (2 m d or d m elements) or 256
    // H rows; only the gathered x rows of the gate/up GEMM are addressed from x itself, and
    // gemm_tile_rows sends a problem to this kernel only when T d elements take less than
    // 2^32 bytes.
    const bf16_t* const Ablk = (MODE == 0) ? A : A + (int64_t)row0 * m;
    const bf16_t* const Bblk = B + (int64_t)e * ((MODE == 0) ? 2 * m : d) * Kd;
    uint32_t a_off[8], b_off[8];  // element offsets of each row's chunk (k = 0)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = 64 * wid + 8 * i + (lane >> 3);
        const int c = swz8(r, lane & 7);
        const int rr = r < rows ? r : rows - 1;  // rows past the expert's end: clamp, unused
        if (MODE == 0) {
            a_off[i] = (uint32_t)row_token[row0 + rr] * (uint32_t)d + c * 8;
            const int hc = ntile * 128;
            const int brow = (r < 128) ? (hc + r) : (m + hc + (r - 128));
            b_off[i] = (uint32_t)brow * (uint32_t)d + c * 8;
        } else {
            a_off[i] = (uint32_t)rr * (uint32_t)m + c * 8;
            int brow = ntile * TN + r;
            brow = brow < d ? brow : d - 1;
            b_off[i] = (uint32_t)brow * (uint32_t)m + c * 8;
        }
    }
    // LDS byte address of this wave's first 8-row group in unit 0
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)sm_bytes +
                          (uint32_t)__builtin_amdgcn_readfirstlane(wid * 64 * TK * 2);
    // The copies are inline assembly: the compiler cannot tell which unit a copy writes, and
    // would otherwise wait for every copy in flight before each LDS read.  Waits are explicit
    // (ELB_WAIT_VMCNT); M0 carries the LDS destination and is set in the same statement.
    // Each call is 8 copy instructions per wave.
    // copy instruction i (of 8) of a unit; nt: the non-temporal hint (the weight copies when
    // NTW)
    auto issue_one = [&](const bf16_t* src, const uint32_t (&off)[8], int unit, int k0, bool nt,
                         int i) {
        const uint32_t la = lds0 + (uint32_t)unit * (UNIT * 2) + i * 1024;
        const uint32_t va = (off[i] + k0) * 2u;
        if (nt)
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                         :: "s"(la), "v"(va), "s"(src) : "memory", "m0");
        else
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(la), "v"(va), "s"(src) : "memory", "m0");
    };
    auto issue = [&](const bf16_t* src, const uint32_t (&off)[8], int unit, int k0, bool nt) {
#pragma unroll
        for (int i = 0; i < 8; ++i) issue_one(src, off, unit, k0, nt, i);
    };

    // fragment rows (element offsets inside a stage)
    const int l32 = lane & 31;
    const int hi = lane >> 5;
    int a_frag[4], b_frag[4];
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) a_frag[mi] = (wm * 128 + mi * 32 + l32) * TK;
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) {
        const int br = (MODE == 0) ? ((ni < 2) ? (wn * 64 + ni * 32) : (128 + wn * 64 + (ni - 2) * 32))
                                   : (wn * 128 + ni * 32);
        b_frag[ni] = (br + l32) * TK;
    }
    // element offset of the chunk this lane reads for k16-step kk (k = 16 kk .. 16 kk + 15);
    // fragment rows are l32 mod 16 modulo 16, so the swizzle depends on l32 only
    int cofs[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) cofs[kk] = swz8(l32, 2 * kk + hi) * 8;

    f32x16_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;

    // Two fragment register sets: the 8 LDS reads of the next k16-step are issued between
    // the first 8 of the 16 MFMAs of the current one, which run on the other set.
    bf16x8_t fa0[4], fb0[4], fa1[4], fb1[4];
    auto load = [&](bf16x8_t (&fa)[4], bf16x8_t (&fb)[4], int ua, int ub, int kk) {
        const bf16_t* sa = sm + ua * UNIT + cofs[kk];
        const bf16_t* sb = sm + ub * UNIT + cofs[kk];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            fa[i] = *reinterpret_cast<const bf16x8_t*>(sa + a_frag[i]);
            fb[i] = *reinterpret_cast<const bf16x8_t*>(sb + b_frag[i]);
        }
    };
    auto mma = [&](const bf16x8_t (&fa)[4], const bf16x8_t (&fb)[4], bool reads) {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ni], fa[mi], acc[mi][ni], 0, 0, 0);
        if (reads) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
        }
    };

    // Pipeline: the B half of k-tile t lives in unit 2t mod 5, its A half in unit 2t + 1
    // mod 5.  Once the fourth k16-step's fragments of tile t are read (after the second
    // step's MFMAs) each wave waits for its own copies of tile t + 1 and for its own LDS
    // reads; the barrier then makes tile t + 1 visible to every wave and frees tile t's two
    // units (every read of them has completed), which receive the A half of tile t + 2 and the
    // B half of tile t + 3 while the third and fourth steps' MFMAs run.  Copies complete in
    // order and each half is 8 instructions per wave; the only copies issued after tile
    // t + 1's are those of B(t + 2), so the wait is vmcnt <= 8 (0 near the end).
    // A bare s_barrier, not __syncthreads(): the latter's fence would make the compiler drain
    // every copy in flight.
    //
    // Rotation: an expert with one M-tile has its weights read once, and the kernel waits on that
    // stream; its odd N-tiles then start in the middle of the contraction and wrap around, so
    // that blocks do not all walk the same columns of rows a multiple of 1 KB apart, i.e. the
    // same part of the memory channels (OLMoE-shaped layer, us: 1024 tokens 239 -> 221, 1600
    // tokens 250 -> 237, 1900 tokens 263 -> 257).  More starting points (4 or 8) cost part of
    // that again from 1600 tokens on (245, 242): the N-tiles share the token rows through L2, and
    // the rows of every point in use have to fit there.  With more M-tiles, where the weights are
    // shared too, all blocks stay in step (4096 tokens with 8 points: 447 -> 466 us).
    const int nk = Kd / TK;  // >= 1
    auto k_of = [&](int t) {
        if (!ROT) return t * TK;
        return (t + rot < nk ? t + rot : t + rot - nk) * TK;
    };
    // as if barriers at t = -3, -2, -1 had issued B(0); A(0), B(1); A(1), B(2)
    issue(Bblk, b_off, 0, k_of(0), NTW);
    issue(Ablk, a_off, 1, k_of(0), false);
    if (nk > 1) {
        issue(Bblk, b_off, 2, k_of(1), NTW);
        issue(Ablk, a_off, 3, k_of(1), false);
        if (nk > 2) {
            issue(Bblk, b_off, 4, k_of(2), NTW);
            ELB_WAIT_VMCNT(24);
        } else {
            ELB_WAIT_VMCNT(16);
        }
    } else {
        ELB_WAIT_VMCNT(0);
    }
    __builtin_amdgcn_s_barrier();
    int ub = 0, ua = 1;  // units of tile t
    load(fa0, fb0, ua, ub, 0);
    int t = 0;
    for (; t < nk - 1; ++t) {
        const int ub1 = ub + 2 >= NU ? ub + 2 - NU : ub + 2;  // units of tile t + 1
        const int ua1 = ua + 2 >= NU ? ua + 2 - NU : ua + 2;
        const int ka = k_of(t + 2), kb = k_of(t + 3);
        load(fa1, fb1, ua, ub, 1);
        mma(fa0, fb0, true);
        load(fa0, fb0, ua, ub, 2);
        mma(fa1, fb1, true);
        load(fa1, fb1, ua, ub, 3);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 2 < nk) ELB_WAIT_VMCNT(8);
        else ELB_WAIT_VMCNT(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // k16-steps 2 and 3 (32 MFMAs), with one of the 16 copy instructions of A(t + 2) and
        // B(t + 3) after every other MFMA: a copy that cannot issue at once then holds up one
        // MFMA slot, not a burst of them.  The next tile's step-0 reads go between the steps.
#pragma unroll
        for (int q = 0; q < 32; ++q) {
            const int mi = (q & 15) >> 2, ni = q & 3;
            if (q < 16)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb0[ni], fa0[mi],
                                                                      acc[mi][ni], 0, 0, 0);
            else
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb1[ni], fa1[mi],
                                                                      acc[mi][ni], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (q == 15) {
                load(fa0, fb0, ua1, ub1, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if ((q & 1) == 1) {
                const int i = q >> 1;
                if (i < 8) {
                    if (t + 2 < nk) issue_one(Ablk, a_off, ub, ka, false, i);  // -> unit 2t
                } else {
                    if (t + 3 < nk) issue_one(Bblk, b_off, ua, kb, NTW, i - 8);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        ub = ub1;
        ua = ua1;
    }
    {   // last k-tile
        load(fa1, fb1, ua, ub, 1);
        mma(fa0, fb0, true);
        load(fa0, fb0, ua, ub, 2);
        mma(fa1, fb1, true);
        load(fa1, fb1, ua, ub, 3);
        mma(fa0, fb0, true);
        mma(fa1, fb1, false);
    }

    // Epilogue through LDS: every wave is past its last LDS read of the stages.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    char* const stg = sm_bytes;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
        char* const rowp = stg + (wm * 128 + mi * 32 + l32) * PITCH + hi * 8;
#pragma unroll
        for (int ni = 0; ni < ((MODE == 0) ? 2 : 4); ++ni)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float a0 = acc[mi][ni][4 * g + r];
                    v[r] = (MODE == 0) ? silu(a0) * acc[mi][ni + 2][4 * g + r] : a0;
                }
                const int col = ((MODE == 0) ? wn * 64 : wn * 128) + ni * 32 + g * 8;
                u32x2_t pk = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                *reinterpret_cast<u32x2_t*>(rowp + col * 2) = pk;
            }
    }
    __syncthreads();
    // each thread stores one fixed 16-byte column chunk of every RPI-th row
    constexpr int CPR = OUTC * 2 / 16;  // 16-byte chunks per row
    constexpr int RPI = 256 / CPR;      // rows per pass of the block
    const int cc = tid % CPR, r0 = tid / CPR;
    const int ldc = (MODE == 0) ? m : d;
    const int col = ntile * OUTC + cc * 8;
    const bool col_ok = (MODE == 0) || col < d;
    const char* src = stg + r0 * PITCH + cc * 16;
    bf16_t* dst = C + (int64_t)(row0 + r0) * ldc + col;
#pragma unroll
    for (int b = 0; b < TM / RPI; b += 16) {
        u32x4_t v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i)
            v[i] = *reinterpret_cast<const u32x4_t*>(src + (b + i) * RPI * PITCH);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (col_ok && r0 + (b + i) * RPI < rows)
                *reinterpret_cast<u32x4_t*>(dst + (int64_t)(b + i) * RPI * ldc) = v[i];
    }
}

// NTOK: weight copies may carry the non-temporal hint (a form of its own without: tested in the
// kernel, the batches that never use it ran 0.3 % slower)
template <int MODE, bool NTOK>
__device__ __forceinline__ void gemm_dma_body(
    const bf16_t* __restrict__ A, const int* __restrict__ row_token,
    const bf16_t* __restrict__ B, const int* __restrict__ offsets,
    const int* __restrict__ tile_off, const int* __restrict__ tail_list, int big_blocks,
    int N, int d, int m, bf16_t* __restrict__ C, char* sm_bytes) {
    constexpr int TM = 256, TN = 256, TK = 64;
    if ((int)blockIdx.x >= big_blocks) {  // the remainder blocks after the tiles
        tail_block<MODE>(A, row_token, B, offsets, tail_list, (int)blockIdx.x - big_blocks, d,
                         m, TM, C, sm_bytes);
        return;
    }

    const int nt_count = (MODE == 0) ? m / 128 : (d + TN - 1) / TN;
    int tile, ntile;
    if (!xcd_tile(blockIdx.x, tile_off[N] * nt_count, nt_count, tile, ntile)) return;
    int e, row0, rows, tiles, last;
    find_tile(tile_off, offsets, N, tile, TM, e, row0, rows, tiles, last);

    const int Kd = (MODE == 0) ? d : m;
    const int rot = tiles == 1 && (ntile & 1) ? Kd / TK / 2 : 0;  // see the pipeline below
    // An expert's last tile with at most 128 rows: the smaller tile forms of the mid-sized kernel,
    // as wide as this one's, 3 x (16 + 32) KB of LDS at most (64 rows: per k-tile 40 KB copied and
    // 64 KB read instead of 64 and 128, and a quarter of the MFMAs).  Taken in order: all of them
    // after the full tiles would balance the units better, but reads their experts' weights from
    // HBM again (3000 tokens 391 -> 439, 4096 top-8 496 -> 490).
    //
    // The non-temporal hint (where NTOK allows it) goes to the weights of experts with one
    // tile, which nobody else reads, and with two tiles of the full form, which walk the weights
    // in step.  A short tile does not keep step with the full one beside it, and three tiles
    // drift apart: with the hint the tile that comes first leaves nothing in L2 for the others,
    // and each of them reads HBM.  OLMoE-shaped layer, us, all tiles of the full form / short
    // forms, every tile with the hint / this rule: top-8 2048 tokens 310 / 307 / 297, 2300 387 /
    // 378 / 347, 2816 388 / 381 / 366, 3000 391 / 395 / 388, 4500 577 / 573 / 546, 5000 596 / 606 /
    // 588, elbow 2300 379 / 359 / 335, 3000 389 / 381 / 367; 8192 top-8 and 16384 tokens, which
    // have no hint, 939 / 898 and 1605 / 1579.  (Two full tiles without the hint: 3500 tokens
    // top-8 404 -> 411.)
    const bool nt = NTOK && (tiles == 1 || (tiles == 2 && last > 128));
    if (rows <= 128) {
        if (rows <= 64)
            gemm_mid_body<MODE, 64, TN, 1>(A, row_token, B, e, row0, rows, ntile, rot, d, m, C,
                                           sm_bytes, nt);
        else
            gemm_mid_body<MODE, 128, TN, 2>(A, row_token, B, e, row0, rows, ntile, rot, d, m, C,
                                            sm_bytes, nt);
        return;
    }
    // (rotation and hint are forms of their own: the wrap cost the loop 0.5 % at 4096 tokens)
    if (rot) {
        if (nt)
            gemm_dma_tile<MODE, true, true>(A, row_token, B, e, ntile, row0, rows, rot, d, m, C,
                                            sm_bytes);
        else
            gemm_dma_tile<MODE, false, true>(A, row_token, B, e, ntile, row0, rows, rot, d, m, C,
                                             sm_bytes);
    } else {
        if (nt)
            gemm_dma_tile<MODE, true, false>(A, row_token, B, e, ntile, row0, rows, 0, d, m, C,
                                             sm_bytes);
        else
            gemm_dma_tile<MODE, false, false>(A, row_token, B, e, ntile, row0, rows, 0, d, m, C,
                                              sm_bytes);
    }
}

template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_dma(
    const bf16_t* __restrict__ A, const int* __restrict__ row_token,
    const bf16_t* __restrict__ B, const int* __restrict__ offsets,
    const int* __restrict__ tile_off, const int* __restrict__ tail_list, int big_blocks,
    int N, int d, int m, bf16_t* __restrict__ C, int nt_weights) {
    // One array: its address is passed to the copy instructions (inline assembly), which tells
    // the compiler that all of it may be written there.
    __shared__ __attribute__((aligned(1024))) char sm_bytes[5 * 256 * 64 * 2];
    if (nt_weights)  // kernel-uniform
        gemm_dma_body<MODE, true>(A, row_token, B, offsets, tile_off, tail_list, big_blocks, N,
                                  d, m, C, sm_bytes);
    else
        gemm_dma_body<MODE, false>(A, row_token, B, offsets, tile_off, tail_list, big_blocks, N,
                                   d, m, C, sm_bytes);
}

// ------------------------------------------------------------------------------------------
// fp32 kernel: 64 x 64 block tile, k-tiles of 32 (128 bytes of a row), 4 waves (2 x 2) of
// 32 x 32 on v_mfma_f32_16x16x4_f32 (fp32 products and sums; the weights first, so a lane ends
// with 4 consecutive output columns of a token row)
//
// The matrix units bound it: 157 TFLOP/s nominal, twice the vector units' rate, against which
// the LDS traffic of even this small tile is a quarter (16 KB copied and 32 KB read per k-tile
// of 1024 matrix cycles).  So the tile is small, for the small layers that run in fp32: more
// blocks to spread (three per CU), little padding.  Copies global -> LDS, three units deep, chunks
// XOR-swizzled, as in the bf16 kernels.  An operand read is 16 bytes, four k of one row; the
// four MFMAs of a 16-deep step each take one of the four from every lane, a permutation of the
// contraction that both operands share.
// Measured against 64 x 64 x 16 vector tiles (gate/up + down us): 1500 tokens, d = 1024, 16
// experts, m = 528, K = 4: 236 + 105 -> 132 + 63; 2048 tokens, d = 1024, 32 experts, m = 640,
// K = 8: 543 + 259 -> 333 + 168 (121 TFLOP/s without the padding in gate/up); the error against
// 64 bits is the same (5.5e-8 and 4.2e-7 of the layer's output before and after).
// ------------------------------------------------------------------------------------------
constexpr int FBM = 64, FBN = 64, FBK = 32;

template <int MODE, bool DMA>
__global__ __launch_bounds__(256) void gemm_f32(const float* __restrict__ A,
                                                const int* __restrict__ row_token,
                                                const float* __restrict__ B,
                                                const int* __restrict__ offsets,
                                                const int* __restrict__ tile_off, int N, int d,
                                                int m, float* __restrict__ C) {
    constexpr int UNIT = 64 * FBK * 4, NU = 3;  // bytes of a unit (64 rows), units per operand
    __shared__ __attribute__((aligned(1024))) char sm[2 * NU * UNIT];
    const int nt_count = (MODE == 0) ? (m + 31) / 32 : (d + FBN - 1) / FBN;
    int tile, ntile;
    const int block = blockIdx.y * kTileGridRow + blockIdx.x;
    if (!xcd_tile(block, tile_off[N] * nt_count, nt_count, tile, ntile)) return;
    int e, row0, rows, tiles, last;
    find_tile(tile_off, offsets, N, tile, FBM, e, row0, rows, tiles, last);
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wid >> 1, wn = wid & 1;
    const int Kd = (MODE == 0) ? d : m;
    const int nout = (MODE == 0) ? m : d;  // output columns of this GEMM
    const int nk = (Kd + FBK - 1) / FBK;
    const bool half = Kd % FBK != 0;  // the last k-tile has 16 columns (d and m are % 16)

    // copy sources: wave w copies rows [16 w, 16 w + 16) of each unit, 8 rows per instruction;
    // lane l fills physical chunk l & 7 of row 8 i + (l >> 3) with that row's logical chunk (of
    // a half k-tile: one of its four, the upper half is never read)
    const char* a_src[2];
    const char* b_src[2];
    int chunk[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 16 * wid + 8 * i + (lane >> 3);
        chunk[i] = swz8(r, lane & 7) * 16;
        const int rr = r < rows ? r : rows - 1;  // rows past the tile's end: never stored
        const int64_t ar = (MODE == 0) ? (int64_t)row_token[row0 + rr] : (int64_t)(row0 + rr);
        a_src[i] = reinterpret_cast<const char*>(A + ar * Kd);
        int col = (MODE == 0) ? ntile * 32 + (r & 31) : ntile * FBN + r;
        col = col < nout ? col : nout - 1;  // columns past the end: never stored
        const int64_t br = (MODE == 0) ? (int64_t)e * 2 * m + (r < 32 ? col : m + col)
                                       : (int64_t)e * d + col;
        b_src[i] = reinterpret_cast<const char*>(B + br * Kd);
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(lds_void_t*)sm + (uint32_t)wid * 2048);
    auto issue = [&](int t, int unit) {
        const int mask = half && t == nk - 1 ? 63 : 127;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t la = lds0 + (uint32_t)unit * UNIT + i * 1024;
            const int64_t o = (int64_t)t * (FBK * 4) + (chunk[i] & mask);
            const char* const va = a_src[i] + o;
            const char* const vb = b_src[i] + o;
            if constexpr (!DMA) {
                char* const at = sm + unit * UNIT + wid * 2048 + i * 1024 + lane * 16;
                copy16_any(at, va);
                copy16_any(at + NU * UNIT, vb);
                continue;
            }
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                         :: "s"(la), "v"(va) : "memory", "m0");
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
                         :: "s"(la + NU * UNIT), "v"(vb) : "memory", "m0");
        }
    };

    const int l16 = lane & 15, hq = lane >> 4;
    int a_at[2], b_at[2], cofs[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        a_at[i] = (32 * wm + 16 * i + l16) * 128;
        b_at[i] = NU * UNIT + ((MODE == 0 ? 32 * i + 16 * wn : 32 * wn + 16 * i) + l16) * 128;
        cofs[i] = swz8(l16, 4 * i + hq) * 16;  // rows 16 apart swizzle alike
    }
    f32x4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto step = [&](const char* p, int ks) {
        f32x4_t fa[2], fb[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            fa[i] = *reinterpret_cast<const f32x4_t*>(p + a_at[i] + cofs[ks]);
            fb[i] = *reinterpret_cast<const f32x4_t*>(p + b_at[i] + cofs[ks]);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][c], fa[i][c],
                                                                     acc[i][j], 0, 0, 0);
    };

    // at the barrier that opens k-tile t every wave has read tile t - 1, whose unit receives
    // tile t + 2; the wait before it leaves tile t + 1's four copies in flight
    const bool any = 32 * wm < rows;  // wave-uniform: a short tile's upper waves only copy
    issue(0, 0);
    if (nk > 1) issue(1, 1);
    int u = 0;
    for (int t = 0; t < nk; ++t) {
        if (t + 1 < nk) ELB_WAIT_VMCNT(4);
        else ELB_WAIT_VMCNT(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (t + 2 < nk) issue(t + 2, u + 2 >= NU ? u + 2 - NU : u + 2);
        if (any) {
            const char* const p = sm + u * UNIT;
            step(p, 0);
            if (!(half && t == nk - 1)) step(p, 1);
        }
        u = u + 1 == NU ? 0 : u + 1;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 32 * wm + 16 * i + l16;
        if (r >= rows) continue;
        float* const dst = C + (int64_t)(row0 + r) * nout;
        if (MODE == 0) {
            const int col = ntile * 32 + 16 * wn + 4 * hq;
            f32x4_t v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = silu(acc[i][0][q]) * acc[i][1][q];
            if (col < nout) *reinterpret_cast<f32x4_t*>(dst + col) = v;
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int col = ntile * FBN + 32 * wn + 16 * j + 4 * hq;
                if (col < nout) *reinterpret_cast<f32x4_t*>(dst + col) = acc[i][j];
            }
        }
    }
}

unsigned grid8(int64_t blocks) { return (unsigned)((blocks + 7) / 8 * 8); }
// the fp32 kernel's grid: its blocks write 8 KB of H, so 137 GB of it are 2^24 blocks (the bf16
// kernels' blocks write 16 KB or more, and theirs fit one dimension)
dim3 grid_f32(int64_t blocks) {
    const TileGrid g = tile_grid(blocks);
    return dim3(g.x, g.y);
}

}  // namespace

int gemm_tile_rows(int dtype, int64_t T, int K, int N, int d, int m, bool aligned) {
    if (dtype != ELB_BF16) return FBM;
    const int64_t avg_rows = T * K / (N > 0 ? N : 1);
    // the large-tile kernel's 32-bit byte offsets: gathered x rows from x itself (T d
    // elements), weights from the expert's own matrix (2 m d elements); larger problems take
    // the 128-row kernel, which addresses with 64-bit pointers
    const bool offsets_fit = (uint64_t)T * (uint64_t)d * 2u < ((uint64_t)1 << 32) &&
                             (uint64_t)m * (uint64_t)d * 4u < ((uint64_t)1 << 32);
    // Which tiles are faster, measured on whole layers (us, 128-row kernel / this one).
    // Rows per expert, OLMoE-shaped: 98 179 / 227, 113 204 / 231, 128 231 / 231, 143 250 / 236;
    // with d = 2560, m = 1536 at 120 rows 404 / 380.  From some 112 rows on many experts need two
    // 128-row tiles, and the second pass over the weights costs what the finer tiles gain.
    // Few large tiles leave compute units idle (one block each): about (T K + 128 N) / 256
    // M-tiles times m / 128 blocks in gate/up.  90 blocks 46 / 66, 96 75 / 94, 120 48 / 66; at
    // 157 and 160 58 / 69 and 111 / 98; at 216 and more within 5 % either way.  So this kernel
    // needs more than 128 blocks, half of the compute units.
    const int64_t blocks = (T * K + (int64_t)N * 128) / 256 * (m / 128);
    return (m % 128 == 0 && d >= 128 && T > 0 && avg_rows >= 112 && blocks > 128 &&
            offsets_fit && aligned) ? LBM : BM;
}

hipError_t launch_gemm_gate_up(const void* x, const void* Wgu, const int* row_token,
                               const int* offsets, const int* tile_off, const int* tail_list,
                               int64_t max_tiles, int tile_rows, int d, int N, int m,
                               int dtype, void* H, hipStream_t s, bool nt_weights) {
    if (max_tiles <= 0) return hipSuccess;
    if (dtype == ELB_BF16 && tile_rows == LBM) {
        ProfileScope prof("gemm_gate_up_bf16", s);
        const unsigned big = grid8(max_tiles * (m / 128));
        const unsigned tail = tail_list ? (unsigned)(kTailMax * (m / 32)) : 0u;
        ELB_LAUNCH(gemm_bf16_dma<0>, dim3(big + tail), dim3(256), 0, s,
                           (const bf16_t*)x, row_token, (const bf16_t*)Wgu, offsets, tile_off,
                           tail_list, (int)big, N, d, m, (bf16_t*)H, (int)nt_weights);
    } else if (dtype == ELB_BF16) {
        ProfileScope prof("gemm_gate_up_bf16_s", s);
        ELB_LAUNCH((aligned16(x, Wgu) ? gemm_bf16_mid<0, true> : gemm_bf16_mid<0, false>),
                   dim3(grid8(max_tiles * (m / 64))), dim3(256), 0, s, (const bf16_t*)x,
                   row_token, (const bf16_t*)Wgu, offsets, tile_off, N, d, m, (bf16_t*)H);
    } else {
        ProfileScope prof("gemm_gate_up_f32", s);
        ELB_LAUNCH((aligned16(x, Wgu) ? gemm_f32<0, true> : gemm_f32<0, false>),
                   grid_f32(max_tiles * ((m + 31) / 32)), dim3(256), 0, s, (const float*)x,
                   row_token, (const float*)Wgu, offsets, tile_off, N, d, m, (float*)H);
    }
    return hipGetLastError();
}

hipError_t launch_gemm_down(const void* H, const void* Wd, const int* offsets,
                            const int* tile_off, const int* tail_list, int64_t max_tiles,
                            int tile_rows, int d, int N, int m, int dtype, void* Y,
                            hipStream_t s, bool nt_weights) {
    if (max_tiles <= 0) return hipSuccess;
    if (dtype == ELB_BF16 && tile_rows == LBM) {
        ProfileScope prof("gemm_down_bf16", s);
        const unsigned big = grid8(max_tiles * ((d + LBN - 1) / LBN));
        const unsigned tail = tail_list ? (unsigned)(kTailMax * (d / 64)) : 0u;
        ELB_LAUNCH(gemm_bf16_dma<1>, dim3(big + tail), dim3(256), 0, s,
                           (const bf16_t*)H, (const int*)nullptr, (const bf16_t*)Wd, offsets,
                           tile_off, tail_list, (int)big, N, d, m, (bf16_t*)Y, (int)nt_weights);
    } else if (dtype == ELB_BF16) {
        ProfileScope prof("gemm_down_bf16_s", s);
        ELB_LAUNCH((aligned16(H, Wd) ? gemm_bf16_mid<1, true> : gemm_bf16_mid<1, false>),
                   dim3(grid8(max_tiles * ((d + BN - 1) / BN))), dim3(256), 0, s,
                   (const bf16_t*)H, (const int*)nullptr, (const bf16_t*)Wd, offsets, tile_off,
                   N, d, m, (bf16_t*)Y);
    } else {
        ProfileScope prof("gemm_down_f32", s);
        ELB_LAUNCH((aligned16(H, Wd) ? gemm_f32<1, true> : gemm_f32<1, false>),
                   grid_f32(max_tiles * ((d + FBN - 1) / FBN)), dim3(256), 0, s,
                   (const float*)H, (const int*)nullptr, (const float*)Wd, offsets, tile_off, N,
                   d, m, (float*)Y);
    }
    return hipGetLastError();
}

}  // namespace elb
