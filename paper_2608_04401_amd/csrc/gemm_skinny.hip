// Grouped expert GEMMs for decode-sized batches: weight streaming.
//
// With a few tokens per expert (T K / N of order 10) the expert GEMMs are matrix-vector
// products in disguise: every used expert's weights are read once from HBM and each weight
// is used for only a handful of FLOPs, so the kernels are bound by HBM bandwidth, not by the
// matrix cores.  The design follows from that:
//  - the weights are the streamed operand.  One block owns a task (expert e, a slice of 64
//    weight rows); its four waves take a quarter of the contraction each, in 64-deep stages.
//    A wave copies a stage (64 rows x 128 bytes, whole cache lines) into its own 8 KB of LDS
//    with global_load_lds_dwordx4, reads it into MFMA operand registers and lets the next
//    stage's copies run while it multiplies: no barrier in the loop, and the four blocks of a
//    CU keep up to 128 KB in flight;
//  - the quarters start at four different columns.  Weight rows lie a multiple of 1 KB or more
//    apart, so waves that all walk the same columns at the same time crowd onto part of the
//    memory channels: a read-only probe of this copy pattern over 537 MB reached 5.2 TB/s
//    with a wave on whole rows and 6.7-6.8 TB/s with the quarters (the same for 128 to 512
//    bytes of a row per instruction; half lines, as operand loads straight into registers
//    read them, reached 4.6);
//  - the expert's token rows are the small operand (chunks of up to 32 rows, 2 tiles of
//    16), read from L2, where the expert's other blocks also find them;
//  - v_mfma_f32_16x16x32_bf16 with the WEIGHTS as the first operand: the output tile is
//    (weight row) x (token), so a lane holds 4 consecutive output columns of one token row;
//    the four waves' partial tiles are summed in LDS in the order of the contraction;
//  - experts without tokens cost nothing: their blocks exit before any weight is read;
//  - gate/up: a task is 32 H columns, i.e. its 32 gate rows and the 32 matching up rows, so
//    SwiGLU is applied to the sums and H is written once (bf16); down: a task is 64 Y
//    columns.
// An expert with more than 32 rows is processed in chunks of 32 rows, re-reading its
// weights per chunk (rare where this path is chosen: at most 16 rows per expert on
// average).
//
// Block -> task mapping: tasks are numbered expert-major and each of the 8 XCDs (block b
// runs on XCD b % 8) takes a contiguous range of them, so an expert's token rows are shared
// through one XCD's L2.  With at most two slots per expert many experts have no token, and an
// XCD whose range holds few used ones is done early while another streams all of its own; then
// (`spread`) consecutive tasks go to consecutive XCDs, so that every XCD streams an eighth of
// each used expert.  OLMoE-shaped layer, us, ranges / spread: 8 tokens 109 / 94, 9 113 / 101, 10
// 114 / 108, 16 126 / 125; from there on the ranges are faster (20 tokens 128 / 129, 64 133 / 139).
// Small layers, whose time is not the stream's, lose by it (d = 2048, N = 8, m = 576: 29.8 / 30.5;
// d = 1024, N = 64, m = 768, 302 MB of weights: 54.2 / 54.7), so it takes twice the last-level
// cache of weights; and one token's experts are as many different ones, which the ranges deal out
// as evenly (33.1 / 33.8).
//
// Measured (OLMoE-shaped layer, T = 64, gate/up + down): 126 + 54 us with one wave per 64-row
// task loading operands straight into registers, 79 + 42 us (6.8 and 6.4 TB/s of weights, the
// probe's rates) in this form.  Eight or sixteen waves per task (shorter serial streams, fewer
// blocks per CU): 79 + 47 and 105 + 63 us.
#include "gemm_stream.h"

namespace elb {

namespace {

constexpr int SK_NW = 4;           // waves per block
constexpr int SK_MAXMT = 2;       // token tiles of 16 rows per chunk (32 rows)
constexpr int SK_STAGE = 64 * 128;  // bytes of one wave's stage: 64 weight rows x 64 bf16

// The assignment slots s = t K + j (j < k_t) routed to expert e, in increasing order (so in
// increasing token order, as the dispatch orders an expert's rows), gathered by the block's
// four waves into its LDS list; returns their number.  T K <= kSlotMax on this path, so each
// wave looks at 256 slots, with all its loads in flight at once.
constexpr int kSlotMax = 16 * ELB_MAX_EXPERTS;  // T K <= 16 N
__device__ __forceinline__ int gather_slots(const int* __restrict__ k,
                                            const int* __restrict__ ids, int T, int K, int e,
                                            int* list, int* wave_n, int lane, int w) {
    static_assert(kSlotMax <= SK_NW * 4 * kWave, "four 64-slot chunks per wave");
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int first = w * 4 * kWave;
    int id4[4], k4[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int slot = first + c * kWave + lane;
        id4[c] = (slot < T * K) ? ids[slot] : -1;
        k4[c] = (slot < T * K) ? k[slot / K] : 0;
    }
    uint64_t b[4];
    int n = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int slot = first + c * kWave + lane;
        b[c] = __ballot(id4[c] == e && slot - (slot / K) * K < k4[c]);
        n += __popcll(b[c]);
    }
    if (lane == 0) wave_n[w] = n;
    __syncthreads();
    int at = 0, total = 0;
#pragma unroll
    for (int q = 0; q < SK_NW; ++q) {
        if (q < w) at += wave_n[q];
        total += wave_n[q];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if ((b[c] >> lane) & 1) list[at + __popcll(b[c] & below)] = first + c * kWave + lane;
        at += __popcll(b[c]);
    }
    __syncthreads();
    return total;
}

// One chunk of up to 16 * MT token rows (assignment slots list[0 .. rows)) of a task.
// src[i] (i < 8): the task's weight rows 8 i .. 8 i + 7 at stage 0, off[i & 1]: the lane's byte
// offset from it.
// ring: this wave's stage; the block's four of them hold the partial sums afterwards.
template <int MODE, int MT, bool DMA>
__device__ __forceinline__ void skinny_chunk(const char* const (&src)[8],
                                             const uint32_t (&off)[2],
                                             int s0, int s1,
                                             const bf16_t* __restrict__ A, const int* list,
                                             int rows, int K, int d, int m, int out_col,
                                             bf16_t* __restrict__ C, char* ring_all, int lane,
                                             int w) {
    const int l16 = lane & 15, hq = lane >> 4;
    char* const ring = ring_all + w * SK_STAGE;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(lds_void_t*)ring_all + (uint32_t)w * SK_STAGE);
    const bf16_t* xp[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int r = 16 * t + l16;
        const int slot = list[r < rows ? r : rows - 1];  // past the chunk: never stored
        xp[t] = A + ((MODE == 0) ? (int64_t)(slot / K) * d : (int64_t)slot * m) + hq * 8;
    }
    // The copies are inline assembly, so that the compiler does not wait for them before LDS
    // reads it cannot tell apart; every wait for them is the explicit one below.
    auto issue = [&](int s) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t la = lds0 + i * 1024;
            const char* const base = src[i] + (int64_t)s * 128;
            if constexpr (!DMA) {
                copy16_any(ring + i * 1024 + lane * 16, base + off[i & 1]);
                continue;
            }
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                         :: "s"(la), "v"(off[i & 1]), "s"(base) : "memory", "m0");
        }
    };
    bf16x8_t x[MT][2];
    auto load_x = [&](int s) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                x[t][h] = *reinterpret_cast<const bf16x8_t*>(xp[t] + s * 64 + 32 * h);
    };
    f32x4_t acc[MT][SK_NF];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int f = 0; f < SK_NF; ++f) acc[t][f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (s1 > s0) {
        load_x(s0);
        issue(s0);
    }
    for (int s = s0; s < s1; ++s) {
        ELB_WAIT_VMCNT(0);  // stage s: this wave's own copies, and its token rows
        asm volatile("" ::: "memory");
        bf16x8_t wf[SK_NF][2], xs[MT][2];
#pragma unroll
        for (int f = 0; f < SK_NF; ++f)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int row = 16 * f + l16;
                wf[f][h] = *reinterpret_cast<const bf16x8_t*>(ring + row * 128 +
                                                              swz8(row, 4 * h + hq) * 16);
            }
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) xs[t][h] = x[t][h];
        // every read of the stage has returned before the next stage's copies overwrite it
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (s + 1 < s1) {
            load_x(s + 1);
            issue(s + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int f = 0; f < SK_NF; ++f)
                    acc[t][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[f][h], xs[t][h],
                                                                        acc[t][f], 0, 0, 0);
    }
    // partial tiles: each wave's own 8 KB holds its MT x 4 fragments of 1 KB
    static_assert(SK_MAXMT * SK_NF * 1024 <= SK_STAGE, "partial tiles exceed the stage");
    f32x4_t* const part = reinterpret_cast<f32x4_t*>(ring_all);
    auto at = [&](int ww, int t, int f) {
        return ww * (SK_STAGE / 16) + (t * SK_NF + f) * 64 + lane;
    };
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int f = 0; f < SK_NF; ++f) part[at(w, t, f)] = acc[t][f];
    __syncthreads();
    auto sum = [&](int t, int f) {
        f32x4_t v = part[at(0, t, f)];
#pragma unroll
        for (int ww = 1; ww < SK_NW; ++ww) v += part[at(ww, t, f)];
        return v;
    };
    // gate/up: wave w takes gate fragment w & 1 and its up fragment of token tile w / 2; down:
    // wave w takes fragment w of every token tile.  The lane holds token row l16 of the tile
    // and columns 16 f + 4 hq .. + 3 of the task.
    if (MODE == 0) {
        const int t = w >> 1, f = w & 1;
        const int r = 16 * t + l16;
        if (w < 2 * MT && r < rows) {
            const f32x4_t g = sum(t, f), u = sum(t, f + 2);
            const u32x2s_t pk = {
                stream_pack2(stream_silu(g[0]) * u[0], stream_silu(g[1]) * u[1]),
                stream_pack2(stream_silu(g[2]) * u[2], stream_silu(g[3]) * u[3])};
            bf16_t* const dst = C + (int64_t)list[r] * m + out_col + 16 * f + 4 * hq;
            *reinterpret_cast<u32x2s_t*>(dst) = pk;
        }
    } else {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const int r = 16 * t + l16;
            if (w < SK_NF && r < rows) {
                const f32x4_t v = sum(t, w);
                const u32x2s_t pk = {stream_pack2(v[0], v[1]), stream_pack2(v[2], v[3])};
                bf16_t* const dst = C + (int64_t)list[r] * d + out_col + 16 * w + 4 * hq;
                *reinterpret_cast<u32x2s_t*>(dst) = pk;
            }
        }
    }
}

// MODE 0: A = x [T, d], W = W_gate_up [N, 2m, d], C = H [T K, m]
// MODE 1: A = H [T K, m], W = W_down [N, d, m], C = Y [T K, d]
// Rows are assignment slots t K + j, found by each block from the routing itself (k, ids):
// no dispatch pass; every expert's blocks write their slots' rows of H and Y, and the combine
// reads row t K + j.  counts (optional): assignments per expert, by each expert's first task.
// With fewer slots than experts (T K < N) the tasks are numbered by slot instead of by expert:
// slot q's blocks take its expert if no earlier slot has it, so that a step of one sequence
// starts 8 experts' blocks and not 64 experts' of which 56 only find that they have no row
// (OLMoE-shaped layer, T = 1: layer 45.6 -> 33.3 us, T = 4: 93 -> 72 us; from T K = N on the
// two numberings start as many blocks).  The counts are then taken by the first block.
// spread: see above.
// DMA: the weights are 16-byte aligned (the token rows are loaded ordinarily); the form without
// holds a stage in registers on its way, for which two waves per SIMD leave room
template <int MODE, bool DMA>
__global__ __launch_bounds__(64 * SK_NW)
    __attribute__((amdgpu_waves_per_eu(DMA ? 4 : 2, DMA ? 4 : 2))) void gemm_skinny(
    const bf16_t* __restrict__ A, const int* __restrict__ k, const int* __restrict__ ids,
    int T, int K, const bf16_t* __restrict__ W, int N, int d, int m, int spread,
    bf16_t* __restrict__ C, int* __restrict__ counts) {
    __shared__ __attribute__((aligned(1024))) char ring[SK_NW * SK_STAGE];
    __shared__ int list[kSlotMax];
    __shared__ int wave_n[SK_NW];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_e = (MODE == 0) ? m / 32 : d / 64;  // tasks per expert
    const bool by_slot = T * K < N;
    const int tasks = (by_slot ? T * K : N) * per_e;
    const int per = (tasks + 7) >> 3;
    const int s = blockIdx.x >> 3;
    const int task = spread ? (int)blockIdx.x : (int)(blockIdx.x & 7) * per + s;
    if (s >= per || task >= tasks) return;  // block-uniform
    const int i_e = task / per_e, c = task - i_e * per_e;
    int e = i_e;
    if (by_slot) {
        if (counts && task == 0 && threadIdx.x < N) {
            int n = 0;
            for (int q = 0; q < T * K; ++q)
                n += ids[q] == (int)threadIdx.x && q - (q / K) * K < k[q / K];
            counts[threadIdx.x] = n;
        }
        e = (i_e - (i_e / K) * K < k[i_e / K]) ? ids[i_e] : -1;
        if (e < 0 || e >= N) return;
    }
    const int n = gather_slots(k, ids, T, K, e, list, wave_n, lane, w);
    if (!by_slot && counts && c == 0 && threadIdx.x == 0) counts[e] = n;
    if (n <= 0 || (by_slot && list[0] != i_e)) return;

    const int kd = (MODE == 0) ? d : m;
    const int ns = kd / 64;
    // lane l fills physical chunk l & 7 of row 8 i + (l >> 3), so it fetches that row's logical
    // chunk (swz8 is its own inverse, and the same for rows 16 apart)
    const char* src[8];
    const int64_t ew = (int64_t)e * ((MODE == 0) ? 2 * m : d);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = (MODE == 0) ? ((i < 4) ? 32 * c + 8 * i : m + 32 * c + 8 * (i - 4))
                                    : 64 * c + 8 * i;
        src[i] = reinterpret_cast<const char*>(W + (ew + row) * kd);
    }
    uint32_t off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        off[i] = ((uint32_t)(lane >> 3) * (uint32_t)kd +
                  swz8(8 * i + (lane >> 3), lane & 7) * 8) * 2u;
    const int s0 = ns * w / SK_NW, s1 = ns * (w + 1) / SK_NW;
    const int out_col = (MODE == 0) ? 32 * c : 64 * c;
    for (int cb = 0; cb < n; cb += 16 * SK_MAXMT) {
        const int rows = n - cb < 16 * SK_MAXMT ? n - cb : 16 * SK_MAXMT;
        if (cb) __syncthreads();  // the last chunk's partial sums have been read
        if (rows <= 16)
            skinny_chunk<MODE, 1, DMA>(src, off, s0, s1, A, list + cb, rows, K, d, m, out_col,
                                       C, ring, lane, w);
        else
            skinny_chunk<MODE, 2, DMA>(src, off, s0, s1, A, list + cb, rows, K, d, m, out_col,
                                       C, ring, lane, w);
    }
}

// Packing (elb_pack_expert_weights): one thread per 16-byte operand of the packed copy, in
// packed order (per task, 64-deep stage, 32-deep half and fragment the 64 lanes' operands),
// gathered from the row-major weights (gate/up then down; the copy has the same size).  The
// kernels above read the row-major weights as fast (T = 64: 134 us a layer, against 139 us
// with the same kernel reading the packed copy), so none reads the copy any more.
__global__ __launch_bounds__(256) void pack_experts(const bf16_t* __restrict__ Wgu,
                                                    const bf16_t* __restrict__ Wd, int N, int d,
                                                    int m, bf16_t* __restrict__ P) {
    const int64_t n_gu = (int64_t)N * 2 * m * d / 8;  // 16-byte operands of W_gate_up
    const int64_t n_all = n_gu + (int64_t)N * d * m / 8;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_all) return;
    const bool gu = i < n_gu;
    const int64_t j = gu ? i : i - n_gu;
    const int lane = (int)(j % 64);
    int64_t q = j / 64;
    const int f = (int)(q % 4);
    q /= 4;
    const int h = (int)(q % 2);
    q /= 2;
    const int ns = (gu ? d : m) / 64;
    const int s = (int)(q % ns);
    q /= ns;
    const int per_e = gu ? m / 32 : d / 64;
    const int c = (int)(q % per_e);
    const int e = (int)(q / per_e);
    const int l16 = lane & 15, kq = (lane >> 4) * 8;
    const int k = 64 * s + 32 * h + kq;
    int64_t src;
    if (gu) {
        const int wrow = (f < 2) ? 32 * c + 16 * f + l16 : m + 32 * c + 16 * (f - 2) + l16;
        src = ((int64_t)e * 2 * m + wrow) * d + k;
    } else {
        src = ((int64_t)e * d + 64 * c + 16 * f + l16) * m + k;
    }
    const u32x4_t v = *reinterpret_cast<const u32x4_t*>((gu ? Wgu : Wd) + src);
    *reinterpret_cast<u32x4_t*>(P + i * 8) = v;
}

unsigned blocks_for(int tasks) { return (unsigned)((tasks + 7) / 8 * 8); }

}  // namespace

bool gemm_use_skinny(int dtype, int64_t T, int K, int N, int d, int m) {
    // at most 16 rows per expert on average: far below the bf16 ridge point (~300 rows), so
    // the weight stream bounds the GEMMs (T K <= 16 N <= kSlotMax, the waves' slot lists)
    // the kernel's 32-bit lane offsets span 8 weight rows of 2 max(d, m) bytes
    return dtype == ELB_BF16 && T > 0 && T * K <= (int64_t)16 * N && d % 64 == 0 &&
           m % 64 == 0 && d < (1 << 28) && m < (1 << 28);
}

hipError_t launch_gemm_skinny(const void* x, const void* Wgu, const void* Wd, const int* k,
                              const int* ids, int64_t T, int K, int d, int N, int m, void* H,
                              void* Y, int* counts, hipStream_t s) {
    const int t = (int)T;
    const int ne = T * K < N ? (int)(T * K) : N;  // see the kernel: tasks by slot or by expert
    const int spread = T > 1 && T * K <= 2 * N &&
                       (double)N * d * m * 6 > 2.0 * (double)kLastLevelCacheBytes;
    {
        ProfileScope prof("gemm_gate_up_skinny", s);
        ELB_LAUNCH((aligned16(Wgu, nullptr) ? gemm_skinny<0, true> : gemm_skinny<0, false>),
                   dim3(blocks_for(ne * (m / 32))), dim3(64 * SK_NW), 0, s, (const bf16_t*)x, k,
                   ids, t, K, (const bf16_t*)Wgu, N, d, m, spread, (bf16_t*)H, counts);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    {
        ProfileScope prof("gemm_down_skinny", s);
        ELB_LAUNCH((aligned16(Wd, nullptr) ? gemm_skinny<1, true> : gemm_skinny<1, false>),
                   dim3(blocks_for(ne * (d / 64))), dim3(64 * SK_NW), 0, s, (const bf16_t*)H, k,
                   ids, t, K, (const bf16_t*)Wd, N, d, m, spread, (bf16_t*)Y, (int*)nullptr);
    }
    return hipGetLastError();
}

hipError_t launch_pack_experts(const void* Wgu, const void* Wd, int N, int d, int m,
                               void* packed, hipStream_t s) {
    const int64_t n_all = ((int64_t)N * 2 * m * d + (int64_t)N * d * m) / 8;
    if (n_all == 0) return hipSuccess;
    ProfileScope prof("pack_experts", s);
    ELB_LAUNCH(pack_experts, dim3((unsigned)((n_all + 255) / 256)), dim3(256), 0, s,
                       (const bf16_t*)Wgu, (const bf16_t*)Wd, N, d, m, (bf16_t*)packed);
    return hipGetLastError();
}

}  // namespace elb
