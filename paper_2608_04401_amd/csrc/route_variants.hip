// Routing variants (Section 2.1, 2.2, 2.3): caps above 16 up to N (the uncapped elbow
// routing is K = N), tail randomisation (the experts after the elbow replaced by experts
// drawn from outside the elbow's selection) and the elbow angle with the uncapped elbow
// index.
//
// One LANE per token with the routing kernel's staging and arithmetic (route_lane.h), but the
// sorting network carries the expert ids along with the logits, so the id at every rank is
// known and any cap up to N costs the same.  Same bits as the routing kernel: the same keys,
// u_i = exp(l_(i) - l_(0)) in rank order (rel_exp), S as the same tree over the ranks
// (tree_sum), the same E_i and first argmin, w = u * (1 / denominator).  The elbow angle (no
// selection asked for) and tail randomisation with K <= 16 sort the keys only.
#include <cfloat>

#include "route_lane.h"

namespace elb {

namespace {

// ---------------------------------------------------------------------------------------
// One LANE per token, (key, id) pairs sorted by a network: the same staging and arithmetic as
// the routing kernel, but the sort carries the expert ids, so every rank's id is known and
// any cap up to N costs no more than K = 1.  A pair is one 64-bit integer: the logit's
// order-preserving integer image in the high word and (NP - 1 - id) in the low word, so one
// signed 64-bit comparison orders by logit descending, then id ascending (pads, -inf with the
// largest ids, sort last).  Each comparator is one v_cmp_gt_i64 and four v_cndmask_b32.
// ---------------------------------------------------------------------------------------

// order-preserving signed integer image of a canonical (non-NaN, no -0) fp32 value; its
// own inverse
__device__ __forceinline__ int ord_flip(int i) { return i ^ ((i >> 31) & 0x7fffffff); }

template <int NP, int Q>
__device__ __forceinline__ void cx_pair(int64_t* v) {
    constexpr int a = NetHolder<NP>::net.a[Q];
    constexpr int b = NetHolder<NP>::net.b[Q];
    const bool sw = v[b] > v[a];
    const int64_t hi = sw ? v[b] : v[a];
    const int64_t lo = sw ? v[a] : v[b];
    v[a] = hi;
    v[b] = lo;
}
template <int NP, int... Q>
__device__ __forceinline__ void sort_pairs_desc(int64_t* v, std::integer_sequence<int, Q...>) {
    (cx_pair<NP, Q>(v), ...);
}

// The experts of the first k ranks from the sorted keys, by the routing kernel's rule
// (select_first_k): their mask `taken`, and up to KM of them in id order (cid) with their keys
// (ck, -inf past k; re-read from the token's LDS row, as the id is not a compile-time
// constant there).
template <int NP, int KM>
__device__ __forceinline__ void first_k_experts(const float (&key)[NP], const float (&okey)[NP],
                                                const float* row, int Nn, int k,
                                                uint64_t& taken, int (&cid)[KM],
                                                float (&ck)[KM]) {
    taken = select_first_k<NP, KM>(key, [&](int c) { return okey[c]; }, Nn, k);
    selected_in_id_order<KM>(taken, [&](int c) { return order_key(row[c]); }, Nn, k, cid, ck);
}

// The KM largest of v[0 .. NP) into v[0 .. KM), descending (the rest is left in no order): groups
// of KM sorted by the network, then folded into the first, group by group: the larger of a_i and
// b_(KM - 1 - i) are the KM largest of two descending groups, in a bitonic order that log2(KM)
// stages of comparators sort.  528 min/max for the 8 largest of 64 and 744 for the 16 largest,
// where K - k passes over the draws, each a masked minimum with its index, took some 450
// instructions each (65536 tokens, N = 64, K = 8: angle and tail randomisation 35.7 -> 24.0 us;
// with K <= 2 a bound of 8 costs more than the pass it replaces: 299776 tokens, N = 32, tail
// randomisation 17.9 us by passes, 31.8 with KM = 8).
template <int NP, int KM>
__device__ __forceinline__ void largest_desc(float (&v)[NP]) {
#pragma unroll
    for (int g = 0; g < NP; g += KM)
        sort_desc<KM>(v + g, std::make_integer_sequence<int, NetHolder<KM>::net.n>{});
#pragma unroll
    for (int g = KM; g < NP; g += KM) {
#pragma unroll
        for (int i = 0; i < KM; ++i) v[i] = fmaxf(v[i], v[g + KM - 1 - i]);
#pragma unroll
        for (int o = KM / 2; o >= 1; o >>= 1)
#pragma unroll
            for (int i = 0; i < KM; ++i)
                if (!(i & o)) {
                    const float hi = fmaxf(v[i], v[i + o]), lo = fminf(v[i], v[i + o]);
                    v[i] = hi;
                    v[i + o] = lo;
                }
    }
}

// PAIRS: sort (key, id) pairs (a selection with any cap is asked for).  Otherwise the keys
// alone are sorted (the routing kernel's value network: the same sorted keys, so the same e
// and theta bits, at two instructions per comparator): for the elbow angle (no selection), and
// for tail randomisation with K <= kLaneMaxK, whose first k experts are then recovered by the
// routing kernel's selection rule.
// KMAX (keys alone): a bound on K: 2, 4, 8 or kLaneMaxK
template <int NP, bool FULL, bool PAIRS, int KMAX>
__global__ __launch_bounds__(256) void route_pair_kernel(
    const float* __restrict__ logits, const float* __restrict__ rand, int64_t T, int N, int K,
    float eps, int mode, int renorm, int vec4, XTable xt, int* __restrict__ kout,
    int* __restrict__ ids, float* __restrict__ wout, int* __restrict__ eout,
    float* __restrict__ thout) {
    constexpr int LD = NP + 1;
    __shared__ float lds[4 * kWave * LD];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x >> 6;
    const int64_t t0 = ((int64_t)blockIdx.x * 4 + wv) * kWave;
    float* tile = lds + wv * kWave * LD;
    int rows = 0;
    if (t0 < T) rows = (int)((T - t0) < kWave ? (T - t0) : kWave);
    stage_rows<NP, FULL>(logits + t0 * N, N, rows, vec4, tile, lane);
    __syncthreads();
    // a wave with no token of its own must not read draws (token t0 lies past the last one); no
    // barrier follows
    if (rows == 0) return;
    // lanes past the last token route a copy of the wave's first one and write nothing: every
    // lane takes part in the staged stores at the end
    const bool active = lane < rows;
    const float* row = tile + (active ? lane : 0) * LD;
    const int64_t t = t0 + (active ? lane : 0);
    const int Nn = FULL ? NP : N;

    // Tail randomisation from sorted keys: the lane's draws (16-byte loads where every row starts
    // on a 16-byte boundary).  Whole tiles load them where a token of the wave has a tail: a
    // batch of several waves per SIMD hides the wait, and a wave without a tail reads none.
    // Otherwise, whose 4-byte loads take longer, they are loaded ahead of the sort, except with
    // K <= 2, where most waves have no tail (299776 tokens, us, ahead / where needed: N = 32, K = 2
    // 27.5 / 14.0, K = 8 40.7 / 30.9; N = 24, K = 2 34.6 / 25.4, K = 8 47.8 / 53.7).
    constexpr bool kEarlyDraws = !FULL && KMAX > 2;
    float draw[NP];
    auto load_draws = [&]() {
        const float* const rr = rand + t * N;
        if (FULL && ((uintptr_t)rand % 16) == 0) {
#pragma unroll
            for (int c = 0; c < NP; c += 4) {
                const float4 q = *reinterpret_cast<const float4*>(rr + c);
                draw[c] = q.x; draw[c + 1] = q.y; draw[c + 2] = q.z; draw[c + 3] = q.w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < NP; ++c) draw[c] = (c < Nn) ? rr[c] : INFINITY;
        }
    };
    if (!PAIRS && kEarlyDraws && rand) load_draws();

    // ---- sort (key, id) pairs: rank r holds key[r] and id[r] ----
    float key[NP];
    int id[NP];
    if (PAIRS) {
        int64_t v[NP];
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            const float f = (c < Nn) ? order_key(row[c]) : -INFINITY;
            v[c] = ((int64_t)ord_flip(__float_as_int(f)) << 32) | (uint32_t)(NP - 1 - c);
        }
        sort_pairs_desc<NP>(v, std::make_integer_sequence<int, NetHolder<NP>::net.n>{});
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            key[r] = __int_as_float(ord_flip((int)(v[r] >> 32)));
            id[r] = NP - 1 - (int)(uint32_t)v[r];
        }
    } else {
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            key[c] = (c < Nn) ? order_key(row[c]) : -INFINITY;
            id[c] = 0;  // not used: no selection without PAIRS
        }
        sort_desc<NP>(key, std::make_integer_sequence<int, NetHolder<NP>::net.n>{});
    }

    // ---- u, S, u_min and the elbow: the routing kernel's arithmetic, in rank order ----
    const float nl = neg_scaled(key[0]);
    float u[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) u[i] = rel_exp(key[i], nl);
    const float S = tree_sum<NP>(u);
    float umin = u[NP - 1];
    if (!FULL) {
#pragma unroll
        for (int i = 0; i < NP; ++i) umin = (i == Nn - 1) ? u[i] : umin;
    }
    const float Rp = (1.0f - umin) + eps * S;
    float best = 1.f;  // E_0 = 1 (D_0 = 0)
    int e = 0;
#pragma unroll
    for (int i = 1; i < NP; ++i) {
        const float Ei = fmaf(xt.x[i], Rp, u[i]);  // pads: x' = +inf, never win
        const bool better = Ei < best;  // strict: the first index wins ties
        best = better ? Ei : best;
        e = better ? i : e;
    }
    if (eout && active) eout[t] = e;
    if (thout && active) {  // the angle at the elbow point (x'_e, p'_e) between (0,0) and (1,1)
        float th = 180.0f;  // e = 0: no point off the chord, a straight curve
        if (e > 0) {
            float xe = 0.f, ue = 0.f;
#pragma unroll
            for (int i = 1; i < NP; ++i) {
                xe = (i == e) ? xt.x[i] : xe;
                ue = (i == e) ? u[i] : ue;
            }
            const float pe = (1.0f - ue) / Rp;
            const float v1x = -xe, v1y = -pe, v2x = 1.0f - xe, v2y = 1.0f - pe;
            const float dot = fmaf(v1x, v2x, v1y * v2y);
            const float crs = fmaf(v1x, v2y, -(v1y * v2x));
            th = atan2f(fabsf(crs), dot) * (180.0f / 3.14159265358979323846f);
        }
        thout[t] = th;
    }
    if (!ids) return;
    const int k = (mode == ELB_MODE_TOPK) ? K : (e + 1 < K ? e + 1 : K);
    if (active) kout[t] = k;

    if (!PAIRS) {
        // tail randomisation with K <= kLaneMaxK from the sorted keys alone: the first k ranks'
        // experts by the routing kernel's selection rule, then the K - k untaken experts with
        // the smallest draws (equal draws: lower id) by the same rule on the negated draws; the
        // same ids and weight bits as the pair path (an expert's u is recomputed from its own
        // key)
        constexpr int KM = NP < KMAX ? NP : KMAX;
        float okey[NP];
#pragma unroll
        for (int c = 0; c < NP; ++c) okey[c] = (c < Nn) ? order_key(row[c]) : -INFINITY;
        uint64_t taken;
        int cid[KM];
        float ck[KM];
        first_k_experts<NP, KM>(key, okey, row, Nn, k, taken, cid, ck);
        const int n_tail = K - k;  // 0 .. KM - 1
        int tail[KM];
        float tu[KM];
        // wave-uniform; tail and tu are read for j < n_tail only.  (With K above 8 and the draws at
        // hand the test costs more than it saves: N = 60, K = 16 161 / 166 us.)
        if ((kEarlyDraws && KMAX > 8) || __any(n_tail > 0)) {
            if (!kEarlyDraws) load_draws();
            // negated draws (-inf: taken or past N), and the KM largest of them sorted
            float dkey[NP], top[NP];
#pragma unroll
            for (int c = 0; c < NP; ++c) {
                // order_key: a draw of 0 gives +0; the bound keeps an infinite draw above the
                // taken
                const float q = fmaxf(order_key(-draw[c]), -FLT_MAX);
                dkey[c] = (c < Nn && !((taken >> c) & 1ull)) ? q : -INFINITY;
                top[c] = dkey[c];
            }
            largest_desc<NP, KM>(top);
            uint64_t sel = select_first_k<NP, KM>(
                top, [&](int c) { return dkey[c]; }, Nn, n_tail > 0 ? n_tail : 1);
            if (n_tail == 0) sel = 0;
            int did[KM];
            float dk[KM];
            selected_in_id_order<KM>(
                sel, [&](int c) { return fmaxf(order_key(-rand[t * N + c]), -FLT_MAX); }, Nn,
                n_tail, did, dk);
            // the tail in its order: tail[j] for j < n_tail
            bool distinct = true;
#pragma unroll
            for (int j = 0; j + 1 < KM; ++j)
                if (j + 1 < n_tail && top[j] == top[j + 1]) distinct = false;
            if (__builtin_expect(__all(distinct), 1)) {
#pragma unroll
                for (int j = 0; j < KM; ++j) {
                    tail[j] = did[0];
#pragma unroll
                    for (int q = 0; q < KM; ++q) tail[j] = (dk[q] == top[j]) ? did[q] : tail[j];
                }
            } else {  // by counting (equal draws: lower id, i.e. lower position, first)
                int rank[KM];
#pragma unroll
                for (int q = 0; q < KM; ++q) {
                    rank[q] = q < n_tail ? 0 : KM;
#pragma unroll
                    for (int o = 0; o < KM; ++o)
                        if (o != q && o < n_tail && (o < q ? dk[o] >= dk[q] : dk[o] > dk[q]))
                            ++rank[q];
                }
#pragma unroll
                for (int j = 0; j < KM; ++j) {
                    tail[j] = did[0];
#pragma unroll
                    for (int q = 0; q < KM; ++q) tail[j] = (rank[q] == j) ? did[q] : tail[j];
                }
            }
#pragma unroll
            for (int j = 0; j < KM; ++j) tu[j] = rel_exp(order_key(row[tail[j]]), nl);
        }
        float denom = S;
        if (renorm) {
            float sel_u[KM];
#pragma unroll
            for (int j = 0; j < KM; ++j) sel_u[j] = j < k ? u[j] : 0.f;
            denom = tree_sum<KM>(sel_u);
#pragma unroll
            for (int j = 0; j < KM; ++j)
                if (j < n_tail) denom += tu[j];
        }
        const float inv = 1.0f / denom;
        if (!active) return;
        // the elbow's experts at their ranks (descending key; equal keys: lower id first)
#pragma unroll
        for (int r = 0; r < KM; ++r) {
            if (r < k) {
                int rank = 0;
#pragma unroll
                for (int q = 0; q < KM; ++q) {
                    if (q < r) rank += (q < k && ck[q] >= ck[r]) ? 1 : 0;
                    if (q > r) rank += (q < k && ck[q] > ck[r]) ? 1 : 0;
                }
                ids[t * K + rank] = cid[r];
                wout[t * K + rank] = rel_exp(ck[r], nl) * inv;
            }
        }
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            if (j < n_tail) {
                ids[t * K + k + j] = tail[j];
                wout[t * K + k + j] = tu[j] * inv;
            }
        }
        return;
    }

    if (rand) {
        // tail randomisation: K - k experts outside the first k ranks, smallest draws first
        // (equal draws: lower id); weights are the experts' own probabilities
        const float* rr = rand + t * N;
        float draw[NP];
#pragma unroll
        for (int c = 0; c < NP; ++c) draw[c] = (c < Nn) ? rr[c] : INFINITY;
        uint64_t taken = 0;
#pragma unroll
        for (int r = 0; r < NP; ++r)
            if (r < k) taken |= 1ull << id[r];

        float denom = S;
        if (renorm) {
            float sel_u[NP];
#pragma unroll
            for (int j = 0; j < NP; ++j) sel_u[j] = j < k ? u[j] : 0.f;
            denom = tree_sum<NP>(sel_u);
        }
        // pass 1: the tail's ids, with unnormalised weights u (the denominator needs them all)
        for (int j = k; j < K; ++j) {
            float bv = INFINITY;
            int bc = -1;
#pragma unroll
            for (int c = 0; c < NP; ++c) {
                const bool ok = c < Nn && !((taken >> c) & 1ull) && (bc < 0 || draw[c] < bv);
                bv = ok ? draw[c] : bv;
                bc = ok ? c : bc;
            }
            taken |= 1ull << bc;
            const float ub = rel_exp(order_key(row[bc]), nl);
            if (active) {
                ids[t * K + j] = bc;
                wout[t * K + j] = ub;
            }
            if (renorm) denom += ub;
        }
        const float inv = 1.0f / denom;
        if (!active) return;
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            if (r < k) {
                ids[t * K + r] = id[r];
                wout[t * K + r] = u[r] * inv;
            }
        }
        for (int j = k; j < K; ++j) wout[t * K + j] *= inv;  // pass 2 (this lane's own writes)
        return;
    }
    float denom = S;
    if (renorm) {
        float sel_u[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) sel_u[j] = j < k ? u[j] : 0.f;
        denom = tree_sum<NP>(sel_u);
    }
    const float inv = 1.0f / denom;
    if (K <= 16) {  // few slots: direct stores
        if (!active) return;
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            if (r < k) {
                ids[t * K + r] = id[r];
                wout[t * K + r] = u[r] * inv;
            } else if (r < K) {
                ids[t * K + r] = -1;
                wout[t * K + r] = 0.f;
            }
        }
        return;
    }
    // many slots: stage the wave's 64 output rows in its LDS tile (its logits have been read;
    // a wave's LDS operations complete in order), rows padded to K + 1 words, then store each
    // token's K contiguous values with the whole wave
    int* sti = reinterpret_cast<int*>(tile);
#pragma unroll
    for (int r = 0; r < NP; ++r)
        if (r < K) sti[lane * (K + 1) + r] = (r < k) ? id[r] : -1;
    for (int q = 0; q < rows; ++q)
        for (int c = lane; c < K; c += kWave) ids[(t0 + q) * K + c] = sti[q * (K + 1) + c];
#pragma unroll
    for (int r = 0; r < NP; ++r)
        if (r < K) tile[lane * (K + 1) + r] = (r < k) ? u[r] * inv : 0.f;
    for (int q = 0; q < rows; ++q)
        for (int c = lane; c < K; c += kWave) wout[(t0 + q) * K + c] = tile[q * (K + 1) + c];
}

template <int NP, bool FULL>
void launch_pair_np(const float* logits, const float* rand, int64_t T, int N,
                    const elb_route_params& p, int* k, int* ids, float* w, int* e, float* theta,
                    hipStream_t s) {
    const int64_t waves = (T + kWave - 1) / kWave;
    const int vec4 = ((uintptr_t)logits % 16) == 0;
    const dim3 grid((unsigned)((waves + 3) / 4));
    // keys only: the elbow angle (no ids), or tail randomisation with K <= kLaneMaxK
    const bool keys_only = !ids || (rand && p.K <= kLaneMaxK);
    auto launch = [&](auto kernel) {
        ELB_LAUNCH(kernel, grid, dim3(256), 0, s, logits, rand, T, N, p.K, p.eps, p.mode,
                   p.renormalize, vec4, make_xtable(N), k, ids, w, e, theta);
    };
    if (!keys_only) launch(route_pair_kernel<NP, FULL, true, NP>);
    else if (!ids) launch(route_pair_kernel<NP, FULL, false, 8>);  // no K
    else if (p.K <= 2) launch(route_pair_kernel<NP, FULL, false, 2>);
    else if (p.K <= 4) launch(route_pair_kernel<NP, FULL, false, 4>);
    else if (p.K <= 8) launch(route_pair_kernel<NP, FULL, false, 8>);
    else launch(route_pair_kernel<NP, FULL, false, kLaneMaxK>);
}

}  // namespace

hipError_t launch_route_pair(const float* logits, const float* rand, int64_t T, int N,
                             const elb_route_params& p, int* k, int* ids, float* w, int* e,
                             float* theta, hipStream_t s) {
    if (T == 0) return hipSuccess;
    ProfileScope prof("route_pair", s);
    switch (N) {
        case 8: launch_pair_np<8, true>(logits, rand, T, N, p, k, ids, w, e, theta, s); break;
        case 16: launch_pair_np<16, true>(logits, rand, T, N, p, k, ids, w, e, theta, s); break;
        case 32: launch_pair_np<32, true>(logits, rand, T, N, p, k, ids, w, e, theta, s); break;
        case 64: launch_pair_np<64, true>(logits, rand, T, N, p, k, ids, w, e, theta, s); break;
        default:
            if (N < 8)
                launch_pair_np<8, false>(logits, rand, T, N, p, k, ids, w, e, theta, s);
            else if (N < 16)
                launch_pair_np<16, false>(logits, rand, T, N, p, k, ids, w, e, theta, s);
            else if (N < 32)
                launch_pair_np<32, false>(logits, rand, T, N, p, k, ids, w, e, theta, s);
            else
                launch_pair_np<64, false>(logits, rand, T, N, p, k, ids, w, e, theta, s);
    }
    return hipGetLastError();
}

}  // namespace elb
