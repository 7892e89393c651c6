// The router: fused score function + top-k + weights + histogram (Sec. 2.1.2 item 2, Sec. 4.3.4), its group-limited and
// biased branches, its backward, and the load-balancing loss.
//
// A group of LPT lanes owns one token: 16 lanes (four tokens per wavefront) up to 256 experts, a whole wavefront above.
// Lane l of the group holds the logits of experts l, l + LPT, l + 2 LPT, ... in registers; what the group has to agree on
// (maximum, sum, the winner of an arg-max round) is a reduction of four DPP steps over 16 lanes (two more before them,
// through the LDS crossbar, over 64).  A wavefront handles one token per group and ends.
// Bound: vector instructions at large T (one read of the logits: 3.6 us for T 16384, E 256 at the copy rate), one
// token's chain of reductions at small T.  Values are compared as order-preserving integers, so that an arg-max round is
// max3 over the lane's values, four DPP maxima, and a DPP minimum over the indices that hold the maximum.
// Measured (us a call; one token per wavefront, eight in turn, butterfly shuffles : this), T 16384, E 256, k 8: top-k 57 : 15;
// group-limited with bias, 8 groups: 147 : 35; backward 22 : 11; auxiliary loss 22 : 16.  T 64, E 128, k 8: 47 : 6.
// The group-limited kernel then: 35 -> 25 with the groups' best two met in registers instead of scans through LDS, a slot's score read
// back from LDS instead of picked out of 16 registers per round, and half as many workgroups adding their histograms.
#include "common.h"

#define ROUTE_MAX_E 1024

// ---- reductions over a token's lanes: every lane gets the result --------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float x) { return __uint_as_float(dpp<CTRL>(__float_as_uint(x))); }
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    return __longlong_as_double((long long)(((uint64_t)dpp<CTRL>((uint32_t)(b >> 32)) << 32) | dpp<CTRL>((uint32_t)b)));
}
// Exchange with the lane 32 and 16 away (a whole wavefront), then 8, 4, 2 and 1 away: row_ror by 8 and by 4 (by then a row
// repeats every 8 lanes, so that 4 to either side are the same value), quad permutations for the rest.
template <int LPT, typename T, typename F>
__device__ __forceinline__ T lanes_reduce(T v, F op) {
    if (LPT == 64) {
        v = op(v, __shfl_xor(v, 32));
        v = op(v, __shfl_xor(v, 16));
    }
    v = op(v, dpp<0x128>(v));
    v = op(v, dpp<0x124>(v));
    v = op(v, dpp<0x4E>(v));
    v = op(v, dpp<0xB1>(v));
    return v;
}
template <int LPT> __device__ __forceinline__ float lanes_max(float v) { return lanes_reduce<LPT>(v, [](float a, float b) { return fmaxf(a, b); }); }
template <int LPT> __device__ __forceinline__ float lanes_sum(float v) { return lanes_reduce<LPT>(v, [](float a, float b) { return a + b; }); }
template <int LPT> __device__ __forceinline__ double lanes_sum(double v) { return lanes_reduce<LPT>(v, [](double a, double b) { return a + b; }); }
template <int LPT> __device__ __forceinline__ uint32_t lanes_max(uint32_t v) { return lanes_reduce<LPT>(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; }); }
template <int LPT> __device__ __forceinline__ uint32_t lanes_min(uint32_t v) { return lanes_reduce<LPT>(v, [](uint32_t a, uint32_t b) { return a < b ? a : b; }); }

// Sum over a token's experts, add(j, sum) = sum + the term of expert l + LPT j.  The order of the additions is the same for
// both layouts, that of 64 lanes: per residue of the expert modulo 64 in ascending order, then residues 32, 16, 8, 4, 2, 1
// apart (a lane of 16 holds four residues).  A weight's last bit moves bf16 roundings all the way through a layer: it must
// not depend on the lane layout.
template <int LPT, int VPL, typename T, typename F>
__device__ __forceinline__ T experts_sum(F add) {
    T part[4] = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
    for (int j = 0; j < VPL; ++j) part[LPT == 64 ? 0 : j & 3] = add(j, part[LPT == 64 ? 0 : j & 3]);
    return lanes_sum<LPT>(LPT == 64 ? part[0] : (part[0] + part[2]) + (part[1] + part[3]));
}
// Sum over a token's slots, one per lane (0 in the lanes without one).  The + 0 rounds a product before it is added, as the
// empty upper lanes of a 64-lane sum do.
template <int LPT>
__device__ __forceinline__ float slots_sum(float v) { return lanes_sum<LPT>(LPT == 64 ? v : v + 0.0f); }

// fp32 values as unsigned integers in the same order (-0 counts as 0); every number, -inf included, is above 0, which
// stands for "no candidate"
__device__ __forceinline__ uint32_t order_key(float x) {
    const uint32_t u = __float_as_uint(x + 0.0f);
    return u ^ (uint32_t)(((int32_t)u >> 31) | (int32_t)0x80000000);
}
__device__ __forceinline__ float key_value(uint32_t k) { return __uint_as_float(k & 0x80000000u ? k ^ 0x80000000u : ~k); }

// one round of arg-max over (value descending, index ascending): best value and its index; the winner leaves the list
template <int LPT, int VPL>
__device__ __forceinline__ void take_best(uint32_t (&key)[VPL], int l, uint32_t& best, uint32_t& idx) {
    uint32_t m = key[0];
#pragma unroll
    for (int j = 1; j < VPL; ++j) m = key[j] > m ? key[j] : m;
    best = lanes_max<LPT>(m);
    uint32_t at = 0xffffffffu;
#pragma unroll
    for (int j = VPL - 1; j >= 0; --j) at = key[j] == best ? (uint32_t)(l + LPT * j) : at;
    idx = lanes_min<LPT>(at);
#pragma unroll
    for (int j = 0; j < VPL; ++j) key[j] = (uint32_t)(l + LPT * j) == idx ? 0u : key[j];
}

// The histogram: LDS per workgroup, then, with more than one workgroup, added to `counts`, which a launch ahead of the kernel
// has cleared.  (An accumulator kept at zero between calls, taken out by the last workgroup, saves that launch, 2-4 us, but
// what one call left there the next would count.)
__device__ __forceinline__ void finish_counts(const int32_t* hist, int E, int32_t* counts) {
    __syncthreads();
    if (!counts) return;
    const bool alone = gridDim.x == 1;
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        if (alone) counts[e] = hist[e];
        else if (hist[e]) atomicAdd(&counts[e], hist[e]);
    }
}

template <int LPT, int VPL>
__global__ __launch_bounds__(1024) void route_topk_kernel(
    const float* __restrict__ logits, int T, int E, int k, int fn, int norm_topk, float scale,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_prob, int32_t* __restrict__ counts) {
    extern __shared__ int32_t hist[];  // [E]
    const int l = threadIdx.x & (LPT - 1);
    const int t = blockIdx.x * (blockDim.x / LPT) + threadIdx.x / LPT;
    for (int e = threadIdx.x; e < E; e += blockDim.x) hist[e] = 0;
    const float* row = logits + (int64_t)(t < T ? t : T - 1) * E;
    float v[VPL];
    uint32_t key[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) v[j] = l + LPT * j < E ? row[l + LPT * j] : -INFINITY;
#pragma unroll
    for (int j = 0; j < VPL; ++j) key[j] = l + LPT * j < E ? order_key(v[j]) : 0u;
    float mx = 0.f, den = 1.f;
    if (fn == MOE_SCORE_SOFTMAX) {
        float m = v[0];
#pragma unroll
        for (int j = 1; j < VPL; ++j) m = fmaxf(m, v[j]);
        mx = lanes_max<LPT>(m);
        den = experts_sum<LPT, VPL, float>([&](int j, float s) { return s + (l + LPT * j < E ? expf(v[j] - mx) : 0.f); });
    }
    float my_logit = 0.f;
    uint32_t my_idx = 0;
    for (int it = 0; it < k; ++it) {
        uint32_t best, idx;
        take_best<LPT, VPL>(key, l, best, idx);
        if (l == it) {
            my_logit = key_value(best);
            my_idx = idx;
        }
    }
    float p = 0.f;
    if (l < k) p = fn == MOE_SCORE_SOFTMAX ? expf(my_logit - mx) / den : 1.f / (1.f + expf(-my_logit));
    if (norm_topk) p = p / slots_sum<LPT>(p);
    __syncthreads();  // hist is zero
    if (l < k && t < T) {
        const int e = (int)min(my_idx, (uint32_t)E - 1);  // (NaN logits: some expert that exists)
        topk_idx[(int64_t)t * k + l] = e;
        topk_prob[(int64_t)t * k + l] = p * scale;
        atomicAdd(&hist[e], 1);
    }
    finish_counts(hist, E, counts);
}

// ---------------------------------------------------------------------------
// moe_route_topk_grouped: the other branches of the fused score kernel (Sec. 4.3.4 item 1): group-limited
// top-k, the load-balancing expert bias (Sec. 7) and score scaling.
//   s_e = score(logits)_e;  c_e = s_e + bias_e decides, s_e weighs;
//   group score = sum of the k / topk_group largest c of the group; keep the topk_group best groups;
//   select the k largest c among the kept groups' experts; ties to the lower index throughout.
// The decisions are taken on fp32 values that do not depend on the precision of a fast exponential: the score is
// evaluated in double and rounded to fp32 once, the bias add and the group sums (largest first) are single fp32
// additions.  The c values of a token go through LDS for the group scores: `lpg` lanes share a group, each looking at
// every lpg-th member.
// ---------------------------------------------------------------------------
template <int LPT, int VPL>
__global__ __launch_bounds__(512) void route_topk_grouped_kernel(
    const float* __restrict__ logits, const float* __restrict__ bias, int T, int E, int k, int n_group, int topk_group,
    int lpg, uint32_t gs_magic, int fn, int norm_topk, float scale,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_prob, int32_t* __restrict__ counts) {
    extern __shared__ int32_t hist[];  // [E] histogram, then one [E + E / 16 + 1] row of c per token of the workgroup
    const int l = threadIdx.x & (LPT - 1);
    const int t = blockIdx.x * (blockDim.x / LPT) + threadIdx.x / LPT;
    for (int e = threadIdx.x; e < E; e += blockDim.x) hist[e] = 0;
    const int gs = E / n_group, m = k / topk_group;
    const float* row = logits + (int64_t)(t < T ? t : T - 1) * E;
    float v[VPL], sc[VPL];
    uint32_t key[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) v[j] = l + LPT * j < E ? row[l + LPT * j] : -INFINITY;
    if (fn == MOE_SCORE_SOFTMAX) {
        float mf = v[0];
#pragma unroll
        for (int j = 1; j < VPL; ++j) mf = fmaxf(mf, v[j]);
        const double mx = (double)lanes_max<LPT>(mf);
        double ex[VPL];
        const double den = experts_sum<LPT, VPL, double>([&](int j, double s) {
            ex[j] = l + LPT * j < E ? exp((double)v[j] - mx) : 0.0;
            return s + ex[j];
        });
#pragma unroll
        for (int j = 0; j < VPL; ++j) sc[j] = (float)(ex[j] / den);
    } else {
#pragma unroll
        for (int j = 0; j < VPL; ++j) sc[j] = (float)(1.0 / (1.0 + exp(-(double)v[j])));
    }
    // Groups of whole rows of lanes (16 members, or a multiple) whose best one or two count: a lane's members of a group are
    // neighbours in its registers, and the two largest of 16 lanes meet in four exchanges.  Other groups meet through LDS
    // (by_lds), which otherwise keeps the scores for the lanes that will hold a slot.
    const bool in_regs = LPT == 16 && m <= 2 && (gs & 15) == 0, by_lds = n_group > 1 && !in_regs;
    float* const cw = (float*)(hist + E) + (threadIdx.x / LPT) * (E + E / 16 + 1);
    auto at = [](int e) { return e + (e >> 4); };  // (a float of padding every 16 keeps the groups on different banks)
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
        const int e = l + LPT * j;
        const float c = (bias && e < E) ? sc[j] + bias[e] : sc[j];
        key[j] = e < E ? order_key(c) : 0u;
        if (e < E) cw[at(e)] = by_lds ? c : sc[j];
    }

    // ---- groups to keep ----
    if (n_group > 1) {
        const int g = l / lpg, sub = l & (lpg - 1);
        uint32_t gkey = 0;
        float gsum = 0.f;
        if (in_regs) {
            uint32_t hi = 0, lo = 0;
            const int per = gs >> 4;
            int grp = 0, left = per;
#pragma unroll
            for (int j = 0; j < VPL; ++j) {
                // (a NaN counts for nothing here; numbers' keys run from that of -inf to that of inf)
                const uint32_t x = key[j] - 0x007fffffu <= 0xff800000u - 0x007fffffu ? key[j] : 0u;
                lo = max(lo, min(hi, x));
                hi = max(hi, x);
                if (--left == 0) {                          // (uniform)
                    uint32_t h2 = hi, l2 = lo;
                    auto meet = [&](uint32_t oh, uint32_t ol) {
                        l2 = max(min(h2, oh), max(l2, ol));
                        h2 = max(h2, oh);
                    };
                    meet(dpp<0x128>(h2), dpp<0x128>(l2));
                    meet(dpp<0x124>(h2), dpp<0x124>(l2));
                    meet(dpp<0x4E>(h2), dpp<0x4E>(l2));
                    meet(dpp<0xB1>(h2), dpp<0xB1>(l2));
                    const float sum = m == 1 ? key_value(h2) : key_value(h2) + key_value(l2);
                    gsum = grp == g ? sum : gsum;
                    ++grp;
                    left = per;
                    hi = lo = 0;
                }
            }
        } else {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // (a token's lanes are of one wavefront: program order suffices)
        // sum of the m largest c of the lane's group, largest first; round r takes the best element that comes after
        // round r - 1's pick in (value desc, index asc) order
        float pv = INFINITY;
        int pi = -1;
        for (int r = 0; r < m; ++r) {
            uint32_t bk = 0, bi = 0x7fffffff;
            if (g < n_group) {
                for (int x = sub; x < gs; x += lpg) {
                    const float cv = cw[at(g * gs + x)];
                    const uint32_t ck = order_key(cv);
                    if ((cv < pv || (cv == pv && x > pi)) && ck > bk) {
                        bk = ck;
                        bi = x;
                    }
                }
            }
            for (int o = 1; o < lpg; o <<= 1) {
                const uint32_t ok = __shfl_xor(bk, o), oi = __shfl_xor(bi, o);
                if (ok > bk || (ok == bk && oi < bi)) {
                    bk = ok;
                    bi = oi;
                }
            }
            pv = key_value(bk);
            pi = (int)bi;
            gsum = r == 0 ? pv : gsum + pv;
        }
        }
        if (g < n_group) gkey = order_key(gsum);
        bool kept = false;
        for (int r = 0; r < topk_group; ++r) {
            const uint32_t best = lanes_max<LPT>(gkey);
            const uint32_t win = lanes_min<LPT>(gkey == best ? (uint32_t)g : 0xffffffffu);
            if ((uint32_t)g == win) {
                kept = true;
                gkey = 0;
            }
        }
        // bit lpg * g of the token's lanes = group g is kept
        const uint64_t b = __ballot(kept) >> (LPT == 64 ? 0 : (threadIdx.x & 63 & ~(LPT - 1)));
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
            const int eg = (int)(((uint32_t)(l + LPT * j) * gs_magic) >> 20);  // (l + LPT j) / gs
            if (l + LPT * j < E && !((b >> (eg * lpg)) & 1ull)) key[j] = 0u;
        }
    }

    // ---- the k best among the kept groups ----
    float my_s = 0.f;
    uint32_t my_idx = 0;
    for (int it = 0; it < k; ++it) {
        uint32_t best, idx;
        take_best<LPT, VPL>(key, l, best, idx);
        if (by_lds) {
            uint32_t sv = 0;  // the winner's unbiased score, from the lane that holds it
#pragma unroll
            for (int j = 0; j < VPL; ++j) sv = (uint32_t)(l + LPT * j) == idx ? __float_as_uint(sc[j]) : sv;
            sv = lanes_max<LPT>(sv);  // (scores are not negative: their bits order like the values, the other lanes hold 0)
            if (l == it) my_s = __uint_as_float(sv);
        }
        if (l == it) my_idx = idx;
    }
    if (!by_lds) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        my_s = cw[at((int)min(my_idx, (uint32_t)E - 1))];
    }
    float p = l < k ? my_s : 0.f;
    if (norm_topk) p = p / slots_sum<LPT>(p);
    __syncthreads();  // hist is zero
    if (l < k && t < T) {
        const int e = (int)min(my_idx, (uint32_t)E - 1);  // (NaN logits: some expert that exists)
        topk_idx[(int64_t)t * k + l] = e;
        topk_prob[(int64_t)t * k + l] = p * scale;
        atomicAdd(&hist[e], 1);
    }
    finish_counts(hist, E, counts);
}

// ---------------------------------------------------------------------------
// moe_route_topk_bwd: dL/dlogits from dL/dweights with the selection frozen (Sec. 2.1.2 item 2).
//   w_s = scale * q_s / D,  q_s = score of the s-th selected expert,  D = sum_s q_s (norm_topk) or 1
//   dq_s = scale * (dw_s / D - [norm] <dw, q> / D^2)
//   softmax: dl_j = p_j * ([j selected] dq_j - <dq, q>)      sigmoid: dl_j = [j selected] dq_j * q_j (1 - q_j)
// Same layout as the forward kernel; lane s < k of a token's group holds slot s.
// ---------------------------------------------------------------------------
template <int LPT, int VPL>
__global__ __launch_bounds__(256) void route_topk_bwd_kernel(
    const float* __restrict__ logits, const int32_t* __restrict__ topk_idx, const float* __restrict__ dprob,
    int T, int E, int k, int fn, int norm_topk, float scale, float* __restrict__ dlogits) {
    const int l = threadIdx.x & (LPT - 1);
    const int t = blockIdx.x * (blockDim.x / LPT) + threadIdx.x / LPT;
    const int tr = t < T ? t : T - 1;  // (whole wavefronts stay together: a token behind the last one computes, unused)
    const float* row = logits + (int64_t)tr * E;
    float v[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) v[j] = l + LPT * j < E ? row[l + LPT * j] : -INFINITY;
    // slot s lives in lane s: its expert, its score q_s and the incoming gradient
    int my_idx = l < k ? topk_idx[(int64_t)tr * k + l] : -1;
    if (my_idx < 0 || my_idx >= E) my_idx = -1;  // a slot that names no expert of this router contributes nothing
    const float dw = my_idx >= 0 ? dprob[(int64_t)tr * k + l] : 0.f;
    const float lg = my_idx >= 0 ? row[my_idx] : 0.f;
    float mx = 0.f, den = 1.f;
    if (fn == MOE_SCORE_SOFTMAX) {
        float m = v[0];
#pragma unroll
        for (int j = 1; j < VPL; ++j) m = fmaxf(m, v[j]);
        mx = lanes_max<LPT>(m);
        den = experts_sum<LPT, VPL, float>([&](int j, float s) {
            v[j] = l + LPT * j < E ? expf(v[j] - mx) : 0.f;
            return s + v[j];
        });
    }
    float q = 0.f;
    if (my_idx >= 0) q = fn == MOE_SCORE_SOFTMAX ? expf(lg - mx) / den : 1.f / (1.f + expf(-lg));
    float dq = scale * dw;
    if (norm_topk) {
        const float D = slots_sum<LPT>(q);
        const float dwq = slots_sum<LPT>(dw * q);
        dq = my_idx >= 0 ? scale * (dw / D - dwq / (D * D)) : 0.f;
    }
    const float dqq = slots_sum<LPT>(dq * q);  // <dq, q>
    // every lane collects the dq of the selected experts it owns, and (sigmoid) their scores: the other experts' gradient is
    // zero, so that k scores of a token are computed and not E
    float gsel[VPL], ssel[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) gsel[j] = ssel[j] = 0.f;
    for (int s = 0; s < k; ++s) {
        const int e = __shfl(my_idx, s, LPT);
        const float d = __shfl(dq, s, LPT), qs = __shfl(q, s, LPT);
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
            const bool mine = e == l + LPT * j;
            gsel[j] += mine ? d : 0.f;
            ssel[j] = mine ? qs : ssel[j];
        }
    }
    if (t >= T) return;
    float* o = dlogits + (int64_t)t * E;
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
        const int e = l + LPT * j;
        if (e < E) {
            float r;
            if (fn == MOE_SCORE_SOFTMAX) {
                r = v[j] / den * (gsel[j] - dqq);
            } else {
                r = v[j] != v[j] ? v[j] : gsel[j] * ssel[j] * (1.f - ssel[j]);   // (a NaN logit: NaN, selected or not)
            }
            o[e] = r;
        }
    }
}

// ---------------------------------------------------------------------------
// moe_aux_loss: load-balancing auxiliary loss and its gradient (Sec. 4.3.4 items 2 and 3, fused here into one
// pass over the logits; the Switch-Transformer form the paper cites):
//   p[t,:] = softmax(l[t,:]) or sigmoid(l[t,:]) / sum_j sigmoid(l[t,j])           (Sec. 2.1.2 item 2)
//   loss   = coeff E sum_e f_e P_e,  f_e = counts[e] / (T k),  P_e = (1/T) sum_t p[t,e]
//          = sum_t <w, p[t,:]>,      w_e = coeff E counts[e] / (T^2 k)
//   dl[t,j] = g p_j (w_j - <w, p>) (softmax),  g (1 - sg_j) p_j (w_j - <w, p>) (sigmoid),  g = dloss
// so both the loss and the gradient need only per-token quantities.  The per-token terms are summed in double: the
// tokens of a workgroup in order, by eights, one partial sum per workgroup (32 tokens) into the context's workspace, and a
// one-wave kernel adds the partial sums in a fixed order (run-to-run identical, no floating-point atomics).
// ---------------------------------------------------------------------------
#define AUX_TOKENS 32  // tokens per workgroup (and 8 bytes of workspace for each)
template <int LPT, int VPL>
__global__ __launch_bounds__(AUX_TOKENS * LPT > 1024 ? 1024 : AUX_TOKENS * LPT) void aux_loss_kernel(
    const float* __restrict__ logits, const int32_t* __restrict__ counts, int T, int E, int fn, float wscale, float g,
    int accumulate, float* __restrict__ dlogits, double* __restrict__ partial, float* __restrict__ loss) {
    __shared__ double terms[AUX_TOKENS];
    const int l = threadIdx.x & (LPT - 1);
    float w[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) w[j] = l + LPT * j < E ? wscale * (float)counts[l + LPT * j] : 0.f;
    for (int i = threadIdx.x / LPT; i < AUX_TOKENS; i += blockDim.x / LPT) {
        const int t = blockIdx.x * AUX_TOKENS + i;
        const int tr = t < T ? t : T - 1;
        const float* row = logits + (int64_t)tr * E;
        float v[VPL], p[VPL], old[VPL];
#pragma unroll
        for (int j = 0; j < VPL; ++j) v[j] = l + LPT * j < E ? row[l + LPT * j] : -INFINITY;
        if (dlogits && accumulate) {
#pragma unroll
            for (int j = 0; j < VPL; ++j) old[j] = l + LPT * j < E ? dlogits[(int64_t)tr * E + l + LPT * j] : 0.f;
        }
        if (fn == MOE_SCORE_SOFTMAX) {
            float m = v[0];
#pragma unroll
            for (int j = 1; j < VPL; ++j) m = fmaxf(m, v[j]);
            m = lanes_max<LPT>(m);
#pragma unroll
            for (int j = 0; j < VPL; ++j) p[j] = l + LPT * j < E ? expf(v[j] - m) : 0.f;
        } else {
#pragma unroll
            for (int j = 0; j < VPL; ++j) p[j] = v[j] = l + LPT * j < E ? 1.f / (1.f + expf(-v[j])) : 0.f;
        }
        const float inv = 1.f / experts_sum<LPT, VPL, float>([&](int j, float s) { return s + p[j]; });
        const float d = experts_sum<LPT, VPL, float>([&](int j, float s) {  // <w, p[t,:]>
            p[j] *= inv;
            return s + w[j] * p[j];
        });
        if (l == 0) terms[i] = t < T ? (double)d : 0.0;
        if (dlogits && t < T) {
#pragma unroll
            for (int j = 0; j < VPL; ++j) {
                const int e = l + LPT * j;
                if (e < E) {
                    float gr = g * p[j] * (w[j] - d);
                    if (fn != MOE_SCORE_SOFTMAX) gr *= 1.f - v[j];
                    dlogits[(int64_t)t * E + e] = accumulate ? old[j] + gr : gr;
                }
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = 0.0;
        for (int i = 0; i < AUX_TOKENS; i += 8) {
            double eight = 0.0;
            for (int x = 0; x < 8; ++x) eight += terms[i + x];
            sum += eight;
        }
        if (gridDim.x == 1) *loss = (float)sum;
        else partial[blockIdx.x] = sum;
    }
}

__global__ __launch_bounds__(64) void aux_loss_sum_kernel(const double* __restrict__ partial, int n, float* __restrict__ loss) {
    double a = 0.0;
    for (int i = threadIdx.x; i < n; i += 512) {   // (eight loads in flight; the order of the additions is i's)
        double v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = i + 64 * x < n ? partial[i + 64 * x] : 0.0;
#pragma unroll
        for (int x = 0; x < 8; ++x) a += v[x];
    }
    a = lanes_sum<64>(a);
    if (threadIdx.x == 0) *loss = (float)a;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Lanes per token and values per lane.  16 lanes where a token's experts, slots and groups fit them: four tokens share
// the instructions of a wavefront, and their reductions stay inside DPP rows.
static inline bool route_narrow(int E, int k, int n_group) { return E <= 256 && k <= 16 && n_group <= 16; }
#define ROUTE_CASES(KERNEL, ...)                                                                                  \
    do {                                                                                                          \
        const int vpl = (E + lpt - 1) / lpt;                                                                      \
        if (lpt == 16) {                                                                                          \
            if (vpl <= 1) hipLaunchKernelGGL((KERNEL<16, 1>), __VA_ARGS__);                                       \
            else if (vpl <= 2) hipLaunchKernelGGL((KERNEL<16, 2>), __VA_ARGS__);                                  \
            else if (vpl <= 4) hipLaunchKernelGGL((KERNEL<16, 4>), __VA_ARGS__);                                  \
            else if (vpl <= 8) hipLaunchKernelGGL((KERNEL<16, 8>), __VA_ARGS__);                                  \
            else hipLaunchKernelGGL((KERNEL<16, 16>), __VA_ARGS__);                                               \
        } else {                                                                                                  \
            if (vpl <= 1) hipLaunchKernelGGL((KERNEL<64, 1>), __VA_ARGS__);                                       \
            else if (vpl <= 4) hipLaunchKernelGGL((KERNEL<64, 4>), __VA_ARGS__);                                  \
            else if (vpl <= 8) hipLaunchKernelGGL((KERNEL<64, 8>), __VA_ARGS__);                                  \
            else hipLaunchKernelGGL((KERNEL<64, 16>), __VA_ARGS__);                                               \
        }                                                                                                         \
    } while (0)

extern "C" moe_status moe_route_topk(moe_ctx* ctx, void* stream, const float* logits, int T, int E, int k,
                                     moe_score fn, int norm_topk, float scale,
                                     int32_t* topk_idx, float* topk_prob, int32_t* counts) {
    if (!ctx) return MOE_ERR_ARG;
    if (!logits || !topk_idx || !topk_prob) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk: NULL pointer");
    if (T < 0 || E < 1 || E > ROUTE_MAX_E || k < 1 || k > 32 || k > E)
        MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk: need T>=0, 1<=k<=min(E,32), E<=%d (T=%d E=%d k=%d)", ROUTE_MAX_E, T, E, k);
    if (fn != MOE_SCORE_SOFTMAX && fn != MOE_SCORE_SIGMOID) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk: bad score fn");
    hipStream_t s = (hipStream_t)stream;
    if (T == 0) {
        if (counts) moe_launch_fill_i32(counts, E, 0, s);
        return MOE_OK;
    }
    const int lpt = route_narrow(E, k, 1) ? 16 : 64;
    // many tokens: large workgroups, so that fewer of them add their histograms to the shared one
    // (and one alone where it can: nothing to clear then)
    const int threads = T > 4096 || (T > 256 / lpt && T <= 1024 / lpt) ? 1024 : 256, tokens = threads / lpt;
    const dim3 grid((T + tokens - 1) / tokens), block(threads);
    if (counts && grid.x > 1) moe_launch_fill_i32(counts, E, 0, s);
    ROUTE_CASES(route_topk_kernel, grid, block, (size_t)E * sizeof(int32_t), s, logits, T, E, k, (int)fn, norm_topk, scale,
                topk_idx, topk_prob, counts);
    MOE_LAUNCH_CHECK(ctx, "route_topk_kernel");
    return MOE_OK;
}

extern "C" moe_status moe_route_topk_grouped(moe_ctx* ctx, void* stream, const float* logits, const float* expert_bias,
                                             int T, int E, int k, int n_group, int topk_group,
                                             moe_score fn, int norm_topk, float scale,
                                             int32_t* topk_idx, float* topk_prob, int32_t* counts) {
    if (!ctx) return MOE_ERR_ARG;
    if (!logits || !topk_idx || !topk_prob) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk_grouped: NULL pointer");
    if (T < 0 || E < 1 || E > ROUTE_MAX_E || k < 1 || k > 32 || k > E)
        MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk_grouped: need T>=0, 1<=k<=min(E,32), E<=%d (T=%d E=%d k=%d)",
                 ROUTE_MAX_E, T, E, k);
    if (n_group < 1 || n_group > 64 || E % n_group || topk_group < 1 || topk_group > n_group || k % topk_group ||
        k / topk_group > E / n_group)
        MOE_FAIL(ctx, MOE_ERR_ARG,
                 "moe_route_topk_grouped: need 1<=topk_group<=n_group<=64, E %% n_group == 0, k %% topk_group == 0 and "
                 "k/topk_group <= E/n_group (E=%d k=%d n_group=%d topk_group=%d)", E, k, n_group, topk_group);
    if (fn != MOE_SCORE_SOFTMAX && fn != MOE_SCORE_SIGMOID) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk_grouped: bad score fn");
    hipStream_t s = (hipStream_t)stream;
    if (T == 0) {
        if (counts) moe_launch_fill_i32(counts, E, 0, s);
        return MOE_OK;
    }
    const int lpt = route_narrow(E, k, n_group) ? 16 : 64;
    int lpg = lpt;  // lanes per group: the largest power of two with room for all groups
    while (lpg > 1 && lpg * n_group > lpt) lpg >>= 1;
    // (many tokens: as moe_route_topk, with 35 KB of LDS at 256 experts)
    const int threads = lpt == 16 && T > 4096 ? 512 : 256, tokens = threads / lpt, gs = E / n_group;
    const uint32_t gs_magic = ((1u << 20) + gs - 1) / gs;  // (e * gs_magic) >> 20 == e / gs for e < 1024: the excess, e * gs at most, stays below 2^20
    const dim3 grid((T + tokens - 1) / tokens), block(threads);
    if (counts && grid.x > 1) moe_launch_fill_i32(counts, E, 0, s);
    const size_t shm = (size_t)E * sizeof(int32_t) + (size_t)tokens * (E + E / 16 + 1) * sizeof(float);
    ROUTE_CASES(route_topk_grouped_kernel, grid, block, shm, s, logits, expert_bias, T, E, k, n_group, topk_group, lpg, gs_magic,
                (int)fn, norm_topk, scale, topk_idx, topk_prob, counts);
    MOE_LAUNCH_CHECK(ctx, "route_topk_grouped_kernel");
    return MOE_OK;
}

extern "C" moe_status moe_route_topk_bwd(moe_ctx* ctx, void* stream, const float* logits, const int32_t* topk_idx,
                                         const float* dprob, int T, int E, int k, moe_score fn, int norm_topk,
                                         float scale, float* dlogits) {
    if (!ctx) return MOE_ERR_ARG;
    if (!logits || !topk_idx || !dprob || !dlogits) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk_bwd: NULL pointer");
    if (T < 0 || E < 1 || E > ROUTE_MAX_E || k < 1 || k > 32 || k > E)
        MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk_bwd: need T>=0, 1<=k<=min(E,32), E<=%d (T=%d E=%d k=%d)", ROUTE_MAX_E, T, E, k);
    if (fn != MOE_SCORE_SOFTMAX && fn != MOE_SCORE_SIGMOID) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_route_topk_bwd: bad score fn");
    if (T == 0) return MOE_OK;
    const int lpt = route_narrow(E, k, 1) ? 16 : 64, tokens = 256 / lpt;
    const dim3 grid((T + tokens - 1) / tokens), block(256);
    ROUTE_CASES(route_topk_bwd_kernel, grid, block, 0, (hipStream_t)stream, logits, topk_idx, dprob, T, E, k, (int)fn, norm_topk,
                scale, dlogits);
    MOE_LAUNCH_CHECK(ctx, "route_topk_bwd_kernel");
    return MOE_OK;
}

extern "C" moe_status moe_aux_loss(moe_ctx* ctx, void* stream, const float* logits, const int32_t* counts,
                                   int T, int E, int k, moe_score fn, float coeff, float dloss, int accumulate,
                                   float* loss, float* dlogits) {
    if (!ctx) return MOE_ERR_ARG;
    if (!logits || !counts || !loss) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_aux_loss: NULL pointer");
    if (T < 1 || E < 1 || E > ROUTE_MAX_E || k < 1)
        MOE_FAIL(ctx, MOE_ERR_ARG, "moe_aux_loss: need T>=1, 1<=E<=%d, k>=1 (T=%d E=%d k=%d)", ROUTE_MAX_E, T, E, k);
    if (fn != MOE_SCORE_SOFTMAX && fn != MOE_SCORE_SIGMOID) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_aux_loss: bad score fn");
    const int nblocks = (T + AUX_TOKENS - 1) / AUX_TOKENS;
    if (MOE_WS_RESERVED + (size_t)nblocks * sizeof(double) > ctx->ws_bytes)
        MOE_FAIL(ctx, MOE_ERR_WORKSPACE, "moe_aux_loss: workspace %zu B < %zu B", ctx->ws_bytes,
                 MOE_WS_RESERVED + (size_t)nblocks * sizeof(double));
    const int lpt = E <= 256 ? 16 : 64;
    double* const partial = (double*)((char*)ctx->ws + MOE_WS_RESERVED);
    const float wscale = (float)((double)coeff * E / ((double)T * T * k));
    ROUTE_CASES(aux_loss_kernel, dim3(nblocks), dim3(lpt == 16 ? 16 * AUX_TOKENS : 1024), 0, (hipStream_t)stream, logits, counts, T, E,
                (int)fn, wscale, dloss, accumulate, dlogits, partial, loss);
    if (nblocks > 1) hipLaunchKernelGGL(aux_loss_sum_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, partial, nblocks, loss);
    MOE_LAUNCH_CHECK(ctx, "aux_loss_kernel");
    return MOE_OK;
}
