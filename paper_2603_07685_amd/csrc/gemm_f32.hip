// All-fp32 grouped GEMMs (dt = MOE_F32): the same three calls as gemm.hip with fp32 operands, fp32 accumulation and fp32
// results.  Same conventions as the bf16 path: rows >= offsets[E] untouched, empty experts write zero weight gradients,
// inconsistent offsets raise the error word and nothing is written.
//
// One kernel, OUT[i,j] = sum_c P[i,c] * Q[j,c], on a BT x BT output tile (128 or 64) per 256-thread workgroup:
//     forward : P = A [rows,K]           Q = W_e [N,K]
//     dgrad   : P = dC [rows,N]          Q = W_e as [K,N]^T
//     wgrad   : P = dC as [N,rows]^T     Q = A as [K,rows]^T
// Bound: the fp32 matrix rate (v_mfma_f32_16x16x4_f32: exact products, fp32 sums; 157 TFLOP/s nominal, a large library
// product reaches 153 on these chips).  Four waves as 2 x 2, wave tile BT/2 x BT/2; the contraction is walked 16 elements
// per stage: a stage is BT/32 squared blocks x 4 MFMAs of 32 cycles per wave against (BT = 128) 16 KB of operands, so
// registers hold the next stage's operands while two LDS buffers alternate, one barrier per stage, and the loads have a
// whole stage (2048 cycles at BT = 128) to arrive.  BT = 64 trades operand reuse for four times as many workgroups where
// the larger tile would leave compute units idle (moe_gg_f32_tile below).
// LDS: an operand whose contraction index is contiguous in memory is kept [row][16] with a pitch of 20 floats, one
// 16-byte read giving a lane contraction elements 4 g .. 4 g + 3 (g = lane / 16; MFMA step j takes element j of every
// lane, the order inside a stage is free); the other kind is kept [16][column] with a pitch of BT + 4 floats, read
// element by element in the same order.  The latter is free of bank conflicts; of the former's LDS cycles 49 % are conflicts
// (both operands row-major: forward; 28 % with one, the data gradients), at LDS instructions in 25-35 % of the time and the
// matrix pipes busy 55-69 % (T 2048, h 1024, f 512).
// Measured (T 2048, h 1024, f 512, 8 experts, top-2, MI355X): the six GEMMs of a training step took 29.19 ms with one
// thread per output element (uncoalesced, no reuse); with this kernel 0.47 ms = 82 TFLOP/s (the step: 29.4 -> 0.54 ms).
#include "common.h"

#define F32_THREADS 256
#define F32_MAX_E 1024
#define GF_BK 16

enum { GF_FWD = 0, GF_DGRAD = 1, GF_WGRAD = 2 };
enum { GF_STORE = 0, GF_SWIGLU = 1, GF_SWIGLU_BWD = 2 };

struct gf_args {
    const float* P;  // fwd: A, dgrad / wgrad: dC
    const float* Q;  // fwd / dgrad: W [E,N,K], wgrad: A
    const int32_t* offsets;
    int E, N, K;
    int64_t Rcap;
    float* out;      // fwd: C (may be NULL with SwiGLU), dgrad: dA or dZ, wgrad: dW
    float* out_act;  // fwd SwiGLU: activation [rows, N/2]
    const float* Zsaved;
    const float* row_prob;
    int accumulate;
    int* dev_err;
};

__device__ __forceinline__ float sigmoid32(float g) { return 1.0f / (1.0f + expf(-g)); }

// VEC: every row starts on a 16-byte boundary (row lengths are multiples of 4 floats and so are the bases): operands move
// 16 bytes per lane; else element by element.
template <int MODE, int EPI, int BT, bool VEC>
__global__ __launch_bounds__(F32_THREADS, 2) void gf_kernel(const gf_args a) {
    constexpr bool P_CMAJ = MODE == GF_WGRAD, Q_CMAJ = MODE != GF_FWD;
    constexpr int KP = GF_BK + 4, CP = BT + 4;              // LDS pitches (floats) of the two kinds of tile
    constexpr int TILE = BT * KP > GF_BK * CP ? BT * KP : GF_BK * CP;
    constexpr int NP = BT / 64;                             // 16-byte pieces per thread, operand and stage
    constexpr int NB = BT / 32;                             // 16 x 16 blocks per wave and direction
    __shared__ __attribute__((aligned(16))) float lds[2][2][TILE];
    __shared__ tile_pick_lds pick;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int N = a.N, K = a.K;
    const int half = EPI == GF_SWIGLU ? N >> 1 : 0;
    const int J = MODE == GF_FWD ? N : K;
    const int tiles_j = EPI == GF_SWIGLU ? (half + BT / 2 - 1) / (BT / 2) : (J + BT - 1) / BT;
    const int tiles_iw = (N + BT - 1) / BT;                 // wgrad only

    // ---- this workgroup's tile ----
    int e, ti, tj, row_lo, row_hi;
    {
        int u;
        if (!tile_pick<F32_THREADS>(a.offsets, a.E, a.Rcap, a.dev_err, MODE == GF_WGRAD ? 0 : BT,
                                    MODE == GF_WGRAD ? tiles_iw * tiles_j : tiles_j, pick, e, u, row_lo, row_hi)) return;
        const int tiles_i = MODE == GF_WGRAD ? tiles_iw : (row_hi - row_lo + BT - 1) / BT;
        tj = u / tiles_i;
        ti = u - tj * tiles_i;
    }
    const int64_t i0 = MODE == GF_WGRAD ? (int64_t)ti * BT : row_lo + (int64_t)ti * BT;
    const int64_t i_end = MODE == GF_WGRAD ? N : row_hi;
    const int j0 = EPI == GF_SWIGLU ? tj * (BT / 2) : tj * BT;
    const int64_t c_lo = MODE == GF_WGRAD ? row_lo : 0, c_hi = MODE == GF_WGRAD ? row_hi : (MODE == GF_FWD ? K : N);
    const int KT = (int)((c_hi - c_lo + GF_BK - 1) / GF_BK);
    // column of the output that Q tile row rho stands for (-1: outside)
    auto q_col = [&](int rho) {
        if (EPI == GF_SWIGLU) {
            const int f = j0 + (rho < BT / 2 ? rho : rho - BT / 2);
            return f < half ? (rho < BT / 2 ? f : half + f) : -1;
        }
        return j0 + rho < J ? j0 + rho : -1;
    };

    // ---- operand fetch: NP pieces of 4 floats per thread ----
    // contraction-contiguous: piece = row 64 p + tid / 4, elements 4 (tid % 4) ..; the other kind: piece = contraction row
    // (1024 / BT) p + tid / (BT / 4), columns 4 (tid % (BT / 4)) ..
    const float* const Qe = MODE == GF_WGRAD ? a.Q : a.Q + (int64_t)e * N * K;
    f32x4_t rp[NP], rq[NP];
    auto fetch4 = [&](const float* src, int64_t limit) {  // elements 0 .. limit - 1 of the piece exist
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (VEC) {
            if (limit > 0) v = *(const f32x4_t*)src;
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (x < limit) v[x] = src[x];
        }
        return v;
    };
    auto load = [&](int kt) {
        const int64_t c0 = c_lo + (int64_t)kt * GF_BK;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if (P_CMAJ) {
                const int64_t c = c0 + p * (1024 / BT) + tid / (BT / 4);
                const int64_t i = i0 + 4 * (tid % (BT / 4));
                rp[p] = fetch4(a.P + c * N + i, c < c_hi ? i_end - i : 0);
            } else {
                const int64_t i = i0 + 64 * p + (tid >> 2), c = c0 + 4 * (tid & 3);
                rp[p] = fetch4(a.P + i * (MODE == GF_FWD ? K : N) + c, i < i_end ? c_hi - c : 0);
            }
            if (Q_CMAJ) {
                const int64_t c = c0 + p * (1024 / BT) + tid / (BT / 4);
                const int j = j0 + 4 * (tid % (BT / 4));
                rq[p] = fetch4(Qe + c * K + j, c < c_hi ? J - j : 0);
            } else {
                const int n = q_col(64 * p + (tid >> 2));
                const int64_t c = c0 + 4 * (tid & 3);
                rq[p] = fetch4(Qe + (int64_t)n * K + c, n >= 0 ? c_hi - c : 0);
            }
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int km = (64 * p + (tid >> 2)) * KP + 4 * (tid & 3);
            const int cm = (p * (1024 / BT) + tid / (BT / 4)) * CP + 4 * (tid % (BT / 4));
            *(f32x4_t*)(lds[buf][0] + (P_CMAJ ? cm : km)) = rp[p];
            *(f32x4_t*)(lds[buf][1] + (Q_CMAJ ? cm : km)) = rq[p];
        }
    };
    const int l16 = lane & 15, g = lane >> 4;
    auto p_row = [&](int i) { return wm * (BT / 2) + 16 * i; };
    auto q_row = [&](int j) {
        return EPI == GF_SWIGLU ? (j / (NB / 2)) * (BT / 2) + wn * (BT / 4) + (j % (NB / 2)) * 16 : wn * (BT / 2) + 16 * j;
    };
    auto frag = [&](const float* t, bool cmaj, int row) {
        if (!cmaj) return *(const f32x4_t*)(t + (row + l16) * KP + 4 * g);
        f32x4_t v;
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = t[(4 * g + x) * CP + row + l16];
        return v;
    };

    f32x4_t acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (KT > 0) {
        load(0);
        store(0);
        if (KT > 1) load(1);
        for (int kt = 0; kt < KT; ++kt) {
            __syncthreads();  // stage kt is in its buffer; everyone is past the other buffer's last reads
            if (kt + 1 < KT) store((kt + 1) & 1);
            if (kt + 2 < KT) load(kt + 2);
            const float* const tp = lds[kt & 1][0];
            const float* const tq = lds[kt & 1][1];
            f32x4_t fp[NB], fq[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) fp[i] = frag(tp, P_CMAJ, p_row(i));
#pragma unroll
            for (int j = 0; j < NB; ++j) fq[j] = frag(tq, Q_CMAJ, q_row(j));
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fq[j][x], fp[i][x], acc[i][j], 0, 0, 0);
        }
    }

    // ---- output: a lane holds, per block, one output row (P index l16) and the 4 consecutive columns 4 g .. 4 g + 3 ----
    auto put4 = [&](float* dst, f32x4_t v, int limit, bool add) {
        if (VEC) {
            if (limit <= 0) return;
            if (add) v += *(const f32x4_t*)dst;
            *(f32x4_t*)dst = v;
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (x < limit) dst[x] = add ? dst[x] + v[x] : v[x];
        }
    };
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int64_t r = i0 + p_row(i) + l16;
        if (r >= i_end) continue;
        const float pr = (EPI != GF_STORE && a.row_prob) ? a.row_prob[r] : 1.0f;
        if (EPI == GF_SWIGLU) {
#pragma unroll
            for (int j = 0; j < NB / 2; ++j) {
                const int f = j0 + q_row(j) + 4 * g;         // feature: gate column f, up column half + f
                const f32x4_t gt = acc[i][j], up = acc[i][j + NB / 2];
                f32x4_t act;
#pragma unroll
                for (int x = 0; x < 4; ++x) act[x] = pr * (gt[x] * sigmoid32(gt[x]) * up[x]);
                if (a.out) {
                    put4(a.out + r * N + f, gt, half - f, false);
                    put4(a.out + r * N + half + f, up, half - f, false);
                }
                put4(a.out_act + r * half + f, act, half - f, false);
            }
        } else {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int c = j0 + q_row(j) + 4 * g;
                if (EPI == GF_SWIGLU_BWD) {
                    const f32x4_t gt = fetch4(a.Zsaved + r * 2 * K + c, K - c), up = fetch4(a.Zsaved + r * 2 * K + K + c, K - c);
                    f32x4_t dg, du;
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const float s = sigmoid32(gt[x]), d = acc[i][j][x];
                        dg[x] = pr * d * up[x] * s * (1.0f + gt[x] * (1.0f - s));
                        du[x] = pr * d * gt[x] * s;
                    }
                    put4(a.out + r * 2 * K + c, dg, K - c, false);
                    put4(a.out + r * 2 * K + K + c, du, K - c, false);
                } else {
                    put4(a.out + (MODE == GF_WGRAD ? ((int64_t)e * N + r) * K : r * (int64_t)J) + c, acc[i][j], J - c,
                         MODE == GF_WGRAD && a.accumulate);
                }
            }
        }
    }
}

// Tile size.  128 halves the operand traffic, 64 has four times the workgroups and loses less to partly filled tiles and
// to a last, half-empty round of them; eight 128-tiles per compute unit is where the two meet.  The number of row tiles
// depends on the device's offsets; Rcap / 128 is taken.  Measured, whole training step, 8 experts, top-2 (64 against 128):
// T 256, h 128, f 256: 106 us against 178; T 2048, h 1024, f 512: 537 against 665; T 4096, h 1024, f 512: 906 against 1042;
// T 8192, h 1024, f 1024 (8 tiles per unit in fc1): 3.04 ms against 3.05; T 8192, h 2048, f 2048: 11.4 against 10.7;
// T 8192, h 4096, f 2048: 22.6 against 20.7 ms (119 TFLOP/s).
int moe_gg_f32_tile(int num_cu, bool wgrad, int E, int N, int out_cols, int64_t Rcap) {
    const int64_t cols = ceil_div64(out_cols, 128);
    const int64_t tiles = wgrad ? (int64_t)E * ceil_div64(N, 128) * cols : ceil_div64(Rcap, 128) * cols;
    return tiles >= 8 * (int64_t)(num_cu > 0 ? num_cu : 256) ? 128 : 64;
}

template <int MODE, int EPI>
static moe_status gf_launch(moe_ctx* ctx, hipStream_t s, const char* who, const gf_args& a) {
    if (a.E > F32_MAX_E) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: E > %d", who, F32_MAX_E);
    const int out_cols = EPI == GF_SWIGLU ? a.N : (MODE == GF_FWD ? a.N : a.K);
    const int bt = moe_gg_f32_tile(ctx->num_cu, MODE == GF_WGRAD, a.E, a.N, out_cols, a.Rcap);
    const int64_t tiles_j = EPI == GF_SWIGLU ? ceil_div64(a.N / 2, bt / 2) : ceil_div64(out_cols, bt);
    // (every expert may end in a partly filled row tile)
    const int64_t grid = ceil_div64(tiles_j * (MODE == GF_WGRAD ? a.E * ceil_div64(a.N, bt) : ceil_div64(a.Rcap, bt) + a.E), 8) * 8;
    if (grid > 0x7fffffffLL) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: problem too large for the fp32 path", who);
    const uintptr_t bits = (uintptr_t)a.P | (uintptr_t)a.Q | (uintptr_t)a.out | (uintptr_t)a.out_act | (uintptr_t)a.Zsaved;
    const bool vec = a.N % 4 == 0 && a.K % 4 == 0 && (EPI != GF_SWIGLU || a.N % 8 == 0) && bits % 16 == 0;
    const dim3 g((unsigned)grid), b(F32_THREADS);
    if (vec && bt == 128) hipLaunchKernelGGL((gf_kernel<MODE, EPI, 128, true>), g, b, 0, s, a);
    else if (vec) hipLaunchKernelGGL((gf_kernel<MODE, EPI, 64, true>), g, b, 0, s, a);
    else if (bt == 128) hipLaunchKernelGGL((gf_kernel<MODE, EPI, 128, false>), g, b, 0, s, a);
    else hipLaunchKernelGGL((gf_kernel<MODE, EPI, 64, false>), g, b, 0, s, a);
    MOE_LAUNCH_CHECK(ctx, who);
    return MOE_OK;
}

moe_status moe_gg_f32_fwd(moe_ctx* ctx, hipStream_t s, const void* A, const void* B, const int32_t* offsets, int E, int N,
                          int K, int64_t Rcap, int swiglu, const float* row_prob, void* C, void* C_act) {
    const gf_args a = {(const float*)A, (const float*)B, offsets, E, N, K, Rcap, (float*)C, (float*)C_act, nullptr, row_prob, 0,
                       ctx->dev_err};
    return swiglu ? gf_launch<GF_FWD, GF_SWIGLU>(ctx, s, "moe_grouped_gemm_fwd(f32)", a)
                  : gf_launch<GF_FWD, GF_STORE>(ctx, s, "moe_grouped_gemm_fwd(f32)", a);
}

moe_status moe_gg_f32_dgrad(moe_ctx* ctx, hipStream_t s, const void* dC, const void* B, const int32_t* offsets, int E, int N,
                            int K, int64_t Rcap, const void* Z_saved, const float* row_prob, void* dA) {
    const gf_args a = {(const float*)dC, (const float*)B, offsets, E, N, K, Rcap, (float*)dA, nullptr, (const float*)Z_saved,
                       row_prob, 0, ctx->dev_err};
    return Z_saved ? gf_launch<GF_DGRAD, GF_SWIGLU_BWD>(ctx, s, "moe_grouped_gemm_dgrad(f32)", a)
                   : gf_launch<GF_DGRAD, GF_STORE>(ctx, s, "moe_grouped_gemm_dgrad(f32)", a);
}

moe_status moe_gg_f32_wgrad(moe_ctx* ctx, hipStream_t s, const void* A, const void* dC, const int32_t* offsets, int E, int N,
                            int K, int64_t Rcap, int accumulate, void* dB) {
    const gf_args a = {(const float*)dC, (const float*)A, offsets, E, N, K, Rcap, (float*)dB, nullptr, nullptr, nullptr,
                       accumulate ? 1 : 0, ctx->dev_err};
    return gf_launch<GF_WGRAD, GF_STORE>(ctx, s, "moe_grouped_gemm_wgrad(f32)", a);
}
