// All-fp32 grouped GEMMs (dt = MOE_F32): the same three calls as gemm.hip with fp32 operands, fp32 accumulation and fp32
// results.  Same conventions as the bf16 path: rows >= offsets[E] untouched, empty experts write zero weight gradients,
// inconsistent offsets raise the error word and nothing is written.
//
// OUT[i,j] = sum_c P[i,c] * Q[j,c], one output tile per 256-thread workgroup, by one of two kernels (gs_serves chooses):
//     forward : P = A [rows,K]           Q = W_e [N,K]
//     dgrad   : P = dC [rows,N]          Q = W_e as [K,N]^T
//     wgrad   : P = dC as [N,rows]^T     Q = A as [K,rows]^T
// gf_kernel: BT x BT tiles (128 or 64) on the fp32 matrix instruction; small calls, short contractions, any row length.
// gs_kernel: every operand as three bf16 parts on the bf16 instruction, sixteen times the fp32 one's rate; see there.
//
// gf_kernel.  Bound: the fp32 matrix rate (v_mfma_f32_16x16x4_f32: exact products, fp32 sums; 157 TFLOP/s nominal, a large library
// product reaches 153 on these chips).  Four waves as 2 x 2, wave tile BT/2 x BT/2; the contraction is walked 16 elements
// per stage: a stage is BT/32 squared blocks x 4 MFMAs of 32 cycles per wave against (BT = 128) 16 KB of operands, so
// registers hold the next stage's operands while two LDS buffers alternate, one barrier per stage, and the loads have a
// whole stage (2048 cycles at BT = 128) to arrive.  BT = 64 trades operand reuse for four times as many workgroups where
// the larger tile would leave compute units idle (gf_tile below).
// LDS: an operand whose contraction index is contiguous in memory is kept [row][16] with a pitch of 20 floats, one
// 16-byte read giving a lane contraction elements 4 g .. 4 g + 3 (g = lane / 16; MFMA step j takes element j of every
// lane, the order inside a stage is free); the other kind is kept [16][column] with a pitch of BT + 4 floats, read
// element by element in the same order.  The latter is free of bank conflicts; of the former's LDS cycles 49 % are conflicts
// (both operands row-major: forward; 28 % with one, the data gradients), at LDS instructions in 25-35 % of the time and the
// matrix pipes busy 55-69 % (T 2048, h 1024, f 512).
// Measured (T 2048, h 1024, f 512, 8 experts, top-2, MI355X): the six GEMMs of a training step took 29.19 ms with one
// thread per output element (uncoalesced, no reuse); with this kernel 0.47 ms = 82 TFLOP/s (the step: 29.4 -> 0.54 ms).
#include "gemm.h"
#include <type_traits>

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

// elements 0 .. limit - 1 of four at src (the others: 0)
template <bool VEC>
__device__ __forceinline__ f32x4_t fetch4(const float* src, int64_t limit) {
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    if (VEC) {
        if (limit > 0) v = *(const f32x4_t*)src;
    } else {
#pragma unroll
        for (int x = 0; x < 4; ++x)
            if (x < limit) v[x] = src[x];
    }
    return v;
}

// Output.  A lane holds, per row block i, quads of consecutive columns: value(i, q) are the four from tile column col(q) on of
// tile row row(i); SwiGLU: quad q + NQ / 2 has the up projections of quad q's gates.
template <int MODE, int EPI, bool VEC, int NI, int NQ, typename VALUE, typename ROW, typename COL>
__device__ __forceinline__ void gf_output(const gf_args& a, int e, int64_t i0, int64_t i_end, int j0, VALUE&& value, ROW&& row, COL&& col) {
    const int N = a.N, K = a.K, half = EPI == GF_SWIGLU ? N >> 1 : 0, J = MODE == GF_FWD ? N : K;
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
    // (one quad per row: all the saved pre-activations are asked for at once, not row by row behind the stores)
    constexpr bool AHEAD = EPI == GF_SWIGLU_BWD && VEC && NQ == 1;
    f32x4_t zg[AHEAD ? NI : 1], zu[AHEAD ? NI : 1];
    if (AHEAD) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const float* const z = a.Zsaved + min(i0 + row(i), i_end - 1) * 2 * K + min(j0 + col(0), K - 4);
            zg[i] = *(const f32x4_t*)z;
            zu[i] = *(const f32x4_t*)(z + K);
        }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int64_t r = i0 + row(i);
        if (r >= i_end) continue;
        const float pr = (EPI != GF_STORE && a.row_prob) ? a.row_prob[r] : 1.0f;
        if (EPI == GF_SWIGLU) {
#pragma unroll
            for (int q = 0; q < NQ / 2; ++q) {
                const int f = j0 + col(q);                   // feature: gate column f, up column half + f
                const f32x4_t gt = value(i, q), up = value(i, q + NQ / 2);
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
            for (int q = 0; q < NQ; ++q) {
                const int c = j0 + col(q);
                const f32x4_t v = value(i, q);
                if (EPI == GF_SWIGLU_BWD) {
                    const f32x4_t gt = AHEAD ? zg[i] : fetch4<VEC>(a.Zsaved + r * 2 * K + c, K - c);
                    const f32x4_t up = AHEAD ? zu[i] : fetch4<VEC>(a.Zsaved + r * 2 * K + K + c, K - c);
                    f32x4_t dg, du;
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const float s = sigmoid32(gt[x]), d = v[x];
                        dg[x] = pr * d * up[x] * s * (1.0f + gt[x] * (1.0f - s));
                        du[x] = pr * d * gt[x] * s;
                    }
                    put4(a.out + r * 2 * K + c, dg, K - c, false);
                    put4(a.out + r * 2 * K + K + c, du, K - c, false);
                } else {
                    put4(a.out + (MODE == GF_WGRAD ? ((int64_t)e * N + r) * K : r * (int64_t)J) + c, v, J - c,
                         MODE == GF_WGRAD && a.accumulate);
                }
            }
        }
    }
}

// VEC: every row starts on a 16-byte boundary (row lengths are multiples of 4 floats and so are the bases): operands move
// 16 bytes per lane; else element by element.
// `block`: the workgroup's place among those of its call
template <int BT>
struct gf_lds {
    static constexpr int KP = GF_BK + 4, CP = BT + 4;       // pitches (floats) of the two kinds of tile
    __attribute__((aligned(16))) float tile[2][2][BT * KP > GF_BK * CP ? BT * KP : GF_BK * CP];
    tile_pick_lds pick;
};
template <int MODE, int EPI, int BT, bool VEC>
__device__ __forceinline__ void gf_body(const gf_args& a, gf_lds<BT>& l, const int block) {
    constexpr bool P_CMAJ = MODE == GF_WGRAD, Q_CMAJ = MODE != GF_FWD;
    constexpr int KP = gf_lds<BT>::KP, CP = gf_lds<BT>::CP;
    constexpr int NP = BT / 64;                             // 16-byte pieces per thread, operand and stage
    constexpr int NB = BT / 32;                             // 16 x 16 blocks per wave and direction
    auto& lds = l.tile;
    tile_pick_lds& pick = l.pick;
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
                                    MODE == GF_WGRAD ? tiles_iw * tiles_j : tiles_j, block, pick, e, u, row_lo, row_hi)) return;
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
    auto load = [&](int kt) {
        const int64_t c0 = c_lo + (int64_t)kt * GF_BK;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if (P_CMAJ) {
                const int64_t c = c0 + p * (1024 / BT) + tid / (BT / 4);
                const int64_t i = i0 + 4 * (tid % (BT / 4));
                rp[p] = fetch4<VEC>(a.P + c * N + i, c < c_hi ? i_end - i : 0);
            } else {
                const int64_t i = i0 + 64 * p + (tid >> 2), c = c0 + 4 * (tid & 3);
                rp[p] = fetch4<VEC>(a.P + i * (MODE == GF_FWD ? K : N) + c, i < i_end ? c_hi - c : 0);
            }
            if (Q_CMAJ) {
                const int64_t c = c0 + p * (1024 / BT) + tid / (BT / 4);
                const int j = j0 + 4 * (tid % (BT / 4));
                rq[p] = fetch4<VEC>(Qe + c * K + j, c < c_hi ? J - j : 0);
            } else {
                const int n = q_col(64 * p + (tid >> 2));
                const int64_t c = c0 + 4 * (tid & 3);
                rq[p] = fetch4<VEC>(Qe + (int64_t)n * K + c, n >= 0 ? c_hi - c : 0);
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

    gf_output<MODE, EPI, VEC, NB, NB>(a, e, i0, i_end, j0, [&](int i, int j) { return acc[i][j]; }, [&](int i) { return p_row(i) + l16; },
                                      [&](int j) { return q_row(j) + 4 * g; });
}
template <int MODE, int EPI, int BT, bool VEC>
__global__ __launch_bounds__(F32_THREADS, 2) void gf_kernel(const gf_args a) {
    __shared__ gf_lds<BT> lds;
    gf_body<MODE, EPI, BT, VEC>(a, lds, (int)blockIdx.x);
}

// Independent small calls in one launch (a batch's; gemm_tile.hip: gt_fwd_jobs_kernel, gt_bwd_jobs_kernel), 64 x 64 tiles, 16-byte rows.
// A step, us, one launch each : together: T 425 h 320 f 192 E 4 k 4 140 : 117; T 128 h 256 f 256 E 22 k 8 98 : 87; with a shared expert
// T 285 h 576 f 192 E 6 k 1 194 : 97.
struct gf_jobs {
    gf_args a[GT_JOBS];
    int start[GT_JOBS + 1], turn;
};
__device__ __forceinline__ int gf_job_of(const gf_jobs& m, int block) {
    int j = 0;
#pragma unroll
    for (int x = 1; x < GT_JOBS; ++x) j += block >= m.start[x];
    return j;
}
template <int EPI>
__global__ __launch_bounds__(F32_THREADS, 2) void gf_fwd_jobs_kernel(const gf_jobs m) {
    __shared__ gf_lds<64> lds;
    const int j = gf_job_of(m, (int)blockIdx.x);
    gf_body<GF_FWD, EPI, 64, true>(m.a[j], lds, (int)blockIdx.x - m.start[j]);
}
template <int EPI>
__global__ __launch_bounds__(F32_THREADS, 2) void gf_bwd_jobs_kernel(const gf_jobs m) {
    __shared__ gf_lds<64> lds;
    const int at = gt_place_of((int)blockIdx.x, m.turn, m.start[GT_JOBS]), j = gf_job_of(m, at), block = at - m.start[j];
    if (j < 2) gf_body<GF_DGRAD, EPI, 64, true>(m.a[j], lds, block);
    else gf_body<GF_WGRAD, GF_STORE, 64, true>(m.a[j], lds, block);
}

// ---------------------------------------------------------------------------
// The same GEMMs on the bf16 matrix instruction, without losing a bit of the operands: every fp32 element is the sum of
// three bf16 numbers, x = hi + mid + lo (each the remainder rounded to 8 bits), and a product of two elements is the sum of
// the nine products of their parts, each exact in the matrix unit.  Eight are taken; the ninth, lo lo, is at most 2^-34 of the
// product, where a rounding of the sum is 2^-24 of the sum so far.  (lo mid and mid lo are up to 2^-24 of it together, and count where
// few terms of a sum are not zero.)  Sums in fp32, in the matrix unit's four roundings per 32 elements instead of 32.  Error against 64
// bits in units of 2^-24 sum |ab|, root mean square and largest of some million sums, fp32 instruction : six products : these
// eight; one term that is not zero 0.425 : 0.436 : 0.425, 1.00 : 1.71 : 1.01; two 0.44 : 0.37 : 0.36, 1.99 : 2.9 : 2.6 (the unit drops what
// lies below the last place of the larger product); four 0.45 : 0.30 : 0.29, 3.6 : 3.2 : 3.2; 32 0.47 : 0.20 : 0.20, 6.0 : 3.4 : 3.4.  The
// layer below: 8.7e-7 relative error on the fp32 instruction, 3.5e-7 here.
//
// BM x 128 tiles (BM = 64; weight gradients 128, whose contraction-major rows then fill 256-byte bank lines), four waves as
// 2 x 2, stages of 32 contraction elements.  Global loads run two to three stages ahead into registers; each element is split
// once per workgroup, in the gaps between the MFMAs of the stage before it is used, into three bf16 tiles in one of two LDS buffers;
// one barrier per stage.  What shaped it: a vector instruction issues for free beside a 32 x 32 x 16 MFMA up to about five
// (16 x 16 x 32: two), if it does not wait for the one before it (8 cycles there); v_dot2_f32_bf16, which would give a
// remainder in one instruction, shares the matrix pipe and doubled the time of a stage.
// Bound: the MFMAs of eight products, 1.17 us per 128 x 128 x 32 stage and unit at the clock the card holds, with loads and splitting
// mostly beside them; 6 us around a tile.  Measured (us a call, gf_kernel : six products : these eight), T 2048, h 1024, f 512, 8
// experts, top-2: fc1 + SwiGLU 104 : 84 : 92, fc2 55 : 45 : 48, weight gradients 72, 141 : 47, 92 : 50, 97 (rank^-1.2 loads 132, 260 : 76,
// 149 : 82, 162), fc2 data gradient + SwiGLU backward 70 : 57 : 60, fc1 data gradient 101 : 83 : 91; the
// step 504 : 408 : 434.
// ---------------------------------------------------------------------------
#define GS_BN 128

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

// The tile on the fp32 instruction, one stage of 16 after the other: for the rare tile whose operands the split cannot hold.
template <int MODE, int EPI, int BM, int NI, int NJ, typename PROW, typename QROW, typename COLAT>
__device__ __forceinline__ void gs_again(const gf_args& a, float* lds, f32x16_t (&acc)[NI][NJ], const float* Qe, int64_t i0,
                                         int64_t i_end, int j0, int64_t c_lo, int64_t c_hi, PROW p_row, QROW q_row, COLAT col_at) {
    constexpr bool P_CMAJ = MODE == GF_WGRAD, Q_CMAJ = MODE != GF_FWD;
    constexpr int PITCH = GF_BK + 1;
    const int tid = threadIdx.x, l32 = tid & 31, kh = (tid & 63) >> 5, N = a.N, K = a.K;
    const int half = EPI == GF_SWIGLU ? N >> 1 : 0, J = MODE == GF_FWD ? N : K;
    float *const tp = lds, *const tq = lds + BM * PITCH;    // [row][16]
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[i][j][x] = 0.f;
    for (int64_t c0 = c_lo; c0 < c_hi; c0 += GF_BK) {
        __syncthreads();
        for (int x = tid; x < BM * GF_BK; x += F32_THREADS) {
            const int at = P_CMAJ ? x % BM : x / GF_BK, c = P_CMAJ ? x / BM : x % GF_BK, r = col_at(P_CMAJ, at);
            tp[at * PITCH + c] = i0 + r < i_end && c0 + c < c_hi ? (P_CMAJ ? a.P[(c0 + c) * N + i0 + r] : a.P[(i0 + r) * (MODE == GF_FWD ? K : N) + c0 + c]) : 0.f;
        }
        for (int x = tid; x < GS_BN * GF_BK; x += F32_THREADS) {
            const int at = Q_CMAJ ? x % GS_BN : x / GF_BK, c = Q_CMAJ ? x / GS_BN : x % GF_BK, r = col_at(Q_CMAJ, at);
            const int n = EPI == GF_SWIGLU ? (j0 + (r & 63) < half ? (r >> 6) * half + j0 + (r & 63) : -1) : (j0 + r < J ? j0 + r : -1);
            tq[at * PITCH + c] = n >= 0 && c0 + c < c_hi ? (Q_CMAJ ? Qe[(c0 + c) * K + n] : Qe[(int64_t)n * K + c0 + c]) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int x = 0; x < GF_BK; x += 2)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(tq[(q_row(j) + l32) * PITCH + x + kh], tp[(p_row(i) + l32) * PITCH + x + kh],
                                                                     acc[i][j], 0, 0, 0);
    }
}

template <int MODE, int EPI, int BM>
__global__ __launch_bounds__(F32_THREADS, BM == 64 ? 2 : 1) void gs_kernel(const gf_args a) {
    constexpr bool P_CMAJ = MODE == GF_WGRAD, Q_CMAJ = MODE != GF_FWD;
    static_assert(!P_CMAJ || BM == 128, "contraction-major tiles have rows of 256 bytes");
    constexpr int BN = GS_BN, NI = BM / 64, NJ = 2;         // 32 x 32 blocks per wave and direction
    constexpr int P_PLANE = BM * 64, PLANE = (BM + BN) * 64, STAGE = 3 * PLANE;   // bytes: a part of P, of both, a stage
    constexpr int PP = BM / 64, PIECES = PP + 2;            // 8-element pieces per thread: P, Q
    __shared__ __attribute__((aligned(1024))) char lds[2 * STAGE];
    __shared__ tile_pick_lds pick;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    const int N = a.N, K = a.K;
    const int half = EPI == GF_SWIGLU ? N >> 1 : 0;
    const int J = MODE == GF_FWD ? N : K;
    const int tiles_j = EPI == GF_SWIGLU ? (half + 63) / 64 : (J + BN - 1) / BN;
    const int tiles_iw = (N + BM - 1) / BM;                 // wgrad only

    int e, ti, tj, row_lo, row_hi;
    {
        int u;
        if (!tile_pick<F32_THREADS>(a.offsets, a.E, a.Rcap, a.dev_err, MODE == GF_WGRAD ? 0 : BM,
                                    MODE == GF_WGRAD ? tiles_iw * tiles_j : tiles_j, (int)blockIdx.x, pick, e, u, row_lo, row_hi)) return;
        const int tiles_i = MODE == GF_WGRAD ? tiles_iw : (row_hi - row_lo + BM - 1) / BM;
        tj = u / tiles_i;
        ti = u - tj * tiles_i;
    }
    const int64_t i0 = MODE == GF_WGRAD ? (int64_t)ti * BM : row_lo + (int64_t)ti * BM;
    const int64_t i_end = MODE == GF_WGRAD ? N : row_hi;
    const int j0 = EPI == GF_SWIGLU ? tj * 64 : tj * BN;
    const int64_t c_lo = MODE == GF_WGRAD ? row_lo : 0, c_hi = MODE == GF_WGRAD ? row_hi : (MODE == GF_FWD ? K : N);
    const int KT = __builtin_amdgcn_readfirstlane((int)((c_hi - c_lo + 31) / 32));

    // ---- operand fetch: pieces of 8 floats, two quads that lie half a tile line apart, so that neighbouring lanes read
    // neighbouring 16 bytes ----
    // contraction-contiguous: piece = row 64 p + tid / 4, elements 4 t .. and 16 + 4 t .. (t = tid % 4); the other kind:
    // contraction row 16 p + tid / 16, columns 4 t .. and 64 + 4 t .. (t = tid % 16).  A piece is one 16-byte slot of the LDS tile:
    // contraction elements and columns are kept in that order there.  Rows and columns outside the tensor are replaced by
    // its last ones: what they compute is not stored.
    const float* const Qe = MODE == GF_WGRAD ? a.Q : a.Q + (int64_t)e * N * K;
    const float* src[PIECES];
    int second[2];                                          // elements from the first quad to the second: P, Q
    second[0] = second[1] = 16;
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
        const int r4 = tid >> 2, c4 = 4 * (tid & 3), r16 = tid >> 4, j4 = 4 * (tid & 15);
        if (p < PP) {
            if (P_CMAJ) {
                const int at = min((int)i0 + j4, (int)i_end - 4);
                src[p] = a.P + (c_lo + 16 * p + r16) * N + at;
                second[0] = min((int)i0 + 64 + j4, (int)i_end - 4) - at;
            } else {
                src[p] = a.P + min(i0 + 64 * p + r4, i_end - 1) * (MODE == GF_FWD ? K : N) + c4;
            }
        } else {
            const int q = p - PP;
            if (Q_CMAJ) {
                const int at = min(j0 + j4, J - 4);
                src[p] = Qe + (c_lo + 16 * q + r16) * K + at;
                second[1] = min(j0 + 64 + j4, J - 4) - at;
            } else if (EPI == GF_SWIGLU) {
                src[p] = Qe + ((int64_t)q * half + min(j0 + r4, half - 1)) * K + c4;
            } else {
                src[p] = Qe + (int64_t)min(j0 + 64 * q + r4, J - 1) * K + c4;
            }
        }
    }
    const int64_t p_step = P_CMAJ ? 32 * (int64_t)N : 32, q_step = Q_CMAJ ? 32 * (int64_t)K : 32;   // elements per stage
    f32x4_t raw[2][PIECES][2];                              // stage s in set s & 1
    const int total = (int)(c_hi - c_lo);
    auto load = [&](int set, int p, int s) __attribute__((always_inline)) {   // of stage s; behind the contraction's end: zeros
        const bool cmaj = p < PP ? P_CMAJ : Q_CMAJ;
        const int left = total - 32 * s;
        if (left >= 32) {
            raw[set][p][0] = *(const f32x4_t*)src[p];
            raw[set][p][1] = *(const f32x4_t*)(src[p] + (cmaj ? second[p >= PP] : 16));
        } else {
            raw[set][p][0] = raw[set][p][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            const int c = cmaj ? 16 * (p < PP ? p : p - PP) + (tid >> 4) : 4 * (tid & 3);   // contraction index in the stage
            if (c < left) raw[set][p][0] = *(const f32x4_t*)src[p];
            if (c + (cmaj ? 0 : 16) < left) raw[set][p][1] = *(const f32x4_t*)(src[p] + (cmaj ? second[p >= PP] : 16));
        }
        src[p] += p < PP ? p_step : q_step;
    };

    // ---- splitting, in units of five instructions that go between the MFMAs.  A result takes 8 cycles to the next
    // instruction while the matrix pipe is busy, so that two pairs of elements are in work at a time ----
    uint32_t parts[3][4];                                   // of the piece in work: hi, mid, lo, a pair of elements per word
    float rest[4], lead[4];
    uint32_t inexact = 0;                                   // low halves: what the third part does not hold
    // LDS.  Row-major tiles have rows of 64 bytes, four 16-byte slots, permuted so that the rows 4 i .. 4 i + 3 of i = 0 .. 3
    // (in the order in which the LDS takes the lanes of a 16-byte read, too) have their slots on different banks;
    // contraction-major ones rows of 256 bytes, slots ^ 4 * (row % 4): the 4 rows x 64 bytes of a transposing read are on
    // different banks.
    auto km_f = [](int row) { const int q = (row >> 2) & 3; return ((q << 1) ^ (3 * (q >> 1))) & 3; };   // 0 2 3 1
    auto cm_f = [](int row) { return 4 * (row & 3); };
    uint32_t put_at[PIECES];
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
        const int q = p < PP ? p : p - PP;
        const int r4 = 64 * q + (tid >> 2), r16 = 16 * q + (tid >> 4);
        const bool cmaj = p < PP ? P_CMAJ : Q_CMAJ;
        put_at[p] = (p < PP ? 0 : P_PLANE) + (cmaj ? r16 * 256 + ((tid & 15) ^ cm_f(r16)) * 16 : r4 * 64 + ((tid & 3) ^ km_f(r4)) * 16);
    }
    constexpr int UNITS = 11;                               // per piece: 2 x 5, then the stores
    auto split_unit = [&](int buf, int p, int u) __attribute__((always_inline)) {
        const int two = u / 5, v = u % 5, part = v >> 1;    // (two = 2: the stores)
        if (two < 2 && (v & 1) == 0) {
            if (v == 0) {
#pragma unroll
                for (int x = 0; x < 4; ++x) rest[x] = raw[buf][p][two][x];
            }
            uint32_t w0 = pack_bf16(rest[0], rest[1]), w1 = pack_bf16(rest[2], rest[3]);
            asm("" : "+v"(w0));                             // (else the compiler converts once more to widen it again)
            asm("" : "+v"(w1));
            parts[part][2 * two] = w0;
            parts[part][2 * two + 1] = w1;
            if (part < 2) {
                lead[0] = bf16_lo(w0);
                lead[1] = bf16_hi(w0);
                lead[2] = bf16_lo(w1);
                lead[3] = bf16_hi(w1);
            } else {
                inexact |= __float_as_uint(rest[0]) | __float_as_uint(rest[1]);
                inexact |= __float_as_uint(rest[2]) | __float_as_uint(rest[3]);
                asm("" : "+v"(inexact));                    // (here: left to the end of the stage, all of them stay alive)
            }
        } else if (two < 2) {
#pragma unroll
            for (int x = 0; x < 4; ++x) rest[x] -= lead[x];   // (exact: what a rounding to 8 bits leaves of 24)
        } else {
#pragma unroll
            for (int part = 0; part < 3; ++part)
                *(u32x4_t*)(lds + buf * STAGE + part * PLANE + put_at[p]) = u32x4_t{parts[part][0], parts[part][1], parts[part][2], parts[part][3]};
        }
    };

    // ---- fragments: 32 rows, contraction elements 4 t .. and 16 + 4 t .., t = 2 ks + lane / 32, of the stage ----
    const int l32 = lane & 31, kh = lane >> 5;
    auto p_row = [&](int i) { return wm * (BM / 2) + 32 * i; };
    auto q_row = [&](int j) { return EPI == GF_SWIGLU ? j * 64 + wn * 32 : wn * 64 + 32 * j; };
    // place in a contraction-major tile -> column, and what lies there in the others
    auto col_at = [](bool cmaj, int at) { return cmaj ? 64 * ((at >> 2) & 1) + 4 * (at >> 3) + (at & 3) : at; };
    const int km[2] = {l32 * 64 + (kh ^ km_f(l32)) * 16, l32 * 64 + ((2 + kh) ^ km_f(l32)) * 16};
    const int cm_row = 4 * kh + ((lane & 15) >> 2), cm_x = cm_f(cm_row);
    const int cm_at = cm_row * 256 + (lane & 1) * 8, cm_slot = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    auto frag = [&](const char* t, bool cmaj, int ks, int row) __attribute__((always_inline)) -> bf16x8_t {
        if (!cmaj) return *(const bf16x8_t*)(t + row * 64 + km[ks]);
        const char* p = t + ks * (8 * 256) + cm_at + ((row / 8 + cm_slot) ^ cm_x) * 16;
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p);
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p + 16 * 256));
        return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    bf16x8_t fp[3][2][NI], fq[3][2][NJ];                    // parts 0 hi, 1 mid, 2 lo
    auto read_p = [&](int buf, int part, int r) __attribute__((always_inline)) {   // r < 2 NI, in the order of use
        fp[part][r / NI][r % NI] = frag(lds + buf * STAGE + part * PLANE, P_CMAJ, r / NI, p_row(r % NI));
    };
    auto read_q = [&](int buf, int part, int r) __attribute__((always_inline)) {
        fq[part][r / NJ][r % NJ] = frag(lds + buf * STAGE + part * PLANE + P_PLANE, Q_CMAJ, r / NJ, q_row(r % NJ));
    };

    // The product of the leading parts has an accumulator of its own: the other products, 2^-8 and less of it, then do not
    // round at its magnitude.
    f32x16_t acc[NI][NJ], low[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[i][j][x] = low[i][j][x] = 0.f;
    constexpr int NM = 2 * NI * NJ;                         // MFMAs per product
    auto products = [&](int pp, int pq, auto&& slot) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    f32x16_t& d = pp + pq == 0 ? acc[i][j] : low[i][j];
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[pq][ks][j], fp[pp][ks][i], d, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    slot((ks * NI + i) * NJ + j);
                    __builtin_amdgcn_sched_barrier(0);
                }
    };
    auto barrier = []() __attribute__((always_inline)) {    // (no vector-memory wait: loads in flight go to registers)
        __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };
    auto stage = [&](int s, auto parity) __attribute__((always_inline)) {
        constexpr int b = decltype(parity)::value;          // s & 1: this stage's buffer, the set of the loads in flight
        // work between the MFMAs of the first seven products (weight gradients: six, 3 % faster there, 2 % slower elsewhere): the
        // splitting of stage s + 1 and the loads of stage s + 3
        constexpr int W = PIECES * (UNITS + 1), M = (MODE == GF_WGRAD ? 6 : 7) * NM;
        auto work = [&](int m) __attribute__((always_inline)) {
#pragma unroll
            for (int w = 0; w < W; ++w)
                if (w * M / W == m) {
                    if (w % (UNITS + 1) < UNITS) split_unit(b ^ 1, w / (UNITS + 1), w % (UNITS + 1));
                    else load(b ^ 1, w / (UNITS + 1), s + 3);
                }
        };
        auto reads_p = [&](int m, int buf, int part) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 2 * NI; ++r)
                if (r * NM / (2 * NI) == m) read_p(buf, part, r);
        };
        auto reads_q = [&](int m, int buf, int part) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 2 * NJ; ++r)
                if (r * NM / (2 * NJ) == m) read_q(buf, part, r);
        };
        // each product needs one new set of fragments, read during the one before it
        products(1, 1, [&](int m) __attribute__((always_inline)) { reads_q(m, b, 0); work(m); });
        products(1, 0, [&](int m) __attribute__((always_inline)) { reads_p(m, b, 2); work(NM + m); });
        products(2, 0, [&](int m) __attribute__((always_inline)) { reads_p(m, b, 0); work(2 * NM + m); });
        products(0, 0, [&](int m) __attribute__((always_inline)) { reads_q(m, b, 2); work(3 * NM + m); });
        products(0, 1, [&](int m) __attribute__((always_inline)) { work(4 * NM + m); });
        products(2, 1, [&](int m) __attribute__((always_inline)) { work(5 * NM + m); });
        products(1, 2, [&](int m) __attribute__((always_inline)) { work(6 * NM + m); });
        barrier();                                          // stage s + 1 is in its buffer, this one's has been read
        products(0, 2, [&](int m) __attribute__((always_inline)) { reads_p(m, b ^ 1, 1); reads_q(m, b ^ 1, 1); });
    };
    if (KT > 0) {
#pragma unroll
        for (int p = 0; p < PIECES; ++p) load(0, p, 0);
#pragma unroll
        for (int p = 0; p < PIECES; ++p) load(1, p, 1);
#pragma unroll
        for (int p = 0; p < PIECES; ++p) {
#pragma unroll
            for (int u = 0; u < UNITS; ++u) split_unit(0, p, u);
            load(0, p, 2);
        }
        barrier();
#pragma unroll
        for (int r = 0; r < 2 * NI; ++r) read_p(0, 1, r);
#pragma unroll
        for (int r = 0; r < 2 * NJ; ++r) read_q(0, 1, r);
        for (int s = 0; s < KT; s += 2) {
            stage(s, std::integral_constant<int, 0>{});
            stage(s + 1, std::integral_constant<int, 1>{});   // (an odd count: a stage of zeros, without an exit in mid-loop)
        }
    }

    // A result is kept if every element was the sum of its three parts, as it is from 2^-110 up to where rounding the
    // leading part overflows (and below, where 24 bits are not used), and if no sum left the range.  Otherwise (infinities and
    // NaN too) the tile is computed again on the fp32 instruction.
    bool again = (inexact & 0xffffu) != 0;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                acc[i][j][x] += low[i][j][x];
                again |= !(__builtin_fabsf(acc[i][j][x]) < INFINITY);
            }
    if (__syncthreads_or(again)) gs_again<MODE, EPI, BM>(a, (float*)lds, acc, Qe, i0, i_end, j0, c_lo, c_hi, p_row, q_row, col_at);
    // ---- output through LDS, whole rows at a time ----
    __syncthreads();
    constexpr int PITCH = BN + 4;
    float* const stg = (float*)lds;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {                   // a lane holds, per block, one row and quads of columns
                const f32x16_t& v = acc[i][j];
                *(f32x4_t*)(stg + col_at(P_CMAJ, p_row(i) + l32) * PITCH + col_at(Q_CMAJ, q_row(j) + 8 * q + 4 * kh)) =
                    f32x4_t{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
            }
    __syncthreads();
    // rows tid / 32 + 8 i of the tile; columns 4 (tid % 32) .., SwiGLU: two rows' gates and up projections in turn
    const int x32 = tid & 31;
    if (EPI == GF_SWIGLU) {
        gf_output<MODE, EPI, true, BM / 16, 2>(a, e, i0, i_end, j0,
            [&](int i, int q) { return *(const f32x4_t*)(stg + (16 * i + (tid >> 4)) * PITCH + 64 * q + 4 * (tid & 15)); },
            [&](int i) { return 16 * i + (tid >> 4); }, [&](int) { return 4 * (tid & 15); });
    } else {
        gf_output<MODE, EPI, true, BM / 8, 1>(a, e, i0, i_end, j0,
            [&](int i, int) { return *(const f32x4_t*)(stg + (8 * i + (tid >> 5)) * PITCH + 4 * x32); },
            [&](int i) { return 8 * i + (tid >> 5); }, [&](int) { return 4 * x32; });
    }
}

// Tile size.  128 halves the operand traffic, 64 has four times the workgroups and loses less to partly filled tiles and
// to a last, half-empty round of them; eight 128-tiles per compute unit is where the two meet.  The number of row tiles
// depends on the device's offsets; Rcap / 128 is taken.  Measured, whole training step, 8 experts, top-2 (64 against 128):
// T 256, h 128, f 256: 106 us against 178; T 2048, h 1024, f 512: 537 against 665; T 4096, h 1024, f 512: 906 against 1042;
// (all calls on gf_kernel) T 8192, h 1024, f 1024 (8 tiles per unit in fc1): 3.04 ms against 3.05; T 8192, h 2048, f 2048: 11.4 against 10.7;
// T 8192, h 4096, f 2048: 22.6 against 20.7 ms (119 TFLOP/s).
static int gf_tile(int num_cu, bool wgrad, int E, int N, int out_cols, int64_t Rcap) {
    const int64_t cols = ceil_div64(out_cols, 128);
    const int64_t tiles = wgrad ? (int64_t)E * ceil_div64(N, 128) * cols : ceil_div64(Rcap, 128) * cols;
    return tiles >= 8 * (int64_t)(num_cu > 0 ? num_cu : 256) ? 128 : 64;
}

// rows of 16-byte pieces
static bool gf_vec(int epi, int N, int K) { return N % 4 == 0 && K % 4 == 0 && (epi != GF_SWIGLU || N % 8 == 0); }

// Which kernel: the split needs enough work per workgroup, workgroups for most of the compute units, and columns that fill its
// wider tiles.  Measured (us, gf : gs):
//   forward / data gradient: 64 x 128 tiles for 0.6 of the units and a contraction of 320 (SwiGLU backward 512).  128 tiles: T 300
//     h 256 f 512 E 16 k 2 fc2 dgrad 13 : 16, T 100 h 2048 f 1024 E 8 k 2 61 : 70; 158: T 1000 h 512 f 256 E 32 k 4 fc2 dgrad 30 : 26;
//     320: T 30 h 1024 f 4096 E 8 k 2 80 : 59.  Contraction 320: T 2000 f 704 E 8 k 4 82 : 68 (fc2 dgrad there, 320: 51 : 55); 256:
//     T 8192 h 192 f 256 E 8 k 4 fc2 41 : 44.
//   weight gradient: 128 x 128 tiles that fill their rounds to three quarters (T 4096 h 1024 f 1536 E 4 k 1, 384 tiles 196 : 170; T 2048
//     h 768 f 512 E 8 k 2, 192 57 : 51; T 2000 h 320 f 704 E 8 k 4, 144 84 : 88, 264 148 : 176), from 32 experts on, the largest of which is
//     further above the mean and sets the time of a round, to seven eighths (192 tiles: T 8192 h 384 f 128 E 64 k 4 45 : 54, T 8192 h 512
//     f 192 E 32 k 2 45 : 54), and 384 rows per expert in the mean (T 3072 h 512 f 512 E 16 k 2 49 : 45, T 2048 33.8 : 34.5).
//   columns (and the weight gradient's rows) whose 64-wide tiles cover at least 0.8 of what the 128-wide ones do: 192 of 256 T 8192
//     h 192 f 256 E 8 k 4 fc1 dgrad 74 : 84, E 64 weight gradients 45, 72 : 56, 84; 320 of 384 T 4096 h 320 f 512 E 16 k 4 fc2 64 : 58,
//     weight gradients 107, 159 : 99, 144.
static bool gs_serves(int num_cu, int mode, int epi, const gf_args& a) {
    const double cu = num_cu > 0 ? num_cu : 256;
    auto cover = [](int64_t cols, int bn) { return (double)ceil_div64(cols, bn / 2) / (2 * ceil_div64(cols, bn)); };
    if (mode == GF_WGRAD) {
        const double n = (double)a.E * ceil_div64(a.N, 128) * ceil_div64(a.K, 128), rounds = __builtin_ceil(n / cu);
        return (double)a.Rcap >= 384.0 * a.E && n >= (a.E < 32 ? 0.75 : 0.875) * cu * rounds && cover(a.N, 128) * cover(a.K, 128) >= 0.8;
    }
    const int64_t cols = epi == GF_SWIGLU ? a.N / 2 : mode == GF_FWD ? a.N : a.K, c = mode == GF_FWD ? a.K : a.N;
    const int bn = epi == GF_SWIGLU ? 64 : GS_BN;
    const int64_t tiles = (ceil_div64(a.Rcap, 64) + a.E / 2) * ceil_div64(cols, bn);
    return tiles >= 0.6 * cu && c >= (epi == GF_SWIGLU_BWD ? 512 : 320) && cover(cols, bn) >= 0.8;
}

// 64 or 128: gf_kernel on tiles of that size; 3: gs_kernel (bases, too, on 16 bytes then)
int moe_gg_f32_choice(int num_cu, int mode, int epi, int E, int N, int K, int64_t Rcap) {
    gf_args a = {};
    a.E = E;
    a.N = N;
    a.K = K;
    a.Rcap = Rcap;
    if (gf_vec(epi, N, K) && gs_serves(num_cu, mode, epi, a)) return 3;
    return gf_tile(num_cu, mode == GF_WGRAD, E, N, mode == GF_FWD ? N : K, Rcap);
}

template <int MODE, int EPI>
static moe_status gf_launch(moe_ctx* ctx, hipStream_t s, const char* who, const gf_args& a) {
    if (a.E > F32_MAX_E) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: E > %d", who, F32_MAX_E);
    const int out_cols = EPI == GF_SWIGLU ? a.N : (MODE == GF_FWD ? a.N : a.K);
    const int bt = gf_tile(ctx->num_cu, MODE == GF_WGRAD, a.E, a.N, out_cols, a.Rcap);
    const int64_t tiles_j = EPI == GF_SWIGLU ? ceil_div64(a.N / 2, bt / 2) : ceil_div64(out_cols, bt);
    // (every expert may end in a partly filled row tile)
    const int64_t grid = ceil_div64(tiles_j * (MODE == GF_WGRAD ? a.E * ceil_div64(a.N, bt) : ceil_div64(a.Rcap, bt) + a.E), 8) * 8;
    if (grid > 0x7fffffffLL) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: problem too large for the fp32 path", who);
    const uintptr_t bits = (uintptr_t)a.P | (uintptr_t)a.Q | (uintptr_t)a.out | (uintptr_t)a.out_act | (uintptr_t)a.Zsaved;
    const bool vec = gf_vec(EPI, a.N, a.K) && bits % 16 == 0;
    const dim3 g((unsigned)grid), b(F32_THREADS);
    constexpr int GS_BM = MODE == GF_WGRAD ? 128 : 64;
    if (vec && gs_serves(ctx->num_cu, MODE, EPI, a)) {
        const int64_t cols = EPI == GF_SWIGLU ? ceil_div64(a.N / 2, 64) : ceil_div64(out_cols, GS_BN);
        const int64_t n = cols * (MODE == GF_WGRAD ? a.E * ceil_div64(a.N, GS_BM) : ceil_div64(a.Rcap, GS_BM) + a.E);
        hipLaunchKernelGGL((gs_kernel<MODE, EPI, GS_BM>), dim3((unsigned)(ceil_div64(n, 8) * 8)), b, 0, s, a);
    } else if (vec && bt == 64 && ctx->batch) {
        gg_args j;   // (the fields a batch's list has in common with this path's)
        memset(&j, 0, sizeof(j));
        j.P = a.P;
        j.Q = a.Q;
        j.offsets = a.offsets;
        j.E = a.E;
        j.N = a.N;
        j.K = a.K;
        j.Rcap = a.Rcap;
        j.out = a.out;
        j.out_act = (bf16_t*)a.out_act;
        j.Zsaved = (const bf16_t*)a.Zsaved;
        j.row_prob = a.row_prob;
        j.accumulate = a.accumulate;
        j.dev_err = a.dev_err;
        batch_gemm(ctx, {s, MODE, EPI, 0, 1, JOB_F32, MODE == GF_WGRAD, false, j});
    } else if (vec && bt == 128) hipLaunchKernelGGL((gf_kernel<MODE, EPI, 128, true>), g, b, 0, s, a);
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

// ---- calls of a batch ----
int64_t gf_blocks(int mode, int epi, const gg_args& a) {
    const int64_t cols = epi == GF_SWIGLU ? ceil_div64(a.N / 2, 32) : ceil_div64(mode == GF_FWD ? a.N : a.K, 64);
    return ceil_div64(cols * (mode == GF_WGRAD ? a.E * ceil_div64(a.N, 64) : ceil_div64(a.Rcap, 64) + a.E), 8) * 8;
}
void gf_launch_jobs(hipStream_t s, bool fwd, int epi, const gt_jobs& m) {
    gf_jobs f;
    for (int x = 0; x < GT_JOBS; ++x) {
        const gg_args& a = m.a[x];
        f.a[x] = {(const float*)a.P, (const float*)a.Q, a.offsets, a.E, a.N, a.K, a.Rcap, (float*)a.out, (float*)a.out_act,
                  (const float*)a.Zsaved, a.row_prob, a.accumulate, a.dev_err};
        f.start[x] = m.start[x];
    }
    f.start[GT_JOBS] = m.start[GT_JOBS];
    f.turn = m.turn;
    const dim3 g((unsigned)f.start[GT_JOBS]), b(F32_THREADS);
    if (fwd && epi == GF_SWIGLU) hipLaunchKernelGGL(gf_fwd_jobs_kernel<GF_SWIGLU>, g, b, 0, s, f);
    else if (fwd) hipLaunchKernelGGL(gf_fwd_jobs_kernel<GF_STORE>, g, b, 0, s, f);
    else if (epi == GF_SWIGLU_BWD) hipLaunchKernelGGL(gf_bwd_jobs_kernel<GF_SWIGLU_BWD>, g, b, 0, s, f);
    else hipLaunchKernelGGL(gf_bwd_jobs_kernel<GF_STORE>, g, b, 0, s, f);
}
