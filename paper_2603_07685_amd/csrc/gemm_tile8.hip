// Grouped GEMM on one-byte operands (blockwise fp8 and MXFP8), four waves per workgroup: 64 x 128 and 128 x 128 tiles, the
// counterpart of gemm_tile.hip, for the calls whose 256 x 256 tiles are too few for the compute units or whose contraction is a
// few stages; and, MXFP8, 256 x 256 tiles for the rest.
//
// A workgroup computes one BM x BN tile with its waves as 2 x 2, wave tile BM/2 x BN/2 in 32 x 32 blocks of
// v_mfma_scale_f32_32x32x64_f8f6f4: fragments, contraction order and the software rescaling of the blockwise
// recipe are those of gemm.hip's kernel, so all of them give the same bits.  A stage is 128 contraction elements (128 bytes of a
// row), two MFMA steps of 64; operands come by DMA into two stage buffers, the scales of a stage (a dword per row and column)
// into a ring of four, because the blockwise weight gradient needs the previous stage's beside the current.
// The quantising epilogues are not built here: their 1 x 128 blocks span two small tiles; the caller runs the quantiser on the
// stored tensor instead (the same bits by construction), one more launch.
//
// Small tiles.  Bound: as gemm_tile.hip, the fixed cost around a few stages; the 256 x 256 kernel's output phase, quantisation
// included, is 30-55 us of one workgroup per tile.  Measured (us, gemm.hip's kernel : this), T 1024, h 512, f 256, 8 experts,
// top-4, blockwise: fc1 + SwiGLU + quantised copy 31 : 10 (+ 4 for the quantiser), fc2 15 : 7, fc2 data gradient + SwiGLU
// backward + copies 55 : 10 (+ 5), weight gradients 28, 29 : 13, 13, fc1 data gradient 18 : 8.
//
// 256 x 256 tiles (MXFP8).  One workgroup per compute unit goes from tile to tile; the accumulators fill the 256 accumulation
// registers, both steps' fragments 128 others.  A wave alone on its SIMD issues in order, so fragment reads and DMA
// instructions are written between MFMAs.  A stage's buffer is free as soon as its second step is in registers (a barrier in
// the first step), and the refill is spread over the rest of the stage: an even flow is what matters (all 18 DMA instructions
// of a wave in the second step: 5-7 % slower, bunched in its first half: 9 % slower; where exactly they lie, below 1 %).  The next
// tile's first stage is under way during the output phase, which is staged through the other buffer.
// Against eight waves in two groups that take turns reading and multiplying, with the copies in their output phase (us, old :
// this, profiled steps), T 16384, h 7168, f 2048, 32 experts, top-8: fc1 + SwiGLU with quantised copies 4153 : 3733 + 207 for the
// quantiser, fc2 2006 : 1909, fc2 data gradient + SwiGLU backward with copies 2665 : 2180 + 443, fc1 data gradient 3595 : 3452; the
// shared expert 525 : 426 + 34, 247 : 224, 331 : 270 + 62, 433 : 397; weight gradients 1787 : 1611, 3279 : 3063, the shared
// expert's 226 : 203, 427 : 390.  T 8192, h 2048, f 1024, 16 experts, rank^-1.2: 193 : 164, 220 : 191.  Without the order of cost
// and the draw the routed weight gradients took 1869 and 3740.  Bound now: 1.75 us per stage and tile; the matrix pipe is busy
// 46-66 % of the time in forward and data-gradient calls and 65-83 % in weight gradients, at the 1.75-2.0 GHz the card holds
// under this load; operands at 37 bytes/ns and compute unit.
#include "gemm_tile.h"

#include <type_traits>

// 4 bytes per lane from a per-lane address; LDS side: M0 + 4 * lane
__device__ __forceinline__ void dma4_addr(const void* src, uint32_t lds_wave, uint32_t lds_const) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 ::"s"(m0_value(lds_wave, lds_const)), "v"(src) : "memory", "m0");
}
// the 32 contraction values of a lane from a contraction-major tile of 128-byte rows (gemm.hip: lds_read_tr8x32)
template <int PITCH>
__device__ __forceinline__ i32x8_t read_tr8x32_pitch(const char* p, int second) {
    const i32x2_t r0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2_t*)p);
    const i32x2_t r1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2_t*)(p + 8 * PITCH));
    const i32x2_t r2 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2_t*)(p + second * PITCH));
    const i32x2_t r3 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2_t*)(p + (second + 8) * PITCH));
    const i32x8_t v = {r0.x, r0.y, r1.x, r1.y, r2.x, r2.y, r3.x, r3.y};
    return v;
}

// F8: 1 = blockwise (fp32 block scales applied to the accumulators), 2 = MXFP8 (E8M0 scales, by the matrix instruction)
// The LDS of a workgroup: two stage buffers, a ring of four stages' scales (P's from 0 on, Q's from GQ_PS(BM) on), and the rest.
// (Arrays of their own rather than one struct: with the ring's addresses behind others' the 256 x 256 kernels need up to 8 more
// registers, and spill.)
#define GQ_PS(BM) ((BM) < 128 ? 128 : (BM))
template <bool LPT>
struct gq_lds {
    tile_pick_lds pick;
    int offs[LPT ? GG_MAX_E + 1 : 1], order[LPT ? GG_MAX_E : 1], drawn;
};
// block, G: the workgroup's place among the G of its call
template <int MODE, int EPI, bool OUT_F32, int F8, int BM, int BN>
__device__ __forceinline__ void gq_body(const gg_args& a, char* const ring, float (*const scales)[GQ_PS(BM) + BN],
                                        gq_lds<BM == 256 && MODE == GG_WGRAD>& lds, const int block, const int G) {
    constexpr bool MX = F8 == 2, P_CMAJ = MODE == GG_WGRAD, Q_CMAJ = MODE != GG_FWD, BW_WGRAD = F8 == 1 && MODE == GG_WGRAD;
    static_assert(MODE != GG_WGRAD || BM >= 128, "contraction-major tiles have rows of 128 or 256 bytes");
    constexpr int P_BYTES = BM * 128, STAGE = P_BYTES + BN * 128;
    constexpr int PS = GQ_PS(BM), SC = (PS + BN) / 256;
    constexpr int PC = BM / 32, QC = BN / 32, XC = PC + QC + SC;    // DMA instructions per wave and stage: P, Q, scales
    constexpr int NI = BM / 64, NJ = BN / 64;                       // 32-row and 32-column blocks per wave
    constexpr bool MANY = BM == 256;                                // one workgroup per compute unit, tile after tile
    constexpr bool LPT = MANY && MODE == GG_WGRAD;
    constexpr int HB = BN / 2;                                      // SwiGLU: features per tile
    tile_pick_lds& pick = lds.pick;
    int *const offs = lds.offs, *const order = lds.order;
    int& drawn = lds.drawn;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    const int N = a.N, K = a.K;
    const int J = MODE == GG_FWD ? N : K;
    const int half_cols = EPI == GG_EPI_SWIGLU ? N >> 1 : 0;
    const int tiles_j = EPI == GG_EPI_SWIGLU ? (half_cols + HB - 1) / HB : (J + BN - 1) / BN;
    const int tiles_iw = (N + BM - 1) / BM;                 // wgrad
    if (MODE == GG_WGRAD || a.out_qc) {   // (scale blocks down the rows must not straddle two experts)
        bool off_grid = false;
        for (int e = tid; e <= a.E; e += 256) off_grid |= (a.offsets[e] & 127) != 0;
        if (__syncthreads_or(off_grid)) {
            if (block == 0 && tid == 0) atomicExch(a.dev_err, 1);
            return;
        }
    }
    tile_sums<256> sums;
    if (!tile_scan(a.offsets, a.E, a.Rcap, a.dev_err, MODE == GG_WGRAD ? 0 : BM, MODE == GG_WGRAD ? tiles_iw * tiles_j : tiles_j,
                   pick, sums, block == 0)) return;
    // Weight gradients, tile after tile: a tile costs its expert's rows, so the experts are taken in descending order of rows
    // (rank sort, ties by index) and the list is dealt to the XCDs in chunks, in a snake; with an expert above twice the mean no
    // deal balances, and the workgroups draw from a device counter in the same order (gemm.hip: tile_of, draw).
    const int tpe = tiles_iw * tiles_j;
    bool dyn = false;
    int ticket = 0;
    if constexpr (LPT) {
        for (int x = tid; x <= a.E; x += 256) offs[x] = a.offsets[x];
        __syncthreads();
        for (int x = tid; x < a.E; x += 256) {
            const int rows = offs[x + 1] - offs[x];
            int rank = 0;
            for (int o = 0; o < a.E; ++o) {
                const int ro = offs[o + 1] - offs[o];
                rank += ro > rows || (ro == rows && o < x);
            }
            order[rank] = x;
        }
        __syncthreads();
        const int most = __builtin_amdgcn_readfirstlane(offs[order[0] + 1] - offs[order[0]]);
        dyn = (int64_t)most * a.E > 2 * (int64_t)__builtin_amdgcn_readfirstlane(offs[a.E] - offs[0]);
    }
    auto draw = [&]() __attribute__((always_inline)) {
        if (LPT && dyn && tid == 0) ticket = atomicAdd(a.tile_counter, 1);
    };
    // the tile in work
    int e, u, row_lo, row_hi, ti, tj, i0, i_end, j0, c_lo, KT;
    const int CB = (MODE == GG_FWD ? K : N) / 128;          // contraction blocks (forward, data gradient)
    auto q_col = [&](int rho) { return EPI == GG_EPI_SWIGLU ? (rho < HB ? j0 + rho : half_cols + j0 + rho - HB) : j0 + rho; };

    // ---- operand transfers: 1 KB chunks of 8 rows x 128 B, lane -> row l / 8, 16-byte slot l % 8.  Row-major: slot ^
    // KM_SWZ(row); contraction-major: slot ^ 2 * (row / 2 % 4): a transposing read of 8 rows x 32 bytes then covers all 16
    // slots of the 256-byte bank line once (two rows share a line) ----
    const int ldp = MODE == GG_FWD ? K : N;
    auto cm_slot = [](int width, int l, int row) { return width == 256 ? (l & 15) ^ (2 * (row & 7)) : (l & 7) ^ (2 * ((row >> 1) & 3)); };
    uint32_t po[PC], qo[QC], p_all;
    const uint32_t q_all = (uint32_t)N * (uint32_t)K;
    const char *p_base0, *q_base0;
    const float* sc_src[SC];
    int64_t sc_step;
    auto set_tile = [&](int n) __attribute__((always_inline)) -> bool {   // this workgroup's n-th
    if constexpr (LPT) {
        const int x = block & 7;
        int t = (8 * n + ((n & 1) ? 7 - x : x)) * (G >> 3) + (block >> 3);
        if (dyn) {
            if (tid == 0) drawn = ticket;
            wait_lgkm0();
            stage_barrier();
            t = __builtin_amdgcn_readfirstlane(drawn);
        }
        if (t >= sums.total) return false;
        u = __builtin_amdgcn_readfirstlane(t % tpe);
        e = __builtin_amdgcn_readfirstlane(order[t / tpe]);
        row_lo = __builtin_amdgcn_readfirstlane(offs[e]);
        row_hi = __builtin_amdgcn_readfirstlane(offs[e + 1]);
    } else if (!tile_find(sums, block + n * G, pick, e, u, row_lo, row_hi)) return false;
    gt_place(u, MODE == GG_WGRAD ? tiles_iw : (row_hi - row_lo + BM - 1) / BM, tiles_j, ti, tj);
    i0 = MODE == GG_WGRAD ? ti * BM : row_lo + ti * BM;
    i_end = MODE == GG_WGRAD ? N : row_hi;
    j0 = tj * (EPI == GG_EPI_SWIGLU ? HB : BN);
    c_lo = MODE == GG_WGRAD ? row_lo : 0;
    KT = __builtin_amdgcn_readfirstlane(((MODE == GG_WGRAD ? row_hi - row_lo : MODE == GG_FWD ? K : N)) / 128);
#pragma unroll
    for (int i = 0; i < PC; ++i) {
        const int row = (wave * PC + i) * (P_CMAJ ? 1024 / BM : 8) + (P_CMAJ ? lane / (BM / 16) : lane >> 3);
        if (P_CMAJ) po[i] = (uint32_t)(row * ldp + i0 + cm_slot(BM, lane, row) * 16);
        else po[i] = (uint32_t)(row * ldp) + ((lane & 7) ^ KM_SWZ(row)) * 16;
    }
#pragma unroll
    for (int i = 0; i < QC; ++i) {
        const int row = (wave * QC + i) * (Q_CMAJ ? 1024 / BN : 8) + (Q_CMAJ ? lane / (BN / 16) : lane >> 3);
        if (Q_CMAJ) qo[i] = (uint32_t)(row * K + j0 + cm_slot(BN, lane, row) * 16);
        else qo[i] = (uint32_t)q_col(row) * (uint32_t)K + ((lane & 7) ^ KM_SWZ(row)) * 16;
    }
    p_base0 = (const char*)a.P + (int64_t)(P_CMAJ ? c_lo : i0) * ldp;
    q_base0 = (const char*)a.Q + (MODE == GG_WGRAD ? (int64_t)c_lo * K : (int64_t)e * N * K);
    p_all = (uint32_t)min(BM, i_end - i0) * (uint32_t)ldp;
    // scales: this lane's dwords of stage 0 and the advance per stage (elements); waves 0, 1: P rows, waves 2, 3: Q rows
#pragma unroll
    for (int x = 0; x < SC; ++x) {
        if (wave < 2) {
            const int q = min((wave * SC + x) * 64 + lane, BM - 1);
            if (MODE == GG_WGRAD) {
                sc_src[x] = a.p_scale + (int64_t)(c_lo >> 7) * N + min(i0 + q, N - 1);
                sc_step = N;
            } else {
                sc_src[x] = a.p_scale + (int64_t)min(i0 + q, i_end - 1) * CB;
                sc_step = 1;
            }
        } else {
            const int q = ((wave - 2) * SC + x) * 64 + lane;
            if (MODE == GG_WGRAD) {
                sc_src[x] = a.q_scale + (int64_t)(c_lo >> 7) * K + min(j0 + q, K - 1);
                sc_step = K;
            } else if (MX) {
                const int col = min(q_col(q), J - 1);
                sc_src[x] = MODE == GG_FWD ? a.q_scale + ((int64_t)e * N + col) * CB : a.q_scale + (int64_t)e * (N >> 7) * K + col;
                sc_step = MODE == GG_FWD ? 1 : K;
            } else {   // one scale per 128 x 128 block: even lanes the block of the tile's first columns, odd lanes of the last
                const int col = min(q_col((lane & 1) * HB), J - 1);
                sc_src[x] = MODE == GG_FWD ? a.q_scale + ((int64_t)e * (N / 128) + col / 128) * (K / 128)
                                           : a.q_scale + (int64_t)e * (N / 128) * (K / 128) + col / 128;
                sc_step = MODE == GG_FWD ? 1 : K / 128;
            }
        }
    }
    return true;
    };
    auto make = [](const char* base, uint32_t bytes) __attribute__((always_inline)) {
        const uint64_t b = (uint64_t)base;
        i32x4_t r = {(int)__builtin_amdgcn_readfirstlane((uint32_t)b), (int)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)),
                     (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000};
        return r;
    };
    const uint32_t lds0 = lds_addr(ring), sc0 = lds_addr(scales);
    i32x4_t rp, rq;
    int64_t sc_at;
    auto describe = [&](int s) __attribute__((always_inline)) {   // (behind the last stage nothing is fetched: zeros)
        const uint32_t rows = s < KT ? 128u : 0u;
        rp = make(p_base0 + (int64_t)s * (P_CMAJ ? 128 * (int64_t)ldp : 128), P_CMAJ ? rows * (uint32_t)ldp : s < KT ? p_all - (uint32_t)s * 128 : 0u);
        rq = make(q_base0 + (int64_t)s * (Q_CMAJ ? 128 * (int64_t)K : 128), Q_CMAJ ? rows * (uint32_t)K : s < KT ? q_all - (uint32_t)s * 128 : 0u);
        sc_at = (int64_t)min(s, KT - 1) * sc_step;
    };
    auto issue_one = [&](int s, uint32_t at, int x) __attribute__((always_inline)) {
        if (x < PC) dma16_buf(rp, po[x], at + wave * (PC * 1024), x * 1024);
        else if (x < PC + QC) dma16_buf(rq, qo[x - PC], at + wave * (QC * 1024), P_BYTES + (x - PC) * 1024);
        else dma4_addr(sc_src[x - PC - QC] + sc_at, sc0 + (s & 3) * ((PS + BN) * 4) + wave * (SC * 256), (x - PC - QC) * 256);
    };

    // ---- fragments (gemm.hip: fetch) ----
    const int fr_row = lane & 31, fr_khalf = lane >> 5, fr_swz = KM_SWZ(lane & 31);
    const int tr_i = lane & 15, tr_blk = lane >> 4;
    const int tr_row = (MX ? 16 : 32) * (tr_blk >> 1) + (tr_i >> 1);
    auto col_of = [&](int j) __attribute__((always_inline)) {
        return EPI == GG_EPI_SWIGLU ? (j / (NJ / 2)) * HB + wn * (HB / 2) + (j % (NJ / 2)) * 32 : wn * HB + j * 32;
    };
    auto frag = [&](const char* t, auto width, bool cmaj, int half, int row) __attribute__((always_inline)) -> i32x8_t {
        constexpr int W = decltype(width)::value;
        if (cmaj) return read_tr8x32_pitch<W>(t + (half * 64 + tr_row) * W + (tr_i & 1) * 8 +
                                              (((row / 16) ^ (W == 256 ? 2 * (tr_i >> 1) : 2 * (tr_i >> 2))) + (tr_blk & 1)) * 16, MX ? 32 : 16);
        const int sl0 = MX ? 4 * half + fr_khalf : 4 * half + 2 * fr_khalf, sl1 = MX ? sl0 + 2 : sl0 + 1;
        const i32x4_t lo = *(const i32x4_t*)(t + (row + fr_row) * 128 + (sl0 ^ fr_swz) * 16);
        const i32x4_t hi = *(const i32x4_t*)(t + (row + fr_row) * 128 + (sl1 ^ fr_swz) * 16);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    i32x8_t fp[2][NI], fq[2][NJ];
    auto read_one = [&](int set, const char* t, int half, int r) __attribute__((always_inline)) {
        if (r < NJ) fq[set][r] = frag(t + P_BYTES, std::integral_constant<int, BN>{}, Q_CMAJ, half, col_of(r));
        else fp[set][r - NJ] = frag(t, std::integral_constant<int, BM>{}, P_CMAJ, half, wm * (BM / 2) + 32 * (r - NJ));
    };
    auto read_set = [&](int set, const char* t, int half) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < NJ + NI; ++r) read_one(set, t, half, r);
    };
    f32x16_t acc[NI][NJ];
    // MXFP8: the lane's E8M0 bytes, shifted so that its block is byte 0 (first step) / 2 (second).  Blockwise: the running
    // scales the accumulators are in units of (see gemm.hip)
    int ps[NI], qs[NJ];
    float ps_cur[NI], qs_cur[NJ];
    auto scale_cols = [&](const float* now, const float* before, const float (&rp_)[NI]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int c = PS + col_of(j) + 8 * g + 4 * fr_khalf;
                f32x4_t q4 = *(const f32x4_t*)(now + c);
                if (before) {
                    const f32x4_t qp4 = *(const f32x4_t*)(before + c);
#pragma unroll
                    for (int x = 0; x < 4; ++x) q4[x] = qp4[x] * __builtin_amdgcn_rcpf(q4[x]);
                }
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int x = 0; x < 4; ++x) acc[i][j][4 * g + x] *= rp_[i] * q4[x];
            }
    };
    int ps_raw[NI], qs_raw[NJ];   // MXFP8: the next stage's scales, read a step ahead of their use
    auto read_scales = [&](int s) __attribute__((always_inline)) {
        const int* const at = (const int*)scales[s & 3];
#pragma unroll
        for (int i = 0; i < NI; ++i) ps_raw[i] = at[wm * (BM / 2) + 32 * i + fr_row];
#pragma unroll
        for (int j = 0; j < NJ; ++j) qs_raw[j] = at[PS + col_of(j) + fr_row];
    };
    auto enter_stage = [&](int s) __attribute__((always_inline)) {   // the scales of stage s are in LDS
        if (MX) {
#pragma unroll
            for (int i = 0; i < NI; ++i) ps[i] = (int)((uint32_t)ps_raw[i] >> (8 * fr_khalf));
#pragma unroll
            for (int j = 0; j < NJ; ++j) qs[j] = (int)((uint32_t)qs_raw[j] >> (8 * fr_khalf));
            return;
        }
        const float* const now = scales[s & 3];
        if (BW_WGRAD) {
            if (s == 0) return;
            const float* const before = scales[(s - 1) & 3];
            float rp_[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int r = wm * (BM / 2) + 32 * i + fr_row;
                rp_[i] = before[r] * __builtin_amdgcn_rcpf(now[r]);
            }
            scale_cols(now, before, rp_);
        } else {
            float qr[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float qn = now[PS + (EPI == GG_EPI_SWIGLU ? j : 0)];
                qr[j] = qs_cur[j] * __builtin_amdgcn_rcpf(qn);
                qs_cur[j] = qn;
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const float pn = now[wm * (BM / 2) + 32 * i + fr_row], pr = ps_cur[i] * __builtin_amdgcn_rcpf(pn);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const float ratio = pr * qr[j];
#pragma unroll
                    for (int x = 0; x < 16; ++x) acc[i][j][x] *= ratio;
                }
                ps_cur[i] = pn;
            }
        }
    };
    auto step = [&](int half, auto&& slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (!MX) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fq[half][j], fp[half][i], acc[i][j], 0, 0, 0, 127, 0, 127);
                else if (half == 0) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fq[half][j], fp[half][i], acc[i][j], 0, 0, 0, qs[j], 0, ps[i]);
                else acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fq[half][j], fp[half][i], acc[i][j], 0, 0, 2, qs[j], 2, ps[i]);
                __builtin_amdgcn_sched_barrier(0);
                slot(i * NJ + j);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    constexpr int NM = NI * NJ;   // MFMAs per step

    auto issue_stage = [&](int s) __attribute__((always_inline)) {
        describe(s);
#pragma unroll
        for (int x = 0; x < XC; ++x) issue_one(s, lds0 + s * STAGE, x);
    };
    draw();
    bool more = set_tile(0);
    if (more && KT > 0) issue_stage(0);     // (an expert without rows: not even its scales' address is inside the tensor)
    for (int n = 1; more; ++n) {
    draw();                                 // (collected behind the contraction)
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        ps_cur[i] = 1.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            qs_cur[j] = 1.f;
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[i][j][x] = 0.f;
        }
    }
    if (KT > 0) {
        issue_stage(1);
        wait_vm<XC>();
        stage_barrier();
        if (MX) read_scales(0);
        read_set(0, ring, 0);
        for (int s = 0; s < KT; ++s) {
            const char* const t0 = ring + (s & 1) * STAGE;
            const char* const t1 = ring + ((s + 1) & 1) * STAGE;
            enter_stage(s);
            if (BN == 128) {
                read_set(1, t0, 1);
                step(0, [&](int) {});
                describe(s + 2);
                wait_vm<0>();       // stage s + 1 and its scales have landed, this wave's reads of this buffer are done
                wait_lgkm0();
                stage_barrier();
                if (MX) read_scales(s + 1);
                read_set(0, t1, 0);
                step(1, [&](int m) __attribute__((always_inline)) {
#pragma unroll
                    for (int x = 0; x < XC; ++x)
                        if (x * NM / XC == m) issue_one(s + 2, lds0 + (s & 1) * STAGE, x);
                });
            } else {
                constexpr int FREE = 5, EARLY = 9, LATE = 15;
                step(0, [&](int m) __attribute__((always_inline)) {
                    if (2 * m < NI + NJ) {
                        read_one(1, t0, 1, 2 * m);
                        read_one(1, t0, 1, 2 * m + 1);
                    }
                    if (m == FREE) {
                        describe(s + 2);
                        wait_lgkm0();
                        stage_barrier();
                    }
                    if (m > FREE) {
#pragma unroll
                        for (int x = 0; x < EARLY; ++x)
                            if (FREE + 1 + x * (15 - FREE) / EARLY == m) issue_one(s + 2, lds0 + (s & 1) * STAGE, x);
                    }
                });
                wait_vm<EARLY>();
                stage_barrier();
                if (MX) read_scales(s + 1);
                step(1, [&](int m) __attribute__((always_inline)) {
                    if (m < NI + NJ) read_one(0, t1, 0, m);
#pragma unroll
                    for (int x = EARLY; x < XC; ++x)
                        if ((x - EARLY) * LATE / (XC - EARLY) == m) issue_one(s + 2, lds0 + (s & 1) * STAGE, x);
                });
            }
        }
        if (BW_WGRAD) {         // out of the last stage's units
            const float* const now = scales[(KT - 1) & 3];
            float rp_[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) rp_[i] = now[wm * (BM / 2) + 32 * i + fr_row];
            scale_cols(now, nullptr, rp_);
        }
    }
    wait_vm0();                 // (the zeros of the stages past the end must not land in the staging area)
    wait_lgkm0();
    stage_barrier();

    // a workgroup with further tiles: the next one's first stage is on its way while this one's output goes through the other
    // stage buffer
    const int e_ = e, i0_ = i0, i_end_ = i_end, j0_ = j0, tj_ = tj;
    more = MANY && set_tile(n);
    if (more && KT > 0) issue_stage(0);
    gt_output<MODE, EPI, OUT_F32, BM, BN>(a, (float*)(ring + (MANY ? STAGE : 0)), e_, i0_, i_end_, j0_, tj_, tiles_j, [&](int pass, float* stg) __attribute__((always_inline)) {
        // a lane's accumulators of a block: one row (lane % 32), four groups of columns 8 g + 4 (lane / 32) .. + 3
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4_t v;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    v[x] = acc[pass][j][4 * g + x];
                    if (!MX && !BW_WGRAD) v[x] *= ps_cur[pass] * qs_cur[j];
                }
                *(f32x4_t*)(stg + stg_at<BN>(wm * 32 + fr_row, col_of(j) + 8 * g + 4 * fr_khalf)) = v;
            }
    });
    if (more) {                 // (the next stage 1 goes where the output was staged)
        wait_lgkm0();
        stage_barrier();
    }
    }
}
template <int MODE, int EPI, bool OUT_F32, int F8, int BM, int BN>
__global__ __launch_bounds__(256, BM == 64 ? 3 : BM == 128 ? 2 : 1) void gq_kernel(const gg_args a) {
    __shared__ __attribute__((aligned(1024))) char ring[2 * (BM + BN) * 128];
    __shared__ __attribute__((aligned(16))) float scales[4][GQ_PS(BM) + BN];
    __shared__ gq_lds<BM == 256 && MODE == GG_WGRAD> lds;
    gq_body<MODE, EPI, OUT_F32, F8, BM, BN>(a, ring, scales, lds, (int)blockIdx.x, (int)gridDim.x);
}
// Independent calls in one launch (gemm_tile.hip: gt_fwd_jobs_kernel, gt_bwd_jobs_kernel)
template <int EPI, int F8, int BM>
__global__ __launch_bounds__(256, BM == 64 ? 3 : 2) void gq_fwd_jobs_kernel(const gt_jobs m) {
    __shared__ __attribute__((aligned(1024))) char ring[2 * (BM + 128) * 128];
    __shared__ __attribute__((aligned(16))) float scales[4][256];
    __shared__ gq_lds<false> lds;
    const int j = gt_job_of(m, (int)blockIdx.x);
    gq_body<GG_FWD, EPI, false, F8, BM, 128>(m.a[j], ring, scales, lds, (int)blockIdx.x - m.start[j], m.start[j + 1] - m.start[j]);
}
template <int EPI, bool F32, int F8>
__global__ __launch_bounds__(256, 2) void gq_bwd_jobs_kernel(const gt_jobs m) {
    __shared__ __attribute__((aligned(1024))) char ring[2 * 256 * 128];
    __shared__ __attribute__((aligned(16))) float scales[4][256];
    __shared__ gq_lds<false> lds;
    const int at = gt_place_of((int)blockIdx.x, m.turn, m.start[GT_JOBS]), j = gt_job_of(m, at), block = at - m.start[j];
    const int G = m.start[j + 1] - m.start[j];
    if (j < 2) gq_body<GG_DGRAD, EPI, false, F8, 64, 128>(m.a[j], ring, scales, lds, block, G);
    else gq_body<GG_WGRAD, GG_EPI_STORE, F32, F8, 128, 128>(m.a[j], ring, scales, lds, block, G);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int64_t gq_tiles(int mode, int epi, int bm, int bn, const gg_args& a) {
    const int64_t cols = epi == GG_EPI_SWIGLU ? ceil_div64(a.N / 2, bn / 2) : ceil_div64(mode == GG_FWD ? a.N : a.K, bn);
    return cols * (mode == GG_WGRAD ? a.E * ceil_div64(a.N, bm) : ceil_div64(a.Rcap, bm) + a.E);
}
int64_t gq_blocks(int mode, int epi, int bm, const gg_args& a) { return ceil_div64(gq_tiles(mode, epi, bm, 128, a), 8) * 8; }
template <int MODE, int EPI, bool F32, int F8, int BM, int BN = 128>
static void gq_go(hipStream_t s, const gg_args& a, int cu) {
    int64_t n = gq_tiles(MODE, EPI, BM, BN, a);
    if (BM == 256 && n > cu) n = cu;
    hipLaunchKernelGGL((gq_kernel<MODE, EPI, F32, F8, BM, BN>), dim3((unsigned)(ceil_div64(n, 8) * 8)), dim3(256), 0, s, a);
}
template <int F8, int BM, int BN = 128>
static void gq_call(hipStream_t s, int mode, int epi, bool out_f32, const gg_args& a, int cu) {
    if constexpr (BM >= 128) {   // (contraction-major rows of 64 bytes are not built)
        if (mode == GG_WGRAD && out_f32) return gq_go<GG_WGRAD, GG_EPI_STORE, true, F8, BM, BN>(s, a, cu);
        if (mode == GG_WGRAD) return gq_go<GG_WGRAD, GG_EPI_STORE, false, F8, BM, BN>(s, a, cu);
    }
    if (mode == GG_FWD && epi == GG_EPI_SWIGLU) gq_go<GG_FWD, GG_EPI_SWIGLU, false, F8, BM, BN>(s, a, cu);
    else if (mode == GG_FWD) gq_go<GG_FWD, GG_EPI_STORE, false, F8, BM, BN>(s, a, cu);
    else if (epi == GG_EPI_SWIGLU_BWD) gq_go<GG_DGRAD, GG_EPI_SWIGLU_BWD, false, F8, BM, BN>(s, a, cu);
    else gq_go<GG_DGRAD, GG_EPI_STORE, false, F8, BM, BN>(s, a, cu);
}
// Which kernel serves a call: 1 = 64 x 128 tiles, 2 = 128 x 128, 3 = 256 x 256 (MXFP8), 0 = the 256 x 256
// kernel of gemm.hip (blockwise).  Decided from the call's sizes by
// two estimates of its time in microseconds, fitted to measured calls (MI355X; the rows of an expert are unknown on the host:
// R is taken to hold half a 128-row tile of slack per expert, and an expert's rows to be multiples of 128):
//   256 x 256: one workgroup per compute unit, whole rounds of tiles, a tile = per stage 1.75 (MXFP8 here), 2.35
//              (blockwise) or 3.4 (blockwise weight gradient: two multiplies per accumulator and stage) + its output phase: 8
//              (weight gradient 10, blockwise 11.5), SwiGLU 13 (blockwise 19 with quantised copies, 14
//              without), SwiGLU backward 38 (blockwise 57 when most units are in it at once, 35 without quantised copies)
//   128 x 128: two workgroups per compute unit, a round = 1.5 per stage (SwiGLU 1.7; weight gradient 1.25, blockwise 2.1) + 6.5
//              (SwiGLU backward 16); plus the quantiser's launch and its way over memory where the other kernel needs none
// Measured against each other (us, gemm.hip's 256 x 256 : small tiles, quantiser included), fc1 forward / fc2 dgrad + SwiGLU
// backward / fc1 wgrad, MXFP8:
//   T 256 h 128 f 128 E 8 k 2       20 : 11    34 : 12     9 : 6       T 2048 h 1024 f 512 E 8 k 2      36 : 25    54 : 23    19 : 14
//   T 4096 h 512 f 512 E 16 k 4     55 : 44    53 : 44    26 : 18      T 4096 h 2048 f 1024 E 8 k 2    106 : 88    91 : 72    51 : 64
//   T 16384 h 256 f 256 E 32 k 4    74 : 61   121 : 76    45 : 23      T 8192 h 1024 f 1024 E 16 k 4   184 : 190  215 : 173   83 : 106
//   T 2048 h 2048 f 1024 E 8 k 2    53 : 54    71 : 42    34 : 46      T 1024 h 4096 f 1536 E 16 k 8   208 : 270  141 : 152  192 : 263
// and the 256 x 256 tiles of this file, T 3968 k 3 h 1920 f 896 E 13: fc1 92 (107 : 104); T 8192: 164, 213; T 1024: 169, 133.
// 64 x 128 while the 128 x 128 tiles make less than one and a half rounds (T 4096 h 512 f 512: backward 24 against 29, fc1 dgrad
// 25.5 against 27; at four rounds, T 8192 h 1024 f 1024, 118 against 112 and 140 against 129).
int gq_tile(const moe_ctx* ctx, int mode, int epi, bool mx, bool quant, const gg_args& a) {
    const double cu = ctx->num_cu > 0 ? ctx->num_cu : 256;
    const double E = a.E, R = (double)a.Rcap, one = E < R ? E : R;
    auto row_tiles = [&](double bm, double slack) {
        const double n = E == 1 ? __builtin_ceil(R / bm) : R / bm + slack * E;
        return n > one ? n : one;
    };
    const bool wg = mode == GG_WGRAD, sw = epi == GG_EPI_SWIGLU, swb = epi == GG_EPI_SWIGLU_BWD;
    const double cols = mode == GG_FWD ? a.N : a.K;
    const double stages = wg ? R / E / 128 + 0.5 : (mode == GG_FWD ? a.K : a.N) / 128.0;
    const double n256 = __builtin_ceil(cols / 256) * (wg ? E * __builtin_ceil(a.N / 256.0) : row_tiles(256, 0.125));
    const double n128 = __builtin_ceil(cols / 128) * (wg ? E * __builtin_ceil(a.N / 128.0) : row_tiles(128, -0.25));
    const double r256 = __builtin_ceil(n256 / cu), r128 = n128 / (2 * cu);
    const double out256 = mx ? (sw ? 13 : swb ? 38 : wg ? 10 : 8)
                             : sw ? (quant ? 19 : 14) : swb ? (!quant ? 35 : 2 * n256 > cu ? 57 : 38) : wg ? 11.5 : 8;
    const double t256 = r256 * ((mx ? 1.75 : wg ? 3.4 : 2.35) * stages + out256);
    const double per_stage = wg ? (mx ? 1.25 : 2.1) : sw ? 1.7 : 1.5;
    double t128 = (3 * r128 + __builtin_ceil(r128)) / 4;
    t128 = (t128 < 0.5 ? 0.5 : t128) * (per_stage * stages + (swb ? 16 : 6.5));
    if (quant && !mx) t128 += 4 + R * (sw ? a.N / 2 : 2 * a.K) * 3 / 5e6;   // (bytes at 5 TB/s)
    if (t128 > t256) return mx ? 3 : 0;
    return wg || r128 >= 1.5 ? 2 : 1;
}
void gq_launch(const moe_ctx* ctx, hipStream_t s, int mode, int epi, bool out_f32, bool mx, int tile, const gg_args& a) {
    const int cu = ctx && ctx->num_cu >= 8 ? ctx->num_cu & ~7 : 256;   // (ctx: 256 x 256 tiles only)
    if (mx && tile == 3 && mode == GG_WGRAD) moe_launch_fill_i32(a.tile_counter, 1, 0, s);
    if (mx && tile == 3) gq_call<2, 256, 256>(s, mode, epi, out_f32, a, cu);
    else if (mx) tile == 1 ? gq_call<2, 64>(s, mode, epi, out_f32, a, cu) : gq_call<2, 128>(s, mode, epi, out_f32, a, cu);
    else tile == 1 ? gq_call<1, 64>(s, mode, epi, out_f32, a, cu) : gq_call<1, 128>(s, mode, epi, out_f32, a, cu);
}
template <int F8>
static void gq_jobs(hipStream_t s, bool fwd, int epi, bool f32, int tile, const gt_jobs& m) {
    const dim3 grid((unsigned)m.start[GT_JOBS]), block(256);
    if (fwd && epi == GG_EPI_SWIGLU) {
        if (tile == 1) hipLaunchKernelGGL((gq_fwd_jobs_kernel<GG_EPI_SWIGLU, F8, 64>), grid, block, 0, s, m);
        else hipLaunchKernelGGL((gq_fwd_jobs_kernel<GG_EPI_SWIGLU, F8, 128>), grid, block, 0, s, m);
    } else if (fwd) {
        if (tile == 1) hipLaunchKernelGGL((gq_fwd_jobs_kernel<GG_EPI_STORE, F8, 64>), grid, block, 0, s, m);
        else hipLaunchKernelGGL((gq_fwd_jobs_kernel<GG_EPI_STORE, F8, 128>), grid, block, 0, s, m);
    } else if (epi == GG_EPI_SWIGLU_BWD) {
        if (f32) hipLaunchKernelGGL((gq_bwd_jobs_kernel<GG_EPI_SWIGLU_BWD, true, F8>), grid, block, 0, s, m);
        else hipLaunchKernelGGL((gq_bwd_jobs_kernel<GG_EPI_SWIGLU_BWD, false, F8>), grid, block, 0, s, m);
    } else {
        if (f32) hipLaunchKernelGGL((gq_bwd_jobs_kernel<GG_EPI_STORE, true, F8>), grid, block, 0, s, m);
        else hipLaunchKernelGGL((gq_bwd_jobs_kernel<GG_EPI_STORE, false, F8>), grid, block, 0, s, m);
    }
}
void gq_launch_jobs(hipStream_t s, bool mx, bool fwd, int epi, bool f32, int tile, const gt_jobs& m) {
    mx ? gq_jobs<2>(s, fwd, epi, f32, tile, m) : gq_jobs<1>(s, fwd, epi, f32, tile, m);
}
// Kept by a batch: calls on small tiles (data gradients: 64 rows), without copies of their output or with both MXFP8 ones
bool gq_submit(moe_ctx* ctx, hipStream_t s, int mode, int epi, bool out_f32, bool mx, int tile, const gg_args& a) {
    if (ctx->batch && tile != 3 && !(mode == GG_DGRAD && tile == 2) && (!a.out_q || (mx && a.out_qc))) {
        batch_gemm(ctx, {s, mode, epi, 0, tile, mx ? JOB_MX : JOB_FP8, out_f32, false, a});
        return true;
    }
    gq_launch(ctx, s, mode, epi, out_f32, mx, tile, a);
    return false;
}
