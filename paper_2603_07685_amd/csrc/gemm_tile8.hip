// Grouped GEMM on small tiles, one-byte operands (blockwise fp8 and MXFP8): the counterpart of gemm_tile.hip, for the calls
// whose 256 x 256 tiles are too few for the compute units or whose contraction is a few stages.
//
// A 256-thread workgroup computes one BM x 128 tile (BM = 64 or 128), four waves as 2 x 2, wave tile BM/2 x 64 in 32 x 32
// blocks of v_mfma_scale_f32_32x32x64_f8f6f4: fragments, contraction order and the software rescaling of the blockwise
// recipe are those of gemm.hip's kernel, so the two give the same bits.  A stage is 128 contraction elements (128 bytes of a
// row), two MFMA steps of 64; operands come by DMA into two stage buffers, the scales of a stage (256 dwords) into a ring of
// four, because the blockwise weight gradient needs the previous stage's beside the current.
// The quantising epilogues are not built here: their 1 x 128 blocks span two tiles; the caller runs the quantiser on the
// stored tensor instead (the same bits by construction), one more launch.
//
// Bound: as gemm_tile.hip, the fixed cost around a few stages; the 256 x 256 kernel's output phase, quantisation included, is
// 30-55 us of one workgroup per tile.  Measured (us, that kernel : this), T 1024, h 512, f 256, 8 experts, top-4, blockwise:
// fc1 + SwiGLU + quantised copy 31 : 10 (+ 4 for the quantiser), fc2 15 : 7, fc2 data gradient + SwiGLU backward + copies
// 55 : 10 (+ 5), weight gradients 28, 29 : 13, 13, fc1 data gradient 18 : 8.
#include "gemm_tile.h"

// 4 bytes per lane from a per-lane address; LDS side: M0 + 4 * lane
__device__ __forceinline__ void dma4_addr(const void* src, uint32_t lds_wave, uint32_t lds_const) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 ::"s"(m0_value(lds_wave, lds_const)), "v"(src) : "memory", "m0");
}
// the 32 contraction values of a lane from a contraction-major tile of 128-byte rows (gemm.hip: lds_read_tr8x32)
__device__ __forceinline__ i32x8_t read_tr8x32_p128(const char* p, int second) {
    const i32x2_t r0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2_t*)p);
    const i32x2_t r1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2_t*)(p + 8 * 128));
    const i32x2_t r2 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2_t*)(p + second * 128));
    const i32x2_t r3 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2_t*)(p + (second + 8) * 128));
    const i32x8_t v = {r0.x, r0.y, r1.x, r1.y, r2.x, r2.y, r3.x, r3.y};
    return v;
}

// F8: 1 = blockwise (fp32 block scales applied to the accumulators), 2 = MXFP8 (E8M0 scales, by the matrix instruction)
template <int MODE, int EPI, bool OUT_F32, int F8, int BM>
__global__ __launch_bounds__(256, BM == 64 ? 3 : 2) void gq_kernel(const gg_args a) {
    constexpr bool MX = F8 == 2, P_CMAJ = MODE == GG_WGRAD, Q_CMAJ = MODE != GG_FWD, BW_WGRAD = F8 == 1 && MODE == GG_WGRAD;
    static_assert(MODE != GG_WGRAD || BM == 128, "contraction-major tiles have 128-byte rows");
    constexpr int P_BYTES = BM * 128, STAGE = P_BYTES + GT_BN * 128;
    constexpr int PC = BM / 32, QC = 4, XC = PC + QC + 1;   // DMA instructions per wave and stage: P, Q, scales
    constexpr int NI = BM / 64;                             // 32-row blocks per wave
    __shared__ __attribute__((aligned(1024))) char ring[2 * STAGE];
    __shared__ __attribute__((aligned(16))) float scales[4][256];   // per stage: P rows from 0 on, Q rows (or column blocks) from 128 on
    __shared__ tile_pick_lds pick;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    const int N = a.N, K = a.K;
    const int J = MODE == GG_FWD ? N : K;
    const int half_cols = EPI == GG_EPI_SWIGLU ? N >> 1 : 0;
    const int tiles_j = EPI == GG_EPI_SWIGLU ? (half_cols + 63) / 64 : (J + GT_BN - 1) / GT_BN;
    const int tiles_iw = (N + BM - 1) / BM;                 // wgrad
    if (MODE == GG_WGRAD || a.out_qc) {   // (scale blocks down the rows must not straddle two experts)
        bool off_grid = false;
        for (int e = tid; e <= a.E; e += 256) off_grid |= (a.offsets[e] & 127) != 0;
        if (__syncthreads_or(off_grid)) {
            if (blockIdx.x == 0 && tid == 0) atomicExch(a.dev_err, 1);
            return;
        }
    }
    int e, u, row_lo, row_hi;
    if (!tile_pick<256>(a.offsets, a.E, a.Rcap, a.dev_err, MODE == GG_WGRAD ? 0 : BM,
                        MODE == GG_WGRAD ? tiles_iw * tiles_j : tiles_j, pick, e, u, row_lo, row_hi)) return;
    int ti, tj;
    gt_place(u, MODE == GG_WGRAD ? tiles_iw : (row_hi - row_lo + BM - 1) / BM, tiles_j, ti, tj);
    const int i0 = MODE == GG_WGRAD ? ti * BM : row_lo + ti * BM;
    const int i_end = MODE == GG_WGRAD ? N : row_hi;
    const int j0 = EPI == GG_EPI_SWIGLU ? tj * 64 : tj * GT_BN;
    const int c_lo = MODE == GG_WGRAD ? row_lo : 0, c_hi = MODE == GG_WGRAD ? row_hi : (MODE == GG_FWD ? K : N);
    const int KT = __builtin_amdgcn_readfirstlane((c_hi - c_lo) / 128);
    const int CB = (MODE == GG_FWD ? K : N) / 128;          // contraction blocks (forward, data gradient)
    auto q_col = [&](int rho) { return EPI == GG_EPI_SWIGLU ? (rho < 64 ? j0 + rho : half_cols + j0 + rho - 64) : j0 + rho; };

    // ---- operand transfers: 1 KB chunks of 8 rows x 128 B, lane -> row l / 8, 16-byte slot l % 8.  Row-major: slot ^
    // KM_SWZ(row); contraction-major: slot ^ 2 * (row / 2 % 4): a transposing read of 8 rows x 32 bytes then covers all 16
    // slots of the 256-byte bank line once (two rows share a line) ----
    const int ldp = MODE == GG_FWD ? K : N;
    uint32_t po[PC], qo[QC];
#pragma unroll
    for (int i = 0; i < PC; ++i) {
        const int row = (wave * PC + i) * 8 + (lane >> 3);
        if (P_CMAJ) po[i] = (uint32_t)(row * ldp + i0 + ((lane & 7) ^ (2 * ((row >> 1) & 3))) * 16);
        else po[i] = (uint32_t)(row * ldp) + ((lane & 7) ^ KM_SWZ(row)) * 16;
    }
#pragma unroll
    for (int i = 0; i < QC; ++i) {
        const int row = (wave * QC + i) * 8 + (lane >> 3);
        if (Q_CMAJ) qo[i] = (uint32_t)(row * K + j0 + ((lane & 7) ^ (2 * ((row >> 1) & 3))) * 16);
        else qo[i] = (uint32_t)q_col(row) * (uint32_t)K + ((lane & 7) ^ KM_SWZ(row)) * 16;
    }
    const char* const p_base0 = (const char*)a.P + (int64_t)(P_CMAJ ? c_lo : i0) * ldp;
    const char* const q_base0 = (const char*)a.Q + (MODE == GG_WGRAD ? (int64_t)c_lo * K : (int64_t)e * N * K);
    const uint32_t p_all = (uint32_t)min(BM, i_end - i0) * (uint32_t)ldp, q_all = (uint32_t)N * (uint32_t)K;
    auto make = [](const char* base, uint32_t bytes) __attribute__((always_inline)) {
        const uint64_t b = (uint64_t)base;
        i32x4_t r = {(int)__builtin_amdgcn_readfirstlane((uint32_t)b), (int)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)),
                     (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000};
        return r;
    };
    // scales: this lane's dword of stage 0 and the advance per stage (elements); waves 0, 1: P rows, waves 2, 3: Q rows
    const float* sc_src;
    int64_t sc_step;
    if (wave < 2) {
        const int q = min(wave * 64 + lane, BM - 1);
        if (MODE == GG_WGRAD) {
            sc_src = a.p_scale + (int64_t)(c_lo >> 7) * N + min(i0 + q, N - 1);
            sc_step = N;
        } else {
            sc_src = a.p_scale + (int64_t)min(i0 + q, i_end - 1) * CB;
            sc_step = 1;
        }
    } else {
        const int q = (wave - 2) * 64 + lane;
        if (MODE == GG_WGRAD) {
            sc_src = a.q_scale + (int64_t)(c_lo >> 7) * K + min(j0 + q, K - 1);
            sc_step = K;
        } else if (MX) {
            const int col = min(q_col(q), J - 1);
            sc_src = MODE == GG_FWD ? a.q_scale + ((int64_t)e * N + col) * CB : a.q_scale + (int64_t)e * (N >> 7) * K + col;
            sc_step = MODE == GG_FWD ? 1 : K;
        } else {   // one scale per 128 x 128 block: even lanes the block of the tile's first columns, odd lanes of the last
            const int col = min(q_col((lane & 1) * 64), J - 1);
            sc_src = MODE == GG_FWD ? a.q_scale + ((int64_t)e * (N / 128) + col / 128) * (K / 128)
                                    : a.q_scale + (int64_t)e * (N / 128) * (K / 128) + col / 128;
            sc_step = MODE == GG_FWD ? 1 : K / 128;
        }
    }
    const uint32_t lds0 = lds_addr(ring), sc0 = lds_addr(scales);
    i32x4_t rp, rq;
    const float* sc_at;
    auto describe = [&](int s) __attribute__((always_inline)) {   // (behind the last stage nothing is fetched: zeros)
        const uint32_t rows = s < KT ? 128u : 0u;
        rp = make(p_base0 + (int64_t)s * (P_CMAJ ? 128 * (int64_t)ldp : 128), P_CMAJ ? rows * (uint32_t)ldp : s < KT ? p_all - (uint32_t)s * 128 : 0u);
        rq = make(q_base0 + (int64_t)s * (Q_CMAJ ? 128 * (int64_t)K : 128), Q_CMAJ ? rows * (uint32_t)K : s < KT ? q_all - (uint32_t)s * 128 : 0u);
        sc_at = sc_src + (int64_t)min(s, KT - 1) * sc_step;
    };
    auto issue_one = [&](int s, uint32_t at, int x) __attribute__((always_inline)) {
        if (x < PC) dma16_buf(rp, po[x], at + wave * (PC * 1024), x * 1024);
        else if (x < PC + QC) dma16_buf(rq, qo[x - PC], at + wave * (QC * 1024), P_BYTES + (x - PC) * 1024);
        else dma4_addr(sc_at, sc0 + (s & 3) * 1024 + wave * 256, 0);
    };

    // ---- fragments (gemm.hip: fetch) ----
    const int fr_row = lane & 31, fr_khalf = lane >> 5, fr_swz = KM_SWZ(lane & 31);
    const int tr_i = lane & 15, tr_blk = lane >> 4;
    const int tr_off = ((MX ? 16 : 32) * (tr_blk >> 1) + (tr_i >> 1)) * 128 + (tr_i & 1) * 8;
    auto col_of = [&](int j) __attribute__((always_inline)) { return EPI == GG_EPI_SWIGLU ? j * 64 + wn * 32 : wn * 64 + j * 32; };
    auto frag = [&](const char* t, bool cmaj, int half, int row) __attribute__((always_inline)) -> i32x8_t {
        if (cmaj) return read_tr8x32_p128(t + half * 64 * 128 + tr_off + (((row / 16) ^ (2 * (tr_i >> 2))) + (tr_blk & 1)) * 16, MX ? 32 : 16);
        const int sl0 = MX ? 4 * half + fr_khalf : 4 * half + 2 * fr_khalf, sl1 = MX ? sl0 + 2 : sl0 + 1;
        const i32x4_t lo = *(const i32x4_t*)(t + (row + fr_row) * 128 + (sl0 ^ fr_swz) * 16);
        const i32x4_t hi = *(const i32x4_t*)(t + (row + fr_row) * 128 + (sl1 ^ fr_swz) * 16);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    i32x8_t fp[2][NI], fq[2][2];
    auto read_set = [&](int set, const char* t, int half) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) fq[set][j] = frag(t + P_BYTES, Q_CMAJ, half, col_of(j));
#pragma unroll
        for (int i = 0; i < NI; ++i) fp[set][i] = frag(t, P_CMAJ, half, wm * (BM / 2) + 32 * i);
    };
    f32x16_t acc[NI][2];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[i][j][x] = 0.f;
    // MXFP8: the lane's E8M0 bytes, shifted so that its block is byte 0 (first step) / 2 (second).  Blockwise: the running
    // scales the accumulators are in units of (see gemm.hip)
    int ps[NI], qs[2];
    float ps_cur[NI], qs_cur[2] = {1.f, 1.f};
#pragma unroll
    for (int i = 0; i < NI; ++i) ps_cur[i] = 1.f;
    auto scale_cols = [&](const float* now, const float* before, const float (&rp_)[NI]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int c = 128 + col_of(j) + 8 * g + 4 * fr_khalf;
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
    auto enter_stage = [&](int s) __attribute__((always_inline)) {   // the scales of stage s are in LDS
        const float* const now = scales[s & 3];
        if (MX) {
#pragma unroll
            for (int i = 0; i < NI; ++i) ps[i] = (int)(__float_as_uint(now[wm * (BM / 2) + 32 * i + fr_row]) >> (8 * fr_khalf));
#pragma unroll
            for (int j = 0; j < 2; ++j) qs[j] = (int)(__float_as_uint(now[128 + col_of(j) + fr_row]) >> (8 * fr_khalf));
        } else if (BW_WGRAD) {
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
            float qr[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float qn = now[128 + (EPI == GG_EPI_SWIGLU ? j : 0)];
                qr[j] = qs_cur[j] * __builtin_amdgcn_rcpf(qn);
                qs_cur[j] = qn;
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const float pn = now[wm * (BM / 2) + 32 * i + fr_row], pr = ps_cur[i] * __builtin_amdgcn_rcpf(pn);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
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
            for (int j = 0; j < 2; ++j) {
                if (!MX) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fq[half][j], fp[half][i], acc[i][j], 0, 0, 0, 127, 0, 127);
                else if (half == 0) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fq[half][j], fp[half][i], acc[i][j], 0, 0, 0, qs[j], 0, ps[i]);
                else acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fq[half][j], fp[half][i], acc[i][j], 0, 0, 2, qs[j], 2, ps[i]);
                __builtin_amdgcn_sched_barrier(0);
                slot(i * 2 + j);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    constexpr int NM = NI * 2;   // MFMAs per step

    if (KT > 0) {               // (an expert without rows: not even its scales' address is inside the tensor)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            describe(s);
#pragma unroll
            for (int x = 0; x < XC; ++x) issue_one(s, lds0 + s * STAGE, x);
        }
        wait_vm<XC>();
        stage_barrier();
        read_set(0, ring, 0);
        for (int s = 0; s < KT; ++s) {
            const char* const t0 = ring + (s & 1) * STAGE;
            const char* const t1 = ring + ((s + 1) & 1) * STAGE;
            enter_stage(s);
            read_set(1, t0, 1);
            step(0, [&](int) {});
            describe(s + 2);
            wait_vm<0>();       // stage s + 1 and its scales have landed, this wave's reads of this buffer are done
            wait_lgkm0();
            stage_barrier();
            read_set(0, t1, 0);
            step(1, [&](int m) __attribute__((always_inline)) {
#pragma unroll
                for (int x = 0; x < XC; ++x)
                    if (x * NM / XC == m) issue_one(s + 2, lds0 + (s & 1) * STAGE, x);
            });
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

    gt_output<MODE, EPI, OUT_F32, BM>(a, (float*)ring, e, i0, i_end, j0, tj, tiles_j, [&](int pass, float* stg) __attribute__((always_inline)) {
        // a lane's accumulators of a block: one row (lane % 32), four groups of columns 8 g + 4 (lane / 32) .. + 3
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4_t v;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    v[x] = acc[pass][j][4 * g + x];
                    if (!MX && !BW_WGRAD) v[x] *= ps_cur[pass] * qs_cur[j];
                }
                *(f32x4_t*)(stg + (wm * 32 + fr_row) * STG_PITCH + col_of(j) + 8 * g + 4 * fr_khalf) = v;
            }
    });
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <int MODE, int EPI, bool F32, int F8, int BM>
static void gq_go(hipStream_t s, const gg_args& a) {
    const int64_t cols = EPI == GG_EPI_SWIGLU ? ceil_div64(a.N / 2, 64) : ceil_div64(MODE == GG_FWD ? a.N : a.K, GT_BN);
    const int64_t n = cols * (MODE == GG_WGRAD ? a.E * ceil_div64(a.N, BM) : ceil_div64(a.Rcap, BM) + a.E);
    hipLaunchKernelGGL((gq_kernel<MODE, EPI, F32, F8, BM>), dim3((unsigned)(ceil_div64(n, 8) * 8)), dim3(256), 0, s, a);
}
template <int F8>
static void gq_pick(hipStream_t s, int mode, int epi, bool out_f32, int tile, const gg_args& a) {
    if (mode == GG_WGRAD) {
        if (out_f32) gq_go<GG_WGRAD, GG_EPI_STORE, true, F8, 128>(s, a);
        else gq_go<GG_WGRAD, GG_EPI_STORE, false, F8, 128>(s, a);
        return;
    }
#define GQ_ROWS(MODE, EPI) (tile == 1 ? gq_go<MODE, EPI, false, F8, 64>(s, a) : gq_go<MODE, EPI, false, F8, 128>(s, a))
    if (mode == GG_FWD) epi == GG_EPI_SWIGLU ? GQ_ROWS(GG_FWD, GG_EPI_SWIGLU) : GQ_ROWS(GG_FWD, GG_EPI_STORE);
    else epi == GG_EPI_SWIGLU_BWD ? GQ_ROWS(GG_DGRAD, GG_EPI_SWIGLU_BWD) : GQ_ROWS(GG_DGRAD, GG_EPI_STORE);
#undef GQ_ROWS
}

// Which kernel serves a call: 1 = 64 x 128 tiles, 2 = 128 x 128, 0 = the 256 x 256 kernel.  Decided from the call's sizes by
// two estimates of its time in microseconds, fitted to measured calls (MI355X; the rows of an expert are unknown on the host:
// R is taken to hold half a 128-row tile of slack per expert, and an expert's rows to be multiples of 128):
//   256 x 256: one workgroup per compute unit, whole rounds of tiles, a tile = per stage 2.1 (MXFP8), 2.35 (blockwise) or 3.4
//              (blockwise weight gradient: two multiplies per accumulator and stage) + its output phase: 8 (weight gradient,
//              blockwise: 11.5), SwiGLU 19, SwiGLU backward 38, or 57 when most units are in it at once (then bound by
//              memory); 14 and 35 without quantised copies
//   128 x 128: two workgroups per compute unit, a round = 1.5 per stage (SwiGLU 1.7; weight gradient 1.25, blockwise 2.1) + 6.5
//              (SwiGLU backward 16); plus the quantiser's launch and its way over memory
// Measured against each other (us, 256 x 256 : small tiles, quantiser included), fc1 forward / fc2 dgrad + SwiGLU backward /
// fc1 wgrad, MXFP8:
//   T 256 h 128 f 128 E 8 k 2       20 : 11    34 : 12     9 : 6       T 2048 h 1024 f 512 E 8 k 2      36 : 25    54 : 23    19 : 14
//   T 4096 h 512 f 512 E 16 k 4     55 : 44    53 : 44    26 : 18      T 4096 h 2048 f 1024 E 8 k 2    106 : 88    91 : 72    51 : 64
//   T 16384 h 256 f 256 E 32 k 4    74 : 61   121 : 76    45 : 23      T 8192 h 1024 f 1024 E 16 k 4   184 : 190  215 : 173   83 : 106
//   T 2048 h 2048 f 1024 E 8 k 2    53 : 54    71 : 42    34 : 46      T 1024 h 4096 f 1536 E 16 k 8   208 : 270  141 : 152  192 : 263
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
    const double out256 = sw ? (quant ? 19 : 14) : swb ? (!quant ? 35 : 2 * n256 > cu ? 57 : 38) : wg && !mx ? 11.5 : 8;
    const double t256 = r256 * ((mx ? 2.1 : wg ? 3.4 : 2.35) * stages + out256);
    const double per_stage = wg ? (mx ? 1.25 : 2.1) : sw ? 1.7 : 1.5;
    double t128 = (3 * r128 + __builtin_ceil(r128)) / 4;
    t128 = (t128 < 0.5 ? 0.5 : t128) * (per_stage * stages + (swb ? 16 : 6.5));
    if (quant) t128 += 4 + R * (sw ? a.N / 2 : 2 * a.K) * (mx ? 4 : 3) / 5e6;   // (bytes at 5 TB/s)
    if (t128 > t256) return 0;
    return wg || r128 >= 1.5 ? 2 : 1;
}
void gq_launch(hipStream_t s, int mode, int epi, bool out_f32, bool mx, int tile, const gg_args& a) {
    if (mx) gq_pick<2>(s, mode, epi, out_f32, tile, a);
    else gq_pick<1>(s, mode, epi, out_f32, tile, a);
}
