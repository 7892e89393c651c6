// Grouped GEMM on small tiles (bf16 operands): the calls that the 256 x 256 kernel of gemm.hip serves badly, because its
// tiles are too few for the 256 compute units, mostly padding (a few rows per expert), or because a contraction of a few
// stages does not pay for that kernel's set-up and output phases.
//
// Same operation, operand layouts and LDS swizzles as there: OUT[i,j] = sum_c P[i,c] * Q[j,c], the contraction in stages
// of 64 elements (128 bytes of a row: whole cache lines), row-major operands read with ds_read_b128, contraction-major
// ones with the transposing ds_read_b64_tr_b16.  The contraction order inside a result is that kernel's too, so the two
// give the same bits (dprob's partial sums, which group other columns, aside).
//
// A 256-thread workgroup computes one BM x 128 tile (BM = 64 or 128), four waves as 2 x 2, wave tile BM/2 x 64 in 16 x 16
// blocks; operands come by global -> LDS DMA into a ring of NBUF stage buffers, NBUF - 1 stages ahead of their use, awaited
// by count (vmcnt), with one barrier per stage.  The DMA goes through buffer descriptors: rows behind a tensor's or a
// contraction's end arrive as zeros, without a branch.
//
// Bound: the fixed cost around a short contraction (finding the tile, the first operands' latency, the output: about 5 us)
// and the rate at which a compute unit's L1 takes lines from the L2 (35-45 bytes per ns here, in the 256 x 256 kernel too;
// the matrix pipes are 13-36 % busy over the calls of T 2048, h 1024, f 512 and T 1999, h 2880, f 1472, the LDS 12-29 %).  What helped
// is waves: NBUF = 2 keeps two (BM = 128) or three (64) workgroups on a compute unit, which cover each other's waits; with a ring of
// four stages and one workgroup, the same bytes ahead, a call takes 1.25-1.5 times as long (fc1 forward, T 2048, h 1024, f 512, 8
// experts, top-2: 24 us against 33, BM = 128).  A persistent form, whose operand stream runs on across tiles, was no faster (27 us) and
// its static share of the tiles made it slower where there are many (BM = 64, 24 experts, 8000 rows: 309 us against 251).
// Where the rows of an expert fit one tile and the call streams the weights, or the tiles leave at most two to a unit, a third
// buffer is worth more than the third workgroup (decoding, 32 rows on each of 16 experts, 403 MB of fc1 weights: 92 us against
// 98, 4.4 TB/s).  The other way round, weight gradients of a few stages and many tiles are mostly output: one buffer, no operand
// ahead, and three workgroups to a unit (gt_one_buffer).
#include "gemm_tile.h"

// Weight gradients that are split (gt_spread): an expert of more than split_limit rows is cut into pieces of at most that many,
// each with its own tiles, which leave their results as fp32 in a slice of the workspace; gt_add_kernel adds an expert's slices in
// order.  One workgroup would otherwise walk all its rows (0.54 us per 64).  The limit is at least `least` and such that the pieces of any
// load fit the slices: with R <= n lim, the m <= min(n - 1, E) experts above lim have at most n - 1 + m pieces, which is cap for
// n = cap / 2 + 1 and for n = cap - E alike.
__device__ __forceinline__ int split_limit(const int32_t* __restrict__ offsets, int E, int cap, int least) {
    if (cap < 2) return 0;
    const int rows = offsets[E] - offsets[0], n = max(cap / 2 + 1, cap - E);
    return max((int)(((int64_t)rows + n * 64 - 1) / (n * 64)) * 64, least);
}

// The LDS of a workgroup
template <int MODE, int GATH, int BM, int NBUF>
struct gt_lds {
    static constexpr int STAGE = (BM + GT_BN) * 128;
    static constexpr int STAGED = 64 * STG_PITCH * 4;    // (the output phase stages 64 rows in the ring)
    __attribute__((aligned(1024))) char ring[NBUF * STAGE > STAGED ? NBUF * STAGE : STAGED];
    tile_pick_lds pick;
    // weight gradient with a gathered operand: byte offsets of the rows of two blocks of 16 stages (see rows_in)
    uint32_t rows_at[GATH != 0 && MODE == GG_WGRAD ? 2048 : 1];
    int slices_before;
};
// GATH: 0 no gathered operand, 1 P, 2 Q (weight gradient), 3 P if the call has a map (row-major P).
// `block`: the workgroup's place among those of its call
template <int MODE, int EPI, bool OUT_F32, int GATH, int BM, int NBUF, bool SPLIT>
__device__ __forceinline__ void gt_body(const gg_args& a, gt_lds<MODE, GATH, BM, NBUF>& lds, const int block) {
    static_assert(!SPLIT || MODE == GG_WGRAD, "the weight gradient's contraction is the one whose length depends on the load");
    static_assert(GATH == 2 ? MODE == GG_WGRAD : GATH != 3 || MODE != GG_WGRAD, "Q is gathered in the weight gradient only");
    constexpr bool P_CMAJ = MODE == GG_WGRAD, Q_CMAJ = MODE != GG_FWD;
    constexpr int P_BYTES = BM * 128, STAGE = P_BYTES + GT_BN * 128;
    constexpr int PC = BM / 32, QC = 4;                 // 1 KB DMA chunks per wave, operand and stage
    constexpr int NI = BM / 32;                         // 16-row blocks per wave
    char* const ring = lds.ring;
    tile_pick_lds& pick = lds.pick;
    uint32_t* const rows_at = lds.rows_at;
    constexpr bool G_CM = GATH != 0 && MODE == GG_WGRAD;
    const bool gath_p = GATH == 1 || (GATH == 3 && a.g_src_of);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    const int N = a.N, K = a.K;
    const int J = MODE == GG_FWD ? N : K;
    const int half_cols = EPI == GG_EPI_SWIGLU ? N >> 1 : 0;
    const int tiles_j = EPI == GG_EPI_SWIGLU ? (half_cols + 63) / 64 : (J + GT_BN - 1) / GT_BN;
    const int tiles_iw = (N + BM - 1) / BM;             // wgrad

    int e, u, row_lo, row_hi;
    const int lim = SPLIT ? split_limit(a.offsets, a.E, a.split_cap, a.split_rows) : 0;
    tile_sums<256> sums;
    // A weight gradient without pieces has the same number of tiles for every expert: its tile is found without a sum over the
    // experts.  The check of all offsets goes on while the first operands are on their way (from rows made safe by
    // clamping), and is asked for its answer at the first barrier.
    constexpr bool EVEN = MODE == GG_WGRAD && !SPLIT;
    bool bad = false;
    if (EVEN) {
        const int tpe = tiles_iw * tiles_j, total = a.E * tpe, run = (total + 7) >> 3, at = block >> 3;
        const int unit = (block & 7) * run + at;
        if (at >= run || unit >= total) return;
        e = unit / tpe;
        u = unit - e * tpe;
        row_lo = min(max(__builtin_amdgcn_readfirstlane(a.offsets[e]), 0), (int)a.Rcap);
        row_hi = min(max(__builtin_amdgcn_readfirstlane(a.offsets[e + 1]), row_lo), (int)a.Rcap);
        for (int x = tid; x < a.E; x += 256) bad |= a.offsets[x + 1] < a.offsets[x];
        bad |= a.offsets[0] < 0 || a.offsets[a.E] > a.Rcap;
        pick.wave_bad[wave] = __builtin_amdgcn_ballot_w64(bad) != 0;
    } else {
        if (!tile_scan<256>(a.offsets, a.E, a.Rcap, a.dev_err, MODE == GG_WGRAD ? 0 : BM,
                            MODE == GG_WGRAD ? tiles_iw * tiles_j : tiles_j, pick, sums, block == 0, lim)) return;
        if (SPLIT && tid == 0) lds.slices_before = 0;
        if (!tile_find(sums, block, pick, e, u, row_lo, row_hi)) return;
    }
    int slice = -1;   // >= 0: a piece, its place among the partial results
    if (SPLIT && lim > 0) {   // (0: a call without pieces beside one that has them)
        const int pieces = __builtin_amdgcn_readfirstlane(split_pieces(row_hi - row_lo, lim));
        if (pieces > 1) {
            int n = 0;
#pragma unroll
            for (int x = 0; x < tile_sums<256>::PER; ++x) {
                const int p = split_pieces(sums.o[x + 1] - sums.o[x], lim);
                n += tid * tile_sums<256>::PER + x < e && p > 1 ? p : 0;
            }
            if (n) atomicAdd(&lds.slices_before, n);
            __syncthreads();
            const int tpe = tiles_iw * tiles_j, piece = __builtin_amdgcn_readfirstlane(u / tpe);
            const int len = ((row_hi - row_lo + pieces - 1) / pieces + 63) / 64 * 64;   // (whole stages; none is empty)
            slice = __builtin_amdgcn_readfirstlane(lds.slices_before) + piece;
            u -= piece * tpe;
            row_lo += piece * len;
            row_hi = min(row_lo + len, row_hi);
        }
    }
    int ti, tj;
    {
        const int tiles_i = MODE == GG_WGRAD ? tiles_iw : (row_hi - row_lo + BM - 1) / BM;
        gt_place(u, tiles_i, tiles_j, ti, tj);
    }
    const int i0 = MODE == GG_WGRAD ? ti * BM : row_lo + ti * BM;
    const int i_end = MODE == GG_WGRAD ? N : row_hi;
    const int j0 = EPI == GG_EPI_SWIGLU ? tj * 64 : tj * GT_BN;
    const int c_lo = MODE == GG_WGRAD ? row_lo : 0, c_hi = MODE == GG_WGRAD ? row_hi : (MODE == GG_FWD ? K : N);
    const int KT = __builtin_amdgcn_readfirstlane((c_hi - c_lo + 63) / 64);

    // ---- DMA sources: 32-bit lane offsets from a wave-uniform base ----
    // row-major: a chunk = 8 rows x 128 B, lane -> row l / 8, slot l % 8 ^ KM_SWZ(row).  contraction-major: a chunk =
    // 1024 / pitch rows (pitch = 2 x the tile's columns), lane -> 16-byte slot, ^ 2 * (row % 4 | separating bit << 2):
    // the eight 4-row groups that the LDS serves in one pass of a transposing read (4 rows of two lane groups) then hit
    // different 32-byte bank segments.  The separating bit is the row bit that tells the two lane groups apart.
    constexpr int SEP = MODE == GG_WGRAD ? 4 : 3;
    auto cm_f = [](int row) { return 2 * ((row & 3) | (((row >> SEP) & 1) << 2)); };
    const int ldp = MODE == GG_FWD ? K : N;             // row length of P in memory (wgrad: dC [rows, N])
    uint32_t po[PC], qo[QC];
#pragma unroll
    for (int i = 0; i < PC; ++i) {
        const int c = wave * PC + i;
        if (P_CMAJ) {
            constexpr int SL = BM * 2 / 16;             // 16-byte slots per row
            const int row = c * (64 / SL) + lane / SL, slot = (lane % SL) ^ cm_f(row);
            po[i] = (uint32_t)((GATH == 1 ? 0 : row * ldp) + i0 + slot * 8) * 2u;
        } else {
            const int row = c * 8 + (lane >> 3), slot = (lane & 7) ^ KM_SWZ(row);
            if (gath_p) {
                const int s = i0 + row < i_end ? a.g_src_of[i0 + row] : -1;
                const uint32_t tok = __umulhi(2u * (uint32_t)s + 1u, a.g_magic);  // s / g_k
                po[i] = s >= 0 ? tok * (uint32_t)(ldp * 2) + slot * 16 : GG_NO_ROW;
            } else {
                po[i] = (uint32_t)(row * ldp) * 2u + slot * 16;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < QC; ++i) {
        const int c = wave * QC + i;
        if (Q_CMAJ) {
            const int row = c * 4 + (lane >> 4), slot = (lane & 15) ^ cm_f(row);
            qo[i] = (uint32_t)((GATH == 2 ? 0 : row * K) + j0 + slot * 8) * 2u;
        } else {
            const int p = c * 8 + (lane >> 3), slot = (lane & 7) ^ KM_SWZ(p);
            const int n = EPI == GG_EPI_SWIGLU ? (p < 64 ? j0 + p : half_cols + j0 + p - 64) : j0 + p;
            qo[i] = (uint32_t)n * (uint32_t)(K * 2) + slot * 16;
        }
    }
    // base and byte count of each operand at stage s (past the last stage: nothing, the buffer fills with zeros)
    const char* const p_base0 = gath_p ? (const char*)a.P
                                          : (const char*)a.P + (int64_t)(P_CMAJ ? c_lo : i0) * ldp * 2;
    const char* const q_base0 = GATH == 2 ? (const char*)a.Q : MODE == GG_WGRAD ? (const char*)a.Q + (int64_t)c_lo * K * 2
                                                 : (const char*)a.Q + (int64_t)e * N * K * 2;
    const uint32_t p_all = gath_p ? (uint32_t)a.g_T * (uint32_t)(ldp * 2) : (uint32_t)min(BM, i_end - i0) * (uint32_t)(ldp * 2);
    const uint32_t q_all = GATH == 2 ? (uint32_t)a.g_T * (uint32_t)(K * 2) : (uint32_t)N * (uint32_t)(K * 2);
    auto make = [](const char* base, uint32_t bytes) {
        const uint64_t b = (uint64_t)base;
        i32x4_t r = {(int)__builtin_amdgcn_readfirstlane((uint32_t)b), (int)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)),
                     (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000};
        return r;
    };
    // Gathered operand of the weight gradient: every stage brings 64 new rows, found through the row map.  The byte offsets
    // of the rows of 16 stages at a time are looked up ahead by the whole workgroup and kept in LDS, two blocks in turn
    // (rows without a source and rows behind the contraction range: an offset that reads as zeros).  Looking them up in
    // the stage loop would wait for the map entry, and with it for every transfer in flight, in each stage.
    auto rows_in = [&](int blk) {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int at = blk * 1024 + x * 256 + tid, c = c_lo + at;
            const int s = c < c_hi ? a.g_src_of[c] : -1;
            const uint32_t tok = __umulhi(2u * (uint32_t)s + 1u, a.g_magic);  // s / g_k
            rows_at[at & 2047] = s >= 0 ? tok * (uint32_t)((GATH == 1 ? ldp : K) * 2) : GG_NO_ROW;
        }
    };
    const uint32_t lds0 = lds_addr(ring);
    // descriptors of stage s, and its transfers one by one (x < PC: P, then Q) into buffer `at`
    i32x4_t rp, rq;
    auto describe = [&](int s) {
        const uint32_t left = (uint32_t)max(min(64, c_hi - c_lo - s * 64), 0);   // contraction rows of this stage
        rp = G_CM && GATH == 1 ? make(p_base0, p_all)
                               : make(p_base0 + (int64_t)s * (P_CMAJ ? 128 * (int64_t)ldp : 128),
                                      P_CMAJ ? left * (uint32_t)(ldp * 2) : s < KT ? p_all - (uint32_t)s * 128 : 0u);
        rq = G_CM && GATH == 2 ? make(q_base0, q_all)
                               : make(q_base0 + (int64_t)s * (Q_CMAJ ? 128 * (int64_t)K : 128),
                                      Q_CMAJ ? left * (uint32_t)(K * 2) : s < KT ? q_all - (uint32_t)s * 128 : 0u);
    };
    uint32_t g_off[G_CM ? 4 : 1];   // gathered rows of this lane's four chunks of the stage about to be requested
    auto g_rows = [&](int s) {
        if (G_CM) {
#pragma unroll
            for (int i = 0; i < 4; ++i) g_off[i] = rows_at[(s * 64 + (wave * 4 + i) * 4 + (lane >> 4)) & 2047];
        }
    };
    auto issue_one = [&](uint32_t at, int x) {
        if (x < PC) dma16_buf(rp, po[x] + (G_CM && GATH == 1 ? g_off[x] : 0u), at + wave * (PC * 1024), x * 1024);
        else dma16_buf(rq, qo[x - PC] + (G_CM && GATH == 2 ? g_off[x - PC] : 0u), at + wave * (QC * 1024), P_BYTES + (x - PC) * 1024);
    };
    if (G_CM) {
        rows_in(0);
        __syncthreads();
    }

    // ---- fragment side (the lane groups' share of a 32-element step is the 256 x 256 kernel's: same sums) ----
    const int l16 = lane & 15, kq = lane >> 4;
    const int kperm = MODE == GG_WGRAD ? 2 * (kq & 1) + (kq >> 1) : kq;
    auto col_of = [&](int jb) { return EPI == GG_EPI_SWIGLU ? (jb >> 1) * 64 + wn * 32 + (jb & 1) * 16 : wn * 64 + jb * 16; };
    const int km[2] = {(kperm ^ KM_SWZ(l16)) * 16, ((4 + kperm) ^ KM_SWZ(l16)) * 16};
    const int cm_row = 8 * kperm + (l16 >> 2), cm_x = cm_f(cm_row), cm_lo = ((l16 & 3) >> 1) * 16 + (l16 & 1) * 8;
    auto frag = [&](const char* t, bool cmaj, int pitch, int ks, int row) -> bf16x8_t {
        if (!cmaj) return *(const bf16x8_t*)(t + (row + l16) * 128 + km[ks]);
        const char* p = t + (32 * ks + cm_row) * pitch + ((row / 8) ^ cm_x) * 16 + cm_lo;
        return lds_read_tr16x8(p, p + 4 * pitch);
    };

    f32x4_t acc[NI][4];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NBUF; ++s) {
        describe(s);
        g_rows(s);
#pragma unroll
        for (int x = 0; x < PC + QC; ++x) issue_one(lds0 + s * STAGE, x);
    }
    // A stage is two contraction steps of 32 elements.  The fragments of a step are read while the MFMAs of the step
    // before it run, and the transfers of the stage that takes over this buffer are slipped between the MFMAs of the
    // second step.  In mid-stage: this wave's share of stage s + 1 has landed, its reads of this buffer are done, barrier.
    bf16x8_t fp[2][NI], fq[2][4];
    constexpr int NR = NI + 4, NM = NI * 4;               // fragment reads and MFMAs per step
    auto read_one = [&](int set, const char* t, int ks, int r) {   // in the order of use: Q 0, P 0, Q 1..3, P 1..
        const int j = r == 0 ? 0 : r - 1, i = r == 1 ? 0 : r - 4;
        if (r == 0 || (r >= 2 && r < 5)) fq[set][j] = frag(t + P_BYTES, Q_CMAJ, GT_BN * 2, ks, col_of(j));
        else fp[set][i] = frag(t, P_CMAJ, BM * 2, ks, wm * (BM / 2) + 16 * i);
    };
    auto step = [&](int set, auto&& slot) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fq[set][j], fp[set][i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                slot(i * 4 + j);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    wait_vm<(NBUF - 1) * (PC + QC)>();
    wait_lgkm0();
    stage_barrier();
    if (EVEN && (pick.wave_bad[0] | pick.wave_bad[1] | pick.wave_bad[2] | pick.wave_bad[3])) {
        wait_vm0();                                         // (nothing may land in this LDS once it is someone else's)
        if (block == 0 && tid == 0) atomicExch(a.dev_err, 1);
        return;
    }
    if constexpr (NBUF == 1) {
        // One buffer, for contractions of a stage or two: what counts is a third workgroup per compute unit.  Both steps'
        // fragments leave the buffer, then the next stage's transfers run beside the MFMAs.
        for (int s = 0; s < KT; ++s) {
            if (s) {
                wait_vm0();
                stage_barrier();
            }
#pragma unroll
            for (int r = 0; r < 2 * NR; ++r) read_one(r / NR, ring, r / NR, r % NR);
            if (s + 1 < KT) {
                wait_lgkm0();
                stage_barrier();
                describe(s + 1);
                g_rows(s + 1);
#pragma unroll
                for (int x = 0; x < PC + QC; ++x) issue_one(lds0, x);
                if (G_CM && ((s + 1) & 15) == 8) rows_in(((s + 1) >> 4) + 1);
            }
            step(0, [](int) {});
            step(1, [](int) {});
        }
    } else {
#pragma unroll
        for (int r = 0; r < NR; ++r) read_one(0, ring, 0, r);
        int buf = 0;
        for (int s = 0; s < KT; ++s) {
            const char* const t0 = ring + buf * STAGE;
            const int nbuf = buf + 1 == NBUF ? 0 : buf + 1;
            const char* const t1 = ring + nbuf * STAGE;
            step(0, [&](int m) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (r * (NM - 2) / NR == m) read_one(1, t0, 1, r);
                if (m == NM - 2) describe(s + NBUF);
                if (m == NM - 1) g_rows(s + NBUF);
            });
            wait_vm<(NBUF - 2) * (PC + QC)>();
            wait_lgkm0();
            stage_barrier();
            step(1, [&](int m) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (r * (NM - 2) / NR == m) read_one(0, t1, 0, r);
#pragma unroll
                for (int x = 0; x < PC + QC; ++x)
                    if (x * NM / (PC + QC) == m) issue_one(lds0 + buf * STAGE, x);
            });
            // (the half written here was last read 8 stages ago, and is read from 8 stages on)
            if (G_CM && ((s + NBUF) & 15) == 8 && s + NBUF < KT) rows_in(((s + NBUF) >> 4) + 1);
            buf = nbuf;
        }
    }
    wait_vm0();        // (the stages past the end: their zeros must not land in the staging area)
    wait_lgkm0();
    stage_barrier();

    auto stage = [&](int ps, float* stg) {
        // a lane's accumulators of a block: one row (l16), columns 4 kq .. 4 kq + 3
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *(f32x4_t*)(stg + (wm * 32 + 16 * i2 + l16) * STG_PITCH + col_of(j) + 4 * kq) = acc[2 * ps + i2][j];
    };
    if (SPLIT && slice >= 0) {   // (a slice is laid out as one expert's fp32 result)
        gg_args part = a;
        part.out = a.partials;
        part.accumulate = 0;
        gt_output<MODE, EPI, SPLIT, BM>(part, (float*)ring, slice, i0, i_end, j0, tj, tiles_j, stage);
        return;
    }
    gt_output<MODE, EPI, OUT_F32, BM>(a, (float*)ring, e, i0, i_end, j0, tj, tiles_j, stage);
}
template <int MODE, int EPI, bool OUT_F32, int GATH, int BM, int NBUF, bool SPLIT>
__global__ __launch_bounds__(256, NBUF == 1 ? 3 : NBUF == 2 ? (BM == 64 ? 3 : 2) : 2) void gt_kernel(const gg_args a) {
    __shared__ gt_lds<MODE, GATH, BM, NBUF> lds;
    gt_body<MODE, EPI, OUT_F32, GATH, BM, NBUF, SPLIT>(a, lds, (int)blockIdx.x);
}

// Independent calls in one launch.  Small calls leave compute units idle in their start, their output phase and the last of their
// rounds, and each launch costs about 2 us behind another; together they fill each other's gaps.  A step, us, one launch each :
// together: T 256 h 128 f 256 E 8 k 2 52.8 : 45.1; T 377 h 2240 f 512 E 8 k 2 130 : 106; T 7394 h 128 f 192 E 24 125 : 104; with a
// shared expert T 27 h 576 f 512 E 7 k 2 105 : 60, T 873 h 896 f 2688 E 12 k 2 342 : 300.
// forward calls with one epilogue
template <int EPI, int BM, int NBUF>
__global__ __launch_bounds__(256, NBUF == 2 && BM == 64 ? 3 : 2) void gt_fwd_jobs_kernel(const gt_jobs m) {
    __shared__ gt_lds<GG_FWD, 3, BM, NBUF> lds;
    const int j = gt_job_of(m, (int)blockIdx.x);
    gt_body<GG_FWD, EPI, false, 3, BM, NBUF, false>(m.a[j], lds, (int)blockIdx.x - m.start[j]);
}
// data gradients with one epilogue (calls 0, 1) and weight gradients (2, 3)
template <int EPI, int BM, int NBUF, bool F32, int WGATH, int WBUF, bool SPLIT>
__global__ __launch_bounds__(256, 2) void gt_bwd_jobs_kernel(const gt_jobs m) {
    __shared__ union {
        gt_lds<GG_DGRAD, 3, BM, NBUF> d;
        gt_lds<GG_WGRAD, WGATH, 128, WBUF> w;
    } lds;
    const int at = gt_place_of((int)blockIdx.x, m.turn, m.start[GT_JOBS]), j = gt_job_of(m, at), block = at - m.start[j];
    if (j < 2) gt_body<GG_DGRAD, EPI, false, 3, BM, NBUF, false>(m.a[j], lds.d, block);
    else gt_body<GG_WGRAD, GG_EPI_STORE, F32, WGATH, 128, WBUF, SPLIT>(m.a[j], lds.w, block);
}

// Second step of a weight gradient with pieces: every workgroup finds the split experts in the offsets (at most half of
// GT_MAX_PIECES, as each has two pieces or more) and goes over its share of their results, piece 0 first.  Bound: HBM, a slice read per
// piece; without a split expert, one look.
template <bool OUT_F32>
__global__ __launch_bounds__(256) void gt_add_kernel(const gg_args a) {
    __shared__ int at[GT_MAX_PIECES], rows_at[GT_MAX_PIECES], count;
    const int lim = split_limit(a.offsets, a.E, a.split_cap, a.split_rows);   // (> 0: launched with split_cap >= 2)
    if (threadIdx.x == 0) count = 0;
    bool bad = a.offsets[0] < 0 || a.offsets[a.E] > a.Rcap;
    for (int e = threadIdx.x; e < a.E; e += 256) bad |= a.offsets[e + 1] < a.offsets[e];
    if (__syncthreads_or(bad)) return;   // (as the first step did)
    for (int e = threadIdx.x; e < a.E; e += 256) {
        const int rows = a.offsets[e + 1] - a.offsets[e];
        if (split_pieces(rows, lim) > 1) {
            const int i = atomicAdd(&count, 1);
            at[i] = e;
            rows_at[i] = rows;
        }
    }
    __syncthreads();
    const int64_t n4 = (int64_t)a.N * a.K / 4;
    for (int i = 0; i < count; ++i) {
        int before = 0;
        for (int j = 0; j < count; ++j) before += at[j] < at[i] ? split_pieces(rows_at[j], lim) : 0;
        const int pieces = split_pieces(rows_at[i], lim);
        const f32x4_t* const src = (const f32x4_t*)a.partials + before * n4;
        for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < n4; x += (int64_t)gridDim.x * 256) {
            f32x4_t v = src[x];
            for (int p = 1; p < pieces; ++p) v += src[p * n4 + x];
            if (OUT_F32) {
                f32x4_t* const o = (f32x4_t*)a.out + at[i] * n4 + x;
                if (a.accumulate) v += *o;
                *o = v;
            } else {
                bf16_t* const o = (bf16_t*)a.out + (at[i] * n4 + x) * 4;
                float t[4] = {v[0], v[1], v[2], v[3]};
                if (a.accumulate) {
                    float old[4];
                    ld4_bf16(o, old);
#pragma unroll
                    for (int y = 0; y < 4; ++y) t[y] += old[y];
                }
                st4_bf16(o, t);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Weight gradients of more than two tiles per unit and short contractions, mostly output: one buffer, three workgroups per
// unit (fc2, fc1; two buffers : one; h 3072 f 1024 E 32, T 128 k 4 75 : 59, 143 : 109; h 4096 f 1536 E 16, T 64 k 8 63 : 45, 127 : 93).
// A hot expert's workgroups walk their rows at half the pace then, which the host cannot see; it shows once that walk is long beside
// the output of all tiles.  Hence at most 160 rows in all for every tile per unit: up to there no load was slower, also with 95 % of
// the rows on one expert; at 192 one such was (512 x 512 of 40 experts, 9.4 : 9.9), from 256 on most.  Two buffers : one, equal loads |
// half on one expert | 95 %, R rows in all (per tile and unit), N x K of E experts: 512 x 512 of 64, R 512 (128) 13 : 11 | 13 : 10 | 12
// : 10, R 1024 (256) 13 : 11 | 14 : 11 | 14 : 16, R 4096 (1024) 14 : 12 | 23 : 27 | 39 : 46; 768 x 512 of 24, R 320 (142) 10 : 8 | 10 :
// 8 | 10 : 8.4, R 864 (384) 10 : 8 | 10 : 9 | 11.5 : 12.4; 2048 x 1024 of 8, R 512 (128) 14 : 12 | 16 : 14 | 22 : 21, R 1024 (256) 15 :
// 13 | 22 : 21 | 32 : 33.5, R 2048 (512) 18 : 17 | 32 : 34 | 51 : 56; 1024 x 1024 of 64, R 2304 (144) 38 : 27 | 50 : 38 | 61 : 48.
// (256 rows per expert and 6144 in all are the most that was measured.)
static bool gt_one_buffer(const moe_ctx* ctx, const gg_args& a) {
    const int64_t tiles = a.E * ceil_div64(a.N, 128) * ceil_div64(a.K, 128), cu = ctx->num_cu > 0 ? ctx->num_cu : 256;
    return tiles > 2 * cu && a.Rcap * cu <= 160 * tiles && a.Rcap <= 256 * (int64_t)a.E && a.Rcap <= 6144;
}

// Which kernel serves a call: 1 = 64 x 128 tiles, 2 = 128 x 128, 3 = 64 x 128 with a third stage buffer, 4 = 128 x 128 on one
// (gt_one_buffer), 0 = the 256 x 256 kernel.  Decided from the call's sizes by two estimates of its time in microseconds, each fitted
// to measured calls (MI355X, bf16).  The rows of an expert are unknown on the host: several experts are taken half way between equal
// ones and ones that scatter, with half a partly filled row tile each and at least one tile.
//   256 x 256: one workgroup per compute unit, whole rounds of tiles (a twentieth of one over is not rounded up: it comes from
//              the guess), a tile = 1.5 per stage + 15 (SwiGLU backward: 34); weight gradient: + 6 for the second launch
//   128 x 128: two workgroups per compute unit, rounds between the exact and the rounded-up count, a round = 2 x (0.62 per
//              stage + 4)
//   up to 96 rows per expert, where the weights' way from memory is the time: 4.9 TB/s and 6
// Over 1814 drawn forward and data-gradient calls, from cold caches, this choice takes 1.4 % more than the best kernel of each would
// (scattered loads alone, a tenth of a round forgiven, 48 rows: 2.3 %; T 1999 h 2880 f 1472 E 24 k 4, fc2 dgrad: 192 : 144; 450 MB of
// weights for 272 rows, T 34 h 3328 f 1472 E 23 k 8, fc1: 159 : 103).
// Measured against each other (us, 256 x 256 : small tiles), fc1 forward unless said otherwise:
//   T 256 h 128 f 256 E 8 k 2       16 : 6       T 2048 h 1024 f 512 E 8 k 2       41 : 23   (its weight gradients 38, 37 : 14, 16)
//   T 4096 h 512 f 512 E 16 k 4     56 : 43      T 4096 h 2048 f 1024 E 8 k 2     122 : 113
//   T 2048 h 2048 f 1024 E 8 k 2    65 : 74      T 1024 h 4096 f 1536 E 16 k 8    222 : 284  (fc2 dgrad of the former 72 : 36)
//   T 8192 h 1024 f 1024 E 16 k 4  200 : 230     T 64 h 7168 f 2048 E 32 k 8      429 : 312  (fc2 274 : 168)
// These are scattered loads.  One that fills whole 256-row tiles exactly is not told apart and can lose (T 4096 h 2048 f 1024
// E 8 k 2, 1024 rows each, plain fc1 forward 60 : 67; any other load there 93 : 82).  Skewed weight gradients: split_limit.
// Few rows per expert: the third buffer (T 64 h 4096 f 14336 E 8 k 2: 464 : 330 against 363 with two
// buffers and 359 with 128 x 128).  The same where the 64 x 128 tiles are at most two per unit, so that a third workgroup would
// find no work (fc1, fc2, fc2 dgrad, fc1 dgrad, two buffers : three: T 256 h 1024 f 704 E 16 k 4 18.0 : 15.4, 12.3 : 9.7, 14.6 :
// 12.2, 15.6 : 11.4; T 400 h 512 f 512 E 8 k 2 10.9 : 8.6, 7.7 : 6.2, 10.2 : 9.1, 11.8 : 9.1; but at 2.25 per unit, T 2048 h 1024
// f 512 E 8 k 2, 21.8 : 23.8, 12.2 : 14.1, 18.2 : 21.0).  Otherwise 64 x 128 while the 128 x 128 tiles would not fill six tenths of the
// chip's two workgroups per unit (one above it: 7 experts 3298 rows 1920 x 896 fc2 39 : 28); SwiGLU backward, whose output
// phase is long, up to twice what fills them if the contraction is not (128 x 128 : 64 x 128, T 3000 h 512 f 1536 E 12 k 2 34 : 28.5,
// T 4096 h 512 f 512 E 8 k 4 32 : 27, T 4008 h 1536 f 2048 E 17 52 : 48; but h 3264 f 640 E 51, 10230 rows, equal loads 83 : 116, scattered
// 119 : 115).
int gt_tile(const moe_ctx* ctx, int mode, int epi, const gg_args& a) {
    const double cu = ctx->num_cu > 0 ? ctx->num_cu : 256;
    const double E = a.E, R = (double)a.Rcap, one = E < R ? E : R;
    const double cols = mode == GG_FWD ? a.N : a.K, c256 = __builtin_ceil(cols / 256), c128 = __builtin_ceil(cols / 128);
    auto rounds = [&](double n) { return n / cu < 1 ? 1 : __builtin_ceil(n / cu); };
    if (mode == GG_WGRAD) {
        const double stages = R / E / 64 + 0.5, n256 = c256 * E * __builtin_ceil(a.N / 256.0), r128 = c128 * E * __builtin_ceil(a.N / 128.0) / (2 * cu);
        const double t256 = rounds(n256 - 0.1 * cu) * (1.5 * stages + 15) + 6, t128 = (r128 + __builtin_ceil(r128)) * (0.62 * stages + 4);
        if (t128 > 1.1 * t256) return 0;   // (weight gradients of a few stages are better than the estimate)
        return gt_one_buffer(ctx, a) ? 4 : 2;
    }
    const double stages = (mode == GG_FWD ? a.K : a.N) / 64.0;
    auto scattered = [&](double bm) {
        const double n = E == 1 ? __builtin_ceil(R / bm) : R / bm + E / 2;
        return n > one ? n : one;
    };
    auto even = [&](double bm) { return E * __builtin_ceil(R / E / bm); };
    const double t256 = 0.5 * (rounds(c256 * scattered(256) - 0.05 * cu) + rounds(c256 * even(256) - 0.05 * cu)) * (1.5 * stages + (epi == GG_EPI_SWIGLU_BWD ? 34 : 15));
    const double r128 = 0.5 * (scattered(128) + even(128)) * c128 / (2 * cu), n64 = 0.5 * (scattered(64) + even(64)) * c128;
    const double t128 = (r128 + __builtin_ceil(r128)) * (0.62 * stages + 4);
    if (R <= 96 * E) {
        const double stream = 6 + E * a.N * a.K * 2 / 4.9e6;
        return t256 < (stream < t128 ? stream : t128) ? 0 : 3;
    }
    if (t128 > t256) return 0;
    if (n64 <= 2 * cu) return 3;
    return r128 < (epi == GG_EPI_SWIGLU_BWD && stages <= 24 ? 2 : 0.6) ? 1 : 2;
}

// Weight gradients are split in two cases (pieces' results out and in again and the second launch cost about 5 us and what their
// bytes take; 540 drawn calls from cold caches):
//   few tiles, so that one workgroup's walk over an expert's rows is the call's time: as many pieces as fill two workgroups per unit,
//   of at least 8 stages, where that saves more than it costs.  Us, whole : pieces: one expert (a shared one) 13675 rows 256 x 576
//   199 : 32, 10108 384 x 192 151 : 27, 3085 768 x 128 51 : 24; 6 experts 19362 320 x 192 139 : 38; 5 experts 4890 512 x 128 27.3 : 25.8;
//   most lost: one expert 4513 rows 6144 x 512 72 : 79.
//   more than GT_SPLIT_ROWS rows of several experts, where a hot one is walked for long: pieces of the time that all work takes spread
//   evenly, but of no less than one and a half times the mean load, so that equal loads are not cut.  The second launch costs every
//   load 2.7 us.  Below the bound that is 6 % of a backward pass under equal loads, 5 % under ones scattered by 30 %, against 1.18x under
//   rank^-1.2 (means of 40 drawn layers; T 1876 h 576 f 256 E 26 k 8 90 : 98 | 91 : 99 | 144 : 125): not worth it for the loads that a
//   balanced router gives.  Above it, steps of 30 drawn layers, whole : pieces:
//   0.990 | 0.992 | 1.17 in the mean (T 16310 h 192 f 128 E 62 k 8, backward, 223 : 230 | 250 : 257 | 1093 : 539); pieces of a fifth of all
//   rows instead of these: 0.98 | 0.98 | 0.93 (0.73-1.004).
#define GT_SPLIT_ROWS 24576
void gt_spread(const moe_ctx* ctx, gg_args& a, int64_t slices) {
    const double cu = ctx->num_cu > 0 ? ctx->num_cu : 256, R = (double)a.Rcap, E = a.E, stages = R / E / 64;
    const double tiles = E * ceil_div64(a.N, 128) * ceil_div64(a.K, 128);
    if (slices > GT_MAX_PIECES) slices = GT_MAX_PIECES;
    if (slices < 2) return;
    double few = 2 * cu / tiles < stages / 8 ? 2 * cu / tiles : stages / 8;   // pieces of an expert
    if (few > slices / E) few = slices / E;
    const double all = 0.55 * tiles * (stages + 8) / (2 * cu);                // us, were everything spread evenly
    if (few >= 1.5 && 0.5 * stages * (1 - 1 / few) > 6 + 1.7e-6 * E * a.N * a.K * few) a.split_rows = (int)(R / E / few / 64 + 1) * 64;
    else if (E > 1 && R > GT_SPLIT_ROWS) {
        const double share = 1.5 * R / E, even = all < 16 ? 1024 : all * 64, rows = share > even ? share : even;
        a.split_rows = (int)((rows < R ? rows : R) / 64 + 1) * 64;
    } else return;
    // (no more room than any load can ask for: see split_limit)
    const int64_t n = a.Rcap / a.split_rows + 1, most = n + (n < a.E ? n : a.E);
    a.split_cap = (int)(slices < most ? slices : most);
}

// (a multiple of 8: every XCD gets as many workgroups of a call)
int64_t gt_blocks(int mode, int epi, int bm, const gg_args& a) {
    const int64_t cols = epi == GG_EPI_SWIGLU ? ceil_div64(a.N / 2, 64) : ceil_div64(mode == GG_FWD ? a.N : a.K, GT_BN);
    const int64_t pieces = a.split_cap >= 2 ? (a.Rcap / a.split_rows < a.split_cap ? a.Rcap / a.split_rows : a.split_cap) : 0;
    const int64_t n = cols * (mode == GG_WGRAD ? (a.E + pieces) * ceil_div64(a.N, bm) : ceil_div64(a.Rcap, bm) + a.E);
    return ceil_div64(n, 8) * 8;
}
template <int MODE, int EPI, bool F32, int GATH, int BM, int NBUF, bool SPLIT = false>
static void gt_go(hipStream_t s, const gg_args& a) {
    hipLaunchKernelGGL((gt_kernel<MODE, EPI, F32, GATH, BM, NBUF, SPLIT>), dim3((unsigned)gt_blocks(MODE, EPI, BM, a)), dim3(256), 0, s, a);
}
template <int MODE, int EPI, int GATH>
static void gt_rows(hipStream_t s, int tile, const gg_args& a) {
    if (tile == 1) gt_go<MODE, EPI, false, GATH, 64, 2>(s, a);
    else if (tile == 2) gt_go<MODE, EPI, false, GATH, 128, 2>(s, a);
    else gt_go<MODE, EPI, false, GATH, 64, 3>(s, a);
}
template <bool F32>
static void gt_add(hipStream_t s, const gg_args& a) {
    const int64_t blocks = ceil_div64((int64_t)a.N * a.K / 4, 256);
    hipLaunchKernelGGL(gt_add_kernel<F32>, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256), 0, s, a);
}
// (a kernel of its own for calls that may split: the others are 5 % faster at their smallest without the choice in them)
template <bool F32, bool SPLIT, int NBUF>
static void gt_wgrad(hipStream_t s, int gath, const gg_args& a) {
    if (gath == 1) gt_go<GG_WGRAD, GG_EPI_STORE, F32, 1, 128, NBUF, SPLIT>(s, a);
    else if (gath == 2) gt_go<GG_WGRAD, GG_EPI_STORE, F32, 2, 128, NBUF, SPLIT>(s, a);
    else gt_go<GG_WGRAD, GG_EPI_STORE, F32, 0, 128, NBUF, SPLIT>(s, a);
    if (SPLIT) gt_add<F32>(s, a);
}
void gt_launch(hipStream_t s, int mode, int epi, bool out_f32, int gath, int tile, const gg_args& a) {
    if (mode == GG_WGRAD) {
        if (a.split_cap >= 2) out_f32 ? gt_wgrad<true, true, 2>(s, gath, a) : gt_wgrad<false, true, 2>(s, gath, a);
        else if (tile == 4) out_f32 ? gt_wgrad<true, false, 1>(s, gath, a) : gt_wgrad<false, false, 1>(s, gath, a);
        else out_f32 ? gt_wgrad<true, false, 2>(s, gath, a) : gt_wgrad<false, false, 2>(s, gath, a);
    } else if (mode == GG_FWD) {
        if (epi == GG_EPI_SWIGLU) gath ? gt_rows<GG_FWD, GG_EPI_SWIGLU, 1>(s, tile, a) : gt_rows<GG_FWD, GG_EPI_SWIGLU, 0>(s, tile, a);
        else gath ? gt_rows<GG_FWD, GG_EPI_STORE, 1>(s, tile, a) : gt_rows<GG_FWD, GG_EPI_STORE, 0>(s, tile, a);
    } else {
        if (epi == GG_EPI_SWIGLU_BWD) gath ? gt_rows<GG_DGRAD, GG_EPI_SWIGLU_BWD, 1>(s, tile, a) : gt_rows<GG_DGRAD, GG_EPI_SWIGLU_BWD, 0>(s, tile, a);
        else gath ? gt_rows<GG_DGRAD, GG_EPI_STORE, 1>(s, tile, a) : gt_rows<GG_DGRAD, GG_EPI_STORE, 0>(s, tile, a);
    }
}

// ---- calls of a batch (see moe_batch_create) ----
template <int EPI>
static void gt_fwd_jobs(hipStream_t s, int tile, int64_t n, const gt_jobs& m) {
    const dim3 grid((unsigned)n), block(256);
    if (tile == 1) hipLaunchKernelGGL((gt_fwd_jobs_kernel<EPI, 64, 2>), grid, block, 0, s, m);
    else if (tile == 2) hipLaunchKernelGGL((gt_fwd_jobs_kernel<EPI, 128, 2>), grid, block, 0, s, m);
    else hipLaunchKernelGGL((gt_fwd_jobs_kernel<EPI, 64, 3>), grid, block, 0, s, m);
}
template <int EPI, bool F32, int WGATH>
static void gt_bwd_jobs(hipStream_t s, int tile, int wtile, int64_t n, const gt_jobs& m) {
    const dim3 grid((unsigned)n), block(256);
    bool split = false;
    for (int x = 2; x < GT_JOBS; ++x) split |= m.a[x].split_cap >= 2;
    if (split && tile == 1) hipLaunchKernelGGL((gt_bwd_jobs_kernel<EPI, 64, 2, F32, WGATH, 2, true>), grid, block, 0, s, m);
    else if (split) hipLaunchKernelGGL((gt_bwd_jobs_kernel<EPI, 64, 3, F32, WGATH, 2, true>), grid, block, 0, s, m);
    else if (wtile == 4) hipLaunchKernelGGL((gt_bwd_jobs_kernel<EPI, 64, 3, F32, WGATH, 1, false>), grid, block, 0, s, m);
    else if (tile == 1) hipLaunchKernelGGL((gt_bwd_jobs_kernel<EPI, 64, 2, F32, WGATH, 2, false>), grid, block, 0, s, m);
    else hipLaunchKernelGGL((gt_bwd_jobs_kernel<EPI, 64, 3, F32, WGATH, 2, false>), grid, block, 0, s, m);
    for (int x = 2; split && x < GT_JOBS; ++x)
        if (m.a[x].split_cap >= 2) gt_add<F32>(s, m.a[x]);
}
void gt_launch_jobs(hipStream_t s, bool fwd, int epi, bool f32, int wgath, int tile, int wtile, const gt_jobs& m) {
    const int64_t n = m.start[GT_JOBS];
    if (fwd) {
        epi == GG_EPI_SWIGLU ? gt_fwd_jobs<GG_EPI_SWIGLU>(s, tile, n, m) : gt_fwd_jobs<GG_EPI_STORE>(s, tile, n, m);
    } else if (epi == GG_EPI_SWIGLU_BWD) {
        if (wgath) f32 ? gt_bwd_jobs<GG_EPI_SWIGLU_BWD, true, 1>(s, tile, wtile, n, m) : gt_bwd_jobs<GG_EPI_SWIGLU_BWD, false, 1>(s, tile, wtile, n, m);
        else f32 ? gt_bwd_jobs<GG_EPI_SWIGLU_BWD, true, 0>(s, tile, wtile, n, m) : gt_bwd_jobs<GG_EPI_SWIGLU_BWD, false, 0>(s, tile, wtile, n, m);
    } else {
        if (wgath) f32 ? gt_bwd_jobs<GG_EPI_STORE, true, 2>(s, tile, wtile, n, m) : gt_bwd_jobs<GG_EPI_STORE, false, 2>(s, tile, wtile, n, m);
        else f32 ? gt_bwd_jobs<GG_EPI_STORE, true, 0>(s, tile, wtile, n, m) : gt_bwd_jobs<GG_EPI_STORE, false, 0>(s, tile, wtile, n, m);
    }
}
// Calls that a batch does not keep: data gradients on 128-row tiles, which fill the chip by themselves; weight gradients on one buffer of
// more than eight tiles per unit, which live off three workgroups to a unit, one more than beside a data gradient (a step, us, alone :
// together: T 112 h 5504 f 1152 E 57 k 4, 86 tiles per unit, 1433 : 1545; T 262 h 5696 f 704 E 16 k 2, 17 per unit, 422 : 435; T 2541 h
// 1088 f 384 E 54, 6 per unit, 171 : 157).
bool gt_submit(moe_ctx* ctx, hipStream_t s, int mode, int epi, bool out_f32, int gath, int tile, const gg_args& a) {
    const int64_t cu = ctx->num_cu > 0 ? ctx->num_cu : 256;
    if (ctx->batch && !(mode == GG_DGRAD && tile == 2) && !(tile == 4 && a.split_cap < 2 && gt_blocks(mode, epi, 128, a) > 8 * cu)) {
        batch_gemm(ctx, {s, mode, epi, gath, tile, JOB_BF16, out_f32, false, a});
        return true;
    }
    gt_launch(s, mode, epi, out_f32, gath, tile, a);
    return false;
}
