// Shared by the small-tile grouped-GEMM kernels (gemm_tile.hip: bf16 operands, gemm_tile8.hip: one-byte operands).
#pragma once
#include "gemm.h"

#define GT_BN 128
#define GT_BAND 8   // row tiles per band of the tile order (tiles of a band that share a column run together)
#define STG_PITCH 132  // floats per staged output row

// 16 bytes per lane, descriptor in scalar registers, lane offset in bytes; LDS side: M0 + 16 * lane
__device__ __forceinline__ void dma16_buf(i32x4_t rsrc, uint32_t off, uint32_t lds_wave, uint32_t lds_const) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(m0_value(lds_wave, lds_const)), "v"(off), "s"(rsrc) : "memory", "m0");
}
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// Tile `u` of an expert with tiles_i x tiles_j tiles: bands of GT_BAND row tiles, column by column inside a band.
__device__ __forceinline__ void gt_place(int u, int tiles_i, int tiles_j, int& ti, int& tj) {
    const int band_sz = GT_BAND * tiles_j, band = u / band_sz, in_band = u - band * band_sz;
    const int band_rows = min(GT_BAND, tiles_i - band * GT_BAND);
    ti = __builtin_amdgcn_readfirstlane(band * GT_BAND + in_band % band_rows);
    tj = __builtin_amdgcn_readfirstlane(in_band / band_rows);
}

// Output phase of a BM x 128 tile.  stage(ps, stg) puts rows (q / 32) * (BM / 2) + 32 ps + q % 32 of the tile, q = 0..63, into
// stg (fp32, pitch STG_PITCH) in tile column order; called by every thread.  e, i0, i_end, j0, tj: the tile.
// (a 256-wide tile has no room for a padded pitch beside a free stage buffer: its 16-byte slots are permuted by the row instead)
template <int BN> __device__ __forceinline__ int stg_at(int row, int col) {
    return BN == 128 ? row * STG_PITCH + col : row * 256 + (((col >> 2) ^ (row & 15)) << 2) + (col & 3);
}
template <int MODE, int EPI, bool OUT_F32, int BM, int BN = 128, typename STAGE_FN>
__device__ __forceinline__ void gt_output(const gg_args& a, float* const stg, int e, int i0, int i_end, int j0, int tj, int tiles_j,
                                          STAGE_FN&& stage) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = a.N, K = a.K, J = MODE == GG_FWD ? N : K, half_cols = EPI == GG_EPI_SWIGLU ? N >> 1 : 0;
    // ---- output: 64 rows at a time (32 of each wave half) through LDS in fp32, back as whole rows ----
    // A staged row comes back to 16 lanes of 8 consecutive columns each: a store instruction is 4 rows x 256 contiguous
    // bytes (bf16).
    const int c8 = (lane & 15) * 8;
    constexpr int CH = BN / 128, HB = BN / 2;   // column parts; SwiGLU: features per tile
    // (256-wide tiles: no fence, which would wait for the stores of the previous pass and the next tile's first stage; the small
    // tiles have nothing in flight that matters and are 1-4 % faster with it, T 256 h 128 f 256: 5.2 us against 5.8)
    auto staged = []() __attribute__((always_inline)) {
        if (BN == 128) {
            __syncthreads();
        } else {
            wait_lgkm0();
            stage_barrier();
        }
    };
#pragma unroll
    for (int ps = 0; ps < BM / 64; ++ps) {
        // staged row q (0..63) is tile row (q / 32) * (BM / 2) + 32 ps + q % 32
        auto out_row = [&](int q) { return i0 + (q >> 5) * (BM / 2) + 32 * ps + (q & 31); };
        u32x4_t zg[CH][4], zu[CH][4];
        if (EPI == GG_EPI_SWIGLU_BWD) {   // the saved pre-activations: on their way while the accumulators are staged
#pragma unroll
            for (int ch = 0; ch < CH; ++ch)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int r = out_row(wave * 16 + t * 4 + (lane >> 4)), c = j0 + 128 * ch + c8;
                    if (r < i_end && c < K) {
                        const bf16_t* z = a.Zsaved + (int64_t)r * 2 * K + c;
                        zg[ch][t] = *(const u32x4_t*)z;
                        zu[ch][t] = *(const u32x4_t*)(z + K);
                    }
                }
        }
        if (ps) staged();
        stage(ps, stg);
        staged();
        auto pack8 = [](const float* v) {
            return u32x4_t{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7])};
        };
#pragma unroll
        for (int ch = 0; ch < CH; ++ch)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int q = wave * 16 + t * 4 + (lane >> 4), r = out_row(q), cc = 128 * ch + c8, c = j0 + cc;
            const bool live = r < i_end;
            float v[8];
            *(f32x4_t*)v = *(const f32x4_t*)(stg + stg_at<BN>(q, cc));
            *(f32x4_t*)(v + 4) = *(const f32x4_t*)(stg + stg_at<BN>(q, cc + 4));
            if (EPI == GG_EPI_SWIGLU) {
                const int f = j0 + (cc & (HB - 1));
                if (a.out && live && f < half_cols)
                    *(u32x4_t*)((bf16_t*)a.out + (int64_t)r * N + (cc < HB ? f : half_cols + f)) = pack8(v);
            } else if (EPI == GG_EPI_SWIGLU_BWD) {
                float dot = 0.f;
                if (live && c < K) {
                    const float gt[8] = {bf16_lo(zg[ch][t].x), bf16_hi(zg[ch][t].x), bf16_lo(zg[ch][t].y), bf16_hi(zg[ch][t].y),
                                         bf16_lo(zg[ch][t].z), bf16_hi(zg[ch][t].z), bf16_lo(zg[ch][t].w), bf16_hi(zg[ch][t].w)};
                    const float up[8] = {bf16_lo(zu[ch][t].x), bf16_hi(zu[ch][t].x), bf16_lo(zu[ch][t].y), bf16_hi(zu[ch][t].y),
                                         bf16_lo(zu[ch][t].z), bf16_hi(zu[ch][t].z), bf16_lo(zu[ch][t].w), bf16_hi(zu[ch][t].w)};
                    const float pr = a.row_prob ? a.row_prob[r] : 1.0f;
                    float dg[8], du[8];
#pragma unroll
                    for (int x = 0; x < 8; ++x) {
                        const float sg = sigmoid_f(gt[x]);
                        dg[x] = pr * v[x] * up[x] * sg * (1.0f + gt[x] * (1.0f - sg));
                        du[x] = pr * v[x] * gt[x] * sg;
                        dot += v[x] * (gt[x] * sg * up[x]);
                    }
                    bf16_t* o = (bf16_t*)a.out + (int64_t)r * 2 * K + c;
                    *(u32x4_t*)o = pack8(dg);
                    *(u32x4_t*)(o + K) = pack8(du);
                }
                if (a.dprob_part) {   // one partial sum per row and 128-column tile; an odd tile count leaves one entry over
#pragma unroll
                    for (int x = 1; x < 16; x <<= 1) dot += __shfl_xor(dot, x);
                    if (live && (lane & 15) == 0) {
                        float* d = a.dprob_part + (int64_t)r * (2 * ((K + 255) / 256));
                        d[tj * CH + ch] = dot;
                        if (CH == 1 && tj + 1 == tiles_j && (tiles_j & 1)) d[tj + 1] = 0.f;
                    }
                }
            } else if (live && c < J) {
                const int64_t at = (MODE == GG_WGRAD ? ((int64_t)e * N + r) * K : (int64_t)r * J) + c;
                if (OUT_F32) {
                    f32x4_t* o = (f32x4_t*)((float*)a.out + at);
                    f32x4_t lo = *(f32x4_t*)v, hi = *(f32x4_t*)(v + 4);
                    if (a.accumulate) {
                        lo += o[0];
                        hi += o[1];
                    }
                    o[0] = lo;
                    o[1] = hi;
                } else {
                    u32x4_t* o = (u32x4_t*)((bf16_t*)a.out + at);
                    if (a.accumulate) {
                        const u32x4_t w = *o;
                        v[0] += bf16_lo(w.x); v[1] += bf16_hi(w.x); v[2] += bf16_lo(w.y); v[3] += bf16_hi(w.y);
                        v[4] += bf16_lo(w.z); v[5] += bf16_hi(w.z); v[6] += bf16_lo(w.w); v[7] += bf16_hi(w.w);
                    }
                    *o = pack8(v);
                }
            }
        }
        if (EPI == GG_EPI_SWIGLU) {   // activation: 8 features per lane, 8 (256-wide tile: 4) rows per instruction
#pragma unroll
            for (int t = 0; t < 2 * CH; ++t) {
                const int q = wave * 16 + t * (8 / CH) + lane / (HB / 8), r = out_row(q), f8 = (lane % (HB / 8)) * 8;
                if (r < i_end && j0 + f8 < half_cols) {
                    const float pr = a.row_prob ? a.row_prob[r] : 1.0f;
                    float act[8];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const f32x4_t gt = *(const f32x4_t*)(stg + stg_at<BN>(q, f8 + 4 * h));
                        const f32x4_t up = *(const f32x4_t*)(stg + stg_at<BN>(q, HB + f8 + 4 * h));
#pragma unroll
                        for (int x = 0; x < 4; ++x) act[4 * h + x] = pr * (gt[x] * sigmoid_f(gt[x]) * up[x]);
                    }
                    *(u32x4_t*)(a.out_act + (int64_t)r * half_cols + j0 + f8) = pack8(act);
                }
            }
        }
    }
}

__device__ __forceinline__ int gt_job_of(const gt_jobs& m, int block) {
    int j = 0;
#pragma unroll
    for (int x = 1; x < GT_JOBS; ++x) j += block >= m.start[x];
    return j;
}
