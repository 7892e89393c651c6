// Shared by the grouped-GEMM kernels of gemm.hip (256 x 256 tiles) and gemm_tile.hip (smaller tiles): arguments, LDS access
// and synchronisation primitives.
#pragma once
#include "common.h"

#define GG_MAX_E 1024
// k-major swizzle: two 128-byte rows share a 256-byte bank line; slot ^= bits 1..3 of the row makes
// 16 consecutive rows hit 16 different (position in line, slot) pairs (SQ_LDS_BANK_CONFLICT = 0)
#define KM_SWZ(row) (((row) >> 1) & 7)

enum { GG_FWD = 0, GG_DGRAD = 1, GG_WGRAD = 2 };
enum { GG_EPI_STORE = 0, GG_EPI_SWIGLU = 1, GG_EPI_SWIGLU_BWD = 2 };

typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) void gbl_void_t;
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef int i32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
typedef __attribute__((address_space(3))) i32x2_t lds_i32x2_t;

// The LDS destination is passed as a wave-uniform register part plus a constant part (buffer + chunk).
// The register part goes through an empty asm first: the sum is then formed at each use (one scalar add)
// instead of sixteen loop-invariant sums each holding a scalar register across the stage loop.
__device__ __forceinline__ uint32_t lds_addr(void* p) { return (uint32_t)(uintptr_t)(lds_void_t*)p; }
__device__ __forceinline__ uint32_t m0_value(uint32_t lds_wave, uint32_t lds_const) {
    asm volatile("" : "+s"(lds_wave));
    return lds_wave + lds_const;
}
// Workgroup barrier without the memory fence __syncthreads() carries: the fence would drain every
// DMA load in flight (vmcnt(0)) and serialise the pipeline.  The wave has already waited for its own
// loads of the stage being published; LDS reads after the barrier are ordered by the hardware.
// The empty asm statements and sched_barriers keep the compiler from moving anything across.
__device__ __forceinline__ void stage_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }  // lgkmcnt(0)
// s_waitcnt vmcnt(0) only (gfx9 encoding, other counters at their maxima): this wave's DMA loads landed
__device__ __forceinline__ void wait_vm0() { __builtin_amdgcn_s_waitcnt(0x0F70); }
// (hardware reciprocal, 1 ulp: an IEEE division is ten instructions per element in an epilogue one wave runs alone)
__device__ __forceinline__ float sigmoid_f(float g) { return __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// ds_read_b64_tr_b16: within each group of 16 lanes, lane i supplies the address of 4 consecutive
// 16-bit elements (row i/4, columns 4*(i%4)..+3 of a 4x16 block) and receives column i of that block
// (rows 0..3).  Two of them give the 8 contraction values a lane feeds to the 32x32x16 MFMA.
__device__ __forceinline__ bf16x8_t lds_read_tr16x8(const char* p_lo, const char* p_hi) {
    s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p_lo);
    s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p_hi);
    s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
}
// 4 consecutive bf16 <-> 4 floats, one 8-byte access
__device__ __forceinline__ void st4_bf16(bf16_t* p, const float* v) {
    u32x2_t w = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    *(u32x2_t*)p = w;
}
__device__ __forceinline__ void ld4_bf16(const bf16_t* p, float* v) {
    const u32x2_t w = *(const u32x2_t*)p;
    v[0] = bf16_lo(w.x);
    v[1] = bf16_hi(w.x);
    v[2] = bf16_lo(w.y);
    v[3] = bf16_hi(w.y);
}

struct gg_args {
    const void* P;         // fwd: A, dgrad: dC, wgrad: dC   (bf16, or E4M3 codes)
    const void* Q;         // fwd/dgrad: W [E,N,K], wgrad: A
    const float* p_scale;  // fp8: [rows, C/128] for the row-indexed operand (C = contraction length)
    const float* q_scale;  // fp8: [E, N/128, K/128] for the weights
    const int32_t* offsets;
    int E, N, K;
    int64_t Rcap;
    void* out;             // fwd: C (may be NULL with SWIGLU), dgrad: dA or dZ, wgrad: dW
    bf16_t* out_act;       // fwd SWIGLU: activation output
    const bf16_t* Zsaved;  // dgrad SWIGLU_BWD: saved pre-activation [rows, 2K]
    const char* zeros;     // >= 16 zero bytes (feeds the wgrad contraction tail)
    int* dev_err;
    int accumulate;        // wgrad: out += result
    const float* row_prob; // eq. (2): routing weight of each row (fwd SWIGLU: scales the activation;
                           //   dgrad SWIGLU_BWD: scales dZ); NULL = 1
    // blockwise fp8 only: the epilogue also emits the 1x128 codes and scales of its bf16 output (fwd SWIGLU: of the
    // activation [rows, N/2]; dgrad SWIGLU_BWD: of dZ [rows, 2K]), the operand of the next GEMM (Sec. 5.4.2)
    uint8_t* out_q;
    float* out_q_scale;
    // MXFP8: the same tensors as 1x32 codes + E8M0 bytes [rows, cols/32] (out_q, out_q_e8) and, optionally, as the
    // 32x1 copy for the weight gradient (out_qc, scales [rows/128, cols, 4]: one dword = the four 32-row blocks)
    uint8_t* out_q_e8;
    uint8_t* out_qc;
    uint8_t* out_qc_e8;
    int* tile_counter;     // wgrad: device counter, zero at the start, for the dynamic tile order under skewed loads (see the kernel)
    // wgrad, bf16: deterministic split of the contraction for experts far above the mean load (see the kernels)
    int split_rows;        // wgrad, small tiles: an expert of up to this many rows is not split
    int split_cap;         // how many expert-sized slices of fp32 partial results `partials` can hold (0: never split)
    float* partials;       // [split_cap] slices: 256 x 256 kernel [tiles per expert][256 x 256], small tiles [N][K]
    int* split_info;       // [1 + 3 * GG_MAX_SPLIT_EXPERTS]: count, then (expert, pieces, first slice) for the reduce kernel
    float* dprob_part;     // eq. (2), dgrad SWIGLU_BWD: [Rcap, 2 ceil(K/256)] partial <dA, act(Z)> per row, two per column tile
    // Permutation fused into the operand fetch (Sec. 4.3.3; GATH variants): the gathered operand (P or Q) points to
    // the unpermuted tensor [g_T, row length], and row r of the operand is its row g_src_of[r] / g_k, or zeros where
    // g_src_of[r] < 0 (padding, rows behind offsets[E])
    const int32_t* g_src_of;
    uint32_t g_magic;      // ceil(2^31 / g_k): ((2 s + 1) * g_magic) >> 32 == s / g_k for every 0 <= s with s * g_k < 2^30
    int g_k;
    int g_T;
};
// offset of a gathered row that has no source: behind every record count a gathered operand can have (checked on the
// host), and far enough from 2^32 that a column offset added to it cannot wrap
#define GG_NO_ROW 0xF0000000u


// Small-tile kernels for bf16 operands (gemm_tile.hip).  gt_tile: which of them serves a call (0: none, the 256 x 256
// kernel of gemm.hip is the better one); gt_launch: run it.
int gt_tile(const moe_ctx* ctx, int mode, int epi, const gg_args& a);
// Weight gradients on small tiles: whether experts are split (sets split_rows, split_cap); `slices`: room for so many fp32 results of
// an expert.
#define GT_MAX_PIECES 32
void gt_spread(const moe_ctx* ctx, gg_args& a, int64_t slices);
void gt_launch(hipStream_t s, int mode, int epi, bool out_f32, int gath, int tile, const gg_args& a);
// the same for one-byte operands (gemm_tile8.hip); `quant`: the call also asks for quantised copies of its output
int gq_tile(const moe_ctx* ctx, int mode, int epi, bool mx, bool quant, const gg_args& a);
void gq_launch(const moe_ctx* ctx, hipStream_t s, int mode, int epi, bool out_f32, bool mx, int tile, const gg_args& a);

// ---- batches (moe_batch_create; batch.hip): calls kept until the batch's end, launched together ----
// Up to four grouped GEMMs of a launch: the workgroups of call x are start[x] .. start[x + 1] - 1, multiples of 8 of them, so
// that the XCDs' shares of a call stay.  Forward calls from 0 on; or data gradients 0 and 1, weight gradients 2 and 3.
// turn: the place in that list of the grid's first workgroup, 0 or start[2] (weight gradients go first; batch.hip: longer_first).
#define GT_JOBS 4
struct gt_jobs {
    gg_args a[GT_JOBS];
    int start[GT_JOBS + 1];
    int turn;
};
__device__ __forceinline__ int gt_place_of(int block, int turn, int total) { return block + turn < total ? block + turn : block + turn - total; }
enum { JOB_BF16 = 0, JOB_FP8 = 1, JOB_MX = 2, JOB_F32 = 3 };
struct gemm_job {
    hipStream_t s;
    int mode, epi, gath, tile, kind;
    bool f32, done;
    gg_args a;
};
// a call of the tile quantisers (fp8.hip), and up to six of a launch, in the order of the calls
enum { QUANT_WEIGHTS = 0, QUANT_FP8 = 1, QUANT_FP8_GATHER = 2, QUANT_MX = 3, QUANT_MX_GATHER = 4 };
struct quant_args {
    int kind, cols, E, groups, k_shift;
    uint32_t k_magic;
    const u32x4_t* X;
    int64_t rows, blocks;
    const int32_t *rows_dev, *src_of;
    const float* pair_scale;
    u32x2_t *q_row, *q_col;
    void *s_row, *s_col;
};
#define QUANT_JOBS 6
struct quant_jobs {
    quant_args a[QUANT_JOBS];
    int start[QUANT_JOBS + 1];
};
struct quant_job {
    hipStream_t s;
    bool done;
    quant_args a;
};
#define MOE_BATCH_MAX 16
struct moe_batch {
    gemm_job gemm[MOE_BATCH_MAX];
    quant_job quant[MOE_BATCH_MAX];   // (launched behind the GEMMs: among them the quantised copies of their outputs)
    int n_gemm, n_quant;
    size_t partials;                  // bytes of the workspace that kept weight gradients leave pieces' results in
    int64_t kept_gemm, kept_quant;    // since its creation
};
void batch_flush(moe_batch* b);
void batch_gemm(moe_ctx* ctx, gemm_job j);
// gt_submit, gq_submit: launch a call, or keep it in the context's batch (true)
bool gt_submit(moe_ctx* ctx, hipStream_t s, int mode, int epi, bool out_f32, int gath, int tile, const gg_args& a);
bool gq_submit(moe_ctx* ctx, hipStream_t s, int mode, int epi, bool out_f32, bool mx, int tile, const gg_args& a);
int64_t gt_blocks(int mode, int epi, int bm, const gg_args& a);
int64_t gq_blocks(int mode, int epi, int bm, const gg_args& a);
void gt_launch_jobs(hipStream_t s, bool fwd, int epi, bool f32, int wgath, int tile, int wtile, const gt_jobs& m);
void gq_launch_jobs(hipStream_t s, bool mx, bool fwd, int epi, bool f32, int tile, const gt_jobs& m);
// after: the copies of a kept GEMM's output
void quant_submit(moe_ctx* ctx, hipStream_t s, const quant_args& a, bool after);
void quant_flush(quant_job* jobs, int n);
// fp32 calls on 64 x 64 tiles (gemm_f32.hip)
int64_t gf_blocks(int mode, int epi, const gg_args& a);
void gf_launch_jobs(hipStream_t s, bool fwd, int epi, const gt_jobs& m);
