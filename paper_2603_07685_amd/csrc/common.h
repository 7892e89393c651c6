// Internal definitions shared by the library's translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "moe_hip.h"

struct moe_ctx {
    int device;
    void* ws;          // device workspace
    size_t ws_bytes;
    int* dev_err;      // device error word (first 256 bytes of ws are reserved for it)
    int num_cu;
    struct moe_batch* batch;   // a batch (moe_batch_create): its recorded calls, and the workspace is its parent's; else NULL
    char err[512];
};

#define MOE_WS_RESERVED 256  // bytes at the head of the workspace: error word at 0, ...
#define MOE_WS_ZEROS 128     // ... and 128 bytes that stay zero for the whole life of the context

#define MOE_FAIL(ctx, code, ...)                                   \
    do {                                                           \
        if (ctx) snprintf((ctx)->err, sizeof((ctx)->err), __VA_ARGS__); \
        return (code);                                             \
    } while (0)

#define MOE_HIP_CHECK(ctx, expr)                                                        \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess) MOE_FAIL(ctx, MOE_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

#define MOE_LAUNCH_CHECK(ctx, name)                                                     \
    do {                                                                                \
        hipError_t e_ = hipGetLastError();                                              \
        if (e_ != hipSuccess) MOE_FAIL(ctx, MOE_ERR_HIP, "launch %s: %s", name, hipGetErrorString(e_)); \
    } while (0)

static inline size_t moe_dtype_size(moe_dtype dt) { return dt == MOE_F32 ? 4 : (dt == MOE_BF16 ? 2 : 1); }
static inline int64_t ceil_div64(int64_t a, int64_t b) { return (a + b - 1) / b; }

// --- device helpers --------------------------------------------------------
typedef __bf16 bf16_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// two fp32 -> packed bf16 pair, round to nearest even (hardware conversion on gfx950)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    bf16x2_t v;
    v[0] = (bf16_t)lo;
    v[1] = (bf16_t)hi;
    return __builtin_bit_cast(uint32_t, v);
}

// blockwise fp8 (Sec. 5.3.2): scale of a block from its amax, and four fp32 -> four E4M3 codes packed in a dword
// (fp32 division, clamp to +-448, hardware round-to-nearest-even conversion).  Shared by the quantiser kernels and
// the GEMM epilogues that quantise their own output, so both produce the same bits.
__device__ __forceinline__ float block_scale(float amax) { return amax > 0.0f ? amax / 448.0f : 1.0f; }
// x / scale without a division per element.  The quantisers are bound by vector arithmetic when every element pays the
// dozen instructions of a correctly rounded fp32 division, so the division is done once per block, r = 1 / scale, and
// an element costs a product and two fused multiply-adds: q0 = x r, q = fma(fma(-q0, scale, x), r, q0).  With r the
// correctly rounded reciprocal, q0 is a faithful quotient, the inner fma is the exact residual x - q0 scale, and the
// corrected q is the correctly rounded quotient (Markstein's division theorem), i.e. bit for bit what x / scale gives,
// as long as nothing under- or overflows on the way.  That holds for scales in [2^-40, 2^120] (block maxima from about
// 2^-31 up to the top of the bf16 range): r is normal; the residual of an element of magnitude 2^-77 or more is exact
// and a normal number whenever it matters (a residual below 2^-126 means q0 was already the correctly rounded
// quotient, so it would not matter even if denormals were flushed); a smaller element has a quotient below 2^-37, and
// whatever fp32 value comes out near that converts to the code 0 like the exact one (E4M3's smallest step is 2^-9).
// A wave in which any lane holds a scale outside the range takes the plain division for that piece (quant_fast_ok +
// a ballot: a uniform branch).
__device__ __forceinline__ bool quant_fast_ok(float scale) { return scale >= 0x1p-40f && scale <= 0x1p120f; }
__device__ __forceinline__ bool quant_fast_all(bool ok) { return __builtin_amdgcn_ballot_w64(!ok) == 0; }
__device__ __forceinline__ float quant_div(float x, float scale, float rcp) {
    const float q0 = x * rcp;
    // (the sign is x's: the scale is positive, and for x = -0 the sum of the two zeros would come out positive)
    return __builtin_copysignf(__builtin_fmaf(__builtin_fmaf(-q0, scale, x), rcp, q0), x);
}
__device__ __forceinline__ uint32_t cvt4_e4m3(float a, float b, float c, float d, float scale) {
    const float rcp = 1.0f / scale;
    if (quant_fast_all(quant_fast_ok(scale))) {
        a = quant_div(a, scale, rcp);
        b = quant_div(b, scale, rcp);
        c = quant_div(c, scale, rcp);
        d = quant_div(d, scale, rcp);
    } else {
        a = a / scale;
        b = b / scale;
        c = c / scale;
        d = d / scale;
    }
    a = __builtin_fminf(__builtin_fmaxf(a, -448.0f), 448.0f);
    b = __builtin_fminf(__builtin_fmaxf(b, -448.0f), 448.0f);
    c = __builtin_fminf(__builtin_fmaxf(c, -448.0f), 448.0f);
    d = __builtin_fminf(__builtin_fmaxf(d, -448.0f), 448.0f);
    int w = 0;
    w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, w, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
    return (uint32_t)w;
}

// MXFP8 (Sec. 5.3.3): the E8M0 exponent of a block from its largest magnitude, e = ceil(log2(amax / 448)) taken from
// the bits of amax (clamped to +-127, 0 for an all-zero block), and the E4M3 codes of x * 2^-e (exact scaling, RNE).
// One copy for every kernel that quantises (stand-alone quantisers and GEMM epilogues): identical bits everywhere.
__device__ __forceinline__ int mx_exponent(float amax) {
    if (!(amax > 0.0f)) return 0;
    const uint32_t b = __float_as_uint(amax);
    int e = (int)((b >> 23) & 0xFF) - 127 - 8 + ((b & 0x7FFFFFu) > 0x600000u ? 1 : 0);
    if (((b >> 23) & 0xFF) == 0) e = -127;  // subnormal maximum: far below the clamp
    return e < -127 ? -127 : (e > 127 ? 127 : e);
}
// Four bf16 values (two packed pairs) -> four E4M3 codes of x / 2^e, with the hardware's scaled conversion
// (v_cvt_scalef32_pk_fp8_bf16 divides by the power of two in the scale operand's exponent field, round to nearest
// even); one exponent for all four, or one per element (two conversions per pair, one byte kept of each).
typedef short s16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float mx_scale_f32(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }  // 2^e
__device__ __forceinline__ uint32_t mx_cvt4_bf16(uint32_t w01, uint32_t w23, float scale) {
    s16x2_t o = {0, 0};
    o = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(o, __builtin_bit_cast(bf16x2_t, w01), scale, false);
    o = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(o, __builtin_bit_cast(bf16x2_t, w23), scale, true);
    return __builtin_bit_cast(uint32_t, o);
}
__device__ __forceinline__ uint32_t mx_cvt4_bf16_each(uint32_t w01, uint32_t w23, float s0, float s1, float s2, float s3) {
    s16x2_t ev = {0, 0}, od = {0, 0};
    ev = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(ev, __builtin_bit_cast(bf16x2_t, w01), s0, false);
    ev = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(ev, __builtin_bit_cast(bf16x2_t, w23), s2, true);
    od = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(od, __builtin_bit_cast(bf16x2_t, w01), s1, false);
    od = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(od, __builtin_bit_cast(bf16x2_t, w23), s3, true);
    return (__builtin_bit_cast(uint32_t, ev) & 0x00FF00FFu) | (__builtin_bit_cast(uint32_t, od) & 0xFF00FF00u);
}
// largest magnitude of the eight bf16 values of a 16-byte piece, as fp32 (the bits of |x| order like unsigned integers)
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_absmax_bits(uint32_t m, uint32_t w) {   // both halves at once
    const u16x2_t a = __builtin_bit_cast(u16x2_t, m), b = __builtin_bit_cast(u16x2_t, w & 0x7FFF7FFFu);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, b));
}
__device__ __forceinline__ float bf16_absmax_finish(uint32_t m) {
    const uint32_t hi = m >> 16, lo = m & 0xFFFFu;
    return __uint_as_float((hi > lo ? hi : lo) << 16);
}

// Tile lookup of the one-tile-per-workgroup GEMM kernels: the whole workgroup reads the device-resident offsets (E <= 1024,
// a few per thread), checks them (inconsistent: error word, nothing is computed; decided alike by every workgroup) and
// finds its tile in the list of all experts' tiles, expert by expert: mult * ceil(rows / bm) of them each, or mult if
// bm = 0.  u = the tile's number inside its expert.  A parallel prefix sum: one pass of loads and two barriers whatever E
// is.  Workgroups land on the 8 XCDs round-robin; each XCD gets a contiguous run of the tiles that exist (the grid is an
// upper bound, rounded up to a multiple of 8), so that neighbours share their operands in its L2.  With bm = 0, lim > 0 cuts
// experts of more than lim rows into split_pieces pieces of mult tiles each.  Returns false
// (uniformly) if there is nothing to do.  Every thread of the workgroup must call it.
__device__ __forceinline__ int split_pieces(int rows, int lim) { return rows > lim ? (rows - 1) / lim + 1 : 1; }
struct tile_pick_lds {
    int wave_sum[16];
    int wave_bad[16];
    int found[4];  // expert, tile, first row, end row
};
// In two parts for a workgroup that computes several tiles: the sums over the experts once (kept in registers), then one
// look-up per tile.
template <int THREADS>
struct tile_sums {
    static constexpr int PER = 1024 / THREADS;   // experts per thread
    int o[PER + 1], cnt[PER];                    // their offsets and tile counts
    int n, first, total;                         // this thread's tiles, the first of them, all
};
template <int THREADS>
__device__ __forceinline__ bool tile_scan(const int32_t* __restrict__ offsets, int E, int64_t Rcap, int* dev_err, int bm,
                                          int mult, tile_pick_lds& l, tile_sums<THREADS>& st, bool first_block, int lim = 0) {
    constexpr int PER = tile_sums<THREADS>::PER;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto& o = st.o;
    auto& cnt = st.cnt;
#pragma unroll
    for (int x = 0; x <= PER; ++x) {
        const int i = tid * PER + x;
        o[x] = offsets[i < E ? i : E];
    }
    bool bad = (tid == 0 && o[0] < 0) || o[PER] > Rcap;
    int n = 0;
#pragma unroll
    for (int x = 0; x < PER; ++x) {
        const int rows = o[x + 1] - o[x];
        bad |= rows < 0;
        cnt[x] = mult * (bm ? (rows > 0 ? (rows + bm - 1) / bm : 0) : (tid * PER + x < E ? 1 : 0));
    }
    if (lim > 0) {   // (uniform: the divisions stay out of the calls that cut nothing)
#pragma unroll
        for (int x = 0; x < PER; ++x) cnt[x] *= split_pieces(o[x + 1] - o[x], lim);
    }
#pragma unroll
    for (int x = 0; x < PER; ++x) n += cnt[x];
    int incl = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int v = __shfl_up(incl, d);
        if (lane >= d) incl += v;
    }
    const bool any_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
    if (lane == 63) l.wave_sum[wave] = incl;
    if (lane == 0) l.wave_bad[wave] = any_bad;
    __syncthreads();
    int first = incl - n, total = 0, wrong = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        if (w < wave) first += l.wave_sum[w];
        total += l.wave_sum[w];
        wrong |= l.wave_bad[w];
    }
    if (wrong) {
        if (first_block && tid == 0) atomicExch(dev_err, 1);
        return false;
    }
    st.n = n;
    st.first = first;
    st.total = total;
    return true;
}
// `block`: the place in the launch (of a workgroup's further tiles: its own plus a multiple of 8)
template <int THREADS>
__device__ __forceinline__ bool tile_find(const tile_sums<THREADS>& st, int block, tile_pick_lds& l, int& e, int& u,
                                          int& row_lo, int& row_hi) {
    constexpr int PER = tile_sums<THREADS>::PER;
    const int run = (st.total + 7) >> 3, at_run = block >> 3;
    const int unit = (block & 7) * run + at_run;
    if (at_run >= run || unit >= st.total) return false;
    if (unit >= st.first && unit < st.first + st.n) {
        int at = unit - st.first;
#pragma unroll
        for (int x = 0; x < PER; ++x) {
            if (at >= 0 && at < st.cnt[x]) {
                l.found[0] = threadIdx.x * PER + x;
                l.found[1] = at;
                l.found[2] = st.o[x];
                l.found[3] = st.o[x + 1];
            }
            at -= st.cnt[x];
        }
    }
    __syncthreads();
    e = __builtin_amdgcn_readfirstlane(l.found[0]);
    u = __builtin_amdgcn_readfirstlane(l.found[1]);
    row_lo = __builtin_amdgcn_readfirstlane(l.found[2]);
    row_hi = __builtin_amdgcn_readfirstlane(l.found[3]);
    return true;
}
template <int THREADS>
__device__ __forceinline__ bool tile_pick(const int32_t* __restrict__ offsets, int E, int64_t Rcap, int* dev_err, int bm,
                                          int mult, int block, tile_pick_lds& l, int& e, int& u, int& row_lo, int& row_hi) {
    tile_sums<THREADS> st;
    return tile_scan(offsets, E, Rcap, dev_err, bm, mult, l, st, block == 0) && tile_find(st, block, l, e, u, row_lo, row_hi);
}

// Quantised copies of the tensor X [rows, cols] that a grouped GEMM has just stored (fp8.hip): blockwise 1x128 codes and
// scales, or MXFP8 1x32 (and, q_col not NULL, 32x1) ones, of the rows offsets[0] .. offsets[E] - 1; nothing at all where the
// GEMM refuses the offsets too (they fall, leave 0 .. rows, or, with q_col, lie off the 128-row grid).  `after`: the GEMM is kept in
// ctx's batch (only a two-copy MXFP8 call can be), and so the copies have to be.
moe_status moe_quantise_live(moe_ctx* ctx, hipStream_t s, const void* X, int64_t rows, int cols, const int32_t* offsets, int E,
                             bool mx, void* q, void* scale, void* q_col, uint8_t* e8_col, bool after);

// all-fp32 grouped GEMMs (gemm_f32.hip), reached from the public entry points with dt = MOE_F32
int moe_gg_f32_choice(int num_cu, int mode, int epi, int E, int N, int K, int64_t Rcap);   // the kernel: 64 or 128 (tile of gf_kernel), 3 (gs_kernel)
moe_status moe_gg_f32_fwd(moe_ctx* ctx, hipStream_t s, const void* A, const void* B, const int32_t* offsets, int E, int N,
                          int K, int64_t Rcap, int swiglu, const float* row_prob, void* C, void* C_act);
moe_status moe_gg_f32_dgrad(moe_ctx* ctx, hipStream_t s, const void* dC, const void* B, const int32_t* offsets, int E, int N,
                            int K, int64_t Rcap, const void* Z_saved, const float* row_prob, void* dA);
moe_status moe_gg_f32_wgrad(moe_ctx* ctx, hipStream_t s, const void* A, const void* dC, const int32_t* offsets, int E, int N,
                            int K, int64_t Rcap, int accumulate, void* dB);

// gate GEMM of small calls (gate.hip): the best of its tiles with an estimate of its time, and the launch
int moe_gate_tile(int num_cu, int T, int E, int h, double* us);
void moe_gate_launch(hipStream_t s, int tile, const void* X, const void* W, int T, int E, int h, float* out);

// message buffer (512 bytes, one per host thread) of the calls that take no context; moe_last_error(NULL) returns it
char* moe_ctxless_error();

// shared by the fill launches of several files
void moe_launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s);
