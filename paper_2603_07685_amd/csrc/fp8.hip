// Blockwise FP8 quantisation (Sec. 5.3.2): E4M3 codes + fp32 block scales, grouped over all experts
// in one launch with the live row count read from the device (Sec. 5.4.2).
//
//   scale = amax(block) / 448   (1 for an all-zero block)
//   code  = nearest E4M3 to clamp(x / scale, +-448): fp32 division, hardware round-to-nearest-even
//           conversion (v_cvt_pk_fp8_f32; gfx950 implements the OCP "fn" format: no inf, max 448)
// All three kernels are bandwidth-bound: 2 bytes read + 1 byte written per element.
//   1x128   : 16 lanes own one block (8 elements per lane), amax by butterfly over those 16 lanes.
//   128x1   : a wave owns a 128-row x 512-column panel, 8 columns per lane; first pass keeps the running
//             column amax in registers, second pass re-reads the panel (from L2) and converts.
//   128x128 : a 512-thread workgroup owns one block, 32 elements per thread held in registers.
#include "gemm.h"

// Threads per 128 x 128 tile of the two-copy quantisers and the weight quantiser, 2048 / this 16-byte pieces per lane.  At 256 a call
// of few tiles was bound by one lane's chain of eight pieces and sixteen divisions; at 1024 every lane's share of the column scales
// outweighs its pieces.  Measured (us, 256 threads with every lane dividing : 512 and one division pair per column), T 1024 h 512 f 256 E 8
// k 4: tokens and p * dY through the row map 13.8, 13.1 : 9.2, 9.3, X and dY 11.0, 10.9 : 7.2, 6.8, columns only 6.1 : 5.0, weights 6.1,
// 5.3, 5.0 : 5.1, 4.2, 4.2; T 8192 h 1024 f 512 E 8 k 2: 27.6, 15.2 : 25.1, 13.0; T 16384 h 4096 k 4 unchanged.  MXFP8 (256 : 512), T 256
// h 512 f 256 E 8 k 2 7.6, 7.9 : 6.3, 6.9; T 16384 h 7168 f 2048 E 32 k 8: weights 793, 376 : 739, 365, tokens and p * dY 740, 764 :
// 675, 715, A and dZ 208, 438 : 198, 412.
#define QUANT_THREADS 512

// Calls of a batch: up to this many tiles are kept, 16 per compute unit.  A step of 37 drawn fp8 and MXFP8 layers (T 512-14464, h 256-4096,
// half of them with a shared expert), against 1024 tiles 0.985 in time in the mean (0.897-1.003; MXFP8 T 2304 h 2560 f 128 E 26 k 1, shared
// 128, 223 : 200 us), 2048 0.996, 8192 and 32768 no difference (0.995-1.012): larger calls fill the chip long enough for their start not to
// count, and a launch holds six calls of this many tiles at most.
#define QUANT_KEEP 4096

__device__ __forceinline__ float amax8(u32x4_t v) {
    float m = fabsf(bf16_lo(v.x));
    m = fmaxf(m, fabsf(bf16_hi(v.x)));
    m = fmaxf(m, fmaxf(fabsf(bf16_lo(v.y)), fabsf(bf16_hi(v.y))));
    m = fmaxf(m, fmaxf(fabsf(bf16_lo(v.z)), fabsf(bf16_hi(v.z))));
    m = fmaxf(m, fmaxf(fabsf(bf16_lo(v.w)), fabsf(bf16_hi(v.w))));
    return m;
}

__device__ __forceinline__ u32x2_t cvt8_e4m3(u32x4_t v, float scale) {
    u32x2_t o;
    o.x = cvt4_e4m3(bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y), scale);
    o.y = cvt4_e4m3(bf16_lo(v.z), bf16_hi(v.z), bf16_lo(v.w), bf16_hi(v.w), scale);
    return o;
}

// Rows of the copies that go with a GEMM call (moe_quantise_live): rows_dev points to the last of E + 1 offsets, and whatever
// makes the GEMM refuse them (see tile_scan) has to stop its copies as well.  Decided alike by every workgroup, from E + 1
// loads in flight together; every thread must call it.
__device__ __forceinline__ bool offsets_refused(const int32_t* __restrict__ rows_dev, int E, int64_t rows, bool grid128) {
    const int32_t* const o = rows_dev - E;
    bool bad = o[0] < 0 || o[E] > rows;
    for (int i = threadIdx.x; i < E; i += blockDim.x) bad |= o[i + 1] < o[i] || (grid128 && ((o[i] | o[i + 1]) & 127) != 0);
    return __syncthreads_or(bad);
}

// ---- 1x128 ---------------------------------------------------------------------------------
// (E > 0: the copy of a GEMM's output, see offsets_refused)
__global__ __launch_bounds__(256) void quant_1x128_kernel(const u32x4_t* __restrict__ X, int64_t rows, int cols,
                                                          const int32_t* __restrict__ rows_dev, int E,
                                                          u32x2_t* __restrict__ q, float* __restrict__ scale) {
    const int64_t live = rows_dev ? min((int64_t)*rows_dev, rows) : rows;
    if (E > 0 && offsets_refused(rows_dev, E, rows, false)) return;
    const int bpr = cols / 128;                       // blocks per row
    const int64_t nblocks = live * bpr;
    const int sub = threadIdx.x & 15;                 // lane inside its 16-lane block group
    int64_t b = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
    if (E > 0) b += (int64_t)rows_dev[-E] * bpr;
    const int64_t stride = ((int64_t)gridDim.x * blockDim.x) >> 4;
    for (; b < nblocks; b += stride) {                // uniform inside a 16-lane group
        const int64_t vec = b * 16 + sub;             // 16-byte vector index (row-major, 16 per block)
        const u32x4_t v = X[vec];
        float m = amax8(v);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        const float s = block_scale(m);
        q[vec] = cvt8_e4m3(v, s);
        if (sub == 0) scale[b] = s;
    }
}

// ---- 128x1 ---------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void quant_128x1_kernel(const u32x4_t* __restrict__ X, int64_t rows, int cols,
                                                          const int32_t* __restrict__ rows_dev,
                                                          u32x2_t* __restrict__ q, float* __restrict__ scale) {
    const int64_t live = rows_dev ? min((int64_t)*rows_dev, rows) : rows;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int vpr = cols / 8;                          // 16-byte vectors per row
    const int panels_c = (vpr + 63) / 64;              // 512-column panels per row block
    const int64_t npanels = (live / 128) * panels_c;
    for (int64_t p = (int64_t)blockIdx.x * 4 + wave; p < npanels; p += (int64_t)gridDim.x * 4) {
        const int64_t rb = p / panels_c;
        const int vc = (int)(p % panels_c) * 64 + lane;
        if (vc >= vpr) continue;
        const u32x4_t* src = X + rb * 128 * vpr + vc;
        float m[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int r = 0; r < 128; ++r) {
            const u32x4_t v = src[(int64_t)r * vpr];
            m[0] = fmaxf(m[0], fabsf(bf16_lo(v.x))); m[1] = fmaxf(m[1], fabsf(bf16_hi(v.x)));
            m[2] = fmaxf(m[2], fabsf(bf16_lo(v.y))); m[3] = fmaxf(m[3], fabsf(bf16_hi(v.y)));
            m[4] = fmaxf(m[4], fabsf(bf16_lo(v.z))); m[5] = fmaxf(m[5], fabsf(bf16_hi(v.z)));
            m[6] = fmaxf(m[6], fabsf(bf16_lo(v.w))); m[7] = fmaxf(m[7], fabsf(bf16_hi(v.w)));
        }
        float s[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] = block_scale(m[i]);
        f32x4_t* sd = (f32x4_t*)(scale + rb * cols + (int64_t)vc * 8);
        sd[0] = f32x4_t{s[0], s[1], s[2], s[3]};
        sd[1] = f32x4_t{s[4], s[5], s[6], s[7]};
        u32x2_t* dst = q + rb * 128 * vpr + vc;
        float rc[8];   // (one division per column block, then a product and two fmas per element: see quant_div)
        bool fast = true;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            rc[i] = 1.0f / s[i];
            fast &= quant_fast_ok(s[i]);
        }
        fast = quant_fast_all(fast);
        for (int r = 0; r < 128; ++r) {
            const u32x4_t v = src[(int64_t)r * vpr];
            float x[8] = {bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y),
                          bf16_lo(v.z), bf16_hi(v.z), bf16_lo(v.w), bf16_hi(v.w)};
            if (fast) {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = quant_div(x[i], s[i], rc[i]);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = x[i] / s[i];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = __builtin_fminf(__builtin_fmaxf(x[i], -448.0f), 448.0f);
            int w0 = 0, w1 = 0;
            w0 = __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], w0, false);
            w0 = __builtin_amdgcn_cvt_pk_fp8_f32(x[2], x[3], w0, true);
            w1 = __builtin_amdgcn_cvt_pk_fp8_f32(x[4], x[5], w1, false);
            w1 = __builtin_amdgcn_cvt_pk_fp8_f32(x[6], x[7], w1, true);
            dst[(int64_t)r * vpr] = u32x2_t{(uint32_t)w0, (uint32_t)w1};
        }
    }
}

// ---- 128x128 -------------------------------------------------------------------------------
// grid = groups * (rows/128) * (cols/128) workgroups of QUANT_THREADS
struct quant_lds {
    union {
        float part[32];
        struct {
            float cmax[16][128];
            __attribute__((aligned(16))) float cscale[4][128];
            __attribute__((aligned(16))) float crcp[128];
            uint8_t sc[4][128];
        };
    };
};
__device__ __forceinline__ void quant_128x128_body(const quant_args& a, quant_lds& lds, int block) {
    const u32x4_t* const __restrict__ W = a.X;
    u32x2_t* const __restrict__ q = a.q_row;
    float* const __restrict__ scale = (float*)a.s_row;
    float* const part = lds.part;
    const int rows = (int)a.rows, cols = a.cols;
    constexpr int PIECES = 2048 / QUANT_THREADS, NW = 32 / PIECES, RP = 128 / PIECES;   // per lane; waves; rows of a pass
    const int nbr = rows / 128, nbc = cols / 128;
    const int b = block;
    const int g = b / (nbr * nbc), rb = (b / nbc) % nbr, cb = b % nbc;
    const int vpr = cols / 8;
    const int tr = threadIdx.x >> 4, tc = threadIdx.x & 15;   // RP rows x 16 vectors per pass
    const int64_t base = ((int64_t)g * rows + rb * 128) * vpr + cb * 16 + tc;
    u32x4_t v[PIECES];
    float m = 0.f;
#pragma unroll
    for (int it = 0; it < PIECES; ++it) {
        v[it] = W[base + (int64_t)(it * RP + tr) * vpr];
        m = fmaxf(m, amax8(v[it]));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    m = part[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, part[w]);
    const float s = block_scale(m);
    if (threadIdx.x == 0) scale[b] = s;
#pragma unroll
    for (int it = 0; it < PIECES; ++it) q[base + (int64_t)(it * RP + tr) * vpr] = cvt8_e4m3(v[it], s);
}
__global__ __launch_bounds__(QUANT_THREADS) void quant_128x128_kernel(const quant_args a) {
    __shared__ quant_lds lds;
    quant_128x128_body(a, lds, (int)blockIdx.x);
}

// floor(s / k) for a map entry 0 <= s < 2^31 as one widening multiplication (division by an invariant integer,
// rounded-up constant): with l = ceil(log2 k) and m = ceil(2^(31 + l) / k) <= 2^32 - 1, (s * m) >> (31 + l) == s / k
// for every such s, and the product stays below 2^63.
struct gather_div_t { uint32_t m; int sh; };
static inline gather_div_t gather_div(int k) {
    int l = 0;
    while ((1 << l) < k) ++l;
    return gather_div_t{(uint32_t)(((1ull << (31 + l)) + (uint64_t)k - 1) / (uint64_t)k), 31 + l};
}
static quant_args quant_make(int kind, const void* X, int64_t rows, int cols, const int32_t* rows_dev, void* q_row, void* s_row,
                             void* q_col, void* s_col, int64_t blocks) {
    quant_args a;
    memset(&a, 0, sizeof(a));
    a.kind = kind;
    a.X = (const u32x4_t*)X;
    a.rows = rows;
    a.cols = cols;
    a.rows_dev = rows_dev;
    a.q_row = (u32x2_t*)q_row;
    a.s_row = s_row;
    a.q_col = (u32x2_t*)q_col;
    a.s_col = s_col;
    a.groups = 1;
    a.blocks = blocks;
    return a;
}
static void quant_gather(quant_args& a, const int32_t* src_of, int k, const float* pair_scale, int groups) {
    a.src_of = src_of;
    a.k_magic = gather_div(k).m;
    a.k_shift = gather_div(k).sh;
    a.pair_scale = pair_scale;
    a.groups = groups;
}

static moe_status fp8_rowcol_launch(moe_ctx* ctx, hipStream_t s, const char* who, const void* X, int64_t rows, int cols,
                                    const int32_t* rows_dev, void* q_row, float* s_row, void* q_col, float* s_col,
                                    const int32_t* src_of, int k, const float* pair_scale, int groups);

extern "C" moe_status moe_fp8_quantize(moe_ctx* ctx, void* stream, const void* X, moe_qblock block,
                                       int groups, int64_t rows, int cols, const int32_t* rows_dev,
                                       void* q, float* scale) {
    if (!ctx) return MOE_ERR_ARG;
    if (!X || !q || !scale) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize: NULL pointer");
    if (rows < 0 || cols < 1 || groups < 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize: bad sizes");
    if (cols % 8) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize: cols must be a multiple of 8");
    hipStream_t s = (hipStream_t)stream;
    const int cu = ctx->num_cu > 0 ? ctx->num_cu : 256;
    if (rows == 0) return MOE_OK;
    switch (block) {
        case MOE_Q_1x128: {
            if (cols % 128) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize(1x128): cols %% 128 != 0");
            if (groups != 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize(1x128): groups must be 1");
            const int64_t nb = rows * (cols / 128);
            int64_t grid = ceil_div64(nb * 16, 256);
            if (grid > (int64_t)cu * 32) grid = (int64_t)cu * 32;
            hipLaunchKernelGGL(quant_1x128_kernel, dim3((unsigned)grid), dim3(256), 0, s, (const u32x4_t*)X, rows, cols,
                               rows_dev, 0, (u32x2_t*)q, scale);
            break;
        }
        case MOE_Q_128x1: {
            if (rows % 128) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize(128x1): rows %% 128 != 0");
            if (groups != 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize(128x1): groups must be 1");
            if (cols % 128 == 0) {  // the tiled kernel below: the same bits at about twice the rate
                moe_status st = fp8_rowcol_launch(ctx, s, "moe_fp8_quantize(128x1)", X, rows, cols, rows_dev, nullptr, nullptr, q, scale,
                                                  nullptr, 1, nullptr, 1);
                if (st != MOE_OK) return st;
                break;
            }
            const int64_t npanels = (rows / 128) * ceil_div64(cols / 8, 64);
            int64_t grid = ceil_div64(npanels, 4);
            if (grid > (int64_t)cu * 16) grid = (int64_t)cu * 16;
            hipLaunchKernelGGL(quant_128x1_kernel, dim3((unsigned)grid), dim3(256), 0, s, (const u32x4_t*)X, rows, cols,
                               rows_dev, (u32x2_t*)q, scale);
            break;
        }
        case MOE_Q_128x128: {
            if (rows % 128 || cols % 128) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize(128x128): rows, cols %% 128 != 0");
            if (rows_dev) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize(128x128): rows_dev is not used for weights");
            const int64_t nb = (int64_t)groups * (rows / 128) * (cols / 128);
            if (nb > 0x7fffffffLL) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize(128x128): too many blocks");
            quant_args a = quant_make(QUANT_WEIGHTS, X, rows, cols, nullptr, q, scale, nullptr, nullptr, nb);
            quant_submit(ctx, s, a, false);
            break;
        }
        default:
            MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize: bad block kind");
    }
    MOE_LAUNCH_CHECK(ctx, "moe_fp8_quantize");
    return MOE_OK;
}

// ---------------------------------------------------------------------------
// Blockwise recipe, row- and column-wise copies in one pass (Sec. 5.3.3: a tensor that two GEMMs read with different
// contraction dimensions is quantised once per direction; Sec. 5.4.2: one grouped launch; Sec. 5.4.1: padding and
// the permutation fused in).  A 512-thread workgroup owns a tile of 128 rows x 128 columns: exactly one 1x128 block
// of each of its rows and one 128x1 block of each of its columns.  Wave w owns rows 16 w .. 16 w + 15; a lane reads
// four 16-byte pieces: piece i is row 16 w + 4 i + lane / 16, columns 8 (lane % 16) .. + 7.
//   row-wise : the block is the 16 lanes of one piece (four butterfly steps);
//   col-wise : the block is the same element of the lane's 4 pieces, of the 4 lanes 16 apart and of the 8 waves
//              (maxima meet in LDS, where one thread per column forms the scale).
// Either copy may be switched off (q_row or q_col NULL).  GATHER: row r of the input is pair_scale[s] * X[s / k, :]
// rounded to bf16 (no scale, no rounding when pair_scale is NULL) with s = src_of[r], zero where s < 0.
// Scales and codes are formed exactly as in the single-direction kernels above (amax / 448, fp32 division,
// hardware conversion), so both copies are bit-identical to theirs.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t scale2_bf16_bw(uint32_t w, float sc) { return pack_bf16(sc * bf16_lo(w), sc * bf16_hi(w)); }

template <bool GATHER>
__device__ __forceinline__ void fp8_rowcol_body(const quant_args& a, quant_lds& lds, int block) {
    const u32x4_t* const __restrict__ X = a.X;
    const int64_t rows = a.rows;
    const int cols = a.cols, groups = a.groups, k_shift = a.k_shift;
    const uint32_t k_magic = a.k_magic;
    const int32_t *const __restrict__ rows_dev = a.rows_dev, *const __restrict__ src_of = a.src_of;
    const float* const __restrict__ pair_scale = a.pair_scale;
    u32x2_t *const __restrict__ q_row = a.q_row, *const __restrict__ q_col = a.q_col;
    float *const __restrict__ s_row = (float*)a.s_row, *const __restrict__ s_col = (float*)a.s_col;
    auto& cmax = lds.cmax;
    float *const cscale = lds.cscale[0], *const crcp = lds.crcp;
    constexpr int PIECES = 2048 / QUANT_THREADS, NW = 32 / PIECES, RW = 4 * PIECES;   // per lane; waves; rows of a wave
    const int64_t live = rows_dev ? min((int64_t)*rows_dev, rows) : rows;
    const int ctiles = cols / 128;
    int64_t rt = block / ctiles;
    const int ct = block % ctiles;
    if (GATHER && groups > 1) {  // row tiles expert-interleaved: the k copies of a token are read close together in time
        const int64_t S = (rows / 128 + groups - 1) / groups;
        rt = (rt % groups) * S + rt / groups;
    }
    const int64_t row0 = rt * 128;
    if (row0 >= live || row0 >= rows) return;  // uniform over the workgroup
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int vpr = cols / 8;
    const int64_t v0 = (row0 + wave * RW + (lane >> 4)) * vpr + ct * 16 + (lane & 15);
    u32x4_t x[PIECES];
    if (GATHER) {
        // Three passes, so that the map entries, then the rows, then the weights of a lane are each in
        // flight together (one pass per piece would chain the memory latencies), and no branch: a lane
        // whose row is padding reads 16 aligned bytes of this tile's 512 bytes of map entries instead, which always
        // exist, and drops them.
        const void* const spare = (const void*)(((uintptr_t)(src_of + row0) + 15) & ~(uintptr_t)15);
        int32_t sidx[PIECES];
#pragma unroll
        for (int i = 0; i < PIECES; ++i) sidx[i] = src_of[row0 + wave * RW + 4 * i + (lane >> 4)];
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int64_t tok = (int64_t)(((uint64_t)(uint32_t)sidx[i] * k_magic) >> k_shift);  // sidx / k (gather_div)
            uint64_t live_at = (uint64_t)(X + (tok * vpr + ct * 16 + (lane & 15)));
            asm volatile("" : "+v"(live_at));  // (formed for every lane: a select then, not a branch around the multiplications)
            x[i] = *(const u32x4_t*)(sidx[i] >= 0 ? live_at : (uint64_t)spare);
        }
        if (pair_scale) {
            float psc[PIECES];
#pragma unroll
            for (int i = 0; i < PIECES; ++i) psc[i] = *(sidx[i] >= 0 ? pair_scale + sidx[i] : (const float*)spare);
#pragma unroll
            for (int i = 0; i < PIECES; ++i)
                x[i] = u32x4_t{scale2_bf16_bw(x[i].x, psc[i]), scale2_bf16_bw(x[i].y, psc[i]), scale2_bf16_bw(x[i].z, psc[i]),
                               scale2_bf16_bw(x[i].w, psc[i])};
        }
#pragma unroll
        for (int i = 0; i < PIECES; ++i)
            if (sidx[i] < 0) x[i] = u32x4_t{0, 0, 0, 0};
    } else {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) x[i] = X[v0 + (int64_t)i * 4 * vpr];
    }
    if (q_col) {  // (first: the other waves' maxima are on their way while this wave converts its rows)
        float m[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) m[c] = 0.f;
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            m[0] = fmaxf(m[0], fabsf(bf16_lo(x[i].x))); m[1] = fmaxf(m[1], fabsf(bf16_hi(x[i].x)));
            m[2] = fmaxf(m[2], fabsf(bf16_lo(x[i].y))); m[3] = fmaxf(m[3], fabsf(bf16_hi(x[i].y)));
            m[4] = fmaxf(m[4], fabsf(bf16_lo(x[i].z))); m[5] = fmaxf(m[5], fabsf(bf16_hi(x[i].z)));
            m[6] = fmaxf(m[6], fabsf(bf16_lo(x[i].w))); m[7] = fmaxf(m[7], fabsf(bf16_hi(x[i].w)));
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            m[c] = fmaxf(m[c], __shfl_xor(m[c], 16));
            m[c] = fmaxf(m[c], __shfl_xor(m[c], 32));
            if (lane < 16) cmax[wave][8 * lane + c] = m[c];
        }
    }
    if (q_row) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            float m = amax8(x[i]);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
            const float sc = block_scale(m);
            q_row[v0 + (int64_t)i * 4 * vpr] = cvt8_e4m3(x[i], sc);
            if ((lane & 15) == 0) s_row[(row0 + wave * RW + 4 * i + (lane >> 4)) * ctiles + ct] = sc;
        }
    }
    if (q_col) {
        // (a column's two divisions by one thread, not by every lane that has a piece of it)
        __syncthreads();
        if (threadIdx.x < 128) {
            const int c = threadIdx.x;
            float m = cmax[0][c];
#pragma unroll
            for (int w = 1; w < NW; ++w) m = fmaxf(m, cmax[w][c]);
            const float one = block_scale(m);
            s_col[rt * cols + ct * 128 + c] = one;
            cscale[c] = one;
            crcp[c] = 1.0f / one;
        }
        __syncthreads();
        float sc[8], rc[8];
        bool fast = true;
        const int cb = 8 * (lane & 15);
        *(f32x4_t*)sc = *(const f32x4_t*)(cscale + cb);
        *(f32x4_t*)(sc + 4) = *(const f32x4_t*)(cscale + cb + 4);
        *(f32x4_t*)rc = *(const f32x4_t*)(crcp + cb);
        *(f32x4_t*)(rc + 4) = *(const f32x4_t*)(crcp + cb + 4);
#pragma unroll
        for (int c = 0; c < 8; ++c) fast &= quant_fast_ok(sc[c]);
        fast = quant_fast_all(fast);   // (see quant_div: one division per column block instead of one per element)
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            float v[8] = {bf16_lo(x[i].x), bf16_hi(x[i].x), bf16_lo(x[i].y), bf16_hi(x[i].y),
                          bf16_lo(x[i].z), bf16_hi(x[i].z), bf16_lo(x[i].w), bf16_hi(x[i].w)};
            if (fast) {
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] = quant_div(v[c], sc[c], rc[c]);
            } else {
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] = v[c] / sc[c];
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = __builtin_fminf(__builtin_fmaxf(v[c], -448.0f), 448.0f);
            int w0 = 0, w1 = 0;
            w0 = __builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], w0, false);
            w0 = __builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], w0, true);
            w1 = __builtin_amdgcn_cvt_pk_fp8_f32(v[4], v[5], w1, false);
            w1 = __builtin_amdgcn_cvt_pk_fp8_f32(v[6], v[7], w1, true);
            q_col[v0 + (int64_t)i * 4 * vpr] = u32x2_t{(uint32_t)w0, (uint32_t)w1};
        }
    }
}
template <bool GATHER>
__global__ __launch_bounds__(QUANT_THREADS) void fp8_quant_rowcol_kernel(const quant_args a) {
    __shared__ quant_lds lds;
    fp8_rowcol_body<GATHER>(a, lds, (int)blockIdx.x);
}

static moe_status fp8_rowcol_launch(moe_ctx* ctx, hipStream_t s, const char* who, const void* X, int64_t rows, int cols,
                                    const int32_t* rows_dev, void* q_row, float* s_row, void* q_col, float* s_col,
                                    const int32_t* src_of, int k, const float* pair_scale, int groups) {
    if (rows % 128 || cols % 128) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: rows and cols must be multiples of 128", who);
    if ((q_row == nullptr) != (s_row == nullptr) || (q_col == nullptr) != (s_col == nullptr) || (!q_row && !q_col))
        MOE_FAIL(ctx, MOE_ERR_ARG, "%s: codes and scales of a copy go together, and at least one copy is needed", who);
    if (groups < 1) groups = 1;
    const int64_t tiles_r = src_of ? (rows / 128 + groups - 1) / groups * groups : rows / 128;
    const int64_t nblk = tiles_r * (cols / 128);
    if (nblk > 0x7fffffffLL) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: too many tiles", who);
    quant_args a = quant_make(src_of ? QUANT_FP8_GATHER : QUANT_FP8, X, rows, cols, rows_dev, q_row, s_row, q_col, s_col, nblk);
    if (src_of) quant_gather(a, src_of, k, pair_scale, groups);
    quant_submit(ctx, s, a, false);
    return MOE_OK;
}

extern "C" moe_status moe_fp8_quantize_rowcol(moe_ctx* ctx, void* stream, const void* X, int64_t rows, int cols,
                                              const int32_t* rows_dev, void* q_row, float* scale_row,
                                              void* q_col, float* scale_col) {
    if (!ctx) return MOE_ERR_ARG;
    if (!X) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize_rowcol: NULL pointer");
    if (rows < 0 || cols < 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize_rowcol: bad sizes");
    if (rows == 0) return MOE_OK;
    moe_status st = fp8_rowcol_launch(ctx, (hipStream_t)stream, "moe_fp8_quantize_rowcol", X, rows, cols, rows_dev, q_row,
                                      scale_row, q_col, scale_col, nullptr, 1, nullptr, 1);
    if (st != MOE_OK) return st;
    MOE_LAUNCH_CHECK(ctx, "moe_fp8_quantize_rowcol");
    return MOE_OK;
}

extern "C" moe_status moe_fp8_quantize_rowcol_gather(moe_ctx* ctx, void* stream, const void* X, const int32_t* src_of, int k,
                                                     const float* pair_scale, int groups, int64_t rows, int cols,
                                                     const int32_t* rows_dev, void* q_row, float* scale_row,
                                                     void* q_col, float* scale_col) {
    if (!ctx) return MOE_ERR_ARG;
    if (!X || !src_of) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize_rowcol_gather: NULL pointer");
    if (rows < 0 || cols < 1 || k < 1 || k > 32 || groups < 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_fp8_quantize_rowcol_gather: bad sizes");
    if (rows == 0) return MOE_OK;
    moe_status st = fp8_rowcol_launch(ctx, (hipStream_t)stream, "moe_fp8_quantize_rowcol_gather", X, rows, cols, rows_dev,
                                      q_row, scale_row, q_col, scale_col, src_of, k, pair_scale, groups);
    if (st != MOE_OK) return st;
    MOE_LAUNCH_CHECK(ctx, "moe_fp8_quantize_rowcol_gather");
    return MOE_OK;
}

// ---------------------------------------------------------------------------
// MXFP8 (Sec. 5.3.3): E4M3 elements in 1x32 blocks with E8M0 (power-of-two) scales.
//   e = ceil(log2(amax / 448)) from the bits of amax = 1.f * 2^(E-127): e = E - 127 - 8 (+1 if 1.f > 1.75),
//   clamped to +-127; an all-zero block gets e = 0.  code = nearest E4M3 to x * 2^-e (exact scaling).
//   1x32 : 4 lanes own one block (8 elements each); a wave reads 1 KB and writes 512 B contiguous.
//   32x1 : blocks of 32 consecutive rows of a column, for a tensor read with its row index as the contraction
//          (weights in the data gradient, both operands of the weight gradient); made alone or together with
//          the 1x32 copy in one pass over the input (mx_quant_rowcol_kernel).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mx_quant_1x32_kernel(const u32x4_t* __restrict__ X, int64_t rows, int cols,
                                                            const int32_t* __restrict__ rows_dev, int E,
                                                            u32x2_t* __restrict__ q, uint8_t* __restrict__ e8) {
    const int64_t live = rows_dev ? min((int64_t)*rows_dev, rows) : rows;
    if (E > 0 && offsets_refused(rows_dev, E, rows, false)) return;
    const int64_t nvec = live * (cols / 8);            // 16-byte vectors; 4 per block, blocks never straddle rows
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (E > 0) v += (int64_t)rows_dev[-E] * (cols / 8);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; v < ((nvec + 3) & ~(int64_t)3); v += stride) {  // whole 4-lane groups stay together
        const bool in = v < nvec;
        const u32x4_t x = in ? X[v] : u32x4_t{0, 0, 0, 0};
        float m = amax8(x);
        m = fmaxf(m, __shfl_xor(m, 1));
        m = fmaxf(m, __shfl_xor(m, 2));
        const int e = mx_exponent(m);
        if (in) {
            u32x2_t o;
            o.x = mx_cvt4_bf16(x.x, x.y, mx_scale_f32(e));
            o.y = mx_cvt4_bf16(x.z, x.w, mx_scale_f32(e));
            q[v] = o;
            if ((v & 3) == 0) e8[v >> 2] = (uint8_t)(e + 127);
        }
    }
}

// Row- and column-wise copies in one pass (either may be switched off).  A 512-thread workgroup owns a tile of
// 128 rows x 128 columns; wave w owns its rows 16 w .. 16 w + 15, i.e. half a 32-row block of every column.  A lane
// reads four 16-byte pieces: piece i is row 4 i + lane / 16, columns 8 (lane % 16) .. + 7.
//   row-wise  : a 1x32 block is 4 adjacent lanes of one piece (two butterfly steps);
//   col-wise  : a 32x1 block is the same element of the lane's 4 pieces, of the 4 lanes 16 apart and of two waves (maxima meet
//               in LDS, where one thread per block forms the exponent).
// The column scales of a tile leave as one dword per column:
// e8_col[(row / 128) * cols + col] holds the four 32-row blocks of rows 128 (row / 128) .. + 127, the unit in
// which the GEMMs walk a contraction over rows.
// GATHER: the input is not stored in row order: row r of it is pair_scale[s] * X[s / k, :] rounded to bf16
// (no scale, no rounding when pair_scale is NULL) with s = src_of[r], and zero where s < 0 -- the permuted
// tokens (Sec. 4.3.3) or the combine's backward, quantised without ever being written out in bf16.
__device__ __forceinline__ uint32_t scale2_bf16(uint32_t w, float sc) { return pack_bf16(sc * bf16_lo(w), sc * bf16_hi(w)); }

template <bool GATHER>
__device__ __forceinline__ void mx_rowcol_body(const quant_args& a, quant_lds& lds, int block) {
    const u32x4_t* const __restrict__ X = a.X;
    const int64_t rows = a.rows;
    const int cols = a.cols, groups = a.groups, k_shift = a.k_shift, E = a.E;
    const uint32_t k_magic = a.k_magic;
    const int32_t *const __restrict__ rows_dev = a.rows_dev, *const __restrict__ src_of = a.src_of;
    const float* const __restrict__ pair_scale = a.pair_scale;
    u32x2_t *const __restrict__ q_row = a.q_row, *const __restrict__ q_col = a.q_col;
    uint32_t *const __restrict__ e8_row = (uint32_t*)a.s_row, *const __restrict__ e8_col = (uint32_t*)a.s_col;
    auto& cmax = lds.cmax;
    auto& cscale = lds.cscale;
    auto& sc = lds.sc;
    constexpr int PIECES = 2048 / QUANT_THREADS, RW = 4 * PIECES;   // per lane; rows of a wave
    static_assert(QUANT_THREADS == 512, "a thread per column and 32-row block");
    const int64_t live = rows_dev ? min((int64_t)*rows_dev, rows) : rows;
    const int ctiles = cols / 128;
    int64_t rt = block / ctiles;
    const int ct = block % ctiles;
    if (GATHER && groups > 1) {
        // Visit the row tiles expert-interleaved: with `groups` experts of roughly equal extent, consecutive
        // workgroups take the same relative position in different experts, which (stable order inside an expert)
        // is roughly the same window of source tokens, so the k copies of a token are read while it is cached.
        // Only the order changes: rt -> (rt % groups) * S + rt / groups is one-to-one onto [0, groups * S).
        const int64_t S = (rows / 128 + groups - 1) / groups;
        rt = (rt % groups) * S + rt / groups;
    }
    const int64_t row0 = rt * 128;
    if (row0 >= live || row0 >= rows) return;  // uniform over the workgroup
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int vpr = cols / 8;                                       // 16-byte pieces per row
    const int64_t v0 = (row0 + wave * RW + (lane >> 4)) * vpr + ct * 16 + (lane & 15);
    u32x4_t x[PIECES];
    if (GATHER) {
        // Three passes, so that the map entries, then the rows, then the weights of a lane are each in
        // flight together (one pass per piece would chain the memory latencies), and no branch: a lane
        // whose row is padding reads 16 aligned bytes of this tile's 512 bytes of map entries instead, which always
        // exist, and drops them.
        const void* const spare = (const void*)(((uintptr_t)(src_of + row0) + 15) & ~(uintptr_t)15);
        int32_t sidx[PIECES];
#pragma unroll
        for (int i = 0; i < PIECES; ++i) sidx[i] = src_of[row0 + wave * RW + 4 * i + (lane >> 4)];
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int64_t tok = (int64_t)(((uint64_t)(uint32_t)sidx[i] * k_magic) >> k_shift);  // sidx / k (gather_div)
            uint64_t live_at = (uint64_t)(X + (tok * vpr + ct * 16 + (lane & 15)));
            asm volatile("" : "+v"(live_at));  // (formed for every lane: a select then, not a branch around the multiplications)
            x[i] = *(const u32x4_t*)(sidx[i] >= 0 ? live_at : (uint64_t)spare);
        }
        if (pair_scale) {
            float psc[PIECES];
#pragma unroll
            for (int i = 0; i < PIECES; ++i) psc[i] = *(sidx[i] >= 0 ? pair_scale + sidx[i] : (const float*)spare);
#pragma unroll
            for (int i = 0; i < PIECES; ++i)
                x[i] = u32x4_t{scale2_bf16(x[i].x, psc[i]), scale2_bf16(x[i].y, psc[i]), scale2_bf16(x[i].z, psc[i]),
                               scale2_bf16(x[i].w, psc[i])};
        }
#pragma unroll
        for (int i = 0; i < PIECES; ++i)
            if (sidx[i] < 0) x[i] = u32x4_t{0, 0, 0, 0};
    } else {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) x[i] = X[v0 + (int64_t)i * 4 * vpr];
        if (E > 0 && (offsets_refused(rows_dev, E, rows, true) || row0 < rows_dev[-E])) return;  // (the rows are on their way meanwhile)
    }
    if (q_col) {
        float m[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) m[c] = 0.f;
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            m[0] = fmaxf(m[0], fabsf(bf16_lo(x[i].x))); m[1] = fmaxf(m[1], fabsf(bf16_hi(x[i].x)));
            m[2] = fmaxf(m[2], fabsf(bf16_lo(x[i].y))); m[3] = fmaxf(m[3], fabsf(bf16_hi(x[i].y)));
            m[4] = fmaxf(m[4], fabsf(bf16_lo(x[i].z))); m[5] = fmaxf(m[5], fabsf(bf16_hi(x[i].z)));
            m[6] = fmaxf(m[6], fabsf(bf16_lo(x[i].w))); m[7] = fmaxf(m[7], fabsf(bf16_hi(x[i].w)));
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            m[c] = fmaxf(m[c], __shfl_xor(m[c], 16));
            m[c] = fmaxf(m[c], __shfl_xor(m[c], 32));
            if (lane < 16) cmax[wave][8 * lane + c] = m[c];
        }
    }
    if (q_row) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            float m = amax8(x[i]);
            m = fmaxf(m, __shfl_xor(m, 1));
            m = fmaxf(m, __shfl_xor(m, 2));
            const int e = mx_exponent(m);
            u32x2_t o;
            o.x = mx_cvt4_bf16(x[i].x, x[i].y, mx_scale_f32(e));
            o.y = mx_cvt4_bf16(x[i].z, x[i].w, mx_scale_f32(e));
            q_row[v0 + (int64_t)i * 4 * vpr] = o;
            // the row's four block bytes of this tile, gathered into the first of its 16 lanes
            const int b = e + 127, base = lane & 48;
            const uint32_t w = (uint32_t)__shfl(b, base) | ((uint32_t)__shfl(b, base + 4) << 8) |
                               ((uint32_t)__shfl(b, base + 8) << 16) | ((uint32_t)__shfl(b, base + 12) << 24);
            if ((lane & 15) == 0) e8_row[((row0 + wave * RW + 4 * i + (lane >> 4)) * (cols / 32) + ct * 4) >> 2] = w;
        }
    }
    if (q_col) {
        __syncthreads();
        {   // (a 32-row block is two waves' rows; its exponent is formed by one thread)
            const int blk = threadIdx.x >> 7, c = threadIdx.x & 127;
            const int e = mx_exponent(fmaxf(cmax[2 * blk][c], cmax[2 * blk + 1][c]));
            sc[blk][c] = (uint8_t)(e + 127);
            cscale[blk][c] = mx_scale_f32(e);
        }
        __syncthreads();
        float sf[8];
        *(f32x4_t*)sf = *(const f32x4_t*)(cscale[wave >> 1] + 8 * (lane & 15));
        *(f32x4_t*)(sf + 4) = *(const f32x4_t*)(cscale[wave >> 1] + 8 * (lane & 15) + 4);
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const u32x2_t o = {mx_cvt4_bf16_each(x[i].x, x[i].y, sf[0], sf[1], sf[2], sf[3]),
                               mx_cvt4_bf16_each(x[i].z, x[i].w, sf[4], sf[5], sf[6], sf[7])};
            q_col[v0 + (int64_t)i * 4 * vpr] = o;
        }
        if (threadIdx.x < 128) {
            const int c = threadIdx.x;
            e8_col[rt * cols + ct * 128 + c] = (uint32_t)sc[0][c] | ((uint32_t)sc[1][c] << 8) | ((uint32_t)sc[2][c] << 16) |
                                               ((uint32_t)sc[3][c] << 24);
        }
    }
}
template <bool GATHER>
__global__ __launch_bounds__(QUANT_THREADS) void mx_quant_rowcol_kernel(const quant_args a) {
    __shared__ quant_lds lds;
    mx_rowcol_body<GATHER>(a, lds, (int)blockIdx.x);
}

// Independent calls of one recipe in one launch (a batch's), in the order of the calls
template <bool MX>
__global__ __launch_bounds__(QUANT_THREADS) void quant_jobs_kernel(const quant_jobs m) {
    __shared__ quant_lds lds;
    int j = 0;
#pragma unroll
    for (int x = 1; x < QUANT_JOBS; ++x) j += (int)blockIdx.x >= m.start[x];
    const quant_args& a = m.a[j];
    const int block = (int)blockIdx.x - m.start[j];
    if constexpr (MX) {
        if (a.kind == QUANT_MX_GATHER) mx_rowcol_body<true>(a, lds, block);
        else mx_rowcol_body<false>(a, lds, block);
    } else {
        if (a.kind == QUANT_FP8_GATHER) fp8_rowcol_body<true>(a, lds, block);
        else if (a.kind == QUANT_FP8) fp8_rowcol_body<false>(a, lds, block);
        else quant_128x128_body(a, lds, block);
    }
}

static void quant_launch(hipStream_t s, const quant_args& a) {
    const dim3 grid((unsigned)a.blocks), block(QUANT_THREADS);
    switch (a.kind) {
        case QUANT_WEIGHTS: hipLaunchKernelGGL(quant_128x128_kernel, grid, block, 0, s, a); break;
        case QUANT_FP8: hipLaunchKernelGGL(fp8_quant_rowcol_kernel<false>, grid, block, 0, s, a); break;
        case QUANT_FP8_GATHER: hipLaunchKernelGGL(fp8_quant_rowcol_kernel<true>, grid, block, 0, s, a); break;
        case QUANT_MX: hipLaunchKernelGGL(mx_quant_rowcol_kernel<false>, grid, block, 0, s, a); break;
        default: hipLaunchKernelGGL(mx_quant_rowcol_kernel<true>, grid, block, 0, s, a); break;
    }
}
void quant_submit(moe_ctx* ctx, hipStream_t s, const quant_args& a, bool after) {
    moe_batch* const b = ctx->batch;
    if (!b || (!after && a.blocks > QUANT_KEEP)) return quant_launch(s, a);
    if (b->n_quant == MOE_BATCH_MAX) batch_flush(b);
    b->quant[b->n_quant++] = {s, false, a};
    ++b->kept_quant;
}
void quant_flush(quant_job* jobs, int n) {
    for (int i = 0; i < n; ++i) {
        if (jobs[i].done) continue;
        quant_jobs m;
        memset(&m, 0, sizeof(m));
        const bool mx = jobs[i].a.kind >= QUANT_MX;
        int count = 0;
        int64_t at = 0;
        for (int x = i; x < n && count < QUANT_JOBS; ++x) {
            quant_job& j = jobs[x];
            if (j.done || j.s != jobs[i].s || (j.a.kind >= QUANT_MX) != mx || (count && at + j.a.blocks > QUANT_JOBS * QUANT_KEEP)) continue;
            m.a[count] = j.a;
            m.start[count++] = (int)at;
            at += j.a.blocks;
            j.done = true;
        }
        if (count == 1) {
            quant_launch(jobs[i].s, m.a[0]);
            continue;
        }
        for (int x = count; x <= QUANT_JOBS; ++x) m.start[x] = (int)at;
        if (mx) hipLaunchKernelGGL(quant_jobs_kernel<true>, dim3((unsigned)at), dim3(QUANT_THREADS), 0, jobs[i].s, m);
        else hipLaunchKernelGGL(quant_jobs_kernel<false>, dim3((unsigned)at), dim3(QUANT_THREADS), 0, jobs[i].s, m);
    }
}

static moe_status mx_rowcol_launch(moe_ctx* ctx, hipStream_t s, const char* who, const void* X, int64_t rows, int cols,
                                   const int32_t* rows_dev, void* q_row, uint8_t* e8_row, void* q_col, uint8_t* e8_col,
                                   const int32_t* src_of = nullptr, int k = 1, const float* pair_scale = nullptr,
                                   int groups = 1, int E = 0, bool after = false) {
    if (rows % 128 || cols % 128) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: rows and cols must be multiples of 128", who);
    if (groups < 1) groups = 1;
    const int64_t tiles_r = src_of ? (rows / 128 + groups - 1) / groups * groups : rows / 128;
    const int64_t nblk = tiles_r * (cols / 128);
    if (nblk > 0x7fffffffLL) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: too many tiles", who);
    quant_args a = quant_make(src_of ? QUANT_MX_GATHER : QUANT_MX, X, rows, cols, rows_dev, q_row, e8_row, q_col, e8_col, nblk);
    if (src_of) quant_gather(a, src_of, k, pair_scale, groups);
    a.E = E;
    quant_submit(ctx, s, a, after);
    return MOE_OK;
}

extern "C" moe_status moe_mx_quantize(moe_ctx* ctx, void* stream, const void* X, moe_mxblock block,
                                      int groups, int64_t rows, int cols, const int32_t* rows_dev,
                                      void* q, uint8_t* e8m0) {
    if (!ctx) return MOE_ERR_ARG;
    if (!X || !q || !e8m0) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize: NULL pointer");
    if (rows < 0 || cols < 1 || groups < 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize: bad sizes");
    hipStream_t s = (hipStream_t)stream;
    const int cu = ctx->num_cu > 0 ? ctx->num_cu : 256;
    if (rows == 0) return MOE_OK;
    switch (block) {
        case MOE_MX_1x32: {
            if (cols % 32) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize(1x32): cols %% 32 != 0");
            if (groups != 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize(1x32): groups must be 1 (fold them into rows)");
            int64_t grid = ceil_div64(rows * (cols / 8), 256);
            if (grid > (int64_t)cu * 32) grid = (int64_t)cu * 32;
            hipLaunchKernelGGL(mx_quant_1x32_kernel, dim3((unsigned)grid), dim3(256), 0, s, (const u32x4_t*)X, rows, cols,
                               rows_dev, 0, (u32x2_t*)q, e8m0);
            break;
        }
        case MOE_MX_32x1: {
            if (rows % 128) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize(32x1): rows %% 128 != 0");
            if (groups != 1 && rows_dev) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize(32x1): rows_dev needs groups == 1");
            moe_status st = mx_rowcol_launch(ctx, s, "moe_mx_quantize(32x1)", X, (int64_t)groups * rows, cols, rows_dev, nullptr,
                                             nullptr, q, e8m0);
            if (st != MOE_OK) return st;
            break;
        }
        default:
            MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize: bad block kind");
    }
    MOE_LAUNCH_CHECK(ctx, "moe_mx_quantize");
    return MOE_OK;
}

extern "C" moe_status moe_mx_quantize_rowcol(moe_ctx* ctx, void* stream, const void* X, int64_t rows, int cols,
                                             const int32_t* rows_dev, void* q_row, uint8_t* e8m0_row,
                                             void* q_col, uint8_t* e8m0_col) {
    if (!ctx) return MOE_ERR_ARG;
    if (!X || !q_row || !e8m0_row || !q_col || !e8m0_col) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize_rowcol: NULL pointer");
    if (rows < 0 || cols < 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize_rowcol: bad sizes");
    if (rows == 0) return MOE_OK;
    moe_status st = mx_rowcol_launch(ctx, (hipStream_t)stream, "moe_mx_quantize_rowcol", X, rows, cols, rows_dev, q_row,
                                     e8m0_row, q_col, e8m0_col);
    if (st != MOE_OK) return st;
    MOE_LAUNCH_CHECK(ctx, "moe_mx_quantize_rowcol");
    return MOE_OK;
}

extern "C" moe_status moe_mx_quantize_rowcol_gather(moe_ctx* ctx, void* stream, const void* X, const int32_t* src_of, int k,
                                                    const float* pair_scale, int groups, int64_t rows, int cols,
                                                    const int32_t* rows_dev, void* q_row, uint8_t* e8m0_row,
                                                    void* q_col, uint8_t* e8m0_col) {
    if (!ctx) return MOE_ERR_ARG;
    if (!X || !src_of || !q_row || !e8m0_row || !q_col || !e8m0_col)
        MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize_rowcol_gather: NULL pointer");
    if (rows < 0 || cols < 1 || k < 1 || k > 32 || groups < 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_mx_quantize_rowcol_gather: bad sizes");
    if (rows == 0) return MOE_OK;
    moe_status st = mx_rowcol_launch(ctx, (hipStream_t)stream, "moe_mx_quantize_rowcol_gather", X, rows, cols, rows_dev, q_row,
                                     e8m0_row, q_col, e8m0_col, src_of, k, pair_scale, groups);
    if (st != MOE_OK) return st;
    MOE_LAUNCH_CHECK(ctx, "moe_mx_quantize_rowcol_gather");
    return MOE_OK;
}

moe_status moe_quantise_live(moe_ctx* ctx, hipStream_t s, const void* X, int64_t rows, int cols, const int32_t* offsets, int E,
                             bool mx, void* q, void* scale, void* q_col, uint8_t* e8_col, bool after) {
    const char* who = "quantised copies of a grouped GEMM";
    const int32_t* const end = offsets + E;
    const int64_t most = (int64_t)(ctx->num_cu > 0 ? ctx->num_cu : 256) * 32, grid = ceil_div64(rows * (cols / 8), 256);
    const dim3 g((unsigned)(grid < most ? grid : most)), b(256);
    if (cols % 128) MOE_FAIL(ctx, MOE_ERR_ARG, "%s: %d columns are not a multiple of 128", who, cols);
    if (mx && q_col) {
        const moe_status st = mx_rowcol_launch(ctx, s, who, X, rows, cols, end, q, (uint8_t*)scale, q_col, e8_col, nullptr, 1, nullptr, 1, E, after);
        if (st != MOE_OK) return st;
    } else if (mx) {
        hipLaunchKernelGGL(mx_quant_1x32_kernel, g, b, 0, s, (const u32x4_t*)X, rows, cols, end, E, (u32x2_t*)q, (uint8_t*)scale);
    } else {
        hipLaunchKernelGGL(quant_1x128_kernel, g, b, 0, s, (const u32x4_t*)X, rows, cols, end, E, (u32x2_t*)q, (float*)scale);
    }
    MOE_LAUNCH_CHECK(ctx, who);
    return MOE_OK;
}
