// Gate GEMM, logits[T,E] = X[T,h] * Wr[E,h]^T (Sec. 2.1.2 item 1), for the calls that have too few rows or too short a contraction
// for the 256 x 256 tiles of gemm.hip: one launch, the contraction split among the waves of a workgroup.
//
// A workgroup owns a tile of 16 MB tokens x 16 NB experts; each of its waves takes every WAVES-th chunk of 64 contraction
// elements, straight from memory into MFMA fragments (both operands are contraction-contiguous: a lane's 8 elements are 16
// bytes of a row; a chunk's two steps of 32 share its cache lines), and the waves' sums meet in LDS and are added in order.
// Nothing is staged, so nothing is waited for but the loads themselves; AHEAD chunks per wave are in flight.
// Bound: the rate at which a compute unit takes these 64-byte row pieces, 38 bytes per ns, over (16 MB + 16 NB) rows of 2 h bytes
// per tile; hence the choice of tile by moe_gate_tile below.  Measured (us, 256 x 256 kernel with its second launch : this),
// T, E, h: 512, 48, 960 23.6 : 3.8; 64, 128, 4096 19.6 : 8.9; 512, 256, 7168 32 : 21; 2048, 64, 4096 25 : 13; 4000, 40, 2048
// 24 : 9.4; 16384, 32, 512 19 : 5.9; 16384, 64, 4096 39 : 34; 16384, 256, 1024 41 : 32; but 2048, 256, 7168 36 : 40 and 16384,
// 256, 7168 86 : 156, 16384, 128, 7168 61 : 81, 8192, 64, 7168 33 : 42.
#include "common.h"

template <int MB, int NB, int WAVES, int AHEAD>
__global__ __launch_bounds__(WAVES * 64, WAVES / 4) void gate_kernel(const char* __restrict__ X, const char* __restrict__ W, int T, int E,
                                                                     int h, int tiles_j, int tiles, float* __restrict__ out) {
    constexpr int BM = 16 * MB, BN = 16 * NB, PITCH = BN + 4;
    __shared__ __attribute__((aligned(16))) float part[WAVES * BM * PITCH];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (each XCD takes a contiguous run of the tiles: neighbours share their tokens in its L2)
    const int run = (tiles + 7) >> 3, at = (int)blockIdx.x >> 3, u = ((int)blockIdx.x & 7) * run + at;
    if (at >= run || u >= tiles) return;
    const int i0 = u / tiles_j * BM, j0 = u % tiles_j * BN;
    // byte offsets of this lane's rows (rows outside: the last one, not stored)
    const char* const x0 = X + (int64_t)i0 * h * 2;
    const char* const w0 = W + (int64_t)j0 * h * 2;
    uint32_t xo[MB], wo[NB];
#pragma unroll
    for (int i = 0; i < MB; ++i) xo[i] = (uint32_t)min(16 * i + l16, T - 1 - i0) * (uint32_t)(2 * h) + kq * 32;
#pragma unroll
    for (int j = 0; j < NB; ++j) wo[j] = (uint32_t)min(16 * j + l16, E - 1 - j0) * (uint32_t)(2 * h) + kq * 32;
    f32x4_t acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    bf16x8_t fx[AHEAD][2][MB], fw[AHEAD][2][NB];
    auto load = [&](int set, int c) __attribute__((always_inline)) {
        const char* const xs = x0 + (int64_t)c * 128;
        const char* const ws = w0 + (int64_t)c * 128;
#pragma unroll
        for (int k = 0; k < 2; ++k) {   // (16 of the lane's 32 bytes: the order inside a chunk is free)
#pragma unroll
            for (int i = 0; i < MB; ++i) fx[set][k][i] = *(const bf16x8_t*)(xs + xo[i] + 16 * k);
#pragma unroll
            for (int j = 0; j < NB; ++j) fw[set][k][j] = *(const bf16x8_t*)(ws + wo[j] + 16 * k);
        }
    };
    const int chunks = h / 64;
    int c = wave;
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
        if (c + s * WAVES < chunks) load(s, c + s * WAVES);
    while (c < chunks) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s, c += WAVES) {
            if (c >= chunks) continue;
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[s][k][j], fx[s][k][i], acc[i][j], 0, 0, 0);
            if (c + AHEAD * WAVES < chunks) load(s, c + AHEAD * WAVES);
        }
    }
    // a lane holds, per block, one token (l16) and 4 consecutive experts
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) *(f32x4_t*)(part + (wave * BM + 16 * i + l16) * PITCH + 16 * j + 4 * kq) = acc[i][j];
    __syncthreads();
    for (int x = tid; x < BM * BN / 4; x += WAVES * 64) {
        const int r = x / (BN / 4), q = x % (BN / 4) * 4;
        f32x4_t v = *(const f32x4_t*)(part + r * PITCH + q);
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v += *(const f32x4_t*)(part + (w * BM + r) * PITCH + q);
        if (i0 + r < T && j0 + q < E) *(f32x4_t*)(out + (int64_t)(i0 + r) * E + j0 + q) = v;
    }
}

template <int MB, int NB, int WAVES, int AHEAD>
static void gate_go(hipStream_t s, const void* X, const void* W, int T, int E, int h, float* out) {
    const int64_t tj = ceil_div64(E, 16 * NB), n = ceil_div64(T, 16 * MB) * tj;
    hipLaunchKernelGGL((gate_kernel<MB, NB, WAVES, AHEAD>), dim3((unsigned)(ceil_div64(n, 8) * 8)), dim3(WAVES * 64), 0, s, (const char*)X,
                       (const char*)W, T, E, h, (int)tj, (int)n, out);
}
// The best tile's number, and its time in microseconds: 2.1 + the bytes of a compute unit's tiles at 38.8 per ns, a started round
// counted half, + X and the logits at 15.5 TB/s (what memory adds to the units' own rate).  Between 31 % low and 14 % high of 135 measured
// sizes, 7 % in the root mean square.
static const int GATE_TILES[6][2] = {{16, 16}, {32, 16}, {32, 32}, {64, 32}, {64, 64}, {64, 128}};
int moe_gate_tile(int num_cu, int T, int E, int h, double* us) {
    int best = -1;
    for (int x = 0; x < 6; ++x) {
        const int64_t n = ceil_div64(T, GATE_TILES[x][0]) * ceil_div64(E, GATE_TILES[x][1]);
        double r = (double)n / num_cu;
        r = r < 1 ? 1 : (r + __builtin_ceil(r)) / 2;
        const double t = 2.1 + r * (GATE_TILES[x][0] + GATE_TILES[x][1]) * 2.0 * h / 38.8e3 + (2.0 * T * h + 4.0 * T * E) / 15.5e6;
        if (n <= 0x7ffffff0 && (best < 0 || t < *us)) {
            best = x;
            *us = t;
        }
    }
    return best;
}
void moe_gate_launch(hipStream_t s, int tile, const void* X, const void* W, int T, int E, int h, float* out) {
    if (tile == 0) gate_go<1, 1, 8, 2>(s, X, W, T, E, h, out);
    else if (tile == 1) gate_go<2, 1, 8, 4>(s, X, W, T, E, h, out);
    else if (tile == 2) gate_go<2, 2, 8, 2>(s, X, W, T, E, h, out);
    else if (tile == 3) gate_go<4, 2, 8, 2>(s, X, W, T, E, h, out);
    else if (tile == 4) gate_go<4, 4, 8, 2>(s, X, W, T, E, h, out);
    else gate_go<4, 8, 4, 1>(s, X, W, T, E, h, out);
}
