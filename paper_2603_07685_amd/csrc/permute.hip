// moe_permute / moe_unpermute_combine(+bwd): the row-ID map and the row moves
// (Sec. 4.3.3: preprocessing, permute, unpermute; Sec. 5.4.1: padding fused into permute).
//
// Row-ID map = stable counting sort of the T*k (token, slot) pairs by expert, with
// no atomics on positions so the map is bit-reproducible:
//   1. hist : a workgroup per chunk of PERMUTE_CHUNK consecutive pairs builds that chunk's per-expert histogram (LDS) and
//             stores it to the workspace;
//   2. scan : per expert, exclusive scan of the chunk histograms (chunk bases),
//             totals -> counts, padded exclusive scan over experts -> offsets;
//   3. rank : a workgroup per chunk again, one wavefront per 64 pairs; a lane's rank among equal experts inside the 64
//             comes from ballots over the bits of the expert id, the wavefronts' counts are scanned in LDS.  Further
//             workgroups mark the rows that no pair owns (src_of = -1).
// Up to PERMUTE_ALL_PAIRS pairs, unless their rows are large (permute_all_rows), all of it and the row move are one launch
// (permute_all_kernel).
// Bound: launches and dependent latencies (the map of 131072 pairs is 1.5 MB).  Measured, all kernels of the map: T 16384, k 8, E 32:
// 35 : 16.6 us (fill, one wavefront per chunk, a serial scan over the chunks : this).
// Row moves are token-major: a workgroup reads one source row once and writes
// its k copies (permute), or reads the k expert rows once and writes one row
// (combine), 16 bytes per lane per access, fp32 accumulation in registers.
#include "common.h"
#include "layout.h"

#ifndef MOVE_THREADS
#define MOVE_THREADS 256
#endif

__device__ __forceinline__ u32x4_t mk4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    u32x4_t v = {a, b, c, d};
    return v;
}

// ---------------------------------------------------------------------------
// 1. per-chunk histograms
// ---------------------------------------------------------------------------
static_assert(PERMUTE_CHUNK == 1024, "one pair per thread of a 1024-thread workgroup");
__global__ __launch_bounds__(1024) void permute_hist_kernel(const int32_t* __restrict__ idx, int64_t pairs, int E,
                                                            int32_t* __restrict__ chunk_hist) {
    extern __shared__ int32_t lds[];
    const int tid = threadIdx.x;
    const int64_t j = (int64_t)blockIdx.x * PERMUTE_CHUNK + tid;
    const int e = j < pairs ? idx[j] : -1;
    if (tid < E) lds[tid] = 0;
    __syncthreads();
    if (e >= 0 && e < E) atomicAdd(&lds[e], 1);
    __syncthreads();
    if (tid < E) chunk_hist[(int64_t)blockIdx.x * E + tid] = lds[tid];
}

// Exclusive scan over the 1024 threads of a workgroup (int64: sums of padded counts); *total = the sum of all.
__device__ __forceinline__ int64_t block_scan_1024(int64_t v, int64_t (&wsum)[16], int64_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int64_t base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        if (w < wave) base += wsum[w];
        all += wsum[w];
    }
    *total = all;
    return base + incl - v;
}

// ---------------------------------------------------------------------------
// 2. scans: chunk bases per expert, counts, padded offsets
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void permute_scan_kernel(int32_t* __restrict__ chunk_hist, int nchunks, int E, int log_e,
                                                            int align, int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ offsets) {
    // One workgroup.  Thread (segment, expert): the chunks are cut into up to 32 segments; a thread sums its segment, the
    // segments' sums meet in LDS, then it walks its segment again and leaves the running base of every chunk.
    __shared__ int32_t part[1024];
    __shared__ int64_t wsum[16];
    const int tid = threadIdx.x;
    const int e = tid & ((1 << log_e) - 1), seg = tid >> log_e;   // (E <= 1024 is checked by the caller)
    const int nseg = min(1024 >> log_e, 32), len = (nchunks + nseg - 1) / nseg;
    const int c0 = min(seg * len, nchunks), c1 = seg < nseg ? min(c0 + len, nchunks) : c0;
    int32_t sum = 0;
    if (e < E)
        for (int c = c0; c < c1; ++c) sum += chunk_hist[(int64_t)c * E + e];
    part[tid] = sum;
    __syncthreads();
    int32_t run = 0, tot = 0;
    for (int s = 0; s < nseg; ++s) {
        const int32_t v = part[(s << log_e) + e];
        run += s < seg ? v : 0;
        tot += v;
    }
    if (e < E) {
        for (int c = c0; c < c1; ++c) {
            int32_t* h = chunk_hist + (int64_t)c * E + e;
            const int32_t v = *h;
            *h = run;
            run += v;
        }
    }
    // (segment 0: thread = expert)
    const bool mine = seg == 0 && e < E;
    int64_t total;
    const int64_t at = block_scan_1024(mine ? ((int64_t)tot + align - 1) / align * align : 0, wsum, &total);
    if (mine) {
        counts[e] = tot;
        offsets[e] = (int32_t)at;
    }
    if (tid == 0) offsets[E] = (int32_t)total;
}

// The 64 pairs of a wavefront: each valid lane's peers (lanes with the same expert), and its rank among them.
__device__ __forceinline__ uint64_t expert_peers(int e, bool valid, int nbits) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
        const uint64_t m = __ballot((e >> b) & 1);
        peers &= ((e >> b) & 1) ? m : ~m;
    }
    return peers;
}

// ---------------------------------------------------------------------------
// 3. stable ranks -> row_of, src_of
// ---------------------------------------------------------------------------
#define FILL_ROWS 4096  // rows behind offsets[E] per filling workgroup
__global__ __launch_bounds__(1024) void permute_rank_kernel(const int32_t* __restrict__ idx, int64_t pairs, int E,
                                                            int nbits, int nchunks, int64_t Rcap,
                                                            const int32_t* __restrict__ chunk_base,
                                                            const int32_t* __restrict__ offsets, const int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ row_of, int32_t* __restrict__ src_of) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x;
    if (b >= nchunks) {  // rows that no pair owns: an expert's padding rows, then what lies behind the last expert
        int64_t r0, r1;
        if (b < nchunks + E) {
            const int e = b - nchunks;
            r0 = (int64_t)offsets[e] + counts[e];
            r1 = offsets[e + 1];
        } else {
            r0 = offsets[E] + (int64_t)(b - nchunks - E) * FILL_ROWS;
            r1 = min(r0 + FILL_ROWS, Rcap);
        }
        for (int64_t r = r0 + tid; r < r1; r += 1024) src_of[r] = -1;
        return;
    }
    extern __shared__ int32_t wcnt[];  // [16][E]: pairs per wavefront and expert, then the rows they start at
    for (int i = tid; i < 16 * E; i += 1024) wcnt[i] = 0;
    const int64_t j = (int64_t)b * PERMUTE_CHUNK + tid;
    const int e = j < pairs ? idx[j] : -1;
    const bool valid = e >= 0 && e < E;
    const uint64_t peers = expert_peers(e, valid, nbits);
    const int rank = __popcll(peers & ((1ull << lane) - 1ull));
    __syncthreads();
    if (valid && rank == 0) wcnt[wave * E + e] = __popcll(peers);
    __syncthreads();
    if (tid < E) {
        int32_t run = offsets[tid] + chunk_base[(int64_t)b * E + tid];
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int32_t v = wcnt[w * E + tid];
            wcnt[w * E + tid] = run;
            run += v;
        }
    }
    __syncthreads();
    if (valid) {
        const int row = wcnt[wave * E + e] + rank;
        row_of[j] = row;
        src_of[row] = (int32_t)j;
    } else if (j < pairs) {
        row_of[j] = -1;
    }
}

// ---------------------------------------------------------------------------
// Small calls: map and row move in one launch.  A workgroup owns a few tokens; it counts all pairs by itself, those in front of its own
// apart from the others, ranks its own and copies its tokens' rows.  Every workgroup reads all expert ids (up to 128 KB, from L2),
// which buys two launches' gaps.  Rows that no pair owns are dealt to all workgroups; where there are many of them for the tokens'
// workgroups, further ones without tokens follow (permute_all_grid).
// ---------------------------------------------------------------------------
#define PERMUTE_ALL_THREADS 512
// Us, three launches for the map and one for the rows : this; loads scattered by 30 % | 95 % of the pairs on one expert.  h 512, k 8, 16384
// pairs: E 8 14.5 : 9.6 | 14.6 : 9.5; E 512 17.3 : 10.4 | 17.3 : 14.3; 32768 pairs: E 8 17.7 : 15.4 | 17.7 : 15.2; E 256 20.5 : 16.3 |
// 20.4 : 17.8; E 512 23.3 : 16.8 | 23.1 : 24.1 (the only loss).  Twice as many pairs would cost twice the time here, a fifth more
// there.  The map alone, 16384 pairs: E 8 10.4 : 7.1 | 10.6 : 7.1; E 512 13.1 : 7.9 | 13.3 : 11.8.
// The rows of a large call move faster with a workgroup for every token, and the map is a small part of it (permute_all_rows; E 32, all
// pairs valid | one in eight): 32768 pairs, k 1, h 1024 31.3 : 30.3 | 26.4 : 23.8, h 2048 44.1 : 48.1 | 32.2 : 34.2, h 4096 73 : 126 |
// 49 : 60; k 8, h 1024 23.8 : 22.3 | 14.6 : 12.9, h 2048 36.2 : 36.1 | 15.3 : 17.6, h 7168 103 : 103 | 26.8 : 32.9; 16384 pairs, k 1, h
// 2048 28.5 : 26.6 | 22.6 : 20.3, h 4096 42.9 : 44.3 | 30.5 : 30.9, h 7168 66 : 70 | 45.6 : 47.1; k 8, h 7168 57.0 : 53.4 | 18.1 :
// 17.4; 8192 pairs, k 1, h 7168 39.2 : 38.0 | 28.3 : 26.7.
#define PERMUTE_ALL_PAIRS 32768  // (the map alone: half)
#define PERMUTE_ALL_E 512
#define PERMUTE_ALL_GRID 256     // most workgroups because of rows without a pair
__host__ __device__ __forceinline__ int permute_copies(int E) { return E <= 128 ? 8 : E <= 256 ? 4 : 2; }
__global__ __launch_bounds__(PERMUTE_ALL_THREADS) void permute_all_kernel(
    const u32x4_t* __restrict__ X, const int32_t* __restrict__ idx, int T, int k, int E, int nbits, int align, int per_wg, int vec,
    uint64_t vec_magic, int64_t Rcap, u32x4_t* __restrict__ Xp, int32_t* __restrict__ row_of, int32_t* __restrict__ src_of,
    int32_t* __restrict__ offsets, int32_t* __restrict__ counts) {
    constexpr int NT = PERMUTE_ALL_THREADS, NW = NT / 64, AHEAD = 8;
    extern __shared__ int32_t lds[];
    // [E][2][copies] counts, [E] the experts' ends, [E + 1] offsets, [NW][E].  An expert's count is kept in several copies, a lane's
    // by its number: equal addresses of a wavefront are added one by one, 64 of them under a hot expert
    const int copies = permute_copies(E);
    int32_t *const cnt = lds, *const ends = lds + 2 * copies * E, *const offs = ends + E, *const wcnt = offs + E + 1;
    __shared__ int32_t rows[NT], wsum[NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, G = (int)gridDim.x, b = (int)blockIdx.x;
    const int pairs = T * k, t0 = min(b * per_wg, T), nt = min(per_wg, T - t0), own0 = t0 * k, own = nt * k;
    for (int i = tid; i < 2 * copies * E; i += NT) cnt[i] = 0;
    for (int i = tid; i < NW * E; i += NT) wcnt[i] = 0;
    __syncthreads();
    // ---- counts of the pairs in front of this workgroup's, and of the others ----
    for (int j0 = 0; j0 < pairs; j0 += NT * AHEAD) {
        int ex[AHEAD];
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            const int j = j0 + s * NT + tid;
            ex[s] = j < pairs ? idx[j] : -1;
        }
#pragma unroll
        for (int s = 0; s < AHEAD; ++s)
            if (ex[s] >= 0 && ex[s] < E)
                atomicAdd(&cnt[(2 * ex[s] + (j0 + s * NT + tid < own0 ? 0 : 1)) * copies + (lane & (copies - 1))], 1);
    }
    // ---- this workgroup's pairs: peers inside a wavefront ----
    const int e = tid < own ? idx[own0 + tid] : -1;
    const bool valid = e >= 0 && e < E;
    const uint64_t peers = expert_peers(e, valid, nbits);
    const int rank = __popcll(peers & ((1ull << lane) - 1ull));
    if (valid && rank == 0) wcnt[wave * E + e] = __popcll(peers);
    __syncthreads();
    // ---- offsets, and the rows that the wavefronts' pairs start at ----
    int before = 0, tot = 0;
    if (tid < E)
        for (int c = 0; c < copies; ++c) {
            before += cnt[2 * tid * copies + c];
            tot += cnt[(2 * tid + 1) * copies + c];
        }
    tot += before;
    const int padded = (tot + align - 1) / align * align;
    int incl = padded;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int at = incl - padded, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (w < wave) at += wsum[w];
        total += wsum[w];
    }
    if (tid < E) {
        offs[tid] = at;
        ends[tid] = at + tot;
        if (b == 0) {
            offsets[tid] = at;
            counts[tid] = tot;
        }
        int run = at + before;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int v = wcnt[w * E + tid];
            wcnt[w * E + tid] = run;
            run += v;
        }
    }
    if (tid == 0) {
        offs[E] = total;
        if (b == 0) offsets[E] = total;
    }
    __syncthreads();
    if (tid < own) {
        const int row = valid ? wcnt[wave * E + e] + rank : -1;
        rows[tid] = row;
        row_of[own0 + tid] = row;
        if (valid) src_of[row] = own0 + tid;
    }
    // ---- rows that no pair owns: padding rows, spread over the workgroups, and what lies behind the last expert ----
    if (align > 1) {
        for (int x = wave; x < E; x += NW)   // (an expert's first row goes to the workgroup behind its predecessor's last)
            for (int r = ends[x] + (int)((b + (uint32_t)x * (uint32_t)(align - 1)) % (uint32_t)G); r < offs[x + 1]; r += G) {
                if (lane == 0) src_of[r] = -1;
                if (Xp)
                    for (int c = lane; c < vec; c += 64) Xp[(int64_t)r * vec + c] = mk4(0, 0, 0, 0);
            }
    }
    for (int64_t r = total + (int64_t)b * NT + tid; r < Rcap; r += (int64_t)G * NT) src_of[r] = -1;
    if (!Xp) return;
    __syncthreads();
    // ---- the tokens' rows, each read once ----
    const u32x4_t* const src = X + (int64_t)t0 * vec;
    for (int c0 = tid; c0 < nt * vec; c0 += 4 * NT) {
        u32x4_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c0 + u * NT < nt * vec) v[u] = src[c0 + u * NT];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * NT;
            if (c >= nt * vec) break;
            const int t = (int)(((uint64_t)c * vec_magic) >> 32), at_c = c - t * vec;   // c / vec (see permute_launch)
            for (int s = 0; s < k; ++s) {
                const int r = rows[t * k + s];
                if (r >= 0) __builtin_nontemporal_store(v[u], &Xp[(int64_t)r * vec + at_c]);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// permute: token-major row scatter + zero fill of padding rows
// ---------------------------------------------------------------------------
// grid = T token blocks followed by E padding blocks.
__global__ __launch_bounds__(MOVE_THREADS) void permute_rows_kernel(
    const u32x4_t* __restrict__ X, const int32_t* __restrict__ row_of, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ counts, int T, int k, int E, int vec_per_row, u32x4_t* __restrict__ Xp) {
    __shared__ int32_t rows[32 * 4];
    const int b = blockIdx.x;
    if (b < T) {
        for (int s = threadIdx.x; s < k; s += MOVE_THREADS) rows[s] = row_of[(int64_t)b * k + s];
        __syncthreads();
        const u32x4_t* src = X + (int64_t)b * vec_per_row;
        // four 16-byte pieces of the source row per thread are loaded before the first copy is written, so a
        // row of up to 16 KB is in flight at once instead of one piece per thread
        for (int c0 = threadIdx.x; c0 < vec_per_row; c0 += 4 * MOVE_THREADS) {
            u32x4_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * MOVE_THREADS;
                if (c < vec_per_row) v[u] = src[c];
            }
            for (int s = 0; s < k; ++s) {
                const int r = rows[s];
                if (r < 0) continue;
                u32x4_t* dst = Xp + (int64_t)r * vec_per_row;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = c0 + u * MOVE_THREADS;
                    if (c < vec_per_row) __builtin_nontemporal_store(v[u], &dst[c]);
                }
            }
        }
    } else {
        const int e = b - T;
        const int64_t r0 = (int64_t)offsets[e] + counts[e], r1 = offsets[e + 1];
        const int64_t n = (r1 - r0) * vec_per_row;
        u32x4_t z = mk4(0, 0, 0, 0);
        u32x4_t* dst = Xp + r0 * vec_per_row;
        for (int64_t i = threadIdx.x; i < n; i += MOVE_THREADS) dst[i] = z;
    }
}

// ---------------------------------------------------------------------------
// combine: Y[t] = sum_s w[t,s] * O[row_of[t,s]] (+ residual[t]); fp32 accumulation
// ---------------------------------------------------------------------------
template <bool F32>
__device__ __forceinline__ void acc_vec(float (&a)[8], u32x4_t v, float w);
template <>
__device__ __forceinline__ void acc_vec<false>(float (&a)[8], u32x4_t v, float w) {
    a[0] += w * bf16_lo(v.x); a[1] += w * bf16_hi(v.x);
    a[2] += w * bf16_lo(v.y); a[3] += w * bf16_hi(v.y);
    a[4] += w * bf16_lo(v.z); a[5] += w * bf16_hi(v.z);
    a[6] += w * bf16_lo(v.w); a[7] += w * bf16_hi(v.w);
}
template <>
__device__ __forceinline__ void acc_vec<true>(float (&a)[8], u32x4_t v, float w) {
    a[0] += w * __uint_as_float(v.x); a[1] += w * __uint_as_float(v.y);
    a[2] += w * __uint_as_float(v.z); a[3] += w * __uint_as_float(v.w);
}

#define COMBINE_MAX_K 32

template <bool F32>
__global__ __launch_bounds__(MOVE_THREADS) void combine_kernel(
    const u32x4_t* __restrict__ O, const int32_t* __restrict__ row_of, const float* __restrict__ prob,
    const u32x4_t* __restrict__ residual, int T, int k, int vec_per_row, u32x4_t* __restrict__ Y) {
    __shared__ int32_t rows[COMBINE_MAX_K];
    __shared__ float wts[COMBINE_MAX_K];
    const int t = blockIdx.x;
    for (int s = threadIdx.x; s < k; s += MOVE_THREADS) {
        rows[s] = row_of[(int64_t)t * k + s];
        wts[s] = prob ? prob[(int64_t)t * k + s] : 1.0f;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < vec_per_row; c += MOVE_THREADS) {
        float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (residual) acc_vec<F32>(a, residual[(int64_t)t * vec_per_row + c], 1.0f);
        int s = 0;
        for (; s + 8 <= k; s += 8) {  // eight independent row reads in flight
            u32x4_t v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int r = rows[s + j];
                v[j] = r >= 0 ? __builtin_nontemporal_load(&O[(int64_t)r * vec_per_row + c]) : mk4(0, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) acc_vec<F32>(a, v[j], wts[s + j]);
        }
        for (; s + 4 <= k; s += 4) {  // four independent row reads in flight
            int r0 = rows[s], r1 = rows[s + 1], r2 = rows[s + 2], r3 = rows[s + 3];
            u32x4_t z = mk4(0, 0, 0, 0);
            u32x4_t v0 = r0 >= 0 ? __builtin_nontemporal_load(&O[(int64_t)r0 * vec_per_row + c]) : z;
            u32x4_t v1 = r1 >= 0 ? __builtin_nontemporal_load(&O[(int64_t)r1 * vec_per_row + c]) : z;
            u32x4_t v2 = r2 >= 0 ? __builtin_nontemporal_load(&O[(int64_t)r2 * vec_per_row + c]) : z;
            u32x4_t v3 = r3 >= 0 ? __builtin_nontemporal_load(&O[(int64_t)r3 * vec_per_row + c]) : z;
            acc_vec<F32>(a, v0, wts[s]);
            acc_vec<F32>(a, v1, wts[s + 1]);
            acc_vec<F32>(a, v2, wts[s + 2]);
            acc_vec<F32>(a, v3, wts[s + 3]);
        }
        for (; s < k; ++s) {
            int r = rows[s];
            if (r >= 0) acc_vec<F32>(a, O[(int64_t)r * vec_per_row + c], wts[s]);
        }
        u32x4_t out;
        if (F32) {
            out = mk4(__float_as_uint(a[0]), __float_as_uint(a[1]), __float_as_uint(a[2]), __float_as_uint(a[3]));
        } else {
            out = mk4(pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3]), pack_bf16(a[4], a[5]), pack_bf16(a[6], a[7]));
        }
        Y[(int64_t)t * vec_per_row + c] = out;
    }
}

// ---------------------------------------------------------------------------
// combine backward: dO[row_of[t,s]] = w[t,s] * dY[t];  dprob[t,s] = <dY[t], O[row_of[t,s]]>
// ---------------------------------------------------------------------------
template <bool F32>
__device__ __forceinline__ u32x4_t scale_vec(u32x4_t v, float w);
template <>
__device__ __forceinline__ u32x4_t scale_vec<false>(u32x4_t v, float w) {
    return mk4(pack_bf16(w * bf16_lo(v.x), w * bf16_hi(v.x)), pack_bf16(w * bf16_lo(v.y), w * bf16_hi(v.y)),
                      pack_bf16(w * bf16_lo(v.z), w * bf16_hi(v.z)), pack_bf16(w * bf16_lo(v.w), w * bf16_hi(v.w)));
}
template <>
__device__ __forceinline__ u32x4_t scale_vec<true>(u32x4_t v, float w) {
    return mk4(__float_as_uint(w * __uint_as_float(v.x)), __float_as_uint(w * __uint_as_float(v.y)),
                      __float_as_uint(w * __uint_as_float(v.z)), __float_as_uint(w * __uint_as_float(v.w)));
}
template <bool F32>
__device__ __forceinline__ float dot_vec(u32x4_t a, u32x4_t b);
template <>
__device__ __forceinline__ float dot_vec<false>(u32x4_t a, u32x4_t b) {
    return bf16_lo(a.x) * bf16_lo(b.x) + bf16_hi(a.x) * bf16_hi(b.x) + bf16_lo(a.y) * bf16_lo(b.y) +
           bf16_hi(a.y) * bf16_hi(b.y) + bf16_lo(a.z) * bf16_lo(b.z) + bf16_hi(a.z) * bf16_hi(b.z) +
           bf16_lo(a.w) * bf16_lo(b.w) + bf16_hi(a.w) * bf16_hi(b.w);
}
template <>
__device__ __forceinline__ float dot_vec<true>(u32x4_t a, u32x4_t b) {
    return __uint_as_float(a.x) * __uint_as_float(b.x) + __uint_as_float(a.y) * __uint_as_float(b.y) +
           __uint_as_float(a.z) * __uint_as_float(b.z) + __uint_as_float(a.w) * __uint_as_float(b.w);
}

#define ZERO_ROWS 64
template <bool F32>
__global__ __launch_bounds__(MOVE_THREADS) void combine_bwd_kernel(
    const u32x4_t* __restrict__ dY, const u32x4_t* __restrict__ O, const int32_t* __restrict__ row_of,
    const float* __restrict__ prob, int T, int k, int vec_per_row, u32x4_t* __restrict__ dO,
    float* __restrict__ dprob, const int32_t* __restrict__ src_of, int64_t Rcap) {
    __shared__ int32_t rows[COMBINE_MAX_K];
    __shared__ float wts[COMBINE_MAX_K];
    __shared__ float part[COMBINE_MAX_K][MOVE_THREADS / 64];
    const int t = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (t >= T) {  // behind the tokens: workgroups that zero the rows no pair owns, ZERO_ROWS rows each
        const int64_t r0 = (int64_t)(t - T) * ZERO_ROWS + wave * (ZERO_ROWS / (MOVE_THREADS / 64));
        const int64_t r = r0 + lane;
        uint64_t pad = __ballot(lane < ZERO_ROWS / (MOVE_THREADS / 64) && r < Rcap && src_of[min(r, Rcap - 1)] < 0);
        for (; pad; pad &= pad - 1) {
            u32x4_t* const row = dO + (r0 + __builtin_ctzll(pad)) * vec_per_row;
            for (int c = lane; c < vec_per_row; c += 64) row[c] = mk4(0, 0, 0, 0);
        }
        return;
    }
    for (int s = threadIdx.x; s < k; s += MOVE_THREADS) {
        rows[s] = row_of[(int64_t)t * k + s];
        wts[s] = prob ? prob[(int64_t)t * k + s] : 1.0f;
    }
    __syncthreads();
    const bool want_dot = dprob != nullptr && O != nullptr;
    // slots in chunks of 8: per 16-byte piece of dY[t] the 8 expert rows are read together (9 loads in flight per
    // thread) and the 8 scaled copies written; a slot's partial dot product stays in one register, summed over
    // the pieces in increasing order
    for (int s0 = 0; s0 < k; s0 += 8) {
        float acc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.f;
        for (int c = threadIdx.x; c < vec_per_row; c += MOVE_THREADS) {
            const u32x4_t g = dY[(int64_t)t * vec_per_row + c];
            u32x4_t o[8];
            if (want_dot) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int r = s0 + j < k ? rows[s0 + j] : -1;
                    if (r >= 0) o[j] = __builtin_nontemporal_load(&O[(int64_t)r * vec_per_row + c]);
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int r = s0 + j < k ? rows[s0 + j] : -1;
                if (r >= 0) {
                    if (want_dot) acc[j] += dot_vec<F32>(g, o[j]);
                    if (dO) __builtin_nontemporal_store(scale_vec<F32>(g, wts[s0 + j]), &dO[(int64_t)r * vec_per_row + c]);
                }
            }
        }
        if (dprob) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (s0 + j < k) {
                    float a = acc[j];
#pragma unroll
                    for (int o2 = 32; o2 > 0; o2 >>= 1) a += __shfl_xor(a, o2);
                    if (lane == 0) part[s0 + j][wave] = a;
                }
            }
        }
    }
    if (dprob) {
        __syncthreads();
        for (int s = threadIdx.x; s < k; s += MOVE_THREADS) {
            float a = 0.f;
            for (int w = 0; w < MOVE_THREADS / 64; ++w) a += part[s][w];
            dprob[(int64_t)t * k + s] = a;
        }
    }
}

// ---------------------------------------------------------------------------
// host entry points
// ---------------------------------------------------------------------------
static int bits_for(int E) {
    int b = 0;
    while ((1 << b) < E) ++b;
    return b;
}

// Argument checks shared by moe_permute and moe_permute_static (err: where the message goes, 512 bytes, or NULL).
static moe_status permute_check(char* err, const void* X, moe_dtype dt, const int32_t* idx, int T, int k, int h, int E,
                                int align, const void* Xp, int64_t Rcap, const int32_t* row_of, const int32_t* src_of,
                                const int32_t* offsets, const int32_t* counts) {
#define PERMUTE_FAIL(code, ...)                        \
    do {                                               \
        if (err) snprintf(err, 512, __VA_ARGS__);      \
        return (code);                                 \
    } while (0)
    if (!idx || !row_of || !src_of || !offsets || !counts) PERMUTE_FAIL(MOE_ERR_ARG, "moe_permute: NULL map pointer");
    if ((X == nullptr) != (Xp == nullptr)) PERMUTE_FAIL(MOE_ERR_ARG, "moe_permute: X and Xp must both be given or both NULL");
    if (T < 0 || k < 1 || k > 32 || E < 1 || E > 1024 || align < 1 || h < 1)
        PERMUTE_FAIL(MOE_ERR_ARG, "moe_permute: need T>=0, 1<=k<=32, 1<=E<=1024, align>=1, h>=1");
    if (dt != MOE_BF16 && dt != MOE_F32) PERMUTE_FAIL(MOE_ERR_UNSUPPORTED, "moe_permute: dtype must be bf16 or f32");
    const size_t row_bytes = (size_t)h * moe_dtype_size(dt);
    if (X && row_bytes % 16) PERMUTE_FAIL(MOE_ERR_ARG, "moe_permute: row size %zu B is not a multiple of 16", row_bytes);
    const int64_t pairs = (int64_t)T * k;
    const int64_t need = pairs + (int64_t)E * (align - 1);
    if (Rcap < need) PERMUTE_FAIL(MOE_ERR_ARG, "moe_permute: Rcap=%lld < T*k+E*(align-1)=%lld", (long long)Rcap, (long long)need);
    if (Rcap > 0x7fffffffLL) PERMUTE_FAIL(MOE_ERR_ARG, "moe_permute: Rcap exceeds int32");
#undef PERMUTE_FAIL
    return MOE_OK;
}

// Workgroups of permute_all_kernel: the tokens', or so many that none fills more than 64 KB of rows without a pair, up to one per
// compute unit.  Us, three launches and the row move : the tokens' workgroups alone : 256 : 1024; T 1 k 8 h 7168 E 8, padded to 128 rows,
// 20.6 : 80.9 : 7.7 : 7.7; T 64 k 8 h 4096 E 128, padded to 128, 25.4 : 26.3 : 21.9 : 24.3; T 256 k 8 h 7168 E 256, padded to 128,
// 98.8 : 92.6 : 92.9 : 96.4; T 16 k 2 h 1024 E 8, 2^22 rows more than pairs, 13.5 : 20.5 : 7.9 : 7.9; T 1 k 8 h 1024 E 8, 2^24 more,
// 21.6 : 846 : 15.6 : 14.7.
static unsigned permute_all_grid(int T, int per_wg, int E, int align, int vec, int64_t free_rows) {
    const int64_t tokens = T > per_wg ? (T + per_wg - 1) / per_wg : 1;
    const int64_t fill = ceil_div64((int64_t)E * (align - 1) * vec * 16 + free_rows * 4, 65536);
    return (unsigned)(fill < tokens ? tokens : fill < PERMUTE_ALL_GRID ? fill : PERMUTE_ALL_GRID > tokens ? PERMUTE_ALL_GRID : tokens);
}

// Whether the rows of a call are few enough for permute_all_kernel (PERMUTE_ALL_PAIRS): X up to 128 MB up to 8192 pairs, up to 64 MB
// up to 16384, 64 MB of rows to be written above.
static bool permute_all_rows(int64_t pairs, int T, int64_t row_bytes) {
    const int64_t MB = 1 << 20;
    return pairs <= 8192 ? T * row_bytes <= 128 * MB : pairs <= 16384 ? T * row_bytes <= 64 * MB : pairs * row_bytes <= 64 * MB;
}

// The launches of one permute call; chunk_hist = int32 [chunks, E] of device scratch (every entry is written by the
// histogram kernel before it is read: the buffer needs no clearing).
static void permute_launch(hipStream_t s, const void* X, moe_dtype dt, const int32_t* idx, int T, int k, int h, int E,
                           int align, void* Xp, int64_t Rcap, int32_t* row_of, int32_t* src_of, int32_t* offsets,
                           int32_t* counts, int32_t* chunk_hist) {
    const int64_t pairs = (int64_t)T * k;
    const int nchunks = (int)moe_permute_chunks(pairs), nbits = bits_for(E);
    const int vec = X ? (int)((size_t)h * moe_dtype_size(dt) / 16) : 0;
    const int per_wg = T > 256 ? (T + 255) / 256 : 1;   // a workgroup per compute unit
    if (pairs <= (X ? PERMUTE_ALL_PAIRS : PERMUTE_ALL_PAIRS / 2) && E <= PERMUTE_ALL_E && (int64_t)per_wg * vec * vec < (1LL << 32) &&
        permute_all_rows(pairs, T, (int64_t)vec * 16)) {
        // (c / vec = c * ceil(2^32 / vec) / 2^32 for c < per_wg * vec: the rounding adds less than c vec / 2^32 of a step)
        const uint64_t magic = vec ? ((1ull << 32) + vec - 1) / vec : 0;
        hipLaunchKernelGGL(permute_all_kernel, dim3(permute_all_grid(T, per_wg, E, align, vec, Rcap - pairs)), dim3(PERMUTE_ALL_THREADS),
                           (size_t)((2 * permute_copies(E) + 2 + PERMUTE_ALL_THREADS / 64) * E + 1) * sizeof(int32_t), s, (const u32x4_t*)X, idx, T, k, E, nbits,
                           align, per_wg, vec, magic, Rcap, (u32x4_t*)Xp, row_of, src_of, offsets, counts);
        return;
    }
    if (nchunks > 0)
        hipLaunchKernelGGL(permute_hist_kernel, dim3(nchunks), dim3(1024), (size_t)E * sizeof(int32_t), s, idx, pairs, E, chunk_hist);
    hipLaunchKernelGGL(permute_scan_kernel, dim3(1), dim3(1024), 0, s, chunk_hist, nchunks, E, nbits, align, counts, offsets);
    // (rows without a pair: at most Rcap of them behind the last expert, if every slot is skipped)
    hipLaunchKernelGGL(permute_rank_kernel, dim3(nchunks + E + (unsigned)ceil_div64(Rcap, FILL_ROWS)), dim3(1024),
                       (size_t)16 * E * sizeof(int32_t), s, idx, pairs, E, nbits, nchunks, Rcap, chunk_hist, offsets, counts,
                       row_of, src_of);
    if (X) {
        hipLaunchKernelGGL(permute_rows_kernel, dim3(T + E), dim3(MOVE_THREADS), 0, s, (const u32x4_t*)X, row_of, offsets,
                           counts, T, k, E, vec, (u32x4_t*)Xp);
    }
}

extern "C" moe_status moe_permute(moe_ctx* ctx, void* stream, const void* X, moe_dtype dt,
                                  const int32_t* idx, int T, int k, int h, int E, int align,
                                  void* Xp, int64_t Rcap,
                                  int32_t* row_of, int32_t* src_of, int32_t* offsets, int32_t* counts) {
    if (!ctx) return MOE_ERR_ARG;
    const moe_status st = permute_check(ctx->err, X, dt, idx, T, k, h, E, align, Xp, Rcap, row_of, src_of, offsets, counts);
    if (st != MOE_OK) return st;
    const int64_t pairs = (int64_t)T * k;
    if (MOE_WS_RESERVED + moe_permute_ws_bytes(pairs, E) > ctx->ws_bytes)
        MOE_FAIL(ctx, MOE_ERR_WORKSPACE, "moe_permute: workspace %zu B < %zu B", ctx->ws_bytes,
                 MOE_WS_RESERVED + moe_permute_ws_bytes(pairs, E));
    permute_launch((hipStream_t)stream, X, dt, idx, T, k, h, E, align, Xp, Rcap, row_of, src_of, offsets, counts,
                   (int32_t*)((char*)ctx->ws + MOE_WS_RESERVED));
    MOE_LAUNCH_CHECK(ctx, "moe_permute kernels");
    return MOE_OK;
}

// ---------------------------------------------------------------------------
// moe_permute_static: moe_permute for callers that cannot allocate (no context, no hipMalloc anywhere on the path).
// The per-chunk histograms live in a file-scope device array instead of a context workspace.  Every GPU the library
// runs on holds its own copy of the array at its own address until the process ends; the address is looked up once
// per device, on the first call made with that device current, and kept.
// ---------------------------------------------------------------------------
#define PERMUTE_STATIC_BYTES (1u << 20)
#define PERMUTE_STATIC_MAX_DEVICES 64
static __device__ __align__(256) unsigned char scratch[PERMUTE_STATIC_BYTES];
static void* scratch_ptr_of_device[PERMUTE_STATIC_MAX_DEVICES];  // host copies of the per-device addresses (0 = not yet looked up)

extern "C" moe_status moe_permute_static(void* stream, const void* X, moe_dtype dt,
                                         const int32_t* idx, int T, int k, int h, int E, int align,
                                         void* Xp, int64_t Rcap,
                                         int32_t* row_of, int32_t* src_of, int32_t* offsets, int32_t* counts) {
    char* err = moe_ctxless_error();  // this host thread's message buffer, read back with moe_last_error(NULL)
    err[0] = 0;
    const moe_status st = permute_check(err, X, dt, idx, T, k, h, E, align, Xp, Rcap, row_of, src_of, offsets, counts);
    if (st != MOE_OK) return st;
    const size_t need = moe_permute_ws_bytes((int64_t)T * k, E);
    if (need > PERMUTE_STATIC_BYTES) {
        snprintf(err, 512, "moe_permute_static: ceil(T*k/%d)*E*4 = %zu B exceeds the fixed scratch of %u B; use moe_permute",
                 PERMUTE_CHUNK, need, PERMUTE_STATIC_BYTES);
        return MOE_ERR_WORKSPACE;
    }
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= PERMUTE_STATIC_MAX_DEVICES) {
        snprintf(err, 512, "moe_permute_static: no current device below %d (%s)", PERMUTE_STATIC_MAX_DEVICES, hipGetErrorString(e));
        return MOE_ERR_HIP;
    }
    // (two host threads racing here both look up the same address and store the same value)
    void* ptr = __atomic_load_n(&scratch_ptr_of_device[dev], __ATOMIC_ACQUIRE);
    if (!ptr) {
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            snprintf(err, 512, "moe_permute_static: hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
            return MOE_ERR_HIP;
        }
        __atomic_store_n(&scratch_ptr_of_device[dev], ptr, __ATOMIC_RELEASE);
    }
    permute_launch((hipStream_t)stream, X, dt, idx, T, k, h, E, align, Xp, Rcap, row_of, src_of, offsets, counts,
                   (int32_t*)ptr);
    e = hipGetLastError();
    if (e != hipSuccess) {
        snprintf(err, 512, "launch moe_permute_static kernels: %s", hipGetErrorString(e));
        return MOE_ERR_HIP;
    }
    return MOE_OK;
}

extern "C" moe_status moe_unpermute_combine(moe_ctx* ctx, void* stream, const void* O, moe_dtype dt,
                                            const int32_t* row_of, const float* prob, const void* residual,
                                            int T, int k, int h, void* Y) {
    if (!ctx) return MOE_ERR_ARG;
    if (!O || !row_of || !Y) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine: NULL pointer");
    if (T < 0 || k < 1 || k > COMBINE_MAX_K || h < 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine: need T>=0, 1<=k<=32, h>=1");
    if (dt != MOE_BF16 && dt != MOE_F32) MOE_FAIL(ctx, MOE_ERR_UNSUPPORTED, "moe_unpermute_combine: dtype must be bf16 or f32");
    const size_t row_bytes = (size_t)h * moe_dtype_size(dt);
    if (row_bytes % 16) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine: row size %zu B is not a multiple of 16", row_bytes);
    if (T == 0) return MOE_OK;
    hipStream_t s = (hipStream_t)stream;
    const int vec = (int)(row_bytes / 16);
    if (dt == MOE_BF16)
        hipLaunchKernelGGL(combine_kernel<false>, dim3(T), dim3(MOVE_THREADS), 0, s, (const u32x4_t*)O, row_of, prob,
                           (const u32x4_t*)residual, T, k, vec, (u32x4_t*)Y);
    else
        hipLaunchKernelGGL(combine_kernel<true>, dim3(T), dim3(MOVE_THREADS), 0, s, (const u32x4_t*)O, row_of, prob,
                           (const u32x4_t*)residual, T, k, vec, (u32x4_t*)Y);
    MOE_LAUNCH_CHECK(ctx, "combine_kernel");
    return MOE_OK;
}

extern "C" moe_status moe_unpermute_combine_bwd(moe_ctx* ctx, void* stream, const void* dY, const void* O,
                                                moe_dtype dt, const int32_t* row_of, const int32_t* src_of,
                                                const float* prob, int T, int k, int h, int64_t Rcap,
                                                void* dO, float* dprob) {
    if (!ctx) return MOE_ERR_ARG;
    if (!dY || !row_of || !src_of) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine_bwd: NULL pointer");
    if (!dO && !dprob) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine_bwd: neither dO nor dprob requested");
    if (dprob && !O) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine_bwd: dprob needs O");
    if (T < 0 || k < 1 || k > COMBINE_MAX_K || h < 1 || Rcap < 0)
        MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine_bwd: need T>=0, 1<=k<=32, h>=1, Rcap>=0");
    if (dt != MOE_BF16 && dt != MOE_F32) MOE_FAIL(ctx, MOE_ERR_UNSUPPORTED, "moe_unpermute_combine_bwd: dtype must be bf16 or f32");
    const size_t row_bytes = (size_t)h * moe_dtype_size(dt);
    if (row_bytes % 16) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine_bwd: row size %zu B is not a multiple of 16", row_bytes);
    hipStream_t s = (hipStream_t)stream;
    const int vec = (int)(row_bytes / 16);
    // (one launch: the padding rows' workgroups follow the tokens')
    const int64_t grid = T + (dO ? ceil_div64(Rcap, ZERO_ROWS) : 0);
    if (grid > 0x7fffffffLL) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_unpermute_combine_bwd: T and Rcap too large");
    if (grid > 0) {
        if (dt == MOE_BF16)
            hipLaunchKernelGGL(combine_bwd_kernel<false>, dim3((unsigned)grid), dim3(MOVE_THREADS), 0, s, (const u32x4_t*)dY,
                               (const u32x4_t*)O, row_of, prob, T, k, vec, (u32x4_t*)dO, dprob, src_of, Rcap);
        else
            hipLaunchKernelGGL(combine_bwd_kernel<true>, dim3((unsigned)grid), dim3(MOVE_THREADS), 0, s, (const u32x4_t*)dY,
                               (const u32x4_t*)O, row_of, prob, T, k, vec, (u32x4_t*)dO, dprob, src_of, Rcap);
    }
    MOE_LAUNCH_CHECK(ctx, "combine_bwd kernels");
    return MOE_OK;
}

// ---------------------------------------------------------------------------
// eq. (2) helpers: routing weights per permuted row, and the way back for their gradients
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gather_row_prob_kernel(const float* __restrict__ prob,
                                                              const int32_t* __restrict__ src_of, int64_t Rcap,
                                                              float* __restrict__ row_prob) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= Rcap) return;
    const int32_t j = src_of[r];
    row_prob[r] = j >= 0 ? prob[j] : 0.0f;
}

__global__ __launch_bounds__(256) void scatter_row_dprob_kernel(const float* __restrict__ part, int parts,
                                                                const int32_t* __restrict__ row_of, int64_t pairs,
                                                                float* __restrict__ dprob) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= pairs) return;
    const int32_t r = row_of[j];
    float acc = 0.f;
    if (r >= 0)
        for (int q = 0; q < parts; ++q) acc += part[(int64_t)r * parts + q];
    dprob[j] = acc;
}

extern "C" moe_status moe_gather_row_prob(moe_ctx* ctx, void* stream, const float* prob, const int32_t* src_of,
                                          int64_t Rcap, float* row_prob) {
    if (!ctx) return MOE_ERR_ARG;
    if (!prob || !src_of || !row_prob) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_gather_row_prob: NULL pointer");
    if (Rcap < 0 || Rcap > 0x7fffffffLL) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_gather_row_prob: need 0 <= Rcap < 2^31");
    if (Rcap == 0) return MOE_OK;
    hipLaunchKernelGGL(gather_row_prob_kernel, dim3((unsigned)ceil_div64(Rcap, 256)), dim3(256), 0, (hipStream_t)stream,
                       prob, src_of, Rcap, row_prob);
    MOE_LAUNCH_CHECK(ctx, "gather_row_prob_kernel");
    return MOE_OK;
}

extern "C" moe_status moe_scatter_row_dprob(moe_ctx* ctx, void* stream, const float* dprob_part, int parts,
                                            const int32_t* row_of, int T, int k, float* dprob) {
    if (!ctx) return MOE_ERR_ARG;
    if (!dprob_part || !row_of || !dprob) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_scatter_row_dprob: NULL pointer");
    if (parts < 1 || T < 0 || k < 1) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_scatter_row_dprob: need parts >= 1, T >= 0, k >= 1");
    const int64_t pairs = (int64_t)T * k;
    if (pairs == 0) return MOE_OK;
    hipLaunchKernelGGL(scatter_row_dprob_kernel, dim3((unsigned)ceil_div64(pairs, 256)), dim3(256), 0, (hipStream_t)stream,
                       dprob_part, parts, row_of, pairs, dprob);
    MOE_LAUNCH_CHECK(ctx, "scatter_row_dprob_kernel");
    return MOE_OK;
}
