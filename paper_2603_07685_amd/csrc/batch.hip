// Batches: a second handle on a context that keeps small calls and launches several of them together at its end (host code; the
// kernels are beside those that serve single calls).
#include <new>

#include "gemm.h"

extern "C" moe_status moe_batch_create(moe_ctx* ctx, moe_ctx** out) {
    if (!ctx || !out) return MOE_ERR_ARG;
    if (ctx->batch) MOE_FAIL(ctx, MOE_ERR_ARG, "moe_batch_create: a batch has no batches of its own");
    moe_ctx* c = new (std::nothrow) moe_ctx(*ctx);
    moe_batch* b = c ? new (std::nothrow) moe_batch() : nullptr;
    if (!b) {
        delete c;
        MOE_FAIL(ctx, MOE_ERR_HIP, "moe_batch_create: no host memory");
    }
    c->batch = b;
    c->err[0] = 0;
    *out = c;
    return MOE_OK;
}

extern "C" moe_status moe_batch_end(moe_ctx* batch, void* stream, int launch) {
    if (!batch) return MOE_ERR_ARG;
    (void)stream;   // (each call has its own)
    moe_batch* const b = batch->batch;
    if (!b) MOE_FAIL(batch, MOE_ERR_ARG, "moe_batch_end: not a batch");
    if (launch) batch_flush(b);
    b->n_gemm = b->n_quant = 0;
    b->partials = 0;
    MOE_LAUNCH_CHECK(batch, "calls of a batch");
    return MOE_OK;
}

extern "C" moe_status moe_batch_kept(moe_ctx* batch, int64_t* gemms, int64_t* quantisers) {
    if (!batch) return MOE_ERR_ARG;
    if (!batch->batch || !gemms || !quantisers) MOE_FAIL(batch, MOE_ERR_ARG, "moe_batch_kept: not a batch, or NULL pointer");
    *gemms = batch->batch->kept_gemm;
    *quantisers = batch->batch->kept_quant;
    return MOE_OK;
}

void batch_gemm(moe_ctx* ctx, gemm_job j) {
    moe_batch* const b = ctx->batch;
    // (pieces of two weight gradients of a launch need room side by side; a call's number of pieces does not depend on it)
    const size_t need = j.a.split_cap >= 2 ? (size_t)j.a.split_cap * j.a.N * j.a.K * sizeof(float) : 0;
    if (b->n_gemm == MOE_BATCH_MAX || (need && b->partials + need > ctx->ws_bytes - MOE_WS_RESERVED)) batch_flush(b);
    if (need) j.a.partials = (float*)((char*)j.a.partials + b->partials);
    b->partials += (need + 255) / 256 * 256;
    b->gemm[b->n_gemm++] = j;
    ++b->kept_gemm;
}

static void launch_alone(const gemm_job& j) {
    if (j.kind == JOB_BF16) gt_launch(j.s, j.mode, j.epi, j.f32, j.gath, j.tile, j.a);
    else if (j.kind == JOB_F32) {
        gt_jobs m;
        memset(&m, 0, sizeof(m));
        const int at = j.mode == GG_WGRAD ? 2 : 0;
        m.a[at] = j.a;
        for (int x = at + 1; x <= GT_JOBS; ++x) m.start[x] = (int)gf_blocks(j.mode, j.epi, j.a);
        gf_launch_jobs(j.s, j.mode == GG_FWD, j.epi, m);
    } else gq_launch(nullptr, j.s, j.mode, j.epi, j.f32, j.kind == JOB_MX, j.tile, j.a);
}

// Whether the weight gradients of a launch go in front of its data gradients: the tiles that take longer go first, so that the
// others fill what they leave.  A tile takes the call's contraction: N of a data gradient, an expert's rows of a weight gradient.
// Of several experts a hot one ends the launch, so their mean counts twice; of a single one 0.8 of its rows, as a data gradient's
// output phase is the longer (bf16 T 1538 h 1536 f 2624 E 6 k 1, shared 2624, 1538 rows against N 1536: 445 : 462 us a step with the
// weight gradients first).  A call that cuts experts into pieces walks no more rows than a piece's, but may have nothing
// to cut: counted as nothing, 40 drawn layers' backward passes of 24576 rows or fewer took 1.02 (equal loads) to 1.03 times as long
// (rank^-1.2), T 3699 h 192 f 256 E 9 k 4 85 : 72 us.
// Steps, us, data gradients always first : this: MXFP8 T 1920 h 512 f 256 E 8 k 8 160 : 145, T 8192 h 256 f 896 E 28, shared 896
// 410 : 356; fp8 T 1920 h 896 f 896 E 4 k 4 250 : 230; bf16 T 773 h 960 f 384 E 5 k 4, rank^-1.2, 104 : 94.  160 drawn layers with a
// shared expert, each with equal, by 30 % scattered and rank^-1.2 loads, mean: MXFP8 1.040, fp8 1.034, bf16 1.005; 159 others 1.018,
// 1.018, 1.005.  Weight gradients always first: 0.89 the least.  Each call on its own, which data gradients first made the better choice
// for some (up to 1.05): 0.95 in the mean, 1.017 the most, so that there is no size from which on a call is better alone.
static bool longer_first(gemm_job* const (&take)[GT_JOBS]) {
    double data = 0, weight = 0;
    for (int x = 0; x < GT_JOBS; ++x) {
        if (!take[x]) continue;
        const gg_args& a = take[x]->a;
        const double rows = a.E == 1 ? 0.8 * a.Rcap : 2.0 * a.Rcap / a.E;
        const double l = x < 2 ? a.N : a.split_cap >= 2 && a.split_rows < rows ? a.split_rows : rows;
        double& most = x < 2 ? data : weight;
        if (l > most) most = l;
    }
    return weight > data;
}

// The calls that go with the first one left: of its kind and stream; forward calls of one epilogue, or data gradients of one epilogue
// and weight gradients of one output type and gathered operand (as many kinds of a kernel as a layer has use for: beside SwiGLU's
// backward, fc2, a weight gradient may gather dC, beside the plain data gradient, fc1, A).
static void gemm_flush(gemm_job* jobs, int n) {
    auto fits = [](int epi, int gath) { return gath == 0 || gath == (epi == GG_EPI_SWIGLU_BWD ? 1 : 2); };
    for (int i = 0; i < n; ++i) {
        const gemm_job& first = jobs[i];
        if (first.done) continue;
        gemm_job* take[GT_JOBS] = {};
        const gemm_job *d = nullptr, *w = nullptr;   // the first data and weight gradient
        const bool fwd = first.mode == GG_FWD;
        int count = 0;
        for (int x = i; x < n; ++x) {
            gemm_job& j = jobs[x];
            if (j.done || j.s != first.s || j.kind != first.kind || (j.mode == GG_FWD) != fwd) continue;
            int at = count;
            if (fwd) {
                if (j.epi != first.epi) continue;
            } else if (j.mode == GG_DGRAD) {
                if (d ? j.epi != d->epi : w && !fits(j.epi, w->gath)) continue;
                at = d ? 1 : 0;
            } else {
                if (w ? j.f32 != w->f32 || j.gath != w->gath : d && !fits(d->epi, j.gath)) continue;
                at = w ? 3 : 2;
            }
            if (at >= GT_JOBS || take[at]) continue;
            if (j.mode == GG_DGRAD && !d) d = &j;
            if (j.mode == GG_WGRAD && !w) w = &j;
            take[at] = &j;
            ++count;
        }
        for (gemm_job* j : take)
            if (j) j->done = true;
        if (count == 1) {
            launch_alone(first);
            continue;
        }
        // The tiles of the call with the most of them serve all of a mode.  Where the routed experts' weight gradients are on one stage
        // buffer (gt_one_buffer) the shared expert's is walked on one too, at half its pace, but it is few tiles beside many and over
        // before them.  A backward pass of 30 drawn layers with a shared expert and such a pair (T 67-847, h 256-1472, f 320-1792, E
        // 11-61), this : the two in launches of their own : both on two buffers: 1 : 1.10 : 1.03 in the mean, at least 1.02 and 0.993;
        // us, T 847 h 1216 f 384 E 27 62.8 : 66.1 : 63.0; T 158 h 1152 f 640 E 13, shared 384, 41.3 : 51.8 : 42.9.
        const gemm_job *most = nullptr, *wmost = nullptr;
        for (const gemm_job* j : take) {
            const gemm_job*& m = j && j->mode == GG_WGRAD ? wmost : most;
            if (j && (!m || gt_blocks(j->mode, j->epi, 64, j->a) > gt_blocks(m->mode, m->epi, 64, m->a))) m = j;
        }
        const int tile = most ? most->tile : 3, wtile = wmost ? wmost->tile : 2;
        gt_jobs m;
        memset(&m, 0, sizeof(m));
        int64_t at = 0;
        for (int x = 0; x < GT_JOBS; ++x) {
            m.start[x] = (int)at;
            if (!take[x]) continue;
            const gemm_job& j = *take[x];
            m.a[x] = j.a;
            const int bm = j.mode == GG_WGRAD || tile == 2 ? 128 : 64;
            at += j.kind == JOB_BF16  ? gt_blocks(j.mode, j.epi, bm, j.a)
                  : j.kind == JOB_F32 ? gf_blocks(j.mode, j.epi, j.a)
                                      : gq_blocks(j.mode, j.epi, bm, j.a);
        }
        m.start[GT_JOBS] = (int)at;
        if (!fwd && d && w && longer_first(take)) m.turn = m.start[2];
        const int epi = fwd ? first.epi : d ? d->epi : w->gath == 1 ? GG_EPI_SWIGLU_BWD : GG_EPI_STORE;
        if (first.kind == JOB_BF16) gt_launch_jobs(first.s, fwd, epi, w && w->f32, w ? w->gath : 0, tile, wtile, m);
        else if (first.kind == JOB_F32) gf_launch_jobs(first.s, fwd, epi, m);
        else gq_launch_jobs(first.s, first.kind == JOB_MX, fwd, epi, w && w->f32, tile, m);
    }
}

void batch_flush(moe_batch* b) {
    gemm_flush(b->gemm, b->n_gemm);
    quant_flush(b->quant, b->n_quant);
    b->n_gemm = b->n_quant = 0;
    b->partials = 0;
}
