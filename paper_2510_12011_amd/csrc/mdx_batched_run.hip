// The batched form's time loop: per step the ionic update, right-hand side
// and initial residual of every instance, chunks of PCG iterations (five
// launches per iteration, or one persistent launch) and the residual
// replacement, replayed as HIP graphs when enabled; the host reads the
// per-instance records once per chunk.
#include "mdx_host.h"

namespace mdx {
namespace host {

// ---------------------------------------------------------------------------
// batched form: one time step's work up to the host check
// ---------------------------------------------------------------------------

BatchPtrs batch_ptrs(mdx_ctx *c)
{
    const Layout &L = c->L;
    BatchPtrs q;
    q.P = SellView{c->dev<int64_t>(L.slice_ptr), c->dev<int32_t>(L.col)};
    q.IM = iter_matrix(c);
    q.Mv = c->dev<double>(L.Mv);
    q.Kv = c->dev<double>(L.Kv);
    q.Av = c->dev<double>(L.Av);
    q.dinv = c->dev<double>(L.dinv);
    q.dinv32 = c->dev<float>(L.dinv32);
    q.b = c->dev<double>(L.b);
    q.u = ionic_nstates(c->ionic_kind) ? c->dev<double>(L.u) : nullptr;
    q.part0 = c->dev<double>(L.partial);
    q.part_pq = q.part0 + 3 * kPartialCap;
    q.part_rz = q.part0 + 6 * kPartialCap;
    q.r32 = c->dev<float>(L.r32);
    q.p32 = c->dev<float>(L.p32);
    q.q32 = c->dev<float>(L.q32);
    q.delta = c->dev<float>(L.delta);
    q.g32 = c->dev<float>(L.g32);
    q.bsc = c->dev<BScalars>(L.bsc);
    return q;
}

BParams batch_params(const mdx_ctx *c)
{
    return BParams{c->opts.atol, c->opts.rtol, c->opts.max_iter, c->opts.rr_interval,
                   c->opts.rel_mode};
}

constexpr int kPersistentSpinCap = 1000000;   // polls (about 60 ms) before a barrier gives up

void launch_persistent(mdx_ctx *c, hipStream_t st, const BatchPtrs &q, const BParams &bp)
{
    unsigned *bar = c->dev<unsigned>(c->L.pbar);
    launch_b_persistent(st, c->pseg, q.P, c->dev<float>(c->L.A32), q.dinv32, bp, q.p32, q.q32,
                        q.delta, q.r32, q.part_pq, q.part_rz, q.bsc, bar,
                        reinterpret_cast<int *>(bar + c->n_inst), kPersistentSpinCap);
}

// the persistent iteration's barrier timed out (its groups were not all
// resident); the flag arrives with the instance records (fetch_bscalars)
mdx_status persistent_fault(mdx_ctx *c)
{
    if (*reinterpret_cast<const int *>(c->bsc_host + c->n_inst))
        return fail(c, MDX_ERR_DEVICE,
                    "a barrier of the persistent batched iteration timed out (%d workgroups; "
                    "not all were resident)", c->pseg.groups);
    return MDX_OK;
}

// right-hand side and initial residual; keep_r: for the single-launch solve
void enqueue_rhs(mdx_ctx *c, hipStream_t st, const BatchPtrs &q, bool keep_r)
{
    launch_b_rhs_init(st, c->seg, q.P, q.Mv, q.Kv, q.dinv, q.dinv32, step_params(c),
                      c->dev<double>(c->L.gv), c->vec(2), q.b, q.r32, q.delta, q.part0,
                      use_nt(c, 20.0 * slots(c)), keep_r);
    if (keep_r) return;
    launch_b_init_finalize(st, c->seg, q.part0, batch_params(c), q.bsc);
    launch_b_set_direction(st, c->seg, q.dinv32, q.r32, q.p32, q.bsc);
}

// The solve as one launch where the instances fit on chip; the tunings that
// choose among the streaming kernels select those.
bool batch_onchip(const mdx_ctx *c, bool profiling)
{
    return c->onchip_ready && c->onchip.shape[2] && c->onchip_polls > 0 && !c->onchip_off &&
           !c->persistent && !c->layout_set && !profiling;
}

void enqueue_onchip(mdx_ctx *c, hipStream_t st, const BatchPtrs &q)
{
    OnchipBatch a{};
    a.map = c->onchip_map;
    a.grp = c->dev<int4>(c->L.oc_team);
    a.part = q.part0;
    a.part_groups = c->seg.groups;
    a.inst_grp = c->seg.inst_grp;
    a.bp = batch_params(c);
    a.r = q.b;
    a.x = c->vec(2);
    a.dinv = q.dinv;
    a.r32 = q.r32;
    a.dinv32 = q.dinv32;
    a.zb = c->dev<float>(c->L.oc_z);
    a.words = c->dev<unsigned long long>(c->L.words);
    a.polls = c->onchip_polls;
    a.once = c->onchip_give_up.exchange ? c->onchip_give_up.group : -1;
    a.lanes = c->fmt <= 1 ? c->lpr : 1;   // sliced ELL or CSR; 4-entry loads add in column order
    a.turn = c->dev<int32_t>(c->L.oc_turn);
    a.sc = q.bsc;
    launch_onchip_batch(st, c->onchip, a);
}

// ionic update at V (Vprev the one before it); times: the activation and
// repolarisation times of the step that gave V, recorded with it
void enqueue_ionic(mdx_ctx *c, hipStream_t st, const BatchPtrs &q, const double *V,
                   const double *Vprev, const double *istim, const int32_t *guard,
                   const StepTimes &times)
{
    const GatherOut gather{c->dev<double>(c->L.gv), Vprev, c->cm, c->dt, c->opts.warm_start};
    if (c->opts.precision == MDX_PREC_MIXED_GATES32)
        launch_ionic_step_mixed(st, c->ionic_kind, c->ionic_params.data(), c->npad, c->npad, c->dt,
                                c->cm, V, q.u, q.g32, istim, nullptr, row_mask(c), guard, times,
                                gather);
    else
        launch_ionic_step(st, c->ionic_kind, c->ionic_params.data(), c->npad, c->npad, c->dt, c->cm,
                          V, q.u, istim, nullptr, 0, row_mask(c), guard, times, gather);
}

// right-hand side and initial residual, then the solve in one launch (iters <
// 0) or `iters` PCG iterations of every running instance and one
// residual-replacement pass.  With `timed`, event pairs bracket the SpMV
// launches.
void enqueue_batched_step(mdx_ctx *c, hipStream_t st, int iters, bool timed)
{
    const BatchPtrs q = batch_ptrs(c);
    const BParams bp = batch_params(c);
    double *X = c->vec(2);
    enqueue_rhs(c, st, q, iters < 0);
    if (iters < 0) {
        enqueue_onchip(c, st, q);
        return;
    }
    if (c->persistent) {
        launch_persistent(c, st, q, bp);
        iters = 0;
    }
    for (int i = 0; i < iters; ++i) {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (timed && 2 * i + 1 < (int)c->ev.size()) {
            e0 = c->ev[2 * i];
            e1 = c->ev[2 * i + 1];
        }
        launch_b_iteration(st, c->seg, q.IM, bp, q.dinv32, q.p32, q.q32, q.delta, q.r32, q.part_pq,
                           q.part_rz, q.bsc, e0, e1);
    }
    launch_b_replacement(st, c->seg, q.P, bp, q.Av, X, q.delta, q.b, q.dinv, q.dinv32, q.r32, q.p32,
                         q.part0, q.bsc, use_nt(c, 12.0 * slots(c)));
}

mdx_status fetch_bscalars(mdx_ctx *c, hipStream_t st)
{
    mdx_ctx *ctx = c;   // for HIPCHK
    HIPCHK(hipMemcpyAsync(c->bsc_host, c->dev<BScalars>(c->L.bsc), sizeof(BScalars) * c->n_inst,
                          hipMemcpyDeviceToHost, st));
    if (c->persistent)
        HIPCHK(hipMemcpyAsync(c->bsc_host + c->n_inst, c->dev<unsigned>(c->L.pbar) + c->n_inst,
                              sizeof(int), hipMemcpyDeviceToHost, st));
    auto w0 = std::chrono::steady_clock::now();
    HIPCHK(hipStreamSynchronize(st));
    c->stats.host_wait_seconds +=
        std::chrono::duration<double>(std::chrono::steady_clock::now() - w0).count();
    return MDX_OK;
}

bool all_done(const mdx_ctx *c)
{
    for (int i = 0; i < c->n_inst; ++i)
        if (!c->bsc_host[i].done) return false;
    return true;
}

mdx_status run_batched(mdx_ctx *ctx, int64_t n_steps, int64_t out_every, double *v_out)
{
    if (ctx->opts.precision == MDX_PREC_FP64)
        return fail(ctx, MDX_ERR_UNSUPPORTED,
                    "a batched context runs the mixed-precision solver (MDX_PREC_MIXED)");
    if (ctx->opts.warm_start == MDX_WS_MLP || ctx->rec_X)
        return fail(ctx, MDX_ERR_UNSUPPORTED, "no learned warm start or recorder in a batched context");
    // graphs cannot be captured on the legacy default stream: use an own one
    hipStream_t st = ctx->stream;
    if (!st) {
        if (!ctx->own_stream) HIPCHK(hipStreamCreateWithFlags(&ctx->own_stream, hipStreamNonBlocking));
        HIPCHK(hipStreamSynchronize(ctx->stream));
        st = ctx->own_stream;
    }
    const Layout &L = ctx->L;
    const BatchPtrs q = batch_ptrs(ctx);
    const BParams bp = batch_params(ctx);
    const int max_iter = ctx->opts.max_iter;
    double *istim_dev = ctx->dev<double>(L.istim);
    Scalars *sc = ctx->dev<Scalars>(L.scalars);
    mdx_status result = MDX_OK;
    ctx->iters_hist.clear();
    ctx->inst_iters_hist.clear();
    int64_t n_out = 0;
    auto t_start = std::chrono::steady_clock::now();

    // a step's activation and repolarisation times are recorded by the next
    // step's ionic update, or by a launch of their own
    double *lat = ctx->dev<double>(L.lat), *lrt = ctx->dev<double>(L.lrt);
    int32_t *ready = ctx->dev<int32_t>(L.oc_turn) + ctx->n_inst;
    bool times_due = false;
    bool ionic_queued = false;   // this step's ionic update was queued by the previous step
    auto record_times = [&]() {
        if (times_due)
            launch_epilogue(st, ctx->npad, (double)ctx->step * ctx->dt, ctx->vec(1), ctx->vec(0),
                            lat, lrt, sc);
        times_due = false;
    };

    OnchipCus cus(ctx);
    for (int64_t j = 0; j < n_steps; ++j) {
        const int64_t k = ctx->step;
        bool any_stim = false;
        if (mdx_status e = update_stimulus(ctx, st, k, any_stim)) return e;
        double *X = ctx->vec(2);
        const bool profiling = ctx->profile_every > 0 && k % ctx->profile_every == 0;
        const bool onchip = batch_onchip(ctx, profiling);
        const int C = onchip ? -1 : std::max(1, std::min(ctx->last_iters, max_iter));
        // (six launches: a replay of them as a graph costs 8-10 us a step more)
        if (ctx->use_graph && !profiling && !onchip) {
            record_times();   // the replayed ionic update does not
            const std::pair<int, int> key{ctx->persistent ? -1 : C, ctx->vb[0]};
            auto it = ctx->graphs.find(key);
            if (it == ctx->graphs.end()) {
                hipGraph_t g = nullptr;
                HIPCHK(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
                enqueue_ionic(ctx, st, q, ctx->vec(0), ctx->vec(1), istim_dev, nullptr, StepTimes{});
                enqueue_batched_step(ctx, st, C, false);
                HIPCHK(hipStreamEndCapture(st, &g));
                hipGraphExec_t ex = nullptr;
                hipError_t ie = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
                (void)hipGraphDestroy(g);
                HIPCHK(ie);
                it = ctx->graphs.emplace(key, ex).first;
            }
            if (ctx->persistent)
                if (mdx_status e = cus.enter(-1, 1)) return e;
            HIPCHK(hipGraphLaunch(it->second, st));
        } else {
            if (!ionic_queued) {
                StepTimes times;
                if (times_due)
                    times = StepTimes{(double)k * ctx->dt, ctx->vec(1), lat, lrt, sc};
                times_due = false;
                enqueue_ionic(ctx, st, q, ctx->vec(0), ctx->vec(1), any_stim ? istim_dev : nullptr,
                              nullptr, times);
            }
            if (onchip)
                if (mdx_status e = cus.enter(ctx->onchip.groups, ctx->onchip.per_cu[2])) return e;
            if (ctx->persistent)
                if (mdx_status e = cus.enter(-1, 1)) return e;
            enqueue_batched_step(ctx, st, C, profiling);
        }
        HIPCHK(hipGetLastError());
        int units = C;
        ionic_queued = false;
        if (onchip) {
            // the records published, and the next step's ionic update queued
            // behind (it acts only if every instance is done), so that the
            // device is busy while the host reads them and queues the rest
            launch_b_publish(st, q.bsc, ctx->n_inst, ctx->bsc_host_dev, ready, sc, ctx->pub_dev,
                             ++ctx->pub_seq);
            if (j + 1 < n_steps) {
                bool any_next = false;
                if (mdx_status e = update_stimulus(ctx, st, k + 1, any_next)) return e;
                enqueue_ionic(ctx, st, q, X, ctx->vec(0), any_next ? istim_dev : nullptr, ready,
                              StepTimes{(double)(k + 1) * ctx->dt, ctx->vec(0), lat, lrt, sc});
                ionic_queued = true;
            }
            HIPCHK(hipGetLastError());
            auto w0 = std::chrono::steady_clock::now();
            if (mdx_status e = wait_published(ctx, st, ctx->pub_seq)) return e;
            ctx->stats.host_wait_seconds +=
                std::chrono::duration<double>(std::chrono::steady_clock::now() - w0).count();
            cus.ended();
            units = 0;
            for (int i = 0; i < ctx->n_inst; ++i)
                if (ctx->bsc_host[i].gave_up) ctx->onchip_off = true;
            if (ctx->onchip_off) {   // the step's solve again, by the streaming kernels
                ionic_queued = false;
                enqueue_rhs(ctx, st, q, false);
                if (mdx_status e = fetch_bscalars(ctx, st)) return e;
            }
        } else {
            if (mdx_status e = fetch_bscalars(ctx, st)) return e;
            cus.ended();
            if (ctx->persistent)
                if (mdx_status e = persistent_fault(ctx)) return e;
        }
        while (!all_done(ctx) && units < max_iter + 1) {
            hipEvent_t e0 = nullptr, e1 = nullptr;
            if (profiling && 2 * units + 1 < (int)ctx->ev.size()) {
                e0 = ctx->ev[2 * units];
                e1 = ctx->ev[2 * units + 1];
            }
            if (ctx->persistent) {
                if (mdx_status e = cus.enter(-1, 1)) return e;
                launch_persistent(ctx, st, q, bp);
            } else {
                launch_b_iteration(st, ctx->seg, q.IM, bp, q.dinv32, q.p32, q.q32, q.delta, q.r32,
                                   q.part_pq, q.part_rz, q.bsc, e0, e1);
            }
            launch_b_replacement(st, ctx->seg, q.P, bp, q.Av, X, q.delta, q.b, q.dinv, q.dinv32, q.r32,
                                 q.p32, q.part0, q.bsc, use_nt(ctx, 12.0 * slots(ctx)));
            HIPCHK(hipGetLastError());
            ++units;
            if (mdx_status e = fetch_bscalars(ctx, st)) return e;
            cus.ended();
            if (ctx->persistent)
                if (mdx_status e = persistent_fault(ctx)) return e;
        }
        if (!all_done(ctx))
            return fail(ctx, MDX_ERR_STATE, "batched solve of step %lld did not finish",
                        (long long)k);
        int max_it = 0, step_iters = 0;
        bool failed = false;
        double bytes = 0.0;
        for (int i = 0; i < ctx->n_inst; ++i) {
            const BScalars &b = ctx->bsc_host[i];
            if (b.nonfinite)
                return fail(ctx, MDX_ERR_NONFINITE,
                            "non-finite value in the solve of instance %d, step %lld", i,
                            (long long)k);
            const int itv = b.failed ? -1 : b.iters;
            ctx->inst_iters_hist.push_back(itv);
            max_it = std::max(max_it, b.it);
            if (itv < 0) {
                failed = true;
                ctx->stats.not_converged++;
            } else {
                step_iters = std::max(step_iters, itv);
            }
            ctx->stats.cg_iters_total += b.it;
            const int64_t ni = ctx->inst_node_ptr[i + 1] - ctx->inst_node_ptr[i];
            bytes += (double)b.it * (8.0 * (double)ctx->inst_nnz[i] + 8.0 * (double)ni);
        }
        ctx->stats.cg_iters_max = std::max<int64_t>(ctx->stats.cg_iters_max, max_it);
        ctx->last_iters = max_it;
        if (failed) result = MDX_WARN_NOT_CONVERGED;
        // the persistent iteration has no separate SpMV launches to time
        if (profiling && !ctx->persistent) {
            const int timed = std::min(units, (int)ctx->ev.size() / 2);
            for (int u_ = 0; u_ < timed; ++u_) {
                float ms = 0.0f;
                HIPCHK(hipEventElapsedTime(&ms, ctx->ev[2 * u_], ctx->ev[2 * u_ + 1]));
                ctx->stats.spmv_seconds += 1e-3 * ms;
                ctx->stats.spmv_timed++;
            }
            if (timed == units) {
                ctx->stats.spmv_work += units;
                ctx->stats.spmv_bytes += bytes;
            }
        }
        times_due = !ionic_queued;
        int old_prev = ctx->vb[1];
        ctx->vb[1] = ctx->vb[0];
        ctx->vb[0] = ctx->vb[2];
        ctx->vb[2] = old_prev;
        ctx->step++;
        ctx->iters_hist.push_back(failed ? -1 : step_iters);
        ctx->stats.steps++;
        if (out_every > 0 && (j + 1) % out_every == 0 && v_out) {
            HIPCHK(hipStreamSynchronize(st));
            if (mdx_status e = copy_vec_out(ctx, ctx->vec(0), v_out + n_out * ctx->n)) return e;
            ++n_out;
        }
    }
    record_times();
    HIPCHK(hipMemcpyAsync(ctx->sc_host, sc, sizeof(Scalars), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    ctx->stats.step_loop_seconds +=
        std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
    if (ctx->sc_host->nonfinite || ctx->sc_host->nonfinite_v)
        return fail(ctx, MDX_ERR_NONFINITE, "non-finite V after step %lld", (long long)ctx->step);
    return result;
}

}  // namespace host
}  // namespace mdx
