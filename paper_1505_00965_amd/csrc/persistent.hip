// Persistent all-levels sampler: every level (and payoff) of one MLMC
// iteration in a single launch.
//
// Levels are independent (Sec. 5, after eq. (eq:Yldef)), so one iteration's
// work is a set of (payoff, level, sample range) items.  Their costs differ by
// orders of magnitude: level l costs M^l + M^(l-1) steps per sample (the
// paper's cost measure, Sec. 3) and N_l falls with l.  A plan kernel cuts the
// outstanding samples into items of roughly equal cost, deepest levels first
// (longest-processing-time order), and a grid that about fills the device takes
// items (block b item b first, then from its group's counter) until none are left, so
// cheap levels fill in around the long deep-level items.  GBM levels with too few paths to fill the
// device run each path on several lanes (process_split), with the per-level
// launch's rule on the level's count.  The problem's parameters live in
// device memory and are uploaded when they change; the sampler reads the plan
// that the launch before it wrote: a batch is plan, sampler and publication,
// the adaptive driver's run two launches per iteration (the sampler, then one
// block that absorbs the batch and plans the next).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "context.hpp"
#include "driver.hpp"
#include "driver_dev.hpp"
#include "persistent.hpp"
#include "trace.hpp"

namespace mlmc {

// Outstanding samples and first indices per (slot, level) of one batch, and
// the blocks that its sampler is launched with.
struct BatchRequest {
    double dN[kPairs], offset[kPairs];
    unsigned blocks;
};

__global__ __launch_bounds__(64) void plan_kernel(const BatchDesc* d, BatchRequest q)
{
    __shared__ BatchRequest s;
    s.dN[threadIdx.x] = q.dN[threadIdx.x];
    s.offset[threadIdx.x] = q.offset[threadIdx.x];
    __syncthreads();
    PlanArgs a = plan_args(d);
    clear_heads(a);
    a.grid_blocks = a.fit_blocks = q.blocks;
    plan_body(a, s.dN, s.offset);
}

// The plan of a randomised estimate: the drawn samples per level, from 0.
__global__ __launch_bounds__(64) void plan_counts_kernel(const BatchDesc* d, const unsigned long long* counts)
{
    __shared__ BatchRequest s;
    unsigned long long n = 0;
    for (int k = 0; k < kCountCopies && threadIdx.x < kMaxLevels; ++k) n += counts[k * kMaxLevels + threadIdx.x];
    s.dN[threadIdx.x] = (double)n;
    s.offset[threadIdx.x] = 0.0;
    __syncthreads();
    const PlanArgs a = plan_args(d);
    clear_heads(a);
    plan_body(a, s.dN, s.offset);
}

// The adaptive run's first kernel when its spread groups are not known to
// hold zeros: a fresh state (n_pilot samples outstanding on levels
// 0..L_min) built in LDS and planned from there (the plan also zeroes the
// dispensers), then the state written out and the spread groups cleared (the
// stores last: nothing waits for them).
__global__ __launch_bounds__(256) void driver_start_kernel(DriverState* st, LevelAcc* spread,
                                                           DriverInit c, const BatchDesc* d)
{
    __shared__ DriverState s;
    const PlanArgs pa = plan_args(d);
    clear_heads(pa);
    init_state(s, c);   // ends with a barrier
    plan_body(pa, s.dN, s.n);
    constexpr int kWords = sizeof(DriverState) / 8;
    const unsigned long long* w = (const unsigned long long*)&s;
    unsigned long long* dst = (unsigned long long*)st;
    for (int i = threadIdx.x; i < kWords; i += blockDim.x) dst[i] = w[i];
    clear_groups(spread, kMaxLevels - 1);
}

// One iteration's end: sum the spread groups, absorb the batch, re-plan
// (update_state), plan the next batch's items from the new state in LDS
// (nothing for a finished one, whose result the host waits for), then write
// the state back and clear the groups.  The host reads the
// update count every iteration and the state once, at the end: the mirror
// is written whole by the finishing update only.  Every load goes out at
// the start, none waiting for another: the state (one word per thread), the
// records of every level's spread group (8 waves, levels w and w + 8; the
// groups past the sampled levels hold zeros), the descriptor's plan fields
// and the state's level count and done flag; the stores come last.  A
// finished state has no outstanding samples: the plan its finishing update
// wrote is empty, so a sampler launched after it does nothing, and the
// update launched after it (the host queues exactly one iteration past the
// last) prepares the next run's start instead.
__global__ __launch_bounds__(512) void driver_update_plan_kernel(DriverState* st, DriverState* mirror,
                                                                 LevelAcc* spread, const BatchDesc* d)
{
    constexpr int kWords = sizeof(DriverState) / 8;
    static_assert(kWords <= 512, "one state word per thread");
    static_assert(kMaxLevels == 16 && kSpread == 64, "8 waves, two levels' groups each");
    __shared__ DriverState s;
    __shared__ GroupSums g;
    const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
    const unsigned long long word =
        threadIdx.x < (unsigned)kWords ? ((const unsigned long long*)st)[threadIdx.x] : 0ull;
    const LevelAcc& r0 = spread[wave * kSpread + lane];
    const LevelAcc& r1 = spread[(wave + 8) * kSpread + lane];
    double y0 = r0.sum[0], q0 = r0.sum[1], c0 = (double)r0.n_nonfinite;
    double y1 = r1.sum[0], q1 = r1.sum[1], c1 = (double)r1.n_nonfinite;
    // the levels the batch sampled: 0..L of the stored state
    const int L0 = __builtin_amdgcn_readfirstlane(st->L);
    const int done = __builtin_amdgcn_readfirstlane(st->done);
    const PlanArgs pa = plan_args(d);
    // only the plan reads the descriptor's fields, at the end: taking them
    // into registers here keeps their loads beside the others
    asm volatile("" ::"s"(pa.L), "s"(pa.M), "s"(pa.nslots), "s"(pa.dim), "s"(pa.split_ok), "s"(pa.num_cu),
                 "s"(pa.grid_blocks), "s"(pa.fit_blocks), "s"(pa.chunk), "s"(pa.block), "s"(pa.cond_slots), "s"(pa.plan),
                 "s"(pa.head), "s"(pa.split));
    clear_heads(pa);
    // the sums of each group, in record order as the per-level form folds them
    y0 = wave_sum(y0);
    q0 = wave_sum(q0);
    c0 = wave_sum(c0);
    if (L0 >= 8) {   // above it the second level's records are zeros
        y1 = wave_sum(y1);
        q1 = wave_sum(q1);
        c1 = wave_sum(c1);
    }
    if (done) {   // block-uniform
        // The update queued past a run's finishing one: the state becomes
        // the fresh state of a next run of this descriptor and the plan its
        // pilot batch (the start kernel's work; the groups already hold
        // zeros), so that run can start with its sampler.  The mirror, which
        // holds the finished run's result, is not touched.
        init_state(s, d->init);   // ends with a barrier
        plan_body(pa, s.dN, s.n);
        if (threadIdx.x < (unsigned)kWords)
            ((unsigned long long*)st)[threadIdx.x] = ((const unsigned long long*)&s)[threadIdx.x];
        return;
    }
    if (lane == 0) {
        g.y[wave] = y0;
        g.y2[wave] = q0;
        g.c[wave] = c0;
        g.y[wave + 8] = y1;
        g.y2[wave + 8] = q1;
        g.c[wave + 8] = c1;
    }
    if (threadIdx.x < (unsigned)kWords) ((unsigned long long*)&s)[threadIdx.x] = word;
    __syncthreads();
    // absorb the groups into the batch records (held at zero between updates)
    if ((int)threadIdx.x <= L0) {
        const int l = (int)threadIdx.x;
        s.batch[l].sum[0] += g.y[l];
        s.batch[l].sum[1] += g.y2[l];
        s.batch[l].n_nonfinite += (unsigned long long)g.c[l];
    }
    __syncthreads();
    update_state(s);   // ends with a barrier
    if (s.done) plan_nothing(pa);
    else plan_body(pa, s.dN, s.n);
    publish_state(st, mirror, s, false);
    clear_groups(spread, L0);
}

extern template PersistentFn pick_persistent_variant<kGBM>(int, int, int, bool);
extern template PersistentFn pick_persistent_variant<kGBMMil>(int, int, int, bool);
extern template PersistentFn pick_persistent_variant<kHeston>(int, int, int, bool);

// variant: sampler_variant() of the model (GBM Euler, GBM Milstein, Heston);
// payoff: the kind every slot holds, or kAnyPayoff; cv: with the tabulated
// control variate (nullptr where that kernel does not exist).
static PersistentFn pick_persistent(int variant, int M, int ppt, int payoff, bool cv = false)
{
    if (variant == kGBM) return pick_persistent_variant<kGBM>(M, ppt, payoff, cv);
    if (variant == kGBMMil) return pick_persistent_variant<kGBMMil>(M, ppt, payoff, cv);
    return pick_persistent_variant<kHeston>(M, ppt, payoff, cv);
}

// A problem's descriptor and the plan made from it.  Batches and driver runs
// have one each: a batch between two runs of one problem leaves the plan that
// the first run's end prepared for the second, and neither uploads again.
struct PlannedProblem {
    BatchDesc* d_desc = nullptr;
    BatchDesc* h_desc = nullptr;
    PlanTable* d_plan = nullptr;
    unsigned* d_head = nullptr;       // dispensers
    unsigned* d_split = nullptr;      // lanes per path [kMaxSlots][kMaxLevels]
    BatchDesc last_desc;              // the bytes of the last descriptor upload
    // 0: unknown; 1: the device descriptor holds last_desc
    int desc_state = 0;
};

// Batch spread groups [kMaxSlots][kMaxLevels][kSpread], and behind them the
// level draws of a randomised estimate: cleared by one launch where both are to be.
constexpr int kGroupRecords = kMaxSlots * kMaxLevels * kSpread;
constexpr int kCountRecords = (int)(sizeof(unsigned long long) * kCountCopies * kMaxLevels / sizeof(LevelAcc));
static_assert(kCountRecords * sizeof(LevelAcc) == sizeof(unsigned long long) * kCountCopies * kMaxLevels,
              "the counts are whole records");

// State of the persistent form; the buffers are parts of the context's.
struct PersistentBufs {
    PlannedProblem run, batch;
    LevelAcc* d_acc = nullptr;
    bool acc_clean = false;           // they hold zeros (publish_groups clears what it folds)
    unsigned long long* d_counts = nullptr;
    bool counts_clean = false;        // they hold zeros
};

static PersistentBufs* bufs_of(mlmc_ctx* ctx);

struct PersistentShape {
    int block, ppt, blocks_per_cu, fit_per_cu;
};

static int persistent_ppt(const mlmc_ctx* ctx) { return ctx->persist_ppt ? ctx->persist_ppt : 1; }

// The launch of sampler `fn` with `lds` bytes of dynamic LDS: the shape that
// was set, or five blocks of 256 per compute unit -- 346 us for the estimate
// at RMSE 2e-5 S0 against 353 with four and 366 with eight -- and how many of
// those a unit holds at once (see kItems).
static PersistentShape persistent_shape(const mlmc_ctx* ctx, PersistentFn fn, size_t lds)
{
    PersistentShape s;
    s.block = ctx->persist_block ? ctx->persist_block : 256;
    s.ppt = persistent_ppt(ctx);
    s.blocks_per_cu = s.fit_per_cu = ctx->persist_bpc;
    if (!s.blocks_per_cu) {
        const int fit = resident_blocks((const void*)fn, s.block, lds);
        s.blocks_per_cu = 5;
        s.fit_per_cu = fit > 0 ? std::min(fit, 5) : 5;
    }
    return s;
}

// The persistent form's buffers cut from the context's two blocks (from null:
// their sizes alone).
static PersistentBufs cut_bufs(char* d, char* h, size_t* d_bytes, size_t* h_bytes)
{
    size_t da = 0, ha = 0;
    auto cut = [](char* base, size_t& at, size_t bytes) {
        char* p = base + at;
        at += (bytes + 255) / 256 * 256;
        return p;
    };
    PersistentBufs b;
    for (PlannedProblem* q : {&b.run, &b.batch}) {
        q->d_desc = (BatchDesc*)cut(d, da, sizeof(BatchDesc));
        q->h_desc = (BatchDesc*)cut(h, ha, sizeof(BatchDesc));
        q->d_plan = (PlanTable*)cut(d, da, sizeof(PlanTable));
        q->d_head = (unsigned*)cut(d, da, sizeof(unsigned) * kHeads * kHeadStride);
        q->d_split = (unsigned*)cut(d, da, sizeof(unsigned) * kMaxSlots * kMaxLevels);
    }
    b.d_acc = (LevelAcc*)cut(d, da, sizeof(LevelAcc) * (kGroupRecords + kCountRecords));
    b.d_counts = (unsigned long long*)(b.d_acc + kGroupRecords);
    if (d_bytes) *d_bytes = da;
    if (h_bytes) *h_bytes = ha;
    return b;
}

size_t persistent_device_bytes()
{
    size_t n;
    cut_bufs(nullptr, nullptr, &n, nullptr);
    return n;
}

size_t persistent_host_bytes()
{
    size_t n;
    cut_bufs(nullptr, nullptr, nullptr, &n);
    return n;
}

static mlmc_status ensure_bufs(mlmc_ctx* ctx)
{
    if (ctx->persist) return MLMC_OK;
    ctx->persist = new (std::nothrow) PersistentBufs(cut_bufs(ctx->d_persist, ctx->h_persist, nullptr, nullptr));
    if (!ctx->persist) return fail(ctx, MLMC_ENOMEM, "host allocation failed");
    return MLMC_OK;
}

static PersistentBufs* bufs_of(mlmc_ctx* ctx) { return (PersistentBufs*)ctx->persist; }

void free_persistent(mlmc_ctx* ctx)
{
    delete bufs_of(ctx);
    ctx->persist = nullptr;
}

// Fill the host copy of the descriptor (parameters for every slot and level).
// A driver run passes the fresh state's configuration, a batch nullptr.
static void fill_desc(mlmc_ctx* ctx, const PlannedProblem& q, const PersistentShape& s, const mlmc_model& m,
                      const mlmc_payoff* p, int np, int L, int M, LevelAcc* acc, const DriverInit* init)
{
    BatchDesc* h = q.h_desc;
    std::memset(h, 0, sizeof(*h));
    h->nslots = np;
    h->L = L;
    h->M = M;
    h->dim = m.kind == MLMC_HESTON ? 2 : 1;
    for (int k = 0; k < np; ++k) {
        h->payoff_kind[k] = p[k].kind;
        for (int l = 0; l <= L; ++l) h->params[k][l] = make_step_params<float>(m, p[k], l, M);
    }
    h->acc = acc;
    h->plan = q.d_plan;
    h->head = q.d_head;
    h->grid_blocks = (unsigned)(ctx->num_cu * s.blocks_per_cu);
    h->fit_blocks = (unsigned)(ctx->num_cu * s.fit_per_cu);
    h->chunk = (unsigned)(s.block * s.ppt);
    h->split = q.d_split;
    h->split_ok = m.kind == MLMC_GBM && !m.antithetic;
    h->num_cu = ctx->num_cu;
    h->block = (unsigned)s.block;
    if (init) h->init = *init;
}

// Copy the host descriptor to the device unless the last upload from this
// context carried the same bytes (repeated runs of one problem skip it: a
// driver run passes its seed with each launch, not in the descriptor).
// *uploaded (if given) tells which.
static mlmc_status upload_desc(mlmc_ctx* ctx, PlannedProblem& q, bool* uploaded = nullptr)
{
    if (uploaded) *uploaded = false;
    if (q.desc_state == 1 && std::memcmp(&q.last_desc, q.h_desc, sizeof(BatchDesc)) == 0) return MLMC_OK;
    if (uploaded) *uploaded = true;
    q.desc_state = 0;
    MLMC_HIP(ctx, hipMemcpyAsync(q.d_desc, q.h_desc, sizeof(BatchDesc), hipMemcpyHostToDevice, ctx->stream));
    std::memcpy(&q.last_desc, q.h_desc, sizeof(BatchDesc));
    q.desc_state = 1;
    return MLMC_OK;
}

// mlmc_run with persistent = 1: the start kernel (fresh state, pilot plan),
// then per driver iteration the all-levels sampler and the update-and-plan
// block, as plain launches on the context's stream.
mlmc_status run_persistent(mlmc_ctx* ctx, const mlmc_model& m, const mlmc_payoff& p,
                           const mlmc_run_opts& o, DriverState* d_st, DriverState* h_st,
                           const DriverInit& init, bool prepared)
{
    if (o.precision != 32) return fail(ctx, MLMC_EINVAL, "the persistent form runs fp32 paths");
    if (o.cv) {
        if (!cv_tabulated(o.cv))
            return fail(ctx, MLMC_EINVAL,
                        "the device-planned form takes the tabulated control variate (mlmc_cv_set_tabulated)");
        if (m.scheme != MLMC_EULER || m.antithetic)
            return fail(ctx, MLMC_EINVAL, "the control variate runs with plain Euler paths");
        if (p.kind == MLMC_DIGITAL_COND)
            return fail(ctx, MLMC_EINVAL, "the control variate takes the four plain payoffs");
        if (cv_in_dim(o.cv) != (m.kind == MLMC_HESTON ? 3 : 2))
            return fail(ctx, MLMC_EINVAL, "network inputs do not match the model (2: GBM, 3: Heston)");
    }
    mlmc_status st = ensure_bufs(ctx);
    if (st) return st;
    PlannedProblem& prob = bufs_of(ctx)->run;
    const auto sampler = pick_persistent(sampler_variant(m), o.M, persistent_ppt(ctx), p.kind, o.cv != nullptr);
    if (!sampler) return fail(ctx, MLMC_EINVAL, "no persistent sampler for this model and payoff");
    const float *cv_table = nullptr, *cv_phi0 = nullptr;
    TableSpec cv_spec{};
    size_t lds = 0;
    if (o.cv) {
        int max_nf = 1;
        for (int l = 0; l < o.L_max; ++l) max_nf *= o.M;
        const hipError_t e = cv_table_view(o.cv, m, ctx->stream, max_nf, &cv_table, &cv_spec, &cv_phi0, &lds);
        if (e != hipSuccess) return hip_fail(ctx, e, "control-variate table");
    }
    const PersistentShape s = persistent_shape(ctx, sampler, lds);
    // the seed goes in with each launch: runs of one problem share the
    // descriptor's bytes and upload it once
    fill_desc(ctx, prob, s, m, &p, 1, o.L_max, o.M, ctx->d_drv_spread, &init);
    if (o.cv) {
        prob.h_desc->cv_table = cv_table;
        prob.h_desc->cv_spec = cv_spec;
        prob.h_desc->cv_phi0 = cv_phi0;
        prob.h_desc->cv_levels = o.cv_levels;
    }
    bool uploaded = false;
    st = upload_desc(ctx, prob, &uploaded);
    if (st) return st;
    const dim3 grid(ctx->num_cu * s.blocks_per_cu), block(s.block);
    const BatchDesc* d = prob.d_desc;
    DriverState* mirror = (DriverState*)ctx->h_drv_dev;
    // prepared: the context's last run was a device-planned one that ended
    // normally, so the update queued past its end has built a fresh state
    // and planned its pilot batch, and its updates left the spread groups at
    // zero; if the descriptor is that run's, this run starts with its
    // sampler.  Otherwise the start kernel comes first.
    if (!(prepared && !uploaded)) {
        hipLaunchKernelGGL(driver_start_kernel, dim3(1), dim3(256), 0, ctx->stream, d_st,
                           ctx->d_drv_spread, init, d);
        MLMC_HIP(ctx, hipGetLastError());
    }
    // Iteration k + 1 is enqueued before the host waits for iteration k's
    // update: its sampler reads the items that update planned, so the GPU
    // runs the iterations back to back while the host reads the mirror.  The
    // one iteration past the last update finds an empty plan and a finished
    // state and does nothing.
    int first_tix = -1;
    for (int it = 0;; ++it) {
        if (it > h_st->max_iterations + 1)
            return fail(ctx, MLMC_EDEVICE, "driver state did not reach the host");
        const TraceRange iter_range("mlmc_run driver iteration (device-planned)");
        for (int k = it ? 1 : 0; k < 2; ++k) {
            // the sampler stamps slot 16, the update-and-plan block slot 17
            hipEvent_t t0, t1;
            timed_kernel(ctx, 16, 0.0, 0.0, &t0, &t1);
            if (first_tix < 0 && t0) first_tix = (int)ctx->pending.size() - 1;
            if (t0) hipExtLaunchKernelGGL(sampler, grid, block, lds, ctx->stream, t0, t1, 0, d, o.seed);
            else hipLaunchKernelGGL(sampler, grid, block, lds, ctx->stream, d, o.seed);
            hipError_t e = hipGetLastError();
            if (e == hipSuccess) {
                timed_kernel(ctx, 17, 0.0, 0.0, &t0, &t1);
                if (t0)
                    hipExtLaunchKernelGGL(driver_update_plan_kernel, dim3(1), dim3(512), 0, ctx->stream,
                                          t0, t1, 0, d_st, mirror, ctx->d_drv_spread, d);
                else
                    hipLaunchKernelGGL(driver_update_plan_kernel, dim3(1), dim3(512), 0, ctx->stream,
                                       d_st, mirror, ctx->d_drv_spread, d);
                e = hipGetLastError();
            }
            if (e != hipSuccess) return hip_fail(ctx, e, "persistent iteration");
        }
        // the update kernel also writes the host mirror h_st
        const hipError_t e = wait_update(ctx->stream, h_st, (unsigned long long)it + 1);
        if (e != hipSuccess) return hip_fail(ctx, e, "persistent iteration");
        // the flag comes in the word that publishes the update, so a mirror
        // seen done is complete; later updates leave it as it is
        if (mirror_done(h_st)) break;
    }
    // the update queued past the last one prepares the next run's start
    ctx->drv_pilot_ready = true;
    // the iteration past the last update may still run: the result is read
    // from the mirror; stamped launches are read once finished (harvest_ready
    // now, the rest by a later harvest), the run does not wait for them
    if (ctx->pending.empty()) return MLMC_OK;
    if (first_tix >= 0) {
        // the launches' path steps are known only as a whole: every sampled
        // batch is absorbed into n_l, so they are charged to the run's first
        // stamped sampler launch
        double fine = 0.0, coarse = 0.0;
        for (int l = 0; l <= h_st->L; ++l) {
            const double nf = std::pow((double)o.M, (double)l);
            fine += h_st->n[l] * nf;
            coarse += l ? h_st->n[l] * nf / o.M : 0.0;
        }
        ctx->pending[first_tix].fine_steps = fine;
        ctx->pending[first_tix].coarse_steps = coarse;
    }
    harvest_ready(ctx);
    return MLMC_OK;
}

// One payoff kind in every slot: a kernel that holds that payoff's code only.
static PersistentFn batch_sampler(const mlmc_ctx* ctx, const mlmc_model& m, const mlmc_payoff* p, int np, int M)
{
    int payoff = p[0].kind;
    for (int k = 1; k < np; ++k)
        if (p[k].kind != payoff) payoff = kAnyPayoff;
    return pick_persistent(sampler_variant(m), M, persistent_ppt(ctx), payoff);
}

// Plan and sample one batch, then publish its groups: three launches (four
// with a fill launch after a call that failed) on the context's stream, the
// seed and the request in their arguments, so batches of one problem upload
// nothing.  counts: device counts of slot 0's samples per level instead of
// the request (then published and cleared).
static mlmc_status run_batch(mlmc_ctx* ctx, const mlmc_model& m, const mlmc_payoff* p, int np, int L, int M,
                             uint64_t seed, BatchRequest* req, unsigned long long* counts, double fine,
                             double coarse)
{
    auto* b = bufs_of(ctx);
    const PersistentFn sampler = batch_sampler(ctx, m, p, np, M);
    const PersistentShape s = persistent_shape(ctx, sampler, 0);
    fill_desc(ctx, b->batch, s, m, p, np, L, M, b->d_acc, nullptr);
    mlmc_status st = upload_desc(ctx, b->batch);
    if (st) return st;
    if (!b->acc_clean) MLMC_HIP(ctx, zero_records(b->d_acc, kGroupRecords, ctx->stream));
    b->acc_clean = false;
    const BatchDesc* d = b->batch.d_desc;
    unsigned blocks = (unsigned)(ctx->num_cu * s.blocks_per_cu);
    if (req) {
        // small: the blocks that fit (see kItems)
        if (fine + coarse < kFewItems * kSmallItem * blocks) blocks = (unsigned)(ctx->num_cu * s.fit_per_cu);
        req->blocks = blocks;
    }
    const int tix = timed_begin(ctx, 16, fine, coarse);
    if (counts) hipLaunchKernelGGL(plan_counts_kernel, dim3(1), dim3(64), 0, ctx->stream, d, counts);
    else hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(64), 0, ctx->stream, d, *req);
    MLMC_HIP(ctx, hipGetLastError());
    hipLaunchKernelGGL(sampler, dim3(blocks), dim3(s.block), 0, ctx->stream, d, seed);
    MLMC_HIP(ctx, hipGetLastError());
    timed_end(ctx, tix);
    static_assert(kMaxSlots * kMaxLevels <= kPublishGroups, "the mirror holds every pair");
    // the groups past the last slot's last level were not touched
    st = publish_groups(ctx, b->d_acc, (np - 1) * kMaxLevels + L + 1, counts, false);
    if (!st) b->acc_clean = true;
    return st;
}

mlmc_status run_counts(mlmc_ctx* ctx, const mlmc_model& m, const mlmc_payoff& p, int L, int M, uint64_t seed,
                       unsigned long long* counts)
{
    const mlmc_status st = run_batch(ctx, m, &p, 1, L, M, seed, nullptr, counts, 0.0, 0.0);
    if (!st) counts_published(ctx);
    return st;
}

void counts_published(mlmc_ctx* ctx) { bufs_of(ctx)->counts_clean = true; }

mlmc_status level_counts(mlmc_ctx* ctx, unsigned long long** counts)
{
    const mlmc_status st = ensure_bufs(ctx);
    if (st) return st;
    auto* b = bufs_of(ctx);
    if (!b->counts_clean) {
        LevelAcc* from = b->acc_clean ? b->d_acc + kGroupRecords : b->d_acc;
        MLMC_HIP(ctx, zero_records(from, (int)(b->d_acc + kGroupRecords + kCountRecords - from), ctx->stream));
        b->acc_clean = true;
    }
    b->counts_clean = false;
    *counts = b->d_counts;
    return MLMC_OK;
}

}  // namespace mlmc

using namespace mlmc;

extern "C" {

mlmc_status mlmc_set_persistent_launch(mlmc_ctx* ctx, int block, int ppt, int blocks_per_cu)
{
    if (!ctx) return MLMC_EINVAL;
    if (block == 0) {
        ctx->persist_block = ctx->persist_ppt = ctx->persist_bpc = 0;
    } else {
        if (block != 64 && block != 128 && block != 256 && block != 512 && block != 1024)
            return fail(ctx, MLMC_EINVAL, "block must be 64, 128, 256, 512 or 1024");
        if (ppt != 1 && ppt != 2 && ppt != 4) return fail(ctx, MLMC_EINVAL, "ppt must be 1, 2 or 4");
        if (blocks_per_cu < 1 || blocks_per_cu * block > 4096)
            return fail(ctx, MLMC_EINVAL, "blocks_per_cu * block must be in 1..4096 threads");
        ctx->persist_block = block;
        ctx->persist_ppt = ppt;
        ctx->persist_bpc = blocks_per_cu;
    }
    return MLMC_OK;
}

mlmc_status mlmc_persistent_shape(mlmc_ctx* ctx, const mlmc_model* model, const mlmc_payoff* payoffs, int npayoffs,
                                  int M, int L, const mlmc_cv* cv, mlmc_launch_shape* out)
{
    if (!ctx) return MLMC_EINVAL;
    if (!payoffs || !out) return fail(ctx, MLMC_EINVAL, "payoffs and out must not be NULL");
    if (npayoffs < 1 || npayoffs > kMaxSlots) return fail(ctx, MLMC_EINVAL, "npayoffs must be in 1..4");
    for (int k = 0; k < npayoffs; ++k) {
        const mlmc_status st = check_level_args(ctx, model, &payoffs[k], L, M, 32);
        if (st) return st;
    }
    MLMC_ENTER(ctx);
    PersistentFn fn = batch_sampler(ctx, *model, payoffs, npayoffs, M);
    size_t lds = 0;
    if (cv) {
        fn = pick_persistent(sampler_variant(*model), M, persistent_ppt(ctx), payoffs[0].kind, true);
        if (!fn || npayoffs != 1 || cv_in_dim(cv) != (model->kind == MLMC_HESTON ? 3 : 2))
            return fail(ctx, MLMC_EINVAL, "no persistent sampler with this control variate");
        int max_nf = 1;
        for (int l = 0; l < L; ++l) max_nf *= M;
        const float *table, *phi0;
        TableSpec spec;
        const hipError_t e = cv_table_view(cv, *model, ctx->stream, max_nf, &table, &spec, &phi0, &lds);
        if (e != hipSuccess) return hip_fail(ctx, e, "control-variate table");
    }
    const PersistentShape s = persistent_shape(ctx, fn, lds);
    out->block = s.block;
    out->ppt = s.ppt;
    out->split = 1;
    out->few_chains = 0;
    out->grid = ctx->num_cu * s.blocks_per_cu;
    out->resident = s.fit_per_cu;
    return MLMC_OK;
}

mlmc_status mlmc_levels_batch(mlmc_ctx* ctx, const mlmc_model* model, const mlmc_payoff* payoffs,
                              int npayoffs, int M, int L, const uint64_t* N,
                              const uint64_t* offsets, uint64_t seed, mlmc_level_result* out)
{
    if (!ctx) return MLMC_EINVAL;
    if (!payoffs || !N || !out) return fail(ctx, MLMC_EINVAL, "payoffs, N and out must not be NULL");
    if (npayoffs < 1 || npayoffs > kMaxSlots)
        return fail(ctx, MLMC_EINVAL, "npayoffs must be in 1..4");
    mlmc_status st = MLMC_OK;
    for (int k = 0; k < npayoffs && !st; ++k) st = check_level_args(ctx, model, &payoffs[k], L, M, 32);
    if (st) return st;
    if (model->antithetic)
        return fail(ctx, MLMC_EINVAL, "the antithetic estimator runs with per-level launches only");
    if (L >= kMaxLevels) return fail(ctx, MLMC_EINVAL, "L must be < 16");
    for (int i = 0; i < npayoffs * (L + 1); ++i) {
        if (N[i] > (1ull << 40)) return fail(ctx, MLMC_EINVAL, "N too large (max 2^40 per level)");
        if (((offsets ? offsets[i] : 0) + N[i]) >> 56)
            return fail(ctx, MLMC_EINVAL, "path index beyond 2^56");
    }
    ctx->err.clear();
    MLMC_ENTER(ctx);
    st = ensure_bufs(ctx);
    if (st) return st;
    BatchRequest req;
    std::memset(&req, 0, sizeof(req));
    double fine = 0.0, coarse = 0.0;
    for (int k = 0; k < npayoffs; ++k)
        for (int l = 0; l <= L; ++l) {
            const uint64_t n = N[k * (L + 1) + l];
            req.dN[k * kMaxLevels + l] = (double)n;
            req.offset[k * kMaxLevels + l] = offsets ? (double)offsets[k * (L + 1) + l] : 0.0;
            const double nf = std::pow((double)M, (double)l);
            fine += (double)n * nf;
            coarse += l ? (double)n * nf / M : 0.0;
        }
    st = run_batch(ctx, *model, payoffs, npayoffs, L, M, seed, &req, nullptr, fine, coarse);
    if (st) return st;
    uint64_t nonfinite = 0;
    for (int k = 0; k < npayoffs; ++k)
        for (int l = 0; l <= L; ++l) {
            const double* sum = ctx->h_pub->sum[k * kMaxLevels + l];
            mlmc_level_result& o = out[k * (L + 1) + l];
            o.sum_y = sum[0];
            o.sum_y2 = sum[1];
            o.sum_pf = sum[2];
            o.sum_pf2 = sum[3];
            o.sum_pc = sum[4];
            o.sum_pc2 = sum[5];
            const double nf = std::pow((double)M, (double)l);
            o.n = N[k * (L + 1) + l];
            o.cost = (double)o.n * (l ? nf + nf / M : 1.0);
            o.n_nonfinite = ctx->h_pub->n_nonfinite[k * kMaxLevels + l];
            nonfinite += o.n_nonfinite;
        }
    if (nonfinite) return fail(ctx, MLMC_ENONFINITE, "non-finite samples left out of the sums");
    return MLMC_OK;
}

}  // extern "C"
