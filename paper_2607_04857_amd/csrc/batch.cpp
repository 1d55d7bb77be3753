// batch.cpp -- many independent instances in one persistent walk launch.
//
// Every instance is planned on the host, laid out in one device allocation,
// and its work items are queued largest instance first (longest-processing-
// time order), so the persistent walk grid drains the big instances while
// the small ones fill the tail.  The H2D upload, table build, walk, per-
// instance finish and D2H download are captured once into a HIP graph and
// replayed by qubo_batch_run.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <numeric>
#include <tuple>

#include "runtime.h"

struct qubo_batch {
    qrt::Job job;
    std::vector<int> order;                    // walk position -> caller's index
    std::vector<std::vector<float>> qf_copy;   // owned float32 inputs
    hipStream_t stream = nullptr;
    void *d_mem = nullptr;
    unsigned char *h_stage = nullptr;          // pinned staging image
    qk::FinalRes *h_out = nullptr;             // pinned results
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    float last_ms = 0.f;
    bool ran = false;
};

namespace {

// Work items that a batch has at least, where its steps allow (eight per
// resident wave of the default variant): 100 instances of n = 15..25 walk in
// 55 us instead of 137, 1000 of n = 12..26 in 261 us instead of 328.  A replay
// of equal instances with this rule, and with the best and the longest of the
// items of 2^6 to 2^13 steps, us: 64 of n = 24 77, 76, 734; 300 of n = 24 188,
// 164 (2^8), 787; 1000 of n = 22 242, 225 (2^7), 383; 4096 of n = 22 677, 664
// (2^9), 726; 4096 of n = 24 1293, 1263 (2^10), 1707; 1000 of n = 26 923, 914
// (2^10), 1245.  Items of 2^6 steps, with as much set-up as walk, would take 791
// and 1844 for the 4096 of n = 22 and 24.
constexpr double kBatchItems = 32768.0;

void batch_free(qubo_batch *b)
{
    if (!b) return;
    if (b->stream) (void)hipStreamSynchronize(b->stream);
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    if (b->ev0) (void)hipEventDestroy(b->ev0);
    if (b->ev1) (void)hipEventDestroy(b->ev1);
    if (b->d_mem) (void)hipFree(b->d_mem);
    if (b->h_stage) (void)hipHostFree(b->h_stage);
    if (b->h_out) (void)hipHostFree(b->h_out);
    if (b->stream) (void)hipStreamDestroy(b->stream);
    delete b;
}

// Plan and lay out the batch's job.  own: keep copies of float32 inputs (for
// replays), instead of reading the caller's.
qubo_status_t batch_plan(qubo_batch *b, int count, const void *const *Q, const int *n,
                         const qubo_dtype_t *dtype, const qubo_options_t *opt, bool own)
{
    if (opt && (opt->item_first || opt->item_count)) {
        qrt::set_error("item ranges are for single solves");
        return QUBO_EINVAL;
    }
    std::vector<qplan::Plan> plans(static_cast<size_t>(count));
    std::string msg;
    qrt::tune_autoload();
    for (int i = 0; i < count; i++) {
        if (!Q[i]) {
            qrt::set_error("null Q in batch at " + std::to_string(i));
            return QUBO_EINVAL;
        }
        qubo_status_t st = qplan::make_plan(Q[i], n[i], dtype[i], opt, &plans[size_t(i)], &msg, true);
        if (st != QUBO_OK) {
            qrt::set_error("instance " + std::to_string(i) + ": " + msg);
            return st;
        }
    }
    // Shorter items where the whole batch has too few steps for kBatchItems
    // items of the planned length: the grid is then filled and ends together.
    if (!(opt && opt->L)) {
        double steps = 0.0;
        for (const qplan::Plan &P : plans)
            if (!P.direct) steps += std::ldexp(1.0, P.A);
        const int L = std::max(qplan::kSuper, std::ilogb(std::max(steps / kBatchItems, 1.0)));
        for (qplan::Plan &P : plans)
            if (!P.direct && P.L > L) {
                P.L = L;
                P.items = uint64_t(1) << (P.A - L);
            }
    }
    // Walk order: grouped by walk kernel variant (one persistent launch per
    // group), most walk work first inside a group; direct (tiny) instances last.
    b->order.resize(size_t(count));
    std::iota(b->order.begin(), b->order.end(), 0);
    std::stable_sort(b->order.begin(), b->order.end(), [&](int x, int y) {
        const qplan::Plan &px = plans[size_t(x)], &py = plans[size_t(y)];
        if (px.direct != py.direct) return !px.direct;
        const auto kx = std::make_tuple(px.mcols, px.vgpr_levels, px.tier);
        const auto ky = std::make_tuple(py.mcols, py.vgpr_levels, py.tier);
        if (kx != ky) return kx > ky;
        return px.n > py.n;
    });
    b->qf_copy.resize(size_t(count));
    for (int w = 0; w < count; w++) {
        const int i = b->order[size_t(w)];
        b->job.plans.push_back(std::move(plans[size_t(i)]));
        if (dtype[i] == QUBO_FP32) {
            const float *q = static_cast<const float *>(Q[i]);
            if (own) {
                b->qf_copy[size_t(w)].assign(q, q + size_t(n[i]) * n[i]);
                q = b->qf_copy[size_t(w)].data();
            }
            b->job.qf.push_back(q);
        } else {
            b->job.qf.push_back(nullptr);
        }
    }
    return qrt::job_layout(&b->job, opt ? opt->waves_per_cu : 0);
}

qubo_status_t batch_build(qubo_batch *b, int count, const void *const *Q, const int *n,
                          const qubo_dtype_t *dtype, const qubo_options_t *opt)
{
    qubo_status_t st = batch_plan(b, count, Q, n, dtype, opt, true);
    if (st != QUBO_OK) return st;
    QRT_HIP(hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking), "hipStreamCreate");
    QRT_HIP(hipEventCreate(&b->ev0), "hipEventCreate");
    QRT_HIP(hipEventCreate(&b->ev1), "hipEventCreate");
    hipError_t e = hipMalloc(&b->d_mem, b->job.bytes);
    if (e != hipSuccess) {
        b->d_mem = nullptr;
        qrt::set_error("device allocation of " + std::to_string(b->job.bytes) + " bytes failed");
        return QUBO_ENOMEM;
    }
    st = qrt::job_bind(&b->job, b->d_mem);
    if (st != QUBO_OK) return st;
    QRT_HIP(hipHostMalloc(reinterpret_cast<void **>(&b->h_stage), b->job.stage_bytes, 0),
            "hipHostMalloc");
    std::memcpy(b->h_stage, b->job.stage.data(), b->job.stage_bytes);
    QRT_HIP(hipHostMalloc(reinterpret_cast<void **>(&b->h_out), size_t(count) * sizeof(qk::FinalRes), 0),
            "hipHostMalloc");
    // Capture: upload, kernels, download.  No memset nodes: the table kernel
    // clears the work-item counter.
    QRT_HIP(hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
    qubo_status_t cst = QUBO_OK;
    e = hipMemcpyAsync(b->d_mem, b->h_stage, b->job.stage_bytes, hipMemcpyHostToDevice, b->stream);
    if (e != hipSuccess) cst = qrt::device_error("capture H2D", e);
    if (cst == QUBO_OK) cst = qrt::job_enqueue_kernels(b->job, b->stream);
    if (cst == QUBO_OK) {
        e = hipMemcpyAsync(b->h_out, b->job.d_out, size_t(count) * sizeof(qk::FinalRes),
                           hipMemcpyDeviceToHost, b->stream);
        if (e != hipSuccess) cst = qrt::device_error("capture D2H", e);
    }
    hipError_t ee = hipStreamEndCapture(b->stream, &b->graph);
    if (cst != QUBO_OK) return cst;
    if (ee != hipSuccess) return qrt::device_error("hipStreamEndCapture", ee);
    QRT_HIP(hipGraphInstantiateWithFlags(&b->exec, b->graph, 0), "hipGraphInstantiate");
    return QUBO_OK;
}

}  // namespace

extern "C" {

qubo_status_t qubo_batch_create(int count, const void *const *Q, const int *n,
                                const qubo_dtype_t *dtype, const qubo_options_t *opt,
                                qubo_batch_t **batch)
{
    try {
        qrt::set_error("");
        if (count < 1 || !Q || !n || !dtype || !batch) {
            qrt::set_error("bad batch arguments");
            return QUBO_EINVAL;
        }
        qubo_batch *b = new qubo_batch();
        qubo_status_t st = batch_build(b, count, Q, n, dtype, opt);
        if (st != QUBO_OK) {
            const std::string keep = qrt::last_error_cstr();
            batch_free(b);
            qrt::set_error(keep);
            return st;
        }
        *batch = b;
        return QUBO_OK;
    } catch (const std::bad_alloc &) {
        qrt::set_error("host allocation failed");
        return QUBO_ENOMEM;
    } catch (...) {
        qrt::set_error("unexpected exception");
        return QUBO_EINTERNAL;
    }
}

qubo_status_t qubo_batch_run(qubo_batch_t *b, void *hip_stream)
{
    if (!b) {
        qrt::set_error("null batch");
        return QUBO_EINVAL;
    }
    qrt::set_error("");
    hipStream_t s = hip_stream ? static_cast<hipStream_t>(hip_stream) : b->stream;
    QRT_HIP(hipEventRecord(b->ev0, s), "hipEventRecord");
    QRT_HIP(hipGraphLaunch(b->exec, s), "hipGraphLaunch");
    QRT_HIP(hipEventRecord(b->ev1, s), "hipEventRecord");
    QRT_HIP(hipStreamSynchronize(s), "hipStreamSynchronize");
    QRT_HIP(hipEventElapsedTime(&b->last_ms, b->ev0, b->ev1), "hipEventElapsedTime");
    b->ran = true;
    return QUBO_OK;
}

qubo_status_t qubo_batch_results(qubo_batch_t *b, qubo_result_t *out)
{
    if (!b || !out) {
        qrt::set_error("null argument");
        return QUBO_EINVAL;
    }
    if (!b->ran) {
        qrt::set_error("batch has not run");
        return QUBO_EINVAL;
    }
    const int count = int(b->order.size());
    for (int w = 0; w < count; w++) {
        qubo_result_t r;
        qubo_status_t st = qrt::job_result(b->job, w, b->h_out[w], &r);
        if (st != QUBO_OK) return st;
        r.kernel_ms = b->last_ms;
        r.total_ms = b->last_ms;
        out[b->order[size_t(w)]] = r;
    }
    return QUBO_OK;
}

qubo_status_t qubo_batch_stats(qubo_batch_t *b, double *states, double *kernel_ms)
{
    if (!b) {
        qrt::set_error("null batch");
        return QUBO_EINVAL;
    }
    if (states) *states = b->job.states;
    if (kernel_ms) *kernel_ms = b->last_ms;
    return QUBO_OK;
}

void qubo_batch_destroy(qubo_batch_t *b) { batch_free(b); }

// One pass needs no graph and no allocations of its own: planning, one upload
// launch and the kernels (100 instances of n = 15..25: 790 us with a batch
// handle made and destroyed, now 545).
qubo_status_t qubo_solve_batch(int count, const void *const *Q, const int *n,
                               const qubo_dtype_t *dtype, qubo_result_t *out)
{
    using clock = std::chrono::steady_clock;
    const auto t0 = clock::now();
    try {
        qrt::set_error("");
        if (!out) {
            qrt::set_error("null output");
            return QUBO_EINVAL;
        }
        if (count < 1 || !Q || !n || !dtype) {
            qrt::set_error("bad batch arguments");
            return QUBO_EINVAL;
        }
        qubo_batch b;
        qubo_status_t st = batch_plan(&b, count, Q, n, dtype, nullptr, false);
        if (st != QUBO_OK) return st;
        hipStream_t s = qrt::thread_stream(&st);
        if (st != QUBO_OK) return st;
        std::vector<qk::FinalRes> res;
        if ((st = qrt::run_once(b.job, s, &res)) != QUBO_OK) return st;
        const double walk = qrt::walk_ms(res[0].walk_ticks);
        for (int w = 0; w < count; w++) {
            qubo_result_t r;
            if ((st = qrt::job_result(b.job, w, res[size_t(w)], &r)) != QUBO_OK) return st;
            r.kernel_ms = walk;
            out[b.order[size_t(w)]] = r;
        }
        const double total =
            std::chrono::duration<double, std::milli>(clock::now() - t0).count();
        for (int i = 0; i < count; i++) out[i].total_ms = total;
        return QUBO_OK;
    } catch (const std::bad_alloc &) {
        qrt::set_error("host allocation failed");
        return QUBO_ENOMEM;
    } catch (...) {
        qrt::set_error("unexpected exception");
        return QUBO_EINTERNAL;
    }
}

}  // extern "C"
