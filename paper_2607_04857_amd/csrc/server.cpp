// server.cpp -- continuous-batching solve server.
//
// Requests are planned on the submitting thread and queued.  One scheduler
// thread owns the device stream and runs ticks:
//   1. admission: queued requests enter device slots, first come first
//      served, while a slot is free and the device-memory budget allows;
//      each admitted request gets one block of device memory (its tables,
//      per-item results), a finished request's where one of that size is kept,
//      and a round's requests one table-build launch; the tables stay
//      resident until the request finishes;
//   2. one persistent walk launch over a slice of work items from EVERY
//      admitted request (water-filling: requests with few items left get all
//      of them, the rest share the remaining per-tick item budget), so a
//      request arriving while others are on the GPU joins the next tick;
//   3. a finish launch for requests whose last items ran in this tick, which
//      writes the results to mapped host memory.
// Ticks alternate between two buffer sets: tick k+1 is enqueued before the
// host waits for tick k, so the GPU does not idle between ticks.  A request
// is solved by the same kernels and the same integer arithmetic whether it
// runs alone or mixed with others, so its result does not depend on the mix.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <thread>
#include <tuple>
#include <unordered_map>

#include "runtime.h"
#include "serve_policy.h"

namespace {

using Clock = std::chrono::steady_clock;

// Walk launches per tick are one per distinct walk kernel variant among the
// active requests; this bounds the number of built variants (B x cache x tier).
constexpr int kMaxTickLaunches = 32;
constexpr int kUnitLog = 12;        // the tick budget counts units of 2^12 Gray steps, or
                                    // items where these are longer (A > 32)
constexpr int kMaxRound = 128;      // requests admitted in one round, at most: their host
                                    // images share one mapped block per tick buffer
// A request's image at most: its descriptor, T and float32 Q, each aligned.
constexpr size_t kImageBytes = 1024 + 2 * (size_t(qplan::kMaxN) * qplan::kMaxN * 4 + 256);

enum class RState { Queued, Active, Done, Failed };

struct Request {
    uint64_t ticket = 0;
    qrt::Job job;                 // single-instance job
    std::vector<float> qf;        // owned float32 input
    Clock::time_point arrival;
    RState state = RState::Queued;
    void *d_mem = nullptr;
    int kslot = -1;
    qk::Inst base{};              // device descriptor of the whole instance
    uint64_t next_item = 0;       // next work item to issue
    qubo_result_t result{};
    qubo_status_t status = QUBO_OK;
    std::string error;
};

struct TickBuf {
    hipEvent_t done = nullptr;
    // Mapped host blocks, with their device addresses: the images of a round's
    // requests and where they go, the tick's descriptors (walk, then finish:
    // 2 max_slots), and the finish results (max_slots), which the finish
    // writes there.  A copy each had cost about 10 us of the stream.
    unsigned char *h_block = nullptr;   // all of them
    unsigned char *h_images = nullptr, *hd_images = nullptr;
    qk::Upload *h_ups = nullptr, *hd_ups = nullptr;
    qk::Inst *h_descs = nullptr, *hd_descs = nullptr;
    qk::FinalRes *h_out = nullptr, *hd_out = nullptr;
    unsigned char *d_block = nullptr;   // the descriptors in place, then the item counters
    std::vector<Request *> finishing;
    bool inflight = false;
};

}  // namespace

struct qubo_server {
    int dev = 0;
    size_t budget = 0;
    int max_slots = 0;
    int cus = 0;                  // compute units of the device
    uint64_t tick_items = 0;      // units (kUnitLog) per tick, two per resident wave
    hipStream_t stream = nullptr;
    int32_t *d_karena = nullptr;  // max_slots K tables
    size_t counters_at = 0;       // offset of the item counters in TickBuf::d_block
    std::vector<int> free_kslots;
    TickBuf ticks[2];
    int cur = 0;
    // Device memory of finished requests, by size, for the next ones (the
    // scheduler thread's, on its stream): with what the active requests hold,
    // within the budget, and given back whenever the server idles.
    std::map<size_t, std::vector<void *>> kept;
    size_t kept_bytes = 0;

    std::mutex mu;
    std::condition_variable cv_work, cv_done;
    std::deque<Request *> queue;
    std::vector<Request *> active;
    std::unordered_map<uint64_t, Request *> reqs;
    uint64_t next_ticket = 1;
    size_t mem_used = 0, mem_peak = 0;
    int active_peak = 0;
    uint64_t n_ticks = 0;
    bool stop = false;
    std::string fatal;
    std::vector<double> lat_ms;
    double states_done = 0.0;
    bool have_t0 = false;
    Clock::time_point t0;
    std::thread th;
};

namespace {

double ms_since(Clock::time_point a) { return std::chrono::duration<double, std::milli>(Clock::now() - a).count(); }

void fail_all(qubo_server *s, const std::string &msg)
{
    std::lock_guard<std::mutex> lk(s->mu);
    s->fatal = msg;
    for (auto &kv : s->reqs) {
        Request *r = kv.second;
        if (r->state == RState::Queued || r->state == RState::Active) {
            r->state = RState::Failed;
            r->status = QUBO_EDEVICE;
            r->error = msg;
        }
    }
    s->queue.clear();
    s->active.clear();
    s->cv_done.notify_all();
}

// Give back at least `need` bytes of the kept blocks (all where they are fewer).
void give_back(qubo_server *s, size_t need)
{
    std::vector<size_t> sizes;
    for (const auto &kv : s->kept) sizes.insert(sizes.end(), kv.second.size(), kv.first);
    for (size_t k : qsched::blocks_to_free(sizes, need)) {
        auto it = s->kept.find(sizes[k]);
        (void)hipFreeAsync(it->second.back(), s->stream);
        s->kept_bytes -= sizes[k];
        it->second.pop_back();
        if (it->second.empty()) s->kept.erase(it);
    }
}

// A kept block of exactly that size, or null.
void *take_kept(qubo_server *s, size_t bytes)
{
    auto it = s->kept.find(bytes);
    if (it == s->kept.end()) return nullptr;
    void *p = it->second.back();
    s->kept_bytes -= bytes;
    it->second.pop_back();
    if (it->second.empty()) s->kept.erase(it);
    return p;
}

// New device memory for a request about to be set up (counted in mem_used already).
hipError_t take_memory(qubo_server *s, size_t bytes, void **p)
{
    const size_t held = s->kept_bytes + s->mem_used;
    if (held > s->budget) give_back(s, held - s->budget);
    hipError_t e = hipMallocAsync(p, bytes, s->stream);
    if (e != hipSuccess && s->kept_bytes) {
        (void)hipGetLastError();
        give_back(s, s->kept_bytes);
        e = hipMallocAsync(p, bytes, s->stream);
    }
    return e;
}

// Called with the tick's event complete: publish results, keep the memory for
// other requests (a hipFreeAsync each, about 10 us, had held back the results
// of a tick of 25 requests by 250 us, and the next tick as long).  What the
// budget has no room for is freed after the results are out.
void complete_tick(qubo_server *s, TickBuf &t)
{
    std::vector<Request *> done = std::move(t.finishing);
    std::vector<void *> freed;
    t.finishing.clear();
    t.inflight = false;
    {
        std::lock_guard<std::mutex> lk(s->mu);
        for (size_t i = 0; i < done.size(); i++) {
            Request *r = done[i];
            qubo_status_t st = qrt::job_result(r->job, 0, t.h_out[i], &r->result);
            const double lat = ms_since(r->arrival);
            if (st != QUBO_OK) {
                r->status = st;
                r->error = qrt::last_error_cstr();
                r->state = RState::Failed;
            } else {
                r->result.total_ms = lat;
                r->result.kernel_ms = 0.0;
                r->state = RState::Done;
            }
            s->lat_ms.push_back(lat);
            s->states_done += std::ldexp(1.0, r->job.plans[0].n);
            s->mem_used -= r->job.bytes;
            if (s->kept_bytes + r->job.bytes + s->mem_used <= s->budget) {
                s->kept[r->job.bytes].push_back(r->d_mem);
                s->kept_bytes += r->job.bytes;
            } else {
                freed.push_back(r->d_mem);
            }
            r->d_mem = nullptr;
            s->free_kslots.push_back(r->kslot);
            s->active.erase(std::find(s->active.begin(), s->active.end(), r));
        }
    }
    s->cv_done.notify_all();
    for (void *p : freed) (void)hipFreeAsync(p, s->stream);
}

// Admit queued requests (policy: qsched::admit_count); returns the newly
// admitted ones (device set-up pending).
std::vector<Request *> take_admissions(qubo_server *s)
{
    std::vector<Request *> adm;
    std::vector<size_t> bytes;
    bytes.reserve(s->queue.size());
    for (const Request *r : s->queue) bytes.push_back(r->job.bytes);
    const size_t free_slots = std::min(size_t(s->max_slots) - std::min(size_t(s->max_slots),
                                                                      s->active.size()),
                                       s->free_kslots.size());
    size_t n_adm = qsched::admit_count(bytes, s->mem_used, s->budget,
                                       std::min(free_slots, size_t(kMaxRound)));
    for (; n_adm > 0; n_adm--) {
        Request *r = s->queue.front();
        s->queue.pop_front();
        s->mem_used += r->job.bytes;
        s->mem_peak = std::max(s->mem_peak, s->mem_used);
        r->kslot = s->free_kslots.back();
        s->free_kslots.pop_back();
        r->state = RState::Active;
        s->active.push_back(r);
        s->active_peak = std::max(s->active_peak, int(s->active.size()));
        adm.push_back(r);
    }
    return adm;
}

// Device memory of the k-th request admitted in a round, and its image in the
// tick buffer's mapped block.
qubo_status_t setup_request(qubo_server *s, TickBuf &t, Request *r, size_t k)
{
    if (!r->d_mem) QRT_HIP(take_memory(s, r->job.bytes, &r->d_mem), "hipMallocAsync");
    qubo_status_t st = qrt::job_bind(&r->job, r->d_mem);
    if (st != QUBO_OK) return st;
    // The K table lives in the server's arena so one walk launch sees every
    // request's table in a single array.
    qk::Inst I;
    std::memcpy(&I, r->job.stage.data(), sizeof(I));
    I.K = s->d_karena + size_t(r->kslot) * qk::kKTable;
    I.kslot = r->kslot;
    std::memcpy(r->job.stage.data(), &I, sizeof(I));
    r->base = I;
    if (r->job.stage_bytes > kImageBytes) {
        qrt::set_error("internal: request image larger than its share of the block");
        return QUBO_EINTERNAL;
    }
    std::memcpy(t.h_images + k * kImageBytes, r->job.stage.data(), r->job.stage_bytes);
    qk::Upload up{};
    up.src = t.hd_images + k * kImageBytes;
    up.dst = static_cast<unsigned char *>(r->d_mem);
    up.copy_bytes = uint32_t(r->job.stage_bytes);
    t.h_ups[k] = up;
    return QUBO_OK;
}

// One table-build launch for every request admitted in a round, which also
// puts their images in place.
qubo_status_t build_tables(qubo_server *s, TickBuf &t, size_t n_adm)
{
    if (n_adm == 0) return QUBO_OK;
    QRT_HIP(qk::launch_tables_upload(t.hd_ups, int(n_adm), s->stream), "tables kernel");
    return QUBO_OK;
}

// Enqueue one tick into buffer t; *launched stays false when there was nothing to do.
qubo_status_t enqueue_tick(qubo_server *s, TickBuf &t, bool *launched)
{
    *launched = false;
    std::vector<Request *> act;
    {
        std::lock_guard<std::mutex> lk(s->mu);
        act = s->active;
    }
    // requests still owning unissued items or an unrun finish
    std::vector<Request *> walkers, finishers;
    for (Request *r : act) {
        const qplan::Plan &P = r->job.plans[0];
        if (P.direct) {
            if (r->next_item == 0) {   // not yet finished: finish-only request
                r->next_item = 1;
                finishers.push_back(r);
            }
        } else if (r->next_item < P.items) {
            walkers.push_back(r);
        }
    }
    // water-filling over the per-tick item budget, fewest remaining first,
    // then grouped by walk variant (one launch per variant group), in units of
    // 2^kUnitLog steps: requests differ in the length of their items
    auto unit_log = [](const Request *r) { return std::max(kUnitLog - r->job.plans[0].L, 0); };
    auto units_left = [&](const Request *r) {
        const int u = unit_log(r);
        return (r->job.plans[0].items - r->next_item + (uint64_t(1) << u) - 1) >> u;
    };
    std::sort(walkers.begin(), walkers.end(),
              [&](Request *a, Request *b) { return units_left(a) < units_left(b); });
    // Under a backlog the tick grows (qsched::tick_scale): fewer tick
    // boundaries (each costs a drain of the walk grid and a finish launch),
    // at no cost in latency since requests queue anyway.
    std::vector<uint64_t> left(walkers.size());
    for (size_t k = 0; k < walkers.size(); k++) left[k] = units_left(walkers[k]);
    std::vector<uint64_t> share = qsched::tick_shares(left, s->tick_items);
    for (size_t k = 0; k < walkers.size(); k++)
        share[k] = std::min(share[k] << unit_log(walkers[k]),
                            walkers[k]->job.plans[0].items - walkers[k]->next_item);
    uint64_t total = 0;
    for (uint64_t c : share) total += c;
    if (total == 0 && finishers.empty()) return QUBO_OK;
    // descriptors grouped by variant; item numbering restarts in every group
    std::vector<size_t> idx(walkers.size());
    for (size_t k = 0; k < idx.size(); k++) idx[k] = k;
    std::stable_sort(idx.begin(), idx.end(), [&](size_t x, size_t y) {
        const qplan::Plan &a = walkers[x]->job.plans[0], &b = walkers[y]->job.plans[0];
        return std::make_tuple(a.mcols, a.vgpr_levels, a.tier) < std::make_tuple(b.mcols, b.vgpr_levels, b.tier);
    });
    struct Launch { int first, count; uint64_t items; int max_L; const qplan::Plan *P; };
    std::vector<Launch> launches;
    int nw = 0;
    uint64_t g = 0;
    for (size_t k : idx) {
        Request *r = walkers[k];
        const uint64_t c = share[k];
        const qplan::Plan &P = r->job.plans[0];
        if (launches.empty() || !qrt::same_variant(*launches.back().P, P)) {
            launches.push_back({nw, 0, 0, 0, &P});
            g = 0;
        }
        qk::Inst I = r->base;
        I.item_begin = g;
        I.item_end = g + c;
        I.item_local0 = r->next_item;
        I.res = r->base.res + r->next_item;
        I.bit0 = r->next_item;          // I.bits: the request's whole bitmap
        t.h_descs[nw++] = I;
        g += c;
        launches.back().count++;
        launches.back().items += c;
        launches.back().max_L = std::max(launches.back().max_L, P.L);
        r->next_item += c;
        if (r->next_item == P.items) finishers.push_back(r);
    }
    // one launch puts the descriptors (walk, then finish) in place and clears
    // the item counters
    for (size_t i = 0; i < finishers.size(); i++) t.h_descs[size_t(nw) + i] = finishers[i]->base;
    qk::Upload up{};
    up.src = reinterpret_cast<const unsigned char *>(t.hd_descs);
    up.dst = t.d_block;
    up.copy_bytes = uint32_t(((size_t(nw) + finishers.size()) * sizeof(qk::Inst) + 15) / 16 * 16);
    up.zero_from = uint32_t(s->counters_at);
    up.zero_bytes =
        uint32_t(launches.size() * qk::kCounterWords * sizeof(unsigned long long));
    QRT_HIP(qk::launch_upload(up, s->stream), "upload kernel");
    const qk::Inst *d_descs = reinterpret_cast<const qk::Inst *>(t.d_block);
    unsigned long long *counters =
        reinterpret_cast<unsigned long long *>(t.d_block + s->counters_at);
    // the two default variants in one launch (grouped in order of tier)
    for (size_t k = 0; k + 1 < launches.size(); k++) {
        Launch &a = launches[k], &b = launches[k + 1];
        if (a.P->mcols != 16 || a.P->vgpr_levels != 4 || a.P->tier != 2 || b.P->mcols != 16 ||
            b.P->vgpr_levels != 4 || b.P->tier != 4)
            continue;
        const int occ = qk::walk_occupancy(16, 4, 2);
        const int waves = int(std::min<uint64_t>(a.items + b.items, uint64_t(s->cus) * uint64_t(occ)));
        QRT_HIP(qk::launch_walk_pair(
                    {d_descs + a.first, a.count, a.items, a.max_L, counters + k * qk::kCounterWords},
                    {d_descs + b.first, b.count, b.items, b.max_L,
                     counters + (k + 1) * qk::kCounterWords},
                    s->d_karena, waves, s->stream),
                "walk kernel");
        a.items = b.items = 0;
    }
    for (size_t k = 0; k < launches.size(); k++) {
        const Launch &L = launches[k];
        if (L.items == 0) continue;
        const int occ = qk::walk_occupancy(L.P->mcols, L.P->vgpr_levels, L.P->tier);
        const int waves = int(std::min<uint64_t>(L.items, uint64_t(s->cus) * uint64_t(occ)));
        QRT_HIP(qk::launch_walk(L.P->mcols, L.P->vgpr_levels, L.P->tier, d_descs + L.first, L.count,
                                L.items, L.max_L, counters + k * qk::kCounterWords, s->d_karena,
                                waves, s->stream),
                "walk kernel");
    }
    if (!finishers.empty())
        QRT_HIP(qk::launch_finish(d_descs + nw, int(finishers.size()), t.hd_out, qk::Upload{}, nullptr,
                                  nullptr, s->stream),
                "finish kernel");
    t.finishing = std::move(finishers);
    QRT_HIP(hipEventRecord(t.done, s->stream), "hipEventRecord");
    t.inflight = true;
    *launched = true;
    {
        std::lock_guard<std::mutex> lk(s->mu);
        s->n_ticks++;
    }
    return QUBO_OK;
}

void scheduler(qubo_server *s)
{
    if (hipSetDevice(s->dev) != hipSuccess) {
        fail_all(s, "hipSetDevice failed in the scheduler");
        return;
    }
    for (;;) {
        std::vector<Request *> adm;
        {
            std::unique_lock<std::mutex> lk(s->mu);
            adm = take_admissions(s);
            const bool idle = adm.empty() && s->active.empty() && !s->ticks[0].inflight &&
                              !s->ticks[1].inflight;
            if (idle) {
                if (s->stop && s->queue.empty()) break;
                if (s->cv_work.wait_for(lk, std::chrono::milliseconds(20)) ==
                    std::cv_status::timeout) {
                    lk.unlock();   // (`kept` is this thread's)
                    give_back(s, s->kept_bytes);
                }
                continue;
            }
        }
        TickBuf &t = s->ticks[s->cur];
        if (t.inflight) {
            // the buffer's previous tick was enqueued two ticks ago
            if (hipEventSynchronize(t.done) != hipSuccess) {
                fail_all(s, "tick failed on the device");
                return;
            }
            complete_tick(s, t);
        }
        // the whole round's kept blocks first: a new block makes room by giving
        // back others
        for (Request *r : adm) r->d_mem = take_kept(s, r->job.bytes);
        for (size_t k = 0; k < adm.size(); k++) {
            if (setup_request(s, t, adm[k], k) != QUBO_OK) {
                fail_all(s, qrt::last_error_cstr());
                return;
            }
        }
        if (build_tables(s, t, adm.size()) != QUBO_OK) {
            fail_all(s, qrt::last_error_cstr());
            return;
        }
        bool launched = false;
        if (enqueue_tick(s, t, &launched) != QUBO_OK) {
            fail_all(s, qrt::last_error_cstr());
            return;
        }
        if (launched) {
            s->cur ^= 1;
        } else {
            // nothing new to run: retire the other buffer's tick, if any
            TickBuf &o = s->ticks[s->cur ^ 1];
            if (o.inflight) {
                if (hipEventSynchronize(o.done) != hipSuccess) {
                    fail_all(s, "tick failed on the device");
                    return;
                }
                complete_tick(s, o);
            } else {
                std::unique_lock<std::mutex> lk(s->mu);
                if (s->queue.empty() || int(s->active.size()) >= s->max_slots)
                    s->cv_work.wait_for(lk, std::chrono::milliseconds(2));
            }
        }
    }
}

void server_free(qubo_server *s)
{
    if (!s) return;
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    for (TickBuf &t : s->ticks) {
        if (t.done) (void)hipEventDestroy(t.done);
        if (t.h_block) (void)hipHostFree(t.h_block);
        if (t.d_block) (void)hipFree(t.d_block);
    }
    for (auto &kv : s->reqs) {
        if (kv.second->d_mem) (void)hipFree(kv.second->d_mem);
        delete kv.second;
    }
    for (auto &kv : s->kept)
        for (void *m : kv.second) (void)hipFree(m);
    if (s->d_karena) (void)hipFree(s->d_karena);
    if (s->stream) (void)hipStreamDestroy(s->stream);
    delete s;
}

qubo_status_t server_init(qubo_server *s, size_t budget, int max_slots)
{
    QRT_HIP(hipGetDevice(&s->dev), "hipGetDevice");
    s->budget = budget;
    s->max_slots = max_slots;
    qrt::DeviceInfo di;
    qubo_status_t st = qrt::device_info(&di);
    if (st != QUBO_OK) return st;
    s->cus = di.cus;
    // two units (a served request's items are mostly a quarter of one) per
    // resident wave of the default walk variant (B = 10, LDS row cache)
    s->tick_items = uint64_t(di.cus) * uint64_t(qk::walk_occupancy(16, 4, 2)) * 2;
    QRT_HIP(hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking), "hipStreamCreate");
    QRT_HIP(hipMalloc(&s->d_karena, size_t(max_slots) * qk::kKTable * sizeof(int32_t)), "hipMalloc");
    for (int k = max_slots - 1; k >= 0; k--) s->free_kslots.push_back(k);
    for (TickBuf &t : s->ticks) {
        QRT_HIP(hipEventCreateWithFlags(&t.done, hipEventDisableTiming), "hipEventCreate");
        const size_t slots = size_t(max_slots), round = std::min(slots, size_t(kMaxRound));
        // (16 bytes past the descriptors: an image is copied in 16-byte words)
        const size_t ib = 2 * slots * sizeof(qk::Inst) + 16;
        s->counters_at = (ib + 255) / 256 * 256;
        // images | where they go | descriptors | results
        const size_t ups_at = round * kImageBytes;
        const size_t descs_at = (ups_at + round * sizeof(qk::Upload) + 255) / 256 * 256;
        const size_t out_at = descs_at + s->counters_at;
        void *h = nullptr, *d = nullptr;
        QRT_HIP(hipHostMalloc(&h, out_at + slots * sizeof(qk::FinalRes), hipHostMallocMapped),
                "hipHostMalloc");
        t.h_block = static_cast<unsigned char *>(h);
        QRT_HIP(hipHostGetDevicePointer(&d, h, 0), "hipHostGetDevicePointer");
        unsigned char *hd = static_cast<unsigned char *>(d);
        t.h_images = t.h_block;
        t.hd_images = hd;
        t.h_ups = reinterpret_cast<qk::Upload *>(t.h_block + ups_at);
        t.hd_ups = reinterpret_cast<qk::Upload *>(hd + ups_at);
        t.h_descs = reinterpret_cast<qk::Inst *>(t.h_block + descs_at);
        t.hd_descs = reinterpret_cast<qk::Inst *>(hd + descs_at);
        t.h_out = reinterpret_cast<qk::FinalRes *>(t.h_block + out_at);
        t.hd_out = reinterpret_cast<qk::FinalRes *>(hd + out_at);
        // item counters of every walk variant launched in a tick
        QRT_HIP(hipMalloc(&t.d_block, s->counters_at + kMaxTickLaunches * qk::kCounterWords *
                                                           sizeof(unsigned long long)),
                "hipMalloc");
    }
    return QUBO_OK;
}

}  // namespace

extern "C" {

qubo_status_t qubo_server_create(size_t mem_budget_bytes, int max_slots, qubo_server_t **srv)
{
    try {
        qrt::set_error("");
        if (!srv || max_slots < 1 || max_slots > 65536 || mem_budget_bytes == 0) {
            qrt::set_error("bad server arguments");
            return QUBO_EINVAL;
        }
        qubo_server *s = new qubo_server();
        qubo_status_t st = server_init(s, mem_budget_bytes, max_slots);
        if (st != QUBO_OK) {
            const std::string keep = qrt::last_error_cstr();
            server_free(s);
            qrt::set_error(keep);
            return st;
        }
        s->th = std::thread(scheduler, s);
        *srv = s;
        return QUBO_OK;
    } catch (const std::bad_alloc &) {
        qrt::set_error("host allocation failed");
        return QUBO_ENOMEM;
    } catch (...) {
        qrt::set_error("unexpected exception");
        return QUBO_EINTERNAL;
    }
}

qubo_status_t qubo_server_submit(qubo_server_t *s, const void *Q, int n, qubo_dtype_t dtype,
                                 uint64_t *ticket)
{
    try {
        qrt::set_error("");
        if (!s || !ticket) {
            qrt::set_error("null argument");
            return QUBO_EINVAL;
        }
        Request *r = new Request();
        r->job.plans.resize(1);
        std::string msg;
        qrt::tune_autoload();
        qubo_status_t st = qplan::make_plan(Q, n, dtype, nullptr, &r->job.plans[0], &msg, true);
        if (st != QUBO_OK) {
            delete r;
            qrt::set_error(msg);
            return st;
        }
        qplan::Plan &P = r->job.plans[0];
        if (dtype == QUBO_FP32) {
            const float *q = static_cast<const float *>(Q);
            r->qf.assign(q, q + size_t(n) * n);
            r->job.qf.push_back(r->qf.data());
        } else {
            r->job.qf.push_back(nullptr);
        }
        // Shorter items than the plan's; longer ones of these where the budget
        // does not hold so many records.
        const int planned = P.L, longest = std::min(planned, qsched::longest_item_log(P.A));
        for (int L = std::min(planned, qsched::item_log(P.A));; L++) {
            if (!P.direct) {
                P.L = L;
                P.items = uint64_t(1) << (P.A - L);
            }
            st = qrt::job_layout(&r->job, 0);
            if (st != QUBO_OK) {
                delete r;
                return st;
            }
            if (P.direct || L >= longest || r->job.bytes <= s->budget) break;
        }
        std::lock_guard<std::mutex> lk(s->mu);
        if (!s->fatal.empty()) {
            delete r;
            qrt::set_error(s->fatal);
            return QUBO_EDEVICE;
        }
        if (r->job.bytes > s->budget) {
            delete r;
            qrt::set_error("request needs more device memory than the server budget");
            return QUBO_ENOMEM;
        }
        r->ticket = s->next_ticket++;
        r->arrival = Clock::now();
        if (!s->have_t0) {
            s->have_t0 = true;
            s->t0 = r->arrival;
        }
        s->reqs[r->ticket] = r;
        s->queue.push_back(r);
        *ticket = r->ticket;
        s->cv_work.notify_one();
        return QUBO_OK;
    } catch (const std::bad_alloc &) {
        qrt::set_error("host allocation failed");
        return QUBO_ENOMEM;
    } catch (...) {
        qrt::set_error("unexpected exception");
        return QUBO_EINTERNAL;
    }
}

static qubo_status_t take_result(qubo_server *s, uint64_t ticket, qubo_result_t *out, bool *ready)
{
    auto it = s->reqs.find(ticket);
    if (it == s->reqs.end()) {
        qrt::set_error("unknown ticket");
        *ready = true;
        return QUBO_EINVAL;
    }
    Request *r = it->second;
    if (r->state == RState::Queued || r->state == RState::Active) {
        *ready = false;
        return QUBO_EAGAIN;
    }
    *ready = true;
    qubo_status_t st = r->status;
    if (r->state == RState::Done) {
        if (out) *out = r->result;
    } else {
        qrt::set_error(r->error);
    }
    s->reqs.erase(it);
    delete r;
    return st;
}

qubo_status_t qubo_server_poll(qubo_server_t *s, uint64_t ticket, qubo_result_t *out)
{
    if (!s) {
        qrt::set_error("null server");
        return QUBO_EINVAL;
    }
    qrt::set_error("");
    std::lock_guard<std::mutex> lk(s->mu);
    bool ready = false;
    return take_result(s, ticket, out, &ready);
}

qubo_status_t qubo_server_wait(qubo_server_t *s, uint64_t ticket, double timeout_ms,
                               qubo_result_t *out)
{
    if (!s) {
        qrt::set_error("null server");
        return QUBO_EINVAL;
    }
    qrt::set_error("");
    const auto deadline = Clock::now() + std::chrono::microseconds(int64_t(timeout_ms * 1000.0));
    std::unique_lock<std::mutex> lk(s->mu);
    for (;;) {
        bool ready = false;
        qubo_status_t st = take_result(s, ticket, out, &ready);
        if (ready) return st;
        if (s->cv_done.wait_until(lk, deadline) == std::cv_status::timeout) {
            st = take_result(s, ticket, out, &ready);
            return st;
        }
    }
}

qubo_status_t qubo_server_stats(qubo_server_t *s, double *p50_ms, double *p99_ms,
                                double *states_per_s)
{
    if (!s) {
        qrt::set_error("null server");
        return QUBO_EINVAL;
    }
    std::lock_guard<std::mutex> lk(s->mu);
    std::vector<double> v = s->lat_ms;
    std::sort(v.begin(), v.end());
    auto pct = [&](double p) {
        if (v.empty()) return 0.0;
        // nearest-rank percentile
        size_t k = size_t(std::ceil(p / 100.0 * double(v.size())));
        if (k < 1) k = 1;
        return v[k - 1];
    };
    if (p50_ms) *p50_ms = pct(50.0);
    if (p99_ms) *p99_ms = pct(99.0);
    if (states_per_s) {
        const double sec = s->have_t0 ? ms_since(s->t0) / 1e3 : 0.0;
        *states_per_s = sec > 0 ? s->states_done / sec : 0.0;
    }
    return QUBO_OK;
}

qubo_status_t qubo_server_info(qubo_server_t *s, size_t *mem_in_use, size_t *mem_peak,
                               int *active_peak, uint64_t *ticks)
{
    if (!s) {
        qrt::set_error("null server");
        return QUBO_EINVAL;
    }
    std::lock_guard<std::mutex> lk(s->mu);
    if (mem_in_use) *mem_in_use = s->mem_used;
    if (mem_peak) *mem_peak = s->mem_peak;
    if (active_peak) *active_peak = s->active_peak;
    if (ticks) *ticks = s->n_ticks;
    return QUBO_OK;
}

void qubo_server_destroy(qubo_server_t *s)
{
    if (!s) return;
    {
        std::lock_guard<std::mutex> lk(s->mu);
        s->stop = true;
    }
    s->cv_work.notify_all();
    if (s->th.joinable()) s->th.join();
    server_free(s);
}

}  // extern "C"
