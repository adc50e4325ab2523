// bed_server.cpp -- continuous-batching request server.
//
// Requests (count matrices of one size n, caller-owned device buffers) are
// admitted while the in-flight matrix count and the admitted bytes stay under
// the configured limits (bed_admit.hpp).  At admission an event is recorded on
// the caller's stream, so the step that reads a request's A first waits for
// the work the caller enqueued before submitting (the kernel or copy that
// produced A).  A scheduler thread packs admitted, not-yet-launched requests into a
// step on a free stream (up to max_step matrices): a pointer work list in pinned
// host memory that the step's kernels read in place, one launch per size class and
// one event.  While several streams are free a step takes the oldest request's data
// type and size class only.  Steps on different streams overlap on the
// device; completion is observed by polling the events.  The per-matrix
// kernel configuration depends only on (n, dtype), so each request's result is
// bitwise the same alone or in any mix.
#include <chrono>
#include <condition_variable>
#include <deque>
#include <map>
#include <mutex>
#include <string>
#include <algorithm>
#include <thread>
#include <vector>

#include "bed_admit.hpp"
#include "bed_host.hpp"

using namespace bed;

namespace {

using Clock = std::chrono::steady_clock;

struct Request {
    uint64_t ticket;
    bed_dtype dt;
    int32_t count, n;
    const void *A;
    void *lam, *Q;
    int32_t *info;
    int64_t bytes;
    hipEvent_t ready;  // recorded on the caller's stream at submission
    hipStream_t producer;
    Clock::time_point t_submit;
    bool launched = false, done = false;
    double latency_us = 0.0;
};

struct Slot {
    hipStream_t stream = nullptr;
    hipEvent_t done_ev = nullptr;
    // work list of the step in flight, in pinned memory that its kernels read: 48
    // bytes a matrix, once, are not worth a copy ahead of each step
    PtrItem *items = nullptr;
    bool busy = false;
    std::vector<uint64_t> tickets;
};

}  // namespace

struct bed_server {
    bed_server_opts opts;
    std::vector<Slot> slots;
    std::mutex mu;
    std::condition_variable cv, cv_done;
    std::deque<uint64_t> pending;
    std::map<uint64_t, Request> reqs;
    std::vector<hipEvent_t> free_events;  // recycled readiness events
    uint64_t next_ticket = 1;
    Admission adm;
    bool stop = false;
    std::thread worker;
    int device = 0;
    std::string error;
};

static void server_loop(bed_server *s)
{
    (void)hipSetDevice(s->device);
    std::unique_lock<std::mutex> lk(s->mu);
    while (true) {
        // completions
        bool progressed = false;
        for (auto &sl : s->slots) {
            if (!sl.busy) continue;
            if (hipEventQuery(sl.done_ev) == hipSuccess) {
                const auto now = Clock::now();
                for (uint64_t tk : sl.tickets) {
                    auto it = s->reqs.find(tk);
                    if (it == s->reqs.end()) continue;
                    Request &r = it->second;
                    r.done = true;
                    r.latency_us =
                        std::chrono::duration<double, std::micro>(now - r.t_submit).count();
                    s->adm.release(r.count, r.bytes);
                    s->free_events.push_back(r.ready);
                    r.ready = nullptr;
                }
                sl.tickets.clear();
                sl.busy = false;
                progressed = true;
            }
        }
        if (progressed) s->cv_done.notify_all();
        // launches: pending requests go into the next step on a free slot
        Slot *free_slot = nullptr;
        int nfree = 0;
        for (auto &sl : s->slots)
            if (!sl.busy) {
                if (!free_slot) free_slot = &sl;
                ++nfree;
            }
        if (free_slot && !s->pending.empty()) {
            Slot &sl = *free_slot;
            // One type and size class a step, so that classes run side by side on the
            // streams (one after the other on one stream they took 100 us for the last
            // step of a burst, 65 so); everything on the last free stream, where the
            // rest would wait for a step's end.
            int count = 0;
            const bed_dtype dt0 = s->reqs[s->pending.front()].dt;
            const int cls0 = size_class(s->reqs[s->pending.front()].n);
            for (auto p = s->pending.begin(); p != s->pending.end();) {
                Request &r = s->reqs[*p];
                if (nfree > 1 && (r.dt != dt0 || size_class(r.n) != cls0)) {
                    ++p;
                    continue;
                }
                if (count > 0 && count + r.count > s->opts.max_step) break;
                count += r.count;
                r.launched = true;
                sl.tickets.push_back(*p);
                p = s->pending.erase(p);
            }
            // the list in pinned memory grouped by (dtype, class)
            struct Launch {
                bed_dtype dt;
                int cls, off, count;
            };
            std::vector<Launch> launches;
            int off = 0;
            for (const bed_dtype dt : {BED_F32, BED_F64})
                for (int c = 2; c >= 0; --c) {
                    const int first = off;
                    const size_t es = dtype_size(dt);
                    for (uint64_t tk : sl.tickets) {
                        const Request &r = s->reqs[tk];
                        if (r.dt != dt || size_class(r.n) != c) continue;
                        for (int32_t i = 0; i < r.count; ++i) {
                            PtrItem &it = sl.items[off++];
                            it.A = (const char *)r.A + (size_t)i * r.n * r.n * es;
                            it.lam = (char *)r.lam + (size_t)i * r.n * es;
                            it.Q = (char *)r.Q + (size_t)i * r.n * r.n * es;
                            it.info = r.info ? r.info + i : nullptr;
                            it.n = r.n;
                        }
                    }
                    if (off > first) launches.push_back(Launch{dt, c, first, off - first});
                }
            // every request's input is complete on its producer stream first:
            // per producer stream, the event of its latest request covers the
            // earlier ones (work on one stream completes in order)
            hipError_t e = hipSuccess;
            std::map<hipStream_t, uint64_t> latest;
            for (uint64_t tk : sl.tickets) {
                auto &v = latest[s->reqs[tk].producer];
                v = std::max(v, tk);
            }
            std::vector<hipEvent_t> waits;
            for (const auto &kv : latest) waits.push_back(s->reqs[kv.second].ready);
            // The calls below take longer than a submission: the lock is free meanwhile,
            // and what is submitted joins the next step.  Nobody else touches the slot,
            // and the requests' events are recycled only when this thread has seen the
            // step's end.
            lk.unlock();
            for (hipEvent_t ev : waits)
                if (e == hipSuccess) e = hipStreamWaitEvent(sl.stream, ev, 0);
            for (const Launch &L : launches)
                if (e == hipSuccess)
                    e = launch_ptrlist(L.dt, class_shape(L.cls, default_tune(L.dt)), sl.items + L.off, L.count,
                                       sl.stream);
            if (e == hipSuccess) e = hipEventRecord(sl.done_ev, sl.stream);
            lk.lock();
            if (e != hipSuccess) s->error = hipGetErrorString(e);
            sl.busy = true;
            continue;
        }
        if (s->stop && s->pending.empty()) {
            bool any = false;
            for (auto &sl : s->slots) any |= sl.busy;
            if (!any) break;
        }
        // idle: wait for a submission, or poll in-flight events shortly
        bool any_busy = false;
        for (auto &sl : s->slots) any_busy |= sl.busy;
        if (any_busy)
            s->cv.wait_for(lk, std::chrono::microseconds(20));
        else
            s->cv.wait(lk, [&] { return s->stop || !s->pending.empty(); });
    }
}

extern "C" bed_status bed_server_create(bed_server **out, const bed_server_opts *o)
{
    if (!out) return fail(BED_ERR_INVALID_ARG, "server is NULL");
    *out = nullptr;
    bed_server_opts opts{};
    if (o) opts = *o;
    if (opts.streams <= 0) opts.streams = 4;
    if (opts.streams > 16) return fail(BED_ERR_INVALID_ARG, "streams must be 1..16");
    if (opts.max_step <= 0) opts.max_step = 4096;
    auto *s = new (std::nothrow) bed_server();
    if (!s) return fail(BED_ERR_NOMEM, "host allocation failed");
    s->opts = opts;
    s->adm.max_mats = opts.max_inflight;
    s->adm.max_bytes = opts.mem_budget;
    s->device = opts.device;
    if (hipSetDevice(s->device) != hipSuccess) {
        delete s;
        return fail(BED_ERR_HIP, "hipSetDevice(%d) failed", opts.device);
    }
    s->slots.resize(opts.streams);
    for (auto &sl : s->slots) {
        hipError_t e = hipStreamCreateWithFlags(&sl.stream, hipStreamNonBlocking);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&sl.done_ev, hipEventDisableTiming);
        if (e == hipSuccess)
            e = hipHostMalloc((void **)&sl.items, sizeof(PtrItem) * opts.max_step, 0);
        if (e != hipSuccess) {
            bed_server_destroy(s);
            return hip_fail(e, "server resources");
        }
    }
    s->worker = std::thread(server_loop, s);
    *out = s;
    return BED_OK;
}

extern "C" bed_status bed_server_submit(bed_server *s, bed_dtype dt, int32_t count, int32_t n,
                                        const void *A, void *lambda, void *Q, int32_t *info,
                                        void *stream, uint64_t *ticket)
{
    if (!s || !ticket) return fail(BED_ERR_INVALID_ARG, "NULL argument");
    if (count < 1) return fail(BED_ERR_INVALID_ARG, "count < 1");
    if (count > s->opts.max_step) return fail(BED_ERR_INVALID_ARG, "count > max_step");
    int32_t nn = n;
    bed_status st = check_sizes(dt, 1, &nn);
    if (st != BED_OK) return st;
    if ((st = check_ptr(A, dt, "A", false)) != BED_OK) return st;
    if ((st = check_ptr(lambda, dt, "lambda", false)) != BED_OK) return st;
    if ((st = check_ptr(Q, dt, "Q", false)) != BED_OK) return st;
    const int64_t bytes = request_bytes(count, n, dtype_size(dt));
    std::lock_guard<std::mutex> lk(s->mu);
    hipEvent_t ev = nullptr;
    if (!s->free_events.empty()) {
        ev = s->free_events.back();
        s->free_events.pop_back();
    } else {
        hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
    }
    switch (s->adm.admit(count, bytes)) {
    case ADMIT_OK: break;
    case ADMIT_INFLIGHT:
        s->free_events.push_back(ev);
        return fail(BED_ERR_BUSY, "in-flight matrix limit reached");
    case ADMIT_MEMORY:
        s->free_events.push_back(ev);
        return fail(BED_ERR_BUSY, "memory budget reached");
    }
    hipError_t e = hipEventRecord(ev, (hipStream_t)stream);
    if (e != hipSuccess) {
        s->adm.release(count, bytes);
        s->free_events.push_back(ev);
        return hip_fail(e, "hipEventRecord on the submitting stream");
    }
    Request r;
    r.ticket = s->next_ticket++;
    r.dt = dt;
    r.count = count;
    r.n = n;
    r.A = A;
    r.lam = lambda;
    r.Q = Q;
    r.info = info;
    r.bytes = bytes;
    r.ready = ev;
    r.producer = (hipStream_t)stream;
    r.t_submit = Clock::now();
    s->reqs.emplace(r.ticket, r);
    s->pending.push_back(r.ticket);
    *ticket = r.ticket;
    s->cv.notify_all();
    return BED_OK;
}

extern "C" bed_status bed_server_poll(bed_server *s, uint64_t ticket, int32_t *done,
                                      double *latency_us)
{
    if (!s || !done) return fail(BED_ERR_INVALID_ARG, "NULL argument");
    std::lock_guard<std::mutex> lk(s->mu);
    if (!s->error.empty()) return fail(BED_ERR_HIP, "server: %s", s->error.c_str());
    auto it = s->reqs.find(ticket);
    if (it == s->reqs.end()) return fail(BED_ERR_INVALID_ARG, "unknown ticket %llu",
                                         (unsigned long long)ticket);
    *done = it->second.done ? 1 : 0;
    if (latency_us) *latency_us = it->second.latency_us;
    if (it->second.done) s->reqs.erase(it);
    return BED_OK;
}

extern "C" bed_status bed_server_drain(bed_server *s)
{
    if (!s) return fail(BED_ERR_INVALID_ARG, "server is NULL");
    std::unique_lock<std::mutex> lk(s->mu);
    s->cv_done.wait(lk, [&] { return s->adm.idle() || !s->error.empty(); });
    if (!s->error.empty()) return fail(BED_ERR_HIP, "server: %s", s->error.c_str());
    return BED_OK;
}

extern "C" void bed_server_destroy(bed_server *s)
{
    if (!s) return;
    {
        std::lock_guard<std::mutex> lk(s->mu);
        s->stop = true;
        s->cv.notify_all();
    }
    if (s->worker.joinable()) s->worker.join();
    for (auto &kv : s->reqs)
        if (kv.second.ready) (void)hipEventDestroy(kv.second.ready);
    for (hipEvent_t ev : s->free_events) (void)hipEventDestroy(ev);
    for (auto &sl : s->slots) {
        if (sl.stream) (void)hipStreamSynchronize(sl.stream);
        if (sl.done_ev) (void)hipEventDestroy(sl.done_ev);
        if (sl.items) (void)hipHostFree(sl.items);
        if (sl.stream) (void)hipStreamDestroy(sl.stream);
    }
    delete s;
}
