// The request server's policy on the host: slg_server.cpp with the queries'
// device work replaced by scripted reservations. One scenario per run.
#include <cstdio>
#include <cstring>

#include "slg_server.cpp"

struct slg_context {};
struct slg_graph {};
struct slg_result {
    std::shared_ptr<slg::ServeCore> core;
    uint64_t bytes = 0;
};

namespace {
struct Script {  // one query's reservations, and what happens before and after them
    uint64_t plan, stores, output;
    std::function<void()> before_output, after_refusal;
};
std::vector<Script> scripts;  // by the query's first threshold less one
}  // namespace

// --- stand-ins ---------------------------------------------------------
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }

namespace slg {
Arena::Arena(int device, uint64_t limit) : device_(device), limit_(limit) {}
Arena::~Arena() {}
Arena::Event::~Event() {}
int context_device(const slg_context *) { return 0; }
const slg_context *graph_context(const slg_graph *) { return nullptr; }
slg_status set_error(slg_context *, slg_status code, const char *) { return code; }
slg_status create_context(int, uint64_t, const slg_allocator *, bool, slg_context **out) {
    *out = new slg_context();
    return SLG_OK;
}
void copy_tuning(slg_context *, const slg_context *) {}
void share_arena(slg_context *, const std::shared_ptr<Arena> &) {}

slg_status serve_query(slg_context *, slg_graph *, const int32_t *s, int32_t, hipStream_t, const ReserveFn &reserve,
                       const std::shared_ptr<ServeCore> &core, slg_result **out, uint64_t *scratch_bytes,
                       uint64_t *output_bytes, bool lean, uint64_t *stores) {
    const Script &q = scripts[s[0] - 1];
    *out = nullptr;
    *scratch_bytes = *output_bytes = 0;
    auto take = [&](uint64_t bytes, uint64_t *sum) {
        if (!reserve(bytes)) {
            if (q.after_refusal) q.after_refusal();
            return false;
        }
        *sum += bytes;
        return true;
    };
    if (!take(q.plan, scratch_bytes)) return SLG_ERR_OUT_OF_MEMORY;
    if (!lean) *stores = q.stores;
    if (!take(q.plan + (lean ? 0 : q.stores), scratch_bytes)) return SLG_ERR_OUT_OF_MEMORY;
    if (q.before_output) q.before_output();
    if (!take(q.output, output_bytes)) return SLG_ERR_OUT_OF_MEMORY;
    *out = new slg_result{core, q.output};
    return SLG_OK;
}
}  // namespace slg

extern "C" {
slg_status slg_context_destroy(slg_context *c) {
    delete c;
    return SLG_OK;
}
slg_status slg_result_info(const slg_result *, int32_t, int64_t *e, int64_t *w) {
    *e = *w = 0;
    return SLG_OK;
}
slg_status slg_result_free(slg_result *r) {
    r->core->release(r->bytes, true);
    delete r;
    return SLG_OK;
}
const char *slg_last_error(const slg_context *) { return "out of memory"; }
}

namespace {
uint64_t submit(slg_server *sv, int query) {
    static slg_graph g;
    const int32_t s = query + 1;
    uint64_t t = 0;
    if (slg_server_submit(sv, &g, &s, 1, &t) != SLG_OK) std::exit(2);
    return t;
}

void report(slg_server *sv, uint64_t ticket, slg_result **out) {
    slg_request_info info{};
    const slg_status st = slg_server_wait(sv, ticket, 20000, out, &info);
    std::printf("status %d attempts %d message %s\n", (int)st, info.attempts, info.message[0] ? info.message : "-");
}

void stop(slg_server *sv) {  // as slg_server_destroy begins
    std::lock_guard<std::mutex> lk(sv->core->mu);
    sv->stop = true;
    sv->core->cv.notify_all();
}
}  // namespace

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "";
    slg_context ctx;
    slg_server *sv = nullptr;
    if (slg_server_create(&ctx, 2, 100, &sv) != SLG_OK) return 2;
    slg_result *held = nullptr, *r = nullptr;
    scripts.resize(3);
    scripts[0] = {5, 0, 60, nullptr, nullptr};
    if (!std::strcmp(what, "output_waits")) {
        // a result holds 60 of 100: the second query's stores fit, its output
        // (40 more) does not until the result is freed
        std::mutex mu;
        std::condition_variable cv;
        bool reached = false;
        scripts[1] = {5, 10, 40, [&] {
                          std::lock_guard<std::mutex> lk(mu);
                          reached = true;
                          cv.notify_all();
                      }, nullptr};
        report(sv, submit(sv, 0), &held);
        const uint64_t t = submit(sv, 1);
        {
            std::unique_lock<std::mutex> lk(mu);
            if (!cv.wait_for(lk, std::chrono::seconds(20), [&] { return reached; })) return 3;
        }
        for (int i = 0; i < 2000; ++i) {  // until it waits for the memory, or has been sent back
            std::unique_lock<std::mutex> lk(sv->core->mu);
            if (sv->waiter || sv->live[t]->attempts > 1) break;
            lk.unlock();
            std::this_thread::sleep_for(std::chrono::milliseconds(1));
        }
        slg_result_free(held);
        report(sv, t, &r);
    } else if (!std::strcmp(what, "output_fits_without")) {
        // 60 held, 20 of scratch of which 10 are stores, 25 of output: 105
        scripts[1] = {5, 10, 25, nullptr, nullptr};
        report(sv, submit(sv, 0), &held);
        report(sv, submit(sv, 1), &r);
        slg_result_free(held);
    } else if (!std::strcmp(what, "output_never_fits_beside")) {
        // 40 of scratch of which 30 are stores, 70 of output
        scripts[0].output = 10;
        scripts[1] = {5, 30, 70, nullptr, nullptr};
        report(sv, submit(sv, 0), &held);
        report(sv, submit(sv, 1), &r);
        slg_result_free(held);
    } else if (!std::strcmp(what, "output_never_fits")) {
        scripts[1] = {5, 30, 95, nullptr, nullptr};
        report(sv, submit(sv, 0), &held);
        report(sv, submit(sv, 1), &r);
        slg_result_free(held);
    } else if (!std::strcmp(what, "stores_refused")) {
        // the stores do not fit beside the result: planned again without them
        scripts[1] = {5, 50, 20, nullptr, nullptr};
        report(sv, submit(sv, 0), &held);
        report(sv, submit(sv, 1), &r);
        slg_result_free(held);
    } else if (!std::strcmp(what, "shutdown_after_refusal")) {
        // the same, but the server stops before the query is back in the queue
        scripts[1] = {5, 50, 20, nullptr, [&] { stop(sv); }};
        report(sv, submit(sv, 0), &held);
        report(sv, submit(sv, 1), &r);
        slg_result_free(held);
    } else if (!std::strcmp(what, "shutdown_after_yield")) {
        // one query waits for memory, a second is sent back because of it, and
        // the server stops before it is back in the queue
        std::mutex mu;
        std::condition_variable cv;
        bool waits = false;
        scripts[1] = {5, 0, 50, nullptr, nullptr};
        scripts[2] = {5, 0, 80, [&] {
                          std::unique_lock<std::mutex> lk(mu);
                          cv.wait_for(lk, std::chrono::seconds(20), [&] { return waits; });
                      }, [&] { stop(sv); }};
        report(sv, submit(sv, 0), &held);
        const uint64_t back = submit(sv, 2);
        while (true) {  // it has its scratch and is about to ask for the output
            std::lock_guard<std::mutex> lk(sv->core->mu);
            if (sv->core->used == 70) break;
        }
        const uint64_t first = submit(sv, 1);
        while (true) {
            std::lock_guard<std::mutex> lk(sv->core->mu);
            if (sv->waiter) break;
        }
        {
            std::lock_guard<std::mutex> lk(mu);
            waits = true;
            cv.notify_all();
        }
        report(sv, back, &r);
        report(sv, first, &r);
        slg_result_free(held);
    } else {
        return 2;
    }
    if (r) slg_result_free(r);
    std::printf("used %llu\n", (unsigned long long)sv->core->used);
    slg_server_destroy(sv);
    return 0;
}
