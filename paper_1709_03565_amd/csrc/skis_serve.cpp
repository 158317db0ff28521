// skis_serve.cpp -- an influence-estimate service over a resident sketch: the query phase
// of Alg. 2 (answer any seed set from the fixed sketch, Eq. eq21) under a stream of
// requests.
//
// Continuous batching: submitters append queries to a host queue; one worker thread owns
// `depth` pipeline slots, each with its own HIP stream, pinned host staging
// and zeroed bitmap scratch.  Whenever a slot is free and queries are waiting, the
// worker takes as many as the slot admits (by count, by total entries and by large sets),
// except that a heavy set (one whose members' sample lists hold more than HEAVY_WORK entries,
// a hub's set) runs in a batch of its own: a batch completes when its slowest set does, so a
// hub set among light ones would hold them all for milliseconds, while alone it holds one
// slot and the other slots keep serving.  It packs them into the slot's pinned CSR and enqueues the estimate kernels, which read it
// and write the answers to pinned memory, on the slot's stream without waiting.  It polls the slots' completion events,
// and when a batch is done it stores each query's (Cov, I_hat) and completion time and
// wakes the waiters.  A query's result does not depend on the batch it ran in: each set
// takes its own workgroup and bitmap, and its sums run in a fixed order.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstring>
#include <deque>
#include <mutex>
#include <memory>
#include <thread>
#include <unordered_map>
#include <unordered_set>

#include "skis_internal.h"
#include "skis_query.h"

namespace {

using Clock = std::chrono::steady_clock;

struct Pending {
    uint64_t ticket;
    std::vector<int32_t> nodes;
    uint64_t work = 0; // sum of |H(v)| over the members (from the inverse index's offsets)
    Clock::time_point arrive;
};

// A set whose members' lists hold more entries than this is batched alone (about a
// millisecond of walking for one workgroup; a set of 1000 uniform members on the 4M-node TRI
// sketch holds about 60 thousand, its top hub 3 million).
constexpr uint64_t HEAVY_WORK = 1ull << 18;

// Batches of light sets in flight before the next one is held back, for as many queries as a batch
// admits, for one of them to end, for QUIET without a new query or one on its way in, HOLD_MAX at most:
// the streams share two hardware queues in most processes, where a third small batch only waits (a
// burst of 1024 Zipf sets with four in flight 1.4-1.6 ms, with two 1.25-1.5; a burst of few queries has
// nothing to wait for).  Behind a set above EST_MAX_SET members, which takes hundreds of microseconds, one
// in flight is enough (8 sets of 5000 members on 2^18 samples of a 300 thousand-node TRI graph in five
// batches 0.61 ms, in three 0.41).
constexpr auto QUIET = std::chrono::microseconds(3);
constexpr auto HOLD_MAX = std::chrono::microseconds(200);
constexpr int LIGHT_IN_FLIGHT = 2;

// a slot's error words: k_estimate's at 0, k_est_set's flags after it
constexpr int ERR_FLAGS = 4, ERR_WORDS = ERR_FLAGS + (int)(sizeof(skis::EstFlags) / sizeof(int));

struct Done {
    uint64_t cov;
    double est;
    double latency_us;
};

template <typename T>
struct Pinned {
    T *ptr = nullptr;
    T *dev = nullptr; // the same memory as the device addresses it
    size_t count = 0;
    Pinned() = default;
    Pinned(const Pinned &) = delete;
    Pinned &operator=(const Pinned &) = delete;
    ~Pinned()
    {
        if (ptr) (void)hipHostFree(ptr);
    }
    void alloc(size_t n)
    {
        SKIS_HIP_TRY(hipHostMalloc((void **)&ptr, sizeof(T) * (n ? n : 1), hipHostMallocDefault));
        SKIS_HIP_TRY(hipHostGetDevicePointer((void **)&dev, ptr, 0));
        count = n;
    }
};

struct Slot {
    hipStream_t stream = nullptr;
    hipEvent_t done = nullptr;
    Pinned<int64_t> h_ptr;
    Pinned<int32_t> h_nodes;
    Pinned<int64_t> h_large;
    Pinned<unsigned long long> h_cov;
    Pinned<double> h_est;
    skis::DevBuf<int> d_err;
    skis::DevBuf<uint32_t> bitmaps;  // max_batch_queries bitmaps of T bits
    skis::DevBuf<uint32_t> nodebits; // max_large node bitmaps of n bits
    std::vector<Pending> batch;
    bool busy = false;
    bool heavy = false; // its batch is one heavy set
};

} // namespace

struct skis_server {
    const skis_sketch *sk = nullptr;
    skis_server_options opt{};
    int device = 0;
    uint64_t wordsT = 1, wordsN = 1;
    skis::Arena arena;
    std::vector<int64_t> node_ptr;     // host copy of the inverse index's offsets (n + 1), for the work of a set
    std::vector<uint16_t> list_len;    // the lists' lengths, LONG_LIST where node_ptr tells (2 B of reads a member for
                                       // 16 from a table four times the size: a member's read was most of a submission)
    std::vector<std::unique_ptr<Slot>> slots;
    std::thread worker;
    std::mutex mu;
    std::condition_variable cv_work; // of mu
    std::condition_variable cv_done; // of done_mu
    std::deque<Pending> queue;
    std::unordered_set<uint64_t> outstanding; // submitted, not yet taken by a wait
    // of the queue, for the worker to see without the lock (written under mu): where it polled the slots
    // under the lock, submitters met it there
    alignas(64) std::atomic<size_t> queued{0};
    std::atomic<bool> front_heavy{false}, front_large{false}, batch_full{false}; // full: large sets or entries
                                                                                 // for a whole batch wait
    std::atomic<int> coming{0};                              // submissions that have begun
    uint64_t queued_large = 0, queued_entries = 0;           // under mu
    uint64_t next_ticket = 1;
    std::atomic<bool> stop{false}; // written under mu and done_mu
    std::string fault; // set when the worker stopped on an error
    // the answers, under a lock of their own: a batch's end holds it for its queries' entries, and under
    // mu submitters had waited there
    alignas(64) std::mutex done_mu;
    std::unordered_map<uint64_t, Done> results;
    // statistics (under done_mu)
    uint64_t batches = 0, queries = 0, max_batch = 0;
    uint64_t hist[16] = {};

    // a set of `entries` members has joined or left the queue
    void count(uint64_t entries, bool joined)
    {
        const uint64_t large = entries > (uint64_t)skis::EST_MAX_SET ? 1 : 0;
        queued_large = joined ? queued_large + large : queued_large - large;
        queued_entries = joined ? queued_entries + entries : queued_entries - entries;
    }
    void queue_changed()
    {
        batch_full.store(queued_large >= opt.max_large_sets || queued_entries >= opt.max_batch_entries,
                         std::memory_order_relaxed);
        queued.store(queue.size(), std::memory_order_relaxed);
        front_heavy.store(!queue.empty() && queue.front().work > HEAVY_WORK, std::memory_order_relaxed);
        front_large.store(!queue.empty() && queue.front().nodes.size() > (size_t)skis::EST_MAX_SET, std::memory_order_relaxed);
    }
    void run();
    void launch(Slot &sl);
    void complete(Slot &sl);
    ~skis_server()
    {
        for (auto &p : slots) {
            if (p->stream) (void)hipStreamSynchronize(p->stream);
            if (p->done) (void)hipEventDestroy(p->done);
            if (p->stream) (void)hipStreamDestroy(p->stream);
        }
    }
};

void skis_server::launch(Slot &sl)
{
    const skis::Sketch &k = sk->core;
    const int32_t nq = (int32_t)sl.batch.size();
    int64_t off = 0;
    int32_t nl = 0;
    for (int32_t i = 0; i < nq; ++i) {
        const auto &v = sl.batch[i].nodes;
        sl.h_ptr.ptr[i] = off;
        if (!v.empty()) std::memcpy(sl.h_nodes.ptr + off, v.data(), sizeof(int32_t) * v.size());
        off += (int64_t)v.size();
        if ((int64_t)v.size() > skis::EST_MAX_SET || sl.batch[i].work > skis::EST_WALK_MAX) sl.h_large.ptr[nl++] = i;
        sl.h_cov.ptr[i] = skis::EST_PARKED; // unanswered
    }
    sl.h_ptr.ptr[nq] = off;
    // The kernels read the sets from the pinned staging and write the answers there: a set is read once,
    // and six copies a batch had cost the worker and the queues more than the reads do (a burst of
    // 1024 Zipf sets, with k_est_set's walk: 1.55 -> 1.45 ms).
    hipStream_t s = sl.stream;
    skis::estimate_launch(k, nq, sl.h_ptr.dev, sl.h_nodes.dev, sl.h_large.dev, nl, sl.bitmaps.ptr, wordsT,
                          sl.nodebits.ptr, sl.h_cov.dev, sl.h_est.dev, sl.d_err.ptr,
                          reinterpret_cast<skis::EstFlags *>(sl.d_err.ptr + ERR_FLAGS), s);
    SKIS_HIP_TRY(hipEventRecord(sl.done, s));
    sl.busy = true;
}

void skis_server::complete(Slot &sl)
{
    for (size_t i = 0; i < sl.batch.size(); ++i)
        if (sl.h_cov.ptr[i] == skis::EST_PARKED) {
            // ids were checked at submission, so this is an internal fault: scratch may hold bits
            int err[ERR_WORDS] = {};
            SKIS_HIP_TRY(hipMemcpy(err, sl.d_err.ptr, sizeof(err), hipMemcpyDeviceToHost));
            const skis::EstFlags &fl = *reinterpret_cast<const skis::EstFlags *>(err + ERR_FLAGS);
            throw skis::Error{SKIS_EHIP, "internal error in the estimate kernel (flags " +
                                             std::to_string(err[0] | fl.ptr | 2 * fl.node) + ")"};
        }
    const auto now = Clock::now();
    const size_t nq = sl.batch.size();
    {
        std::lock_guard<std::mutex> g(done_mu);
        for (size_t i = 0; i < nq; ++i) {
            const double lat = std::chrono::duration<double, std::micro>(now - sl.batch[i].arrive).count();
            results[sl.batch[i].ticket] = Done{(uint64_t)sl.h_cov.ptr[i], sl.h_est.ptr[i], lat};
        }
        batches += 1;
        queries += nq;
        if (nq > max_batch) max_batch = nq;
        int b = 0;
        while (b < 15 && (1ull << (b + 1)) <= nq) ++b;
        hist[b] += 1;
    }
    sl.batch.clear();
    sl.busy = false;
    cv_done.notify_all();
}

void skis_server::run()
{
    try {
        SKIS_HIP_TRY(hipSetDevice(device));
        size_t had = 0;       // queries waiting at the last look
        bool holding = false; // they were held back
        Clock::time_point since{}, held{}; // since when no other has come, since when held
        for (;;) {
            // the slots are this thread's alone
            Slot *free_slot = nullptr;
            bool any_busy = false;
            int in_flight = 0; // batches of light sets
            for (auto &p : slots) {
                if (!p->busy && !free_slot) free_slot = p.get();
                any_busy |= p->busy;
                in_flight += p->busy && !p->heavy ? 1 : 0;
            }
            if (!any_busy) {
                std::unique_lock<std::mutex> g(mu);
                cv_work.wait(g, [&] { return stop || !queue.empty(); });
                if (stop && queue.empty()) return;
            }
            const size_t have = queued.load(std::memory_order_relaxed);
            bool hold = false;
            if (free_slot && have && in_flight >= (front_large.load(std::memory_order_relaxed) ? 1 : LIGHT_IN_FLIGHT) &&
                have < opt.max_batch_queries && !front_heavy.load(std::memory_order_relaxed) && !batch_full.load(std::memory_order_relaxed)) {
                const auto now = Clock::now();
                if (!holding) held = now;
                if (!holding || have != had || coming.load(std::memory_order_relaxed) > 0) since = now;
                hold = now - since < QUIET && now - held < HOLD_MAX;
            }
            holding = hold;
            had = have;
            if (!have || hold) free_slot = nullptr;
            if (free_slot) {
                std::lock_guard<std::mutex> g(mu);
                if (!queue.empty()) {
                    // admission: by count, by entries (pinned staging) and by large sets
                    Slot &sl = *free_slot;
                    uint64_t entries = 0;
                    uint32_t large = 0;
                    sl.heavy = queue.front().work > HEAVY_WORK;
                    while (!queue.empty() && sl.batch.size() < opt.max_batch_queries) {
                        const uint64_t e = queue.front().nodes.size();
                        const bool is_large = e > (uint64_t)skis::EST_MAX_SET;
                        const bool heavy = queue.front().work > HEAVY_WORK;
                        if (heavy && !sl.batch.empty()) break; // it goes alone, in the next free slot
                        if (entries + e > opt.max_batch_entries) break;
                        if (is_large && large >= opt.max_large_sets) break;
                        entries += e;
                        large += is_large ? 1u : 0u;
                        sl.batch.push_back(std::move(queue.front()));
                        queue.pop_front();
                        count(e, false);
                        if (heavy) break;
                    }
                    queue_changed();
                }
            }
            if (free_slot && !free_slot->batch.empty()) {
                launch(*free_slot);
                continue;
            }
            // nothing to launch now: finish every batch that is done (in any order, so a
            // slow batch holds only its own queries), else poll again
            bool progressed = false;
            for (auto &p : slots) {
                if (!p->busy) continue;
                const hipError_t q = hipEventQuery(p->done);
                if (q == hipSuccess) {
                    complete(*p);
                    progressed = true;
                } else if (q != hipErrorNotReady) {
                    SKIS_HIP_TRY(q);
                }
            }
            if (!progressed) std::this_thread::yield();
        }
    } catch (const skis::Error &e) {
        std::scoped_lock g(mu, done_mu);
        fault = e.msg;
        stop = true;
        cv_done.notify_all();
    } catch (const std::exception &e) {
        std::scoped_lock g(mu, done_mu);
        fault = e.what();
        stop = true;
        cv_done.notify_all();
    }
}

namespace {

template <typename F>
int serve_guarded(F &&f)
{
    try {
        skis::set_error("");
        return f();
    } catch (const skis::Error &e) {
        skis::set_error(e.msg);
        return e.code;
    } catch (const std::bad_alloc &) {
        skis::set_error("host allocation failed");
        return SKIS_ENOMEM;
    } catch (const std::exception &e) {
        skis::set_error(e.what());
        return SKIS_EHIP;
    }
}

int submit_one(skis_server *sv, const int32_t *nodes, int32_t count, Clock::time_point arrive, uint64_t *ticket)
{
    struct Coming {
        std::atomic<int> &n;
        explicit Coming(std::atomic<int> &x) : n(x) { n.fetch_add(1, std::memory_order_relaxed); }
        ~Coming() { n.fetch_sub(1, std::memory_order_relaxed); }
    } on_its_way(sv->coming);
    if (count < 0) throw skis::Error{SKIS_EINVAL, "count must be >= 0"};
    if (count > 0 && !nodes) throw skis::Error{SKIS_EINVAL, "nodes must not be NULL"};
    if ((uint64_t)count > sv->opt.max_batch_entries)
        throw skis::Error{SKIS_EINVAL, "set larger than max_batch_entries"};
    const int32_t n = sv->sk->core.n;
    for (int32_t i = 0; i < count; ++i)
        if (nodes[i] < 0 || nodes[i] >= n) throw skis::Error{SKIS_EINVAL, "a seed set holds a node id outside [0, n)"};
    Pending p;
    p.nodes.assign(nodes, nodes + count);
    if (!sv->node_ptr.empty()) p.work = skis::list_entries(sv->list_len.data(), sv->node_ptr.data(), nodes, count);
    p.arrive = arrive;
    {
        std::lock_guard<std::mutex> g(sv->mu);
        if (sv->stop) throw skis::Error{SKIS_EHIP, "server stopped: " + sv->fault};
        p.ticket = sv->next_ticket++;
        sv->outstanding.insert(p.ticket);
        if (ticket) *ticket = p.ticket;
        sv->queue.push_back(std::move(p));
        sv->count((uint64_t)count, true);
        sv->queue_changed();
    }
    sv->cv_work.notify_one();
    return SKIS_OK;
}

int wait_one(skis_server *sv, uint64_t ticket, uint64_t *cov, double *est, double *latency_us)
{
    {
        std::lock_guard<std::mutex> g(sv->mu);
        if (!sv->outstanding.erase(ticket)) throw skis::Error{SKIS_EINVAL, "unknown or already collected ticket"};
    }
    {
        std::unique_lock<std::mutex> g(sv->done_mu);
        sv->cv_done.wait(g, [&] { return sv->results.count(ticket) || sv->stop; });
        auto it = sv->results.find(ticket);
        if (it != sv->results.end()) {
            if (cov) *cov = it->second.cov;
            if (est) *est = it->second.est;
            if (latency_us) *latency_us = it->second.latency_us;
            sv->results.erase(it);
            return SKIS_OK;
        }
    }
    std::lock_guard<std::mutex> g(sv->mu);
    sv->outstanding.insert(ticket); // not collected
    throw skis::Error{SKIS_EHIP, "server stopped: " + sv->fault};
}

} // namespace

extern "C" {

void skis_server_default_options(skis_server_options *opt)
{
    if (!opt) return;
    std::memset(opt, 0, sizeof(*opt));
    opt->pipeline_depth = 4;
    opt->max_batch_queries = 256;
    opt->max_batch_entries = 1u << 20;
    opt->max_large_sets = 4;
}

int skis_server_create(const skis_sketch *sk, const skis_server_options *opt_in, skis_server **out)
{
    return serve_guarded([&]() -> int {
        if (!out) throw skis::Error{SKIS_EINVAL, "out must not be NULL"};
        *out = nullptr;
        if (!sk) throw skis::Error{SKIS_EINVAL, "NULL sketch"};
        if (!sk->core.has_inverse && sk->core.T > 0)
            throw skis::Error{SKIS_EINVAL, "the sketch was built without the inverse index"};
        skis_server_options opt;
        skis_server_default_options(&opt);
        if (opt_in) {
            if (opt_in->pipeline_depth) opt.pipeline_depth = opt_in->pipeline_depth;
            if (opt_in->max_batch_queries) opt.max_batch_queries = opt_in->max_batch_queries;
            if (opt_in->max_batch_entries) opt.max_batch_entries = opt_in->max_batch_entries;
            if (opt_in->max_large_sets) opt.max_large_sets = opt_in->max_large_sets;
            opt.max_device_bytes = opt_in->max_device_bytes;
        }
        if (opt.pipeline_depth > 16 || opt.max_batch_queries > (1u << 20))
            throw skis::Error{SKIS_EINVAL, "pipeline_depth must be <= 16 and max_batch_queries <= 2^20"};
        auto sv = std::make_unique<skis_server>();
        sv->sk = sk;
        sv->opt = opt;
        SKIS_HIP_TRY(hipGetDevice(&sv->device));
        sv->arena.cap = opt.max_device_bytes;
        sv->wordsT = sk->core.T ? (sk->core.T + 31) / 32 : 1;
        sv->wordsN = ((uint64_t)sk->core.n + 31) / 32;
        if (sk->core.T > 0 && sk->core.node_ptr.ptr) {
            sv->node_ptr.resize((size_t)sk->core.n + 1);
            SKIS_HIP_TRY(hipMemcpy(sv->node_ptr.data(), sk->core.node_ptr.ptr, sizeof(int64_t) * ((size_t)sk->core.n + 1),
                                   hipMemcpyDeviceToHost));
            sv->list_len.resize((size_t)sk->core.n);
            for (int32_t v = 0; v < sk->core.n; ++v)
                sv->list_len[v] = (uint16_t)std::min<int64_t>(sv->node_ptr[v + 1] - sv->node_ptr[v], skis::LONG_LIST);
        }
        const uint64_t nb = std::max<uint64_t>(opt.max_batch_queries, opt.max_large_sets);
        sv->arena.stream = nullptr; // allocations complete before any slot stream uses them (below)
        for (uint32_t i = 0; i < opt.pipeline_depth; ++i) {
            sv->slots.push_back(std::make_unique<Slot>());
            Slot &s = *sv->slots.back();
            SKIS_HIP_TRY(hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking));
            SKIS_HIP_TRY(hipEventCreateWithFlags(&s.done, hipEventDisableTiming));
            s.h_ptr.alloc(opt.max_batch_queries + 1);
            s.h_nodes.alloc(opt.max_batch_entries);
            s.h_large.alloc(opt.max_large_sets);
            s.h_cov.alloc(opt.max_batch_queries);
            s.h_est.alloc(opt.max_batch_queries);
            s.d_err.alloc(sv->arena, ERR_WORDS);
            s.bitmaps.alloc(sv->arena, nb * sv->wordsT);
            s.nodebits.alloc(sv->arena, (uint64_t)opt.max_large_sets * sv->wordsN);
            SKIS_HIP_TRY(hipDeviceSynchronize());
            skis::fill_u32(s.bitmaps.ptr, nb * sv->wordsT, s.stream);
            skis::fill_u32(s.nodebits.ptr, (uint64_t)opt.max_large_sets * sv->wordsN, s.stream);
            skis::fill_u32(reinterpret_cast<uint32_t *>(s.d_err.ptr), ERR_WORDS, s.stream);
            SKIS_HIP_TRY(hipStreamSynchronize(s.stream));
        }
        skis_server *raw = sv.get();
        sv->worker = std::thread([raw] { raw->run(); });
        *out = sv.release();
        return SKIS_OK;
    });
}

int skis_server_submit(skis_server *sv, const int32_t *nodes, int32_t count, uint64_t *ticket)
{
    return serve_guarded([&]() -> int {
        if (!sv) throw skis::Error{SKIS_EINVAL, "NULL server"};
        return submit_one(sv, nodes, count, Clock::now(), ticket);
    });
}

int skis_server_wait(skis_server *sv, uint64_t ticket, uint64_t *cov, double *est, double *latency_us)
{
    return serve_guarded([&]() -> int {
        if (!sv) throw skis::Error{SKIS_EINVAL, "NULL server"};
        return wait_one(sv, ticket, cov, est, latency_us);
    });
}

int skis_server_replay(skis_server *sv, int32_t num_queries, const int64_t *set_ptr, const int32_t *set_nodes,
                       const double *arrival_us, uint64_t *cov, double *est, double *latency_us)
{
    return serve_guarded([&]() -> int {
        if (!sv) throw skis::Error{SKIS_EINVAL, "NULL server"};
        if (num_queries < 0 || (num_queries > 0 && (!set_ptr || !arrival_us)))
            throw skis::Error{SKIS_EINVAL, "bad replay arguments"};
        for (int32_t i = 0; i < num_queries; ++i) {
            if (set_ptr[i + 1] < set_ptr[i] || set_ptr[i] < 0 || set_ptr[i + 1] - set_ptr[i] > INT32_MAX)
                throw skis::Error{SKIS_EINVAL, "set_ptr must be nondecreasing from 0"};
            if (i > 0 && arrival_us[i] < arrival_us[i - 1])
                throw skis::Error{SKIS_EINVAL, "arrival times must be nondecreasing"};
        }
        std::vector<uint64_t> tickets((size_t)num_queries);
        const Clock::time_point t0 = Clock::now();
        Clock::time_point now = t0;
        for (int32_t i = 0; i < num_queries; ++i) {
            const auto due = t0 + std::chrono::duration_cast<Clock::duration>(
                                      std::chrono::duration<double, std::micro>(arrival_us[i]));
            while (now < due) now = Clock::now(); // open loop: submit at the scheduled time, whatever is still in flight
            submit_one(sv, set_nodes + set_ptr[i], (int32_t)(set_ptr[i + 1] - set_ptr[i]), due, &tickets[i]);
        }
        for (int32_t i = 0; i < num_queries; ++i) {
            uint64_t c = 0;
            double e = 0, l = 0;
            wait_one(sv, tickets[i], &c, &e, &l);
            if (cov) cov[i] = c;
            if (est) est[i] = e;
            if (latency_us) latency_us[i] = l;
        }
        return SKIS_OK;
    });
}

int skis_server_get_stats(skis_server *sv, skis_server_stats *st)
{
    return serve_guarded([&]() -> int {
        if (!sv || !st) throw skis::Error{SKIS_EINVAL, "NULL argument"};
        std::lock_guard<std::mutex> g(sv->done_mu);
        std::memset(st, 0, sizeof(*st));
        st->batches = sv->batches;
        st->queries = sv->queries;
        st->max_batch = sv->max_batch;
        st->device_bytes = sv->arena.used;
        for (int i = 0; i < 16; ++i) st->batch_hist[i] = sv->hist[i];
        return SKIS_OK;
    });
}

void skis_server_destroy(skis_server *sv)
{
    if (!sv) return;
    {
        std::scoped_lock g(sv->mu, sv->done_mu);
        sv->stop = true;
    }
    sv->cv_work.notify_all();
    if (sv->worker.joinable()) sv->worker.join();
    delete sv;
}

} // extern "C"
