// Batched solves: many independent problems (each with all of its modes)
// driven together, in two forms side by side.
//
// Grouped (mixed-precision problems on the pair march or the strip kernels): each
// stage of the refinement step is one launch for all of them.  A few steps are
// captured into one HIP graph and replayed; inside a replay the device runs the
// convergence test and retires converged modes (and so finished problems, whose
// workgroups then exit at once); the host reads the active counts after each replay
// and re-captures when the set has shrunk enough to pay off.
//
// Per problem (all others, FP64 among them): problems are dealt to a few streams
// and the host queues a V-cycle and a test of every unfinished one before it looks
// at the states of the tests before, as for a single solve, so the streams do not
// wait for the host.  Nothing is captured: replayed graphs of one branch per stream
// (13 FP64 boxes) ended a process once with a corrupted heap, cause unknown; that
// form made its kernels' first occupancy queries inside a capture, and destroyed
// graphs the moment their last replay had ended.  24 FP64 boxes of 64 to 384 cells:
// 44.0 ms a batch in branches over strip kernels, 26.8 here; 32 of 32 to 96 cells
// 14.0 and 6.2.
//
// The number of streams and the steps per replay come from a small online
// autotuner, cached per batch signature; streams and events are pooled.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

#include "internal.h"

namespace mbp {

namespace {

struct BatchTune {
    int streams = 4;       // per-problem form
    int chunk = 4;         // grouped form: cycles a replay
    bool grouped = false;  // every problem of the set's last batch ran in the grouped form
};

std::mutex g_tune_mu;
std::map<uint64_t, BatchTune> g_tune;

uint64_t mix(uint64_t h, uint64_t v) {
    h ^= v + 0x9e3779b97f4a7c15ULL + (h << 6) + (h >> 2);
    return h;
}

uint64_t batch_signature(mbp_plan* const* plans, int count) {
    uint64_t h = 1469598103934665603ULL;
    for (int i = 0; i < count; ++i) {
        h = mix(h, uint64_t(plans[i]->ncells));
        h = mix(h, uint64_t(plans[i]->g.nz));
        h = mix(h, uint64_t(plans[i]->opt.precision));
    }
    return h;
}

constexpr int kMaxStreams = 8;

struct Graph {
    hipGraph_t g = nullptr;
    hipGraphExec_t e = nullptr;
    std::vector<int> members;
    long long modes = 0;  // active modes captured (grid sizes)
    void reset() {
        if (e) (void)hipGraphExecDestroy(e);
        if (g) (void)hipGraphDestroy(g);
        e = nullptr;
        g = nullptr;
        members.clear();
        modes = 0;
    }
};

// Streams and events of one batch call, kept for later calls on the same
// device (creating them costs about as much as a small problem's cycle).
struct StreamSet {
    int dev = -1;
    hipStream_t st[kMaxStreams] = {};
    hipStream_t cap = nullptr;  // captures graphs, runs nothing
    hipEvent_t ev_join[kMaxStreams] = {};
    hipEvent_t ev_fork = nullptr, t0 = nullptr, t1 = nullptr;
};
std::mutex g_pool_mu;
std::vector<StreamSet*> g_pool;

StreamSet* acquire_streams() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        for (size_t i = 0; i < g_pool.size(); ++i)
            if (g_pool[i]->dev == dev) {
                StreamSet* p = g_pool[i];
                g_pool.erase(g_pool.begin() + long(i));
                return p;
            }
    }
    StreamSet* p = new StreamSet;
    p->dev = dev;
    bool ok = true;
    for (int k = 0; k < kMaxStreams; ++k) {
        ok = ok && hipStreamCreateWithFlags(&p->st[k], hipStreamNonBlocking) == hipSuccess;
        ok = ok && hipEventCreateWithFlags(&p->ev_join[k], hipEventDisableTiming) == hipSuccess;
    }
    ok = ok && hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&p->ev_fork, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreate(&p->t0) == hipSuccess && hipEventCreate(&p->t1) == hipSuccess;
    if (!ok) {
        for (int k = 0; k < kMaxStreams; ++k) {
            if (p->st[k]) (void)hipStreamDestroy(p->st[k]);
            if (p->ev_join[k]) (void)hipEventDestroy(p->ev_join[k]);
        }
        if (p->cap) (void)hipStreamDestroy(p->cap);
        if (p->ev_fork) (void)hipEventDestroy(p->ev_fork);
        if (p->t0) (void)hipEventDestroy(p->t0);
        if (p->t1) (void)hipEventDestroy(p->t1);
        delete p;
        return nullptr;
    }
    return p;
}

void release_streams(StreamSet* p) {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    g_pool.push_back(p);
}

}  // namespace

int solve_batch(mbp_plan* const* plans, const double* const* rhs, double* const* p, int count,
                double rtol, int flags, hipStream_t s, mbp_solve_info* infos) {
    std::vector<SolveCtx> cx(count);
    for (int i = 0; i < count; ++i)
        ctx_init(cx[i], plans[i], rhs[i], p[i], rtol, flags | plans[i]->opt.flags | MBP_RETIRE);

    const uint64_t sig = batch_signature(plans, count);
    BatchTune tune;
    bool have = false;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune.find(sig);
        if (it != g_tune.end()) {
            tune = it->second;
            have = true;
        }
    }

    // all of the streams are forked from s
    StreamSet* ss = acquire_streams();
    if (!ss) return MBP_ERR_HIP;
    hipStream_t* st = ss->st;
    hipEvent_t* ev_join = ss->ev_join;
    hipEvent_t ev_fork = ss->ev_fork, t0 = ss->t0, t1 = ss->t1;
    auto fork = [&](hipStream_t from, int S) {
        (void)hipEventRecord(ev_fork, from);
        for (int k = 0; k < S; ++k)
            if (st[k] != from) (void)hipStreamWaitEvent(st[k], ev_fork, 0);
    };
    auto join = [&](hipStream_t to, int S) {
        for (int k = 0; k < S; ++k) {
            if (st[k] == to) continue;
            (void)hipEventRecord(ev_join[k], st[k]);
            (void)hipStreamWaitEvent(to, ev_join[k], 0);
        }
    };
    int status = MBP_OK;
    auto fail = [&](int e) {
        if (status == MBP_OK) status = e;
    };

    // prologue of every problem, then the checks that need the host
    const int S = std::min(std::max(1, tune.streams), std::min(count, kMaxStreams));
    fork(s, S);
    for (int i = 0; i < count; ++i) ctx_prologue(cx[i], st[i % S]);
    join(s, S);
    if (hipStreamSynchronize(s) != hipSuccess) fail(MBP_ERR_HIP);
    for (int i = 0; i < count && status == MBP_OK; ++i) ctx_check(cx[i]);

    // problems whose whole hierarchy fits in LDS: one launch each; the others join
    // the group or run on their own
    std::vector<int> group, single;
    int inner = -1;  // of the group
    if (status == MBP_OK) {
        fork(s, S);
        for (int i = 0; i < count; ++i) {
            SolveCtx& c = cx[i];
            if (c.done) continue;
            if (c.full_lds) {
                mbp_plan* P = c.P;
                launch_lds_full(P, P->phat, P->fhat, P->d_act, P->d_nact, P->g.nz, P->opt.max_cycles, c.rtol2,
                                c.etol2, P->d_cyc, P->d_rnorm, P->d_fnorm, st[i % S]);
                c.done = true;
                continue;
            }
            const bool in = group_ok(c) && (inner < 0 || c.P->opt.inner == inner);
            if (in) inner = c.P->opt.inner;
            (in ? group : single).push_back(i);
        }
        join(s, S);
    }
    const bool all_grouped = !group.empty() && single.empty();
    const bool retuning = (flags & MBP_AUTOTUNE) && !have;
    auto drop_done = [&](std::vector<int>& v) {
        v.erase(std::remove_if(v.begin(), v.end(), [&](int i) { return cx[i].done; }), v.end());
    };
    // candidates of one form: cost per active mode-cell and cycle between t0 and t1
    struct Trials {
        std::vector<int> value;
        size_t at = 0;
        double best_cost = 1e300;
        int best = 0;
        bool open() const { return at < value.size(); }
        void note(double cost) {
            if (cost < best_cost) {
                best_cost = cost;
                best = value[at];
            }
            ++at;
        }
    };
    auto cost_of = [&](const std::vector<int>& v, int cycles) {
        float ms = 0.0f;
        (void)hipEventElapsedTime(&ms, t0, t1);
        double work = 0.0;
        for (int i : v) work += double(cx[i].nitems) * double(cx[i].P->plane0);
        return ms / std::max(1.0, work * cycles);
    };

    // ---- per-problem form ----
    struct Test {
        unsigned seq = 0;
        int slot = 0;
        bool open = false;  // its state has not been looked at
    };
    std::vector<Test> test(count);
    std::vector<int> on(count);  // stream of each problem
    int dealt = 0;
    auto deal = [&](int streams) {
        dealt = std::min(std::max(1, streams), std::min(int(single.size()), kMaxStreams));
        for (size_t a = 0; a < single.size(); ++a) on[single[a]] = int(a) % dealt;
        fork(s, dealt);
    };
    auto queue_cycle = [&](int i) {  // V-cycle and test; the test before it
        const Test t = test[i];
        ctx_vcycle(cx[i], st[on[i]]);
        const int slot = (t.slot + 1) % kStateSlots;
        test[i] = Test{ctx_test(cx[i], st[on[i]], slot), slot, true};
        return t;
    };
    std::vector<Test> before;
    auto round = [&] {  // a cycle of every problem, then the states before it
        before.clear();
        for (int i : single) before.push_back(queue_cycle(i));
        for (size_t a = 0; a < single.size(); ++a) {
            SolveCtx& c = cx[single[a]];
            if (!before[a].open) continue;
            const int r = ctx_wait(c, st[on[single[a]]], before[a].slot, before[a].seq);
            if (r != MBP_OK) fail(r);
            else ctx_state_apply(c, before[a].slot);
        }
        drop_done(single);
    };
    if (status == MBP_OK && !single.empty()) {
        deal(tune.streams);
        for (int i : single) test[i] = Test{ctx_test(cx[i], st[on[i]], 0), 0, true};
    }

    // ---- grouped form, with rounds of the others beside each replay ----
    Graph G, last;          // a graph replaced by a smaller one is destroyed a replay later
    void* table = nullptr;  // stage tables
    size_t table_bytes = 0;
    Trials chunks;
    if (retuning && !group.empty()) chunks.value = {4, 2, 8};
    while (status == MBP_OK && !group.empty()) {
        long long modes = 0;
        for (int i : group) modes += cx[i].nitems;
        const bool retune = chunks.open();
        if (retune) tune.chunk = chunks.value[chunks.at];
        if (G.e == nullptr || retune || group.size() < G.members.size() || modes * 4 < G.modes * 3) {
            last.reset();
            std::swap(last, G);
            std::vector<GStage> stages;
            std::vector<SolveCtx*> cs;
            int maxL = 0;
            for (int i : group) {
                cs.push_back(&cx[i]);
                maxL = std::max(maxL, cx[i].P->lds_level32);
            }
            GroupBlob gb;
            stages.push_back(group_res32(gb, cs));
            stages.push_back(group_finish(gb, cs));
            stages.push_back(group_update(gb, cs));
            for (int k = 0; k < inner; ++k) {
                // each level's problems: those of the pair march, then the strip kernels'
                for (int l = 0; l < maxL; ++l) {
                    stages.push_back(group_pair32(gb, cs, l, true, k, inner));
                    stages.push_back(group_march32(gb, cs, l, false, k == 0));
                }
                for (int form = 0; form < 3; ++form) stages.push_back(group_coarse32(gb, cs, form, k, inner));
                stages.push_back(group_lds32(gb, cs));
                for (int l = maxL - 1; l >= 0; --l) {
                    stages.push_back(group_pair32(gb, cs, l, false, k, inner));
                    stages.push_back(group_march32(gb, cs, l, true, false));
                }
            }
            stages.push_back(group_addcorr(gb, cs));
            if (gb.host.size() > table_bytes) {
                if (table) (void)hipFree(table);
                table = nullptr;
                table_bytes = 0;
                if (hipMalloc(&table, gb.host.size()) != hipSuccess) {
                    fail(MBP_ERR_NOMEM);
                    break;
                }
                table_bytes = gb.host.size();
            }
            if (hipMemcpy(table, gb.host.data(), gb.host.size(), hipMemcpyHostToDevice) != hipSuccess) {
                fail(MBP_ERR_HIP);
                break;
            }
            // (every kernel's occupancy and LDS limit were settled with its stage)
            if (hipStreamBeginCapture(ss->cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
                fail(MBP_ERR_HIP);
                break;
            }
            const unsigned char* dev = static_cast<const unsigned char*>(table);
            for (int it = 0; it < tune.chunk; ++it)
                for (const GStage& g : stages) {
                    if (g.kind == G_PRE32 || g.kind == G_POST32) group_launch_march(g, dev, ss->cap);
                    else if (g.kind >= G_PAIR_PRE) group_launch_pair(g, dev, ss->cap);
                    else if (g.kind >= G_COARSE0) group_launch_coarse(g, dev, ss->cap);
                    else group_launch_mg(g, dev, ss->cap);
                }
            if (hipStreamEndCapture(ss->cap, &G.g) != hipSuccess ||
                hipGraphInstantiate(&G.e, G.g, nullptr, nullptr, 0) != hipSuccess) {
                (void)hipGetLastError();
                G.reset();
                fail(MBP_ERR_HIP);
                break;
            }
            G.members = group;
            G.modes = modes;
        }
        (void)hipEventRecord(t0, s);
        if (hipGraphLaunch(G.e, s) != hipSuccess) {
            fail(MBP_ERR_HIP);
            break;
        }
        (void)hipEventRecord(t1, s);
        for (int k = 0; k < tune.chunk && !retuning && !single.empty() && status == MBP_OK; ++k) round();
        if (hipStreamSynchronize(s) != hipSuccess) {
            fail(MBP_ERR_HIP);
            break;
        }
        if (retune) {
            chunks.note(cost_of(group, tune.chunk));
            if (!chunks.open()) tune.chunk = chunks.best;
        }
        for (int i : group) ctx_state_apply(cx[i]);
        drop_done(group);
    }
    if (chunks.at > 0) tune.chunk = chunks.best;  // (the batch may have finished before every candidate ran)

    // ---- what is left of the others ----
    Trials streams;
    if (retuning && !single.empty()) streams.value = {4, 1, 8, 2};
    while (status == MBP_OK && !single.empty()) {
        if (!streams.open()) {
            round();
            continue;
        }
        // one cycle of every problem alone on this candidate's streams
        join(s, dealt);
        (void)hipEventRecord(t0, s);
        deal(streams.value[streams.at]);
        for (int i : single) (void)queue_cycle(i);
        join(s, dealt);
        (void)hipEventRecord(t1, s);
        if (hipStreamSynchronize(s) != hipSuccess) {
            fail(MBP_ERR_HIP);
            break;
        }
        streams.note(cost_of(single, 1));
        for (int i : single) {
            ctx_state_apply(cx[i], test[i].slot);
            test[i].open = false;
        }
        drop_done(single);
        if (!streams.open() && !single.empty()) deal(streams.best);
    }
    if (streams.at > 0) tune.streams = streams.best;
    join(s, dealt);  // finished problems have a cycle and a test queued that do nothing
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        if (chunks.at + streams.at > 0) g_tune[sig] = tune;
        auto it = g_tune.find(sig);
        if (it != g_tune.end()) it->second.grouped = all_grouped;
    }

    // epilogue and results
    fork(s, S);
    for (int i = 0; i < count; ++i) ctx_epilogue(cx[i], st[i % S]);
    join(s, S);
    for (int i = 0; i < count; ++i) {
        const int r = ctx_info(cx[i], s, infos ? &infos[i] : nullptr);
        if (r != MBP_OK) fail(r);
        else if (cx[i].status != MBP_OK) fail(cx[i].status);
    }
    G.reset();
    last.reset();
    if (table) (void)hipFree(table);
    release_streams(ss);
    return status;
}

// Schedule chosen for a batch signature (for reports and tests).
int batch_tuning(mbp_plan* const* plans, int count, int* streams, int* chunk) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune.find(batch_signature(plans, count));
    if (it == g_tune.end()) return MBP_PENDING;
    *streams = it->second.grouped ? 0 : it->second.streams;
    *chunk = it->second.chunk;
    return MBP_OK;
}

}  // namespace mbp
