// batch.cpp -- spin_trotter_evolve_batch: many independent problems of
// uneven size in one launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <list>
#include <map>
#include <memory>
#include <mutex>
#include <sstream>
#include <vector>

#include "../../include/spin.h"
#include "abi_internal.hpp"
#include "kept.hpp"
#include "kernels.hpp"
#include "planner.hpp"

namespace spinqp {

// ------------------------------------------------------- persistent batch
// What the couplings decide: plans, tables and the schedule.  Read-only once
// built, and shared by the calls that differ in states, seeds and outputs only.
struct BatchTables {
    void *d_jobs = nullptr, *d_jstart = nullptr, *d_passes = nullptr, *d_stages = nullptr, *d_ops = nullptr,
         *d_launch = nullptr;
    std::vector<BatchProblem> probs;    // without pointers, seeds and polarised sites
    int64_t part = 0;
    int ngangs = 0;
    size_t bytes = 0;
    ~BatchTables() {
        for (void* p : {d_jobs, d_jstart, d_passes, d_stages, d_ops, d_launch})
            if (p) (void)hipFree(p);
    }
};

// One call's problems and the memory its gangs write.
struct BatchCache {
    std::shared_ptr<const BatchTables> tables;
    void *d_probs = nullptr, *d_part = nullptr, *d_sync = nullptr;
    int nslots = 0;
    bool half = false;
    hipStream_t side = nullptr;
    hipGraphExec_t exec = nullptr;
    hipGraph_t graph = nullptr;
    hipEvent_t end = nullptr;   // of the latest launch, if it has no gangs
    bool awaited = false;       // listed in g_gangless
    size_t bytes = 0;
    ~BatchCache() {
        // its latest launch may still run
        if (side) (void)hipStreamSynchronize(side);
        if (end) (void)hipEventDestroy(end);
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (side) (void)hipStreamDestroy(side);
        for (void* p : {d_probs, d_part, d_sync})
            if (p) (void)hipFree(p);
    }
};

// Problems of fewer sites than a lane of the persistent launch has register
// bits: a wave each, in a launch of their own straight on the caller's stream.
// They wait for nothing, so they need no chaining, and the launch can be
// captured once its tables are there.
struct SmallBatch {
    void *d_jobs = nullptr, *d_stages = nullptr, *d_ops = nullptr;
    int njobs = 0, bits = 0;
    size_t bytes = 0;
    ~SmallBatch() {
        for (void* p : {d_jobs, d_stages, d_ops})
            if (p) (void)hipFree(p);
    }
};

// Kept of past calls, by everything that their launches hold.  A program that
// draws new states or seeds for every call would otherwise leave an entry of
// device memory, a stream and a graph behind with each.
constexpr size_t kCallsKept = 1024, kCallBytesKept = size_t(1) << 30;
static std::mutex g_bmu;
static Kept<SmallBatch> g_small(kCallsKept, kCallBytesKept);
static Kept<BatchCache> g_bcache(kCallsKept, kCallBytesKept);
// The tables of the latest sets of couplings, latest first.
constexpr size_t kBatchTablesKept = 8;
static std::list<std::pair<std::vector<double>, std::shared_ptr<const BatchTables>>> g_btables;
// Per device: sticky status word of the persistent launches (non-zero once a
// gang barrier has timed out), read and cleared by spin_batch_status.
static std::map<int, int*> g_status;
// Per device: the end of the latest persistent launch with gangs, and the calls
// whose launches without gangs no later one with gangs waits for yet.  A gang
// waits for its members, so the launch's workgroups must all find a slot: it
// runs beside no other persistent launch of any stream (one that held some of
// the slots for long would look like a gang that stands still).  Launches without
// gangs overlap each other.
static std::mutex g_launch_mu;
static std::map<int, hipEvent_t> g_last_launch;
static std::map<int, std::vector<std::weak_ptr<BatchCache>>> g_gangless;

static int status_word(int dev, int** out) {
    std::lock_guard<std::mutex> lk(g_bmu);
    int*& w = g_status[dev];
    if (!w) {
        void* p = nullptr;
        if (hipMalloc(&p, sizeof(int)) != hipSuccess) return fail(SPIN_ENOMEM, "status word allocation failed");
        const int zero = 0;
        if (hipMemcpy(p, &zero, sizeof(int), hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipFree(p);
            return fail(SPIN_EHIP, "status word initialisation failed");
        }
        w = static_cast<int*>(p);
    }
    *out = w;
    return SPIN_OK;
}

void release_batch_caches() {
    std::lock_guard<std::mutex> lk(g_bmu);
    g_bcache.clear();
    g_btables.clear();
    g_small.clear();
    {
        std::lock_guard<std::mutex> ll(g_launch_mu);
        for (auto& kv : g_last_launch)
            if (kv.second) (void)hipEventDestroy(kv.second);
        g_last_launch.clear();
        g_gangless.clear();
    }
    for (auto& kv : g_status)
        if (kv.second) (void)hipFree(kv.second);
    g_status.clear();
}

// Key: everything the tables and the launch depend on.
static std::vector<double> batch_key(const spin_problem* probs, int n,
                                     const std::vector<std::vector<Coupling>>& Js, int prec,
                                     double dt, int64_t n_steps, int init, int dev) {
    std::vector<double> k{double(prec), dt, double(n_steps), double(init), double(dev), double(n)};
    for (int p = 0; p < n; ++p) {
        const spin_problem& pr = probs[p];
        k.push_back(double(reinterpret_cast<uintptr_t>(pr.psi)));
        k.push_back(double(reinterpret_cast<uintptr_t>(pr.P_dev)));
        k.push_back(double(reinterpret_cast<uintptr_t>(pr.N_dev)));
        k.push_back(pr.M);
        k.push_back(pr.observed_site);
        k.push_back(pr.polarized_site);
        k.push_back(double(pr.seed >> 32));
        k.push_back(double(pr.seed & 0xffffffffu));
        for (const Coupling& c : Js[p]) {
            k.push_back(c.i);
            k.push_back(c.j);
            k.push_back(c.a);
            k.push_back(c.b);
        }
    }
    return k;
}

// Key of the tables: what a problem's plan and the schedule depend on.
static std::vector<double> tables_key(const spin_problem* probs, int n, const std::vector<std::vector<Coupling>>& Js,
                                      int prec, double dt, int64_t n_steps, int dev, bool half) {
    std::vector<double> k{double(prec), dt, double(n_steps), double(dev), double(half), double(n)};
    for (int p = 0; p < n; ++p) {
        k.push_back(probs[p].M);
        k.push_back(probs[p].observed_site);
        k.push_back(double(Js[p].size()));
        for (const Coupling& c : Js[p]) {
            k.push_back(c.i);
            k.push_back(c.j);
            k.push_back(c.a);
            k.push_back(c.b);
        }
    }
    return k;
}

static int upload(const void* src, size_t n, void** dst, size_t* total) {
    if (n == 0) n = 16;
    *total += n;
    if (hipMalloc(dst, n) != hipSuccess) return fail(SPIN_ENOMEM, "batch table allocation failed");
    if (src && hipMemcpy(*dst, src, n, hipMemcpyHostToDevice) != hipSuccess)
        return fail(SPIN_EHIP, "batch table upload failed");
    return SPIN_OK;
}

// The plan of one problem: its own tables, indices from 0.
template <typename T>
struct ProblemPlan {
    const spin_problem* pr = nullptr;
    const std::vector<Coupling>* J = nullptr;
    BatchProblem b{};
    DevTables<T> tb;
    std::vector<int2> launches;
    double dur = 0;
};

template <typename T>
static void plan_problem(double dt, int64_t n_steps, int64_t gang, bool half, ProblemPlan<T>* out) {
    const bool f32 = sizeof(T) == 4;
    const int K = batch_tile_bits(f32), KL = K - 1;
    const spin_problem& pr = *out->pr;
    BatchProblem& b = out->b;
    double fops = 0;
    if (pr.M <= KL) {
        const int bits = batch_resident_bits(pr.M, half);
        const int r = bits - __builtin_ctz(batch_shape(f32, half).nt);
        const ResidentPlan rp = plan_resident(bits, *out->J, dt, pr.observed_site, true, r);
        b.gsize = 1;
        const ResidentStages rs = encode_resident<T>(rp, bits, pr.observed_site, out->tb, false);
        b.obs_stage0 = rs.obs0;
        b.pro_stage0 = rs.pro0;
        b.pro_nstage = rs.npro;
        b.step_stage0 = rs.step0;
        b.step_nstage = rs.nstep;
        b.last_stage0 = rs.last0;
        for (const Op& op : rp.step.ops) fops += op.kind == 0;
        // on-chip: about half the cost per amplitude of a tiled pass; the
        // observable counts as a factor (a problem without couplings takes time
        // too: 1024 of them had all been given to one slot)
        out->dur = 0.5 * (fops + 1.0) * std::ldexp(1.0, bits) * double(n_steps + 1);
        return;
    }
    PassParams pp;
    pp.k = K;
    pp.r = batch_shape(f32, half).r;
    // the library's default launch shape; a gang plans one scheduling
    // variant (plan_stream), not the single path's variant search
    pp.c = 4;
    pp.half = half;
    pp.gates = half ? kMaxGates : 0;
    const StreamPlan sp = plan_stream(pr.M, *out->J, dt, n_steps, pr.observed_site, true, pp);
    for (const HostPass& hp : sp.passes) encode_pass<T>(hp, pr.M, pr.observed_site, out->tb);
    b.nlaunch = int(sp.launch_tmpl.size());
    for (size_t l = 0; l < sp.launch_tmpl.size(); ++l)
        out->launches.push_back(make_int2(sp.launch_tmpl[l], int(sp.launch_offset[l])));
    b.ntiles = int64_t(1) << (pr.M - K);
    b.gsize = int(std::min<int64_t>(b.ntiles, gang));
    for (int t : sp.launch_tmpl)
        for (const Op& op : sp.passes[t].ops) fops += op.kind == 0;
    // factor work plus one sweep per launch, shared by the gang
    out->dur = (fops + 6.0 * sp.launch_tmpl.size()) * std::ldexp(1.0, pr.M) / b.gsize;
}

template <typename T>
static int build_tables(const std::vector<spin_problem>& probs, const std::vector<std::vector<Coupling>>& Js,
                        double dt, int64_t n_steps, int nslots, bool half, BatchTables* bt) {
    const bool f32 = sizeof(T) == 4;
    const int K = batch_tile_bits(f32);
    const int KL = K - 1;               // largest one-workgroup problem
    // Workgroups per gang, at most: as many as leave every gang a slot of its
    // own, or nearly (a third of them may wait for another).  Stars of M = 14 to
    // 20, ms where the batch may ask for 1 / 1.5 / 2 / 3 times the slots: 32
    // problems, 25 steps 21.0 / 16.9 / 18.4 / 18.2; 64
    // problems, 5 steps 11.1 / 7.5 / 7.9 / 8.5; 128, 4 steps 13.2 / 13.1 / 13.1 /
    // 12.8; complex128, 32 problems, 5 steps 10.8 / 8.5 / 8.5 / 9.5.
    auto demand = [&](int64_t g) {
        int64_t n = 0;
        for (const spin_problem& pr : probs)
            n += pr.M <= KL ? 1 : std::min(int64_t(1) << (pr.M - K), g);
        return n;
    };
    int64_t gang = 8;
    while (2 * gang <= nslots && 2 * demand(2 * gang) <= 3 * int64_t(nslots)) gang *= 2;
    gang = std::min<int64_t>(gang, nslots);
    // problems with equal (M, observed site, couplings) share their plan
    // (e.g. the basis-state members of one ensemble)
    std::map<std::vector<double>, int> seen;
    std::vector<ProblemPlan<T>> plans;
    std::vector<int> plan_of(probs.size());
    for (size_t p = 0; p < probs.size(); ++p) {
        std::vector<double> skey{double(probs[p].M), double(probs[p].observed_site)};
        for (const Coupling& c : Js[p]) {
            skey.push_back(c.i);
            skey.push_back(c.j);
            skey.push_back(c.a);
            skey.push_back(c.b);
        }
        const auto at = seen.emplace(skey, int(plans.size()));
        if (at.second) {
            plans.emplace_back();
            plans.back().pr = &probs[p];
            plans.back().J = &Js[p];
        }
        plan_of[p] = at.first->second;
    }
    // The plans do not depend on each other; a few threads make them (32
    // stars of M = 14 to 20, 25 steps: the first call 1.37 s with one, 0.20 with 8).
    run_on_threads(plans.size(), [&](size_t i) { plan_problem<T>(dt, n_steps, gang, half, &plans[i]); });

    DevTables<T> tb;
    std::vector<int2> launches;
    for (ProblemPlan<T>& pl : plans) {
        const int pass0 = int(tb.passes.size()), stage0 = int(tb.stages.size()), op0 = int(tb.ops.size());
        for (DevStage& s : pl.tb.stages) s.op0 += op0;
        for (DevPass& s : pl.tb.passes) s.stage0 += stage0;
        for (int32_t* f : {&pl.b.obs_stage0, &pl.b.pro_stage0, &pl.b.step_stage0, &pl.b.last_stage0}) *f += stage0;
        pl.b.pass0 = pass0;
        pl.b.launch0 = int64_t(launches.size());
        tb.passes.insert(tb.passes.end(), pl.tb.passes.begin(), pl.tb.passes.end());
        tb.stages.insert(tb.stages.end(), pl.tb.stages.begin(), pl.tb.stages.end());
        tb.ops.insert(tb.ops.end(), pl.tb.ops.begin(), pl.tb.ops.end());
        launches.insert(launches.end(), pl.launches.begin(), pl.launches.end());
        pl.tb = DevTables<T>();
    }
    std::vector<double> dur;
    for (size_t p = 0; p < probs.size(); ++p) {
        const ProblemPlan<T>& pl = plans[plan_of[p]];
        BatchProblem b = pl.b;
        b.M = probs[p].M;
        if (b.M > KL) {     // a gang: partial sums and a counter of its own
            b.part0 = bt->part;
            bt->part += int64_t(kBatchRing) * b.gsize * 2;
            b.counter = bt->ngangs++;
        }
        dur.push_back(pl.dur);
        bt->probs.push_back(b);
    }
    // Gang schedule: longest jobs first, each on the slots that are free first.
    std::vector<double> avail(nslots, 0.0);
    std::vector<std::vector<BatchJob>> lists(nslots);
    std::vector<int> order(bt->probs.size()), slots(nslots);
    for (size_t i = 0; i < order.size(); ++i) order[i] = int(i);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return dur[a] > dur[b]; });
    for (int q : order) {
        const int g = bt->probs[q].gsize;
        for (int w = 0; w < nslots; ++w) slots[w] = w;
        std::partial_sort(slots.begin(), slots.begin() + g, slots.end(), [&](int a, int b) {
            return avail[a] < avail[b] || (avail[a] == avail[b] && a < b);
        });
        const double start = avail[slots[g - 1]];
        std::sort(slots.begin(), slots.begin() + g);
        for (int r = 0; r < g; ++r) {
            lists[slots[r]].push_back(BatchJob{q, r});
            avail[slots[r]] = start + dur[q];
        }
    }
    std::vector<BatchJob> jobs;
    std::vector<int> jstart(nslots + 1, 0);
    for (int w = 0; w < nslots; ++w) {
        jstart[w] = int(jobs.size());
        jobs.insert(jobs.end(), lists[w].begin(), lists[w].end());
    }
    jstart[nslots] = int(jobs.size());

    int rc;
    if ((rc = upload(jobs.data(), jobs.size() * sizeof(BatchJob), &bt->d_jobs, &bt->bytes))) return rc;
    if ((rc = upload(jstart.data(), jstart.size() * sizeof(int), &bt->d_jstart, &bt->bytes))) return rc;
    if ((rc = upload(tb.passes.data(), tb.passes.size() * sizeof(DevPass), &bt->d_passes, &bt->bytes))) return rc;
    if ((rc = upload(tb.stages.data(), tb.stages.size() * sizeof(DevStage), &bt->d_stages, &bt->bytes))) return rc;
    if ((rc = upload(tb.ops.data(), tb.ops.size() * sizeof(DevOp<T>), &bt->d_ops, &bt->bytes))) return rc;
    return upload(launches.data(), launches.size() * sizeof(int2), &bt->d_launch, &bt->bytes);
}

static int build_call(const std::vector<spin_problem>& probs, int init, int nslots, bool half, BatchCache* bc) {
    std::vector<BatchProblem> bp = bc->tables->probs;
    for (size_t p = 0; p < bp.size(); ++p) {
        bp[p].psi = probs[p].psi;
        bp[p].P = probs[p].P_dev;
        bp[p].N = probs[p].N_dev;
        bp[p].seed = probs[p].seed;
        bp[p].polarized = probs[p].polarized_site;
        bp[p].init = init;
    }
    int rc;
    if ((rc = upload(bp.data(), bp.size() * sizeof(BatchProblem), &bc->d_probs, &bc->bytes))) return rc;
    if ((rc = upload(nullptr, std::max<int64_t>(bc->tables->part, 2) * sizeof(double), &bc->d_part, &bc->bytes))) return rc;
    if ((rc = upload(nullptr, (kSyncGangs + bc->tables->ngangs) * sizeof(int), &bc->d_sync, &bc->bytes))) return rc;
    bc->nslots = nslots;
    bc->half = half;
    return SPIN_OK;
}

// ------------------------------------------------- small problems
template <typename T>
static int build_small(const std::vector<spin_problem>& probs, const std::vector<std::vector<Coupling>>& Js,
                       double dt, int init, SmallBatch* sb) {
    sb->bits = resident_bits(1);
    sb->njobs = int(probs.size());
    DevTables<T> tb;
    std::vector<ResidentJob> jobs;
    std::map<std::vector<double>, ResidentStages> seen;
    for (size_t p = 0; p < probs.size(); ++p) {
        const spin_problem& pr = probs[p];
        std::vector<double> skey{double(pr.M), double(pr.observed_site)};
        for (const Coupling& c : Js[p]) {
            skey.push_back(c.i);
            skey.push_back(c.j);
            skey.push_back(c.a);
            skey.push_back(c.b);
        }
        auto at = seen.find(skey);
        if (at == seen.end()) {
            tb.carry.clear();
            const ResidentPlan rp = plan_resident(sb->bits, Js[p], dt, pr.observed_site, true, kResidentRegs);
            at = seen.emplace(skey, encode_resident<T>(rp, sb->bits, pr.observed_site, tb, false)).first;
        }
        const ResidentStages& rs = at->second;
        ResidentJob j{};
        j.psi = pr.psi;
        j.P = pr.P_dev;
        j.N = pr.N_dev;
        j.seed = pr.seed;
        j.M = pr.M;
        j.polarized = pr.polarized_site;
        j.init = init;
        j.obs_stage0 = rs.obs0;
        j.pro_stage0 = rs.pro0;
        j.pro_nstage = rs.npro;
        j.step_stage0 = rs.step0;
        j.step_nstage = rs.nstep;
        j.last_stage0 = rs.last0;
        jobs.push_back(j);
    }
    int rc;
    if ((rc = upload(jobs.data(), jobs.size() * sizeof(ResidentJob), &sb->d_jobs, &sb->bytes))) return rc;
    if ((rc = upload(tb.stages.data(), tb.stages.size() * sizeof(DevStage), &sb->d_stages, &sb->bytes))) return rc;
    return upload(tb.ops.data(), tb.ops.size() * sizeof(DevOp<T>), &sb->d_ops, &sb->bytes);
}

template <typename T>
static int batch_small(const spin_problem* probs, const std::vector<int>& sel,
                       const std::vector<std::vector<Coupling>>& Js, int prec, double dt, int64_t n_steps,
                       int init, hipStream_t st) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(SPIN_EHIP, "hipGetDevice failed");
    std::vector<spin_problem> ps;
    std::vector<std::vector<Coupling>> js;
    for (int p : sel) {
        ps.push_back(probs[p]);
        js.push_back(Js[p]);
    }
    const std::vector<double> key = batch_key(ps.data(), int(ps.size()), js, prec, dt, n_steps, init, dev);
    // a captured launch keeps its tables' addresses
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) return fail(SPIN_EHIP, "stream query failed");
    const bool pin = cs != hipStreamCaptureStatusNone;
    std::shared_ptr<SmallBatch> sb;
    {
        std::lock_guard<std::mutex> lk(g_bmu);
        sb = g_small.find(key, pin);
    }
    if (!sb) {
        sb = std::make_shared<SmallBatch>();
        try {
            if (int rc = build_small<T>(ps, js, dt, init, sb.get())) return rc;
        } catch (const std::exception& e) {
            return fail(SPIN_EUNSUPPORTED, std::string("batch planning failed: ") + e.what());
        }
        std::vector<std::shared_ptr<SmallBatch>> gone;
        std::lock_guard<std::mutex> lk(g_bmu);
        gone = g_small.insert(key, sb, sb->bytes, pin);
    }
    const hipError_t e = launch_resident<T>(sb->bits, ResidentJob{}, static_cast<const ResidentJob*>(sb->d_jobs), sb->njobs,
                                            static_cast<const DevStage*>(sb->d_stages),
                                            static_cast<const DevOp<T>*>(sb->d_ops), n_steps, st);
    if (e != hipSuccess) return fail(SPIN_EHIP, std::string("batch launch: ") + hipGetErrorString(e));
    return SPIN_OK;
}

template <typename T>
static int batch_persistent(const spin_problem* probs, const std::vector<int>& sel,
                            const std::vector<std::vector<Coupling>>& Js, int prec, double dt,
                            int64_t n_steps, int init, bool use_graph, bool half, hipStream_t st) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(SPIN_EHIP, "hipGetDevice failed");
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return fail(SPIN_EHIP, "device query failed");
    const int nslots = prop.multiProcessorCount * (half ? 2 : 1);

    // key over the selected problems only
    std::vector<spin_problem> ps;
    std::vector<std::vector<Coupling>> js;
    for (int p : sel) {
        ps.push_back(probs[p]);
        js.push_back(Js[p]);
    }
    std::vector<double> key = batch_key(ps.data(), int(ps.size()), js, prec, dt, n_steps, init, dev);
    key.push_back(use_graph ? 1 : 0);
    key.push_back(half ? 1 : 0);
    std::shared_ptr<BatchCache> bc;
    {
        std::lock_guard<std::mutex> lk(g_bmu);
        bc = g_bcache.find(key);
    }
    if (!bc) {
        bc = std::make_shared<BatchCache>();
        const std::vector<double> tkey = tables_key(ps.data(), int(ps.size()), js, prec, dt, n_steps, dev, half);
        {
            std::lock_guard<std::mutex> lk(g_bmu);
            for (auto it = g_btables.begin(); it != g_btables.end(); ++it)
                if (it->first == tkey) {
                    bc->tables = it->second;
                    g_btables.splice(g_btables.begin(), g_btables, it);
                    break;
                }
        }
        int rc;
        if (!bc->tables) {
            auto bt = std::make_shared<BatchTables>();
            try {
                rc = build_tables<T>(ps, js, dt, n_steps, nslots, half, bt.get());
            } catch (const std::exception& e) {
                return fail(SPIN_EUNSUPPORTED, std::string("batch planning failed: ") + e.what());
            }
            if (rc) return rc;
            bc->tables = bt;
            std::lock_guard<std::mutex> lk(g_bmu);
            g_btables.emplace_front(tkey, bt);
            if (g_btables.size() > kBatchTablesKept) g_btables.pop_back();
        }
        if ((rc = build_call(ps, init, nslots, half, bc.get()))) return rc;
        std::vector<std::shared_ptr<BatchCache>> gone;      // let go of after the lock
        std::lock_guard<std::mutex> lk(g_bmu);
        gone = g_bcache.insert(key, bc, bc->bytes + bc->tables->bytes);
    }
    int* status = nullptr;
    if (int rc = status_word(dev, &status)) return rc;
    auto enqueue = [&](hipStream_t s) {
        return launch_batch<T>(bc->nslots, bc->half, static_cast<const BatchProblem*>(bc->d_probs),
                               static_cast<const BatchJob*>(bc->tables->d_jobs),
                               static_cast<const int*>(bc->tables->d_jstart),
                               static_cast<const DevPass*>(bc->tables->d_passes),
                               static_cast<const DevStage*>(bc->tables->d_stages),
                               static_cast<const DevOp<T>*>(bc->tables->d_ops),
                               static_cast<const int2*>(bc->tables->d_launch),
                               static_cast<double*>(bc->d_part), static_cast<int*>(bc->d_sync),
                               bc->tables->ngangs, status, n_steps, s);
    };
    std::lock_guard<std::mutex> launch_lock(g_launch_mu);
    const bool gangs = bc->tables->ngangs > 0;
    hipEvent_t& last = g_last_launch[dev];
    hipEvent_t& end = gangs ? last : bc->end;
    const bool first = last == nullptr;
    if (!end && hipEventCreateWithFlags(&end, hipEventDisableTiming) != hipSuccess)
        return fail(SPIN_EHIP, "event create failed");
    std::vector<std::weak_ptr<BatchCache>>& gangless = g_gangless[dev];
    // the launches that this one waits for
    auto chain = [&](hipStream_t s) {
        hipError_t e = first ? hipSuccess : hipStreamWaitEvent(s, last, 0);
        if (!gangs) return e;
        for (const std::weak_ptr<BatchCache>& w : gangless)
            if (const std::shared_ptr<BatchCache> other = w.lock()) {     // else it has ended
                if (e == hipSuccess) e = hipStreamWaitEvent(s, other->end, 0);
                other->awaited = false;
            }
        gangless.clear();
        return e;
    };
    auto launched = [&](hipStream_t s) {
        if (!gangs && !bc->awaited) {
            if (gangless.size() >= 2 * kCallsKept)
                gangless.erase(std::remove_if(gangless.begin(), gangless.end(), [](auto& w) { return w.expired(); }),
                               gangless.end());
            gangless.push_back(bc);
            bc->awaited = true;
        }
        return hipEventRecord(end, s);
    };
    hipError_t e = hipSuccess;
    if (use_graph) {
        // capture on a library stream ordered after the caller's stream
        if (!bc->side && (e = hipStreamCreateWithFlags(&bc->side, hipStreamNonBlocking)) != hipSuccess)
            return fail(SPIN_EHIP, std::string("stream: ") + hipGetErrorString(e));
        if (!bc->exec) {
            e = hipStreamBeginCapture(bc->side, hipStreamCaptureModeThreadLocal);
            if (e == hipSuccess) e = enqueue(bc->side);
            hipGraph_t g = nullptr;
            hipError_t e2 = hipStreamEndCapture(bc->side, &g);
            if (e == hipSuccess) e = e2;
            if (e == hipSuccess) e = hipGraphInstantiate(&bc->exec, g, nullptr, nullptr, 0);
            bc->graph = g;
            if (e != hipSuccess) return fail(SPIN_EHIP, std::string("graph capture: ") + hipGetErrorString(e));
        }
        hipEvent_t ev;
        if ((e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess)
            return fail(SPIN_EHIP, "event create failed");
        e = hipEventRecord(ev, st);
        if (e == hipSuccess) e = hipStreamWaitEvent(bc->side, ev, 0);
        if (e == hipSuccess) e = chain(bc->side);
        if (e == hipSuccess) e = hipGraphLaunch(bc->exec, bc->side);
        if (e == hipSuccess) e = launched(bc->side);
        if (e == hipSuccess) e = hipEventRecord(ev, bc->side);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, ev, 0);
        (void)hipEventDestroy(ev);
    } else {
        e = chain(st);
        if (e == hipSuccess) e = enqueue(st);
        if (e == hipSuccess) e = launched(st);
    }
    if (e != hipSuccess) return fail(SPIN_EHIP, std::string("batch launch: ") + hipGetErrorString(e));
    return SPIN_OK;
}

}  // namespace spinqp

using namespace spinqp;

extern "C" int spin_trotter_evolve_batch(const spin_problem* probs, int32_t n,
                                         const spin_coupling* J_all, int64_t K_total,
                                         int32_t prec, double dt, int64_t n_steps,
                                         int32_t init, void* stream) {
    try {
        if (init < SPIN_INIT_NONE || init > SPIN_INIT_PRODUCT) return fail(SPIN_EINVAL, "bad init");
        if (n < 0) return fail(SPIN_EINVAL, "n < 0");
        if (n > 0 && !probs) return fail(SPIN_EINVAL, "probs is NULL");
        if (K_total < 0 || (K_total > 0 && !J_all)) return fail(SPIN_EINVAL, "bad J_all / K_total");
        if (!std::isfinite(dt)) return fail(SPIN_EINVAL, "dt is not finite");
        if (n_steps < 0) return fail(SPIN_EINVAL, "n_steps < 0");
        if (prec != SPIN_C64 && prec != SPIN_C128) return fail(SPIN_EINVAL, "bad prec");
        std::vector<std::vector<Coupling>> Js(n);
        const int cap = prec == SPIN_C64 ? 14 : 13;
        for (int p = 0; p < n; ++p) {
            const spin_problem& pr = probs[p];
            std::ostringstream os;
            os << "problem " << p << ": ";
            int rc = validate_common(pr.psi, prec, pr.M);
            if (rc) return fail(rc, os.str() + spin_last_error());
            if (!pr.P_dev) return fail(SPIN_EINVAL, os.str() + "P_dev is NULL");
            if (pr.observed_site < 0 || pr.observed_site >= pr.M)
                return fail(SPIN_EINVAL, os.str() + "observed_site out of range");
            if ((init == SPIN_INIT_RANDOM_PHASE || init == SPIN_INIT_PRODUCT) &&
                (pr.polarized_site < 0 || pr.polarized_site >= pr.M))
                return fail(SPIN_EINVAL, os.str() + "polarized_site out of range");
            if (init == SPIN_INIT_BASIS && (pr.seed >> pr.M) != 0)
                return fail(SPIN_EINVAL, os.str() + "basis index (seed) >= 2^M");
            if (pr.K < 0 || pr.coupling_offset < 0 || pr.coupling_offset + pr.K > K_total)
                return fail(SPIN_EINVAL, os.str() + "coupling range outside J_all");
            rc = validate_couplings(pr.M, J_all + pr.coupling_offset, pr.K, &Js[p]);
            if (rc) return fail(rc, os.str() + spin_last_error());
        }
        (void)cap;
        if (n == 0) return SPIN_OK;
        hipStream_t st = static_cast<hipStream_t>(stream);
        // Two workgroups per CU with half-tile gangs when both fit (every
        // slot of the persistent launch must be resident at once), else one
        // with whole tiles.
        const bool f32 = prec == SPIN_C64;
        const bool half = batch_blocks_per_cu(f32, true) >= 2;
        if (!half && batch_blocks_per_cu(f32, false) < 1)
            return fail(SPIN_EUNSUPPORTED, "batch kernel does not fit a CU");
        std::vector<int> small, large;
        for (int p = 0; p < n; ++p) (probs[p].M < batch_shape(f32, half).r ? small : large).push_back(p);
        const bool graph = true;
        int rc = SPIN_OK;
        if (!small.empty())
            rc = f32 ? batch_small<float>(probs, small, Js, prec, dt, n_steps, init, st)
                     : batch_small<double>(probs, small, Js, prec, dt, n_steps, init, st);
        if (rc == SPIN_OK && !large.empty())
            rc = f32 ? batch_persistent<float>(probs, large, Js, prec, dt, n_steps, init, graph, half, st)
                     : batch_persistent<double>(probs, large, Js, prec, dt, n_steps, init, graph, half, st);
        if (rc == SPIN_OK) fail(SPIN_OK, "");
        return rc;
    } catch (const std::exception& e) {
        return fail(SPIN_EUNSUPPORTED, std::string("internal error: ") + e.what());
    }
}

extern "C" int spin_batch_status(void* stream) {
    try {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return fail(SPIN_EHIP, std::string("batch status: ") + hipGetErrorString(e));
        int* w = nullptr;
        {
            std::lock_guard<std::mutex> lk(g_bmu);
            auto it = g_status.find(dev);
            if (it != g_status.end()) w = it->second;
        }
        if (!w) {
            fail(SPIN_OK, "");
            return SPIN_OK;      // no persistent launch on this device yet
        }
        int v = 0;
        const int zero = 0;
        e = hipMemcpy(&v, w, sizeof(int), hipMemcpyDeviceToHost);
        if (e == hipSuccess && v != 0) e = hipMemcpy(w, &zero, sizeof(int), hipMemcpyHostToDevice);
        if (e != hipSuccess) return fail(SPIN_EHIP, std::string("batch status: ") + hipGetErrorString(e));
        if (v != 0)
            return fail(SPIN_EHIP, "batch: a gang barrier timed out (workgroups not co-resident?); "
                                   "the affected problems' P were set to NaN");
        fail(SPIN_OK, "");
        return SPIN_OK;
    } catch (const std::exception& e) {
        return fail(SPIN_EUNSUPPORTED, std::string("internal error: ") + e.what());
    }
}
