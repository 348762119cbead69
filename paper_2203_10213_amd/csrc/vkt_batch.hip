// vkt_batch.hip -- vktApplyFilterBatched: many independent ApplyFilter calls
// of uneven volume sizes and mixed filter sizes in persistent launches.
//
// Planning (host, once per distinct batch):
//   * every (dst, src, filter) triple is validated and planned exactly as by
//     vktApplyFilter; triples fall into arithmetic classes (cell format, k,
//     vector-ALU or matrix-core path and its variant), one persistent kernel
//     per class;
//   * each volume is cut into tile-slabs (the kernel's output tile -- one of
//     two tile heights -- times a z-slab depth, both chosen per class and
//     batch size class, by default or by the autotuner, which times every
//     tile height at candidate depths on the real batch); the class's work
//     list is sorted longest first;
//   * descriptors, work lists, the classes' weight pools and the work-queue
//     counters go to one device buffer.
// Launch: the class kernels side by side, on streams that fork from the calling
// thread's stream and join it again.  Plans are cached by
// the batch's signature (pointers, dims, formats, filter identities, mode,
// precision, stream), so a repeated batch is its launches alone.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "vkt_internal.h"

namespace vkt {
namespace {

struct ClassKey {
    // path 0 = vector ALU (flag: int accumulate), 1 = matrix (flag bit 0: 6
    // products, bit 1: row-pair kernel), 2 = 8-bit dot products (flag:
    // signed weights)
    int fmt, k, path, flag;
    bool operator<(const ClassKey& o) const
    {
        return std::tie(fmt, k, path, flag) < std::tie(o.fmt, o.k, o.path, o.flag);
    }
};

// variant: the class's tile-height variant (0: default tile, 1: the other
// height; kTileVariants in all)
const void* class_kernel(const ClassKey& c, int variant)
{
    if (c.path == 2) return dot4_batched_kernel(c.k, c.flag != 0, variant);
    return c.path ? mfma_batched_kernel((vktDataFormat)c.fmt, c.k, (c.flag & 1) != 0,
                                        (c.flag & 2) != 0, variant)
                  : valu_batched_kernel((vktDataFormat)c.fmt, c.k, c.flag != 0, variant);
}

ClassGeom class_geom(const ClassKey& c, int variant)
{
    if (c.path == 2) return dot4_geom(c.k, variant);
    return c.path ? mfma_geom((vktDataFormat)c.fmt, c.k, (c.flag & 1) != 0, (c.flag & 2) != 0,
                              variant)
                  : valu_geom(c.k, variant);
}

// Weights per filter in the class's pools: k^3 (float and int pools), or the
// packed 8-bit rows (int pool) of the dot-product path.
int class_weights(const ClassKey& c) { return c.path == 2 ? dot4_words(c.k) : c.k * c.k * c.k; }

// ---- tuning table: (class, size class) -> tile variant and z-slab depth ----

struct TuneKey {
    ClassKey c;
    int size_class;
    bool operator<(const TuneKey& o) const
    {
        return std::tie(c, size_class) < std::tie(o.c, o.size_class);
    }
};

struct TuneVal {
    int tz;        // z-slab depth (0: no entry)
    int variant;   // tile-height variant
};

std::mutex g_tune_mu;
std::map<TuneKey, TuneVal> g_tune;
bool g_tune_loaded = false;

// Size class of a set of volumes: log2 of the mean cube-root edge length.
int size_class_of(const std::vector<FilterJob>& jobs)
{
    double s = 0;
    for (const auto& j : jobs) s += std::cbrt((double)j.X * j.Y * j.Z);
    return jobs.empty() ? 0 : (int)std::floor(std::log2(s / (double)jobs.size()));
}

void tune_load_locked()
{
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char* path = std::getenv("VKT_TUNE_CACHE");
    if (!path) return;
    FILE* f = std::fopen(path, "r");
    if (!f) return;
    char line[256];
    while (std::fgets(line, sizeof line, f)) {
        TuneKey k;
        TuneVal v{0, 0};
        int tx = 0, ty = 0;
        // fmt k path flag size_class tz variant tx ty: the entry and the tile that
        // it was timed on.  Lines for another tile than the variant has now, or
        // without one (older files), say nothing about these kernels.
        const int n = std::sscanf(line, "%d %d %d %d %d %d %d %d %d", &k.c.fmt, &k.c.k, &k.c.path,
                                  &k.c.flag, &k.size_class, &v.tz, &v.variant, &tx, &ty);
        if (n < 9 || v.tz <= 0 || v.variant < 0 || v.variant >= kTileVariants) continue;
        const ClassGeom g = class_geom(k.c, v.variant);
        if (g.tx == tx && g.ty == ty) g_tune[k] = v;
    }
    std::fclose(f);
}

void tune_store_locked()
{
    const char* path = std::getenv("VKT_TUNE_CACHE");
    if (!path) return;
    FILE* f = std::fopen(path, "w");
    if (!f) return;
    for (const auto& e : g_tune) {
        const ClassGeom g = class_geom(e.first.c, e.second.variant);
        std::fprintf(f, "%d %d %d %d %d %d %d %d %d\n", e.first.c.fmt, e.first.c.k, e.first.c.path,
                     e.first.c.flag, e.first.size_class, e.second.tz, e.second.variant, g.tx, g.ty);
    }
    std::fclose(f);
}

// ---- plans ------------------------------------------------------------------

struct ClassPlan {
    ClassKey key;
    const void* func = nullptr;
    std::vector<int> members;      // indices into the batch
    int tz = 0;
    int variant = 0;               // tile-height variant
    unsigned grid = 0;
    size_t lane = 0;               // side stream it runs on; past them: the caller's
    BatchArgs args{};
    // offsets inside the plan's device buffer
    size_t off_desc = 0, off_items = 0, off_cnt = 0, off_wf = 0, off_wi = 0;
    uint32_t nitems = 0;
};

// The streams on which the classes of a batch run beside its caller's stream,
// with the events that fork and join them.  The plans of one caller's stream share
// a set, as their batches run one after another anyhow; shared by two callers, a set
// would make one's kernels wait for the other's stream.  (With a set per plan more
// streams share the hardware queues: 64 float32 volumes of 16 to 64 116 us, with this
// 113; 2 of 17 to 40 79 and 77; larger batches the same.)  A set that the last of its plans has left is used for the next new stream, so there
// are no more than streams with plans at once; none is ever destroyed.
constexpr size_t kSideStreams = 3;  // (with the caller's, the 4 hardware queues)
struct SideStreams {
    int device = 0;
    hipStream_t caller = nullptr;
    size_t plans = 0;  // that use it
    hipEvent_t fork = nullptr;
    hipStream_t stream[kSideStreams] = {};
    hipEvent_t joined[kSideStreams] = {};
    size_t n = 0;
};
std::mutex g_side_mu;
std::vector<std::unique_ptr<SideStreams>> g_side;

// The set of the caller's stream on the current device `dev`, with at least n
// streams; null where they cannot be made (the classes then run one after another).
SideStreams* take_side_streams(int dev, hipStream_t caller, size_t n)
{
    std::lock_guard<std::mutex> lk(g_side_mu);
    SideStreams* s = nullptr;
    for (auto& x : g_side)
        if (x->device == dev && x->plans && x->caller == caller) s = x.get();
    for (auto& x : g_side)
        if (!s && x->device == dev && !x->plans) s = x.get();
    if (!s) {
        g_side.push_back(std::make_unique<SideStreams>());
        s = g_side.back().get();
        s->device = dev;
    }
    bool ok = s->fork || hipEventCreateWithFlags(&s->fork, hipEventDisableTiming) == hipSuccess;
    while (ok && s->n < n) {
        hipStream_t& st = s->stream[s->n];
        hipEvent_t& ev = s->joined[s->n];
        ok = (st || hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess) &&
             (ev || hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess);
        if (ok) ++s->n;
    }
    if (!ok) return nullptr;
    s->caller = caller;
    ++s->plans;
    return s;
}

struct Plan {
    std::vector<uintptr_t> sig;
    int device = 0;
    char* dbuf = nullptr;
    size_t dbytes = 0;
    std::vector<ClassPlan> classes;
    SideStreams* side = nullptr;  // null: one class, or none to be had
    // recorded after every launch: an evicted plan is destroyed only once its
    // last launch has finished (it may still be queued on another thread's
    // stream when the plan leaves the cache)
    hipEvent_t done = nullptr;
    bool captured = false;  // a graph of the caller's holds launches of it
    ~Plan()
    {
        if (done) {
            (void)hipEventSynchronize(done);
            (void)hipEventDestroy(done);
        }
        if (dbuf) (void)hipFree(dbuf);
        if (side) {
            std::lock_guard<std::mutex> lk(g_side_mu);
            --side->plans;
        }
    }
};

// Plan cache, least recently used first.  Plans are shared: a caller holds
// its plan until its launches have been enqueued, so a plan evicted by
// another thread meanwhile stays alive until then (they may still be running
// when the last holder lets go; ~Plan waits for them).  Plans whose
// launches were captured are held in g_captured as well: the caller's graph
// reads the plan's buffer as long as it is replayed.
std::mutex g_plan_mu;
std::vector<std::shared_ptr<Plan>> g_plans, g_captured;
constexpr size_t kMaxPlans = 16;

// Batched calls from several threads run one at a time inside the library:
// planning, launch and the destruction of evicted plans are serialised.  The
// enqueued work itself still runs concurrently on the callers' streams.
//
// The launches were the parallel nodes of one hipGraph per plan once.  The host
// process then ended in a segfault inside the batched call three times, with no
// GPU fault: twice with two threads that evicted each other's plans, once with
// one thread at the 24th or 25th plan of its process.  No mistake was found in
// this file's own code (built with the address sanitizer against a stub of the
// runtime it makes 69 plans and evicts 50 without a finding), which leaves the
// graph calls -- instantiate, launch, destroy -- as suspects: they are out.
std::mutex g_batch_mu;

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Work list of one class at slab depth tz, longest items first.
std::vector<WorkItem> make_items(const std::vector<VolDesc>& descs,
                                 const std::vector<int>& members, int k)
{
    struct Costed {
        WorkItem w;
        int64_t cost;
    };
    std::vector<Costed> v;
    for (size_t m = 0; m < members.size(); ++m) {
        const VolDesc& a = descs[m];
        const int64_t nt = (int64_t)a.tiles_x * a.tiles_y;
        const int slabs = (a.Z + a.tz - 1) / a.tz;
        for (int sl = 0; sl < slabs; ++sl) {
            const int planes = std::min(a.tz, a.Z - sl * a.tz) + k - 1;
            for (int64_t t = 0; t < nt; ++t) {
                Costed c;
                c.w.vol = (uint32_t)m;
                c.w.lid = (uint32_t)(sl * nt + t);
                c.cost = planes;
                v.push_back(c);
            }
        }
    }
    std::stable_sort(v.begin(), v.end(),
                     [](const Costed& a, const Costed& b) { return a.cost > b.cost; });
    std::vector<WorkItem> out(v.size());
    for (size_t i = 0; i < v.size(); ++i) out[i] = v[i].w;
    return out;
}

struct Triple {
    FilterJob j;
    ClassKey key;
    const vktFilter_* f;
};

// Tuning-table key of one class of a batch, and the entry the table holds
// for it (tz 0: none).
TuneKey tune_key(const std::vector<Triple>& tr, const ClassPlan& cp)
{
    std::vector<FilterJob> jobs;
    for (int idx : cp.members) jobs.push_back(tr[idx].j);
    return TuneKey{cp.key, size_class_of(jobs)};
}

TuneVal tuned(const TuneKey& tk)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    tune_load_locked();
    auto it = g_tune.find(tk);
    return it != g_tune.end() ? it->second : TuneVal{0, 0};
}

// Slab depth where the table has no entry.  Each slab reads and multiplies k - 1
// planes besides its own, so the matrix-core classes take 64 planes where that
// still leaves an item for each CU (the classes run side by side, so that one
// class's tail is filled by another's items).  Against 16 planes (20 and 28 for
// k = 5 and 7): 256 uint16 volumes of 32 to 256 2450 -> 2270 us, 128 float32 of 40
// to 160 769 -> 730 us, 48 of 64 to 180 553 -> 529 us, 24 uint8 of 96 to 256
// 446 -> 433 us.  With the line at four items per CU the last three stayed as
// they were.  The vector classes, whose planes cost less, keep 16.
int default_tz(const std::vector<Triple>& tr, const ClassPlan& cp, const ClassGeom& g)
{
    constexpr int kDeep = 64;
    const int base = std::max(g.tz_min, 16);
    if (cp.key.path != 1 || base >= kDeep) return base;
    int64_t n = 0;
    for (int idx : cp.members) {
        const FilterJob& j = tr[idx].j;
        n += (int64_t)tiles_along(j.X, g.tx) * tiles_along(j.Y, g.ty) *
             ((j.Z + kDeep - 1) / kDeep);
    }
    return n >= (int64_t)device_cus() ? kDeep : base;
}

// Build (or rebuild for another slab depth) the host-side arrays of one class.
void class_arrays(const std::vector<Triple>& tr, ClassPlan& cp, std::vector<VolDesc>& descs,
                  std::vector<WorkItem>& items, std::vector<float>& wf,
                  std::vector<int32_t>& wi)
{
    const ClassGeom g = class_geom(cp.key, cp.variant);
    descs.clear();
    wf.clear();
    wi.clear();
    std::map<uint64_t, uint32_t> woff;  // filter serial -> pool offset
    const int n3 = class_weights(cp.key);
    for (int idx : cp.members) {
        const Triple& t = tr[idx];
        VolDesc a = make_desc(t.j, std::min(cp.tz, t.j.Z), g);
        auto it = woff.find(t.f->serial);
        if (it == woff.end()) {
            const uint32_t off = (uint32_t)wf.size();
            wf.resize(wf.size() + n3);
            wi.resize(wi.size() + n3);
            it = woff.emplace(t.f->serial, off).first;
        }
        a.woff = it->second;
        descs.push_back(a);
    }
    items = make_items(descs, cp.members, cp.key.k);
}

// Device copies of the weights go into the pools with device-to-device
// copies (the filters' weights live on the device).
hipError_t upload_class(const std::vector<Triple>& tr, ClassPlan& cp, char* base,
                        const std::vector<VolDesc>& descs, const std::vector<WorkItem>& items)
{
    hipError_t e = hipMemcpy(base + cp.off_desc, descs.data(), descs.size() * sizeof(VolDesc),
                             hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(base + cp.off_items, items.data(), items.size() * sizeof(WorkItem),
                      hipMemcpyHostToDevice);
    const int n3 = class_weights(cp.key);
    for (size_t m = 0; m < cp.members.size() && e == hipSuccess; ++m) {
        const vktFilter_* f = tr[cp.members[m]].f;
        const uint32_t off = descs[m].woff;
        if (cp.key.path == 2) {
            e = hipMemcpy(base + cp.off_wi + off * sizeof(int32_t), f->d_wq,
                          n3 * sizeof(uint32_t), hipMemcpyDeviceToDevice);
            continue;
        }
        e = hipMemcpy(base + cp.off_wf + off * sizeof(float), f->d_wf, n3 * sizeof(float),
                      hipMemcpyDeviceToDevice);
        if (e == hipSuccess && f->d_wi)
            e = hipMemcpy(base + cp.off_wi + off * sizeof(int32_t), f->d_wi,
                          n3 * sizeof(int32_t), hipMemcpyDeviceToDevice);
    }
    // (copies on the device need not have ended when they return, and the class
    // may run on a stream that does not wait for the null stream)
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    cp.nitems = (uint32_t)items.size();
    cp.args.vols = reinterpret_cast<const VolDesc*>(base + cp.off_desc);
    cp.args.items = reinterpret_cast<const WorkItem*>(base + cp.off_items);
    cp.args.nitems = cp.nitems;
    cp.args.counters = reinterpret_cast<uint32_t*>(base + cp.off_cnt);
    cp.args.wpool = reinterpret_cast<const float*>(base + cp.off_wf);
    cp.args.wipool = reinterpret_cast<const int32_t*>(base + cp.off_wi);
    return e;
}

hipError_t launch_class(const ClassPlan& cp, hipStream_t s)
{
    BatchArgs a = cp.args;
    void* params[] = {&a};
    return hipLaunchKernel(cp.func, dim3(cp.grid), dim3(256), params, 0, s);
}

// All classes of a plan, side by side on its side streams (one class: on the
// caller's stream).  Up to three leave the caller's lane empty, so that they start
// together: the class there runs ahead of the others by the fork, and whichever it was
// some batch became slower (256 uint8 volumes of 16 to 96, k = 3, 5, 7: with 3,
// 5 or 7 there 258, 238 and 273 us, with none 242; 64 float32 of 16 to 64: 124,
// 113 and 107, with none 113; 16 uint16 of 8 to 48: 86, 100 and 92, with none
// 84).  One after another on the caller's stream the last three sets take 287,
// 141 and 115 us, as nodes of one graph they took 234, 114 and 88.
hipError_t launch_plan(const Plan& p, hipStream_t s)
{
    if (!p.side) {
        hipError_t e = hipSuccess;
        for (size_t i = 0; i < p.classes.size() && e == hipSuccess; ++i)
            e = launch_class(p.classes[i], s);
        return e;
    }
    SideStreams& sd = *p.side;
    const size_t lanes = std::min(p.classes.size(), sd.n);
    hipError_t e = hipEventRecord(sd.fork, s);
    size_t forked = 0;
    for (; forked < lanes && e == hipSuccess; ++forked)
        e = hipStreamWaitEvent(sd.stream[forked], sd.fork, 0);
    for (size_t i = 0; i < p.classes.size() && e == hipSuccess; ++i)
        e = launch_class(p.classes[i], p.classes[i].lane < lanes ? sd.stream[p.classes[i].lane] : s);
    // joined whatever failed: s must not run ahead of what was launched
    for (size_t l = 0; l < forked; ++l) {
        hipError_t j = hipEventRecord(sd.joined[l], sd.stream[l]);
        if (j == hipSuccess) j = hipStreamWaitEvent(s, sd.joined[l], 0);
        if (e == hipSuccess) e = j;
    }
    return e;
}

// Time one class alone at a given slab depth (two launches on the caller's
// stream, the second timed; waits for both).
float time_class(const std::vector<Triple>& tr, ClassPlan& cp, char* base, int tz, int variant,
                 hipStream_t s)
{
    cp.tz = tz;
    cp.variant = variant;
    cp.func = class_kernel(cp.key, variant);
    int per_cu = 0, cus = 0, dev = 0;
    (void)hipGetDevice(&dev);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, cp.func, 256, 0) != hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 1;
    cp.grid = (unsigned)(per_cu * cus);
    std::vector<VolDesc> descs;
    std::vector<WorkItem> items;
    std::vector<float> wf;
    std::vector<int32_t> wi;
    class_arrays(tr, cp, descs, items, wf, wi);
    if (upload_class(tr, cp, base, descs, items) != hipSuccess) return -1.f;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return -1.f;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return -1.f;
    }
    float ms = -1.f;
    if (launch_class(cp, s) == hipSuccess && hipEventRecord(e0, s) == hipSuccess &&
        launch_class(cp, s) == hipSuccess && hipEventRecord(e1, s) == hipSuccess &&
        hipEventSynchronize(e1) == hipSuccess)
        (void)hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return ms;
}

// Lanes of a plan's classes: a side stream each, or, where there are more classes
// than those, the side streams and the caller's shared out: the longest class first,
// each to the lane that is free soonest; a class takes some 40 us however small it is (a slab's chain of
// planes), as long as 8e8 taps.  (9 classes of 24 volumes of 16 to 64, and of 96
// of 32 to 128: 141 and 313 us, as nodes of one graph 143 and 310; by taps alone 154
// and 315, dealt out in turn 132 and 334, to 3 lanes 181 and 344.)
void assign_lanes(const std::vector<Triple>& tr, Plan& plan)
{
    if (plan.classes.size() <= plan.side->n) {
        for (size_t i = 0; i < plan.classes.size(); ++i) plan.classes[i].lane = i;
        return;
    }
    std::vector<std::pair<double, ClassPlan*>> order;
    for (auto& cp : plan.classes) {
        double taps = 8e8;
        for (int idx : cp.members) {
            const FilterJob& j = tr[idx].j;
            taps += (double)j.X * j.Y * j.Z * j.k * j.k * j.k;
        }
        order.push_back({taps, &cp});
    }
    std::stable_sort(order.begin(), order.end(),
                     [](const auto& a, const auto& b) { return a.first > b.first; });
    std::vector<double> load(plan.side->n + 1, 0.0);
    for (auto& o : order) {
        const size_t l = std::min_element(load.begin(), load.end()) - load.begin();
        load[l] += o.first;
        o.second->lane = l;
    }
}

vktError build_plan(const std::vector<Triple>& tr, std::vector<uintptr_t>&& sig, bool tune,
                    hipStream_t stream, std::shared_ptr<Plan>& out)
{
    auto plan = std::make_shared<Plan>();
    plan->sig = std::move(sig);
    if (hipGetDevice(&plan->device) != hipSuccess) return vktDeviceError;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, plan->device) !=
        hipSuccess)
        return vktDeviceError;

    std::map<ClassKey, std::vector<int>> groups;
    for (size_t i = 0; i < tr.size(); ++i) groups[tr[i].key].push_back((int)i);

    // size the device buffer for the most items any candidate makes (the
    // shorter tile variant at its smallest slab depth), so tuning and the
    // final plan fit
    size_t bytes = 0;
    for (auto& g : groups) {
        ClassPlan cp;
        cp.key = g.first;
        cp.members = g.second;
        cp.func = class_kernel(cp.key, 0);
        if (!cp.func) return vktUnsupported;
        size_t nitems = 0;
        for (int v = 0; v < kTileVariants; ++v) {
            const ClassGeom geom = class_geom(cp.key, v);
            size_t n = 0;
            for (int idx : cp.members) {
                const FilterJob& j = tr[idx].j;
                const int tzmin = std::min(geom.tz_min, j.Z);
                n += (size_t)tiles_along(j.X, geom.tx) * tiles_along(j.Y, geom.ty) *
                     ((j.Z + tzmin - 1) / tzmin);
            }
            nitems = std::max(nitems, n);
        }
        const size_t n3 = (size_t)class_weights(cp.key);
        cp.off_desc = bytes = align_up(bytes, 256);
        bytes += cp.members.size() * sizeof(VolDesc);
        cp.off_items = bytes = align_up(bytes, 256);
        bytes += nitems * sizeof(WorkItem);
        cp.off_cnt = bytes = align_up(bytes, 256);
        bytes += 2 * sizeof(uint32_t);
        cp.off_wf = bytes = align_up(bytes, 256);
        bytes += (cp.members.size() * n3 + kWeightPad) * sizeof(float);
        cp.off_wi = bytes = align_up(bytes, 256);
        bytes += (cp.members.size() * n3 + kWeightPad) * sizeof(int32_t);
        plan->classes.push_back(cp);
    }
    plan->dbytes = bytes;
    hipError_t e = hipMalloc(&plan->dbuf, bytes);
    if (e != hipSuccess) return from_hip(e);
    e = hipMemset(plan->dbuf, 0, bytes);  // queue counters start at zero
    if (e != hipSuccess) return from_hip(e);

    for (auto& cp : plan->classes) {
        const TuneKey tk = tune_key(tr, cp);
        TuneVal tv = tuned(tk);
        if (tv.tz == 0 && tune) {
            // autotune: time every tile variant at candidate slab depths on
            // the real batch
            float best = -1.f;
            for (int v = 0; v < kTileVariants; ++v) {
                const ClassGeom geom = class_geom(cp.key, v);
                for (int cand : {8, 16, 32, 64}) {
                    if (cand < geom.tz_min && cand != 64) continue;
                    const float ms = time_class(tr, cp, plan->dbuf, std::max(cand, geom.tz_min),
                                                v, stream);
                    if (ms > 0.f && (best < 0.f || ms < best)) {
                        best = ms;
                        tv = TuneVal{std::max(cand, geom.tz_min), v};
                    }
                }
            }
            if (tv.tz > 0) {
                std::lock_guard<std::mutex> lk(g_tune_mu);
                g_tune[tk] = tv;
                tune_store_locked();
            }
        }
        cp.variant = tv.tz > 0 ? tv.variant : 0;
        const ClassGeom geom = class_geom(cp.key, cp.variant);
        cp.tz = std::max(tv.tz > 0 ? tv.tz : default_tz(tr, cp, geom), geom.tz_min);
        cp.func = class_kernel(cp.key, cp.variant);
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, cp.func, 256, 0) !=
                hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        cp.grid = (unsigned)(per_cu * cus);
        std::vector<VolDesc> descs;
        std::vector<WorkItem> items;
        std::vector<float> wf;
        std::vector<int32_t> wi;
        class_arrays(tr, cp, descs, items, wf, wi);
        e = upload_class(tr, cp, plan->dbuf, descs, items);
        if (e != hipSuccess) return from_hip(e);
        if (cp.grid > cp.nitems) cp.grid = cp.nitems > 0 ? cp.nitems : 1;
    }

    if (plan->classes.size() > 1)
        plan->side = take_side_streams(plan->device, stream,
                                       std::min(plan->classes.size(), kSideStreams));
    if (plan->side) assign_lanes(tr, *plan);
    e = hipEventCreateWithFlags(&plan->done, hipEventDisableTiming);
    if (e != hipSuccess) return from_hip(e);

    out = plan;
    std::shared_ptr<Plan> evicted;  // released after the lock (hipFree waits)
    {
        std::lock_guard<std::mutex> lk(g_plan_mu);
        if (g_plans.size() >= kMaxPlans) {
            evicted = std::move(g_plans.front());
            g_plans.erase(g_plans.begin());
        }
        g_plans.push_back(std::move(plan));
    }
    return vktNoError;
}

// Validate and plan every triple of a batch exactly as vktApplyFilter would,
// check that no output overlaps any volume of the batch, and collect the
// batch signature (the plan cache key).
vktError prepare_batch(int32_t n, const vktStructuredVolume* dst, const vktStructuredVolume* src,
                       const vktFilter* filters, vktAddressMode mode, vktPrecision prec,
                       hipStream_t stream, std::vector<Triple>& tr, std::vector<uintptr_t>& sig)
{
    tr.assign(n, Triple{});
    sig.clear();
    sig.reserve(4 + 6 * (size_t)n);
    sig.push_back((uintptr_t)n);
    sig.push_back((uintptr_t)mode);
    sig.push_back((uintptr_t)prec);
    sig.push_back((uintptr_t)thread_row_pair_min_cells());
    sig.push_back((uintptr_t)stream);
    for (int i = 0; i < n; ++i) {
        bool mfma = false, six = false;
        // (the batched form always runs the dense arithmetic)
        const vktError e =
            build_job(dst[i], src[i], filters[i], mode, prec, tr[i].j, mfma, six, nullptr, false);
        if (e != vktNoError) return e;
        const FilterJob& j = tr[i].j;
        tr[i].f = filters[i];
        if (mfma)
            tr[i].key = ClassKey{(int)j.fmt, j.k, 1, (six ? 1 : 0) | (mfma_row_pairs(j, six) ? 2 : 0)};
        else if (j.dot4) tr[i].key = ClassKey{(int)j.fmt, j.k, 2, j.q_signed ? 1 : 0};
        else tr[i].key = ClassKey{(int)j.fmt, j.k, 0, j.int_acc ? 1 : 0};
        sig.push_back((uintptr_t)j.src);
        sig.push_back((uintptr_t)j.dst);
        sig.push_back((uintptr_t)filters[i]->serial);
        sig.push_back((uintptr_t)j.X);
        sig.push_back((uintptr_t)j.Y);
        sig.push_back((uintptr_t)j.Z | ((uintptr_t)j.fmt << 40));
    }
    // outputs must not overlap any volume of the batch (they run concurrently)
    std::vector<std::pair<uintptr_t, uintptr_t>> dr, sr;
    for (int i = 0; i < n; ++i) {
        const uintptr_t b = (uintptr_t)cell_bytes(tr[i].j.fmt) * tr[i].j.X * tr[i].j.Y * tr[i].j.Z;
        dr.push_back({(uintptr_t)tr[i].j.dst, (uintptr_t)tr[i].j.dst + b});
        sr.push_back({(uintptr_t)tr[i].j.src, (uintptr_t)tr[i].j.src + b});
    }
    std::sort(dr.begin(), dr.end());
    for (size_t i = 1; i < dr.size(); ++i)
        if (dr[i].first < dr[i - 1].second) return vktInvalidValue;
    // sources sorted by start with the running maximum of their ends: an
    // output [a, b) meets a source iff some source starting before b ends
    // after a
    std::sort(sr.begin(), sr.end());
    std::vector<uintptr_t> max_end(sr.size());
    for (size_t i = 0; i < sr.size(); ++i)
        max_end[i] = std::max(sr[i].second, i ? max_end[i - 1] : (uintptr_t)0);
    for (const auto& d : dr) {
        const size_t m = (size_t)(std::lower_bound(sr.begin(), sr.end(),
                                                   std::make_pair(d.second, (uintptr_t)0)) -
                                  sr.begin());
        if (m > 0 && max_end[m - 1] > d.first) return vktInvalidValue;
    }
    return vktNoError;
}

// ---- allocation-free form ---------------------------------------------------
//
// The batch's descriptors, work lists, work-queue counters and weight pools
// go to this file-scope device array instead of a plan buffer.  Host code
// never passes the array's name to a kernel or a copy (on the host it is a
// stand-in, not a device address): it uses the address that
// hipGetSymbolAddress returns for the current device, looked up once per
// device.
constexpr size_t kNoAllocBytes = size_t(8) << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocBytes];

struct NoAllocDevice {
    unsigned char* ptr = nullptr;       // this device's copy of `scratch`
    std::vector<unsigned char> staging; // host image of the array's head
    hipEvent_t copied = nullptr;        // the last upload from `staging` is done
    bool pending = false;
    std::mutex mu;                      // one call per device at a time (host side)
};
std::mutex g_noalloc_mu;
std::map<int, std::unique_ptr<NoAllocDevice>> g_noalloc;

// Set-up on the first call on a device, with that device current.
vktError noalloc_device(int dev, NoAllocDevice*& out)
{
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    auto it = g_noalloc.find(dev);
    if (it == g_noalloc.end()) {
        auto d = std::make_unique<NoAllocDevice>();
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return vktDeviceError;
        e = hipEventCreateWithFlags(&d->copied, hipEventDisableTiming);
        if (e != hipSuccess) return vktDeviceError;
        d->ptr = static_cast<unsigned char*>(p);
        d->staging.resize(kNoAllocBytes);
        it = g_noalloc.emplace(dev, std::move(d)).first;
    }
    out = it->second.get();
    return vktNoError;
}

vktError batched_no_alloc(const std::vector<Triple>& tr, hipStream_t stream)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return vktDeviceError;
    NoAllocDevice* nd = nullptr;
    vktError ve = noalloc_device(dev, nd);
    if (ve != vktNoError) return ve;

    // plan every class as the cached form does (same tile variants and slab
    // depths: the tuning table's entry, else the defaults; this form never
    // times candidates)
    std::map<ClassKey, std::vector<int>> groups;
    for (size_t i = 0; i < tr.size(); ++i) groups[tr[i].key].push_back((int)i);
    std::vector<ClassPlan> classes;
    std::vector<std::vector<VolDesc>> descs(groups.size());
    std::vector<std::vector<WorkItem>> items(groups.size());
    std::vector<size_t> npool(groups.size());
    // layout: the heads of all classes (descriptors, work list, counters),
    // then the weight pools; returns the bytes it takes (0: no kernel)
    auto lay_out = [&](bool taller) -> size_t {
        size_t bytes = 0, c = 0;
        classes.clear();
        for (auto& g : groups) {
            ClassPlan cp;
            cp.key = g.first;
            cp.members = g.second;
            const TuneVal tv = tuned(tune_key(tr, cp));
            cp.variant = tv.tz > 0 ? tv.variant : 0;
            int tz = tv.tz;  // 0: none
            if (taller && class_geom(cp.key, 1 - cp.variant).ty > class_geom(cp.key, cp.variant).ty) {
                // (the table's depth was timed on the other tile; it stays where it
                // is the deeper one, which makes fewer items)
                cp.variant = 1 - cp.variant;
                tz = std::max(tz, default_tz(tr, cp, class_geom(cp.key, cp.variant)));
            }
            cp.func = class_kernel(cp.key, cp.variant);
            if (!cp.func) return 0;
            const ClassGeom geom = class_geom(cp.key, cp.variant);
            cp.tz = std::max(tz > 0 ? tz : default_tz(tr, cp, geom), geom.tz_min);
            std::vector<float> wf;
            std::vector<int32_t> wi;
            class_arrays(tr, cp, descs[c], items[c], wf, wi);
            const size_t n3 = (size_t)class_weights(cp.key);
            npool[c] = 0;
            for (const auto& d : descs[c]) npool[c] = std::max(npool[c], (size_t)d.woff / n3 + 1);
            cp.off_desc = bytes = align_up(bytes, 256);
            bytes += descs[c].size() * sizeof(VolDesc);
            cp.off_items = bytes = align_up(bytes, 256);
            bytes += items[c].size() * sizeof(WorkItem);
            cp.off_cnt = bytes = align_up(bytes, 256);
            bytes += 2 * sizeof(uint32_t);
            cp.grid = (unsigned)resident_wgs(cp.func);
            classes.push_back(cp);
            ++c;
        }
        for (size_t i = 0; i < classes.size(); ++i) {
            ClassPlan& cp = classes[i];
            const size_t n3 = (size_t)class_weights(cp.key);
            cp.off_wf = bytes = align_up(bytes, 256);
            bytes += (npool[i] * n3 + kWeightPad) * sizeof(float);
            cp.off_wi = bytes = align_up(bytes, 256);
            bytes += (npool[i] * n3 + kWeightPad) * sizeof(int32_t);
        }
        return bytes;
    };
    size_t bytes = lay_out(false);
    // taller tiles make fewer items (6-product float32 13^3 and 15^3 run on the
    // shorter ones, which halves the rows that the scratch holds items for)
    if (bytes > kNoAllocBytes) bytes = lay_out(true);
    if (bytes == 0) return vktUnsupported;
    if (bytes > kNoAllocBytes) return vktUnsupported;  // the batch does not fit

    std::lock_guard<std::mutex> lk(nd->mu);
    // the previous upload must have read the staging image before it changes
    if (nd->pending && hipEventSynchronize(nd->copied) != hipSuccess) return vktDeviceError;
    nd->pending = false;
    // image of the used region: descriptors, work lists, zeroed counters and
    // zeroed weight pools (the upload clears the counters and the pools' pads;
    // the weights come from the filters' device buffers below)
    std::memset(nd->staging.data(), 0, bytes);
    for (size_t i = 0; i < classes.size(); ++i) {
        const ClassPlan& cp = classes[i];
        std::memcpy(&nd->staging[cp.off_desc], descs[i].data(), descs[i].size() * sizeof(VolDesc));
        std::memcpy(&nd->staging[cp.off_items], items[i].data(),
                    items[i].size() * sizeof(WorkItem));
    }
    hipError_t e =
        hipMemcpyAsync(nd->ptr, nd->staging.data(), bytes, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) e = hipEventRecord(nd->copied, stream);
    if (e != hipSuccess) return from_hip(e);
    nd->pending = true;
    for (size_t i = 0; i < classes.size() && e == hipSuccess; ++i) {
        ClassPlan& cp = classes[i];
        const size_t n3 = (size_t)class_weights(cp.key);
        std::map<uint32_t, const vktFilter_*> pool;
        for (size_t m = 0; m < cp.members.size(); ++m)
            pool.emplace(descs[i][m].woff, tr[cp.members[m]].f);
        for (const auto& pf : pool) {
            const vktFilter_* f = pf.second;
            const uint32_t off = pf.first;
            if (cp.key.path == 2) {
                e = hipMemcpyAsync(nd->ptr + cp.off_wi + off * sizeof(int32_t), f->d_wq,
                                   n3 * sizeof(uint32_t), hipMemcpyDeviceToDevice, stream);
            } else {
                e = hipMemcpyAsync(nd->ptr + cp.off_wf + off * sizeof(float), f->d_wf,
                                   n3 * sizeof(float), hipMemcpyDeviceToDevice, stream);
                if (e == hipSuccess && f->d_wi)
                    e = hipMemcpyAsync(nd->ptr + cp.off_wi + off * sizeof(int32_t), f->d_wi,
                                       n3 * sizeof(int32_t), hipMemcpyDeviceToDevice, stream);
            }
            if (e != hipSuccess) break;
        }
        cp.nitems = (uint32_t)items[i].size();
        cp.args.vols = reinterpret_cast<const VolDesc*>(nd->ptr + cp.off_desc);
        cp.args.items = reinterpret_cast<const WorkItem*>(nd->ptr + cp.off_items);
        cp.args.nitems = cp.nitems;
        cp.args.counters = reinterpret_cast<uint32_t*>(nd->ptr + cp.off_cnt);
        cp.args.wpool = reinterpret_cast<const float*>(nd->ptr + cp.off_wf);
        cp.args.wipool = reinterpret_cast<const int32_t*>(nd->ptr + cp.off_wi);
        if (cp.grid > cp.nitems) cp.grid = cp.nitems > 0 ? cp.nitems : 1;
        if (e == hipSuccess) e = launch_class(cp, stream);
    }
    return from_hip(e);
}

}  // namespace
}  // namespace vkt

extern "C" {

vktError vktApplyFilterBatched(int32_t n, const vktStructuredVolume* dst,
                               const vktStructuredVolume* src, const vktFilter* filters,
                               vktAddressMode mode)
{
    using namespace vkt;
    if (n < 0 || (n > 0 && (!dst || !src || !filters))) return vktInvalidValue;
    if (n == 0) return vktNoError;
    const vktPrecision prec = thread_precision();
    hipStream_t stream = thread_stream();
    std::vector<Triple> tr;
    std::vector<uintptr_t> sig;
    const vktError ve = prepare_batch(n, dst, src, filters, mode, prec, stream, tr, sig);
    if (ve != vktNoError) return ve;

    std::lock_guard<std::mutex> serial(g_batch_mu);
    std::shared_ptr<Plan> plan;
    {
        int dev = 0;
        (void)hipGetDevice(&dev);
        std::lock_guard<std::mutex> lk(g_plan_mu);
        for (auto it = g_plans.begin(); it != g_plans.end(); ++it)
            if ((*it)->sig == sig && (*it)->device == dev) {
                plan = *it;
                g_plans.erase(it);        // a hit becomes the most recently used
                g_plans.push_back(plan);
                break;
            }
    }
    if (!plan) {
        const vktError e = build_plan(tr, std::move(sig), thread_autotune(), stream, plan);
        if (e != vktNoError) return e;
    }
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
        (void)hipGetLastError();  // (the legacy stream, while another one is captured)
        cap = hipStreamCaptureStatusNone;
    }
    hipError_t e = launch_plan(*plan, stream);
    if (cap != hipStreamCaptureStatusNone) {
        // (recorded, not run: nothing to wait for when the plan is evicted, but
        // the caller's graph needs its buffer from now on)
        if (!plan->captured) g_captured.push_back(plan);
        plan->captured = true;
    } else if (e == hipSuccess) {
        e = hipEventRecord(plan->done, stream);
    }
    return from_hip(e);
}

vktError vktApplyFilterBatchedNoAlloc(int32_t n, const vktStructuredVolume* dst,
                                      const vktStructuredVolume* src, const vktFilter* filters,
                                      vktAddressMode mode)
{
    using namespace vkt;
    if (n < 0 || (n > 0 && (!dst || !src || !filters))) return vktInvalidValue;
    if (n == 0) return vktNoError;
    hipStream_t stream = thread_stream();
    std::vector<Triple> tr;
    std::vector<uintptr_t> sig;
    const vktError ve =
        prepare_batch(n, dst, src, filters, mode, thread_precision(), stream, tr, sig);
    if (ve != vktNoError) return ve;
    return batched_no_alloc(tr, stream);
}

}  // extern "C"
