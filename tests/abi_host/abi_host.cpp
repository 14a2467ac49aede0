// CPU build of the C-ABI (csrc/abi.cpp as it is) on a model of the HIP calls that its
// batches make, for tests/test_batch_host.py. Device and pinned memory are host
// allocations with a guard behind them, copies are made at once, and a GF(2)[t] launch,
// direct or from a replayed graph, is checked instead of run: every workgroup of every
// job of the batch has to come exactly once, in a launch of its own step, with its
// workspace inside one allocation.
#include <cstdlib>
#include <mutex>
#include <set>

#include "../../paper_2402_09481_amd/csrc/abi.cpp"

namespace {

constexpr size_t GUARD = size_t(1) << 16;
std::map<char *, size_t> g_blocks;
int g_faults = 0;
int g_running = 0;  // what an event query answers: 0 done, 1 not ready, 2 an error
bool g_capturing = false;
int g_unfenced = 0, g_events = 0;             // events made, and those without a system fence

void *block_new(size_t bytes) {
    char *p = (char *)calloc(1, bytes + GUARD);
    if (!p) return nullptr;
    memset(p + bytes, 0xA5, GUARD);
    g_blocks[p] = bytes;
    return p;
}
bool guard_whole(const char *p, size_t bytes) {
    for (size_t i = 0; i < GUARD; ++i)
        if ((unsigned char)p[bytes + i] != 0xA5) return false;
    return true;
}
void block_free(void *p) {
    auto it = g_blocks.find((char *)p);
    if (it == g_blocks.end()) {
        ++g_faults;
        return;
    }
    if (!guard_whole(it->first, it->second)) ++g_faults;
    g_blocks.erase(it);
    free(p);
}
bool inside(const void *p, size_t bytes) {
    auto it = g_blocks.upper_bound((char *)p);
    if (it == g_blocks.begin()) return false;
    --it;
    return (char *)p + bytes <= it->first + it->second;
}

enum Step { BITS, FWD, MUL, ROWS_FWD, PROD, ROWS_INV, INV, NSTEPS };
const char *const STEP_NAMES[NSTEPS] = {"bits", "fwd", "mul", "rows_fwd", "prod", "rows_inv", "inv"};

struct Launch {
    std::string label;
    int step = -1;  // GF(2)[t] launches
    uint32_t wgs = 0, threads = 0;
    const Gf2Job *jobs = nullptr;
    const uint2 *tab = nullptr;
    int rows_lg = 0, one_group = -1;
};
typedef std::vector<Launch> LaunchList;

GraphRecorder *g_recorder = nullptr;
std::string g_labels;
uint64_t g_most_threads = 0;
struct Seen {
    Gf2Job job;
    std::vector<bool> at[NSTEPS];
};
std::map<const void *, Seen> g_seen;  // by output address
size_t g_transform_jobs = 0;

uint32_t expected(const Gf2Job &j, int step) {
    if (!j.px) return step == BITS ? gf2_bits_workgroups(j, true) : 0;
    switch (step) {
        case FWD: return gf2_fwd_workgroups(j);
        case MUL: return j.rows_lg ? 0 : gf2_mul_workgroups(j);
        case ROWS_FWD: return j.rows_lg ? gf2_rows_fwd_workgroups(j) : 0;
        case PROD: return j.rows_lg ? gf2_rows_prod_workgroups(j) : 0;
        case ROWS_INV: return j.rows_lg ? gf2_rows_inv_workgroups(j) : 0;
        case INV: return gf2_inv_workgroups(j);
    }
    return 0;
}

void execute(const Launch &l) {
    if (g_labels.size() < 4096) g_labels += l.label + " ";
    if (l.step < 0) return;
    g_most_threads = std::max(g_most_threads, (uint64_t)l.wgs * l.threads);
    if (!inside(l.tab, (size_t)l.wgs * sizeof(uint2))) {
        ++g_faults;
        return;
    }
    for (uint32_t w = 0; w < l.wgs; ++w) {
        const uint2 t = l.tab[w];
        if (!inside(l.jobs + t.x, sizeof(Gf2Job))) {
            ++g_faults;
            return;
        }
        const Gf2Job &j = l.jobs[t.x];
        auto it = g_seen.find(j.z);
        if (it == g_seen.end()) {
            it = g_seen.emplace(j.z, Seen{j, {}}).first;
            for (int s = 0; s < NSTEPS; ++s) it->second.at[s].assign(expected(j, s), false);
            if (j.px && !inside(j.X, (char *)j.flags + 256 - (char *)j.X)) ++g_faults;
        }
        std::vector<bool> &at = it->second.at[l.step];
        const bool fits = (!l.rows_lg || (uint32_t)l.rows_lg == j.rows_lg) &&
                          (l.one_group < 0 || (l.one_group == 1) == (j.nz == 1));
        if (!fits || t.y >= at.size() || at[t.y]) ++g_faults;
        else at[t.y] = true;
    }
}

hipError_t launch(const Launch &l) {
    if (g_recorder) ((LaunchList *)g_recorder->graph)->push_back(l);
    else execute(l);
    return hipSuccess;
}
hipError_t launch_gf2(int step, uint32_t wgs, uint32_t threads, const Gf2Job *jobs, const uint2 *tab, int rows_lg = 0,
                      int one_group = -1) {
    Launch l;
    l.label = STEP_NAMES[step];
    l.step = step;
    l.wgs = wgs;
    l.threads = threads;
    l.jobs = jobs;
    l.tab = tab;
    l.rows_lg = rows_lg;
    l.one_group = one_group;
    return launch(l);
}
hipError_t launch_other(const char *label) {
    Launch l;
    l.label = label;
    return launch(l);
}

}  // namespace

namespace ext {
void set_graph_recorder(GraphRecorder *rec) { g_recorder = rec; }
void set_launch_event(LaunchEvent *) {}
hipError_t launch_gf2_bits(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &, const uint2 *tab, hipStream_t) {
    return launch_gf2(BITS, wgs, 512, jobs, tab);
}
hipError_t launch_gf2_fwd(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &, const uint2 *tab, hipStream_t) {
    return launch_gf2(FWD, wgs, 256, jobs, tab);
}
hipError_t launch_gf2_mul(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &, const uint2 *tab, hipStream_t) {
    return launch_gf2(MUL, wgs, 512, jobs, tab);
}
hipError_t launch_gf2_rows_fwd(int p, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &, const uint2 *tab, hipStream_t) {
    return launch_gf2(ROWS_FWD, wgs, 1u << (p - 2), jobs, tab, p);
}
hipError_t launch_gf2_rows_prod(bool one, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &, const uint2 *tab, hipStream_t) {
    return launch_gf2(PROD, wgs, 256, jobs, tab, 0, one);
}
hipError_t launch_gf2_rows_inv(int p, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &, const uint2 *tab, hipStream_t) {
    return launch_gf2(ROWS_INV, wgs, 1u << (p - 2), jobs, tab, p);
}
hipError_t launch_gf2_inv(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &, const uint2 *tab, hipStream_t) {
    return launch_gf2(INV, wgs, 256, jobs, tab);
}
hipError_t launch_small_batch(const SmallClasses &, const JobDev *, uint32_t *, unsigned, const Tables &, hipStream_t) {
    return launch_other("small");
}
hipError_t launch_embed(uint32_t, uint64_t, int, int, const JobDev *, const JobDev *, bool, hipStream_t) {
    return launch_other("embed");
}
hipError_t launch_strided(const PassLaunch &, const Tables &, hipStream_t) { return launch_other("strided"); }
hipError_t launch_contig(const PassLaunch &, const Tables &, hipStream_t) { return launch_other("contig"); }
hipError_t launch_ptrans(int, uint64_t, uint64_t, uint64_t, uint32_t, const JobDev *, const JobDev *, bool, hipStream_t) {
    return launch_other("ptrans");
}
}  // namespace ext

extern "C" {
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMalloc(void **p, size_t bytes) {
    return (*p = block_new(bytes)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { return block_free(p), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { return (*p = block_new(bytes)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { return block_free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t bytes, hipMemcpyKind, hipStream_t) {
    if (!inside(to, bytes) || !inside(from, bytes)) return ++g_faults, hipSuccess;
    memcpy(to, from, bytes);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned flags) {
    ++g_events;
    g_unfenced += (flags & hipEventDisableSystemFence) != 0;
    return *e = (hipEvent_t)1, hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) {
    g_faults += g_capturing;
    return g_running == 2 ? hipErrorInvalidHandle : g_running ? hipErrorNotReady : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGraphCreate(hipGraph_t *g, unsigned) { return *g = (hipGraph_t) new LaunchList, hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { return delete (LaunchList *)g, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
    return *x = (hipGraphExec_t) new LaunchList(*(LaunchList *)g), hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return delete (LaunchList *)x, hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
    for (const Launch &l : *(LaunchList *)x) execute(l);
    return hipSuccess;
}

// ---- what the tests call

void *host_ctx(size_t budget, int gf2) {
    ext_ctx *c = new ext_ctx;
    c->budget = budget;
    c->split_min_lg = SPLIT_MIN_LG;
    c->batch_split_min_lg = BATCH_SPLIT_MIN_LG;
    c->gf2 = gf2 != 0;
    return c;
}
void host_ctx_free(void *p) {
    ext_ctx *c = (ext_ctx *)p;
    for (auto &kv : c->graphs) graph_entry_free(kv.second);
    for (auto &b : c->free_blocks) block_free(b.ptr);
    pinned_release_all(c);
    delete c;
}

// a workspace taken and given back, its last call done, still running or unknown (0, 1, 2), the stream captured or
// not; returns 1 if the release's event has no system fence (-1: a query under capture)
int host_release_event(void *ctx, int running, int capturing) {
    ext_ctx *c = (ext_ctx *)ctx;
    g_running = running;
    g_capturing = capturing;
    g_faults = g_unfenced = g_events = 0;
    Lease l;
    const int rc = pool_acquire(c, 1 << 20, nullptr, l);
    LaunchEvent *done = lease_event(l);
    const bool carried = done && done->ev;
    pool_release(c, l, nullptr);
    g_running = 0;
    g_capturing = false;
    if (rc != EXT_OK || g_faults || g_events != 1 || carried != (g_unfenced == 1)) return -1;
    return g_unfenced;
}

// One batch; shapes: kind, n, m of every job. Returns extract_batch's code. *faults: launches
// or copies that were wrong; *done: jobs whose every GF(2)[t] workgroup ran; *threads: of the
// largest launch; labels: the launches in order.
int host_batch(void *ctx, const uint64_t *shapes, size_t count, uint32_t flags, int *faults, size_t *done,
               uint64_t *threads, size_t *leased, char *labels, size_t cap) {
    ext_ctx *c = (ext_ctx *)ctx;
    std::vector<ext_job> jobs(count);
    for (size_t i = 0; i < count; ++i) {
        auto at = [&](size_t k) { return (uint64_t *)((4 * i + k + 1) << 30); };  // (addresses only)
        jobs[i] = ext_job{(int32_t)shapes[3 * i], 0, shapes[3 * i + 1], shapes[3 * i + 2], at(0), at(1), at(2), nullptr, 0, 0};
    }
    g_faults = 0;
    g_most_threads = 0;
    g_labels.clear();
    g_seen.clear();
    const int rc = extract_batch(c, jobs.data(), count, flags, nullptr);
    *done = 0;
    for (auto &kv : g_seen) {
        bool all = true;
        for (auto &at : kv.second.at)
            for (bool b : at) all &= b;
        *done += all;
        g_faults += !all;
    }
    for (auto &b : g_blocks) g_faults += !guard_whole(b.first, b.second);
    *faults = g_faults;
    *threads = g_most_threads;
    *leased = 0;
    for (auto &b : c->free_blocks) *leased = std::max(*leased, b.size);
    snprintf(labels, cap, "%s", g_labels.c_str());
    return rc;
}
}
