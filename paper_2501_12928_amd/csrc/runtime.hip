// Multi-instance runtime: many theta of many datasets of uneven size in one
// persistent launch, optionally replayed from a captured HIP graph, with the
// launch choices picked by a timing autotuner whose results persist in a
// small JSON cache keyed by (GPU architecture, size bucket): the launch shape
// for the group, and the side of the factorisation tiles (64 or 32) for each
// bucket of instance sizes, which one launch mixes freely.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <iterator>
#include <map>
#include <new>
#include <sstream>
#include <string>
#include <vector>

#include "common.h"
#include "spread.h"

using eor::Context;

namespace eor {

// A device buffer that is kept while it is large enough.
template <class T>
struct DeviceArray {
    T *p = nullptr;
    size_t cap = 0;
    // Room for n elements; true if the buffer is a new one.
    hipError_t ensure(size_t n, bool *fresh = nullptr) {
        if (fresh) *fresh = false;
        if (n <= cap) return hipSuccess;
        release();
        const hipError_t e = hipMalloc(&p, n * sizeof(T));
        if (e != hipSuccess) {
            p = nullptr;
            return e;
        }
        cap = n;
        if (fresh) *fresh = true;
        return hipSuccess;
    }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
        cap = 0;
    }
};

}  // namespace eor

struct eor_group {
    int device = 0;
    int num_cu = 0;
    std::vector<eor_ctx *> inst;
    eor::InstDesc *d_inst = nullptr;
    eor::InstDesc *h_inst = nullptr;     // pinned staging
    int2 *d_task = nullptr;
    int64_t ntask = 0;
    // For theta spread over all workgroups, of the task list: the two estimates,
    // the tile rows of the largest instance, the elements of L and of y and the
    // tiles in all. On the device, each kept while it is large enough: per task
    // where its L and its y start, with the number of tasks of at least r tile
    // rows behind them; w and y; the progress words (zero between launches).
    eor::DeviceArray<int64_t> spread_tab;
    eor::DeviceArray<double2> spread_y;
    eor::DeviceArray<int32_t> prog;
    bool spread_ready = false;           // spread_tab is that of the task list
    int64_t spread_rows = 0, spread_elems = 0, spread_y_elems = 0, spread_units = 0;
    double est_spread = 0.0, est_lone = 0.0;
    int spread_per_cu = 2;
    std::vector<int64_t> task_B, task_N; // B and tile rows per instance the task list was built for
    std::vector<int> order_N;            // the instances in list order, largest first
    unsigned int *counter = nullptr;
    bool counter_clear = false;          // cleared before the first launch, left at zero by each
    double2 *Lw = nullptr;
    double2 *yw = nullptr;
    int64_t slots = 0, slot_tiles = 0, slot_y = 0;
    int64_t N_max = 0;
    eor::Tuning tune;
    int ts_bucket[eor::N_BUCKETS] = {64, 64, 64, 64, 64};  // tile side per size bucket of n
    bool use_graph = true;
    // captured graph and what it was captured for
    hipStream_t cap_stream = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    eor::LikeParams cap_params;
    eor::SpreadParams cap_spread;
    bool cap_is_spread = false;
    int64_t cap_grid = 0;
    int cap_stages = 0;
    int cap_tiles = 0;
    int64_t replays = 0;
    int64_t captures = 0;
    eor::StreamOrder order;              // the last call's work on its stream
};

namespace {

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        (void)hipSetDevice(dev);
    }
    ~DeviceGuard() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

void drop_graph(eor_group &g) {
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
    if (g.graph) (void)hipGraphDestroy(g.graph);
    g.exec = nullptr;
    g.graph = nullptr;
    g.cap_grid = 0;
}

void free_work(eor_group &g) {
    if (g.Lw) (void)hipFree(g.Lw);
    if (g.yw) (void)hipFree(g.yw);
    g.Lw = nullptr;
    g.yw = nullptr;
    g.slots = 0;
    drop_graph(g);
}

eor_status ensure_work(eor_group &g, int64_t want) {
    if (g.slots >= want && g.slot_tiles == eor::n_tiles(g.N_max)) return EOR_OK;
    // queued work may still use the current slots
    const hipError_t ed = g.order.drain();
    if (ed != hipSuccess) return eor::hip_status(ed, "hipEventSynchronize");
    free_work(g);
    const int64_t slot_tiles = eor::n_tiles(g.N_max);
    const int64_t n_pad = g.N_max * eor::TS;
    int64_t slots = want;
    while (slots >= 1) {
        double2 *Lw = nullptr, *yw = nullptr;
        hipError_t e1 = hipMalloc(&Lw, (size_t)slots * slot_tiles * eor::TS2 * sizeof(double2));
        hipError_t e2 = e1 == hipSuccess ? hipMalloc(&yw, (size_t)slots * n_pad * sizeof(double2)) : e1;
        if (e1 == hipSuccess && e2 == hipSuccess) {
            g.Lw = Lw;
            g.yw = yw;
            g.slots = slots;
            g.slot_tiles = slot_tiles;
            g.slot_y = n_pad;
            return EOR_OK;
        }
        if (Lw) (void)hipFree(Lw);
        if (yw) (void)hipFree(yw);
        (void)hipGetLastError();
        if (slots == 1) break;
        slots /= 2;
    }
    return eor::fail_status(EOR_ERR_OOM, "cannot allocate the group workspace");
}

void free_tasks(eor_group &g) {
    if (g.d_task) (void)hipFree(g.d_task);
    g.d_task = nullptr;
    g.spread_ready = false;
    g.task_B.clear();
}

// Whether spreading every theta of the task list over all workgroups is sooner
// done by the estimates (few theta, or few large ones that would keep one
// workgroup each busy long after the others are done), and what it needs.
void plan_spread(eor_group &g) {
    std::vector<eor::Sizes> sizes;
    double chain = 0.0, work = 0.0;
    int64_t N_max = 0;
    g.spread_elems = g.spread_y_elems = g.spread_units = 0;
    for (int i : g.order_N) {
        const int64_t N = g.task_N[i], B = g.task_B[i];
        if (B < 1) continue;
        sizes.push_back({N, B});
        N_max = std::max(N_max, N);
        chain = std::max(chain, eor::spread_chain_us(N));
        work += B * eor::spread_work_us(N);
        g.spread_units += B * eor::n_tiles(N);
        g.spread_y_elems += B * N * eor::TS;
    }
    g.spread_elems = g.spread_units * eor::TS2;
    g.spread_rows = N_max;
    g.est_lone = eor::lone_group_us(sizes, g.num_cu);
    g.est_spread = eor::spread_us(chain, work, N_max);
    g.spread_per_cu = eor::spread_per_cu(chain, work, N_max);
    if (!(g.est_spread < 0.97 * g.est_lone) || g.spread_units >= ((int64_t)1 << 31) - 4096) g.est_spread = INFINITY;
}

// The memory of a planned spread launch: false if it cannot be had. The launch
// with one workgroup per theta needs none of it and is then taken. (No earlier
// spread launch is pending: a new task list has waited for the queued work.)
bool ensure_spread(eor_group &g) {
    if (g.spread_ready) return true;
    const int64_t n = g.ntask;
    const size_t words = (size_t)n * (g.spread_rows + eor::SPREAD_EXTRA);
    bool fresh = false;
    hipError_t e = g.spread_y.ensure(g.spread_y_elems);
    if (e == hipSuccess) e = g.prog.ensure(words, &fresh);
    if (e == hipSuccess && fresh) e = hipMemset(g.prog.p, 0, words * sizeof(int32_t));
    if (e == hipSuccess && fresh) e = hipStreamSynchronize(nullptr);
    // per task in list order (largest first) the starts of L and y, then the counts
    std::vector<int64_t> tab(2 * n + g.spread_rows / 2 + 1);
    int32_t *count = (int32_t *)(tab.data() + 2 * n);
    int64_t t = 0, at = 0, y = 0;
    for (int i : g.order_N) {
        const int64_t N = g.task_N[i];
        for (int64_t b = 0; b < g.task_B[i]; ++b, ++t) {
            tab[2 * t] = at;
            tab[2 * t + 1] = y;
            at += eor::n_tiles(N) * eor::TS2;
            y += N * eor::TS;
        }
        if (g.task_B[i] > 0)
            for (int64_t r = 0; r <= N; ++r) count[r] += (int32_t)g.task_B[i];
    }
    if (e == hipSuccess) e = g.spread_tab.ensure(tab.size());
    if (e == hipSuccess) e = hipMemcpy(g.spread_tab.p, tab.data(), tab.size() * sizeof(int64_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        g.spread_ready = true;
        return true;
    }
    (void)hipGetLastError();
    g.spread_y.release();
    g.prog.release();         // its words may not have been cleared
    g.est_spread = INFINITY;  // until the task list changes
    return false;
}

// Task list: every theta of every instance, longest first (cost ~ N^3), so
// that the persistent workgroups, taking tasks in order, approximate a
// longest-processing-time schedule.
eor_status build_tasks(eor_group &g, const int64_t *B) {
    const int n = (int)g.inst.size();
    std::vector<int64_t> want(B, B + n), rows(n);
    for (int i = 0; i < n; ++i) rows[i] = g.inst[i]->c.N;
    if (g.d_task && want == g.task_B && rows == g.task_N) return EOR_OK;
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int b) { return g.inst[a]->c.N > g.inst[b]->c.N; });
    int64_t total = 0;
    for (int64_t b : want) total += b;
    if (total > (int64_t)1 << 30) return eor::fail_status(EOR_ERR_ARG, "more than 2^30 theta in one group call");
    std::vector<int2> tasks;
    for (int i : order)
        for (int64_t b = 0; b < want[i]; ++b) tasks.push_back(make_int2(i, (int)b));
    // queued work may still read the current task list
    const hipError_t ed = g.order.drain();
    if (ed != hipSuccess) return eor::hip_status(ed, "hipEventSynchronize");
    free_tasks(g);
    g.ntask = (int64_t)tasks.size();
    g.task_B = want;
    g.task_N = rows;
    g.order_N = order;
    drop_graph(g);
    if (tasks.empty()) return EOR_OK;
    hipError_t e = hipMalloc(&g.d_task, tasks.size() * sizeof(int2));
    if (e == hipSuccess) e = hipMemcpy(g.d_task, tasks.data(), tasks.size() * sizeof(int2), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        free_tasks(g);
        return eor::hip_status(e, "task list");
    }
    plan_spread(g);
    return EOR_OK;
}

const char *const kBucketName[eor::N_BUCKETS] = {"n<=512", "n<=1024", "n<=2048", "n<=4096", "n>4096"};

std::string bucket_of(int64_t N) { return kBucketName[eor::bucket_index(N * eor::TS)]; }

std::string arch_name(int device) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return "unknown";
    std::string a = prop.gcnArchName;
    const size_t colon = a.find(':');
    return colon == std::string::npos ? a : a.substr(0, colon);
}

// Cache format: a JSON object of flat entries,
//   "<arch>|<bucket>|<kind>": {"stages": S, "wg_per_cu": W, "tiles": P, "ms": T}
//   "<arch>|<bucket>|tile": {"tile": 32 or 64, "ms64": T64, "ms32": T32}
// read as every "key": {...} pair in the file, whatever its line breaks.
std::map<std::string, std::string> read_cache(const char *path) {
    std::map<std::string, std::string> out;
    std::ifstream f(path);
    const std::string text((std::istreambuf_iterator<char>(f)), std::istreambuf_iterator<char>());
    size_t pos = 0;
    for (;;) {
        const size_t a = text.find('"', pos);
        const size_t b = a == std::string::npos ? a : text.find('"', a + 1);
        const size_t c = b == std::string::npos ? b : text.find_first_not_of(" \t\r\n:", b + 1);
        if (c == std::string::npos) break;
        if (text[c] != '{') {  // not an entry (e.g. a key inside a value): go on after it
            pos = b + 1;
            continue;
        }
        const size_t d = text.find('}', c);
        if (d == std::string::npos) break;
        out[text.substr(a + 1, b - a - 1)] = text.substr(c, d - c + 1);
        pos = d + 1;
    }
    return out;
}

bool parse_entry(const std::string &v, eor::Tuning &t) {
    int s = 0, w = 0, p = 0;
    double ms = 0.0;
    if (std::sscanf(v.c_str(), "{\"stages\": %d, \"wg_per_cu\": %d, \"tiles\": %d, \"ms\": %lf}", &s, &w, &p,
                    &ms) < 3)
        return false;
    if (!eor::valid_tuning(s, w, p)) return false;
    t.stages = s;
    t.wg_per_cu = w;
    t.tiles = p;
    return true;
}

bool write_cache(const char *path, const std::map<std::string, std::string> &m) {
    const std::string tmp = std::string(path) + ".tmp";
    {
        std::ofstream f(tmp);
        if (!f) return false;
        f << "{\n";
        size_t k = 0;
        for (const auto &kv : m) {
            f << "  \"" << kv.first << "\": " << kv.second << (++k < m.size() ? ",\n" : "\n");
        }
        f << "}\n";
        if (!f) return false;
    }
    return std::rename(tmp.c_str(), path) == 0;
}

eor::LikeParams make_params(const eor_group &g, const double *const *theta, double *const *logL,
                            int32_t *const *info) {
    eor::LikeParams p;
    std::memset(&p, 0, sizeof(p));
    p.inst = g.d_inst;
    p.task = g.d_task;
    p.ntask = g.ntask;
    p.counter = g.counter;
    p.Lw = g.Lw;
    p.slot_elems = g.slot_tiles * eor::TS2;
    p.yw = g.yw;
    p.slot_y = g.slot_y;
    for (size_t i = 0; i < g.inst.size(); ++i)
        p.call[i] = eor::CallDesc{theta[i], logL[i], info ? info[i] : nullptr, nullptr};
    return p;
}

eor::SpreadParams make_spread(const eor_group &g, const double *const *theta, double *const *logL,
                              int32_t *const *info) {
    eor::SpreadParams p;
    std::memset(&p, 0, sizeof(p));
    p.inst = g.d_inst;
    p.task = g.d_task;
    p.off = (const longlong2 *)g.spread_tab.p;
    p.count = (const int32_t *)(g.spread_tab.p + 2 * g.ntask);
    p.ntask = (int32_t)g.ntask;
    p.n_max = (int32_t)g.spread_rows;
    p.units = g.spread_units;
    p.per_cu = g.spread_per_cu;
    p.counter = g.counter;
    p.prog = g.prog.p;
    p.Lw = g.Lw;
    p.yw = g.spread_y.p;
    for (size_t i = 0; i < g.inst.size(); ++i)
        p.call[i] = eor::CallDesc{theta[i], logL[i], info ? info[i] : nullptr, nullptr};
    return p;
}

// Marks the end of a group call on s, for the group and for each instance
// (whose A the launch reads until then).
eor_status record_call(eor_group &g, hipStream_t s) {
    hipError_t e = g.order.leave(s);
    g.counter_clear = g.counter_clear || e == hipSuccess;
    for (size_t i = 0; i < g.inst.size() && e == hipSuccess; ++i) e = g.inst[i]->c.order.leave(s);
    return e == hipSuccess ? EOR_OK : eor::hip_status(e, "hipEventRecord");
}

// One launch of the whole group (eager or from the captured graph).
eor_status run_group(eor_group &g, const int64_t *B, const double *const *theta, double *const *logL,
                     int32_t *const *info, const eor::Tuning &t, bool allow_graph, bool allow_spread, hipStream_t s) {
    eor_status st = build_tasks(g, B);
    if (st != EOR_OK) return st;
    if (g.ntask == 0) return EOR_OK;
    int64_t N_max = 0;
    for (auto *c : g.inst) N_max = std::max<int64_t>(N_max, c->c.N);
    if (N_max != g.N_max) {
        free_work(g);
        g.N_max = N_max;
    }
    // The launch waits for the group's previous call and for each instance's
    // last call (a precompute that rewrote A) if they went to other streams.
    hipError_t e = g.order.enter(s);
    for (size_t i = 0; i < g.inst.size() && e == hipSuccess; ++i) e = g.inst[i]->c.order.enter(s);
    if (e != hipSuccess) return eor::hip_status(e, "hipStreamWaitEvent");
    // refresh the instance descriptors (a context may have been re-precomputed),
    // with the tile side of each instance's size bucket
    for (size_t i = 0; i < g.inst.size(); ++i) {
        g.h_inst[i] = eor::inst_desc(g.inst[i]->c);
        g.h_inst[i].ts = g.ts_bucket[eor::bucket_index(g.inst[i]->c.n)];
    }
    e = hipMemcpyAsync(g.d_inst, g.h_inst, g.inst.size() * sizeof(eor::InstDesc), hipMemcpyHostToDevice, s);
    if (e == hipSuccess && !g.counter_clear) e = hipMemsetAsync(g.counter, 0, sizeof(unsigned int), s);
    if (e != hipSuccess) return eor::hip_status(e, "instance descriptors");
    const int64_t resident = eor::resident_per_cu(t) * g.num_cu;
    const int64_t want = std::min<int64_t>(g.ntask, resident);
    st = ensure_work(g, want);
    if (st != EOR_OK) return st;
    const int64_t grid = std::min<int64_t>(want, g.slots);
    // Every theta spread over all workgroups, where that is sooner done, the
    // workspace of the resident workgroups holds every theta's L and the tiles
    // are 64-wide (32-wide ones sum in another order).
    bool spread = allow_spread && std::isfinite(g.est_spread) &&
                  g.spread_elems <= g.slots * g.slot_tiles * eor::TS2;
    for (size_t i = 0; i < g.inst.size(); ++i)
        spread = spread && (B[i] == 0 || g.h_inst[i].ts == eor::TS);
    spread = spread && ensure_spread(g);
    const eor::LikeParams p = make_params(g, theta, logL, info);
    const eor::SpreadParams sp = spread ? make_spread(g, theta, logL, info) : eor::SpreadParams();
    auto launch = [&](hipStream_t st) {
        return spread ? eor::launch_spread(sp, g.num_cu, st) : eor::launch_likelihood(p, t, grid, st);
    };
    if (!(allow_graph && g.use_graph)) {
        e = launch(s);
        if (e != hipSuccess) return eor::hip_status(e, "group launch");
        return record_call(g, s);
    }
    const bool same = g.exec && g.cap_grid == grid && g.cap_stages == t.stages && g.cap_tiles == t.tiles &&
                      g.cap_is_spread == spread && std::memcmp(&g.cap_params, &p, sizeof(p)) == 0 &&
                      (!spread || std::memcmp(&g.cap_spread, &sp, sizeof(sp)) == 0);
    if (!same) {
        drop_graph(g);
        if (!g.cap_stream) {
            e = hipStreamCreateWithFlags(&g.cap_stream, hipStreamNonBlocking);
            if (e != hipSuccess) return eor::hip_status(e, "capture stream");
        }
        e = hipStreamBeginCapture(g.cap_stream, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return eor::hip_status(e, "hipStreamBeginCapture");
        hipError_t el = launch(g.cap_stream);
        e = hipStreamEndCapture(g.cap_stream, &g.graph);
        if (el != hipSuccess) e = el;
        if (e == hipSuccess) e = hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            drop_graph(g);
            return eor::hip_status(e, "graph capture");
        }
        g.cap_params = p;
        if (spread) g.cap_spread = sp;
        g.cap_is_spread = spread;
        g.cap_grid = grid;
        g.cap_stages = t.stages;
        g.cap_tiles = t.tiles;
        ++g.captures;
    }
    e = hipGraphLaunch(g.exec, s);
    if (e != hipSuccess) return eor::hip_status(e, "hipGraphLaunch");
    ++g.replays;
    return record_call(g, s);
}

eor_status check_call(const eor_group *g, const int64_t *B, const double *const *theta, double *const *logL) {
    if (!g) return eor::fail_status(EOR_ERR_ARG, "group is NULL");
    if (!B || !theta || !logL) return eor::fail_status(EOR_ERR_ARG, "NULL argument array");
    for (size_t i = 0; i < g->inst.size(); ++i) {
        if (!g->inst[i]->c.ready) return eor::fail_status(EOR_ERR_STATE, "an instance has no precompute");
        if (B[i] < 0 || B[i] > (int64_t)INT32_MAX) return eor::fail_status(EOR_ERR_ARG, "B out of range");
        if (B[i] > 0 && ((!theta[i] && g->inst[i]->c.n_k > 0) || !logL[i]))
            return eor::fail_status(EOR_ERR_ARG, "NULL theta or logL for a non-empty instance");
    }
    return EOR_OK;
}

}  // namespace

extern "C" {

eor_status eor_group_create(int32_t n_inst, eor_ctx *const *insts, eor_group **out) {
    if (!out) return eor::fail_status(EOR_ERR_ARG, "eor_group_create: out is NULL");
    *out = nullptr;
    if (n_inst < 1 || n_inst > eor::MAX_INST || !insts)
        return eor::fail_status(EOR_ERR_ARG, "eor_group_create: need 1 <= n_inst <= 64 contexts");
    for (int i = 0; i < n_inst; ++i) {
        if (!insts[i]) return eor::fail_status(EOR_ERR_ARG, "eor_group_create: NULL context");
        if (insts[i]->c.device != insts[0]->c.device)
            return eor::fail_status(EOR_ERR_ARG, "eor_group_create: contexts on different devices");
    }
    eor_group *g = new (std::nothrow) eor_group;
    if (!g) return eor::fail_status(EOR_ERR_OOM, "eor_group_create: host allocation failed");
    g->device = insts[0]->c.device;
    g->num_cu = insts[0]->c.num_cu;
    g->inst.assign(insts, insts + n_inst);
    DeviceGuard dg(g->device);
    hipError_t e = hipMalloc(&g->d_inst, n_inst * sizeof(eor::InstDesc));
    if (e == hipSuccess) e = hipHostMalloc((void **)&g->h_inst, n_inst * sizeof(eor::InstDesc));
    if (e == hipSuccess) e = hipMalloc(&g->counter, sizeof(unsigned int));
    if (e != hipSuccess) {
        eor_group_destroy(g);
        return eor::hip_status(e, "eor_group_create");
    }
    *out = g;
    return EOR_OK;
}

void eor_group_destroy(eor_group *g) {
    if (!g) return;
    DeviceGuard dg(g->device);
    (void)hipDeviceSynchronize();
    free_work(*g);
    g->order.destroy();
    if (g->cap_stream) (void)hipStreamDestroy(g->cap_stream);
    if (g->d_inst) (void)hipFree(g->d_inst);
    if (g->h_inst) (void)hipHostFree(g->h_inst);
    free_tasks(*g);
    g->spread_tab.release();
    g->spread_y.release();
    g->prog.release();
    if (g->counter) (void)hipFree(g->counter);
    delete g;
}

eor_status eor_group_loglike(eor_group *g, const int64_t *B, const double *const *theta, double *const *logL,
                             int32_t *const *info, void *stream) {
    eor_status st = check_call(g, B, theta, logL);
    if (st != EOR_OK) return st;
    DeviceGuard dg(g->device);
    // The instance descriptors are staged in pinned memory: wait until the
    // previous launch of this group (on this stream or another) has copied
    // them.
    hipError_t e = g->order.drain();
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) return eor::hip_status(e, "hipStreamSynchronize");
    return run_group(*g, B, theta, logL, info, g->tune, true, true, (hipStream_t)stream);
}

eor_status eor_group_set_graph(eor_group *g, int32_t enable) {
    if (!g) return eor::fail_status(EOR_ERR_ARG, "eor_group_set_graph: group is NULL");
    g->use_graph = enable != 0;
    if (!g->use_graph) drop_graph(*g);
    return EOR_OK;
}

eor_status eor_group_set_tuning(eor_group *g, int32_t stages, int32_t wg_per_cu, int32_t tiles_per_pass) {
    if (!g) return eor::fail_status(EOR_ERR_ARG, "eor_group_set_tuning: group is NULL");
    if (!eor::valid_tuning(stages, wg_per_cu, tiles_per_pass))
        return eor::fail_status(EOR_ERR_ARG, "eor_group_set_tuning: need stages 2|4, and wg_per_cu 1|2 with "
                                             "tiles_per_pass 1, or wg_per_cu 1 with tiles_per_pass 2");
    g->tune.stages = stages;
    g->tune.wg_per_cu = wg_per_cu;
    g->tune.tiles = tiles_per_pass;
    return EOR_OK;
}

eor_status eor_group_set_tile_sizes(eor_group *g, const int32_t *ts_per_bucket) {
    if (!g || !ts_per_bucket) return eor::fail_status(EOR_ERR_ARG, "eor_group_set_tile_sizes: NULL argument");
    for (int b = 0; b < eor::N_BUCKETS; ++b)
        if (ts_per_bucket[b] != 32 && ts_per_bucket[b] != 64)
            return eor::fail_status(EOR_ERR_ARG, "eor_group_set_tile_sizes: each tile side is 32 or 64");
    for (int b = 0; b < eor::N_BUCKETS; ++b) g->ts_bucket[b] = ts_per_bucket[b];
    return EOR_OK;
}

eor_status eor_group_tile_sizes(const eor_group *g, int32_t *ts_per_bucket) {
    if (!g || !ts_per_bucket) return eor::fail_status(EOR_ERR_ARG, "eor_group_tile_sizes: NULL argument");
    for (int b = 0; b < eor::N_BUCKETS; ++b) ts_per_bucket[b] = g->ts_bucket[b];
    return EOR_OK;
}

eor_status eor_group_tuning(const eor_group *g, int32_t *stages, int32_t *wg_per_cu, int32_t *tiles_per_pass,
                            int64_t *graph_launches, int64_t *graph_captures) {
    if (!g) return eor::fail_status(EOR_ERR_ARG, "eor_group_tuning: group is NULL");
    if (stages) *stages = g->tune.stages;
    if (wg_per_cu) *wg_per_cu = g->tune.wg_per_cu;
    if (tiles_per_pass) *tiles_per_pass = g->tune.tiles;
    if (graph_launches) *graph_launches = g->replays;
    if (graph_captures) *graph_captures = g->captures;
    return EOR_OK;
}

eor_status eor_autotune(eor_group *g, const int64_t *B, const double *const *theta, const char *cache_path,
                        int32_t force, void *stream) {
    std::vector<double *> outs;
    {
        // validate with placeholder outputs
        std::vector<double *> fake(g ? g->inst.size() : 0, (double *)1);
        eor_status st = check_call(g, B, theta, fake.data());
        if (st != EOR_OK) return st;
    }
    DeviceGuard dg(g->device);
    hipStream_t s = (hipStream_t)stream;
    const int n_inst = (int)g->inst.size();
    int64_t N_max = 0;
    bool present[eor::N_BUCKETS] = {false, false, false, false, false};
    for (int i = 0; i < n_inst; ++i) {
        N_max = std::max<int64_t>(N_max, g->inst[i]->c.N);
        if (B[i] > 0) present[eor::bucket_index(g->inst[i]->c.n)] = true;
    }
    const std::string arch = arch_name(g->device);
    const std::string key = arch + "|" + bucket_of(N_max) + "|" + (n_inst == 1 ? "single" : "group");
    std::map<std::string, std::string> cache;
    if (cache_path) cache = read_cache(cache_path);
    // cached choices: the launch shape of this group's largest bucket, and
    // the tile side of each bucket it holds
    bool shape_known = false;
    if (!force && cache.count(key)) {
        eor::Tuning t;
        if (parse_entry(cache[key], t)) {
            g->tune = t;
            shape_known = true;
        }
    }
    bool tile_known[eor::N_BUCKETS] = {false, false, false, false, false};
    bool all_known = shape_known;
    for (int b = 0; b < eor::N_BUCKETS; ++b) {
        if (!present[b]) continue;
        const std::string tk = arch + "|" + kBucketName[b] + "|tile";
        int ts = 0;
        if (!force && cache.count(tk) && std::sscanf(cache[tk].c_str(), "{\"tile\": %d", &ts) == 1 &&
            (ts == 32 || ts == 64)) {
            g->ts_bucket[b] = ts;
            tile_known[b] = true;
        }
        all_known = all_known && tile_known[b];
    }
    if (all_known) return EOR_OK;
    // scratch outputs for the timing runs
    hipError_t e = g->order.drain();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return eor::hip_status(e, "hipStreamSynchronize");
    for (int i = 0; i < n_inst; ++i) {
        double *o = nullptr;
        e = hipMalloc(&o, std::max<int64_t>(B[i], 1) * sizeof(double));
        if (e != hipSuccess) {
            for (double *x : outs) (void)hipFree(x);
            return eor::hip_status(e, "autotune outputs");
        }
        outs.push_back(o);
    }
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    eor_status st = EOR_OK;
    // one warm-up launch, then the mean of two timed ones
    auto time_launch = [&](const int64_t *Bv, const eor::Tuning &t, bool spread) {
        st = run_group(*g, Bv, theta, outs.data(), nullptr, t, false, spread, s);
        float ms_sum = 0.f;
        for (int r = 0; r < 2 && st == EOR_OK; ++r) {
            (void)hipEventRecord(e0, s);
            st = run_group(*g, Bv, theta, outs.data(), nullptr, t, false, spread, s);
            (void)hipEventRecord(e1, s);
            if (hipEventSynchronize(e1) != hipSuccess) st = eor::fail_status(EOR_ERR_HIP, "autotune timing");
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            ms_sum += ms;
        }
        return ms_sum / 2.0;
    };
    if (!shape_known) {
        eor::Tuning best;
        double best_ms = 1e300;
        const int cand_stages[2] = {4, 2};
        const int cand_shape[3][2] = {{1, 2}, {1, 1}, {2, 1}};  // (tiles per pass, workgroups per CU)
        for (int a = 0; a < 2 && st == EOR_OK; ++a) {
            for (int b = 0; b < 3 && st == EOR_OK; ++b) {
                eor::Tuning t;
                t.stages = cand_stages[a];
                t.tiles = cand_shape[b][0];
                t.wg_per_cu = cand_shape[b][1];
                const double ms = time_launch(B, t, false);  // the shapes are those of one workgroup per theta
                if (st == EOR_OK && ms < best_ms) {
                    best_ms = ms;
                    best = t;
                }
            }
        }
        if (st == EOR_OK) {
            g->tune = best;
            std::ostringstream v;
            v << "{\"stages\": " << best.stages << ", \"wg_per_cu\": " << best.wg_per_cu << ", \"tiles\": "
              << best.tiles << ", \"ms\": " << best_ms << "}";
            cache[key] = v.str();
        }
    }
    // tile side per bucket, timed on that bucket's instances alone with the
    // chosen launch shape
    std::vector<int64_t> Bsub(n_inst);
    for (int b = 0; b < eor::N_BUCKETS && st == EOR_OK; ++b) {
        if (!present[b] || tile_known[b]) continue;
        for (int i = 0; i < n_inst; ++i) Bsub[i] = eor::bucket_index(g->inst[i]->c.n) == b ? B[i] : 0;
        double ms_ts[2] = {0.0, 0.0};
        const int cand_ts[2] = {64, 32};
        for (int c = 0; c < 2 && st == EOR_OK; ++c) {
            g->ts_bucket[b] = cand_ts[c];
            ms_ts[c] = time_launch(Bsub.data(), g->tune, true);
        }
        if (st != EOR_OK) break;
        g->ts_bucket[b] = ms_ts[1] < ms_ts[0] ? 32 : 64;
        std::ostringstream v;
        v << "{\"tile\": " << g->ts_bucket[b] << ", \"ms64\": " << ms_ts[0] << ", \"ms32\": " << ms_ts[1] << "}";
        cache[arch + "|" + kBucketName[b] + "|tile"] = v.str();
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    for (double *x : outs) (void)hipFree(x);
    if (st != EOR_OK) return st;
    drop_graph(*g);
    if (cache_path && !write_cache(cache_path, cache))
        return eor::fail_status(EOR_ERR_ARG, std::string("eor_autotune: cannot write ") + cache_path);
    return EOR_OK;
}

}  // extern "C"
