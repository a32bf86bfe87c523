// batch.hip -- formal solutions of many atmospheres and wavelength batches
// (the radiance-cascades formal solution of Osborne & Sannikov,
// arXiv:2408.14425, Secs. 2.3 and 3.2), batched.
//
// The whole sequence is captured into a HIP graph and replayed. Atmospheres
// share nothing, so they only meet at the end:
//  - those whose every cascade fills the GPU alone run through their plans'
//    own solve (the launches of rcx_formal_solve, with the plan's workspace),
//    one after another on the graph's main branch;
//  - those below about 256^2, whose launches last a few microseconds and
//    leave most of the chip idle, share launches: one per cascade for all of
//    them (march_table.h, k_march_tasks), in 16-lane batches;
//  - those between run through their plans on up to kSide further branches
//    beside the others.
// A graph branch costs about 30 us to fork and join here, so branches are
// taken only when the atmospheres on them hold at least kForkRays rays and
// wavelengths.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <fstream>
#include <new>
#include <sstream>
#include <string>
#include <vector>

#include "rcx_internal.h"

using namespace rcx;

namespace {
// Branches beside the main one. The box's processes get 4 hardware queues.
constexpr int kSide = 3;
// An atmosphere with a cascade of fewer rays does not fill the GPU alone.
constexpr int64_t kFillRays = 1 << 19;
constexpr int64_t kForkRays = 1 << 22;
}  // namespace

struct rcx_batch {
    int32_t n_atm = 0;
    bool f16 = false;
    std::vector<rcx_plan*> plans;
    std::vector<int32_t> n_wave;
    // 0 fills the GPU with every cascade, 1 runs beside the others, 2 shares
    // its launches with the others of its kind
    std::vector<char> kind;
    bool dirty = true;         // the shared tasks (below) are to be rebuilt
    void* tasks = nullptr;     // device
    size_t tasks_cap = 0;
    struct Step {
        int32_t t0, n;         // tasks
        uint32_t blocks;
        bool j;
    };
    std::vector<Step> steps;   // a launch per cascade (more where its grid would be too large), top first
    std::vector<float*> J_bound;
    int64_t n_march = 0;       // march launches the last solve enqueued
    // graph
    bool use_graph = true;
    hipStream_t cap = nullptr;  // capture stream (the legacy default stream cannot be captured)
    hipStream_t side[kSide] = {};
    hipEvent_t fork = nullptr, join[kSide] = {};
    hipGraphExec_t gexec = nullptr;
    std::vector<const float*> g_chi, g_eta;
    unsigned int* flag = nullptr;  // input check (RCX_FLAG_CHECK_INPUT)
    bool check_input = false;
};

namespace {

int32_t bfail(int32_t c, const std::string& m) { return rcx::fail(c, m); }

// Cascades whose launch order rcx_batch_set_order sets (the tiled ones).
constexpr int32_t kWideDirs = 256;

// The shared launches of the small atmospheres for the current J pointers;
// an atmosphere that cannot share moves to kind 1.
int32_t build_tasks(rcx_batch* s)
{
    const size_t bytes = table_task_bytes();
    std::vector<std::vector<TableLaunch>> by(s->n_atm);
    int32_t top = 0;
    for (int32_t a = 0; a < s->n_atm; ++a) {
        rcx_plan* P = s->plans[a];
        if (s->kind[a] == 0) continue;
        s->kind[a] = plan_table_tasks(P, s->n_wave[a], s->J_bound[a], by[a]) ? 2 : 1;
        if (s->kind[a] == 2) top = std::max(top, P->n_casc);
    }
    std::vector<char> host(bytes);
    auto task = [&](int32_t a, int32_t i, uint32_t block0, char* at) {
        const rcx_plan* P = s->plans[a];
        return table_task(P->levels[i], P->tables[i], P->grid.nx, P->grid.nz, by[a][i], block0, at);
    };
    // (a cascade that no launch holds)
    for (int32_t a = 0; a < s->n_atm; ++a)
        for (int32_t i = 0; s->kind[a] == 2 && i < s->plans[a]->n_casc; ++i)
            if (by[a][i].out && task(a, i, 0, host.data()) > kMaxGridX) s->kind[a] = 1;
    host.clear();
    s->steps.clear();
    for (int32_t i = top - 1; i >= 0; --i) {
        rcx_batch::Step step{0, 0, 0, i == 0};
        for (int32_t a = 0; a < s->n_atm; ++a) {
            if (s->kind[a] != 2 || i >= s->plans[a]->n_casc || !by[a][i].out) continue;
            host.resize(host.size() + bytes);
            char* at = host.data() + host.size() - bytes;
            uint64_t n = task(a, i, step.blocks, at);
            if (step.blocks + n > kMaxGridX) {  // the launch is full: the next one starts here
                s->steps.push_back(step);
                step.n = 0;
                step.blocks = 0;
                n = task(a, i, 0, at);
            }
            if (n == 0) {  // sparse with nothing flagged
                host.resize(host.size() - bytes);
                continue;
            }
            if (step.n++ == 0) step.t0 = (int32_t)(host.size() / bytes) - 1;
            step.blocks += (uint32_t)n;
        }
        if (step.n > 0) s->steps.push_back(step);
    }
    if (host.size() > s->tasks_cap) {
        if (s->tasks) (void)hipFree(s->tasks);
        s->tasks = nullptr;
        s->tasks_cap = 0;
        RCX_HIP_TRY(hipMalloc(&s->tasks, host.size()));
        s->tasks_cap = host.size();
    }
    if (!host.empty()) RCX_HIP_TRY(hipMemcpy(s->tasks, host.data(), host.size(), hipMemcpyHostToDevice));
    s->dirty = false;
    return RCX_OK;
}

// The small atmospheres: fields, then their cascades together.
int32_t enqueue_shared(rcx_batch* s, const float* const* chi, const float* const* eta, hipStream_t st)
{
    const size_t bytes = table_task_bytes();
    for (int32_t a = 0; a < s->n_atm; ++a) {
        if (s->kind[a] != 2) continue;
        const int32_t rc = plan_enqueue_prep(s->plans[a], s->n_wave[a], chi[a], eta[a], st);
        if (rc != RCX_OK) return rc;
    }
    for (const auto& step : s->steps) {
        RCX_HIP_TRY(launch_table_tasks((const char*)s->tasks + bytes * step.t0, step.n, step.blocks, step.j, s->f16, st));
        ++s->n_march;
    }
    for (int32_t a = 0; a < s->n_atm; ++a) {
        const rcx_plan* P = s->plans[a];
        if (s->kind[a] == 2 && P->mask_dev)
            RCX_HIP_TRY(launch_mask_j(s->J_bound[a], P->mask_dev, (int64_t)P->grid.nx * P->grid.nz, s->n_wave[a], st));
    }
    return RCX_OK;
}

// Enqueue one batch solve on st (no synchronisation); forked: with branches
// on the side streams (stream capture).
int32_t enqueue(rcx_batch* s, const float* const* chi, const float* const* eta, hipStream_t st, bool forked)
{
    s->n_march = 0;
    // what runs beside the main branch: the atmospheres of kind 1, and the
    // shared launches; the main branch takes a share when it has nothing else
    std::vector<int32_t> beside;
    int64_t rays = 0;
    bool any_large = false, any_shared = false;
    for (int32_t a = 0; a < s->n_atm; ++a) {
        const LevelDesc& L = s->plans[a]->levels[0];
        if (s->kind[a] == 0) any_large = true;
        else rays += (int64_t)L.px * L.pz * L.nd * s->n_wave[a];
        if (s->kind[a] == 1) beside.push_back(a);
        if (s->kind[a] == 2) any_shared = true;
    }
    const int32_t units = (int32_t)beside.size() + (any_shared ? 1 : 0);
    int32_t branches = std::min(kSide, any_large ? units : units - 1);
    if (!forked || rays < kForkRays || branches < 0) branches = 0;
    if (branches > 0) RCX_HIP_TRY(hipEventRecord(s->fork, st));
    for (int32_t b = 0; b < branches; ++b) RCX_HIP_TRY(hipStreamWaitEvent(s->side[b], s->fork, 0));
    const int32_t share = branches + (any_large && branches > 0 ? 0 : 1);
    int32_t k = 0;
    auto next = [&] {
        const int32_t b = k++ % share;
        return b < branches ? s->side[b] : st;
    };
    auto solve = [&](int32_t a, hipStream_t on) {
        int64_t n = 0;
        const int32_t rc = plan_enqueue_solve(s->plans[a], s->n_wave[a], chi[a], eta[a], s->J_bound[a], on, &n);
        s->n_march += n;
        return rc;
    };
    int32_t rc = RCX_OK;
    for (int32_t a = 0; a < s->n_atm && rc == RCX_OK; ++a)
        if (s->kind[a] == 0) rc = solve(a, st);
    for (size_t q = 0; q < beside.size() && rc == RCX_OK; ++q) rc = solve(beside[q], next());
    if (any_shared && rc == RCX_OK) rc = enqueue_shared(s, chi, eta, next());
    if (rc != RCX_OK) return rc;
    for (int32_t b = 0; b < branches; ++b) {
        RCX_HIP_TRY(hipEventRecord(s->join[b], s->side[b]));
        RCX_HIP_TRY(hipStreamWaitEvent(st, s->join[b], 0));
    }
    return RCX_OK;
}

// Solves run asynchronously: before the graph or a plan's lists change, the
// device must have finished any solve still reading them.
void drop_graph(rcx_batch* s)
{
    if (s->gexec) {
        (void)hipDeviceSynchronize();
        (void)hipGraphExecDestroy(s->gexec);
    }
    s->gexec = nullptr;
}

}  // namespace

extern "C" {

int32_t rcx_batch_create(int32_t n_atm, const rcx_grid* grids, const int32_t* n_wave, const rcx_params* p,
                         rcx_batch** out)
{
    if (out) *out = nullptr;
    if (n_atm < 1 || !grids || !n_wave || !p || !out) return bfail(RCX_E_INVALID, "rcx_batch_create: bad argument");
    if (p->c0_dirs != 4) return bfail(RCX_E_UNSUPPORTED, "rcx_batch_create: the fused J epilogue needs c0_dirs = 4");
    if (p->n_cascades != 0) return bfail(RCX_E_UNSUPPORTED, "rcx_batch_create: cascades are chosen per atmosphere");
    if (p->n_incl != 1) return bfail(RCX_E_UNSUPPORTED, "rcx_batch_create: flatland only (n_incl = 1)");
    if ((p->flags & ~RCX_FLAG_CHECK_INPUT) != 0)
        return bfail(RCX_E_UNSUPPORTED, "rcx_batch_create: only RCX_FLAG_CHECK_INPUT (basic merge only)");
    rcx_batch* s = new (std::nothrow) rcx_batch();
    if (!s) return bfail(RCX_E_NOMEM, "rcx_batch_create: host allocation");
    s->n_atm = n_atm;
    s->f16 = p->storage == RCX_STORE_F16_SCALED;
    s->check_input = (p->flags & RCX_FLAG_CHECK_INPUT) != 0;
    hipError_t e = hipSuccess;
    auto chk = [&](hipError_t r) {
        if (r != hipSuccess && e == hipSuccess) e = r;
    };
    for (int32_t a = 0; a < n_atm; ++a) {
        if (n_wave[a] < 1) {
            rcx_batch_destroy(s);
            return bfail(RCX_E_INVALID, "rcx_batch_create: n_wave must be positive");
        }
        rcx_plan* P = nullptr;
        rcx_params pa = *p;
        pa.flags &= ~RCX_FLAG_CHECK_INPUT;  // the batch checks its inputs itself
        int32_t rc = rcx_plan_create(&grids[a], &pa, n_wave[a], &P);
        if (rc != RCX_OK) {
            rcx_batch_destroy(s);
            return rc;
        }
        s->plans.push_back(P);
        s->n_wave.push_back(n_wave[a]);
        bool large = true;
        for (int32_t i = 0; i < P->n_casc; ++i) {
            if (P->top_skipped && i == P->n_casc - 1) continue;
            const LevelDesc& L = P->levels[i];
            if ((int64_t)L.px * L.pz * L.nd < kFillRays) large = false;
        }
        s->kind.push_back(large ? 0 : 1);
    }
    if (s->check_input) chk(hipMalloc(&s->flag, sizeof(unsigned int)));
    chk(hipStreamCreateWithFlags(&s->cap, hipStreamNonBlocking));
    chk(hipEventCreateWithFlags(&s->fork, hipEventDisableTiming));
    for (int b = 0; b < kSide; ++b) {
        chk(hipStreamCreateWithFlags(&s->side[b], hipStreamNonBlocking));
        chk(hipEventCreateWithFlags(&s->join[b], hipEventDisableTiming));
    }
    if (e != hipSuccess) {
        rcx_batch_destroy(s);
        return bfail(RCX_E_NOMEM, std::string("rcx_batch_create: hipMalloc: ") + hipGetErrorName(e));
    }
    *out = s;
    return RCX_OK;
}

int32_t rcx_batch_set_order(rcx_batch* s, int32_t tile_probes, int32_t tile_dirs)
{
    if (!s || tile_probes < 0 || tile_probes > 64) return bfail(RCX_E_INVALID, "rcx_batch_set_order: bad argument");
    RCX_HIP_TRY(hipDeviceSynchronize());  // a solve in flight reads the plans' lists
    for (rcx_plan* P : s->plans)
        for (int32_t i = 0; i < P->n_casc; ++i) {
            if (P->levels[i].nd < kWideDirs) continue;
            const int32_t rc =
                rcx_plan_set_order(P, i, tile_probes, tile_dirs, P->levels[i].xcd_chunk, P->levels[i].shared_walk);
            if (rc != RCX_OK) return rc;
        }
    drop_graph(s);
    s->dirty = true;
    return RCX_OK;
}

int32_t rcx_batch_set_active_host(rcx_batch* s, int32_t atm, const uint8_t* active_host)
{
    if (!s || atm < 0 || atm >= s->n_atm) return bfail(RCX_E_INVALID, "rcx_batch_set_active_host: bad argument");
    RCX_HIP_TRY(hipDeviceSynchronize());  // a solve in flight reads the plan's lists
    const int32_t rc = rcx_plan_set_active_host(s->plans[atm], active_host, nullptr);
    drop_graph(s);
    s->dirty = true;
    return rc;
}

int32_t rcx_batch_set_graph(rcx_batch* s, int32_t enable)
{
    if (!s) return bfail(RCX_E_INVALID, "rcx_batch_set_graph: null batch");
    s->use_graph = enable != 0;
    drop_graph(s);
    return RCX_OK;
}

int32_t rcx_batch_solve(rcx_batch* s, const float* const* chi_host, const float* const* eta_host, float* const* J_host,
                        hipStream_t st)
{
    if (!s || !chi_host || !eta_host || !J_host) return bfail(RCX_E_INVALID, "rcx_batch_solve: null argument");
    for (int32_t a = 0; a < s->n_atm; ++a)
        if (!chi_host[a] || !eta_host[a] || !J_host[a]) return bfail(RCX_E_INVALID, "rcx_batch_solve: null array");
    if (s->check_input) {
        // every atmosphere's chi and eta finite and non-negative (synchronises)
        RCX_HIP_TRY(launch_zero_flag(s->flag, st));
        for (int32_t a = 0; a < s->n_atm; ++a) {
            const int64_t n = (int64_t)s->n_wave[a] * s->plans[a]->grid.nx * s->plans[a]->grid.nz;
            RCX_HIP_TRY(launch_check_f32(chi_host[a], n, kCheckNonNegative, s->flag, st));
            RCX_HIP_TRY(launch_check_f32(eta_host[a], n, kCheckNonNegative, s->flag, st));
        }
        const int32_t rc = check_flag_result(s->flag, "rcx_batch_solve: chi or eta", st);
        if (rc != RCX_OK) return rc;
    }
    const bool same_J = (int32_t)s->J_bound.size() == s->n_atm &&
                        std::equal(s->J_bound.begin(), s->J_bound.end(), J_host);
    const bool same_in = s->gexec && std::equal(s->g_chi.begin(), s->g_chi.end(), chi_host) &&
                         std::equal(s->g_eta.begin(), s->g_eta.end(), eta_host);
    if (s->dirty || !same_J || (s->use_graph && !same_in)) {
        // the tasks or the graph change: a solve still in flight reads them,
        // so it must end first
        RCX_HIP_TRY(hipStreamSynchronize(st));
        drop_graph(s);
        s->J_bound.assign(J_host, J_host + s->n_atm);
        if (s->dirty || !same_J) {
            s->dirty = true;
            int32_t rc;
            try {
                rc = build_tasks(s);
            } catch (const std::bad_alloc&) {
                rc = bfail(RCX_E_NOMEM, "rcx_batch_solve: host allocation");
            }
            if (rc != RCX_OK) return rc;
        }
    }
    if (s->use_graph) {
        if (!s->gexec) {
            hipGraph_t g = nullptr;
            RCX_HIP_TRY(hipStreamBeginCapture(s->cap, hipStreamCaptureModeThreadLocal));
            const int32_t rc = enqueue(s, chi_host, eta_host, s->cap, true);
            hipError_t e = hipStreamEndCapture(s->cap, &g);
            if (rc != RCX_OK) {
                if (g) (void)hipGraphDestroy(g);
                return rc;
            }
            RCX_HIP_TRY(e);
            e = hipGraphInstantiate(&s->gexec, g, nullptr, nullptr, 0);
            (void)hipGraphDestroy(g);
            RCX_HIP_TRY(e);
            s->g_chi.assign(chi_host, chi_host + s->n_atm);
            s->g_eta.assign(eta_host, eta_host + s->n_atm);
        }
        RCX_HIP_TRY(hipGraphLaunch(s->gexec, st));
    } else {
        return enqueue(s, chi_host, eta_host, st, false);
    }
    return RCX_OK;
}

int32_t rcx_batch_work(const rcx_batch* s, int64_t* rays_nonempty_host, int64_t* cell_steps_host)
{
    if (!s || !rays_nonempty_host || !cell_steps_host) return bfail(RCX_E_INVALID, "rcx_batch_work: null argument");
    int64_t r = 0, c = 0;
    for (int32_t a = 0; a < s->n_atm; ++a) {
        rcx_work w;
        int32_t rc = rcx_plan_work(s->plans[a], &w);
        if (rc != RCX_OK) return rc;
        r += w.rays_nonempty * s->n_wave[a];
        c += w.cell_steps * s->n_wave[a];
    }
    *rays_nonempty_host = r;
    *cell_steps_host = c;
    return RCX_OK;
}

int32_t rcx_batch_launches(const rcx_batch* s, int32_t* march_host, int32_t* all_host)
{
    if (!s || !march_host || !all_host) return bfail(RCX_E_INVALID, "rcx_batch_launches: null argument");
    const int32_t march = (int32_t)s->n_march;
    int32_t other = 0;
    if (march > 0)
        for (int32_t a = 0; a < s->n_atm; ++a) {
            other += 1 + (s->f16 ? 1 : 0);              // field prep (+ exponent bias)
            if (s->plans[a]->mask_dev) other += 2;      // masked fields, masked J
        }
    *march_host = march;
    *all_host = march + other;
    return RCX_OK;
}

int32_t rcx_batch_autotune(rcx_batch* s, const float* const* chi, const float* const* eta, float* const* J,
                           const char* cache_path, int32_t* best_rays_host, hipStream_t st)
{
    if (!s || !chi || !eta || !J || !best_rays_host) return bfail(RCX_E_INVALID, "rcx_batch_autotune: null argument");
    // cache key: the device, the march the orders are tuned on, the cascade
    // intervals and the batch's shapes
    int dev = 0;
    RCX_HIP_TRY(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    RCX_HIP_TRY(hipGetDeviceProperties(&prop, dev));
    bool tables = true;
    for (const rcx_plan* P : s->plans) tables = tables && P->table_mem;
    const rcx_params& prm = s->plans[0]->prm;
    std::ostringstream key;
    key << prop.gcnArchName << "_" << prop.multiProcessorCount << "cu_" << (tables ? "table" : "walk") << "_t"
        << prm.c0_t1 << "_r" << prm.t_rule << "_" << (s->f16 ? "f16" : "f32");
    for (int32_t a = 0; a < s->n_atm; ++a)
        if (s->plans[a]->mask_dev) key << "_sparse" << a << "_" << s->plans[a]->levels[0].n_active;
    for (int32_t a = 0; a < s->n_atm; ++a)
        key << "_" << s->plans[a]->grid.nx << "x" << s->plans[a]->grid.nz << "w" << s->n_wave[a];
    const std::string k = key.str();
    if (cache_path) {
        std::ifstream f(cache_path);
        std::string line;
        while (std::getline(f, line)) {
            const std::string pre = "\"" + k + "\": ";
            const size_t pos = line.find(pre);
            if (pos != std::string::npos) {
                const int32_t r = std::atoi(line.c_str() + pos + pre.size());
                if (r >= 0 && r <= 64064) {
                    *best_rays_host = r;
                    return rcx_batch_set_order(s, r / 1000, r % 1000);
                }
            }
        }
    }
    // candidate (tile_probes, tile_dirs), coded tile_probes * 1000 + tile_dirs
    const int32_t cands[] = {0, 2032, 4016, 4032, 4064, 8032};
    double best_ms = 1e300;
    int32_t best = cands[0];
    const bool g = s->use_graph;
    s->use_graph = false;
    for (int32_t cnd : cands) {
        int32_t rc = rcx_batch_set_order(s, cnd / 1000, cnd % 1000);
        if (rc != RCX_OK) return rc;
        rc = rcx_batch_solve(s, chi, eta, J, st);  // warm-up and work-list build
        if (rc != RCX_OK) return rc;
        RCX_HIP_TRY(hipStreamSynchronize(st));
        const auto t0 = std::chrono::steady_clock::now();
        rc = rcx_batch_solve(s, chi, eta, J, st);
        if (rc != RCX_OK) return rc;
        RCX_HIP_TRY(hipStreamSynchronize(st));
        const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        if (ms < best_ms) {
            best_ms = ms;
            best = cnd;
        }
    }
    s->use_graph = g;
    if (cache_path) {
        std::ofstream f(cache_path, std::ios::app);
        f << "{\"" << k << "\": " << best << ", \"ms\": " << best_ms << "}\n";
    }
    *best_rays_host = best;
    return rcx_batch_set_order(s, best / 1000, best % 1000);
}

int32_t rcx_batch_destroy(rcx_batch* s)
{
    if (!s) return RCX_OK;
    drop_graph(s);
    if (s->flag) (void)hipFree(s->flag);
    if (s->tasks) (void)hipFree(s->tasks);
    for (rcx_plan* P : s->plans) rcx_plan_destroy(P);
    if (s->cap) (void)hipStreamDestroy(s->cap);
    if (s->fork) (void)hipEventDestroy(s->fork);
    for (int b = 0; b < kSide; ++b) {
        if (s->side[b]) (void)hipStreamDestroy(s->side[b]);
        if (s->join[b]) (void)hipEventDestroy(s->join[b]);
    }
    delete s;
    return RCX_OK;
}

}  // extern "C"
