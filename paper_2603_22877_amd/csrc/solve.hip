// Batched annealed solver (Alg. "CLS with Annealing" around the PGD loop of Alg.
// "FourierSMT"), fused on the device.
//
// Persistent schedule: one workgroup per (instance, restart). The restart's relaxed state
// (a, b), its gradient and the projection work arrays stay in LDS for the whole launch, so
// the gradient scatter uses LDS atomics and no global atomic is issued. Per PGD step the
// workgroup's waves sweep the instance's constraint buckets (lane = constraint, uniform
// diagram shape per wave), then project (clamp a; box + unit atoms for b), and reduce the
// gradient map norm. At the end of each level the workgroup rounds, checks every
// constraint exactly, updates the ERWA history and weights of its restart (plain loads and
// stores: the workgroup owns the row), and stops once no constraint is violated.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "eval_task.hpp"
#include "solve_grid.hpp"
#include "solve_wg.hpp"

namespace fsmt {

static fsmt_status launch_status(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(FSMT_EHIP, "%s: %s", what, hipGetErrorString(e));
    return FSMT_OK;
}

// The persistent solver kernel for a message variant, cluster mode, closed-form level and
// gradient type.
static const void *solve_kernel_fn(int msg, bool cl, int cf, bool wide) {
    return cf == 0 ? solve_kernel_cf0(msg, cl, wide)
           : cf == 1 ? solve_kernel_cf1(msg, cl, wide)
           : cf == 2 ? solve_kernel_cf2(msg, cl, wide)
           : cf == 3 ? solve_kernel_cf3(msg, cl, wide)
                     : solve_kernel_cf4(msg, cl, wide);
}

// Dynamic LDS a persistent workgroup may take.
static std::vector<const void *> solve_fns() {
    std::vector<const void *> fns;
    for (int msg : {kMsgLds, kMsgSmall, kMsgMedium, kMsgLarge})
        for (int cl = 0; cl < 2; ++cl)
            for (int cf = 0; cf < 5; ++cf)
                for (int wide = 0; wide < 2; ++wide) fns.push_back(solve_kernel_fn(msg, cl != 0, cf, wide != 0));
    return fns;
}
static size_t lds_budget(int device) {
    static LdsBudget B;
    return B.of(device, solve_fns);
}

static int solve_waves(int msg, int cf) {
    if (msg == kMsgMedium) return SolveWaves<kMsgMedium, 0>::value;
    if (msg == kMsgLarge) return SolveWaves<kMsgLarge, 0>::value;
    return cf == 2 || cf == 3 ? SolveWaves<kMsgSmall, 2>::value : SolveWaves<kMsgSmall, 0>::value;
}

static size_t state_floats_of(const fsmt_xbdd *h, bool wide = false) {
    return wide ? solve_state_floats<double>(h->n_bool, h->n_real, h->n_hs, h->hs_nnz)
                : solve_state_floats<float>(h->n_bool, h->n_real, h->n_hs, h->hs_nnz);
}

// ---- per-device resources kept for the life of the process
// A stream for the grid part of a mixed batch, a stream to capture level graphs on, the
// fork/join events, and instantiated level graphs waiting for their last launch to finish
// before they are destroyed (checked without blocking at the next call).
struct DeviceRes {
    bool init = false;
    hipStream_t fork = nullptr, cap = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    std::vector<GraphRetired> retired;
};
static std::mutex g_res_mutex;
static DeviceRes g_res[kMaxDevices];

// Called with g_res_mutex held and `device` current.
static fsmt_status device_res(int device, DeviceRes **out) {
    if (device < 0 || device >= kMaxDevices) return set_error(FSMT_EINVAL, "device %d out of range", device);
    DeviceRes &R = g_res[device];
    if (!R.init) {
        if (hipStreamCreateWithFlags(&R.fork, hipStreamNonBlocking) != hipSuccess ||
            hipStreamCreateWithFlags(&R.cap, hipStreamNonBlocking) != hipSuccess ||
            hipEventCreateWithFlags(&R.ev_fork, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&R.ev_join, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            return set_error(FSMT_EHIP, "solver stream / event creation failed on device %d", device);
        }
        R.init = true;
    }
    reap_retired(R.retired);
    *out = &R;
    return FSMT_OK;
}

// Device memory of one call: either allocated stream-ordered on the call's stream (and
// freed the same way after the kernels), or carved from a fixed buffer (the allocation-free
// entry point).
struct CallScratch {
    char *fixed = nullptr;     // base of the fixed buffer, or null
    size_t cap = 0, used = 0;
    fsmt_status get(size_t bytes, hipStream_t st, void **out) {
        bytes = (bytes + 255) / 256 * 256;
        if (fixed) {
            if (used + bytes > cap)
                return set_error(FSMT_ELIMIT, "the call needs more than the %zu bytes of the fixed solver scratch", cap);
            *out = fixed + used;
            used += bytes;
            return FSMT_OK;
        }
        if (hipMallocAsync(out, bytes, st) != hipSuccess) {
            (void)hipGetLastError();
            return set_error(FSMT_ENOMEM, "solver scratch allocation (%zu bytes) failed", bytes);
        }
        return FSMT_OK;
    }
    void put(void *p, hipStream_t st) const {
        if (!fixed && p) (void)hipFreeAsync(p, st);
    }
};

}  // namespace fsmt

using namespace fsmt;

// Modelled us of one iteration's sweep and exchange with k workgroups per restart, of total_r in the
// launch: rounds of `waves` tasks (tiles 1.9 us a round, of clause pairs 1 us, bucket tasks 3.2 us,
// 3 us and 0.45 us a node where node-by-node templates are among them), and for k > 1 the exchange of k partial
// gradients through the coherence point, which all restarts share.
// Measured (8 restarts, us per iteration at k = 1, 2, 4, 8, 16): placement 75 10.9, 11.5, 10.6,
// 12.4, 15.0; 150 27.3, 19.4, 14.8, 15.3, 16.1; 300 93.9, 53.7, 32.0, 23.5, 21.1; scheduling
// 200 x 10 9.4, 11.5, 12.2, 15.8, 21.1; 400 x 10 17.9, 17.5, 18.7, 23.6, 31.8. The same, 1 / 16
// restarts: 4,000 clauses node by node 39.9, 25.0, 17.2, 15.0, 15.9 / 40.5, 25.6, 19.4, 19.0, 25.8;
// 400 short parities 39.0, 26.4, 18.7, 15.7, 15.2 / 39.7, 26.8, 20.2, 19.3, 23.5; placement 150 node
// by node, 16 restarts 260, 139, 76, 47, 41.
static double cluster_us(const fsmt_xbdd *h, int waves, int64_t total_r, int k) {
    const double bucket = h->small_max_nodes > 0 ? 3.0 + 0.45 * std::min(h->small_max_nodes, 20) : 3.2, tile = h->tile_kinds == kTileClauses ? 1.0 : 1.9;
    const double tasks = (double)sweep_tasks(h);
    const double round = tasks > 0.0 ? ((double)(h->n_pos / 64) * bucket + (double)h->n_tiles * tile) / tasks : 0.0;
    const double exchange = 2.5 + 0.25 * k + 2e-4 * k * ((double)h->n_bool + h->n_real) + 0.006 * (double)total_r * k * std::sqrt((double)k);
    return std::ceil(tasks / ((double)waves * k)) * round + (k > 1 ? exchange : 0.0);
}

// Workgroups per restart: the power of two with the smallest modelled iteration (of the slowest
// instance) that keeps every workgroup resident.
static int best_cluster(const fsmt_xbdd *const *insts, const std::vector<int> &ids, int waves, int64_t total_r,
                        int64_t resident) {
    int best_k = 1;
    double best = 0.0;
    for (int k = 1; k <= 16 && (k == 1 || total_r * k <= resident); k *= 2) {
        double t = 0.0;
        for (int i : ids) t = std::max(t, cluster_us(insts[i], waves, total_r, k));
        if (k == 1 || t < best) {
            best = t;
            best_k = k;
        }
    }
    return best_k;
}

// Schedule choice per instance (cost model in units of one wave task): the persistent
// schedule needs the restart's state in LDS and costs ceil(tasks / waves) sequential tasks
// per step on one CU; the grid schedule spreads tasks x restarts over all CUs (about 8 waves
// each) and pays two launches per step (about 20 task-times).
static bool prefer_grid(const fsmt_xbdd *h, int R, int64_t R_batch, int waves_a, int n_cu) {
    // persistent: a restart's tasks over its cluster of k workgroups (the launch's own choice,
    // with a workgroup a CU), plus the exchange of k partial gradients per step
    const double tasks_a = (double)sweep_tasks(h);                   // per restart, lane = constraint
    const int wa = std::max(1, waves_a);
    const int k = best_cluster(&h, {0}, wa, R_batch, n_cu);
    const double exchange = k > 1 ? 4.0 + (double)(h->n_bool + h->n_real) * k / (wa * 64.0 * 16.0) : 0.0;
    const double t_a = std::ceil(tasks_a / (wa * k)) + exchange;
    // grid: every (constraint, restart) lane over the device, as many waves per CU as the
    // message store's registers allow, plus the launches of a step
    int rp = 1;
    while (rp < R && rp < 64) rp <<= 1;
    const double lanes = (double)h->n_pos * (R <= 64 ? rp : std::ceil(R / 64.0) * 64.0) + 64.0 * h->n_tiles * R;
    const double t_b = std::ceil(lanes / 64.0 / ((double)wa * n_cu)) + 20.0;
    return t_b < t_a;
}

// Workgroups per restart of the grid schedule's workgroup sweep, or 0 where it does not apply
// (node-by-node templates, an atom without an inline record (its kernel has the register store,
// without the path through the atom table), a real state beyond the LDS): about two workgroups a
// CU over the whole call, each with at least two tasks a wave; up to 24 with a task for half of
// their waves where the bucket tasks' rounds are long (4,000 three-literal clauses of 153 shapes,
// one restart, 20 steps: 550 us with five slices, 385 with 22). More cost the step kernel, which
// adds their rows (600 rectangles, one restart: 1.06 ms with 90 slices, 2.26 with 340; 150
// rectangles, 16 restarts: 0.49 with 6, 0.77 with 24). `work`: tasks x restarts of the call.
static int grid_slices(const fsmt_xbdd *h, int R, int64_t work, size_t budget, int n_cu) {
    const int64_t tasks = sweep_tasks(h);
    const size_t lds = (size_t)h->n_real * 12;
    if (h->small_max_nodes > 0 || h->n_big > 0 || tasks == 0 || h->n_real == 0 || closed_level(h) < 1 ||
        !h->all_inline || lds > std::min<size_t>(budget, 60000))
        return 0;
    const int64_t ideal = std::max<int64_t>(1, work / (2 * n_cu));   // tasks of one workgroup
    const bool buckets = sweep_us(h, 16) - sweep_us(h, 16, true) > kSweepUsMin;
    const int64_t most = buckets ? std::max(tasks / 32, std::min<int64_t>(24, tasks / 8)) : tasks / 32;
    const int64_t s = std::max<int64_t>(1, std::min((tasks + ideal - 1) / ideal, most));
    return (int)std::min<int64_t>(s, INT32_MAX / std::max(1, R));
}

// Geometry of one persistent launch over a set of instances.
struct PersistentGeom {
    int msg = kMsgSmall, waves = 0, maxn = 0, maxs = 1;
    size_t state_f = 0, wave_bytes = 0, lds = 0;
    int cf = 0;
    bool wide = false;   // gradient sums in double
};

static PersistentGeom persistent_geom(const fsmt_xbdd *const *insts, const std::vector<int> &ids, size_t budget) {
    PersistentGeom G;
    bool lds_only = false, all_inline = true;
    size_t wide_f = 0;
    for (int i : ids) {
        const fsmt_xbdd *h = insts[i];
        G.state_f = std::max(G.state_f, state_floats_of(h));
        wide_f = std::max(wide_f, state_floats_of(h, true));
        G.maxn = std::max(G.maxn, h->small_max_nodes);
        G.maxs = std::max(G.maxs, h->small_max_slots);
        lds_only = lds_only || lds_store(h);
        all_inline = all_inline && h->all_inline;
        G.cf = closed_level_of(G.cf, closed_level(h));
    }
    G.msg = msg_variant(G.maxn, G.maxs, lds_only, all_inline);
    G.wave_bytes = G.msg == kMsgLds ? WaveScratch::bytes(G.maxn + 2, G.maxs) : 0;
    auto waves_of = [&](size_t state_f) -> int {
        const size_t state_bytes = state_f * sizeof(float);
        if (state_bytes > budget) return 0;
        if (!G.wave_bytes) return solve_waves(G.msg, G.cf);
        return (int)std::min<size_t>(solve_waves(G.msg, G.cf), (budget - state_bytes) / G.wave_bytes);
    };
    // the double gradient wherever it leaves the workgroup at least half of its waves (a
    // wave-wide LDS add takes 9 cycles in double and 193 in float)
    G.waves = waves_of(G.state_f);
    const int wide_waves = waves_of(wide_f);
    if (wide_waves > 0 && 2 * wide_waves >= G.waves) {
        G.wide = true;
        G.waves = wide_waves;
        G.state_f = wide_f;
    }
    G.lds = G.state_f * sizeof(float) + (size_t)G.waves * G.wave_bytes;
    return G;
}

namespace fsmt {

fsmt_status solve_impl(const fsmt_xbdd *const *insts, int32_t n_inst, const fsmt_solve_opts *opts,
                       const fsmt_solve_state *states, void *stream, void *fixed, size_t fixed_cap) {
    const bool fixed_scratch = fixed != nullptr;
    clear_error();
    if (!insts || !opts || !states || n_inst <= 0) return set_error(FSMT_EINVAL, "null argument or no instance");
    const fsmt_solve_opts &O = *opts;
    if (O.n_levels < 0 || O.n_levels > kMaxLevels) return set_error(FSMT_ELIMIT, "n_levels must be in [0, %d]", kMaxLevels);
    if (O.n_levels > 0 && !O.kappas) return set_error(FSMT_EINVAL, "kappas is NULL");
    if (O.steps_per_level < 0) return set_error(FSMT_EINVAL, "steps_per_level < 0");
    if (!(O.eta_a > 0.0f) || !(O.eta_b > 0.0f)) return set_error(FSMT_EINVAL, "step sizes must be positive");
    if (O.tau < 1) return set_error(FSMT_EINVAL, "tau must be >= 1");
    if (!(O.gamma > 0.0f) || !(O.rho >= 0.0f)) return set_error(FSMT_EINVAL, "bad ERWA parameters");
    if (O.schedule < 0 || O.schedule > 2) return set_error(FSMT_EINVAL, "schedule %d unknown", O.schedule);
    if (O.stop_on_sat < 0 || O.stop_on_sat > 2) return set_error(FSMT_EINVAL, "stop_on_sat must be 0, 1 or 2");
    if (O.level_begin < 0) return set_error(FSMT_EINVAL, "level_begin < 0");
    if (O.spin_limit < 0) return set_error(FSMT_EINVAL, "spin_limit < 0");
    if (fixed_scratch && O.schedule == 2) return set_error(FSMT_EUNSUPPORTED, "the allocation-free call runs the persistent schedule only");
    for (int t = 0; t < O.n_levels; ++t)
        if (!(O.kappas[t] >= 0.0)) return set_error(FSMT_EINVAL, "kappa[%d] must be in [0, +inf]", t);

    // ---- validate states, collect shapes
    int device = -1;
    fsmt_status rc;
    for (int i = 0; i < n_inst; ++i) {
        const fsmt_xbdd *h = insts[i];
        const fsmt_solve_state &S = states[i];
        if (!h) return set_error(FSMT_EINVAL, "instance %d: null handle", i);
        if ((rc = select_device(h))) return rc;
        if (device >= 0 && h->device != device) return set_error(FSMT_EINVAL, "instances on different devices");
        device = h->device;
        const int R = S.a.rows;
        if (R <= 0) return set_error(FSMT_EINVAL, "instance %d: no restarts", i);
        if (S.a.cols != h->n_bool || S.b.rows != R || S.b.cols != h->n_real)
            return set_error(FSMT_EINVAL, "instance %d: state shape does not match the instance", i);
        if ((h->n_bool > 1 && S.a.stride_v != 1) || (h->n_real > 1 && S.b.stride_v != 1) ||
            (R > 1 && ((h->n_bool > 0 && S.a.stride_r < h->n_bool) || (h->n_real > 0 && S.b.stride_r < h->n_real))))
            return set_error(FSMT_EINVAL, "instance %d: a and b must be row-major [R][n] with unit column stride", i);
        const void *ptrs[] = {h->n_bool ? S.a.data : nullptr, h->n_real ? S.b.data : nullptr, S.w, S.hist,
                              S.sat_bits, S.n_unsat, S.verdict, S.level_done, S.steps_done, S.obj, S.grad_a, S.grad_b};
        for (int q = 0; q < 12; ++q) {
            if (!ptrs[q] && q >= 2 && q < 10) return set_error(FSMT_EINVAL, "instance %d: state pointer %d is NULL", i, q);
            if ((rc = check_device_ptr(ptrs[q], h->device, "state"))) return rc;
        }
    }

    // the device's streams, events and retired graphs serve the grid schedule and mixed
    // batches; the allocation-free call runs neither and creates nothing
    std::lock_guard<std::mutex> lock(g_res_mutex);
    DeviceRes *res = nullptr;
    if (!fixed_scratch && (rc = device_res(device, &res))) return rc;
    CallScratch mem;
    mem.fixed = (char *)fixed;
    mem.cap = fixed_cap;

    // ---- schedule choice per instance
    const size_t budget = lds_budget(device);
    int n_cu = 256;
    (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device);
    std::vector<char> use_grid(n_inst, 0);
    int64_t r_batch = 0;
    for (int i = 0; i < n_inst; ++i) r_batch += states[i].a.rows;
    for (int i = 0; i < n_inst; ++i) {
        const fsmt_xbdd *h = insts[i];
        const PersistentGeom G = persistent_geom(insts, std::vector<int>{i}, budget);
        const bool fits = G.waves > 0;
        // the instance's schedule: its entry of inst_schedule if set, else the call's
        const int sched = (O.inst_schedule && O.inst_schedule[i] != 0) ? O.inst_schedule[i] : O.schedule;
        if (sched < 0 || sched > 2) return set_error(FSMT_EINVAL, "instance %d: schedule %d unknown", i, sched);
        if (fixed_scratch && sched == 2)
            return set_error(FSMT_EUNSUPPORTED, "the allocation-free call runs the persistent schedule only");
        if ((sched == 1 || fixed_scratch) && !fits)
            return set_error(FSMT_EUNSUPPORTED, "instance %d: restart state (%zu B) does not fit the persistent "
                             "schedule's LDS (%zu B)", i, G.state_f * sizeof(float), budget);
        // big diagrams are evaluated level by level by their own kernel, in the grid schedule
        if ((sched == 1 || fixed_scratch) && h->n_big > 0)
            return set_error(FSMT_EUNSUPPORTED, "instance %d: %d big diagrams need the grid schedule", i, h->n_big);
        use_grid[i] = sched == 2 || !fits || h->n_big > 0 ||
                      (sched == 0 && !fixed_scratch && prefer_grid(h, states[i].a.rows, r_batch, G.waves, n_cu));
    }
    std::vector<int> ia, ib;
    for (int i = 0; i < n_inst; ++i) (use_grid[i] ? ib : ia).push_back(i);
    // the persistent launch takes the largest state and message store of its instances: while
    // that leaves no room for a wave, the instance with the largest state goes to the grid
    // schedule (the persistent schedule only when it was asked for)
    PersistentGeom G;
    while (!ia.empty()) {
        G = persistent_geom(insts, ia, budget);
        if (G.waves > 0) break;
        bool forced = O.schedule == 1 || fixed_scratch;
        for (int i : ia) forced = forced || (O.inst_schedule && O.inst_schedule[i] == 1);
        if (forced)
            return set_error(FSMT_EUNSUPPORTED, "the instances' combined restart state and message store do not fit "
                             "one persistent workgroup's LDS (%zu B)", budget);
        auto big = std::max_element(ia.begin(), ia.end(), [&](int x, int y) {
            return state_floats_of(insts[x]) < state_floats_of(insts[y]);
        });
        ib.push_back(*big);
        ia.erase(big);
    }
    std::sort(ib.begin(), ib.end());

    hipStream_t st = (hipStream_t)stream;
    // the grid part runs on the device's fork stream, concurrently with the persistent launch
    hipStream_t gst = st;
    if (!ia.empty() && !ib.empty()) {
        gst = res->fork;
        if (hipEventRecord(res->ev_fork, st) != hipSuccess || hipStreamWaitEvent(gst, res->ev_fork, 0) != hipSuccess) {
            (void)hipGetLastError();
            return set_error(FSMT_EHIP, "stream fork failed");
        }
    }

    rc = FSMT_OK;
    // ---- persistent schedule
    if (!ia.empty()) {
        SolveParams P{};
        P.n_inst = (int)ia.size();
        P.n_levels = O.n_levels;
        P.steps = O.steps_per_level;
        P.tau = O.tau;
        P.normalize = O.normalize ? 1 : 0;
        P.stop_mode = O.stop_on_sat;
        P.eta_a = O.eta_a;
        P.eta_b = O.eta_b;
        P.eps2 = O.eps > 0.0f ? O.eps * O.eps : -1.0f;
        P.rho = O.rho;
        P.gamma = O.gamma;
        P.spin_limit = O.spin_limit > 0 ? (uint32_t)O.spin_limit : kSpinLimit;
        for (int t = 0; t < O.n_levels; ++t) P.kappas[t] = O.kappas[t];
        std::vector<InstDesc> desc(ia.size());
        int64_t total_r = 0, part_floats = 0;
        for (int i : ia) total_r += states[i].a.rows;
        const int msg = G.msg, waves = G.waves;
        const size_t lds = G.lds;
        auto kernel_of = [&](bool cl) -> const void * { return solve_kernel_fn(msg, cl, G.cf, G.wide); };
        auto resident_of = [&](bool cl) -> int64_t {
            int occ = 1;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel_of(cl), 64 * waves, lds) != hipSuccess) {
                (void)hipGetLastError();
                occ = 1;
            }
            return (int64_t)n_cu * std::max(occ, 1);
        };
        // workgroups per restart: a cluster of k co-resident workgroups shares one restart's
        // sweep (all of them must be resident at once: their barrier waits for each other)
        int k = 1;
        if (O.cluster > 0) {
            k = O.cluster;
            if (k > 16 || (k > 1 && (total_r * k > resident_of(true) || !ib.empty())))
                return set_error(FSMT_EUNSUPPORTED, "cluster of %d workgroups per restart cannot be co-resident", k);
        } else if (ib.empty()) {
            k = best_cluster(insts, ia, waves, total_r, resident_of(true));
            // the fixed scratch bounds the partial gradients
            auto part_bytes = [&]() {
                int64_t f = 0;
                for (int i : ia) f += (int64_t)states[i].a.rows * 2 * k * ((int64_t)insts[i]->n_bool + insts[i]->n_real + 1);
                return f * (int64_t)sizeof(float);
            };
            const int64_t room = (int64_t)fixed_cap - (int64_t)(sizeof(InstDesc) * ia.size() + 32 * total_r + 4096);
            while (fixed_scratch && k > 1 && part_bytes() > room) k /= 2;
        }
        int64_t wg = 0;
        for (size_t q = 0; q < ia.size(); ++q) {
            const fsmt_xbdd *h = insts[ia[q]];
            const fsmt_solve_state &S = states[ia[q]];
            InstDesc &d = desc[q];
            d.T = TabView::of(h);
            d.hs = halfspaces_of(h);
            d.a = as_gptr(S.a.data);
            d.b = as_gptr(S.b.data);
            d.a_sr = S.a.stride_r;
            d.b_sr = S.b.stride_r;
            d.w = as_gptr(S.w);
            d.hist = as_gptr(S.hist);
            d.sat_bits = as_gptr(S.sat_bits);
            d.n_unsat = as_gptr(S.n_unsat);
            d.verdict = as_gptr(S.verdict);
            d.level_done = as_gptr(S.level_done);
            d.steps_done = as_gptr(S.steps_done);
            d.obj = as_gptr(S.obj);
            d.R = S.a.rows;
            d.k = k;
            d.wg_base = (int32_t)wg;
            wg += (int64_t)d.R * k;
            if (k > 1) part_floats += (int64_t)d.R * 2 * k * ((int64_t)h->n_bool + h->n_real + 1);
        }
        if (wg > INT32_MAX || wg * 64 * waves > (int64_t)UINT32_MAX) return set_error(FSMT_ELIMIT, "too many restarts");
        P.lds_nodes = G.maxn;
        P.lds_slots = G.maxs;
        P.state_floats = (int32_t)G.state_f;
        P.waves = waves;
        // scratch: descriptors | stop flags [n] | abort flag | barriers [R] | level results [2][2R] | partials [2]
        void *dbuf = nullptr;
        const size_t desc_bytes = sizeof(InstDesc) * desc.size();
        const size_t off_flag = (desc_bytes + 255) / 256 * 256;
        const size_t n_int = desc.size() + 1 + 5 * (size_t)total_r;
        const size_t off_part = off_flag + (n_int * sizeof(int32_t) + 255) / 256 * 256;
        rc = mem.get(off_part + sizeof(float) * (size_t)part_floats, st, &dbuf);
        if (!rc) {
            int32_t *ints = (int32_t *)((char *)dbuf + off_flag);
            int32_t *flags = ints, *abort_flag = ints + desc.size(), *bar = abort_flag + 1, *ctl = bar + total_r;
            float *part = (float *)((char *)dbuf + off_part);
            int64_t rb = 0, pb = 0;
            for (InstDesc &d : desc) {
                d.bar = as_gptr(bar + rb);
                d.ctl = as_gptr(ctl + 4 * rb);
                d.part = k > 1 ? as_gptr(part + pb) : nullptr;
                rb += d.R;
                if (k > 1) pb += (int64_t)d.R * 2 * k * ((int64_t)d.T.n_bool + d.T.n_real + 1);
            }
            // flags, barriers and level results start at zero (a fill kernel, not a memset:
            // the call may be captured into a graph); the partials are written before read
            if (hipMemcpyAsync(dbuf, desc.data(), desc_bytes, hipMemcpyHostToDevice, st) != hipSuccess ||
                fill_i32(ints, (int64_t)n_int, 0, st) != FSMT_OK) {
                (void)hipGetLastError();
                rc = set_error(FSMT_EHIP, "descriptor upload failed");
            } else {
                const dim3 g((unsigned)wg), b(64 * waves);
                const InstDesc *d = (const InstDesc *)dbuf;
                void *args[] = {(void *)&d, (void *)&P, (void *)&flags, (void *)&abort_flag};
                const hipError_t le = hipLaunchKernel(kernel_of(k > 1), g, b, args, lds, st);
                rc = le != hipSuccess ? set_error(FSMT_EHIP, "solver kernel: %s", hipGetErrorString(le))
                                      : launch_status("solver kernel");
            }
            mem.put(dbuf, st);
        }
    }

    // ---- grid schedule
    if (!ib.empty() && !rc) {
        std::vector<GridInst> gi(ib.size());
        int total_r = 0;
        int64_t tasks = 0, checks = 0, scratch_floats = 0, level_tasks = 0, big_restarts = 0, tile_tasks = 0;
        int64_t wg_blocks = 0, row_floats = 0, work = 0;
        size_t wg_lds = 0;
        int wg_cf = 1;
        int64_t restarts = 0;
        for (int i : ib) {
            work += (int64_t)states[i].a.rows * sweep_tasks(insts[i]);
            restarts += states[i].a.rows;
        }
        int lvl_nodes = 0, lvl_slots = 1, lvl_sym = 0;
        int maxn = 0, maxs = 1;
        size_t step_lds = 0;
        for (size_t q = 0; q < ib.size(); ++q) {
            const fsmt_xbdd *h = insts[ib[q]];
            const fsmt_solve_state &S = states[ib[q]];
            GridInst &d = gi[q];
            d.T = TabView::of(h);
            d.hs = halfspaces_of(h);
            d.a = as_gptr(S.a.data);
            d.b = as_gptr(S.b.data);
            d.a_sr = S.a.stride_r;
            d.b_sr = S.b.stride_r;
            d.ga = as_gptr(S.grad_a);
            d.gb = as_gptr(S.grad_b);
            d.w = as_gptr(S.w);
            d.hist = as_gptr(S.hist);
            d.sat_bits = as_gptr(S.sat_bits);
            d.n_unsat = as_gptr(S.n_unsat);
            d.verdict = as_gptr(S.verdict);
            d.level_done = as_gptr(S.level_done);
            d.steps_done = as_gptr(S.steps_done);
            d.obj = as_gptr(S.obj);
            d.R = S.a.rows;
            int rp = 1, lg = 0;
            while (rp < d.R && rp < 64) { rp <<= 1; ++lg; }
            d.R_pad = d.R <= 64 ? rp : (d.R + 63) / 64 * 64;
            d.log2_rpad = d.R <= 64 ? lg : 0;
            d.rbase = total_r;
            d.task_base = tasks;
            d.check_base = checks;
            d.lev = as_cptr(h->d.lev);
            d.big_pos = as_cptr(h->d.big_pos);
            d.n_big = h->n_big;
            d.pad = 0;
            big_restarts += (int64_t)h->n_big * d.R;
            if (h->n_big > 0) {
                lvl_nodes = std::max(lvl_nodes, h->big_max_nodes);
                lvl_slots = std::max(lvl_slots, h->big_max_slots);
                lvl_sym = std::max(lvl_sym, h->sym_max);
            }
            d.tile_base = tile_tasks;
            // (a workgroup of 1,024 threads a restart at least: the launch stays below 2^32 threads)
            d.slices = restarts <= (1 << 21) ? grid_slices(h, d.R, work, budget, n_cu) : 0;
            d.wg_base = wg_blocks;
            d.row_base = row_floats;
            // 200 scheduling jobs, one restart, 20 steps: 345 us with chunks of 2 tiles, 1,070 with 32
            const int tchunk = tile_chunk((int64_t)d.R * h->n_tiles, n_cu);
            d.tile_chunks = d.slices ? 0 : (h->n_tiles + tchunk - 1) / tchunk;
            tile_tasks += (int64_t)d.R * d.tile_chunks;
            total_r += d.R;
            if (d.slices) {
                wg_blocks += (int64_t)d.R * d.slices;
                row_floats += (int64_t)d.R * d.slices * h->n_real;
                wg_lds = std::max(wg_lds, (size_t)h->n_real * 12);
                wg_cf = closed_level_of(wg_cf, closed_level(h));
            } else tasks += d.R <= 64 ? (int64_t)h->n_pos * d.R_pad / 64 : (int64_t)h->n_pos * (d.R_pad / 64);
            checks += (int64_t)d.R * ((h->n_cons + 255) / 256);
            if (!S.grad_a || !S.grad_b) scratch_floats += (int64_t)d.R * (h->n_bool + h->n_real);
            if (!d.slices) {
                maxn = std::max(maxn, h->small_max_nodes);
                maxs = std::max(maxs, h->small_max_slots);
            }
            if (h->n_hs) step_lds = std::max(step_lds, (size_t)(2 * h->n_real + h->hs_nnz) * sizeof(float));
        }
        bool lds_only = false, all_inline = true;
        for (size_t q = 0; q < ib.size(); ++q) {
            if (gi[q].slices) continue;
            lds_only = lds_only || lds_store(insts[ib[q]]);
            all_inline = all_inline && insts[ib[q]]->all_inline;
        }
        const int msg = msg_variant(maxn, maxs, lds_only, all_inline);
        const size_t wave_bytes = msg == kMsgLds ? WaveScratch::bytes(maxn + 2, maxs) : 0;
        if (wave_bytes > 65536) rc = set_error(FSMT_ELIMIT, "diagram too large for the grid schedule");
        // level tasks: (big constraint, chunk of restarts), instance-major
        const int lvl_chunk = level_chunk(big_restarts, n_cu);
        for (GridInst &d : gi) {
            d.level_base = level_tasks;
            level_tasks += (int64_t)d.n_big * ((d.R + lvl_chunk - 1) / lvl_chunk);
        }
        const size_t level_bytes = level_tasks > 0 ? big_wave_floats(lvl_nodes, lvl_slots, lvl_sym) * sizeof(float) : 0;
        if (level_tasks > 0 && level_too_large(lvl_nodes, lvl_slots)) rc = set_error(FSMT_ELIMIT, "diagram too large for the level-synchronous pass");
        if (step_lds > 65536) rc = set_error(FSMT_ELIMIT, "projection work arrays exceed LDS");
        // device scratch: descriptors, kappas, per-restart flags and accumulators, gradients
        const size_t off_k = (sizeof(GridInst) * gi.size() + 255) / 256 * 256;
        const size_t off_act = off_k + (sizeof(double) * std::max(1, O.n_levels) + 255) / 256 * 256;
        const size_t off_stp = off_act + (sizeof(int32_t) * total_r + 255) / 256 * 256;
        const size_t off_obj = off_stp + (sizeof(int32_t) * total_r + 255) / 256 * 256;
        const size_t off_flg = off_obj + (sizeof(float) * total_r + 255) / 256 * 256;
        const size_t off_gsq = off_flg + (sizeof(int32_t) * gi.size() + 255) / 256 * 256;
        const size_t off_ws = off_gsq + (sizeof(float) * total_r + 255) / 256 * 256;
        const size_t off_grd = off_ws + (sizeof(float) * (size_t)checks + 255) / 256 * 256;
        const size_t off_row = off_grd + (sizeof(float) * (size_t)scratch_floats + 255) / 256 * 256;
        const size_t total = off_row + sizeof(float) * (size_t)row_floats;
        void *buf = nullptr;
        if (!rc) rc = mem.get(total, gst, &buf);
        if (!rc) {
            char *base = (char *)buf;
            float *grd = (float *)(base + off_grd);
            for (GridInst &d : gi) {
                if (!d.ga || !d.gb) {
                    d.ga = as_gptr(grd);
                    d.gb = as_gptr(grd + (int64_t)d.R * d.T.n_bool);
                    grd += (int64_t)d.R * (d.T.n_bool + d.T.n_real);
                }
            }
            GridShared S{};
            S.kappas = (const double *)(base + off_k);
            S.active = (int32_t *)(base + off_act);
            S.stepping = (int32_t *)(base + off_stp);
            S.obj_acc = (float *)(base + off_obj);
            S.stop_flags = (int32_t *)(base + off_flg);
            S.gsq_acc = (float *)(base + off_gsq);
            S.ws_part = (float *)(base + off_ws);
            S.rows = (float *)(base + off_row);
            S.total_r = total_r;
            S.n_levels = O.n_levels;
            S.stop_mode = O.stop_on_sat;
            S.tau = O.tau;
            S.normalize = O.normalize ? 1 : 0;
            S.lds_nodes = maxn;
            S.lds_slots = maxs;
            S.eta_a = O.eta_a;
            S.eta_b = O.eta_b;
            S.eps2 = O.eps > 0.0f ? O.eps * O.eps : -1.0f;
            S.rho = O.rho;
            S.gamma = O.gamma;
            S.total_tasks = tasks;
            S.level_tasks = level_tasks;
            S.tile_tasks = tile_tasks;
            S.level_nodes = lvl_nodes;
            S.level_slots = lvl_slots;
            S.level_chunk = lvl_chunk;
            S.level_floats = (int32_t)(level_bytes / sizeof(float));
            std::vector<double> kap(O.kappas, O.kappas + O.n_levels);
            if (hipMemcpyAsync(base, gi.data(), sizeof(GridInst) * gi.size(), hipMemcpyHostToDevice, gst) != hipSuccess ||
                (O.n_levels > 0 && hipMemcpyAsync(base + off_k, kap.data(), sizeof(double) * kap.size(),
                                                  hipMemcpyHostToDevice, gst) != hipSuccess) ||
                fill_i32(S.stop_flags, (int64_t)gi.size(), 0, gst) != FSMT_OK ||
                fill_f32((float *)(base + off_grd), scratch_floats, 0.0f, gst) != FSMT_OK) {
                (void)hipGetLastError();
                rc = set_error(FSMT_EHIP, "grid schedule upload failed");
            } else {
                GridPlan plan{};
                plan.steps = O.steps_per_level;
                plan.msg = msg;
                plan.sweep_wpb = wave_bytes ? (int)std::max<size_t>(1, std::min<size_t>(4, 65536 / wave_bytes)) : 4;
                plan.sweep_lds = wave_bytes * plan.sweep_wpb;
                plan.sweep_blocks = (int)std::max<int64_t>(1, std::min<int64_t>((tasks + plan.sweep_wpb - 1) / plan.sweep_wpb,
                                                                               (int64_t)n_cu * 8));
                plan.step_lds = step_lds;
                plan.level_wpb = level_bytes ? (int)std::max<size_t>(1, std::min<size_t>(4, 65536 / level_bytes)) : 1;
                plan.level_lds = level_bytes * plan.level_wpb;
                plan.level_blocks = level_tasks > 0 ? (int)std::min<int64_t>((level_tasks + plan.level_wpb - 1) / plan.level_wpb,
                                                                             (int64_t)n_cu * 16)
                                                    : 0;
                plan.check_blocks = checks;
                plan.use_graph = true;
                plan.wg_blocks = wg_blocks;
                plan.wg_cf = wg_cf;
                plan.wg_lds = wg_lds;
                plan.cf = 0;
                for (size_t q = 0; q < ib.size(); ++q)
                    if (!gi[q].slices)
                        plan.cf = closed_level_of(plan.cf, untiled_level(closed_level(insts[ib[q]]), insts[ib[q]]->n_window > 0));
                // each replay of the level sequence advances every running restart by one
                // level (the kernels read each restart's level from memory and skip finished
                // restarts); levels below level_begin are complete by the caller's word, so
                // they are not replayed
                const int replays = std::max(0, O.n_levels - std::min(O.level_begin, O.n_levels));
                rc = run_grid_schedule((const GridInst *)buf, (int)gi.size(), S, plan, replays, gst, res->cap,
                                       res->retired);
            }
            mem.put(buf, gst);
        }
    }

    if (gst != st) {
        if (hipEventRecord(res->ev_join, gst) != hipSuccess || hipStreamWaitEvent(st, res->ev_join, 0) != hipSuccess) {
            (void)hipGetLastError();
            if (!rc) rc = set_error(FSMT_EHIP, "stream join failed");
        }
    }
    return rc;
}

}  // namespace fsmt

extern "C" fsmt_status fsmt_solve_batched(const fsmt_xbdd *const *insts, int32_t n_inst, const fsmt_solve_opts *opts,
                                          const fsmt_solve_state *states, void *stream) {
    return solve_impl(insts, n_inst, opts, states, stream, nullptr, 0);
}

// ---- allocation-free variant: the call's device memory (descriptors, flags, cluster
// barriers and partial gradients) is carved from this array, one copy per device, held until
// the process ends. In host code the name is only a stand-in for the symbol: its device
// address comes from hipGetSymbolAddress, once per device with that device current.
static __device__ __align__(256) char scratch[FSMT_NOALLOC_SCRATCH_BYTES];

static std::mutex g_scratch_mutex;
static void *g_scratch_ptr[kMaxDevices];

extern "C" fsmt_status fsmt_solve_batched_noalloc(const fsmt_xbdd *const *insts, int32_t n_inst,
                                                  const fsmt_solve_opts *opts, const fsmt_solve_state *states,
                                                  void *stream) {
    clear_error();
    if (!insts || n_inst <= 0 || !insts[0]) return set_error(FSMT_EINVAL, "null argument or no instance");
    fsmt_status rc = select_device(insts[0]);
    if (rc) return rc;
    const int device = insts[0]->device;
    if (device < 0 || device >= kMaxDevices) return set_error(FSMT_EINVAL, "device %d out of range", device);
    void *base = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[device]) {
            void *p = nullptr;
            const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p) {
                (void)hipGetLastError();
                return set_error(FSMT_EHIP, "address of the solver scratch on device %d: %s", device,
                                 hipGetErrorString(e));
            }
            g_scratch_ptr[device] = p;
        }
        base = g_scratch_ptr[device];
    }
    return solve_impl(insts, n_inst, opts, states, stream, base, (size_t)FSMT_NOALLOC_SCRATCH_BYTES);
}

extern "C" fsmt_status fsmt_solve_status(const fsmt_solve_state *states, int32_t n_inst, void *stream) {
    clear_error();
    if (!states || n_inst <= 0) return set_error(FSMT_EINVAL, "null argument or no instance");
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) {
        const hipError_t e = hipGetLastError();
        return set_error(FSMT_EHIP, "stream synchronize: %s", hipGetErrorString(e));
    }
    for (int i = 0; i < n_inst; ++i) {
        const int R = states[i].a.rows;
        if (R <= 0 || !states[i].verdict) return set_error(FSMT_EINVAL, "instance %d: no restarts or no verdict", i);
        std::vector<int32_t> v((size_t)R);
        if (hipMemcpy(v.data(), states[i].verdict, sizeof(int32_t) * R, hipMemcpyDeviceToHost) != hipSuccess) {
            const hipError_t e = hipGetLastError();
            return set_error(FSMT_EHIP, "reading verdicts: %s", hipGetErrorString(e));
        }
        for (int r = 0; r < R; ++r)
            if (v[r] == -2)
                return set_error(FSMT_EABORTED, "instance %d, restart %d: a cluster barrier gave up waiting; the "
                                 "state holds its last completed level", i, r);
    }
    return FSMT_OK;
}
