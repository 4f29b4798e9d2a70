// Grid schedule of the batched solver, for instances whose restart state does not fit in
// LDS (or whose restarts are too few to fill the device from one workgroup each).
//
// One annealing level is a fixed sequence of grid-wide kernels over all such instances:
//   begin  : per restart, decide whether it runs this level; zero its counters
//   K x  { sweep : forward + reverse sweep of every (constraint, restart) lane of every
//                  instance (waves as in the per-call kernel, lanes of inactive restarts
//                  skip their work), gradient scatter into the instance's gradient arrays
//          step  : per restart (one block), projected step on the box / unit atoms,
//                  gradient map norm, early end of the level once ||g||^2 <= eps^2 }
//   check  : exact check and ERWA update of every (constraint, restart); scale normalizes
//   end    : per restart, level counter, verdict, stop flag
// Every kernel reads the level of its restart from device memory, so the sequence is
// captured once into a hipGraph and replayed once per level.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "tile_eval.hpp"
#include "solve_grid.hpp"

namespace fsmt {

__device__ __forceinline__ int find_base32(const GridInst *I, int n, int64_t key, int which) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        const int64_t b = which == 0 ? I[mid].task_base
                          : which == 1 ? (int64_t)I[mid].rbase
                          : which == 2 ? I[mid].check_base
                          : which == 3 ? I[mid].level_base
                          : which == 4 ? I[mid].tile_base
                                       : I[mid].wg_base;
        if (b <= key) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Per restart: does it run this level?
__global__ void grid_begin_kernel(const GridInst *insts, int n_inst, GridShared S) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= S.total_r) return;
    const int ii = find_base32(insts, n_inst, g, 1);
    const GridInst &I = insts[ii];
    const int r = g - I.rbase;
    const bool done = I.verdict[r] == 1 && S.stop_mode != 0;
    const bool stopped = S.stop_mode == 2 && S.stop_flags[ii] != 0;
    const int act = (!done && !stopped && I.level_done[r] < S.n_levels) ? 1 : 0;
    S.active[g] = act;
    S.stepping[g] = act;
    S.obj_acc[g] = 0.0f;
    S.gsq_acc[g] = 0.0f;
    if (act) {
        I.n_unsat[r] = 0;
        if (I.verdict[r] < 0) I.verdict[r] = 0;   // an earlier call gave up: resume as not SAT
    }
}

// Waves a SIMD that the sweep's registers have to leave room for (the compiler stops one register
// short of some of them by itself: two-Boolean disjunctions at level 1, windows at level 3, a
// quarter more time a sweep of 4,000 constraints of 2,800 shapes).
template <int V, int kCF>
constexpr int kSweepWaves = (V == kMsgMedium || V == kMsgLarge) ? 1 : kCF <= 1 ? 5 : kCF == 3 && V == kMsgSmall ? 2 : 3;

// Forward + reverse sweep over every instance's (constraint, restart) lanes.
template <int V, int kCF>
__global__ void __launch_bounds__(256, (kSweepWaves<V, kCF>)) grid_sweep_kernel(const GridInst *insts, int n_inst, GridShared S) {
    using Ms = typename MsgOf<V>::type;
    extern __shared__ float lds[];
    const int lane = threadIdx.x & 63, wib = wave_id(), wpb = blockDim.x >> 6;
    const int NN = S.lds_nodes + 2, SS = S.lds_slots;
    FSMT_MSG_STORE(Ms, W, lds + (size_t)wib * (2 * NN + 4 * SS) * 64, NN, SS, lane);
    const int64_t n_waves = (int64_t)gridDim.x * wpb;
    // objective partials are carried across this wave's tasks while they stay in one
    // instance (R <= 64: a lane's restart is fixed there) and flushed on a change
    int cur = -1, cur_rpad = 64, cur_rbase = 0, cur_R = 0;
    float oacc = 0.0f;
    auto flush = [&]() {
        if (cur < 0) return;
        for (int off = 32; off >= cur_rpad; off >>= 1) oacc += __shfl_xor(oacc, off, 64);
        if (lane < cur_rpad && lane < cur_R && oacc != 0.0f) atomic_add_f32(S.obj_acc + cur_rbase + lane, oacc);
        oacc = 0.0f;
    };
    for (int64_t task = (int64_t)blockIdx.x * wpb + wib; task < S.total_tasks; task += n_waves) {
        const int ii = find_base32(insts, n_inst, task, 0);
        const GridInst &I = insts[ii];
        const int64_t lt = task - I.task_base;
        int pos, r;
        if (I.R_pad <= 64) {
            pos = (int)(lt * (64 >> I.log2_rpad)) + (lane >> I.log2_rpad);
            r = lane & (I.R_pad - 1);
        } else {
            const int wpc = I.R_pad >> 6;
            pos = (int)(lt / wpc);
            r = (int)(lt % wpc) * 64 + lane;
        }
        if (ii != cur) {
            flush();
            cur = ii;
            cur_rpad = I.R_pad <= 64 ? I.R_pad : 64;
            cur_rbase = I.rbase;
            cur_R = I.R <= 64 ? I.R : 0;
        }
        const bool r_ok = r < I.R && S.stepping[I.rbase + r] != 0;
        const TabView T = I.T;
        const GlobalState st{View{I.a, I.R, T.n_bool, I.a_sr, 1}, View{I.b, I.R, T.n_real, I.b_sr, 1}};
        // gradients restart-contiguous: one wave-wide atomic of a constraint group touches
        // the R_pad consecutive restarts of one variable, one cache line for R_pad <= 16
        const GlobalScatter sc{View{I.ga, I.R, T.n_bool, 1, I.R}, View{I.gb, I.R, T.n_real, 1, I.R},
                               I.R_pad < 64 ? I.R_pad : 64};
        const TaskCtx t = task_ctx(T, pos, r, r_ok);
        if (t.B.big) continue;   // evaluated by grid_level_kernel
        const double kappa = t.valid ? S.kappas[I.level_done[r]] : 0.0;
        const bool hard = isinf(kappa);
        const float wc = t.valid ? I.w[(int64_t)r * T.n_cons + t.c] : 0.0f;   // requested before the forward pass
        const float unsat = task_eval<true, kCF>(T, t, st, kappa, hard, wc, sc, W, lane);
        if (I.R_pad <= 64) {
            oacc += wc * unsat;
        } else if (r < I.R && wc * unsat != 0.0f) {
            atomic_add_f32(S.obj_acc + I.rbase + r, wc * unsat);
        }
    }
    flush();
}

// Sweep of the instances whose templates all have closed forms and whose real variables fit
// LDS: `slices` workgroups per restart, the real variables and their gradient sums in LDS
// (written out as the workgroup's row, added by the step kernel), the Booleans in global
// memory. A Boolean that is a cell's own (tiles of kind 3) appears in no other constraint, so
// the lane that has its gradient also takes its projected step here: no gradient array, no
// atomics and no pass over the Booleans in the step kernel. The other Booleans' gradient is added
// to a row of the restart's own (restart-contiguous, the restarts' workgroups would add into the
// same lines from every XCD: 20 rectangles, 16 restarts, 20 steps 418 us, 306 so). Three scheduling
// instances of 114,000 to 255,000 clauses at 16 restarts took 396 us a sweep and 219 us a step with
// restarts in the lanes (row-major states: one line per lane) and one block per restart.
struct GridCellScatter {
    View a, ga;        // ga: gradient of the free Booleans, a row per restart
    double *gb;
    float eta_a;
    float *gsq;        // this lane's gradient map of the Booleans it steps
    __device__ __forceinline__ void add_a(int r, int i, float g, int) const {
        if (i >= 0 && g != 0.0f) atomic_add_f32(&ga.at(r, i), g);
    }
    __device__ __forceinline__ void add_b(int, int j, float g, int) const {
        if (j >= 0 && g != 0.0f) atomicAdd(gb + j, (double)g);
    }
    __device__ __forceinline__ void add_b_direct(int, int j, float g) const { atomicAdd(gb + j, (double)g); }
    __device__ __forceinline__ void add(int r, bool real, int i, float g) const {
        if (g == 0.0f) return;
        if (real) atomicAdd(gb + i, (double)g);
        else atomic_add_f32(&ga.at(r, i), g);
    }
    __device__ __forceinline__ void cell(int r, int i, float x, float g) const {
        const float y = x - eta_a * g;
        const float p = y < -1.0f ? -1.0f : (y > 1.0f ? 1.0f : y);
        a.at(r, i) = p;
        const float q = (x - p) / eta_a;
        *gsq += q * q;
    }
};

template <int kCF>
__global__ void __launch_bounds__(1024) grid_wg_kernel(const GridInst *insts, int n_inst, GridShared S) {
    using Ms = typename MsgOf<kMsgSmall>::type;
    extern __shared__ __align__(16) double lds_d[];
    const int lane = threadIdx.x & 63, wib = wave_id(), wpb = blockDim.x >> 6;
    const int ii = find_base32(insts, n_inst, blockIdx.x, 5);
    const GridInst &I = insts[ii];
    const int lb = (int)(blockIdx.x - I.wg_base), r = lb / I.slices, slice = lb - r * I.slices;
    if (!S.stepping[I.rbase + r]) return;   // uniform
    const TabView T = I.T;
    const int m = T.n_real;
    double *gb = lds_d;
    float *sb = (float *)(gb + m);
    const gptr<float> brow = I.b + (int64_t)r * I.b_sr;
    for (int j = threadIdx.x; j < m; j += blockDim.x) {
        sb[j] = brow[j];
        gb[j] = 0.0;
    }
    __syncthreads();
    FSMT_MSG_STORE(Ms, W, nullptr, 0, 0, lane);
    const View av{I.a, I.R, T.n_bool, I.a_sr, 1};
    float gsq = 0.0f, oacc = 0.0f;
    const MixedState st{av, sb};
    const GridCellScatter sc{av, View{I.ga, I.R, T.n_bool, T.n_bool, 1}, gb, S.eta_a, &gsq};
    const double kappa = S.kappas[I.level_done[r]];
    const bool hard = isinf(kappa);
    const gptr<float> wrow = I.w + (int64_t)r * T.n_cons;
    auto wload = [&](int c) -> float { return wrow[c]; };
    const int n_waves = I.slices * wpb, n_tasks = T.n_pos >> 6;
    for (int task = slice + I.slices * wib; task < n_tasks; task += n_waves) {
        const TaskCtx t = task_ctx(T, task * 64 + lane, r, true);
        const float wc = t.valid ? wload(t.c) : 0.0f;
        oacc += wc * task_eval<true, kCF>(T, t, st, kappa, hard, wc, sc, W, lane);
    }
    oacc += tile_sweep<kCF, true>(T, st, sc, r, kappa, hard, slice * wpb + wib, n_waves, wload, [](int, float) {}, lane);
    const float2 red = block_sum2(oacc, gsq);   // also: every wave's adds have reached the LDS
    if (threadIdx.x == 0) {
        atomic_add_f32(S.obj_acc + I.rbase + r, red.x);
        if (red.y != 0.0f) atomic_add_f32(S.gsq_acc + I.rbase + r, red.y);
    }
    float *row = S.rows + I.row_base + (int64_t)lb * m;
    for (int j = threadIdx.x; j < m; j += blockDim.x) row[j] = (float)gb[j];
}

// Tiled constraints of the other instances: one wavefront per (restart, chunk of tiles); the
// chunks are as long as still gives every CU 16 waves (runs share their column's values), at most
// 32 tiles.
__global__ void __launch_bounds__(256, 3) grid_tile_kernel(const GridInst *insts, int n_inst, GridShared S) {
    const int lane = threadIdx.x & 63, wpb = blockDim.x >> 6;
    for (int64_t task = (int64_t)blockIdx.x * wpb + wave_id(); task < S.tile_tasks; task += (int64_t)gridDim.x * wpb) {
        const int ii = find_base32(insts, n_inst, task, 4);
        const GridInst &I = insts[ii];
        const int64_t lt = task - I.tile_base;
        const int r = (int)(lt / I.tile_chunks), id = (int)(lt - (int64_t)r * I.tile_chunks);
        if (!S.stepping[I.rbase + r]) continue;   // uniform
        const TabView T = I.T;
        const GlobalState st{View{I.a, I.R, T.n_bool, I.a_sr, 1}, View{I.b, I.R, T.n_real, I.b_sr, 1}};
        const GlobalScatter sc{View{I.ga, I.R, T.n_bool, 1, I.R}, View{I.gb, I.R, T.n_real, 1, I.R}, 64};
        const double kappa = S.kappas[I.level_done[r]];
        const float oacc = wave_sum(tile_sweep<3, true>(T, st, sc, r, kappa, isinf(kappa), id, I.tile_chunks,
                                                        [&](int c) -> float { return I.w[(int64_t)r * T.n_cons + c]; },
                                                        [](int, float) {}, lane));
        if (lane == 0 && oacc != 0.0f) atomic_add_f32(S.obj_acc + I.rbase + r, oacc);
    }
}

// Big diagrams: one wavefront per (big constraint, chunk of restarts) over every instance,
// level by level (level_eval), into the same gradient rows and objective accumulators.
__global__ void __launch_bounds__(256) grid_level_kernel(const GridInst *insts, int n_inst, GridShared S) {
    extern __shared__ __align__(16) float lds[];
    const int lane = threadIdx.x & 63, wib = wave_id(), wpb = blockDim.x >> 6;
    float *const rows = lds + (size_t)wib * S.level_floats;
    const LevelRows W = LevelRows::at(rows, S.level_nodes, S.level_slots);
    WaveObjAcc oa{S.obj_acc};
    // chunk-major task order inside an instance: a wave's consecutive tasks share their
    // restart chunk, so the objective's partial sums stay in lanes
    for (int64_t task = (int64_t)blockIdx.x * wpb + wib; task < S.level_tasks; task += (int64_t)gridDim.x * wpb) {
        const int ii = find_base32(insts, n_inst, task, 3);
        const GridInst &I = insts[ii];
        const int64_t lt = task - I.level_base;
        const int ci = (int)(lt / I.n_big), q = (int)(lt - (int64_t)ci * I.n_big);
        const int r0 = ci * S.level_chunk, r1 = r0 + S.level_chunk < I.R ? r0 + S.level_chunk : I.R;
        oa.begin(I.rbase + r0, r1 - r0, lane);
        const TabView T = I.T;
        const GlobalState st{View{I.a, I.R, T.n_bool, I.a_sr, 1}, View{I.b, I.R, T.n_real, I.b_sr, 1}};
        const GlobalScatter sc{View{I.ga, I.R, T.n_bool, 1, I.R}, View{I.gb, I.R, T.n_real, 1, I.R}, 64};
        const LevelCtx L = level_ctx(T, I.lev, I.big_pos[q]);
        const bool sym = L.B.big == 2;
        if (!sym) level_stage_nodes(T, L, W, lane);
        for (int r = r0; r < r1; ++r) {
            if (!S.stepping[I.rbase + r]) continue;   // uniform: one restart at a time
            const double kappa = S.kappas[I.level_done[r]];
            const float wc = I.w[(int64_t)r * T.n_cons + L.c];
            const float unsat = sym ? sym_eval(T, L, st, sc, r, kappa, isinf(kappa), wc, true, rows, lane)
                                    : level_eval(T, L, st, sc, r, kappa, isinf(kappa), wc, true, W, lane);
            oa.add(r - r0, wc * unsat, lane);
        }
    }
    oa.flush(lane);
}

// Projected step, one block per restart: every Boolean, or with grid_wg_kernel the free ones
// (the others have taken theirs), and the real variables, whose gradient is then the sum of
// the slices' rows.
__global__ void __launch_bounds__(1024) grid_step_kernel(const GridInst *insts, int n_inst, GridShared S) {
    extern __shared__ float sm[];
    const int g = blockIdx.x;
    const int ii = find_base32(insts, n_inst, g, 1);
    const GridInst &I = insts[ii];
    const int r = g - I.rbase;
    if (!S.stepping[g]) return;
    const bool wg = I.slices > 0;
    const int n = wg ? I.T.n_free : I.T.n_bool, m = I.T.n_real;
    const gptr<float> arow = I.a + (int64_t)r * I.a_sr, brow = I.b + (int64_t)r * I.b_sr;
    const gptr<float> gacol = wg ? I.ga + (int64_t)r * I.T.n_bool : I.ga + r;   // element i at i * ga_s
    const gptr<float> gbcol = I.gb + r;                                         // element j at j * R
    const int64_t ga_s = wg ? 1 : I.R;
    const float *rows = S.rows + I.row_base + (int64_t)r * I.slices * m;
    auto grad_b = [&](int j) -> float {
        if (!wg) {
            const float v = gbcol[(int64_t)j * I.R];
            gbcol[(int64_t)j * I.R] = 0.0f;
            return v;
        }
        float v = 0.0f;
        for (int s0 = 0; s0 < I.slices; s0 += 8) {   // eight rows requested together
            float x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = s0 + q < I.slices ? rows[(int64_t)(s0 + q) * m + j] : 0.0f;
#pragma unroll
            for (int q = 0; q < 8; ++q) v += x[q];
        }
        return v;
    };
    float acc = 0.0f;
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
        const int i = wg ? I.T.free_bool[e] : e;
        const float x = arow[i], y = x - S.eta_a * gacol[i * ga_s];
        const float p = y < -1.0f ? -1.0f : (y > 1.0f ? 1.0f : y);
        arow[i] = p;
        gacol[i * ga_s] = 0.0f;
        const float q = (x - p) / S.eta_a;
        acc += q * q;
    }
    if (I.hs.n == 0) {
        for (int j = threadIdx.x; j < m; j += blockDim.x) {
            const float x = brow[j], y = x - S.eta_b * grad_b(j);
            const float p = y < I.T.real_lo[j] ? I.T.real_lo[j] : (y > I.T.real_hi[j] ? I.T.real_hi[j] : y);
            brow[j] = p;
            const float q = (x - p) / S.eta_b;
            acc += q * q;
        }
    } else {
        float *y = sm, *pb = sm + m, *ph = sm + 2 * m;
        for (int j = threadIdx.x; j < m; j += blockDim.x) y[j] = brow[j] - S.eta_b * grad_b(j);
        project_dykstra(y, pb, ph, I.T.real_lo, I.T.real_hi, m, I.hs);
        for (int j = threadIdx.x; j < m; j += blockDim.x) {
            const float x = brow[j], p = y[j];
            brow[j] = p;
            const float q = (x - p) / S.eta_b;
            acc += q * q;
        }
    }
    const float gsq = block_sum(acc) + S.gsq_acc[g];
    __syncthreads();   // every thread has read gsq_acc
    if (threadIdx.x == 0) {
        I.obj[r] = S.obj_acc[g];
        S.obj_acc[g] = 0.0f;
        S.gsq_acc[g] = 0.0f;
        I.steps_done[r] += 1;
        if (gsq <= S.eps2) S.stepping[g] = 0;
    }
}

// Block index of the level-end kernels: one 256-thread block per (instance, restart,
// 256-constraint group).
struct GroupOf {
    int ii, r, c;   // c: this thread's constraint
};
__device__ __forceinline__ GroupOf group_of(const GridInst *insts, int n_inst) {
    const int64_t blk = blockIdx.x;
    const int ii = find_base32(insts, n_inst, blk, 2);
    const GridInst &I = insts[ii];
    const int64_t lb = blk - I.check_base;
    const int groups = (I.T.n_cons + 255) / 256;
    return GroupOf{ii, (int)(lb / groups), (int)(lb % groups) * 256 + (int)threadIdx.x};
}

// Exact check and ERWA update of the history and the weights; each block's sum of its weights
// goes to ws_part (normalized by grid_scale_kernel).
__global__ void __launch_bounds__(256) grid_check_kernel(const GridInst *insts, int n_inst, GridShared S) {
    const int lane = threadIdx.x & 63;
    const GroupOf G = group_of(insts, n_inst);
    const GridInst &I = insts[G.ii];
    const int r = G.r, c = G.c, c64 = c - lane;
    if (!S.active[I.rbase + r]) return;
    const int C = I.T.n_cons, nw = (C + 31) >> 5;
    const GlobalState st{View{I.a, I.R, I.T.n_bool, I.a_sr, 1}, View{I.b, I.R, I.T.n_real, I.b_sr, 1}};
    const bool sat = c < C ? walk_state(I.T, st, c, r) : false;
    const uint64_t mask = __ballot(sat);
    const uint64_t valid = __ballot(c < C);
    float wv = 0.0f;
    if (c < C) {
        const bool update = ((I.level_done[r] + 1) % S.tau) == 0;
        gref<float> wr = I.w[(int64_t)r * C + c], hr = I.hist[(int64_t)r * C + c];
        float h = S.rho * hr + (sat ? 0.0f : 1.0f);
        wv = wr;
        if (update) {
            wv *= ErwaPow(S.gamma, S.rho, false)(h);   // one constraint a thread
            h = 1.0f;
            wr = wv;
        }
        hr = h;
    }
    if (lane == 0 && valid) {
        const gptr<uint32_t> row = I.sat_bits + (int64_t)r * nw;
        row[c64 >> 5] = (uint32_t)mask;
        if ((c64 >> 5) + 1 < nw) row[(c64 >> 5) + 1] = (uint32_t)(mask >> 32);
        const int bad = (int)__popcll(valid & ~mask);
        if (bad) atomicAdd((int32_t *)(I.n_unsat + r), bad);
    }
    if (S.normalize) {
        const float ws = block_sum(wv);
        if (threadIdx.x == 0) S.ws_part[blockIdx.x] = ws;
    }
}

// Weights normalized to sum n_cons after an update. Every block adds its restart's block sums in
// the same fixed order (no atomics: equal check bits give equal weights in every run).
__global__ void __launch_bounds__(256) grid_scale_kernel(const GridInst *insts, int n_inst, GridShared S) {
    const GroupOf G = group_of(insts, n_inst);
    const GridInst &I = insts[G.ii];
    const int C = I.T.n_cons, groups = (C + 255) / 256;
    if (!S.active[I.rbase + G.r] || ((I.level_done[G.r] + 1) % S.tau) != 0) return;   // uniform
    const float *part = S.ws_part + I.check_base + (int64_t)G.r * groups;
    float ws = 0.0f;
    for (int q = threadIdx.x; q < groups; q += 256) ws += part[q];
    ws = block_sum(ws);
    if (G.c < C) I.w[(int64_t)G.r * C + G.c] *= (float)C / ws;
}

// Level counter and verdict, one thread per restart.
__global__ void grid_end_kernel(const GridInst *insts, int n_inst, GridShared S) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= S.total_r || !S.active[g]) return;
    const int ii = find_base32(insts, n_inst, g, 1);
    const GridInst &I = insts[ii];
    const int r = g - I.rbase;
    I.level_done[r] += 1;
    if (I.n_unsat[r] == 0) {
        I.verdict[r] = 1;
        if (S.stop_mode == 2) atomicExch(S.stop_flags + ii, 1);
    }
}

static fsmt_status launch_status(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(FSMT_EHIP, "%s: %s", what, hipGetErrorString(e));
    return FSMT_OK;
}

// Enqueue one level's kernel sequence on st.
template <int kCF>
static void launch_sweep(const GridPlan &P, dim3 g, dim3 b, hipStream_t st, const GridInst *d_insts, int n_inst,
                         const GridShared &S) {
    if (P.msg == kMsgSmall)
        hipLaunchKernelGGL((grid_sweep_kernel<kMsgSmall, kCF>), g, b, 0, st, d_insts, n_inst, S);
    else if (P.msg == kMsgMedium)
        hipLaunchKernelGGL((grid_sweep_kernel<kMsgMedium, kCF>), g, b, 0, st, d_insts, n_inst, S);
    else if (P.msg == kMsgLarge)
        hipLaunchKernelGGL((grid_sweep_kernel<kMsgLarge, kCF>), g, b, 0, st, d_insts, n_inst, S);
    else
        hipLaunchKernelGGL((grid_sweep_kernel<kMsgLds, kCF>), g, b, P.sweep_lds, st, d_insts, n_inst, S);
}

static fsmt_status enqueue_level(const GridInst *d_insts, int n_inst, const GridShared &S, const GridPlan &P,
                                 hipStream_t st) {
    fsmt_status rc;
    hipLaunchKernelGGL(grid_begin_kernel, dim3((S.total_r + 255) / 256), dim3(256), 0, st, d_insts, n_inst, S);
    if ((rc = launch_status("grid begin"))) return rc;
    for (int k = 0; k < P.steps; ++k) {
        const dim3 g(P.sweep_blocks), b(64 * P.sweep_wpb);
        if (P.wg_blocks > 0) {
            const dim3 wg((unsigned)P.wg_blocks), wb(1024);
            if (P.wg_cf == 1) hipLaunchKernelGGL(grid_wg_kernel<1>, wg, wb, P.wg_lds, st, d_insts, n_inst, S);
            else if (P.wg_cf == 2) hipLaunchKernelGGL(grid_wg_kernel<2>, wg, wb, P.wg_lds, st, d_insts, n_inst, S);
            else if (P.wg_cf == 3) hipLaunchKernelGGL(grid_wg_kernel<3>, wg, wb, P.wg_lds, st, d_insts, n_inst, S);
            else hipLaunchKernelGGL(grid_wg_kernel<4>, wg, wb, P.wg_lds, st, d_insts, n_inst, S);
            if ((rc = launch_status("grid workgroup sweep"))) return rc;
        }
        if (S.total_tasks == 0) {
            // every untiled constraint is in the workgroup sweep
        } else if (P.cf == 0)
            launch_sweep<0>(P, g, b, st, d_insts, n_inst, S);
        else if (P.cf == 1)
            launch_sweep<1>(P, g, b, st, d_insts, n_inst, S);
        else if (P.cf == 2)
            launch_sweep<2>(P, g, b, st, d_insts, n_inst, S);
        else if (P.cf == 3)
            launch_sweep<3>(P, g, b, st, d_insts, n_inst, S);
        else
            launch_sweep<4>(P, g, b, st, d_insts, n_inst, S);
        if ((rc = launch_status("grid sweep"))) return rc;
        if (S.tile_tasks > 0) {
            hipLaunchKernelGGL(grid_tile_kernel, dim3((unsigned)std::min<int64_t>((S.tile_tasks + 3) / 4, 1 << 20)), dim3(256), 0, st, d_insts,
                               n_inst, S);
            if ((rc = launch_status("grid tiles"))) return rc;
        }
        if (P.level_blocks > 0) {
            hipLaunchKernelGGL(grid_level_kernel, dim3(P.level_blocks), dim3(64 * P.level_wpb), P.level_lds, st, d_insts,
                               n_inst, S);
            if ((rc = launch_status("grid level"))) return rc;
        }
        hipLaunchKernelGGL(grid_step_kernel, dim3(S.total_r), dim3(P.wg_blocks > 0 ? 1024 : 256), P.step_lds, st, d_insts, n_inst, S);
        if ((rc = launch_status("grid step"))) return rc;
    }
    if (P.check_blocks > 0) {
        hipLaunchKernelGGL(grid_check_kernel, dim3((unsigned)P.check_blocks), dim3(256), 0, st, d_insts, n_inst, S);
        if ((rc = launch_status("grid check"))) return rc;
        if (S.normalize) {
            hipLaunchKernelGGL(grid_scale_kernel, dim3((unsigned)P.check_blocks), dim3(256), 0, st, d_insts, n_inst, S);
            if ((rc = launch_status("grid scale"))) return rc;
        }
    }
    hipLaunchKernelGGL(grid_end_kernel, dim3((S.total_r + 255) / 256), dim3(256), 0, st, d_insts, n_inst, S);
    return launch_status("grid end");
}

void reap_retired(std::vector<GraphRetired> &list) {
    size_t keep = 0;
    for (size_t i = 0; i < list.size(); ++i) {
        const hipError_t q = hipEventQuery(list[i].done);
        if (q == hipSuccess) {
            (void)hipGraphExecDestroy(list[i].exec);
            (void)hipGraphDestroy(list[i].graph);
            (void)hipEventDestroy(list[i].done);
        } else {
            (void)hipGetLastError();   // "not ready" is not an error of the next call
            list[keep++] = list[i];
        }
    }
    list.resize(keep);
}

static std::vector<const void *> level_fns() { return {(const void *)grid_level_kernel}; }

fsmt_status run_grid_schedule(const GridInst *d_insts, int n_inst, const GridShared &S, const GridPlan &P,
                              int n_levels, hipStream_t st, hipStream_t cap, std::vector<GraphRetired> &retired) {
    if (n_levels <= 0 || n_inst == 0) return FSMT_OK;
    // capture one level into a graph on the capture stream, replay it once per level
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    if (P.level_lds > 65536) {
        static LdsBudget B;
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || P.level_lds > B.of(dev, level_fns))
            return set_error(FSMT_ELIMIT, "a big diagram's rows (%zu B) exceed the device's LDS", P.level_lds);
    }
    bool use_graph = cap != nullptr && P.use_graph && n_levels > 1;
    if (use_graph && hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) != hipSuccess) use_graph = false;
    if (use_graph) {
        fsmt_status rc = enqueue_level(d_insts, n_inst, S, P, cap);
        hipError_t e = hipStreamEndCapture(cap, &graph);
        if (rc || e != hipSuccess || hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) {
            (void)hipGetLastError();
            if (graph) (void)hipGraphDestroy(graph);
            graph = nullptr;
            exec = nullptr;
            use_graph = false;
        }
    }
    fsmt_status rc = FSMT_OK;
    for (int t = 0; t < n_levels && !rc; ++t) {
        if (use_graph) {
            if (hipGraphLaunch(exec, st) != hipSuccess) {
                (void)hipGetLastError();
                rc = set_error(FSMT_EHIP, "hipGraphLaunch failed");
            }
        } else {
            rc = enqueue_level(d_insts, n_inst, S, P, st);
        }
    }
    if (exec) {
        // the executable may be destroyed only after its launches finished: an event after
        // them marks that point, and a later call destroys it
        hipEvent_t done = nullptr;
        if (hipEventCreateWithFlags(&done, hipEventDisableTiming) == hipSuccess && hipEventRecord(done, st) == hipSuccess) {
            retired.push_back(GraphRetired{exec, graph, done});
        } else {
            (void)hipGetLastError();
            if (done) (void)hipEventDestroy(done);
            (void)hipStreamSynchronize(st);   // no event to wait on: the only safe point is now
            (void)hipGraphExecDestroy(exec);
            (void)hipGraphDestroy(graph);
            if (!rc) rc = set_error(FSMT_EHIP, "event creation failed");
        }
    }
    return rc;
}

}  // namespace fsmt
