// HIP kernels for gfx950 (CDNA4, wave64) and the per-call C ABI entry points:
// cop_forward, cop_backward, pgd_step, round_and_check.
//
// Work decomposition of the diagram passes. A "task" is one wavefront's worth of
// (constraint, restart) pairs. With R_pad = next power of two >= R (R <= 64) a task covers
// 64/R_pad consecutive constraint positions times R_pad restarts (lane = position-major,
// restart-minor); with R > 64 a task is one position times 64 restarts. Buckets are padded
// to 64 positions, so every lane of a wave walks the same diagram shape: node records are
// wave-uniform and are fetched through the scalar unit (s_load), while each lane keeps its
// own messages in an LDS column ([node][lane] layout, conflict-free, indexed by the
// uniform node id). Probabilities are evaluated once per (slot, lane) before the passes.
// Where a restart's point and gradient fit the LDS, a workgroup sweeps a share of one
// restart instead (cop_wg_kernel; tiles: tile_eval.hpp); big diagrams take a wave each.
//
// Per (constraint c, restart r) the kernel computes (paper, Supplementary Note 5):
//   forward  : m_td[root] = 1; m_td[hi] += p m_td[v]; m_td[lo] += (1-p) m_td[v]
//              (Alg. "Forward Traversal of XBDDs"); P[c False] = m_td[False terminal]
//   backward : beta(v) = P[reach False from v]: beta(True)=0, beta(False)=1,
//              beta(v) = p beta(hi) + (1-p) beta(lo) in reverse order, and
//              dP[c False]/dp_s = sum_{v: slot s} m_td(v) (beta(hi) - beta(lo))
//              (Alg. "Backward Traversal of XBDD", Lemma "backward"; the gradient of the
//              false mass, so the sign is the opposite of the paper's true-mass form)
//   scatter  : grad_a += w (-1/2) dP/dp; grad_b[j] += w dP/dp * dp/dz * q_j
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <mutex>
#include <vector>

#include "fsmt_internal.hpp"
#include "tile_eval.hpp"

namespace fsmt {

struct CopArgs {
    TabView T;
    int32_t R, R_pad, log2_rpad;   // log2_rpad valid for R_pad <= 64
    int64_t n_tasks;
    View a, b, w, unsat, ga, gb;
    float *obj;
    double kappa;
    int32_t hard;
    int32_t lds_nodes, lds_slots;  // per-wave LDS geometry (max over templates)
};

template <bool kGrad, int V, int kCF>
__global__ void __launch_bounds__(256) cop_kernel(CopArgs A) {
    using Ms = typename MsgOf<V>::type;
    extern __shared__ __align__(16) float lds[];
    const int lane = threadIdx.x & 63;
    const int wib = wave_id();
    const int wpb = blockDim.x >> 6;
    const int64_t wave0 = (int64_t)blockIdx.x * wpb + wib;
    const int64_t n_waves = (int64_t)gridDim.x * wpb;
    const int NN = A.lds_nodes + 2, SS = A.lds_slots;
    FSMT_MSG_STORE(Ms, W, lds + (size_t)wib * (2 * NN + 4 * SS) * 64, NN, SS, lane);
    const GlobalState st{A.a, A.b};
    const GlobalScatter sc{A.ga, A.gb, A.R_pad < 64 ? A.R_pad : 64};
    float oacc = 0.0f;   // objective partial of this lane's restart (R_pad <= 64: fixed per lane)

    for (int64_t task = wave0; task < A.n_tasks; task += n_waves) {
        int pos, r;
        if (A.R_pad <= 64) {
            pos = (int)(task * (64 >> A.log2_rpad)) + (lane >> A.log2_rpad);
            r = lane & (A.R_pad - 1);
        } else {
            const int wpc = A.R_pad >> 6;
            pos = (int)(task / wpc);
            r = (int)(task % wpc) * 64 + lane;
        }
        const TaskCtx t = task_ctx(A.T, pos, r, r < A.R);
        if (t.B.big) continue;   // evaluated by cop_level_kernel
        const float wc = t.valid ? A.w.at(r, t.c) : 0.0f;   // requested before the forward pass
        const float unsat = task_eval<kGrad, kCF, true>(A.T, t, st, A.kappa, A.hard != 0, wc, sc, W, lane);
        if (t.valid && A.unsat.data) A.unsat.at(r, t.c) = unsat;
        if (A.obj) {
            if (A.R_pad <= 64) {
                oacc += wc * unsat;
            } else if (r < A.R) {
                atomic_add_f32(A.obj + r, wc * unsat);
            }
        }
    }
    // objective: reduce lanes holding the same restart, one atomic per restart and wave
    if (A.obj && A.R_pad <= 64) {
        for (int off = 32; off >= A.R_pad; off >>= 1) oacc += __shfl_xor(oacc, off, 64);
        if (lane < A.R_pad && lane < A.R && oacc != 0.0f) atomic_add_f32(A.obj + lane, oacc);
    }
}

// Tiled constraints of instances whose state does not fit LDS: one wave per (restart, chunk of
// tiles), the state and the gradient in global memory.
constexpr int64_t kMaxBlocks = 1 << 20;   // of the kernels whose waves loop over their tasks
template <bool kGrad>
__global__ void __launch_bounds__(256) cop_tile_kernel(CopArgs A, int chunks) {
    const int lane = threadIdx.x & 63, wpb = blockDim.x >> 6;
    const GlobalState st{A.a, A.b};
    const GlobalScatter sc{A.ga, A.gb, 64};
    for (int64_t w = (int64_t)blockIdx.x * wpb + wave_id(); w < (int64_t)A.R * chunks; w += (int64_t)gridDim.x * wpb) {
        const int r = (int)(w / chunks), id = (int)(w - (int64_t)r * chunks);
        auto fout = [&](int c, float F) {
            if (A.unsat.data) A.unsat.at(r, c) = F;
        };
        const float oacc = wave_sum(tile_sweep<3, kGrad>(A.T, st, sc, r, A.kappa, A.hard != 0, id, chunks,
                                                         [&](int c) -> float { return A.w.at(r, c); }, fout, lane));
        if (A.obj && lane == 0 && oacc != 0.0f) atomic_add_f32(A.obj + r, oacc);
    }
}

// ------------------------------------------------------------------ one restart per workgroup
// The restart's point (and, for the reverse sweep, its gradient sums, of type G: see
// LdsScatter) in LDS; `slices` workgroups share a restart's sweep (slice-minor block numbers,
// so with a multiple of 8 slices the workgroups of one slice read the same tables on one XCD).
// The outputs leave the workgroup in one of three ways:
//   kStore: one slice, no accumulation; stored into the caller's views: the whole call is this one
//           launch;
//   kAdd  : added into the zeroed (or accumulating) views with device atomics, one per
//           variable and slice;
//   kRows : written as the slice's row of `part` (objective: opart), summed by sum_rows_kernel.
// kMixed: only the real variables (and their gradient) in LDS, see MixedState; the Booleans'
// gradient goes straight to the caller's view (free Booleans: zeroed before, device atomics).
enum { kStore = 0, kAdd = 1, kRows = 2 };

// The restart's point into LDS (sa then sb), the gradient sums cleared: four elements per
// thread requested together, then stored. n: Booleans in LDS.
template <bool kGrad, class G>
__device__ __forceinline__ void wg_load_point(const View &a, const View &b, int r, int n, int nm, float *sa, G *ga) {
    for (int e0 = threadIdx.x; e0 < nm; e0 += 4 * blockDim.x) {
        float x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = e0 + q * (int)blockDim.x;
            x[q] = e < nm ? (e < n ? (float)a.at(r, e) : (float)b.at(r, e - n)) : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = e0 + q * (int)blockDim.x;
            if (e < nm) {
                sa[e] = x[q];
                if constexpr (kGrad) ga[e] = 0;
            }
        }
    }
    __syncthreads();
}

// The workgroup's objective (lanes and waves summed in double) and gradient sums leave in one of
// the three ways (kPart: rows are among them).
template <bool kGrad, bool kPart = true, class G>
__device__ __forceinline__ void wg_store(float oacc, int r, int n, int nm, const G *ga, float *obj, const View &va,
                                         const View &vb, int mode, float *part, double *opart) {
    __shared__ double part_o[16];
    const int lane = threadIdx.x & 63, wib = wave_id(), wpb = blockDim.x >> 6;
    double o = oacc;
    for (int off = 32; off > 0; off >>= 1) o += __shfl_xor(o, off, 64);
    if (lane == 0) part_o[wib] = o;
    __syncthreads();   // also: every wave's gradient adds have reached the LDS
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < wpb; ++q) t += part_o[q];
        if (kPart && mode == kRows) opart[blockIdx.x] = t;
        else if (obj && mode == kStore) obj[r] = (float)t;
        else if (obj) atomic_add_f32(obj + r, (float)t);
    }
    if constexpr (kGrad) {
        float *row = part + (int64_t)blockIdx.x * nm;
        for (int e = threadIdx.x; e < nm; e += blockDim.x) {
            const float g = (float)ga[e];
            if (kPart && mode == kRows) {
                row[e] = g;
            } else {
                gref<float> dst = e < n ? va.at(r, e) : vb.at(r, e - n);
                if (mode == kAdd) {
                    if (g != 0.0f) atomic_add_f32(&dst, g);
                } else {
                    dst = g;
                }
            }
        }
    }
}

template <bool kGrad, int V, int kCF, class G, bool kMixed = false>
__global__ void __launch_bounds__(1024) cop_wg_kernel(CopArgs A, int slices, int mode, int accumulate, float *part,
                                                      double *opart) {
    using Ms = typename MsgOf<V>::type;
    extern __shared__ __align__(16) float lds[];
    const int lane = threadIdx.x & 63, wib = wave_id(), wpb = blockDim.x >> 6;
    const int n = kMixed ? 0 : A.T.n_bool, m = A.T.n_real, nm = n + m;   // n: Booleans in LDS
    const int r = blockIdx.x / slices, slice = blockIdx.x - r * slices;
    G *ga = (G *)lds, *gb = ga + n;
    float *sa = kGrad ? (float *)(ga + nm) : lds, *sb = sa + n;
    const int NN = A.lds_nodes + 2, SS = A.lds_slots;
    FSMT_MSG_STORE(Ms, W, sb + m + (size_t)wib * (2 * NN + 4 * SS) * 64, NN, SS, lane);
    wg_load_point<kGrad>(A.a, A.b, r, n, nm, sa, ga);
    const auto st = [&] {
        if constexpr (kMixed) return MixedState{A.a, sb};
        else return LdsState{sa, sb};
    }();
    const auto sc = [&] {
        if constexpr (kMixed) return MixedScatter{A.ga, (double *)gb, accumulate};
        else return LdsScatter<G>{ga, gb};
    }();
    const bool hard = A.hard != 0;
    auto wload = [&](int c) -> float { return A.w.at(r, c); };
    auto fout = [&](int c, float F) {
        if (!kGrad && A.unsat.data) A.unsat.at(r, c) = F;
    };
    const int id = slice * wpb + wib, n_waves = slices * wpb, n_tasks = A.T.n_pos >> 6;
    float oacc = 0.0f;
    for (int task = slice + slices * wib; task < n_tasks; task += n_waves) {
        const TaskCtx t = task_ctx(A.T, task * 64 + lane, r, true);
        if (t.B.big) continue;   // evaluated by cop_level_kernel
        const float wc = t.valid ? wload(t.c) : 0.0f;   // requested before the forward pass
        const float unsat = task_eval<kGrad, kCF, true>(A.T, t, st, A.kappa, hard, wc, sc, W, lane);
        if (t.valid) fout(t.c, unsat);
        oacc += wc * unsat;
    }
    oacc += tile_sweep<kCF, kGrad>(A.T, st, sc, r, A.kappa, hard, id, n_waves, wload, fout, lane);
    wg_store<kGrad>(oacc, r, n, nm, ga, A.obj, A.ga, A.gb, mode, part, opart);
}

// Restart r = blockIdx.y: its slices' rows added and stored into (or added to) the caller's
// views: 64 elements per block, the rows split over 16 stripes and the stripes' sums added
// in LDS; the first block adds the objective.
__global__ void __launch_bounds__(1024) sum_rows_kernel(const float *part, const double *opart, int slices, int n, int m,
                                                        View ga, View gb, float *obj, int accumulate) {
    __shared__ float red[16][64];
    const int c = threadIdx.x & 63, s = threadIdx.x >> 6;
    const int nm = n + m, r = blockIdx.y;
    const int e = blockIdx.x * 64 + c;
    float acc = 0.0f;
    if (e < nm) {
        // a stripe's first 16 rows are requested together (one round trip, not 16)
        const float *col = part + (int64_t)r * slices * nm + e;
        float v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int w = s + 16 * q;
            v[q] = w < slices ? col[(int64_t)w * nm] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) acc += v[q];
        for (int w = s + 256; w < slices; w += 16) acc += col[(int64_t)w * nm];
    }
    red[s][c] = acc;
    __syncthreads();
    if (s == 0 && e < nm) {
        float t = 0.0f;
        for (int q = 0; q < 16; ++q) t += red[q][c];
        gref<float> dst = e < n ? ga.at(r, e) : gb.at(r, e - n);
        if (!accumulate) dst = t;
        else if (t != 0.0f) atomic_add_f32(&dst, t);
    }
    if (obj && blockIdx.x == 0 && threadIdx.x < 64) {
        double t = 0.0;
        for (int w = threadIdx.x; w < slices; w += 64) t += opart[(int64_t)r * slices + w];
        for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
        if (threadIdx.x == 0) {
            if (accumulate) atomic_add_f32(obj + r, (float)t);
            else obj[r] = (float)t;
        }
    }
}

// ------------------------------------------------------------------ big diagrams
// Level-synchronous passes (see level_eval): one wavefront per (big constraint, chunk of
// restarts); the wave stages the constraint's node table in its LDS rows once and evaluates
// the chunk's restarts one after the other, keeping the objective's partial sums in lanes.
struct LevelArgs {
    TabView T;
    cptr<int32_t> lev, big_pos;
    int32_t n_big, R, chunk;
    View a, b, w, unsat, ga, gb;
    float *obj;
    double kappa;
    int32_t hard;
    int32_t lds_nodes, lds_slots;   // per-wave LDS rows (max over big templates that are not symmetric)
    int32_t wave_floats;
};

template <bool kGrad>
__global__ void __launch_bounds__(256) cop_level_kernel(LevelArgs A) {
    extern __shared__ __align__(16) float lds[];
    const int lane = threadIdx.x & 63;
    const int wib = wave_id();
    const int wpb = blockDim.x >> 6;
    float *const rows = lds + (size_t)wib * A.wave_floats;
    const LevelRows W = LevelRows::at(rows, A.lds_nodes, A.lds_slots);
    const GlobalState st{A.a, A.b};
    const GlobalScatter sc{A.ga, A.gb, 64};
    const int chunks = (A.R + A.chunk - 1) / A.chunk;
    const int64_t n_tasks = (int64_t)A.n_big * chunks;
    WaveObjAcc oa{A.obj};
    // chunk-major task order: a wave's consecutive tasks share their restart chunk
    for (int64_t task = (int64_t)blockIdx.x * wpb + wib; task < n_tasks; task += (int64_t)gridDim.x * wpb) {
        const int ci = (int)(task / A.n_big), q = (int)(task - (int64_t)ci * A.n_big);
        const int r0 = ci * A.chunk, r1 = r0 + A.chunk < A.R ? r0 + A.chunk : A.R;
        oa.begin(r0, r1 - r0, lane);
        const LevelCtx L = level_ctx(A.T, A.lev, A.big_pos[q]);
        const bool sym = L.B.big == 2;
        if (!sym) level_stage_nodes(A.T, L, W, lane);
        for (int r = r0; r < r1; ++r) {
            const float wc = A.w.at(r, L.c);
            const float unsat = sym ? sym_eval(A.T, L, st, sc, r, A.kappa, A.hard != 0, wc, kGrad, rows, lane)
                                    : level_eval(A.T, L, st, sc, r, A.kappa, A.hard != 0, wc, kGrad, W, lane);
            if (lane == 0 && A.unsat.data) A.unsat.at(r, L.c) = unsat;
            oa.add(r - r0, wc * unsat, lane);
        }
    }
    oa.flush(lane);
}

// The same with the restart's point and gradient sums in LDS, `slices` workgroups per restart
// (see cop_wg_kernel), for instances whose constraints are all big: every (constraint, restart)
// otherwise adds into its literals' gradients with device atomics on as many lines (random
// hybrid 500 x 100 points: 184 us a call).
template <bool kGrad>
__global__ void __launch_bounds__(768) cop_big_wg_kernel(LevelArgs A, int slices, int mode) {
    extern __shared__ __align__(16) float lds[];
    const int lane = threadIdx.x & 63, wib = wave_id(), wpb = blockDim.x >> 6;
    const int n = A.T.n_bool, m = A.T.n_real, nm = n + m;
    const int r = blockIdx.x / slices, slice = blockIdx.x - r * slices;
    double *ga = (double *)lds, *gb = ga + n;
    float *sa = kGrad ? (float *)(ga + nm) : lds, *sb = sa + n;
    float *const rows = sa + (nm + 3) / 4 * 4 + (size_t)wib * A.wave_floats;
    const LevelRows W = LevelRows::at(rows, A.lds_nodes, A.lds_slots);
    wg_load_point<kGrad>(A.a, A.b, r, n, nm, sa, ga);
    const LdsState st{sa, sb};
    const LdsScatter<double> sc{ga, gb};
    float oacc = 0.0f;
    for (int q = slice * wpb + wib; q < A.n_big; q += slices * wpb) {
        const LevelCtx L = level_ctx(A.T, A.lev, A.big_pos[q]);
        const float wc = A.w.at(r, L.c);
        float unsat;
        if (L.B.big == 2) {
            unsat = sym_eval(A.T, L, st, sc, r, A.kappa, A.hard != 0, wc, kGrad, rows, lane);
        } else {
            level_stage_nodes(A.T, L, W, lane);
            unsat = level_eval(A.T, L, st, sc, r, A.kappa, A.hard != 0, wc, kGrad, W, lane);
        }
        if (lane == 0) {
            if (A.unsat.data) A.unsat.at(r, L.c) = unsat;
            oacc += wc * unsat;
        }
    }
    wg_store<kGrad, false>(oacc, r, n, nm, ga, A.obj, A.ga, A.gb, mode, nullptr, nullptr);
}

// ------------------------------------------------------------------ small kernels
// out(r, v) (+)= stage[v * R + r]: the gradient accumulated restart-contiguous (see
// cop_launch) moved into the caller's view.
__global__ void unstage_kernel(View out, const float *stage, int R, int cols, int accumulate) {
    const int64_t n = (int64_t)R * cols;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int v = (int)(e / R), r = (int)(e - (int64_t)v * R);
        const float g = stage[e];
        if (!accumulate) out.at(r, v) = g;
        else if (g != 0.0f) atomic_add_f32(&out.at(r, v), g);
    }
}

// Zeroes the outputs of a call (objective and gradients) in one launch.
__global__ void zero_outputs_kernel(float *obj, int R, View ga, View gb) {
    const int64_t na = (int64_t)R * ga.cols, nb = (int64_t)R * gb.cols, n = R + na + nb;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < R) {
            if (obj) obj[i] = 0.0f;
        } else if (i < R + na) {
            ga.at((int)((i - R) / ga.cols), (int)((i - R) % ga.cols)) = 0.0f;
        } else {
            gb.at((int)((i - R - na) / gb.cols), (int)((i - R - na) % gb.cols)) = 0.0f;
        }
    }
}

__global__ void fill_f32_kernel(float *p, int64_t n, float value) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = value;
}

__global__ void fill_i32_kernel(int32_t *p, int64_t n, int32_t value) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = value;
}

// One block per restart: clamp / project step, gradient-map norm, zero the gradient.
__global__ void __launch_bounds__(1024) pgd_kernel(View a, View b, View ga, View gb, cptr<float> lo,
                                                  cptr<float> hi, float eta_a, float eta_b, float *gsq,
                                                  HalfSpaces hs) {
    extern __shared__ float sm[];
    const int r = blockIdx.x;
    float acc = 0.0f;
    for (int i = threadIdx.x; i < a.cols; i += blockDim.x) {
        const float x = a.at(r, i);
        const float y = x - eta_a * ga.at(r, i);
        const float p = y < -1.0f ? -1.0f : (y > 1.0f ? 1.0f : y);
        a.at(r, i) = p;
        const float g = (x - p) / eta_a;
        acc += g * g;
        ga.at(r, i) = 0.0f;
    }
    if (hs.n == 0) {
        for (int j = threadIdx.x; j < b.cols; j += blockDim.x) {
            const float x = b.at(r, j);
            const float y = x - eta_b * gb.at(r, j);
            const float p = y < lo[j] ? lo[j] : (y > hi[j] ? hi[j] : y);
            b.at(r, j) = p;
            const float g = (x - p) / eta_b;
            acc += g * g;
            gb.at(r, j) = 0.0f;
        }
    } else {
        const int m = b.cols;
        float *y = sm, *pb = sm + m, *ph = sm + 2 * m;
        for (int j = threadIdx.x; j < m; j += blockDim.x) {
            y[j] = b.at(r, j) - eta_b * gb.at(r, j);
            gb.at(r, j) = 0.0f;
        }
        project_dykstra(y, pb, ph, lo, hi, m, hs);
        for (int j = threadIdx.x; j < m; j += blockDim.x) {
            const float x = b.at(r, j), p = y[j];
            b.at(r, j) = p;
            const float g = (x - p) / eta_b;
            acc += g * g;
        }
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0 && gsq) gsq[r] = acc;
}

struct CheckArgs {
    TabView T;
    int32_t n_words;
    View a, b;
    uint32_t *sat_bits;
    int32_t *n_unsat;
};

// grid.x over 64-constraint groups (one wave each), grid.y over restarts. All latency: eight waves a
// SIMD (two registers more would leave seven).
__global__ void __launch_bounds__(256, 8) check_kernel(CheckArgs A) {
    const int lane = threadIdx.x & 63;
    const int64_t c64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    const GlobalState st{A.a, A.b};
    bool sat = false;
    if (c64 < A.T.n_cons) sat = walk_state(A.T, st, (int)c64, r);
    const uint64_t mask = __ballot(sat);
    const uint64_t valid = __ballot(c64 < A.T.n_cons);
    if (lane == 0 && valid) {
        const int64_t w0 = c64 >> 5;   // lane 0 holds a multiple of 64
        uint32_t *row = A.sat_bits + (int64_t)r * A.n_words;
        row[w0] = (uint32_t)mask;
        if (w0 + 1 < A.n_words) row[w0 + 1] = (uint32_t)(mask >> 32);
        atomicAdd(A.n_unsat + r, (int)__popcll(valid & ~mask));
    }
}

// ERWA update of Alg. "CLS with Annealing" for level t (1-based), one block per restart.
__global__ void __launch_bounds__(1024) erwa_kernel(int C, const uint32_t *bits, float *w, float *hist, int t, float rho,
                                                    float gamma, int tau, int normalize) {
    const int r = blockIdx.x, nw = (C + 31) >> 5;
    const bool update = (t % tau) == 0;
    float *wr = w + (int64_t)r * C, *hr = hist + (int64_t)r * C;
    const uint32_t *br = bits + (int64_t)r * nw;
    constexpr int kU = 8;   // elements a thread has in flight (one block per restart waits on latency)
    // (152 constraints at 25 restarts: 4.9 us with three powers a thread, 4.1 with one)
    const ErwaPow pw(gamma, rho, C > (int)blockDim.x);
    float ws = 0.0f;
    for (int c0 = threadIdx.x; c0 < C; c0 += kU * (int)blockDim.x) {
        float h[kU], wv[kU];
        uint32_t b[kU];
#pragma unroll
        for (int q = 0; q < kU; ++q) {
            const int c = c0 + q * (int)blockDim.x;
            h[q] = wv[q] = 0.0f;
            b[q] = 0;
            if (c < C) {
                h[q] = hr[c];
                wv[q] = wr[c];
                b[q] = br[c >> 5];
            }
        }
#pragma unroll
        for (int q = 0; q < kU; ++q) {
            const int c = c0 + q * (int)blockDim.x;
            if (c >= C) continue;
            const float viol = ((b[q] >> (c & 31)) & 1u) ? 0.0f : 1.0f;
            float hv = rho * h[q] + viol;
            if (update) {
                wv[q] *= pw(hv);
                hv = 1.0f;
                wr[c] = wv[q];
            }
            hr[c] = hv;
            ws += wv[q];
        }
    }
    ws = block_sum(ws);
    if (update && normalize) {
        const float scale = (float)C / ws;
        for (int c0 = threadIdx.x; c0 < C; c0 += kU * (int)blockDim.x) {
            float wv[kU];
#pragma unroll
            for (int q = 0; q < kU; ++q) {
                const int c = c0 + q * (int)blockDim.x;
                wv[q] = c < C ? wr[c] : 0.0f;
            }
#pragma unroll
            for (int q = 0; q < kU; ++q) {
                const int c = c0 + q * (int)blockDim.x;
                if (c < C) wr[c] = wv[q] * scale;
            }
        }
    }
}

__global__ void verdict_kernel(View a, int8_t *x, const int32_t *n_unsat, int32_t *verdict) {
    const int r = blockIdx.x;
    if (threadIdx.x == 0) verdict[r] = n_unsat[r] == 0 ? 1 : 0;
    if (x)
        for (int i = threadIdx.x; i < a.cols; i += blockDim.x) x[(int64_t)r * a.cols + i] = a.at(r, i) < 0.0f ? -1 : 1;
}

// ------------------------------------------------------------------ host side

static fsmt_status check_view(const fsmt_view &v, int rows, int cols, const char *name, bool allow_bcast = false) {
    if (cols > 0 && rows > 0 && !v.data) return set_error(FSMT_EINVAL, "%s: null data", name);
    if (v.rows != rows || v.cols != cols)
        return set_error(FSMT_EINVAL, "%s: shape [%d][%d], expected [%d][%d]", name, v.rows, v.cols, rows, cols);
    if (v.stride_v < 0 || v.stride_r < 0) return set_error(FSMT_EINVAL, "%s: negative stride", name);
    if (cols > 1 && v.stride_v == 0) return set_error(FSMT_EINVAL, "%s: zero column stride", name);
    if (rows > 1 && v.stride_r == 0 && !allow_bcast) return set_error(FSMT_EINVAL, "%s: zero row stride", name);
    return FSMT_OK;
}

fsmt_status check_device_ptr(const void *p, int device, const char *name) {
    if (!p) return FSMT_OK;
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        return set_error(FSMT_EINVAL, "%s: not a device pointer", name);
    }
    if (at.type != hipMemoryTypeDevice && at.type != hipMemoryTypeManaged)
        return set_error(FSMT_EINVAL, "%s: not device memory", name);
    if (at.device != device) return set_error(FSMT_EINVAL, "%s: on device %d, handle on %d", name, at.device, device);
    return FSMT_OK;
}

fsmt_status select_device(const fsmt_xbdd *h) {
    if (h->host_only) return set_error(FSMT_EINVAL, "handle was compiled host-only");
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess) return set_error(FSMT_EHIP, "hipGetDevice failed");
    if (cur != h->device) return set_error(FSMT_EINVAL, "current device %d differs from the handle's device %d", cur, h->device);
    return FSMT_OK;
}

HalfSpaces halfspaces_of(const fsmt_xbdd *h) {
    return HalfSpaces{as_cptr(h->d.hs_ptr), as_cptr(h->d.hs_var), as_cptr(h->d.hs_coef), as_cptr(h->d.hs_rhs),
                      as_cptr(h->d.hs_inv), as_cptr(h->d.hs_cstart), h->n_hs, h->hs_nnz, h->n_hs_colors,
                      h->hs_separable, h->hs_two_terms};
}

static fsmt_status launch_status(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(FSMT_EHIP, "%s: %s", what, hipGetErrorString(e));
    return FSMT_OK;
}

template <bool kGrad, int kCF>
static void launch_cop_v(int msg, dim3 g, dim3 bl, size_t lds, hipStream_t st, const CopArgs &A) {
    if (msg == kMsgSmall) hipLaunchKernelGGL((cop_kernel<kGrad, kMsgSmall, kCF>), g, bl, 0, st, A);
    else if (msg == kMsgMedium) hipLaunchKernelGGL((cop_kernel<kGrad, kMsgMedium, kCF>), g, bl, 0, st, A);
    else if (msg == kMsgLarge) hipLaunchKernelGGL((cop_kernel<kGrad, kMsgLarge, kCF>), g, bl, 0, st, A);
    else hipLaunchKernelGGL((cop_kernel<kGrad, kMsgLds, kCF>), g, bl, lds, st, A);
}
template <bool kGrad>
static void launch_cop(int cf, int msg, dim3 g, dim3 bl, size_t lds, hipStream_t st, const CopArgs &A) {
    if (cf == 0) launch_cop_v<kGrad, 0>(msg, g, bl, lds, st, A);
    else if (cf == 1) launch_cop_v<kGrad, 1>(msg, g, bl, lds, st, A);
    else if (cf == 2) launch_cop_v<kGrad, 2>(msg, g, bl, lds, st, A);
    else if (cf == 3) launch_cop_v<kGrad, 3>(msg, g, bl, lds, st, A);
    else launch_cop_v<kGrad, 4>(msg, g, bl, lds, st, A);
}

size_t lds_opt_in(const std::vector<const void *> &fns, int device) {
    int v = 0;
    size_t b = 65536, stat = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, device) == hipSuccess && (size_t)v > b) b = (size_t)v;
    else (void)hipGetLastError();
    for (const void *f : fns) {
        hipFuncAttributes fa{};
        if (hipFuncGetAttributes(&fa, f) == hipSuccess) stat = std::max(stat, (size_t)fa.sharedSizeBytes);
        else (void)hipGetLastError();
    }
    bool ok = true;
    for (const void *f : fns)
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(b - stat)) != hipSuccess) {
            (void)hipGetLastError();
            ok = false;
        }
    return (ok ? b : 65536) - stat;
}

size_t LdsBudget::of(int device, std::vector<const void *> (*fns)()) {
    if (device < 0 || device >= kMaxDevices) return lds_opt_in(fns(), device);
    std::call_once(once[device], [&] { bytes[device] = lds_opt_in(fns(), device); });
    return bytes[device];
}

static int blocks_for(int64_t n, int threads, int cap = 4096) {
    int64_t b = (n + threads - 1) / threads;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

// Restarts of one launch with a workgroup each: the runtime drops what a grid has past 2^32
// threads without an error.
static int rows_per_launch(int R, int threads) { return (int)std::min<int64_t>(R, (int64_t)UINT32_MAX / threads); }
// Rows r0 .. of a view.
static View rows_from(View v, int64_t r0) {
    if (v.data) v.data += r0 * v.sr;
    return v;
}

fsmt_status fill_i32(int32_t *p, int64_t n, int32_t value, hipStream_t st) {
    if (!p || n <= 0) return FSMT_OK;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, p, n, value);
    return launch_status("fill");
}

fsmt_status fill_f32(float *p, int64_t n, float value, hipStream_t st) {
    if (!p || n <= 0) return FSMT_OK;
    hipLaunchKernelGGL(fill_f32_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, p, n, value);
    return launch_status("fill");
}

template <int kCF>
static const void *cop_wg_fn_cf(bool grad, int msg, bool wide, bool mixed) {
    if (mixed)
        return grad ? (const void *)cop_wg_kernel<true, kMsgSmall, kCF, double, true>
                    : (const void *)cop_wg_kernel<false, kMsgSmall, kCF, double, true>;
    if (msg == kMsgSmall)
        return !grad  ? (const void *)cop_wg_kernel<false, kMsgSmall, kCF, float>
               : wide ? (const void *)cop_wg_kernel<true, kMsgSmall, kCF, double>
                      : (const void *)cop_wg_kernel<true, kMsgSmall, kCF, float>;
    return !grad  ? (const void *)cop_wg_kernel<false, kMsgLds, kCF, float>
           : wide ? (const void *)cop_wg_kernel<true, kMsgLds, kCF, double>
                  : (const void *)cop_wg_kernel<true, kMsgLds, kCF, float>;
}
static const void *cop_wg_fn(bool grad, int msg, int cf, bool wide, bool mixed = false) {
    return cf == 0   ? cop_wg_fn_cf<0>(grad, msg, wide, mixed)
           : cf == 1 ? cop_wg_fn_cf<1>(grad, msg, wide, mixed)
           : cf == 2 ? cop_wg_fn_cf<2>(grad, msg, wide, mixed)
           : cf == 3 ? cop_wg_fn_cf<3>(grad, msg, wide, mixed)
                     : cop_wg_fn_cf<4>(grad, msg, wide, mixed);
}

static const void *level_kernel_fn(bool grad) {
    return grad ? (const void *)cop_level_kernel<true> : (const void *)cop_level_kernel<false>;
}
static const void *big_wg_fn(bool grad) {
    return grad ? (const void *)cop_big_wg_kernel<true> : (const void *)cop_big_wg_kernel<false>;
}

// Dynamic LDS the one-restart-per-workgroup kernels may take, and the kernels of big diagrams.
static std::vector<const void *> cop_wg_fns() {
    std::vector<const void *> fns;
    for (int grad = 0; grad < 2; ++grad)
        for (int msg : {kMsgSmall, kMsgLds})
            for (int cf = 0; cf < 5; ++cf)
                for (int wide = 0; wide < 3; ++wide) fns.push_back(cop_wg_fn(grad != 0, msg, cf, wide == 1, wide == 2));
    return fns;
}
static std::vector<const void *> big_fns() {
    return {level_kernel_fn(false), level_kernel_fn(true), big_wg_fn(false), big_wg_fn(true)};
}
static size_t lds_wg_budget(int device) {
    static LdsBudget B;
    return B.of(device, cop_wg_fns);
}
static size_t lds_big_budget(int device) {
    static LdsBudget B;
    return B.of(device, big_fns);
}

// Geometry of the one-restart-per-workgroup kernel, or slices = 0 where it does not apply: a
// state beyond LDS, or a register message store of the larger bounds.
struct WgGeom {
    int slices = 0, waves = 0, mode = kStore;
    bool wide = false, mixed = false;
    size_t lds = 0;
};
static WgGeom big_geom(const fsmt_xbdd *h, int R, bool grad, size_t level_wave_bytes, int n_cu) {
    WgGeom G;
    const size_t nm = (size_t)h->n_bool + h->n_real, state = (nm * (grad ? 12 : 4) + 31) / 16 * 16;
    // with few restarts the level kernel spreads the constraints over more workgroups (random
    // hybrid 100 at 7 points: 17 us a call against 39 here)
    if (R < 32 || h->n_big == 0 || h->n_big != h->n_cons || nm == 0) return G;
    const size_t cap = lds_big_budget(h->device);
    if (state + 4 * level_wave_bytes > cap) return G;
    G.waves = (int)std::min<size_t>(12, (cap - state) / level_wave_bytes);
    // a wave has about four constraints where the restarts do not fill the device
    const int64_t s = std::min<int64_t>(n_cu / std::max(1, R), h->n_big / (4 * G.waves));
    G.slices = (int)std::max<int64_t>(1, s);
    G.mode = G.slices == 1 ? kStore : kAdd;
    G.lds = state + (size_t)G.waves * level_wave_bytes;
    return G;
}
static WgGeom wg_geom(const fsmt_xbdd *h, int R, bool grad, int msg, size_t wave_bytes, int n_cu) {
    WgGeom G;
    const int64_t tasks = sweep_tasks(h), nm = (int64_t)h->n_bool + h->n_real;
    if (tasks == 0 || nm == 0 || h->n_big == h->n_cons || (msg != kMsgSmall && msg != kMsgLds)) return G;
    const size_t cap = lds_wg_budget(h->device);
    // waves of a workgroup: one per task up to 16, fewer where the message columns need the LDS
    auto waves_of = [&](size_t state) -> int {
        if (state + wave_bytes > cap) return 0;
        const int64_t w = std::min<int64_t>(16, tasks);
        return wave_bytes ? (int)std::min<int64_t>(w, (int64_t)((cap - state) / wave_bytes)) : (int)w;
    };
    size_t state = (size_t)nm * 4 * (grad ? 2 : 1);
    G.waves = waves_of(state);
    if (grad) {
        const int w = waves_of((size_t)nm * 12);
        if (w > 0 && 2 * w >= G.waves) {
            G.wide = true;
            G.waves = w;
            state = (size_t)nm * 12;
        }
    }
    if (G.waves < std::min<int64_t>(4, tasks)) {
        // the Booleans stay in global memory where most of them are cells' own
        state = (size_t)h->n_real * (grad ? 12 : 4);
        G = WgGeom{};
        if (msg != kMsgSmall || h->n_real == 0 || (int64_t)h->n_free * 8 > h->n_bool || state > cap) return G;
        G.mixed = G.wide = true;
        G.waves = (int)std::min<int64_t>(16, tasks);
    }
    // Bucket tasks on many nearly empty buckets fill few of a wave's lanes with one restart; where
    // the restarts fill the lanes instead and the message columns leave a workgroup few waves, the
    // lane kernel is ahead (600 constraints of 587 shapes, 2,048 restarts: 7.8 ms a gradient
    // against 9.2 ms here; 256 restarts 1.20 against 1.16).
    if (G.waves <= 4 && wave_bytes && R >= 4 * n_cu && (int64_t)h->n_cons * 16 < h->n_pos) return WgGeom{};
    // One slice (the call is one launch) unless the restarts leave CUs idle and one workgroup's
    // rounds (sweep_us) cost more than the zeroing launch and the atomics of several. Several slices
    // then leave a wave at most one task. One restart, us a gradient with a task a wave / four tasks
    // a wave / one slice: 4,000 three-literal clauses of 153 shapes 13.6 / 35 / -, 6,000
    // two-selector ITEs 13.8 / 59 / -, scheduling 200 x 10 (65 tasks) 15 / - / 11.
    // Large instances write rows, which device atomics on every variable from every slice would
    // cost more than.
    const bool large = tasks >= (int64_t)8 * n_cu;
    G.slices = 1;
    if (R < n_cu) {
        int64_t s = n_cu / R;
        if (!large) s = sweep_us(h, G.waves) <= kSweepUsMin ? 1 : std::min<int64_t>(s, 2 * tasks / G.waves);
        if (s >= 8) s = s / 8 * 8;
        G.slices = (int)std::max<int64_t>(1, s);
    }
    // with more restarts than the CUs hold at 16 waves each, smaller workgroups: a wave runs several
    // tasks after one load of the point, about 10 us (20 rectangles, 16,384 restarts: 130 us a
    // gradient with 7 waves, 58 with one; scheduling 200 x 10, 2,048 restarts: 65 with 16, 46 with
    // four; 2,824 bucket tasks, 2,048 restarts: 13.2 ms with 16, 16.4 with four)
    const int64_t few = (int64_t)std::ceil(sweep_us(h, 1) / 10.0);
    G.waves = (int)std::min<int64_t>(G.waves, std::max<int64_t>({1, (int64_t)32 * n_cu / R, few}));
    G.mode = G.slices == 1 ? kStore : (grad && large) ? kRows : kAdd;
    G.lds = (state + (size_t)G.waves * wave_bytes + 15) / 16 * 16;
    return G;
}

static fsmt_status cop_launch(const fsmt_xbdd *h, fsmt_view a, fsmt_view b, double kappa, fsmt_view w, float *obj,
                              fsmt_view unsat, fsmt_view ga, fsmt_view gb, bool grad, int32_t flags, hipStream_t st) {
    const int R = a.rows;
    fsmt_status rc;
    if (!h) return set_error(FSMT_EINVAL, "null handle");
    if (R <= 0) return set_error(FSMT_EINVAL, "a: no rows");
    if ((rc = check_view(a, R, h->n_bool, "a"))) return rc;
    if ((rc = check_view(b, R, h->n_real, "b"))) return rc;
    if (w.rows == 1 && R > 1 && w.stride_r == 0) {
        if ((rc = check_view(w, 1, h->n_cons, "w"))) return rc;
    } else if ((rc = check_view(w, R, h->n_cons, "w"))) {
        return rc;
    }
    if (unsat.data && (rc = check_view(unsat, R, h->n_cons, "unsat"))) return rc;
    if (grad) {
        if ((rc = check_view(ga, R, h->n_bool, "grad_a"))) return rc;
        if ((rc = check_view(gb, R, h->n_real, "grad_b"))) return rc;
    }
    if (!(kappa >= 0.0)) return set_error(FSMT_EINVAL, "kappa must be in [0, +inf]");
    if ((rc = select_device(h))) return rc;
    const void *ptrs[] = {a.data, b.data, w.data, obj, unsat.data, grad ? ga.data : nullptr, grad ? gb.data : nullptr};
    const char *names[] = {"a", "b", "w", "obj", "unsat", "grad_a", "grad_b"};
    for (int i = 0; i < 7; ++i)
        if ((rc = check_device_ptr(ptrs[i], h->device, names[i]))) return rc;

    // one lane per constraint for the small diagrams, one wavefront per (constraint,
    // restart) for the big ones
    const int NN = h->small_max_nodes + 2, SS = std::max(h->small_max_slots, 1);
    const int msg = msg_variant(h->small_max_nodes, h->small_max_slots, lds_store(h), h->all_inline);
    const size_t wave_bytes = msg == kMsgLds ? WaveScratch::bytes(NN, SS) : 0;
    const int wpb = wave_bytes ? (int)std::max<size_t>(1, std::min<size_t>(4, 65536 / wave_bytes)) : 4;
    const size_t level_wave_bytes = big_wave_floats(h->big_max_nodes, h->big_max_slots, h->sym_max) * sizeof(float);
    if (h->n_big > 0 && level_too_large(h->big_max_nodes, std::max(h->big_max_slots, 1)))
        return set_error(FSMT_ELIMIT, "diagram too large for the level-synchronous pass (%d nodes, %d slots)",
                         h->big_max_nodes, h->big_max_slots);

    // The restart's state in LDS, one or more workgroups per restart (cop_wg_kernel), where it
    // fits. Otherwise: with several restarts in a wavefront's lanes, the lanes of one
    // constraint add into the same variable of consecutive restarts. Device-scope float
    // atomics are performed past the per-XCD L2, one memory transaction per cache line touched,
    // so when the caller's gradient rows are not restart-contiguous the sums go to a
    // restart-contiguous stage ([n + m][R], one line per variable and 16 restarts) and are moved
    // into the caller's views afterwards, on instances of at least 8 tasks (64-position groups)
    // per CU (on smaller ones the atomics cost little and the extra allocation and launches
    // would dominate the call).
    const int n = h->n_bool, m = h->n_real;
    int n_cu = 256;
    (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, h->device);
    const int cf = closed_level(h);
    WgGeom wg = wg_geom(h, R, grad, msg, wave_bytes, n_cu);
    if (wg.mode == kRows) {
        // no allocation while the stream is being captured: the slices add with atomics
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();
        else if (cap != hipStreamCaptureStatusNone) wg.mode = kAdd;
    }
    WgGeom big = big_geom(h, R, grad, level_wave_bytes, n_cu);
    // accumulation adds with atomics in every path: calls on several streams that accumulate into
    // one buffer add up
    const int accumulate = flags & FSMT_ACCUMULATE;
    if (accumulate && wg.mode == kStore) wg.mode = kAdd;
    if (accumulate && big.mode == kStore) big.mode = kAdd;
    const bool large = sweep_tasks(h) >= (int64_t)8 * n_cu;
    const bool stage = !wg.slices && !big.slices && grad && large && R >= 4 && R <= 64 && (int64_t)(n + m) * R > 0 &&
                       !(ga.stride_r == 1 && gb.stride_r == 1);
    struct Stage {   // freed stream-ordered after whatever the call enqueued
        float *p = nullptr;
        hipStream_t st = nullptr;
        ~Stage() {
            if (p) (void)hipFreeAsync(p, st);
        }
    } sg;
    sg.st = st;
    const int n_row = wg.mixed ? 0 : n;   // Booleans in the workgroups' rows
    if (wg.mode == kRows) {   // objectives (double) first, then the gradient rows
        const size_t bytes = (size_t)R * wg.slices * (sizeof(double) + sizeof(float) * (size_t)(n_row + m));
        if (hipMallocAsync((void **)&sg.p, bytes, st) != hipSuccess) {
            (void)hipGetLastError();
            sg.p = nullptr;
            wg.mode = kAdd;   // without the rows the slices add with atomics
        }
    }
    const bool rows = wg.slices && wg.mode == kRows;
    if (stage) {
        if (hipMallocAsync((void **)&sg.p, sizeof(float) * (size_t)(n + m) * R, st) != hipSuccess) {
            (void)hipGetLastError();
            sg.p = nullptr;
            return set_error(FSMT_ENOMEM, "gradient stage allocation failed");
        }
        if ((rc = fill_f32(sg.p, (int64_t)(n + m) * R, 0.0f, st))) return rc;
    }
    float *const sbuf = sg.p;
    // the workgroups store the outputs
    const bool whole = (wg.slices && wg.mode != kAdd) || (big.slices && big.mode == kStore);
    const bool zero_free = wg.mixed && grad && h->n_free > 0;   // added with atomics
    if (!accumulate && (!whole || zero_free)) {
        const bool zg = grad && !stage;
        const bool za = zg && (!wg.mixed || zero_free), zb = zg && !whole;
        const int64_t cnt = R + (za ? (int64_t)R * n : 0) + (zb ? (int64_t)R * m : 0);
        hipLaunchKernelGGL(zero_outputs_kernel, dim3(blocks_for(cnt, 256)), dim3(256), 0, st, obj, R,
                           za ? View::of(ga) : View{}, zb ? View::of(gb) : View{});
        if ((rc = launch_status("zero outputs"))) return rc;
    }
    if (sweep_tasks(h) == 0) {
        if (stage) {
            hipLaunchKernelGGL(unstage_kernel, dim3(blocks_for((int64_t)R * n, 256)), dim3(256), 0, st, View::of(ga),
                               (const float *)sbuf, R, n, accumulate);
            hipLaunchKernelGGL(unstage_kernel, dim3(blocks_for((int64_t)R * m, 256)), dim3(256), 0, st, View::of(gb),
                               (const float *)(sbuf + (size_t)n * R), R, m, accumulate);
        }
        return launch_status("gradient unstage");
    }

    CopArgs A{};
    A.T = TabView::of(h);
    A.R = R;
    if (R <= 64) {
        int rp = 1, lg = 0;
        while (rp < R) { rp <<= 1; ++lg; }
        A.R_pad = rp;
        A.log2_rpad = lg;
        A.n_tasks = (int64_t)h->n_pos * rp / 64;
    } else {
        A.R_pad = (R + 63) / 64 * 64;
        A.log2_rpad = 0;
        A.n_tasks = (int64_t)h->n_pos * (A.R_pad / 64);
    }
    A.a = View::of(a);
    A.b = View::of(b);
    A.w = View::of(w);
    A.unsat = View::of(unsat);
    A.ga = grad ? View::of(ga) : View{};
    A.gb = grad ? View::of(gb) : View{};
    if (stage) {
        A.ga = View{as_gptr(sbuf), R, n, 1, R};
        A.gb = View{as_gptr(sbuf + (size_t)n * R), R, m, 1, R};
    }
    A.obj = obj;
    A.kappa = kappa;
    A.hard = std::isinf(kappa) ? 1 : 0;
    A.lds_nodes = h->small_max_nodes;
    A.lds_slots = SS;
    const int64_t max_waves = 256 * 32;
    const int64_t waves = std::min<int64_t>(A.n_tasks, max_waves);
    const int blocks = (int)((waves + wpb - 1) / wpb);
    const size_t lds = wave_bytes * wpb;
    const dim3 g(blocks), bl(64 * wpb);
    if (wg.slices) {
        double *const opart = rows ? (double *)sbuf : nullptr;
        float *const part = rows ? (float *)(opart + (size_t)R * wg.slices) : nullptr;
        // several slices only below a restart a CU: then one launch has all of them
        const int rows_max = wg.slices > 1 ? R : rows_per_launch(R, 64 * wg.waves);
        for (int r0 = 0, nr; r0 < R; r0 += nr) {
            nr = std::min(R - r0, rows_max);
            CopArgs *P = &A, B;
            if (nr < R) {
                P = &(B = A);
                for (View *v : {&B.a, &B.b, &B.w, &B.unsat, &B.ga, &B.gb}) *v = rows_from(*v, r0);
                if (B.obj) B.obj += r0;
            }
            void *args[] = {(void *)P, (void *)&wg.slices, (void *)&wg.mode, (void *)&accumulate, (void *)&part, (void *)&opart};
            const hipError_t le = hipLaunchKernel(cop_wg_fn(grad, msg, cf, wg.wide, wg.mixed), dim3((unsigned)(nr * wg.slices)),
                                                  dim3(64 * wg.waves), args, wg.lds, st);
            if (le != hipSuccess) return set_error(FSMT_EHIP, "cop kernel (state in LDS): %s", hipGetErrorString(le));
        }
        if (rows) {
            hipLaunchKernelGGL(sum_rows_kernel, dim3((n_row + m + 63) / 64, R), dim3(1024), 0, st, (const float *)part,
                               (const double *)opart, wg.slices, n_row, m, View::of(ga), View::of(gb), obj, accumulate);
            if ((rc = launch_status("gradient rows"))) return rc;
        }
    } else if (h->n_big < h->n_cons) {
        if (A.n_tasks > 0) {
            const int lcf = untiled_level(cf, h->n_window > 0);
            if (grad) launch_cop<true>(lcf, msg, g, bl, lds, st, A);
            else launch_cop<false>(lcf, msg, g, bl, lds, st, A);
            if ((rc = launch_status("cop kernel"))) return rc;
        }
        if (h->n_tiles > 0) {
            const int chunk = tile_chunk((int64_t)R * h->n_tiles, n_cu), chunks = (h->n_tiles + chunk - 1) / chunk;
            const dim3 tg((unsigned)std::min<int64_t>(((int64_t)R * chunks + 3) / 4, kMaxBlocks)), tb(256);
            if (grad) hipLaunchKernelGGL(cop_tile_kernel<true>, tg, tb, 0, st, A, chunks);
            else hipLaunchKernelGGL(cop_tile_kernel<false>, tg, tb, 0, st, A, chunks);
            if ((rc = launch_status("cop tile kernel"))) return rc;
        }
    }
    if (h->n_big > 0) {
        LevelArgs L{};
        L.T = A.T;
        L.lev = as_cptr(h->d.lev);
        L.big_pos = as_cptr(h->d.big_pos);
        L.n_big = h->n_big;
        L.R = R;
        L.a = A.a;
        L.b = A.b;
        L.w = A.w;
        L.unsat = A.unsat;
        L.ga = A.ga;
        L.gb = A.gb;
        L.obj = obj;
        L.kappa = kappa;
        L.hard = A.hard;
        L.lds_nodes = h->big_max_nodes;
        L.lds_slots = std::max(h->big_max_slots, 1);
        L.wave_floats = (int32_t)(level_wave_bytes / sizeof(float));
        L.chunk = level_chunk((int64_t)h->n_big * R, n_cu);
        if (big.slices) {
            const int rows_max = big.slices > 1 ? R : rows_per_launch(R, 64 * big.waves);
            for (int r0 = 0, nr; r0 < R; r0 += nr) {
                nr = std::min(R - r0, rows_max);
                LevelArgs B = L;
                for (View *v : {&B.a, &B.b, &B.w, &B.unsat, &B.ga, &B.gb}) *v = rows_from(*v, r0);
                if (B.obj) B.obj += r0;
                void *args[] = {(void *)&B, (void *)&big.slices, (void *)&big.mode};
                const hipError_t le = hipLaunchKernel(big_wg_fn(grad), dim3((unsigned)(nr * big.slices)), dim3(64 * big.waves),
                                                      args, big.lds, st);
                if (le != hipSuccess) return set_error(FSMT_EHIP, "cop kernel (big diagrams): %s", hipGetErrorString(le));
            }
            return FSMT_OK;
        }
        const int lwpb = (int)std::max<size_t>(1, std::min<size_t>(4, 65536 / level_wave_bytes));
        if (level_wave_bytes > 65536 && level_wave_bytes > lds_big_budget(h->device))
            return set_error(FSMT_ELIMIT, "a big diagram's rows (%zu B) exceed the device's LDS", level_wave_bytes);
        const int64_t ltasks = (int64_t)h->n_big * ((R + L.chunk - 1) / L.chunk);
        const int lblocks = (int)std::min<int64_t>((ltasks + lwpb - 1) / lwpb, (int64_t)256 * 16);
        if (grad)
            hipLaunchKernelGGL(cop_level_kernel<true>, dim3(lblocks), dim3(64 * lwpb), level_wave_bytes * lwpb, st, L);
        else
            hipLaunchKernelGGL(cop_level_kernel<false>, dim3(lblocks), dim3(64 * lwpb), level_wave_bytes * lwpb, st, L);
        if ((rc = launch_status("cop level kernel"))) return rc;
    }
    if (stage) {
        hipLaunchKernelGGL(unstage_kernel, dim3(blocks_for((int64_t)R * n, 256)), dim3(256), 0, st, View::of(ga),
                           (const float *)sbuf, R, n, accumulate);
        hipLaunchKernelGGL(unstage_kernel, dim3(blocks_for((int64_t)R * m, 256)), dim3(256), 0, st, View::of(gb),
                           (const float *)(sbuf + (size_t)n * R), R, m, accumulate);
        if ((rc = launch_status("gradient unstage"))) return rc;
    }
    return FSMT_OK;
}

}  // namespace fsmt

using namespace fsmt;

extern "C" {

fsmt_status cop_forward(const fsmt_xbdd *h, fsmt_view a, fsmt_view b, double kappa, fsmt_view w, float *obj,
                        fsmt_view unsat, int32_t flags, void *stream) {
    clear_error();
    if (!obj) return set_error(FSMT_EINVAL, "obj is required");
    return cop_launch(h, a, b, kappa, w, obj, unsat, fsmt_view{}, fsmt_view{}, false, flags, (hipStream_t)stream);
}

fsmt_status cop_backward(const fsmt_xbdd *h, fsmt_view a, fsmt_view b, double kappa, fsmt_view w, float *obj,
                         fsmt_view grad_a, fsmt_view grad_b, int32_t flags, void *stream) {
    clear_error();
    return cop_launch(h, a, b, kappa, w, obj, fsmt_view{}, grad_a, grad_b, true, flags, (hipStream_t)stream);
}

fsmt_status pgd_step(const fsmt_xbdd *h, fsmt_view a, fsmt_view b, fsmt_view grad_a, fsmt_view grad_b, float eta_a,
                     float eta_b, float *gmap_sq, int32_t flags, void *stream) {
    clear_error();
    (void)flags;
    if (!h) return set_error(FSMT_EINVAL, "null handle");
    const int R = a.rows;
    fsmt_status rc;
    if (R <= 0) return set_error(FSMT_EINVAL, "a: no rows");
    if ((rc = check_view(a, R, h->n_bool, "a")) || (rc = check_view(b, R, h->n_real, "b")) ||
        (rc = check_view(grad_a, R, h->n_bool, "grad_a")) || (rc = check_view(grad_b, R, h->n_real, "grad_b")))
        return rc;
    if (!(eta_a > 0.0f) || !(eta_b > 0.0f)) return set_error(FSMT_EINVAL, "step sizes must be positive");
    if ((rc = select_device(h))) return rc;
    const void *ptrs[] = {a.data, b.data, grad_a.data, grad_b.data, gmap_sq};
    const char *names[] = {"a", "b", "grad_a", "grad_b", "gmap_sq"};
    for (int i = 0; i < 5; ++i)
        if ((rc = check_device_ptr(ptrs[i], h->device, names[i]))) return rc;
    const HalfSpaces hs = halfspaces_of(h);
    const size_t lds = hs.n ? (size_t)(2 * h->n_real + hs.nnz) * sizeof(float) : 0;
    if (lds > 65536) return set_error(FSMT_ELIMIT, "projection onto %d half-spaces over %d reals exceeds LDS", hs.n, h->n_real);
    // as many threads as the swept half-spaces or the variables can use
    const int64_t per = std::max<int64_t>(hs.n && !hs.separable ? hs.n : 0, ((int64_t)h->n_bool + h->n_real) / 4);
    const int threads = (int)std::max<int64_t>(256, std::min<int64_t>(1024, (per + 63) / 64 * 64));
    const int rows_max = rows_per_launch(R, threads);
    for (int r0 = 0; r0 < R; r0 += rows_max) {
        hipLaunchKernelGGL(pgd_kernel, dim3(std::min(R - r0, rows_max)), dim3(threads), lds, (hipStream_t)stream,
                           rows_from(View::of(a), r0), rows_from(View::of(b), r0), rows_from(View::of(grad_a), r0),
                           rows_from(View::of(grad_b), r0), as_cptr(h->d.real_lo), as_cptr(h->d.real_hi), eta_a, eta_b,
                           gmap_sq ? gmap_sq + r0 : nullptr, hs);
        if ((rc = launch_status("pgd kernel"))) return rc;
        if (rows_max > R - r0) break;   // r0 + rows_max may pass INT32_MAX
    }
    return FSMT_OK;
}

fsmt_status round_and_check(const fsmt_xbdd *h, fsmt_view a, fsmt_view b, int8_t *x, uint32_t *sat_bits,
                            int32_t *n_unsat, int32_t *verdict, void *stream) {
    clear_error();
    if (!h) return set_error(FSMT_EINVAL, "null handle");
    const int R = a.rows;
    fsmt_status rc;
    if (R <= 0) return set_error(FSMT_EINVAL, "a: no rows");
    if ((rc = check_view(a, R, h->n_bool, "a")) || (rc = check_view(b, R, h->n_real, "b"))) return rc;
    if (!sat_bits || !n_unsat || !verdict) return set_error(FSMT_EINVAL, "sat_bits, n_unsat and verdict are required");
    if (R > 65535) return set_error(FSMT_ELIMIT, "at most 65535 rows");
    if ((rc = select_device(h))) return rc;
    const void *ptrs[] = {a.data, b.data, x, sat_bits, n_unsat, verdict};
    const char *names[] = {"a", "b", "x", "sat_bits", "n_unsat", "verdict"};
    for (int i = 0; i < 6; ++i)
        if ((rc = check_device_ptr(ptrs[i], h->device, names[i]))) return rc;
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(blocks_for(R, 256)), dim3(256), 0, st, n_unsat, (int64_t)R, 0);
    if ((rc = launch_status("fill"))) return rc;
    CheckArgs A{};
    A.T = TabView::of(h);
    A.n_words = (h->n_cons + 31) / 32;
    A.a = View::of(a);
    A.b = View::of(b);
    A.sat_bits = sat_bits;
    A.n_unsat = n_unsat;
    if (h->n_cons > 0) {
        const int gx = (int)((h->n_cons + 255) / 256);
        hipLaunchKernelGGL(check_kernel, dim3(gx, R), dim3(256), 0, st, A);
        if ((rc = launch_status("check kernel"))) return rc;
    }
    hipLaunchKernelGGL(verdict_kernel, dim3(R), dim3(256), 0, st, View::of(a), x, n_unsat, verdict);
    return launch_status("verdict kernel");
}

fsmt_status erwa_update(const fsmt_xbdd *h, int32_t R, const uint32_t *sat_bits, float *w, float *hist, int32_t level,
                        float rho, float gamma, int32_t tau, int32_t normalize, void *stream) {
    clear_error();
    if (!h) return set_error(FSMT_EINVAL, "null handle");
    if (R <= 0 || R > 65535) return set_error(FSMT_EINVAL, "R must be in [1, 65535]");
    if (!sat_bits || !w || !hist) return set_error(FSMT_EINVAL, "null pointer");
    if (tau < 1 || level < 1 || !(gamma > 0.0f) || !(rho >= 0.0f)) return set_error(FSMT_EINVAL, "bad ERWA parameters");
    fsmt_status rc;
    if ((rc = select_device(h))) return rc;
    const void *ptrs[] = {sat_bits, w, hist};
    const char *names[] = {"sat_bits", "w", "hist"};
    for (int i = 0; i < 3; ++i)
        if ((rc = check_device_ptr(ptrs[i], h->device, names[i]))) return rc;
    if (h->n_cons == 0) return FSMT_OK;
    hipLaunchKernelGGL(erwa_kernel, dim3(R), dim3(1024), 0, (hipStream_t)stream, h->n_cons, sat_bits, w, hist, level, rho,
                       gamma, tau, normalize);
    return launch_status("erwa kernel");
}

}  // extern "C"
