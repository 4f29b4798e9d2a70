// Sweep of the tile sets (see TileSet): one wave runs consecutive 8 x 8 tiles of one restart,
// lane = 8 * row + column. A run of tiles shares its column group (tiles are sorted by it), so
// a lane keeps its column's values and the column's gradient in registers; the row's gradient
// is summed over the 8 lanes of a row by DPP and added with one scatter instruction a tile.
//
// What bounds it: VALU issue, eight half_erfc (about 17 instructions and two transcendentals
// each) of about 330 instructions a tile of kind 0: 1,200 rectangles at 16 restarts take 112 us
// an iteration, level ends included (336 us with the buckets' guarded disjunctions). Against the
// guarded-disjunction task it replaces: no atom records (264 bytes a constraint; here the constraint's id and weight), one
// LDS scatter instruction instead of six, 64-bit linear forms once per dimension. 8 x 8 tiles
// keep the triangle i < j of a pair set 99 % full at 1,200 entities (92 % at 150; 64 columns
// a row would leave half of the lanes idle there) and a row's lanes within one DPP group.
#pragma once
#include "eval_task.hpp"

namespace fsmt {

constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor7 = 0x141, kDppDown4 = 0x104;

// Sums of four values over each group of 8 lanes: lane j < 4 of the group gets value j's.
__device__ __forceinline__ float reduce4(float v0, float v1, float v2, float v3, int j) {
    const bool b0 = j & 1, b1 = j & 2;
    const float k0 = (b0 ? v1 : v0) + dpp<kDppXor1>(b0 ? v0 : v1);
    const float k1 = (b0 ? v3 : v2) + dpp<kDppXor1>(b0 ? v2 : v3);
    const float k = (b1 ? k1 : k0) + dpp<kDppXor2>(b1 ? k0 : k1);
    return k + dpp<kDppDown4>(k);
}
// Sums of eight values over each group of 8 lanes: lane j gets value j's (each step sends the
// half of the values that the partner keeps; the partners j ^ 7, j ^ 2, j ^ 1 reach all 8).
__device__ __forceinline__ float reduce8(const float (&v)[8], int j) {
    const bool b0 = j & 1, b1 = j & 2, b2 = j & 4;
    float q[4], s[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = (b2 ? v[k + 4] : v[k]) + dpp<kDppXor7>(b2 ? v[k] : v[k + 4]);
#pragma unroll
    for (int k = 0; k < 2; ++k) s[k] = (b1 ? q[k + 2] : q[k]) + dpp<kDppXor2>(b1 ? q[k] : q[k + 2]);
    return (b0 ? s[1] : s[0]) + dpp<kDppXor1>(b0 ? s[0] : s[1]);
}

// ks / sqrt(pi) in 64 bits, rounded once. The constant is the sum of two floats (to 2^-52): as one
// 64-bit literal it stays in scalar registers across the persistent solver's loops, which spill 12
// more then (20 levels of placement 1,200, 16 restarts: 224.6 ms against 222.1).
__device__ __forceinline__ float tile_slope(double ks) {
    constexpr double c = 0.56418958354775628695;
    constexpr float kHi = (float)c, kLo = (float)(c - (double)kHi);
    return (float)fma(ks, (double)kHi, ks * (double)kLo);
}

// Literal-false probability of the atom z <= 0 and e^{-u^2} (0 in hard mode), u = ks z.
__device__ __forceinline__ float tile_atom(double z, double ks, float &em) {
    const float u = (float)(z * ks);
    const float e = half_erfc(fabsf(u), em);   // the smaller of the two sides; NaN stays NaN
    return u >= 0.0f ? 1.0f - e : e;
}

// Tiles [t0, t1) of set S for restart r. wload(c): weight of constraint c; fout(c, F): called
// with every valid cell's false mass. Returns this lane's sum of w F. With kGrad the gradient of
// w F goes through sc.add(r, real, id, g).
template <int kKind, bool kGrad, class St, class Sc, class WLoad, class FOut>
__device__ __forceinline__ float tile_run(const TabView &T, const TileSet &S, const St &st, const Sc &sc, int r,
                                          double kappa, bool hard, int t0, int t1, const WLoad &wload,
                                          const FOut &fout, int lane) {
    constexpr int D = kKind == 1 ? 1 : 2, NV = kKind == 0 ? 2 : 1, LM = kKind == 0 ? 0 : kTileBitsMax;
    constexpr int LA = LM ? LM : 1;   // array sizes
    if (t0 >= t1) return 0.0f;
    const int ri = lane >> 3, cj = lane & 7;
    const int L = LM ? S.L : 0;
    const double ks = kappa * (double)S.scale;
    const float kd = hard ? 0.0f : tile_slope(ks);   // dl/dz = kd e^{-u^2}
    const cptr<uint32_t> rc = T.tile_rc + S.tile0;
    const cptr<int32_t> con = T.tile_con + (int64_t)S.tile0 * 64 + lane;
    auto tile_of = [&](int t) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)rc[t]); };
    auto row_of = [&](uint32_t x) { return load_ent(T.tent + S.row_ent + (int)(x & 0xFFFFu) * 8 + ri); };
    auto weight = [&](int c) { return c >= 0 ? wload(c) : 0.0f; };

    // the column: values, right-hand sides and the gradient of the run
    uint32_t cg = ~0u;
    TileEnt ec{};
    double yc[D], rhc[NV][D];
    float qc = 1.0f, pc = 0.0f, cb[LA], gcb[LA], gc[D], gca = 0.0f;
    int idc[LA];
#pragma unroll
    for (int d = 0; d < D; ++d) yc[d] = 0.0, gc[d] = 0.0f;
#pragma unroll
    for (int i = 0; i < LA; ++i) cb[i] = gcb[i] = 0.0f, idc[i] = 0;
    auto flush = [&]() {
        if constexpr (kGrad) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                sc.add(r, true, ec.v[d], gc[d]);
                gc[d] = 0.0f;
            }
            if constexpr (kKind == 0) {
                if (ec.sel >= 0) sc.add(r, false, ec.sel, gca);
                gca = 0.0f;
            }
#pragma unroll
            for (int i = 0; i < LM; ++i) {
                if (i < L) sc.add(r, false, idc[i], gcb[i]);
                gcb[i] = 0.0f;
            }
        }
    };

    // the next tile's row record, constraint ids and weights are requested a tile ahead, the
    // ids two tiles ahead (the weights are read through them)
    uint32_t x0 = tile_of(t0);
    int c0 = con[(int64_t)t0 * 64], c1 = t0 + 1 < t1 ? con[(int64_t)(t0 + 1) * 64] : -1;
    TileEnt er = row_of(x0);
    float w0 = weight(c0), oacc = 0.0f;
    for (int t = t0; t < t1; ++t) {
        const bool more = t + 1 < t1;
        const uint32_t x1 = more ? tile_of(t + 1) : x0;
        const TileEnt er1 = row_of(x1);
        const float w1 = weight(c1);
        const int c2 = t + 2 < t1 ? con[(int64_t)(t + 2) * 64] : -1;
        if ((x0 >> 16) != cg) {
            if (cg != ~0u) flush();
            cg = x0 >> 16;
            ec = load_ent(T.tent + S.col_ent + (int)cg * 8 + cj);
#pragma unroll
            for (int d = 0; d < D; ++d) yc[d] = (double)st.bv(r, ec.v[d]);
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int d = 0; d < D; ++d) rhc[v][d] = (double)ec.rhs[v][d];
            if constexpr (kKind == 0) {
                const float ac = ec.sel >= 0 ? st.av(r, ec.sel) : 1.0f;
                pc = (1.0f - ac) * 0.5f;
                qc = (1.0f + ac) * 0.5f;
            }
#pragma unroll
            for (int i = 0; i < LM; ++i)
                if (i < L) {
                    idc[i] = T.tbits[S.col_bits + ((int)cg * L + i) * 8 + cj];
                    cb[i] = st.av(r, idc[i]);
                }
        }
        const bool valid = c0 >= 0;
        // linear forms and literal-false probabilities
        float lr[NV][D], lc[NV][D], mr[NV][D], mc[NV][D];
        double lin[D];
#pragma unroll
        for (int d = 0; d < D; ++d) lin[d] = (double)st.bv(r, er.v[d]) - yc[d];
        if (hard) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    lr[v][d] = lin[d] - (double)er.rhs[v][d] <= 0.0 ? 0.0f : 1.0f;
                    lc[v][d] = -lin[d] - rhc[v][d] <= 0.0 ? 0.0f : 1.0f;
                    mr[v][d] = mc[v][d] = 0.0f;
                }
        } else {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    lr[v][d] = tile_atom(lin[d] - (double)er.rhs[v][d], ks, mr[v][d]);
                    lc[v][d] = tile_atom(-lin[d] - rhc[v][d], ks, mc[v][d]);
                }
        }
        float F, gx[2] = {0.0f, 0.0f};   // gx: dU/d(y_row,d) of this cell
        if constexpr (kKind == 0) {
            const float ar = er.sel >= 0 ? st.av(r, er.sel) : 1.0f;
            const float pr = (1.0f - ar) * 0.5f, qr = (1.0f + ar) * 0.5f;
            float R0, R1, C0, C1;
            {   // rounded products: with equal sides (a square, kappa = 0) R0 - R1 is exactly 0
#pragma clang fp contract(off)
                R0 = lr[0][0] * lr[0][1];
                R1 = lr[1][0] * lr[1][1];
                C0 = lc[0][0] * lc[0][1];
                C1 = lc[1][0] * lc[1][1];
            }
            const float SR = qr * R0 + pr * R1, SC = qc * C0 + pc * C1;
            F = SR * SC;
            if constexpr (kGrad) {
                const float wr = w0 * SC, wcl = w0 * SR;
                const float A0 = wr * qr, A1 = wr * pr, B0 = wcl * qc, B1 = wcl * pc;
                // the scale last: a weight times a large kappa would overflow where e^{-u^2} is 0
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const int o = 1 - d;
                    gx[d] = kd * ((A0 * lr[0][o]) * mr[0][d] + (A1 * lr[1][o]) * mr[1][d] -
                                  ((B0 * lc[0][o]) * mc[0][d] + (B1 * lc[1][o]) * mc[1][d]));
                    gx[d] = valid ? gx[d] : 0.0f;
                    gc[d] -= gx[d];
                }
                // dF/dp = R1 - R0 times the other side, dp/da = -1/2
                const float gar = valid ? wr * (R0 - R1) * 0.5f : 0.0f;
                gca += valid ? wcl * (C0 - C1) * 0.5f : 0.0f;
                const float v = reduce4(gx[0], gx[1], gar, 0.0f, cj);
                const int id = cj == 0 ? er.v[0] : cj == 1 ? er.v[1] : er.sel;
                if (cj < 3 && id >= 0) sc.add(r, cj < 2, id, v);
            }
        } else {
            // bits: e_i = P[bit i equal] = (1 + a a')/2, exact up to the fma's one rounding
            float rb[LA], e[LA], suf[LA + 1];
            float Q = 1.0f;
#pragma unroll
            for (int d = 0; d < D; ++d) Q *= lr[0][d] * lc[0][d];
#pragma unroll
            for (int i = 0; i < LM; ++i) {
                rb[i] = 0.0f;
                e[i] = 1.0f;
                if (i < L) {
                    rb[i] = st.av(r, T.tbits[S.row_bits + ((int)(x0 & 0xFFFFu) * L + i) * 8 + ri]);
                    e[i] = fmaf(0.5f * rb[i], cb[i], 0.5f);
                }
            }
            suf[LM] = 1.0f;
#pragma unroll
            for (int i = LM - 1; i >= 0; --i) suf[i] = suf[i + 1] * e[i];
            F = suf[0] * Q;
            if constexpr (kGrad) {
                float pre = valid ? 0.5f * w0 * Q : 0.0f, vb[LA];
#pragma unroll
                for (int i = 0; i < LM; ++i) {
                    const float rest = pre * suf[i + 1];
                    vb[i] = valid ? rest * cb[i] : 0.0f;
                    gcb[i] += valid ? rest * rb[i] : 0.0f;
                    pre *= e[i];
                }
                const float wk = w0 * suf[0];
                if constexpr (D == 1) {
                    gx[0] = kd * ((wk * lc[0][0]) * mr[0][0] - (wk * lr[0][0]) * mc[0][0]);
                } else {
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const float other = wk * (lr[0][1 - d] * lc[0][1 - d]);
                        gx[d] = kd * ((other * lc[0][d]) * mr[0][d] - (other * lr[0][d]) * mc[0][d]);
                    }
                }
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    gx[d] = valid ? gx[d] : 0.0f;
                    gc[d] -= gx[d];
                }
                // the row's first 8 bits by lane, then its variables and the bits past 8
                const cptr<int32_t> rbits = T.tbits + S.row_bits + (int64_t)(x0 & 0xFFFFu) * L * 8 + ri;
                const float v8[8] = {vb[0], vb[1], vb[2], vb[3], vb[4], vb[5], vb[6], vb[7]};
                const float vlo = reduce8(v8, cj);
                if (cj < L) sc.add(r, false, rbits[cj * 8], vlo);
                const float vhi = reduce4(gx[0], gx[1], vb[8], vb[9], cj);
                if (cj < D) sc.add(r, true, (cj & 1) ? er.v[1] : er.v[0], vhi);
                else if (cj >= 2 && cj < 4 && cj + 6 < L) sc.add(r, false, rbits[(cj + 6) * 8], vhi);
            }
        }
        if (valid) {
            oacc += w0 * F;
            fout(c0, F);
        }
        x0 = x1;
        er = er1;
        w0 = w1;
        c0 = c1;
        c1 = c2;
    }
    flush();
    return oacc;
}

// Tiles of kind 3 (clause pairs): U = w_r P[literal_r False] l_r + w_c P[literal_c False] l_c
// over a cell's clauses, l the atoms' literal-false probabilities. The cell's Boolean gets its
// whole gradient here (sc.cell: a store). Two half_erfc a cell; the rest is its loads (ids of the
// two clauses, the cell word, two weights), requested one and two tiles ahead.
template <bool kGrad, class St, class Sc, class WLoad, class FOut>
__device__ __forceinline__ float cell_run(const TabView &T, const TileSet &S, const St &st, const Sc &sc, int r,
                                          double kappa, bool hard, int t0, int t1, const WLoad &wload,
                                          const FOut &fout, int lane) {
    if (t0 >= t1) return 0.0f;
    const int ri = lane >> 3, cj = lane & 7;
    const double ks = kappa * (double)S.scale;
    const float kd = hard ? 0.0f : tile_slope(ks);
    const cptr<uint32_t> rc = T.tile_rc + S.tile0;
    const cptr<int32_t> con = T.tile_con + (int64_t)S.tile0 * 64 + lane;
    const cptr<int32_t> aux = T.tile_cell + (int64_t)S.cell0 * 128 + lane;
    auto tile_of = [&](int t) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)rc[t]); };
    auto row_of = [&](uint32_t x) { return load_ent(T.tent + S.row_ent + (int)(x & 0xFFFFu) * 8 + ri); };
    struct Ids {
        int cr, cc, word;
    };
    auto ids_of = [&](int t) {
        if (t >= t1) return Ids{-1, -1, -1};
        return Ids{con[(int64_t)t * 64], aux[(int64_t)t * 128], aux[(int64_t)t * 128 + 64]};
    };
    auto weight = [&](int c) { return c >= 0 ? wload(c) : 0.0f; };
    auto value = [&](int word) { return word >= 0 ? st.av(r, word & kCellId) : 0.0f; };
    uint32_t cg = ~0u;
    TileEnt ec{};
    double yc = 0.0, rhc = 0.0;
    float gc = 0.0f, oacc = 0.0f;
    uint32_t x0 = tile_of(t0);
    Ids i0 = ids_of(t0), i1 = ids_of(t0 + 1);
    TileEnt er = row_of(x0);
    float wr0 = weight(i0.cr), wc0 = weight(i0.cc), a0 = value(i0.word);
    for (int t = t0; t < t1; ++t) {
        const uint32_t x1 = t + 1 < t1 ? tile_of(t + 1) : x0;
        const TileEnt er1 = row_of(x1);
        const float wr1 = weight(i1.cr), wc1 = weight(i1.cc), a1 = value(i1.word);
        const Ids i2 = ids_of(t + 2);
        if ((x0 >> 16) != cg) {
            if (kGrad && cg != ~0u) sc.add(r, true, ec.v[0], gc);
            gc = 0.0f;
            cg = x0 >> 16;
            ec = load_ent(T.tent + S.col_ent + (int)cg * 8 + cj);
            yc = (double)st.bv(r, ec.v[0]);
            rhc = (double)ec.rhs[0][0];
        }
        const double lin = (double)st.bv(r, er.v[0]) - yc;
        const double zr = lin - (double)er.rhs[0][0], zc = -lin - rhc;
        float lr, lc, mr = 0.0f, mc = 0.0f;
        if (hard) {
            lr = zr <= 0.0 ? 0.0f : 1.0f;
            lc = zc <= 0.0 ? 0.0f : 1.0f;
        } else {
            lr = tile_atom(zr, ks, mr);
            lc = tile_atom(zc, ks, mc);
        }
        const bool hr = i0.cr >= 0, hc = i0.cc >= 0;
        const float p = (1.0f - a0) * 0.5f, q = (1.0f + a0) * 0.5f;
        const bool nr = i0.word & kCellNeg, nc = i0.word & kCellCol;
        const float fr = nr ? p : q, fc = nc ? p : q;   // P[literal False]
        const float Fr = fr * lr, Fc = fc * lc;
        if constexpr (kGrad) {
            float gx = kd * ((hr ? wr0 * fr * mr : 0.0f) - (hc ? wc0 * fc * mc : 0.0f));
            gc -= gx;
            gx += dpp<kDppXor1>(gx);
            gx += dpp<kDppXor2>(gx);
            gx += dpp<kDppXor7>(gx);
            if (cj == 0) sc.add(r, true, er.v[0], gx);
            if (i0.word >= 0) {   // d P[literal False]/da = -+1/2
                const float g = (hr ? (nr ? -0.5f : 0.5f) * (wr0 * lr) : 0.0f) + (hc ? (nc ? -0.5f : 0.5f) * (wc0 * lc) : 0.0f);
                sc.cell(r, i0.word & kCellId, a0, g);
            }
        }
        if (hr) {
            oacc += wr0 * Fr;
            fout(i0.cr, Fr);
        }
        if (hc) {
            oacc += wc0 * Fc;
            fout(i0.cc, Fc);
        }
        x0 = x1;
        er = er1;
        wr0 = wr1;
        wc0 = wc1;
        a0 = a1;
        i0 = i1;
        i1 = i2;
    }
    if (kGrad) sc.add(r, true, ec.v[0], gc);
    return oacc;
}

// Wave `id` of `n` takes its share of every tile set (contiguous, so that its runs are long).
template <int kCF, bool kGrad, class St, class Sc, class WLoad, class FOut>
__device__ __forceinline__ float tile_sweep(const TabView &T, const St &st, const Sc &sc, int r, double kappa,
                                            bool hard, int id, int n, const WLoad &wload, const FOut &fout, int lane) {
    float oacc = 0.0f;
    if constexpr (kCF >= 1) {
        for (int s = 0; s < T.n_tsets; ++s) {
            const TileSet S = load_tset(T.tset + s);
            const int t0 = (int)((int64_t)S.n_tiles * id / n), t1 = (int)((int64_t)S.n_tiles * (id + 1) / n);
            if (S.kind == 0) {
                oacc += tile_run<0, kGrad>(T, S, st, sc, r, kappa, hard, t0, t1, wload, fout, lane);
            } else if (S.kind == 3) {
                oacc += cell_run<kGrad>(T, S, st, sc, r, kappa, hard, t0, t1, wload, fout, lane);
            } else if constexpr (kCF >= 3) {
                if (S.kind == 1) oacc += tile_run<1, kGrad>(T, S, st, sc, r, kappa, hard, t0, t1, wload, fout, lane);
                else oacc += tile_run<2, kGrad>(T, S, st, sc, r, kappa, hard, t0, t1, wload, fout, lane);
            }
        }
    }
    return oacc;
}

}  // namespace fsmt
