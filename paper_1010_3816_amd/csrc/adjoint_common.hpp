// Pieces shared by the adjoint-side kernels (adjoint_kernels.hip) and the
// forward-mode spin derivative (spin_tangent.hip): LDS views of the radial
// tables, the a-derivatives of the coefficients, and the strip-major tiles
// of a workgroup.
#pragma once

#include "device_common.hpp"

namespace teuk {
namespace {

// LDS copy of a strip's radial tables: [value/derivative][integer/half][field][lane].
// `o` is a row-dependent offset that is 0 at run time (row & zero): it keeps
// the reads inside the row loop instead of in (scarce) registers.
typedef const __attribute__((address_space(3))) double* lds_cptr;
typedef __attribute__((address_space(3))) double* lds_t;
typedef __attribute__((address_space(3))) v2d* cd_lds_t;

// Tile of a wavefront.  Tiles are numbered strip-major (the theta chunks of
// a strip consecutive) and workgroup b takes tiles b*wpb .. b*wpb + wpb - 1,
// so the tile count need not be a multiple of wpb per strip and a launch can
// fill every wavefront slot of the device.  A workgroup's tiles lie in at
// most two consecutive strips when wpb <= n_chunks + 1 (the host keeps it
// so); it holds the radial tables of both in LDS, as two slices.
struct TileOf {
    int strip, chunk;  // of this wavefront's tile
    int s0, n_slices;  // the workgroup's first strip and its number of strips (1 or 2)
    int slice;         // this wavefront's slice, strip - s0
    bool valid;        // false for wavefronts past the last tile
};

__device__ __forceinline__ TileOf tile_of(int b, int wpb, int wave, int n_strips, int n_chunks) {
    TileOf T;
    const int n_tiles = n_strips * n_chunks;
    const int first = b * wpb, tile = first + wave;
    T.valid = tile < n_tiles;
    T.s0 = first / n_chunks;
    T.n_slices = min((min(first + wpb, n_tiles) - 1) / n_chunks - T.s0 + 1, 2);
    T.strip = min(tile, n_tiles - 1) / n_chunks;
    T.chunk = tile - T.strip * n_chunks;
    T.slice = min(T.strip - T.s0, 1);
    return T;
}

// Workgroups of wpb consecutive tiles (strip-major), wpb at most n_chunks + 1
// so that a workgroup spans at most two strips.  The LDS holds one strip's
// tables (fields_per_strip doubles per lane) when no workgroup spans two,
// i.e. when wpb divides the chunks of a strip or there is one strip, and two
// otherwise; wave_bytes more for each wavefront.
inline void adjoint_launch_shape(const AdjScalars& k, int waves_per_block, int fields_per_strip, dim3* grid,
                                 dim3* block, size_t* lds_bytes, size_t wave_bytes = 0) {
    const int w = std::min(waves_per_block, k.n_chunks + 1);
    const int64_t tiles = (int64_t)k.n_strips * k.n_chunks;
    const int slices = (k.n_chunks % w == 0 || k.n_strips == 1) ? 1 : 2;
    *block = dim3(kWave * w);
    *grid = dim3((unsigned)((tiles + w - 1) / w));
    *lds_bytes = (size_t)slices * fields_per_strip * kWave * sizeof(double) + w * wave_bytes;
}

// ---- the step with its derivative in the spin ----------------------------

// d/da of stage_coef at one position from the radial factors V, their
// a-derivatives D and the values k.  With w = d(Sigma^2)/Sigma^2, a
// coefficient X/Sigma^2 has derivative dX/Sigma^2 - k w and B/Sigma has
// dB/Sigma - b w/2.
__device__ __forceinline__ Stage stage_coef_da(const SRad& V, const SRad& D, const Ang& G, Sig s, double kap,
                                               const Stage& k) {
    const double w = s.inv * fma(-D.a2d, G.sn2, D.rho2);
    const double hw = 0.5 * w;
    Stage r;
    r.b = fma(s.isig, D.b, -k.b * hw);
    r.tr = fma(s.inv, D.tr, -k.tr * w);
    r.ti = fma(s.inv, fma(D.ti1, G.cs, D.ti0), -k.ti * w);
    const double c1 = fma(-V.k2, G.sn2, V.k1), d1 = fma(-D.k2, G.sn2, D.k1);
    const double t = fma(-s.inv, fma(-c1, w, d1), D.k0);
    const double d0 = fma(-s.isig, fma(-V.k3, hw, D.k3), t);
    r.cr = fma(s.inv, d0, -k.cr * w);
    r.ci = -kap * fma(r.b, k.ti, k.b * r.ti);
    const double a2 = s.inv * D.dl2;
    r.wp = fma(a2, G.cotp, fma(-k.wp, w, a2));
    r.wm = fma(-a2, G.cotp, fma(-k.wm, w, a2));
    r.vr = fma(s.inv, fma(D.dl2, G.pd, D.vr), -k.vr * w);
    r.vi = fma(s.inv, D.vi, -k.vi * w);
    return r;
}

// What a row's completion needs of its coefficients (stage2_late and the
// next-row term of stage 1).
struct Late {
    double wh, b, tr, ti, wp;
};
__device__ __forceinline__ Late late_of(const Stage& h, const Stage& i) { return {h.wp, i.b, i.tr, i.ti, i.wp}; }

// A row between its arrival and its completion: of the state, and of its
// a-derivative (V: also the sum of Phi of v at the half point).
struct TanRow {
    cd P, Q, X, U, S;
    cd tP, tQ, tX, tS;
    cd tU;
    Late k, d;
};

// One step u^{m+1} = A u^m together with
//   V = false: T_m = (dA/da) u^m, the derivative of the step at fixed input;
//   V = true:  v^{m+1} = A v^m + (dA/da) u^m, the tangent-linear step of v = du/da,
// over a tile of 62 columns by A.rows rows.  Every stage is linear in the
// fields and in its coefficients, so its derivative is the same stage function
// of the derivative of the fields plus that of the fields with the
// coefficients' derivatives (T_m: the first from stage 1's derivative alone).
// The state's expressions and row order are those of the forward passes, so
// u^{m+1} equals theirs bit for bit; rows, poles and the two row loops are
// theirs too (one step: a row is completed when the next arrives).
// rvi(f, z), rvh(f, z): factor f of the lane's radial factors at its column and
// half point (z: zero, opaque to the compiler); rdi, rdh: their a-derivatives,
// in LDS, read row by row.  smp: this wavefront's
// sample slots.  T_m is streamed; the next states follow KEEP.
//
// What bounds it: 328 vector instructions per point and step with v (498
// before), half of the cycles of its two wavefronts per SIMD, and the waits for
// its 52 LDS reads a row and for memory (210 MB a step on 6400 x 256, 25 us at
// the rate of a copy within the last-level cache).  Stage 1 is finished, and
// the previous row completed and stored, before the column's coefficients are
// read: 226 registers with v, so the default instruction
// schedule, which has more loads in flight than one for occupancy, does not
// spill.  Without v the factors themselves are in registers (220) and their
// derivatives in the wavefront's own slice, which no other wavefront waits for.
// us per step, before and now: 6400 x 256 48.6 -> 39.5 with v, 38.8 -> 31.0
// without; 3200 x 128 19.4 -> 16.1, 14.3 -> 11.6 (15.1 from the workgroup's
// tables in LDS); 1600 x 64 8.9 -> 8.4, 9.7 -> 7.0; 1200 x 100 9.1 -> 9.7, 9.8 ->
// 7.1.
// Three wavefronts per SIMD (168 registers) spill with v and take 51-60 us.
template <bool V, int KEEP, class RadI, class RadH>
__device__ __forceinline__ void tangent_sweep(gin_t u_in, gin_t v_in, gout_t u_out, gout_t v_out, ctab_t ang,
                                              const ExtPoint* __restrict__ ext, double2* __restrict__ series_u,
                                              double2* __restrict__ series_v, RadI rvi, RadH rvh, lds_cptr rdi,
                                              lds_cptr rdh, __attribute__((address_space(3))) v2d* smp,
                                              const AdjScalars& A, int strip, int chunk, int lane) {
    constexpr int kN = V ? 4 : 2;  // planes read
    const int nr = A.nr, nth = A.nth, P = A.pitch;
    const int col = strip * kStripCols - 1 + lane;
    const int ci = min(max(col, 0), nr - 1);
    const bool store_ok = (lane >= 1) && (lane <= kWave - 2) && (col < nr);
    const bool boundary = (col == 0) || (col == nr - 1);
    const int j0 = chunk * A.rows;
    const int j1 = min(j0 + A.rows, nth);
    const int rs0 = max(j0 - 1, 0), rE = j1;
    const double sg = (double)A.sigma;

    const int32_t row_bytes = P * (int32_t)sizeof(v2d);
    const uint32_t ld_off = (uint32_t)ci * sizeof(v2d);
    const uint32_t st_off = store_ok ? (uint32_t)col * sizeof(v2d) : kOffNone;
    auto load_row = [&](int t, cd (&b)[kN]) {
        const size_t o = (size_t)min(max(t, 0), nth - 1) * P;
        b[0] = ld_row(row_rsrc(u_in + o, row_bytes), ld_off);
        b[1] = ld_row(row_rsrc(u_in + o + A.plane, row_bytes), ld_off);
        if constexpr (V) {
            b[2] = ld_row(row_rsrc(v_in + o, row_bytes), ld_off);
            b[3] = ld_row(row_rsrc(v_in + o + A.plane, row_bytes), ld_off);
        }
    };

    // the (at most one) extraction point of this tile
    int e_id = -1, e_lane = 0, e_ra = -1, e_rb = -1;
    double e_wr = 0.0, e_wa = 0.0, e_wb = 0.0;
    if constexpr (V) {
        for (int e = 0; e < A.n_ext; ++e) {
            const ExtPoint E = ext[e];
            const int es = E.col / kStripCols;
            if (es == strip && E.rowa / A.rows == chunk) {
                e_id = e;
                e_lane = E.col - es * kStripCols + 1;
                e_ra = E.rowa;
                e_rb = E.rowb;
                e_wr = E.wr;
                e_wa = E.wa;
                e_wb = E.wb;
            }
        }
    }
    auto pick = [](bool c, cd a, cd b) -> cd { return {c ? a.re : b.re, c ? a.im : b.im}; };

    cd buf[2][kN];
    load_row(rs0, buf[0]);
    load_row(rs0 + 1, buf[1]);
    const int c0 = strip * kStripCols - 1;
    const int plain = (int)(c0 > 0) & (int)(c0 + kWave - 1 < nr - 1) & (int)(e_id < 0);
    const int rM = plain * (min(rE, nth - 1) + 1) - 1;  // last iteration of the main loop

    TanRow row[2] = {};
    Ang g_next = load_ang(ang, nth, rs0);

    // Iteration t: row t arrives into n, row t - 1 in s is completed.
    // check: 0 in the main loop, 1 where t may be past the last row, in a
    // boundary strip or sampled, 2 for the tile's first row.
    auto iteration = [&](int t, cd (&b)[kN], TanRow& s, TanRow& n, auto check) {
        constexpr int CHECK = decltype(check)::value;
        const Ang G = g_next;
        const int z = t & A.zero;
        // stage 1 with the half point's coefficients first, then stage 2 with
        // the column's: both sets at once need more registers
        Stage kh, dh;
        {
            const SRad R = srad_of([&](int f) { return rvh(f, z); });
            const Sig sig = ssigma(R, G);
            kh = stage_coef(R, G, sig, A.kap_h);
            const SRad D = srad_of([&](int f) { return rdh[z + f * kWave]; });
            dh = stage_coef_da(R, D, G, sig, A.kap_h, kh);
        }
        const cd p = b[0], q = b[1];
        if constexpr (V && CHECK) {
            const int rel = lane - ((t == e_ra || t == e_rb) ? e_lane : 1 << 20);
            const int slot = (rel & ~1) == 0 ? rel + (t == e_rb ? 2 : 0) : 8 + lane;
            smp[slot] = v2d{p.re, p.im};
            smp[slot + ((rel & ~1) == 0 ? 4 : 0)] = (rel & ~1) == 0 ? v2d{b[2].re, b[2].im} : v2d{p.re, p.im};
        }
        const cd pr = from_right(p), qr = from_right(q);
        n.U = cadd(p, pr);
        const cd W = cadd(q, qr), dp = csub(pr, p), dq = csub(qr, q);
        const cd H = stage1_phi(kh.b, A.hdt, n.U, W, dp), Hl = from_left(H);
        n.S = cadd(H, Hl);
        const cd D = csub(H, Hl);
        // the derivative of H
        cd tH, tW, tdp, tdq;
        if constexpr (V) {
            const cd vp = b[2], vq = b[3], vpr = from_right(vp), vqr = from_right(vq);
            n.tU = cadd(vp, vpr);
            tW = cadd(vq, vqr);
            tdp = csub(vpr, vp);
            tdq = csub(vqr, vq);
            tH = fma_real(-dh.b, dp, stage1_phi(kh.b, A.hdt, n.tU, tW, tdp));
        } else {
            tH = {-dh.b * dp.re, -dh.b * dp.im};
        }
        const cd tHl = from_left(tH);
        n.tS = cadd(tH, tHl);
        const cd tD = csub(tH, tHl);
        cd Um = s.U, Sm = s.S, tSm = s.tS, tUm = s.tU;
        if constexpr (CHECK == 2) {  // row 0's previous row is its ghost (elsewhere: not used)
            Um = cscale(sg, n.U);
            Sm = cscale(sg, n.S);
            tSm = cscale(sg, n.tS);
            if constexpr (V) tUm = cscale(sg, n.tU);
        } else if constexpr (CHECK == 1) {  // the last row's next one is its ghost
            const bool gh = t == nth;
            n.U = pick(gh, cscale(sg, Um), n.U);
            n.S = pick(gh, cscale(sg, Sm), n.S);
            n.tS = pick(gh, cscale(sg, tSm), n.tS);
            if constexpr (V) n.tU = pick(gh, cscale(sg, tUm), n.tU);
        }
        const cd dU = csub(n.U, Um), dS = csub(n.S, Sm), tdS = csub(n.tS, tSm);
        cd tdU;
        if constexpr (V) tdU = csub(n.tU, tUm);
        // row t up to its next-row terms
        n.X = cadd(W, stage1_inc(kh, n.U, W, dp, dq, dU));
        n.tX = stage1_inc(dh, n.U, W, dp, dq, dU);
        if constexpr (V) n.tX = cadd(tW, cadd(n.tX, stage1_inc(kh, n.tU, tW, tdp, tdq, tdU)));
        if constexpr (CHECK != 2) {  // row t - 1
            const cd HQ = fma_real(s.k.wh, dU, s.X), HQl = from_left(HQ);
            const cd SQ = cadd(HQ, HQl), DQ = csub(HQ, HQl);
            cd np = fma_real(A.qdt, SQ, s.P);
            cd nq = cadd(s.Q, stage2_late(s.k.b, s.k.tr, s.k.ti, s.k.wp, SQ, DQ, dS));
            cd tHQ = fma_real(s.d.wh, dU, s.tX);
            if constexpr (V) tHQ = fma_real(s.k.wh, tdU, tHQ);
            const cd tHQl = from_left(tHQ);
            const cd tSQ = cadd(tHQ, tHQl), tDQ = csub(tHQ, tHQl);
            cd vp = fma_real(A.qdt, tSQ, s.tP);
            cd vq = cadd(s.tQ, cadd(stage2_late(s.d.b, s.d.tr, s.d.ti, s.d.wp, SQ, DQ, dS),
                                    stage2_late(s.k.b, s.k.tr, s.k.ti, s.k.wp, tSQ, tDQ, tdS)));
            if constexpr (CHECK) {
                const cd zero = {0.0, 0.0};
                np = pick(boundary, zero, np);
                nq = pick(boundary, zero, nq);
                vp = pick(boundary, zero, vp);
                vq = pick(boundary, zero, vq);
            }
            const int32_t bytes = (t - 1 >= j0 && t - 1 < j1) ? row_bytes : 0;
            const size_t o = (size_t)max(t - 1, 0) * P;
            constexpr int kV = V ? KEEP : 0;
            st_row<KEEP>(row_rsrc(u_out + o, bytes), st_off, np);
            st_row<KEEP>(row_rsrc(u_out + o + A.plane, bytes), st_off, nq);
            st_row<kV>(row_rsrc(v_out + o, bytes), st_off, vp);
            st_row<kV>(row_rsrc(v_out + o + A.plane, bytes), st_off, vq);
        }
        __builtin_amdgcn_sched_barrier(0);
        // Stage 2 of row t, but for the rows at the tile's ends that are only
        // neighbours: in tiles of a few rows they are most of the rows (with v,
        // 1600 x 64: 10.3 us a step with one-row tiles and all of it, 9.6
        // without, 8.3 with two rows).  What such a row leaves is not used;
        // the values are there for the registers' sake.
        n.P = p;
        n.Q = q;
        n.tP = n.tS;
        n.tQ = n.tS;
        n.k = s.k;
        n.d = s.d;
        if (CHECK == 0 || (CHECK == 1 ? t < rE : rs0 == j0)) {
            Stage ki, di;
            {
                const SRad R = srad_of([&](int f) { return rvi(f, z); });
                const Sig sig = ssigma(R, G);
                ki = stage_coef(R, G, sig, A.kap_i);
                const SRad D = srad_of([&](int f) { return rdi[z + f * kWave]; });
                di = stage_coef_da(R, D, G, sig, A.kap_i, ki);
            }
            n.P = fma_real(-ki.b, D, p);
            n.Q = cadd(q, stage2_early(ki, n.S, D, dS));
            const cd tq = cadd(stage2_early(di, n.S, D, dS), stage2_early(ki, n.tS, tD, tdS));
            if constexpr (V) {
                n.tP = fma_real(-di.b, D, fma_real(-ki.b, tD, b[2]));
                n.tQ = cadd(b[3], tq);
            } else {
                n.tP = fma_real(-di.b, D, cd{-ki.b * tD.re, -ki.b * tD.im});
                n.tQ = tq;
            }
            n.k = late_of(kh, ki);
            n.d = late_of(dh, di);
        }
        g_next = load_ang(ang, nth, min(t + 1, nth - 1));
        load_row(t + 2, b);
        __builtin_amdgcn_sched_barrier(0);
    };

    int t = rs0;
    iteration(t, buf[0], row[1], row[0], Const<2>{});
    ++t;
    for (; t + 1 <= rM; t += 2) {
        iteration(t, buf[1], row[0], row[1], Const<0>{});
        iteration(t + 1, buf[0], row[1], row[0], Const<0>{});
    }
    while (t <= rE) {
        iteration(t, buf[1], row[0], row[1], Const<1>{});
        if (++t > rE) break;
        iteration(t, buf[0], row[1], row[0], Const<1>{});
        ++t;
    }
    if constexpr (V) {
        wave_lds_handover();
        if (e_id >= 0 && lane < 2) {  // lane 0: the sample of u, lane 1: of v
            double2* out = lane == 0 ? series_u : series_v;
            if (out != nullptr) {
                cd w = {0.0, 0.0};
                auto add = [&](double wt, v2d a, v2d c) {
                    w.re = fma(wt, fma(e_wr, c.x - a.x, a.x), w.re);
                    w.im = fma(wt, fma(e_wr, c.y - a.y, a.y), w.im);
                };
                add(e_wa, smp[4 * lane], smp[4 * lane + 1]);
                if (e_rb >= 0) add(e_wb, smp[4 * lane + 2], smp[4 * lane + 3]);
                out[e_id] = double2{w.re, w.im};
            }
        }
    }
}

// LDS of a wavefront's sample slots: u, v x row a, b x two columns, and a slot per lane.
constexpr int kTanSlots = 8 + kWave;

// The radial tables (kTables = 2: and their a-derivatives) of the workgroup's
// strips of K-step tiles, in LDS: [strip][table][column/half][field][lane].
// A wavefront loads 13 rows at once before it writes them: one by one, each
// load's latency is waited for in turn (26 rows a wavefront, a third of the
// spin-tangent step on 6400 x 256).
template <int K, int kTables>
__device__ __forceinline__ void fill_tables(const TileOf& T, const double* __restrict__ rad,
                                            const double* __restrict__ rad_da, double* rad_s, int nr, int P, int wave,
                                            int wpb, int lane) {
    constexpr int kF = kTables * 2 * kNumSRad, kBatch = kNumSRad;
    const int n = T.n_slices * kF;
    for (int f0 = wave; f0 < n; f0 += kBatch * wpb) {
        double v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int f = min(f0 + u * wpb, n - 1);
            const int g = f % kF, deriv = g / (2 * kNumSRad), kind = (g / kNumSRad) % 2, field = g % kNumSRad;
            const int c = min(max((T.s0 + f / kF) * strip_cols(K) - K + lane, 0), nr - 1);
            const double* src = deriv ? rad_da : rad;
            v[u] = src[((size_t)field * 2 + kind) * P + (kind == 0 ? c : min(c, nr - 2))];
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (f0 + u * wpb < n) rad_s[(f0 + u * wpb) * kWave + lane] = v[u];
    }
    __syncthreads();
}

template <bool V, int KEEP>
__device__ __forceinline__ void tangent_tile(const double2* u_in, const double2* v_in, double2* u_out, double2* v_out,
                                             const double* __restrict__ rad, const double* __restrict__ rad_da,
                                             const double* __restrict__ ang, const ExtPoint* __restrict__ ext,
                                             double2* __restrict__ series_u, double2* __restrict__ series_v,
                                             const AdjScalars& A, double* rad_s) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wpb = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    typedef __attribute__((address_space(3))) v2d* slots_t;
    const TileOf T = tile_of(xcd_block(blockIdx.x, gridDim.x), wpb, wave, A.n_strips, A.n_chunks);
    if constexpr (V) {
        fill_tables<1, 2>(T, rad, rad_da, rad_s, A.nr, A.pitch, wave, wpb, lane);
        if (!T.valid) return;  // wavefront-uniform
        constexpr int kF = 4 * kNumSRad;
        const double* slice = rad_s + T.slice * kF * kWave + lane;
        const double* slots = rad_s + T.n_slices * kF * kWave + wave * 2 * kTanSlots;
        const lds_cptr ri = (lds_cptr)slice, rh = (lds_cptr)(slice + kNumSRad * kWave);
        tangent_sweep<V, KEEP>((gin_t)u_in, (gin_t)v_in, (gout_t)u_out, (gout_t)v_out, (ctab_t)ang, ext, series_u,
                               series_v, [&](int f, int z) { return ri[z + f * kWave]; },
                               [&](int f, int z) { return rh[z + f * kWave]; },
                               (lds_cptr)(slice + 2 * kNumSRad * kWave), (lds_cptr)(slice + 3 * kNumSRad * kWave),
                               (slots_t)slots, A, T.strip, T.chunk, lane);
    } else {
        // without v the lane's own factors fit its registers, and their
        // derivatives its wavefront's own slice: no wait for the workgroup
        if (!T.valid) return;  // wavefront-uniform
        double* slice = rad_s + wave * 2 * kNumSRad * kWave + lane;
        const int c = min(max(T.strip * kStripCols - 1 + lane, 0), A.nr - 1), ch = min(c, A.nr - 2);
        double ri[kNumSRad], rh[kNumSRad], d[2 * kNumSRad];
#pragma unroll
        for (int f = 0; f < kNumSRad; ++f) {
            const size_t o = (size_t)f * 2 * A.pitch;
            ri[f] = rad[o + c];
            rh[f] = rad[o + A.pitch + ch];
            d[f] = rad_da[o + c];
            d[kNumSRad + f] = rad_da[o + A.pitch + ch];
        }
#pragma unroll
        for (int f = 0; f < 2 * kNumSRad; ++f) slice[f * kWave] = d[f];
        tangent_sweep<V, KEEP>((gin_t)u_in, (gin_t)v_in, (gout_t)u_out, (gout_t)v_out, (ctab_t)ang, ext, series_u,
                               series_v, [&](int f, int) { return ri[f]; }, [&](int f, int) { return rh[f]; },
                               (lds_cptr)slice, (lds_cptr)(slice + kNumSRad * kWave), (slots_t)rad_s, A, T.strip,
                               T.chunk, lane);
    }
}

}  // namespace
}  // namespace teuk
