// gfx950 adjoint of the Lax-Wendroff step (arXiv:1010.3816, Eqs. (lw1)-(lw2)
// with the boundary conditions): lambda^m = A^H lambda^{m+1} and the spin
// gradient contribution Re <lambda^{m+1}, (dA/da) u^m>.
//
// The step is complex-linear, so its adjoint for a real loss (gradient
// convention dL/dRe + i dL/dIm) is the conjugate transpose.  The sweep is the
// gather form of the transposed step over the forward passes' tiles (64 r*
// columns per wavefront, theta rows in order, K steps a pass); with n =
// lambda^{m+1}, zeroed on the radial boundary columns:
//   * stage 2 transposed at the columns: the cotangents of SQ, DQ, D and S
//     (the sums and differences of the stage-1 values), the last with the
//     theta weights' shares of rows t-1, t, t+1;
//   * sum and difference transposed to the half points: lane L adds lane
//     L+1's share, giving the cotangents of H and HQ;
//   * stage 1 transposed at the half points, with its own theta shares;
//   * sum and difference transposed back to the columns: lane L adds lane
//     L-1's share; plus the direct term n.
//
// What bounds it.  With the stage coefficients of the forward passes, built
// once per row and pass, a two-step sweep issues 133 vector instructions per
// point and step (195 before); on 6400 x 256 (states in the last-level cache)
// it is bound by the latency and issue of one round of wavefronts, two per
// SIMD, or one with the dot products: us per step, before and now, cotangents
// 16.9 -> 14.9, with the dot products 22.4 -> 21.0, spin gradient from states 48
// -> 43; 3200 x 128 8.3 -> 7.7, 10.0 -> 9.1, 20.3 -> 18.5.
#include "adjoint_common.hpp"

namespace teuk {
namespace {

// Extraction points (of the first n) whose bilinear stencil touches output
// rows r_lo .. r_hi of a tile and the columns c0 .. c0 + 63 of its lanes, as
// bits: the transposed extraction is applied row by row only for these.
__device__ __forceinline__ unsigned ext_mask(const ExtPoint* __restrict__ ext, int n, int r_lo, int r_hi, int c0) {
    unsigned m = 0;
    for (int e = 0; e < n; ++e) {
        const ExtPoint E = ext[e];
        const bool rows = (E.rowa >= r_lo && E.rowa <= r_hi) || (E.rowb >= r_lo && E.rowb <= r_hi);
        if (rows && E.col + 1 >= c0 && E.col <= c0 + kWave - 1) m |= 1u << e;
    }
    return m;
}

// x - conj(re + i im) v
__device__ __forceinline__ cd sub_conj(double re, double im, cd v, cd x) {
    return {fma(-im, v.im, fma(-re, v.re, x.re)), fma(im, v.re, fma(-re, v.im, x.im))};
}

// One row of one step between its arrival and its completion, which adds
// the next row's theta shares (the cotangents of S and U lack them).
struct AdjRow {
    cd np, nq;    // n plus the part of the output known at the arrival
    cd lp, lq;    // the same of the share for the next column
    cd lS, lD;    // cotangents of S and D at the column
    cd up, uph;   // theta shares to the next row: stage 2 (column), stage 1 (half point)
    double bh;    // b at the half point
};

// LDS of a wavefront for the points of a row: each step's weights and gradients
// per lane.  No more than that: with two steps' slots the one-step kernel's
// workgroups that span two strips came to 90 KB, one to a CU (5003 x 197 45 us
// a step against 37).
constexpr int hit_doubles(int steps) { return steps * kRowHits * 3 * kWave; }

// What the adjoint's sweeps accumulate beside the cotangents: nothing, the
// dot products with stored tangents, or the spin gradient from the states.
enum SpinPart { kNone, kDot, kStates };

// Sweeps whose lanes hold their own radial factors: one step without the spin
// gradient from states, which leaves the registers for it (us per step from the
// workgroup's tables in LDS and from registers, one step a pass: cotangents,
// 1600 x 128 8.0 and 6.8, 6400 x 256 22.8 and 20.9; dot products 9.7 and 8.4,
// 31.9 and 31.6).
constexpr bool own_factors(int steps, SpinPart sp) { return steps == 1 && sp != kStates; }

// K adjoint steps in one pass over a tile of 64 - 2K columns: step j takes
// row r - j in iteration r and completes row r - j - 1, as in the forward
// passes (sweep in the forward kernels' source), with the same row loops: the
// second one checks for the last pole, boundary columns and extraction.  A
// row's coefficients are built once and serve all steps.  gs[j]: the gradient
// of the sample of step j's output state, or nullptr.
//   kDot:    tan[j] holds T = (dA/da) u of step j; Re <n, T> is summed over the owned points;
//   kStates: (K = 1) tan[0] holds u^m; T_m is formed on the way (tangent_sweep's
//            expressions) and its dot product with n summed.
// rvi(f, z), rvh(f, z): factor f of the lane's radial factors at its column
// and half point (z: zero, opaque to the compiler); rdi, rdh: their
// a-derivatives in LDS (kStates).  Returns this lane's sum.
template <int K, SpinPart SP, int KEEP, class RadI, class RadH>
__device__ __forceinline__ double adjoint_sweep(const double2* __restrict__ nu_in, double2* __restrict__ lam_out,
                                                const double* __restrict__ ang, const ExtPoint* __restrict__ ext,
                                                const double* const (&gs)[K], const double2* const (&tan)[K],
                                                RadI rvi, RadH rvh, lds_cptr rdi, lds_cptr rdh, lds_t hits,
                                                const AdjScalars& A, int strip, int chunk, int lane) {
    static_assert(SP != kStates || K == 1, "the spin gradient from states is a one-step sweep");
    // rows in flight (and rows the loop is unrolled by); coefficient rows: K
    constexpr int kRing = (SP == kStates) ? 1 : (K == 1) ? 2 : K;
    constexpr int kCols = strip_cols(K);
    const int nr = A.nr, nth = A.nth, P = A.pitch;
    const int col = strip * kCols - K + lane;
    const int ci = min(max(col, 0), nr - 1);
    const bool own = (lane >= K) && (lane < kWave - K) && (col < nr);
    const bool interior = (col >= 1) && (col < nr - 1);
    const int j0 = chunk * A.rows;
    const int j1 = min(j0 + A.rows, nth);
    const int rs0 = max(j0 - K, 0), rE = j1 - 1 + K;
    const double sg = (double)A.sigma;
    const int c0 = strip * kCols - K;
    bool any_g = false;
#pragma unroll
    for (int j = 0; j < K; ++j) any_g = any_g || gs[j] != nullptr;
    const unsigned emask = ext_mask(ext, any_g ? A.n_ext : 0, j0 - K + 1, j1 + K - 2, c0);

    const int32_t row_bytes = P * (int32_t)sizeof(v2d);
    const uint32_t ld_off = (uint32_t)ci * sizeof(v2d);
    const uint32_t st_off = own ? (uint32_t)col * sizeof(v2d) : kOffNone;
    auto load_from = [&](const double2* base, int t, cd& p, cd& q) {
        const double2* b = base + (size_t)min(max(t, 0), nth - 1) * P;
        p = ld_row(row_rsrc(b, row_bytes), ld_off);
        q = ld_row(row_rsrc(b + A.plane, row_bytes), ld_off);
    };
    auto pick = [](bool c, cd a, cd b) -> cd { return {c ? a.re : b.re, c ? a.im : b.im}; };
    const cd zero = {0.0, 0.0};

    cd bp[kRing], bq[kRing];
#pragma unroll
    for (int u = 0; u < kRing; ++u) load_from(nu_in, rs0 + u, bp[u], bq[u]);
    // rows of the tangents (or states): step j's row r - j, one row ahead
    constexpr int kT = SP == kNone ? 1 : K;
    cd tp[kT], tq[kT];
    if constexpr (SP != kNone) {
#pragma unroll
        for (int j = 0; j < K; ++j) load_from(tan[j], rs0 - j, tp[j], tq[j]);
    }
    const int plain = (int)(c0 > 0) & (int)(c0 + kWave - 1 < nr - 1) & (int)(emask == 0);
    const int rM = plain * (min(rE, nth - 1) + 1) - 1;

    double acc = 0.0;
    AdjRow st[K] = {};
    Stage Ch[K] = {}, Ci[K] = {};
    TanRow tr = {};  // kStates: the row of the tangent
    cd n_prev_p = zero, n_prev_q = zero;
    Ang g_next = load_ang(ang, nth, rs0);

    // Transposed extraction of the sample of step j's output state: each
    // stencil point of an extraction point receives its bilinear weight times
    // the sample's gradient (gs, re/im interleaved).  The weights and
    // gradients of the rows an iteration completes go to the lane's slots in
    // the wavefront's LDS beforehand (zeros where there are none), so that the
    // row itself takes no branch; the host sees to it that at most kRowHits
    // points touch a grid point.
    lds_t hit_w = (lds_t)hits + lane;
    cd_lds_t hit_g = (cd_lds_t)((lds_t)hits + K * kRowHits * kWave) + lane;
    auto put_hit = [&](int slot, double w, double re, double im) {
        hit_w[slot * kWave] = w;
        hit_g[slot * kWave] = v2d{re, im};
    };
    bool hit_set = true;  // slots to be cleared
    int e_lo = nth, e_hi = -1;  // rows that the tile's points touch
    for (unsigned m = emask; m != 0; m &= m - 1) {
        const ExtPoint E = ext[__builtin_ctz(m)];
        e_lo = min(e_lo, E.rowb >= 0 ? min(E.rowa, E.rowb) : E.rowa);
        e_hi = max(e_hi, max(E.rowa, E.rowb));
    }
    auto set_hits = [&](int r) {
        if (hit_set) {
            for (int k = 0; k < K * kRowHits; ++k) put_hit(k, 0.0, 0.0, 0.0);
            hit_set = false;
        }
        if (r - 1 < e_lo || r - K > e_hi) return;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (gs[j] == nullptr) continue;
            const int t = r - j - 1;
            int h = 0;
            for (int e = 0; e < A.n_ext; ++e) {
                if (!((emask >> e) & 1u)) continue;
                const ExtPoint E = ext[e];
                if (t != E.rowa && t != E.rowb) continue;  // wavefront-uniform
                hit_set = true;
                if ((col != E.col && col != E.col + 1) || h >= kRowHits) continue;
                const double wrow = (t == E.rowa) ? E.wa : E.wb;
                const double w = (col == E.col) ? wrow * (1.0 - E.wr) : wrow * E.wr;
                put_hit(j * kRowHits + h, w, gs[j][2 * e], gs[j][2 * e + 1]);
                ++h;
            }
        }
    };

    auto iteration = [&](int r, cd& rp, cd& rq, auto ph, auto steps, auto check) {
        constexpr int PH = decltype(ph)::value % K, STEPS = decltype(steps)::value, CHECK = decltype(check)::value;
        if constexpr (CHECK) set_hits(r);
        const Ang G = g_next;
        const int z = r & A.zero;
        Stage dh, di;
        {
            const SRad R = srad_of([&](int f) { return rvi(f, z); });
            const Sig s = ssigma(R, G);
            Ci[PH] = stage_coef(R, G, s, A.kap_i);
            if constexpr (SP == kStates) {
                const SRad D = srad_of([&](int f) { return rdi[z + f * kWave]; });
                di = stage_coef_da(R, D, G, s, A.kap_i, Ci[PH]);
            }
        }
        {
            const SRad R = srad_of([&](int f) { return rvh(f, z); });
            const Sig s = ssigma(R, G);
            Ch[PH] = stage_coef(R, G, s, A.kap_h);
            if constexpr (SP == kStates) {
                const SRad D = srad_of([&](int f) { return rdh[z + f * kWave]; });
                dh = stage_coef_da(R, D, G, s, A.kap_h, Ch[PH]);
            }
        }
        cd p = rp, q = rq;
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            const Stage &kh = Ch[(PH + K - j) % K], &ki = Ci[(PH + K - j) % K];
            const int t = r - j;
            AdjRow& s = st[j];
            if constexpr (CHECK) {
                p = pick(interior, p, zero);
                q = pick(interior, q, zero);
            }
            if constexpr (SP == kDot) {
                double c = p.re * tp[j].re + p.im * tp[j].im;
                c = fma(q.re, tq[j].re, fma(q.im, tq[j].im, c));
                const bool in = own && t >= j0 && t < j1;
                acc += in ? c : 0.0;
                load_from(tan[j], t + 1, tp[j], tq[j]);
            }
            // stage 2 at the column
            const cd lSQ = sub_conj(ki.tr, ki.ti, q, cd{A.qdt * p.re, A.qdt * p.im});
            const cd lDQ = cscale(ki.b, q);
            AdjRow n;
            n.lD = sub_conj(ki.cr, ki.ci, q, cd{-ki.b * p.re, -ki.b * p.im});
            n.up = cscale(ki.wp, q);
            cd dn = cscale(ki.wm, q);
            // stage 1 at the half point
            const cd lHQ = cadd(cadd(lSQ, lDQ), from_right(csub(lSQ, lDQ)));
            n.uph = cscale(kh.wp, lHQ);
            cd dnh = cscale(kh.wm, lHQ);
            cd up0 = s.up, uph0 = s.uph;  // shares of the previous row
            if constexpr (CHECK == 2) {
                // the step's first row: at the pole its previous one is its
                // ghost; elsewhere nothing formed from it is used
                if (j == STEPS - 1) {
                    up0 = cscale(sg, dn);
                    uph0 = cscale(sg, dnh);
                }
            }
            n.lS = sub_conj(ki.vr, ki.vi, q, csub(csub(up0, n.up), dn));
            const cd lU = sub_conj(kh.vr, kh.vi, lHQ, csub(csub(uph0, n.uph), dnh));
            const cd lV = sub_conj(kh.tr, kh.ti, lHQ, lHQ);
            const cd ldp = sub_conj(kh.cr, kh.ci, lHQ, zero), ldq = cscale(kh.b, lHQ);
            n.np = cadd(p, csub(lU, ldp));
            n.nq = cadd(q, csub(lV, ldq));
            n.lp = cadd(lU, ldp);
            n.lq = cadd(lV, ldq);
            n.bh = kh.b;
            if constexpr (CHECK == 1) {  // the last row's next one is its ghost
                dn = pick(t == nth, cscale(sg, up0), dn);
                dnh = pick(t == nth, cscale(sg, uph0), dnh);
            }
            // row t - 1 is complete
            const cd lS = cadd(s.lS, dn);
            const cd lH = cadd(cadd(lS, s.lD), from_right(csub(lS, s.lD)));
            const cd a = cadd(lH, dnh);
            cd op = cadd(s.np, cadd(fma_real(s.bh, lH, a), from_left(cadd(s.lp, fma_real(-s.bh, lH, a)))));
            cd oq = cadd(s.nq, fma_real(A.hdt, lH, from_left(fma_real(A.hdt, lH, s.lq))));
            if constexpr (SP == kStates) {
                // T of row t - 1 (tangent_sweep's expressions without v) with n
                const cd u = tp[0], w = tq[0], ur = from_right(u), wr = from_right(w);
                TanRow m;
                m.U = cadd(u, ur);
                const cd W = cadd(w, wr), dp = csub(ur, u), dq = csub(wr, w);
                const cd H = stage1_phi(kh.b, A.hdt, m.U, W, dp), Hl = from_left(H);
                m.S = cadd(H, Hl);
                const cd D = csub(H, Hl);
                const cd tH = {-dh.b * dp.re, -dh.b * dp.im}, tHl = from_left(tH);
                m.tS = cadd(tH, tHl);
                const cd tD = csub(tH, tHl);
                cd Um = tr.U, Sm = tr.S, tSm = tr.tS;
                if constexpr (CHECK == 2) {
                    Um = cscale(sg, m.U);
                    Sm = cscale(sg, m.S);
                    tSm = cscale(sg, m.tS);
                } else if constexpr (CHECK == 1) {
                    m.U = pick(t == nth, cscale(sg, Um), m.U);
                    m.S = pick(t == nth, cscale(sg, Sm), m.S);
                    m.tS = pick(t == nth, cscale(sg, tSm), m.tS);
                }
                const cd dU = csub(m.U, Um), dS = csub(m.S, Sm), tdS = csub(m.tS, tSm);
                const cd HQ = fma_real(tr.k.wh, dU, tr.X), HQl = from_left(HQ);
                const cd SQ = cadd(HQ, HQl), DQ = csub(HQ, HQl);
                const cd tHQ = fma_real(tr.d.wh, dU, tr.tX), tHQl = from_left(tHQ);
                const cd tSQ = cadd(tHQ, tHQl), tDQ = csub(tHQ, tHQl);
                const cd vp = fma_real(A.qdt, tSQ, tr.tP);
                const cd vq = cadd(tr.tQ, cadd(stage2_late(tr.d.b, tr.d.tr, tr.d.ti, tr.d.wp, SQ, DQ, dS),
                                               stage2_late(tr.k.b, tr.k.tr, tr.k.ti, tr.k.wp, tSQ, tDQ, tdS)));
                double c = n_prev_p.re * vp.re + n_prev_p.im * vp.im;
                c = fma(n_prev_q.re, vq.re, fma(n_prev_q.im, vq.im, c));
                const bool in = own && t - 1 >= j0 && t - 1 < j1;
                acc += in ? c : 0.0;
                m.X = cadd(W, stage1_inc(kh, m.U, W, dp, dq, dU));
                m.tX = stage1_inc(dh, m.U, W, dp, dq, dU);
                m.tP = fma_real(-di.b, D, cd{-ki.b * tD.re, -ki.b * tD.im});
                m.tQ = cadd(stage2_early(di, m.S, D, dS), stage2_early(ki, m.tS, tD, tdS));
                m.k = late_of(kh, ki);
                m.d = late_of(dh, di);
                tr = m;
                n_prev_p = p;
                n_prev_q = q;
                load_from(tan[0], t + 1, tp[0], tq[0]);
            }
            s = n;
            if constexpr (CHECK) {
#pragma unroll
                for (int h = 0; h < kRowHits; ++h) {
                    const double w = hit_w[(j * kRowHits + h) * kWave];
                    const v2d g = hit_g[(j * kRowHits + h) * kWave];
                    op.re = fma(w, g.x, op.re);
                    op.im = fma(w, g.y, op.im);
                }
            }
            p = op;
            q = oq;
            if (j == 0) {
                __builtin_amdgcn_sched_barrier(kAllButScalarLoads);
                g_next = load_ang(ang, nth, min(r + 1, nth - 1));
            }
        }
        load_from(nu_in, r + kRing, rp, rq);
        if constexpr (STEPS == K) {
            const int t = r - K;
            const int32_t bytes = (t >= j0 && t < j1) ? row_bytes : 0;
            const double2* b = lam_out + (size_t)max(t, 0) * P;
            st_row<KEEP>(row_rsrc(b, bytes), st_off, p);
            st_row<KEEP>(row_rsrc(b + A.plane, bytes), st_off, q);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    int r = rs0;
    auto head = [&](auto self, auto i) {
        constexpr int I = decltype(i)::value;
        if constexpr (I < K) {
            iteration(r, bp[I % kRing], bq[I % kRing], Const<I>{}, Const<I + 1>{}, Const<2>{});
            ++r;
            self(self, Const<I + 1>{});
        }
    };
    head(head, Const<0>{});
    auto rows = [&](auto self, auto u, auto check) {
        constexpr int I = decltype(u)::value + K;
        if constexpr (I < K + kRing) {
            iteration(r, bp[I % kRing], bq[I % kRing], Const<I>{}, Const<K>{}, check);
            ++r;
            self(self, Const<I - K + 1>{}, check);
        }
    };
    while (r + kRing - 1 <= rM) rows(rows, Const<0>{}, Const<0>{});
    // The last rows: one that is left after the whole groups goes alone (in
    // pairs, a two-step tile of one row swept six rows where it has five: with
    // dot products, 400 x 32 5.4 and 4.7 us a step).
    while (r + kRing - 1 <= rE) rows(rows, Const<0>{}, Const<1>{});
    if constexpr (kRing > 1)
        if (r <= rE) iteration(r, bp[K % kRing], bq[K % kRing], Const<K>{}, Const<K>{}, Const<1>{});
    return acc;
}

// A wavefront's tile of a K-step adjoint sweep; the sums of the lanes go to
// the tile's slot, in a fixed order.  Where the registers allow it (one step,
// without the spin gradient from states) the lane holds its own radial factors
// and no wavefront waits for another; otherwise the workgroup's radial tables
// (with their a-derivatives for kStates) are in LDS.
template <int K, SpinPart SP, int KEEP>
__device__ __forceinline__ void adjoint_tile(const double2* __restrict__ nu_in, double2* __restrict__ lam_out,
                                             const double* __restrict__ rad, const double* __restrict__ rad_da,
                                             const double* __restrict__ ang, const ExtPoint* __restrict__ ext,
                                             const double* const (&gs)[K], const double2* const (&tan)[K],
                                             double* __restrict__ dlda_slots, const AdjScalars& A, double* rad_s) {
    constexpr int kTables = SP == kStates ? 2 : 1;
    const int lane = threadIdx.x & (kWave - 1);
    const int wpb = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const TileOf T = tile_of(xcd_block(blockIdx.x, gridDim.x), wpb, wave, A.n_strips, A.n_chunks);
    double acc;
    if constexpr (own_factors(K, SP)) {
        if (!T.valid) return;  // wavefront-uniform
        const int c = min(max(T.strip * strip_cols(K) - K + lane, 0), A.nr - 1), ch = min(c, A.nr - 2);
        double ri[kNumSRad], rh[kNumSRad];
#pragma unroll
        for (int f = 0; f < kNumSRad; ++f) {
            ri[f] = rad[(size_t)f * 2 * A.pitch + c];
            rh[f] = rad[((size_t)f * 2 + 1) * A.pitch + ch];
        }
        acc = adjoint_sweep<K, SP, KEEP>(nu_in, lam_out, ang, ext, gs, tan, [&](int f, int) { return ri[f]; },
                                         [&](int f, int) { return rh[f]; }, nullptr, nullptr,
                                         (lds_t)(rad_s + wave * hit_doubles(K)), A, T.strip, T.chunk, lane);
    } else {
        fill_tables<K, kTables>(T, rad, rad_da, rad_s, A.nr, A.pitch, wave, wpb, lane);
        if (!T.valid) return;  // wavefront-uniform
        const double* slice = rad_s + T.slice * kTables * 2 * kNumSRad * kWave + lane;
        const double* da = slice + (kTables - 1) * 2 * kNumSRad * kWave;
        const lds_cptr ri = (lds_cptr)slice, rh = (lds_cptr)(slice + kNumSRad * kWave);
        acc = adjoint_sweep<K, SP, KEEP>(nu_in, lam_out, ang, ext, gs, tan,
                                         [&](int f, int z) { return ri[z + f * kWave]; },
                                         [&](int f, int z) { return rh[z + f * kWave]; }, (lds_cptr)da,
                                         (lds_cptr)(da + kNumSRad * kWave),
                                         (lds_t)(rad_s + T.n_slices * kTables * 2 * kNumSRad * kWave +
                                                 wave * hit_doubles(K)),
                                         A, T.strip, T.chunk, lane);
    }
    if constexpr (SP != kNone) {
        for (int off = kWave / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, kWave);
        if (lane == 0) dlda_slots[(size_t)T.chunk * A.n_strips + T.strip] += acc;
    }
}

// One adjoint step.  SPIN: with the spin gradient from u^m = u_in; DOT: from
// the stored tangent T_m = u_in; neither: the cotangents only (linear in the
// state, so they need no forward state).
template <bool SPIN, bool DOT, int KEEP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))
    lw_adjoint_kernel(const double2* __restrict__ nu_in, const double2* __restrict__ u_in,
                      double2* __restrict__ lam_out, const double* __restrict__ rad,
                      const double* __restrict__ rad_da, const double* __restrict__ ang,
                      double* __restrict__ dlda_slots, const ExtPoint* __restrict__ ext,
                      const double* __restrict__ gsample, AdjScalars A) {
    extern __shared__ double rad_s[];
    adjoint_tile<1, SPIN ? kStates : DOT ? kDot : kNone, KEEP>(nu_in, lam_out, rad, rad_da, ang, ext, {gsample}, {u_in},
                                                               dlda_slots, A, rad_s);
}

// Two adjoint steps per pass (temporal blocking): lambda^{m+2} -> lambda^m.
// DOT: also the spin gradient's terms of both steps from stored tangents,
// tan_a = T_{m+1} and tan_b = T_m.
template <bool DOT, int KEEP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))
    lw_adjoint2_kernel(const double2* __restrict__ nu_in, double2* __restrict__ lam_out,
                       const double* __restrict__ rad, const double* __restrict__ ang,
                       const ExtPoint* __restrict__ ext, const double* __restrict__ gsample_a,
                       const double* __restrict__ gsample_b, const double2* __restrict__ tan_a,
                       const double2* __restrict__ tan_b, double* __restrict__ dlda_slots, AdjScalars A) {
    extern __shared__ double rad_s[];
    adjoint_tile<2, DOT ? kDot : kNone, KEEP>(nu_in, lam_out, rad, nullptr, ang, ext, {gsample_a, gsample_b},
                                              {tan_a, tan_b}, dlda_slots, A, rad_s);
}

// Adjoint steps on register tiles, for small and medium grids: the forward
// tile pass (lw_tile_kernel) with the transposed step.  A group's last row
// sends its theta shares (up, uph) to the row below and its first row (dn,
// dnh) to the row above, through LDS, with one barrier a step; everything
// else is in the lane or a cross-lane move.  K steps take lambda^{m+K} to
// lambda^m; after step s the gradient of the sample of its output state, row
// A.g_row - s of g (if that is not negative), is added at every stencil point
// in the tile, own part or not.  Expressions and their order are those of
// adjoint_sweep, so the cotangents are the same bit for bit.
//
// Bound as the forward tile pass, at about 110 vector instructions per point
// and step.  us per step with three extraction points, the two-step sweep and
// now: 1200 x 100 7.1 -> 2.5, 1600 x 128 8.6 -> 3.6, 3200 x 128 10.7 -> 6.1.
template <int C, int R, int T, int KEEP>
__global__ void __launch_bounds__(T)
    lw_adjoint_tile_kernel(const double2* __restrict__ nu_in, double2* __restrict__ lam_out,
                           const double* __restrict__ rad, const double* __restrict__ ang,
                           const ExtPoint* __restrict__ ext, const double2* __restrict__ gser, AdjScalars A,
                           AdjTileArgs B) {
    const int K = B.steps, W = C - 2 * K;
    const int nr = A.nr, nth = A.nth, P = A.pitch;
    const int lane = threadIdx.x & (kWave - 1);
    const int j = lane % C, G = blockDim.x / C;
    const int g = threadIdx.x / C;
    const int strip = blockIdx.x % B.n_strips, tt = blockIdx.x / B.n_strips, n_tt = B.n_chunks;
    const int H = G * R;  // the tile's rows: its first, and its own
    const int own0 = tt == 0 ? 0 : H - K + (tt - 1) * (H - 2 * K);
    const int own1 = tt == n_tt - 1 ? nth : H - K + tt * (H - 2 * K);
    const int row0 = tt == 0 ? 0 : tt == n_tt - 1 ? nth - H : own0 - K;
    const int t0 = row0 + g * R;
    const int c0 = strip * W;
    const int col = c0 - K + j;
    const int ci = min(max(col, 0), nr - 1), hi = min(max(col, 0), nr - 2);
    const bool interior = (col >= 1) && (col < nr - 1);
    const bool edge = c0 - K <= 0 || c0 - K + C >= nr;
    const double sg = (double)A.sigma;

    extern __shared__ double rad_s[];
    // [buffer][first row: dn, dnh; last row: up, uph][group][column]; then the
    // points and the gradients of the launch's samples
    v2d* xch = reinterpret_cast<v2d*>(rad_s);
    const int plane = G * C, buf = 4 * plane;
    v2d* sg_s = xch + 2 * buf;  // [step][point]
    ExtPoint* sx = reinterpret_cast<ExtPoint*>(sg_s + K * kMaxBlockExt);
    const int me = g * C + j;
    const bool pole0 = t0 == 0, pole1 = t0 + R == nth;
    const int i_up = pole0 || g == 0 ? me : 2 * plane + me - C;
    const int i_dn = pole1 || g == G - 1 ? 2 * plane + me : me + C;
    const double f_up = pole0 ? sg : 1.0, f_dn = pole1 ? sg : 1.0;

    cd p[R], q[R];
    Stage kh[R], ki[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const size_t o = (size_t)min(t0 + r, nth - 1) * P + ci;
        p[r] = ld(nu_in, o);
        q[r] = ld(nu_in, o + A.plane);
    }
    const SRad Rh = srad_of([&](int f) { return rad[((size_t)f * 2 + 1) * P + hi]; });
    const SRad Ri = srad_of([&](int f) { return rad[((size_t)f * 2 + 0) * P + ci]; });
    const int n_ext = gser != nullptr ? A.n_ext : 0;
    for (int i = threadIdx.x; i < K * n_ext; i += blockDim.x) {
        const int s = i / n_ext, e = i % n_ext;
        const int64_t row = B.g_row - s;
        const double2 v = row >= 0 ? gser[row * n_ext + e] : double2{0.0, 0.0};
        sg_s[s * kMaxBlockExt + e] = v2d{v.x, v.y};
    }
    if ((int)threadIdx.x < n_ext) sx[threadIdx.x] = ext[threadIdx.x];
    // stencil points this lane holds: bit e of its row r
    unsigned duty[R] = {};
    unsigned any = 0;
    for (int e = 0; e < n_ext; ++e) {
        const ExtPoint E = ext[e];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int t = t0 + r;
            if ((col == E.col || col == E.col + 1) && (t == E.rowa || t == E.rowb)) duty[r] |= 1u << e;
            any |= duty[r];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const Ang ga = load_ang(ang, nth, min(t0 + r, nth - 1));
        kh[r] = stage_coef(Rh, ga, ssigma(Rh, ga), A.kap_h);
        ki[r] = stage_coef(Ri, ga, ssigma(Ri, ga), A.kap_i);
    }

    for (int s = 0; s < K; ++s) {
        v2d* x = xch + (s & 1) * buf;
        if (edge) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                p[r] = {interior ? p[r].re : 0.0, interior ? p[r].im : 0.0};
                q[r] = {interior ? q[r].re : 0.0, interior ? q[r].im : 0.0};
            }
        }
        cd lD[R], up[R], dn[R], lHQ[R], uph[R], dnh[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const Stage &h = kh[r], &i = ki[r];
            const cd lSQ = sub_conj(i.tr, i.ti, q[r], cd{A.qdt * p[r].re, A.qdt * p[r].im});
            const cd lDQ = cscale(i.b, q[r]);
            lD[r] = sub_conj(i.cr, i.ci, q[r], cd{-i.b * p[r].re, -i.b * p[r].im});
            up[r] = cscale(i.wp, q[r]);
            dn[r] = cscale(i.wm, q[r]);
            lHQ[r] = cadd(cadd(lSQ, lDQ), from_right(csub(lSQ, lDQ)));
            uph[r] = cscale(h.wp, lHQ[r]);
            dnh[r] = cscale(h.wm, lHQ[r]);
            if (r == 0) {
                x[me] = v2d{dn[r].re, dn[r].im};
                x[me + plane] = v2d{dnh[r].re, dnh[r].im};
            }
            if (r == R - 1) {
                x[me + 2 * plane] = v2d{up[r].re, up[r].im};
                x[me + 3 * plane] = v2d{uph[r].re, uph[r].im};
            }
        }
        __syncthreads();
        const v2d x0 = x[i_up], x1 = x[i_up + plane], x2 = x[i_dn], x3 = x[i_dn + plane];
        __builtin_amdgcn_sched_barrier(0);
        const cd Uu = {f_up * x0.x, f_up * x0.y}, Uh = {f_up * x1.x, f_up * x1.y};
        const cd Du = {f_dn * x2.x, f_dn * x2.y}, Dh = {f_dn * x3.x, f_dn * x3.y};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const Stage &h = kh[r], &i = ki[r];
            const cd up0 = r == 0 ? Uu : up[r > 0 ? r - 1 : 0], uph0 = r == 0 ? Uh : uph[r > 0 ? r - 1 : 0];
            const cd dnn = r == R - 1 ? Du : dn[r < R - 1 ? r + 1 : r], dnhn = r == R - 1 ? Dh : dnh[r < R - 1 ? r + 1 : r];
            const cd lS = cadd(sub_conj(i.vr, i.vi, q[r], csub(csub(up0, up[r]), dn[r])), dnn);
            const cd lU = sub_conj(h.vr, h.vi, lHQ[r], csub(csub(uph0, uph[r]), dnh[r]));
            const cd lV = sub_conj(h.tr, h.ti, lHQ[r], lHQ[r]);
            const cd ldp = sub_conj(h.cr, h.ci, lHQ[r], cd{0.0, 0.0}), ldq = cscale(h.b, lHQ[r]);
            const cd np = cadd(p[r], csub(lU, ldp)), nq = cadd(q[r], csub(lV, ldq));
            const cd lp = cadd(lU, ldp), lq = cadd(lV, ldq);
            const cd lH = cadd(cadd(lS, lD[r]), from_right(csub(lS, lD[r])));
            const cd a = cadd(lH, dnhn);
            p[r] = cadd(np, cadd(fma_real(h.b, lH, a), from_left(cadd(lp, fma_real(-h.b, lH, a)))));
            q[r] = cadd(nq, fma_real(A.hdt, lH, from_left(fma_real(A.hdt, lH, lq))));
        }
        if (any != 0 && B.g_row - s >= 0) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                for (unsigned d = duty[r]; d != 0; d &= d - 1) {
                    const int e = __builtin_ctz(d);
                    const ExtPoint E = sx[e];
                    const v2d gv = sg_s[s * kMaxBlockExt + e];
                    const double wrow = (t0 + r == E.rowa) ? E.wa : E.wb;
                    const double w = (col == E.col) ? wrow * (1.0 - E.wr) : wrow * E.wr;
                    p[r].re = fma(w, gv.x, p[r].re);
                    p[r].im = fma(w, gv.y, p[r].im);
                }
        }
    }
    if (j >= K && j < K + W && col < nr) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int t = t0 + r;
            if (t >= own0 && t < own1) {
                st_state<KEEP>(lam_out, (size_t)t * P + col, p[r]);
                st_state<KEEP>(lam_out, (size_t)t * P + col + A.plane, q[r]);
            }
        }
    }
}

// One Lax-Wendroff step, u^{m+1} = A u^m, that also writes the derivative of
// the step with respect to the spin at fixed input, T_m = (dA/da) u^m: the
// spin gradient is then dL/da = sum_m Re <lambda^{m+1}, T_m>, a dot product
// the reverse sweep forms from the cotangents it computes anyway.
template <int KEEP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))
    lw_tangent_kernel(const double2* __restrict__ u_in, double2* __restrict__ u_out, double2* __restrict__ t_out,
                      const double* __restrict__ rad, const double* __restrict__ rad_da,
                      const double* __restrict__ ang, AdjScalars A) {
    extern __shared__ double rad_s[];
    tangent_tile<false, KEEP>(u_in, nullptr, u_out, t_out, rad, rad_da, ang, nullptr, nullptr, nullptr, A, rad_s);
}

// lam_Phi += E^T g for every extraction point, in point order (one thread).
__global__ void extract_adjoint_kernel(double2* __restrict__ lam, int pitch, const ExtPoint* __restrict__ pts, int n,
                                       const double2* __restrict__ g) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    for (int e = 0; e < n; ++e) {
        const ExtPoint E = pts[e];
        const double2 gv = g[e];
        for (int r = 0; r < 2; ++r) {
            const int row = r == 0 ? E.rowa : E.rowb;
            if (row < 0) continue;
            const double w = r == 0 ? E.wa : E.wb;
            double2* a = &lam[(size_t)row * pitch + E.col];
            double2* b = &lam[(size_t)row * pitch + E.col + 1];
            const double wa = w * (1.0 - E.wr), wb = w * E.wr;
            a->x = fma(wa, gv.x, a->x);
            a->y = fma(wa, gv.y, a->y);
            b->x = fma(wb, gv.x, b->x);
            b->y = fma(wb, gv.y, b->y);
        }
    }
}

// Sum of the spin-gradient slots in a fixed order (one workgroup), added to *out.
__global__ void reduce_slots_kernel(const double* __restrict__ slots, int n, double* __restrict__ out) {
    __shared__ double part[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) s += slots[i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = blockDim.x / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out += part[0];
}

// Zero the radial boundary columns of a state.
__global__ void zero_radial_boundary_kernel(double2* __restrict__ u, int nr, int nth, int pitch) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nth) return;
    const double2 z = {0.0, 0.0};
    const size_t plane = (size_t)nth * pitch;
    const size_t a = (size_t)j * pitch, b = (size_t)j * pitch + nr - 1;
    u[a] = z;
    u[a + plane] = z;
    u[b] = z;
    u[b + plane] = z;
}

}  // namespace


hipError_t launch_adjoint(const AdjArgs& a, int waves_per_block, AdjMode mode, hipStream_t s) {
    dim3 grid, block;
    size_t lds;
    const bool spin = mode == AdjMode::kSpin;
    adjoint_launch_shape(a.k, waves_per_block, spin ? 4 * kNumSRad : 0, &grid, &block, &lds,
                         hit_doubles(1) * sizeof(double));
    const bool keep = a.k.keep != 0;
    auto pick = [&](auto k0, auto k1) { return keep ? k1 : k0; };
    auto kern = spin ? pick(lw_adjoint_kernel<true, false, 0>, lw_adjoint_kernel<true, false, 1>)
                     : (mode == AdjMode::kTangentDot ? pick(lw_adjoint_kernel<false, true, 0>,
                                                            lw_adjoint_kernel<false, true, 1>)
                                                     : pick(lw_adjoint_kernel<false, false, 0>,
                                                            lw_adjoint_kernel<false, false, 1>));
    hipLaunchKernelGGL(kern, grid, block, lds, s, a.nu_in, a.u_in, a.lam_out, a.rad, a.rad_da, a.ang, a.slots, a.ext,
                       a.gsample, a.k);
    return hipGetLastError();
}

hipError_t launch_adjoint2(const AdjArgs& a, const double* gsample_b, const double2* tan_b, int waves_per_block,
                           hipStream_t s) {
    dim3 grid, block;
    size_t lds;
    adjoint_launch_shape(a.k, waves_per_block, 2 * kNumSRad, &grid, &block, &lds, hit_doubles(2) * sizeof(double));
    const bool keep = a.k.keep != 0;
    auto kern = a.u_in ? (keep ? lw_adjoint2_kernel<true, 1> : lw_adjoint2_kernel<true, 0>)
                       : (keep ? lw_adjoint2_kernel<false, 1> : lw_adjoint2_kernel<false, 0>);
    hipLaunchKernelGGL(kern, grid, block, lds, s, a.nu_in, a.lam_out, a.rad, a.ang, a.ext, a.gsample, gsample_b,
                       a.u_in, tan_b, a.slots, a.k);
    return hipGetLastError();
}

hipError_t launch_adjoint_tile(const AdjArgs& a, const double2* gser, int64_t g_row, int steps, const TileShape& t,
                               hipStream_t s) {
    AdjTileArgs b{};
    b.steps = steps;
    b.g_row = g_row;
    if (!tile_grid(t, a.k.nr, a.k.nth, steps, &b.n_strips, &b.n_chunks) || a.k.n_ext > kMaxBlockExt)
        return hipErrorInvalidValue;
    const int threads = t.waves * kWave;
    const size_t lds = (size_t)(8 * threads + steps * kMaxBlockExt) * sizeof(double2) + kMaxBlockExt * sizeof(ExtPoint);
    const dim3 grid(b.n_strips * b.n_chunks), block(threads);
    auto go = [&](auto k0, auto k1, int most) {
        if (threads > most) return hipErrorInvalidValue;
        hipLaunchKernelGGL(a.k.keep ? k1 : k0, grid, block, lds, s, a.nu_in, a.lam_out, a.rad, a.ang, a.ext, gser, a.k, b);
        return hipGetLastError();
    };
#define TEUK_TILE(C, R, T) \
    if (t.cols == C && t.rows == R) \
        return go(lw_adjoint_tile_kernel<C, R, T, 0>, lw_adjoint_tile_kernel<C, R, T, 1>, T);
    TEUK_TILE(16, 1, 1024)
    TEUK_TILE(32, 1, 1024)
    TEUK_TILE(64, 1, 1024)
    TEUK_TILE(32, 2, 512)
    TEUK_TILE(64, 2, 512)
    TEUK_TILE(64, 3, 512)
#undef TEUK_TILE
    return hipErrorInvalidValue;
}

hipError_t launch_tangent(const double2* u_in, double2* u_out, double2* t_out, const AdjArgs& a, int waves_per_block,
                          hipStream_t s) {
    dim3 grid, block;
    size_t lds;
    adjoint_launch_shape(a.k, waves_per_block, 0, &grid, &block, &lds, 2 * kNumSRad * kWave * sizeof(double));
    hipLaunchKernelGGL(a.k.keep ? lw_tangent_kernel<1> : lw_tangent_kernel<0>, grid, block, lds, s, u_in, u_out, t_out,
                       a.rad, a.rad_da, a.ang, a.k);
    return hipGetLastError();
}

hipError_t launch_extract_adjoint(double2* lam, int pitch, const ExtPoint* pts, int n, const double2* g,
                                  hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(extract_adjoint_kernel, dim3(1), dim3(64), 0, s, lam, pitch, pts, n, g);
    return hipGetLastError();
}

hipError_t launch_reduce_slots(const double* slots, int n, double* out, hipStream_t s) {
    hipLaunchKernelGGL(reduce_slots_kernel, dim3(1), dim3(256), 0, s, slots, n, out);
    return hipGetLastError();
}

hipError_t launch_zero_radial_boundary(double2* u, int nr, int nth, int pitch, hipStream_t s) {
    hipLaunchKernelGGL(zero_radial_boundary_kernel, dim3((nth + 255) / 256), dim3(256), 0, s, u, nr, nth, pitch);
    return hipGetLastError();
}

}  // namespace teuk
