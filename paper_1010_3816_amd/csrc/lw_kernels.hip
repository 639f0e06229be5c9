// gfx950 kernels for the two-step Lax-Wendroff evolution of the homogeneous
// (2+1)D Teukolsky equation (arXiv:1010.3816, Sec. 3, Eqs. (lw1)-(lw2)).
//
// The sweeps.  A pass takes K = 1, 2 or 3 steps over a tile: one wavefront
// owns 64 consecutive r* columns (64 - 2K output columns plus K halo columns
// on each side) and a chunk of theta rows, which it sweeps row by row:
//   * stage 1 (Eq. lw1) is evaluated once per half point and row: lane L
//     combines its column with the column of lane L+1 (the averaging of the
//     printed kernel_average1) and forms u^{n+1/2}_{i+1/2};
//   * stage 2 (Eq. lw2) at column i combines the stage-1 values of lanes
//     L-1 and L; both neighbour exchanges are cross-lane moves, so the
//     stage-1 field never leaves registers;
//   * the theta stencil of S needs the differences of the averaged fields to
//     the neighbour rows; the sweep carries the last row's sums, and the pole
//     ghost rows (mirror for even |m|, anti-mirror for odd |m|) are formed in
//     registers;
//   * a completed row goes on to the next step of the pass in registers;
//   * Phi = Pi = 0 is set on the radial boundary columns.
// Every input point is read once per tile (plus the halo), every output point
// written once; the coefficients of Eq. (1) are rebuilt once per point and
// pass from 1-D radial tables and 1-D angular tables, so no 2-D coefficient
// array is streamed from HBM.
//
// What bounds it, and why three steps.  A pass moves 64 bytes a point however
// many steps it takes, and rebuilding a point's coefficients costs about as
// much as half a step, also once per pass; more steps divide both.  Per point
// and step the main loops issue 150 (K = 1), 110 (K = 2) and 102 (K = 3)
// vector instructions (the two-step pass before the stage coefficients and
// theta differences of device_common.hpp: 180).  K = 3 is the most whose rows
// and coefficients fit the registers of two wavefronts per SIMD (244 of 256).
// 25600 x 512, us per step (the same box in turn): two steps, before, 95; two
// steps 84-88, bound by memory; three steps 66-68 = 4.2 TB/s, bound by the
// issue of its wavefronts as much as by memory.  6400 x 256: 15.1, 13.9, 12.3.
//
// Extraction is fused: the wavefront whose tile contains the bilinear
// stencil of an extraction point samples Phi of the INPUT of every step.
#include "device_common.hpp"

namespace teuk {
namespace {
// The source term of the inhomogeneous variant at one point: f g, with the
// time factor f = (fr, fi) of the stage and the profile g at the position.
__device__ __forceinline__ cd source(cd g, double fr, double fi) {
    return {fma(fr, g.re, -fi * g.im), fma(fr, g.im, fi * g.re)};
}

typedef __attribute__((address_space(3))) double* lds_t;
typedef __attribute__((address_space(3))) v2d* cd_lds_t;

// LDS of one wavefront of a sweep: its radial factors, [column/half][field][lane]
// (13 KB), the slots of a sample's values, and a slot per lane for values not
// sampled.
constexpr int kSampleSlots = 4 * kMaxPassSteps;
constexpr int kSliceDoubles = 2 * kNumSRad * kWave + 2 * (kSampleSlots + kWave);
constexpr size_t kRadSliceBytes = kSliceDoubles * sizeof(double);

// One row of one step between its arrival and its completion (the next
// row's arrival): the new Phi but for its SQ term, the new Pi but for
// stage2_late, 2 h_Pi but for its next-row term, and the row's sums of Phi
// and of H, from which the next row's theta differences are formed.
struct Row {
    cd P, Q, X, U, S;
};

// Stage coefficients of one row: at the half point and at the column.
struct RowCoef {
    Stage h, i;
};

// K Lax-Wendroff steps in one pass over a tile of 64 - 2K columns by A.rows
// rows (temporal blocking: only the pass's input is read and its output
// written).  Iteration r of the row loop takes input row r from memory; step
// 0 of the pass completes row r - 1, which goes from registers to step 1 as
// its row r - 1, and so on: step j takes row r - j and completes row r - j -
// 1, and row r - K of the output is written.  Each step consumes one column
// at each edge of the wavefront and one row at each end of the tile.
//
// A row's coefficients are the same for all steps and are built once, when
// its input row arrives (from the lane's radial factors, in the wavefront's
// LDS slice rs, [column/half][field][lane], or for K = 1 in its registers, and
// the angular row, scalar),
// and kept in registers until the last step has passed it: a ring of K + 1
// rows (K + 2 of user coefficients, which come a row ahead).  The row loop is
// unrolled over the ring, so nothing is copied.
//
// Poles: the ghost rows are sigma times the first and last row, in the input
// and in the stage-1 values alike, so at row 0 the difference to the
// previous row is U - sigma U, and after the last row a step takes the ghost
// as its next one.  A tile starts at row 0 or K rows above its first one,
// where the first rows of each step hold values formed from rows that were
// not read; the rows they complete are not used by the next step.
//
// series0, 1, 2: where the samples of the inputs of the steps go, or nullptr.
//
// The main loop is for rows away from the last pole, of strips without a
// radial boundary column and tiles that sample or keep nothing; the loop
// after it checks for all of these.
template <int K, bool KERR, bool SRC, int KEEP>
__device__ __forceinline__ void sweep(gin_t __restrict__ u_in, gout_t __restrict__ u_out, ctab_t rad, ctab_t ang,
                                      ctab_t uci, ctab_t uch, cext_t ext, double2* series0, double2* series1,
                                      double2* series2, gout_t __restrict__ win, lds_t rs,
                                      const StepScalars& A, int strip, int chunk, int lane,
                                      gin_t __restrict__ src_i, gin_t __restrict__ src_h) {
    // User coefficients, which come from memory, are loaded a row ahead where
    // the registers allow it: in a short tile nothing else covers their latency
    // (us per step: 400 x 32 3.8 and 3.5; with a source in single steps 1600 x
    // 128 17.3 and 13.8).
    constexpr bool kFetch = !KERR && !(K == 2 && SRC);
    constexpr int kRing = kFetch ? K + 2 : K + 1;  // coefficient rows held
    constexpr int kAhead = (K == 3) ? 2 : kRing;  // input rows in flight (divides the unrolled rows)
    constexpr int kCols = strip_cols(K);
    const int nr = A.nr, nth = A.nth, P = A.pitch;
    const int col = strip * kCols - K + lane;
    // Lanes outside the grid read the clamped edge column; what they hold
    // reaches only the radial boundary columns, which every step sets to zero.
    const int ci = min(max(col, 0), nr - 1);
    const int hi = min(max(col, 0), nr - 2);
    const bool store_ok = (lane >= K) && (lane < kWave - K) && (col < nr);
    const bool boundary = (col == 0) || (col == nr - 1);
    const int j0 = chunk * A.rows;
    const int j1 = min(j0 + A.rows, nth);
    const int rs0 = max(j0 - K, 0);  // first input row
    const int rE = j1 - 1 + K;       // last iteration
    const double sg = (double)A.sigma;

    const int32_t row_bytes = P * (int32_t)sizeof(v2d);
    const uint32_t ld_off = (uint32_t)ci * sizeof(v2d);
    const uint32_t st_off = store_ok ? (uint32_t)col * sizeof(v2d) : kOffNone;
    auto load_row = [&](int t, cd& p, cd& q) {
        const gin_t b = u_in + (size_t)min(max(t, 0), nth - 1) * P;
        p = ld_row(row_rsrc(b, row_bytes), ld_off);
        q = ld_row(row_rsrc(b + A.plane, row_bytes), ld_off);
    };
    // rows the tile does not own are dropped (an empty resource)
    auto put_row = [&](gout_t base, int t, cd vp, cd vq, auto keep) {
        const int32_t bytes = (t >= j0 && t < j1) ? row_bytes : 0;
        const gout_t b = base + (size_t)max(t, 0) * P;
        st_row<decltype(keep)::value>(row_rsrc(b, bytes), st_off, vp);
        st_row<decltype(keep)::value>(row_rsrc(b + A.plane, bytes), st_off, vq);
    };

    // The radial factors of this lane's column and half point, loaded with
    // the first rows so that the latencies overlap.  Passes of several steps
    // write them to the wavefront's slice (lane-private: written and read by
    // the same lane, no barrier); one step leaves them in its registers, where
    // a row does not wait for LDS (us per step from LDS and from registers:
    // 1200 x 100 7.6 and 6.9, 3200 x 128 9.8 and 8.1, 6400 x 256 21.2 and 19.2).
    double tv[2 * kNumSRad];
    if constexpr (KERR) {
#pragma unroll
        for (int f = 0; f < kNumSRad; ++f) {
            tv[f] = rad[((size_t)f * 2 + 0) * P + ci];
            tv[kNumSRad + f] = rad[((size_t)f * 2 + 1) * P + hi];
        }
    }
    cd bp[kAhead], bq[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load_row(rs0 + u, bp[u], bq[u]);
    if constexpr (KERR && K > 1) {
#pragma unroll
        for (int f = 0; f < 2 * kNumSRad; ++f) rs[f * kWave + lane] = tv[f];
    }

    auto ang_row = [&](int t) -> Ang {
        Ang G{};
        if constexpr (KERR) G = load_ang(ang, nth, min(t, nth - 1));
        return G;
    };
    // the row-dependent zero offset keeps the LDS reads next to their use
    auto coefs = [&](int t, const Ang& G, RowCoef& c) {
        if constexpr (KERR) {
            const __attribute__((address_space(3))) double* r = rs + lane + (t & A.zero);
            const SRad Ri = srad_of([&](int f) { return K == 1 ? tv[f] : r[f * kWave]; });
            c.i = stage_coef(Ri, G, ssigma(Ri, G), A.kap_i);
            const SRad Rh = srad_of([&](int f) { return K == 1 ? tv[kNumSRad + f] : r[(kNumSRad + f) * kWave]; });
            c.h = stage_coef(Rh, G, ssigma(Rh, G), A.kap_h);
        } else {
            const int tc = min(t, nth - 1);
            c.i = user_stage(uci, nth, P, tc, ci, A.inv_dth2, A.inv_2dth, A.hdt_dr, A.qdt);
            c.h = user_stage(uch, nth, P, tc, hi, A.inv_dth2, A.inv_2dth, A.dt_dr, A.hdt);
        }
    };

    // the (at most one, apart from equal ones) extraction point of this tile,
    // in scalar registers
    int e_id = -1, e_lane = 0, e_ra = -1, e_rb = -1;
    double e_wr = 0.0, e_wa = 0.0, e_wb = 0.0;
    for (int e = 0; e < A.n_ext; ++e) {
        const int ecol = ext[e].col, era = ext[e].rowa;
        const int es = ecol / kCols;
        if (es == strip && era / A.rows == chunk) {
            e_id = e;
            e_lane = ecol - es * kCols + K;
            e_ra = era;
            e_rb = ext[e].rowb;
            e_wr = ext[e].wr;
            e_wa = ext[e].wa;
            e_wb = ext[e].wb;
        }
    }
    // The values of Phi a sample is formed from go to the wavefront's LDS
    // slots [step][row a, b][column, next column] as the rows pass; every
    // other value goes to a slot of the lane's own, so no branch is taken.
    cd_lds_t smp = (cd_lds_t)(rs + 2 * kNumSRad * kWave);
    auto pick = [](bool c, cd a, cd b) -> cd { return {c ? a.re : b.re, c ? a.im : b.im}; };

    // last iteration of the main loop (none: -1)
    const int c0 = strip * kCols - K;
    const int plain = (int)(c0 > 0) & (int)(c0 + kWave - 1 < nr - 1) & (int)(e_id < 0) & (int)(win == nullptr);
    const int rM = plain * (min(rE, nth - 1) + 1) - 1;

    Row st[K] = {};
    RowCoef C[kRing] = {};
    Ang g_next = ang_row(rs0);
    // source rows in the coefficients' ring, loaded a row ahead: with one
    // wavefront to a SIMD nothing else covers their latency (6400 x 256, steps
    // in pairs: 21.0 us a step with the loads at their use, 16.8 ahead)
    cd gi[kRing], gh[kRing];
    const uint32_t half_off = (uint32_t)hi * sizeof(v2d);
    auto load_source = [&](int t, int slot) {
        const size_t o = (size_t)min(t, nth - 1) * P;
        gi[slot] = ld_row(row_rsrc(src_i + o, row_bytes), ld_off);
        gh[slot] = ld_row(row_rsrc(src_h + o, row_bytes), half_off);
    };
    if constexpr (SRC) load_source(rs0, 0);
    if constexpr (kFetch) coefs(rs0, g_next, C[0]);

    // Iteration r.  PH: the ring slot of row r's coefficients; STEPS: the
    // steps that take a row (fewer while a tile starts); CHECK: the row may
    // be a pole's, a boundary column's, sampled or kept.
    auto iteration = [&](int r, cd& rp, cd& rq, auto ph, auto steps, auto check) {
        constexpr int PH = decltype(ph)::value, STEPS = decltype(steps)::value;
        constexpr bool CHECK = decltype(check)::value != 0, FIRST = decltype(check)::value == 2;
        const Ang G = g_next;
        if constexpr (kFetch)
            coefs(r + 1, G, C[(PH + 1) % kRing]);
        else
            coefs(r, G, C[PH]);
        if constexpr (SRC) load_source(r + 1, (PH + 1) % kRing);
        if constexpr (CHECK) __builtin_amdgcn_sched_barrier(0);
        cd p = rp, q = rq;
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            const RowCoef& c = C[(PH + kRing - j) % kRing];      // of the arriving row
            const RowCoef& d = C[(PH + kRing - j - 1) % kRing];  // of the row completed
            const int t = r - j;
            Row& s = st[j];
            cd um = s.U, sm = s.S;
            Row n;
            if constexpr (CHECK) {
                if constexpr (K <= 2)
                    if (j == K - 1) put_row(win, win != nullptr ? t : -1, p, q, Const<0>{});
                // lanes e_lane, e_lane + 1 of a sampled row (1 << 20: none)
                const int rel = lane - ((t == e_ra || t == e_rb) ? e_lane : 1 << 20);
                smp[(rel & ~1) == 0 ? rel + 4 * j + (t == e_rb ? 2 : 0) : kSampleSlots + lane] = v2d{p.re, p.im};
            }
            const cd pr = from_right(p), qr = from_right(q);
            n.U = cadd(p, pr);
            const cd V = cadd(q, qr), dp = csub(pr, p), dq = csub(qr, q);
            const cd H = stage1_phi(c.h.b, A.hdt, n.U, V, dp), Hl = from_left(H);
            n.S = cadd(H, Hl);
            const cd D = csub(H, Hl);
            if constexpr (FIRST) {
                // the step's first row: at the pole its previous one is its
                // ghost; elsewhere nothing formed from the previous one is used
                if (j == STEPS - 1) {
                    um = cscale(sg, n.U);
                    sm = cscale(sg, n.S);
                }
            } else if constexpr (CHECK) {  // the last row's next one is its ghost
                n.U = pick(t == nth, cscale(sg, um), n.U);
                n.S = pick(t == nth, cscale(sg, sm), n.S);
            }
            const cd dU = csub(n.U, um), dS = csub(n.S, sm);
            // row t - 1 is complete
            const cd HQ = fma_real(d.h.wp, dU, s.X), HQl = from_left(HQ);
            const cd SQ = cadd(HQ, HQl), DQ = csub(HQ, HQl);
            cd np = fma_real(A.qdt, SQ, s.P);
            cd nq = cadd(s.Q, stage2_late(d.i.b, d.i.tr, d.i.ti, d.i.wp, SQ, DQ, dS));
            // row t, up to its next-row terms
            cd e1 = stage1_inc(c.h, n.U, V, dp, dq, dU);
            cd e2 = stage2_early(c.i, n.S, D, dS);
            if constexpr (SRC) {
                const int sl = (PH + kRing - j) % kRing;
                e1 = cadd(e1, source(gh[sl], A.sf[4 * j], A.sf[4 * j + 1]));
                e2 = cadd(e2, source(gi[sl], A.sf[4 * j + 2], A.sf[4 * j + 3]));
            }
            n.X = cadd(V, e1);
            n.P = fma_real(-c.i.b, D, p);
            n.Q = cadd(q, e2);
            s = n;
            if constexpr (CHECK) {
                np = pick(boundary, cd{0.0, 0.0}, np);
                nq = pick(boundary, cd{0.0, 0.0}, nq);
            }
            p = np;
            q = nq;
            if (j == 0) {
                // The next row's scalar loads, after this row's LDS reads:
                // the two share a counter and return out of order, so a wait
                // for LDS reads with a scalar load outstanding waits for both.
                __builtin_amdgcn_sched_barrier(kAllButScalarLoads);
                g_next = ang_row(r + 1);
            }
        }
        load_row(r + kAhead, rp, rq);
        if constexpr (STEPS == K) put_row(u_out, r - K, p, q, Const<KEEP>{});
        __builtin_amdgcn_sched_barrier(0);  // rows stay apart: scheduled across them, they need more registers
    };

    // the first K rows: one step more takes its first row each time
    int r = rs0;
    auto head = [&](auto self, auto i) {
        constexpr int I = decltype(i)::value;
        if constexpr (I < K) {
            iteration(r, bp[I % kAhead], bq[I % kAhead], Const<I % kRing>{}, Const<I + 1>{}, Const<2>{});
            ++r;
            self(self, Const<I + 1>{});
        }
    };
    head(head, Const<0>{});
    auto rows = [&](auto self, auto u, auto check) {
        constexpr int I = decltype(u)::value + K;
        if constexpr (I < K + kRing) {
            iteration(r, bp[I % kAhead], bq[I % kAhead], Const<I % kRing>{}, Const<K>{}, check);
            ++r;
            self(self, Const<I - K + 1>{}, check);
        }
    };
    while (r + kRing - 1 <= rM) rows(rows, Const<0>{}, Const<0>{});
    // The last rows: one by one after the last whole group where a pass takes
    // one or two steps, whose tiles are often as short as one row (store runs,
    // us per step in groups and one by one: 1600 x 64 5.0 and 4.1, 3200 x 128 7.3
    // and 6.9).  In whole groups (rows past rE are dropped) where the registers
    // leave no room for more code: three steps (36 spilled), and two with user
    // coefficients and a source (6400 x 256 54 and 63 us).
    if constexpr (K == kMaxPassSteps || (K == 2 && SRC && !KERR)) {
        while (r <= rE) rows(rows, Const<0>{}, Const<1>{});
    } else {
        while (r + kRing - 1 <= rE) rows(rows, Const<0>{}, Const<1>{});
        auto tail = [&](auto self, auto u) {
            constexpr int I = decltype(u)::value + K;
            if constexpr (I < K + kRing - 1) {
                if (r > rE) return;
                iteration(r, bp[I % kAhead], bq[I % kAhead], Const<I % kRing>{}, Const<K>{}, Const<1>{});
                ++r;
                self(self, Const<I - K + 1>{});
            }
        };
        tail(tail, Const<0>{});
    }

    wave_lds_handover();
    if (e_id >= 0 && lane < K) {
        // lane j: the sample of step j's input
        double2* out = lane == 0 ? series0 : lane == 1 ? series1 : series2;
        if (out != nullptr) {
            cd w = {0.0, 0.0};
            auto add = [&](double wt, v2d a, v2d b) {
                w.re = fma(wt, fma(e_wr, b.x - a.x, a.x), w.re);
                w.im = fma(wt, fma(e_wr, b.y - a.y, a.y), w.im);
            };
            add(e_wa, smp[4 * lane], smp[4 * lane + 1]);
            if (e_rb >= 0) add(e_wb, smp[4 * lane + 2], smp[4 * lane + 3]);
            const int e_col = strip * kCols + e_lane - K;
            for (int e = 0; e <= e_id; ++e)  // the point and those equal to it
                if (ext[e].col == e_col && ext[e].rowa == e_ra) out[e] = double2{w.re, w.im};
        }
    }
}


// A tile of a single-grid launch.  SRC: the inhomogeneous variant (source
// profile src_i, src_h; time factors in A.sf).
template <int K, bool KERR, bool SRC, int KEEP>
__device__ __forceinline__ void pass_tile(const double2* __restrict__ u_in, double2* __restrict__ u_out,
                                          const double* __restrict__ rad, const double* __restrict__ ang,
                                          const double* __restrict__ uci, const double* __restrict__ uch,
                                          const ExtPoint* __restrict__ ext, double2* __restrict__ series_in,
                                          double2* __restrict__ series_mid, double2* __restrict__ win,
                                          const double2* __restrict__ src_i, const double2* __restrict__ src_h,
                                          const StepScalars& A, double* rad_s) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wpb = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int strip, chunk;
    if (A.order == kTileOrderDispatch) {
        const int tile = blockIdx.x * wpb + wave;
        strip = tile % A.n_strips;
        chunk = tile / A.n_strips;
    } else {  // XCD strips: workgroup b runs on XCD b % 8
        const int x = blockIdx.x % 8, q = (blockIdx.x / 8) * wpb + wave;
        const int s_lo = x * A.n_strips / 8, n_x = (x + 1) * A.n_strips / 8 - s_lo;
        if (n_x == 0) return;  // fewer strips than XCDs
        strip = s_lo + q % n_x;
        chunk = q / n_x;
    }
    if (chunk >= A.n_chunks) return;  // tiles beyond the last
    sweep<K, KERR, SRC, KEEP>((gin_t)u_in, (gout_t)u_out, (ctab_t)rad, (ctab_t)ang, (ctab_t)uci, (ctab_t)uch,
                              (cext_t)ext, series_in, series_mid, series_mid ? series_mid + A.n_ext : nullptr,
                              (gout_t)win, (lds_t)(rad_s + (threadIdx.x / kWave) * kSliceDoubles), A, strip, chunk, lane, (gin_t)src_i, (gin_t)src_h);
}

// Two wavefronts to a SIMD bar three steps with a source: its rows take 317
// registers (5 more spilled) and would spill 60 at two.  One alone is as fast as two where
// the grid has only that many tiles, and saves a third of the state's traffic
// (us per step in pairs and in threes: 3200 x 128 7.65 and 7.0, 5003 x 197
// 12.2 and 12.4, 6400 x 256 17.0 and 15.4, 12800 x 256 30.8 and 30.9,
// 25600 x 512 129 and 111).
#define TEUK_PASS_KERNEL(NAME, K)                                                                                     \
    template <bool KERR, bool SRC, int KEEP>                                                                          \
    __global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K == 3 && SRC ? 1 : 2, 4)))            \
        NAME(const double2* __restrict__ u_in, double2* __restrict__ u_out, const double* __restrict__ rad,           \
             const double* __restrict__ ang, const double* __restrict__ uci, const double* __restrict__ uch,          \
             const ExtPoint* __restrict__ ext, double2* __restrict__ series_in, double2* __restrict__ series_mid,     \
             double2* __restrict__ win, const double2* __restrict__ src_i, const double2* __restrict__ src_h,         \
             StepScalars A) {                                                                                         \
        extern __shared__ double rad_s[];                                                                             \
        pass_tile<K, KERR, SRC, KEEP>(u_in, u_out, rad, ang, uci, uch, ext, series_in, series_mid, win, src_i, src_h, \
                                      A, rad_s);                                                                      \
    }
TEUK_PASS_KERNEL(lw_step_kernel, 1)
TEUK_PASS_KERNEL(lw_step2_kernel, 2)
TEUK_PASS_KERNEL(lw_step3_kernel, 3)
#undef TEUK_PASS_KERNEL

// Small grids: k = A.bsteps steps in one launch.  A workgroup holds
// A.bcols = W + 2k consecutive columns by all ntheta rows in LDS, one point
// per thread, and takes k steps there; each step consumes one column at each
// edge (the stencil's radial reach), so after k steps its W middle columns
// hold the new state, which it writes back.  Every point's coefficients are
// built once per launch (the sweeps rebuild them every pass), so a step is
// the stencil arithmetic alone, in two phases with a barrier after each:
// stage 1 (the Pi half-step of row t needs the averages of rows t -/+ 1,
// which each thread forms itself from the state) and stage 2.  The
// expressions are those of the sweeps, operand for operand, so the results
// equal theirs bit for bit; columns outside the grid read the clamped
// edge column and, as in the sweeps, reach only the zeroed boundary columns.
// Extraction: the samples of each step's input state, in the sweeps' order.
// The points are read once per launch into LDS, each thread works out once
// which samples it takes, and the launch's series values stay in LDS until
// its last step: no global memory access inside the step loop, whose
// barriers would otherwise wait for it every step.
template <int KEEP>
__global__ void __launch_bounds__(1024)
    lw_block_kernel(const double2* __restrict__ u_in, double2* __restrict__ u_out, const double* __restrict__ rad,
                    const double* __restrict__ ang, const ExtPoint* __restrict__ ext, double2* __restrict__ series,
                    StepScalars A) {
    const int B = A.bcols, K = A.bsteps, W = B - 2 * K;
    const int nr = A.nr, nth = A.nth, P = A.pitch;
    const int j = threadIdx.x % B, t = threadIdx.x / B;  // blockDim.x == B * nth
    const int c0 = blockIdx.x * W;                       // first column written
    const int col = c0 - K + j;
    const int ci = min(max(col, 0), nr - 1), hi = min(max(col, 0), nr - 2);
    const int jl = max(j - 1, 0), jr = min(j + 1, B - 1);  // neighbours (clamped at the block's edges)
    const int me = t * B + j;
    const bool boundary = (col == 0) || (col == nr - 1);
    const double sg = (double)A.sigma;
    extern __shared__ double2 lds2[];
    cd* sp = reinterpret_cast<cd*>(lds2);  // [nth][B] Phi, Pi, h_Phi, h_Pi; then 2 per point samples
    cd* sq = sp + nth * B;
    cd* sh = sq + nth * B;
    cd* shq = sh + nth * B;
    cd* se = shq + nth * B;                      // [2 per point] this step's row samples
    cd* sbuf = se + 2 * kMaxBlockExt;            // [step][point] the launch's series values
    ExtPoint* sx = reinterpret_cast<ExtPoint*>(sbuf + kMaxBlockSteps * kMaxBlockExt);  // the points

    cd p = ld(u_in, (size_t)t * P + ci), q = ld(u_in, (size_t)t * P + ci + A.plane);
    const Ang G = load_ang(ang, nth, t);
    const SRad Rh = srad_of([&](int f) { return rad[((size_t)f * 2 + 1) * P + hi]; });
    const SRad Ri = srad_of([&](int f) { return rad[((size_t)f * 2 + 0) * P + ci]; });
    const Stage kh = stage_coef(Rh, G, ssigma(Rh, G), A.kap_h);
    const Stage ki = stage_coef(Ri, G, ssigma(Ri, G), A.kap_i);
    sp[me] = p;
    sq[me] = q;
    if ((int)threadIdx.x < A.n_ext) sx[threadIdx.x] = ext[threadIdx.x];
    // this thread's samples: bit 2e (row a of point e) and bit 2e + 1 (row
    // b), for the points whose column the workgroup writes
    unsigned duty = 0;
    for (int e = 0; e < A.n_ext; ++e) {
        const ExtPoint E = ext[e];
        if (E.col >= c0 && E.col < c0 + W && col == E.col) {
            if (t == E.rowa) duty |= 1u << (2 * e);
            else if (t == E.rowb) duty |= 2u << (2 * e);
        }
    }
    __syncthreads();

    for (int s = 0; s < K; ++s) {
        // stage 1 at (i+1/2, t): averages, the Phi half-step and the Pi
        // half-step, with the Phi averages of rows t -/+ 1 (or the pole
        // ghost rows) formed here from the state; samples
        const cd pr = sp[t * B + jr], qr = sq[t * B + jr];
        const cd U = cadd(p, pr), V = cadd(q, qr), dp = csub(pr, p), dq = csub(qr, q);
        const cd H = stage1_phi(kh.b, A.hdt, U, V, dp);
        sh[me] = H;
        for (unsigned d = duty; d != 0; d &= d - 1) {
            const int b = __builtin_ctz(d);
            const double wr = sx[b >> 1].wr;
            se[b] = {fma(wr, pr.re - p.re, p.re), fma(wr, pr.im - p.im, p.im)};
        }
        const cd Um = (t == 0) ? cscale(sg, U) : cadd(sp[me - B], sp[(t - 1) * B + jr]);
        const cd Up = (t == nth - 1) ? cscale(sg, U) : cadd(sp[me + B], sp[(t + 1) * B + jr]);
        const cd X = cadd(V, stage1_inc(kh, U, V, dp, dq, csub(U, Um)));
        const cd HQ = fma_real(kh.wp, csub(Up, U), X);
        shq[me] = HQ;
        __syncthreads();

        // stage 2 at (i, t); one thread per point forms its sample
        if ((int)threadIdx.x < A.n_ext) {
            const ExtPoint E = sx[threadIdx.x];
            if (E.col >= c0 && E.col < c0 + W) {
                const cd va = se[2 * threadIdx.x];
                cd acc = {fma(E.wa, va.re, 0.0), fma(E.wa, va.im, 0.0)};
                if (E.rowb >= 0) {
                    const cd vb = se[2 * threadIdx.x + 1];
                    acc = {fma(E.wb, vb.re, acc.re), fma(E.wb, vb.im, acc.im)};
                }
                sbuf[s * kMaxBlockExt + threadIdx.x] = acc;
            }
        }
        const cd Hl = sh[t * B + jl];
        const cd S = cadd(H, Hl), D = csub(H, Hl);
        const cd Sm = (t == 0) ? cscale(sg, S) : cadd(sh[me - B], sh[(t - 1) * B + jl]);
        const cd Sp = (t == nth - 1) ? cscale(sg, S) : cadd(sh[me + B], sh[(t + 1) * B + jl]);
        const cd HQl = shq[t * B + jl];
        const cd SQ = cadd(HQ, HQl), DQ = csub(HQ, HQl);
        cd np = fma_real(A.qdt, SQ, fma_real(-ki.b, D, p));
        cd nq = cadd(cadd(q, stage2_early(ki, S, D, csub(S, Sm))),
                     stage2_late(ki.b, ki.tr, ki.ti, ki.wp, SQ, DQ, csub(Sp, S)));
        if (boundary) {
            np = {0.0, 0.0};
            nq = {0.0, 0.0};
        }
        p = np;
        q = nq;
        sp[me] = p;
        sq[me] = q;
        __syncthreads();
    }
    if (j >= K && j < K + W && col < nr) {
        st_state<KEEP>(u_out, (size_t)t * P + col, p);
        st_state<KEEP>(u_out, (size_t)t * P + col + A.plane, q);
    }
    // the series values of the launch's steps (state row0 + s + 1 at series
    // row row0 + s; none for the initial state)
    if ((int)threadIdx.x < A.n_ext) {
        const ExtPoint E = sx[threadIdx.x];
        if (E.col >= c0 && E.col < c0 + W)
            for (int s = 0; s < K; ++s)
                if (A.row0 + s >= 0) {
                    const cd v = sbuf[s * kMaxBlockExt + threadIdx.x];
                    series[(size_t)(A.row0 + s) * A.n_ext + threadIdx.x] = double2{v.re, v.im};
                }
    }
}

// Small and medium grids: k = A.bsteps steps in one launch on tiles held in
// registers.  A wavefront holds 64 / C groups of C consecutive columns by R
// consecutive rows, one column a lane; a workgroup's groups are one below the
// other, a tile of C columns by G R rows (G groups).  Every point's state and
// coefficients stay in its lane's registers for the whole launch, so a step is
// the stencil arithmetic alone: column neighbours by cross-lane moves, row
// neighbours within the lane, and across groups through LDS, where each group
// leaves the sums (of Phi, and of H) of its first and last row; one barrier a
// step, with two buffers in turn.  Each step consumes one column at both edges
// and one row at each end that is not a pole; the tile's own part, what is
// left after k steps, is written back.  Tiles overlap by that much: redundant
// work in place of any synchronisation between workgroups, and of passes over
// memory.  The expressions are those of the sweeps, operand for operand.
//
// At a pole the group next to it takes its own row times sigma for the ghost.
// The first tile starts at row 0 and the last one ends at the last row; with
// R = 1 a tile may run past the last row of a grid it holds whole.
//
// Bound by the issue of about 94 vector instructions per point and step (three
// rows a lane, two wavefronts a SIMD: 1.13 us a step, 1.07 by that count at
// 2.1 GHz), and for one row a lane by the latency of a step's chain and its
// barrier (0.54 us against 0.36).  What a launch costs besides, 5-7 us (2.5
// between dependent launches, and the start of its workgroups), is spread over
// its steps.  us per step, before and now: 400 x 32 1.60 -> 1.28 (the block
// pass, then this), 200 x 16 1.18 -> 0.87, 1600 x 64 3.2 -> 2.2, 1600 x 128
// 6.9 -> 3.0, 1200 x 100 5.2 (sweeps of three steps) -> 2.0, 3200 x 128 5.9 ->
// 5.2; 5003 x 197 would take 11 against the sweeps' 9.
//
// T: most threads a workgroup may have: 1024 with one row a lane (at most 128
// registers; 100 used), 512 with two (256; 174) or three (244).
template <int C, int R, int T, int KEEP>
__global__ void __launch_bounds__(T)
    lw_tile_kernel(const double2* __restrict__ u_in, double2* __restrict__ u_out, const double* __restrict__ rad,
                   const double* __restrict__ ang, const ExtPoint* __restrict__ ext, double2* __restrict__ series,
                   StepScalars A) {
    constexpr int kEnds = R == 1 ? 1 : 2;
    const int K = A.bsteps, W = C - 2 * K;
    const int nr = A.nr, nth = A.nth, P = A.pitch;
    const int lane = threadIdx.x & (kWave - 1);
    const int j = lane % C, G = blockDim.x / C;
    const int g = threadIdx.x / C;
    const int strip = blockIdx.x % A.n_strips, tt = blockIdx.x / A.n_strips, n_tt = A.n_chunks;
    const int H = G * R;  // the tile's rows: its first, and its own
    const int own0 = tt == 0 ? 0 : H - K + (tt - 1) * (H - 2 * K);
    const int own1 = tt == n_tt - 1 ? nth : H - K + tt * (H - 2 * K);
    const int row0 = tt == 0 ? 0 : tt == n_tt - 1 ? nth - H : own0 - K;
    const int t0 = row0 + g * R;
    const int c0 = strip * W;  // first column written
    const int col = c0 - K + j;
    const int ci = min(max(col, 0), nr - 1), hi = min(max(col, 0), nr - 2);
    const bool boundary = (col == 0) || (col == nr - 1);
    const bool edge = c0 - K <= 0 || c0 - K + C >= nr;  // uniform: the tile holds a boundary column
    const double sg = (double)A.sigma;

    extern __shared__ double2 lds2[];
    // [buffer][first row, last row][U, S][group][column], then the samples' values
    v2d* xch = reinterpret_cast<v2d*>(lds2);
    const int plane = G * C, buf = kEnds * 2 * plane;
    v2d* smp = xch + 2 * buf;  // [step][point][row a, b][column, next column]
    const int me = g * C + j;
    // where the rows before the first and after the last are, and their factor
    const bool pole0 = t0 == 0, pole1 = t0 + R == nth;
    const int i_up = pole0 || g == 0 ? me : (kEnds - 1) * 2 * plane + me - C;
    const int i_dn = pole1 || g == G - 1 ? (kEnds - 1) * 2 * plane + me : me + C;
    const double f_up = pole0 ? sg : 1.0, f_dn = pole1 ? sg : 1.0;

    cd p[R], q[R];
    Stage kh[R], ki[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const size_t o = (size_t)min(t0 + r, nth - 1) * P + ci;
        p[r] = ld(u_in, o);
        q[r] = ld(u_in, o + A.plane);
    }
    const SRad Rh = srad_of([&](int f) { return rad[((size_t)f * 2 + 1) * P + hi]; });
    const SRad Ri = srad_of([&](int f) { return rad[((size_t)f * 2 + 0) * P + ci]; });
    // this lane's part in the samples: bit 4 e + 2 (row b) + (next column) of
    // its rows, for the points in the tile's own part
    unsigned duty[R] = {};
    unsigned any = 0;
    for (int e = 0; e < A.n_ext; ++e) {
        const ExtPoint E = ext[e];
        if (E.col < c0 || E.col >= c0 + W || E.rowa < own0 || E.rowa >= own1) continue;
        const int dc = col - E.col;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int t = t0 + r;
            if ((dc == 0 || dc == 1) && (t == E.rowa || t == E.rowb))
                duty[r] |= 1u << (4 * e + (t == E.rowa ? 0 : 2) + dc);
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
        if (any != 0) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                for (unsigned d = duty[r]; d != 0; d &= d - 1)
                    smp[s * 4 * kMaxBlockExt + __builtin_ctz(d)] = v2d{p[r].re, p[r].im};
        }
        v2d* x = xch + (s & 1) * buf;
        cd U[R], S[R], V[R], D[R], dp[R], dq[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const cd pr = from_right(p[r]), qr = from_right(q[r]);
            U[r] = cadd(p[r], pr);
            V[r] = cadd(q[r], qr);
            dp[r] = csub(pr, p[r]);
            dq[r] = csub(qr, q[r]);
            const cd H = stage1_phi(kh[r].b, A.hdt, U[r], V[r], dp[r]), Hl = from_left(H);
            S[r] = cadd(H, Hl);
            D[r] = csub(H, Hl);
            if (r == 0 || r == R - 1) {
                const int o = (r == 0 ? 0 : 2 * plane) + me;
                x[o] = v2d{U[r].re, U[r].im};
                x[o + plane] = v2d{S[r].re, S[r].im};
            }
        }
        __syncthreads();
        // the neighbours' rows are read at once, and arrive while the terms of
        // the rows themselves are formed
        const v2d x0 = x[i_up], x1 = x[i_up + plane], x2 = x[i_dn], x3 = x[i_dn + plane];
        __builtin_amdgcn_sched_barrier(0);
        cd e1[R], e2[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            e1[r] = stage1_inc0(kh[r], U[r], V[r], dp[r], dq[r]);
            e2[r] = stage2_early0(ki[r], S[r], D[r]);
            p[r] = fma_real(-ki[r].b, D[r], p[r]);
        }
        const cd Uu = {f_up * x0.x, f_up * x0.y}, Su = {f_up * x1.x, f_up * x1.y};
        const cd Ud = {f_dn * x2.x, f_dn * x2.y}, Sd = {f_dn * x3.x, f_dn * x3.y};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const cd dU = csub(U[r], r == 0 ? Uu : U[r > 0 ? r - 1 : 0]);
            const cd dS = csub(S[r], r == 0 ? Su : S[r > 0 ? r - 1 : 0]);
            const cd dUn = csub(r == R - 1 ? Ud : U[r < R - 1 ? r + 1 : r], U[r]);
            const cd dSn = csub(r == R - 1 ? Sd : S[r < R - 1 ? r + 1 : r], S[r]);
            const cd X = cadd(V[r], fma_real(-kh[r].wm, dU, e1[r]));
            const cd HQ = fma_real(kh[r].wp, dUn, X), HQl = from_left(HQ);
            const cd SQ = cadd(HQ, HQl), DQ = csub(HQ, HQl);
            p[r] = fma_real(A.qdt, SQ, p[r]);
            q[r] = cadd(cadd(q[r], fma_real(-ki[r].wm, dS, e2[r])),
                        stage2_late(ki[r].b, ki[r].tr, ki[r].ti, ki[r].wp, SQ, DQ, dSn));
        }
        if (edge) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                p[r] = {boundary ? 0.0 : p[r].re, boundary ? 0.0 : p[r].im};
                q[r] = {boundary ? 0.0 : q[r].re, boundary ? 0.0 : q[r].im};
            }
        }
    }
    if (j >= K && j < K + W && col < nr) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int t = t0 + r;
            if (t >= own0 && t < own1) {
                st_state<KEEP>(u_out, (size_t)t * P + col, p[r]);
                st_state<KEEP>(u_out, (size_t)t * P + col + A.plane, q[r]);
            }
        }
    }
    // the samples of the launch's input states (state row0 + s + 1 at series
    // row row0 + s; none for the initial state), step by step and point by point
    if (A.n_ext > 0) {
        __syncthreads();
        for (int i = threadIdx.x; i < K * A.n_ext; i += blockDim.x) {
            const int s = i / A.n_ext, e = i % A.n_ext;
            const ExtPoint E = ext[e];
            if (A.row0 + s < 0 || E.col < c0 || E.col >= c0 + W || E.rowa < own0 || E.rowa >= own1) continue;
            const v2d* v = smp + (s * kMaxBlockExt + e) * 4;
            cd w = {0.0, 0.0};
            auto add = [&](double wt, v2d a, v2d b) {
                w.re = fma(wt, fma(E.wr, b.x - a.x, a.x), w.re);
                w.im = fma(wt, fma(E.wr, b.y - a.y, a.y), w.im);
            };
            add(E.wa, v[0], v[1]);
            if (E.rowb >= 0) add(E.wb, v[2], v[3]);
            series[(size_t)(A.row0 + s) * A.n_ext + e] = double2{w.re, w.im};
        }
    }
}

__global__ void zero_ints_kernel(int* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Many grids in one persistent launch: the tiles of all members form one
// work list (member k owns tiles [tile_begin_k, tile_begin_{k+1})); each
// wavefront walks the list with a grid-wide stride.  All tiles have the
// same shape (64 - 2K columns x `rows` rows, ragged only at a member's edges),
// so the static stride balances uneven members.  `parity` selects which of
// each member's two state buffers is the input.  Three steps take 247 registers;
// 22 scalar registers, the member's pointers and scalars, are spilled into lanes.
template <int K, int KEEP>
__device__ __forceinline__ void batch_tiles(const BatchMember* __restrict__ members, int n_members, int total_tiles,
                                            int parity, const BatchSeries& S, double* rad_s) {
    const lds_t rs = (lds_t)(rad_s + (threadIdx.x / kWave) * kSliceDoubles);
    const int lane = threadIdx.x & (kWave - 1);
    const int wpb = blockDim.x / kWave;
    const int nwaves = gridDim.x * wpb;
    const int w0 = __builtin_amdgcn_readfirstlane(blockIdx.x * wpb + (threadIdx.x / kWave));
    for (int tile = w0; tile < total_tiles; tile += nwaves) {
        int lo = 0, hi = n_members - 1;  // last member with tile_begin <= tile
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (members[mid].tile_begin[K - 1] <= tile)
                lo = mid;
            else
                hi = mid - 1;
        }
        const BatchMember& M = members[lo];
        const int local = tile - M.tile_begin[K - 1];
        StepScalars k = M.k;
        k.n_strips = M.strips[K - 1];
        const int strip = local % k.n_strips;
        const int chunk = local / k.n_strips;
        auto row = [&](int j) -> double2* { return j < K && S.row[j] ? S.row[j] + M.ext_off : nullptr; };
        if (row(0) == nullptr && row(1) == nullptr && row(2) == nullptr) k.n_ext = 0;
        sweep<K, true, false, KEEP>((gin_t)M.u[parity], (gout_t)M.u[1 - parity], (ctab_t)M.rad, (ctab_t)M.ang, nullptr,
                                    nullptr, (cext_t)M.ext, row(0), row(1), row(2), nullptr, rs, k, strip, chunk, lane, nullptr,
                                    nullptr);
    }
}

#define TEUK_BATCH_KERNEL(NAME, K)                                                              \
    template <int KEEP>                                                                         \
    __global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 4)))          \
        NAME(const BatchMember* __restrict__ members, int n_members, int total_tiles, int parity, \
             BatchSeries S) {                                                                   \
        extern __shared__ double rad_s[];                                                       \
        batch_tiles<K, KEEP>(members, n_members, total_tiles, parity, S, rad_s);                \
    }
TEUK_BATCH_KERNEL(lw_batch_kernel, 1)
TEUK_BATCH_KERNEL(lw_batch2_kernel, 2)
TEUK_BATCH_KERNEL(lw_batch3_kernel, 3)
#undef TEUK_BATCH_KERNEL

// The state is stored as two planes in one buffer: u[f * nth * pitch + j *
// pitch + i], f = 0 for Phi and 1 for Pi.

// The row-wise kernels below take rows blockIdx.y, blockIdx.y + gridDim.y,
// ...: a launch's y dimension is capped (kMaxGridY) while ntheta may reach 2^20.
constexpr int kMaxGridY = 65535;

// Both planes of a state in one launch (blockIdx.z: Phi, Pi; export: from f0 on).
__global__ void import_kernel(const double2* __restrict__ phi, const double2* __restrict__ pi, double2* __restrict__ u,
                              int nr, int nth, int pitch) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, f = blockIdx.z;
    const double2* src = f == 0 ? phi : pi;
    if (i >= pitch) return;
    for (int j = blockIdx.y; j < nth; j += gridDim.y) {
        double2 v;
        v.x = 0.0;
        v.y = 0.0;
        if (i > 0 && i < nr - 1) v = src[(size_t)j * nr + i];
        u[(size_t)f * nth * pitch + (size_t)j * pitch + i] = v;
    }
}

__global__ void export_kernel(const double2* __restrict__ u, double2* phi, double2* pi,
                              int nr, int nth, int pitch, int f0) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, f = f0 + blockIdx.z;
    double2* dst = f == 0 ? phi : pi;
    if (i >= nr) return;
    for (int j = blockIdx.y; j < nth; j += gridDim.y)
        dst[(size_t)j * nr + i] = u[(size_t)f * nth * pitch + (size_t)j * pitch + i];
}

// Bilinear sample of Phi at one extraction point (rows rowa, rowb with the
// pole ghost signs folded into the weights).
__device__ __forceinline__ double2 sample_point(const double2* __restrict__ u, int pitch, const ExtPoint& E) {
    auto row = [&](int j) {
        const double2 a = u[(size_t)j * pitch + E.col];
        const double2 b = u[(size_t)j * pitch + E.col + 1];
        return cd{fma(E.wr, b.x - a.x, a.x), fma(E.wr, b.y - a.y, a.y)};
    };
    const cd va = row(E.rowa);
    cd v = {E.wa * va.re, E.wa * va.im};
    if (E.rowb >= 0) {
        const cd vb = row(E.rowb);
        v.re = fma(E.wb, vb.re, v.re);
        v.im = fma(E.wb, vb.im, v.im);
    }
    double2 w;
    w.x = v.re;
    w.y = v.im;
    return w;
}

__global__ void extract_kernel(const double2* __restrict__ u, int pitch, const ExtPoint* __restrict__ pts, int n,
                               double2* __restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    out[e] = sample_point(u, pitch, pts[e]);
}

// Psi(t_k, observer o) = sum over modes j of e^{i m_j phi_o} r_o^3 Phi_{m_j}(t_k, o)
// (the field from its azimuthal modes, Sec. 3.2); samples are
// [n_samples][n_modes][n_obs], psi [n_samples][n_obs].  The modes are summed
// in their given order.
__global__ void assemble_kernel(AssembleArgs A, int64_t n_samples, const double2* __restrict__ samples,
                                double2* __restrict__ psi) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= n_samples * A.n_obs) return;
    const int64_t k = id / A.n_obs;
    const int o = (int)(id % A.n_obs);
    double re = 0.0, im = 0.0;
    for (int j = 0; j < A.n_modes; ++j) {
        double sn, cs;
        sincos(A.m[j] * A.phi[o], &sn, &cs);
        const double2 f = samples[(k * A.n_modes + j) * A.n_obs + o];
        re = fma(cs, f.x, fma(-sn, f.y, re));
        im = fma(cs, f.y, fma(sn, f.x, im));
    }
    psi[id] = double2{A.r3[o] * re, A.r3[o] * im};
}

// Samples of every member's extraction points of a batch, in member order.
__global__ void batch_extract_kernel(const BatchExtPoint* __restrict__ pts, int n, int parity,
                                     double2* __restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const BatchExtPoint& P = pts[e];
    out[e] = sample_point(P.u[parity], P.pitch, P.e);
}

__global__ void nonfinite_kernel(const double2* __restrict__ u, int nr, int nth, int pitch, int* flag) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    for (int j = blockIdx.y; j < nth; j += gridDim.y) {
        const size_t o = (size_t)j * pitch + i;
        const double2 a = u[o], b = u[o + (size_t)nth * pitch];
        if (!isfinite(a.x) || !isfinite(a.y) || !isfinite(b.x) || !isfinite(b.y)) *flag = 1;
    }
}

// As nonfinite_kernel for the in-loop check: the first check (in stream
// order) that finds a non-finite value records its step count (>= 1).
__global__ void nonfinite_step_kernel(const double2* __restrict__ u, int nr, int nth, int pitch,
                                      unsigned long long* first, long long step) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    bool bad = false;
    for (int j = blockIdx.y; j < nth; j += gridDim.y) {
        const size_t o = (size_t)j * pitch + i;
        const double2 a = u[o], b = u[o + (size_t)nth * pitch];
        bad = bad || !isfinite(a.x) || !isfinite(a.y) || !isfinite(b.x) || !isfinite(b.y);
    }
    if (bad) atomicCAS(first, 0ull, (unsigned long long)step);
}

__global__ void pitch_copy_kernel(const double* __restrict__ src, double* __restrict__ dst, int rows, int cols,
                                  int pitch) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= pitch) return;
    for (int j = blockIdx.y; j < rows; j += gridDim.y)
        dst[(size_t)j * pitch + i] = (i < cols) ? src[(size_t)j * cols + i] : 0.0;
}

}  // namespace

template <int K>
static hipError_t launch_pass_k(const StepArgs& a, bool kerr, int waves_per_block, hipStream_t s) {
    // XCD orders: 8 equal shares of workgroups, each covering the tiles of
    // the largest XCD run of strips
    const int per_xcd = (a.k.n_strips + 7) / 8 * a.k.n_chunks;
    const int nb = a.k.order == kTileOrderDispatch
                       ? (a.k.n_strips * a.k.n_chunks + waves_per_block - 1) / waves_per_block
                       : 8 * ((per_xcd + waves_per_block - 1) / waves_per_block);
    const dim3 block(kWave * waves_per_block), grid(nb);
    const bool src = a.src_i != nullptr;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, waves_per_block * kRadSliceBytes, s, a.u_in, a.u_out, a.rad,
                           a.ang, a.uci, a.uch, a.ext, a.series, a.series_mid, a.win, a.src_i, a.src_h, a.k);
        return hipGetLastError();
    };
    auto pick = [&](auto k0, auto k1) { return go(a.k.keep ? k1 : k0); };
#define TEUK_PICK(KERR, SRC)                                                                       \
    if constexpr (K == 1) return pick(lw_step_kernel<KERR, SRC, 0>, lw_step_kernel<KERR, SRC, 1>); \
    if constexpr (K == 2) return pick(lw_step2_kernel<KERR, SRC, 0>, lw_step2_kernel<KERR, SRC, 1>); \
    if constexpr (K == 3) return pick(lw_step3_kernel<KERR, SRC, 0>, lw_step3_kernel<KERR, SRC, 1>);
    if (src && kerr) {
        TEUK_PICK(true, true)
    }
    if constexpr (K < 3) {
        if (src) {
            TEUK_PICK(false, true)
        }
        if (!kerr) {
            TEUK_PICK(false, false)
        }
    }
    TEUK_PICK(true, false)
#undef TEUK_PICK
}

hipError_t launch_pass(const StepArgs& a, int steps, bool kerr, int waves_per_block, hipStream_t s) {
    if (steps == 3 && kerr) return launch_pass_k<3>(a, kerr, waves_per_block, s);
    if (steps == 2) return launch_pass_k<2>(a, kerr, waves_per_block, s);
    if (steps == 1) return launch_pass_k<1>(a, kerr, waves_per_block, s);
    return hipErrorInvalidValue;
}

hipError_t launch_block(const StepArgs& a, hipStream_t s) {
    const int w = a.k.bcols - 2 * a.k.bsteps;
    const dim3 grid((a.k.nr + w - 1) / w), block(a.k.bcols * a.k.nth);
    static_assert(sizeof(ExtPoint) == 3 * sizeof(double2), "the points' LDS area");
    if (a.k.bsteps > kMaxBlockSteps || a.k.n_ext > kMaxBlockExt) return hipErrorInvalidValue;
    const size_t lds =
        (size_t)(4 * a.k.nth * a.k.bcols + 2 * kMaxBlockExt + kMaxBlockSteps * kMaxBlockExt + 3 * kMaxBlockExt) *
        sizeof(double2);
    hipLaunchKernelGGL(a.k.keep ? lw_block_kernel<1> : lw_block_kernel<0>, grid, block, lds, s, a.u_in, a.u_out,
                       a.rad, a.ang, a.ext, a.series, a.k);
    return hipGetLastError();
}

bool tile_grid(const TileShape& t, int nr, int nth, int steps, int* n_strips, int* n_chunks) {
    if (t.cols < 1 || t.waves < 1 || steps < 1) return false;
    const int w = t.cols - 2 * steps, rows = t.waves * kWave / t.cols * t.rows;
    if (w < 1) return false;
    *n_strips = (nr + w - 1) / w;
    *n_chunks = 1;
    if (rows >= nth) return rows == nth || t.rows == 1;
    // theta tiles: the first holds rows - steps of its own, the last ends at
    // the last row, those between rows - 2 steps
    const int mid = rows - 2 * steps;
    if (mid < 1) return false;
    *n_chunks = 2 + std::max(0, (nth - 2 * (rows - steps) + mid - 1) / mid);
    return true;
}

hipError_t launch_tile(const StepArgs& a, const TileShape& t, hipStream_t s) {
    StepArgs b = a;
    if (!tile_grid(t, a.k.nr, a.k.nth, a.k.bsteps, &b.k.n_strips, &b.k.n_chunks) || a.k.n_ext > kMaxBlockExt)
        return hipErrorInvalidValue;
    const int threads = t.waves * kWave;
    const size_t lds = (size_t)(2 * (t.rows == 1 ? 1 : 2) * 2 * threads + (a.k.n_ext > 0 ? 4 * kMaxBlockExt * a.k.bsteps : 0)) *
                       sizeof(double2);
    const dim3 grid(b.k.n_strips * b.k.n_chunks), block(threads);
    auto go = [&](auto k0, auto k1, int most) {
        if (threads > most) return hipErrorInvalidValue;
        hipLaunchKernelGGL(a.k.keep ? k1 : k0, grid, block, lds, s, b.u_in, b.u_out, b.rad, b.ang, b.ext, b.series, b.k);
        return hipGetLastError();
    };
#define TEUK_TILE(C, R, T) \
    if (t.cols == C && t.rows == R) return go(lw_tile_kernel<C, R, T, 0>, lw_tile_kernel<C, R, T, 1>, T);
    TEUK_TILE(16, 1, 1024)
    TEUK_TILE(32, 1, 1024)
    TEUK_TILE(64, 1, 1024)
    TEUK_TILE(32, 2, 512)
    TEUK_TILE(64, 2, 512)
    TEUK_TILE(64, 3, 512)
#undef TEUK_TILE
    return hipErrorInvalidValue;
}

hipError_t launch_zero_ints(int* p, int n, hipStream_t s) {
    hipLaunchKernelGGL(zero_ints_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_batch(const BatchMember* members, int n_members, int total_tiles, int parity, int n_blocks,
                        int waves_per_block, int steps, bool keep, const BatchSeries& series, hipStream_t s) {
    const int w = waves_per_block < 4 ? waves_per_block : 4;
    auto go = [&](auto k0, auto k1) {
        hipLaunchKernelGGL(keep ? k1 : k0, dim3(n_blocks), dim3(kWave * w), w * kRadSliceBytes, s, members, n_members,
                           total_tiles, parity, series);
        return hipGetLastError();
    };
    if (steps == 3) return go(lw_batch3_kernel<0>, lw_batch3_kernel<1>);
    if (steps == 2) return go(lw_batch2_kernel<0>, lw_batch2_kernel<1>);
    return go(lw_batch_kernel<0>, lw_batch_kernel<1>);
}

hipError_t launch_import(const double2* phi, const double2* pi, double2* u, int nr, int nth, int pitch,
                         hipStream_t s) {
    const dim3 block(256), grid((pitch + 255) / 256, std::min(nth, kMaxGridY), 2);
    hipLaunchKernelGGL(import_kernel, grid, block, 0, s, phi, pi, u, nr, nth, pitch);
    return hipGetLastError();
}

hipError_t launch_export(const double2* u, double2* phi, double2* pi, int nr, int nth, int pitch, hipStream_t s) {
    // outputs that overlap get Phi first, then Pi, as if copied one after the other
    const uintptr_t a = reinterpret_cast<uintptr_t>(phi), b = reinterpret_cast<uintptr_t>(pi);
    const uintptr_t bytes = (uintptr_t)nr * nth * sizeof(double2);
    const int planes = a < b + bytes && b < a + bytes ? 1 : 2;
    const dim3 block(256), grid((nr + 255) / 256, std::min(nth, kMaxGridY), planes);
    for (int f = 0; f < 2; f += planes)
        hipLaunchKernelGGL(export_kernel, grid, block, 0, s, u, phi, pi, nr, nth, pitch, f);
    return hipGetLastError();
}

hipError_t launch_extract(const double2* u, int pitch, const ExtPoint* pts, int n, double2* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const dim3 block(64), grid((n + 63) / 64);
    hipLaunchKernelGGL(extract_kernel, grid, block, 0, s, u, pitch, pts, n, out);
    return hipGetLastError();
}

hipError_t launch_batch_extract(const BatchExtPoint* pts, int n, int parity, double2* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const dim3 block(64), grid((n + 63) / 64);
    hipLaunchKernelGGL(batch_extract_kernel, grid, block, 0, s, pts, n, parity, out);
    return hipGetLastError();
}

hipError_t launch_assemble(const AssembleArgs& a, int64_t n_samples, const double2* samples, double2* psi,
                           hipStream_t s) {
    const int64_t n = n_samples * a.n_obs;
    if (n <= 0) return hipSuccess;
    const dim3 block(256), grid((unsigned)((n + 255) / 256));
    hipLaunchKernelGGL(assemble_kernel, grid, block, 0, s, a, n_samples, samples, psi);
    return hipGetLastError();
}

hipError_t launch_nonfinite(const double2* u, int nr, int nth, int pitch, int* flag, hipStream_t s) {
    const dim3 block(256), grid((nr + 255) / 256, std::min(nth, kMaxGridY));
    hipLaunchKernelGGL(nonfinite_kernel, grid, block, 0, s, u, nr, nth, pitch, flag);
    return hipGetLastError();
}

hipError_t launch_nonfinite_step(const double2* u, int nr, int nth, int pitch, long long* first, int64_t step,
                                 hipStream_t s) {
    const dim3 block(256), grid((nr + 255) / 256, std::min(nth, kMaxGridY));
    hipLaunchKernelGGL(nonfinite_step_kernel, grid, block, 0, s, u, nr, nth, pitch,
                       reinterpret_cast<unsigned long long*>(first), (long long)step);
    return hipGetLastError();
}

hipError_t launch_pitch_copy(const double* src, double* dst, int rows, int cols, int pitch, hipStream_t s) {
    const dim3 block(256), grid((pitch + 255) / 256, std::min(rows, kMaxGridY));
    hipLaunchKernelGGL(pitch_copy_kernel, grid, block, 0, s, src, dst, rows, cols, pitch);
    return hipGetLastError();
}

}  // namespace teuk
