// Internal declarations shared by the host library (teuk_api.cpp) and the
// gfx950 kernels (lw_kernels.hip).  Not part of the public ABI.
#pragma once

#include <cstddef>
#include <cstdint>

#include <hip/hip_runtime.h>

namespace teuk {

// Output columns per wavefront strip.  A wavefront's 64 lanes hold the 64
// consecutive columns c0-1 .. c0+62 of its strip; lane L computes the
// stage-1 value at the half point to the right of its column, so the
// columns c0 .. c0+61 (lanes 1..62) have both neighbouring half points.
constexpr int kWave = 64;
constexpr int kStripCols = kWave - 2;
// Output columns per strip of the two-step kernel: its second step needs the
// first step's results one column further out on each side, so lanes 2..61
// hold the output columns c0 .. c0+59 of a strip whose lanes hold c0-2 .. c0+61.
constexpr int kStripCols2 = kWave - 4;
// A pass of k steps has strips of 64 - 2k columns.
constexpr int kMaxPassSteps = 3;
constexpr int strip_cols(int k) { return kWave - 2 * k; }

// Radial table of the step's stage coefficients (stage_coef), each field a
// row of `pitch` doubles, field f of kind k (0: the columns r*_i, 1: the half
// points r*_{i+1/2}) in row 2 f + k, with the factors of its stage (d on b
// and c, t on the rest, see Stage).  With r, Delta, rho = r^2 + a^2 at the
// position:
enum SRadField : int {
    S_RHO2 = 0,  // rho^2
    S_A2D,       // a^2 Delta                 Sigma^2 = rho^2 - a^2 Delta sin^2
    S_B,         // d rho                     b = B / Sigma
    S_K0,        // -d rho (6 Delta/r + 2 s (r - 1))
    S_K1,        // d 2 r rho^2 Delta         Re c = (K0 - (K1 - K2 sin^2)/Sigma^2 - K3/Sigma)/Sigma^2
    S_K2,        // d a^2 (r - 1) rho Delta
    S_K3,        // d 2 s rho (r Delta - (r^2 - a^2))
    S_TR,        // t 2 s (r Delta - (r^2 - a^2))
    S_TI0,       // t 4 a m r                 Im Ct = (TI0 + TI1 cos)/Sigma^2
    S_TI1,       // t 2 s a Delta
    S_DL2,       // t Delta / dth^2
    S_VR,        // t (-m^2 a^2 - 6 Delta ((s+2) r^2 - (s+3) r + a^2) / r^2)
    S_VI,        // -t 2 s m a (r - 1)
    kNumSRad
};

// Angular table fields, stored row by row: [ntheta][kNumAng] doubles, so
// that one scalar load fetches all fields of a row.
enum AngField : int {
    A_SN2 = 0,  // sin^2 th
    A_CS,       // cos th
    A_COTP,     // cot th * dth / 2               A1/(2 dth) = A2/dth^2 * COTP
    A_PD,       // ((m + s cos th)^2 / sin^2 th - s) * dth^2   Re V0 = (DL2 PD + V0R)/Sigma^2
    kNumAng
};

// USER-mode coefficient order (matches TEUK_NCOEF in teuk.h).
enum UserCoef : int { U_B = 0, U_CRE, U_CIM, U_CTRE, U_CTIM, U_A2, U_A1, U_V0RE, U_V0IM, kNumUser };

// One extraction point: bilinear weights between columns col, col+1 and the
// rows rowa, rowb (rowb < 0: single row, ghost rows folded into the weights).
struct ExtPoint {
    int32_t col, rowa, rowb, pad;
    double wr, wa, wb, pad2;
};

// Scalar launch parameters of the step kernel (passed by value).
struct StepScalars {
    int32_t nr, nth, pitch, sigma;
    int32_t rows, n_strips, n_chunks, n_ext;
    int32_t zero;               // always 0 (an opaque row offset of LDS reads)
    int32_t keep;               // 1: the new state is written with ordinary stores (selects the kernel instance)
    int32_t order;              // passes of several steps: tile order (kTileOrder*)
    int32_t bsteps;             // block pass: steps per launch
    int32_t bcols;              // block pass: columns a workgroup holds (bsteps halo columns each side)
    int32_t pad_;
    int64_t row0;               // block pass: series row of the launch's first input state (-1: not sampled)
    int64_t plane;              // nth * pitch: offset of the Pi plane in a state
    double hdt, dt_dr, hdt_dr;
    double qdt;                 // dt / 4
    double kap_h, kap_i;        // 1 over the factor of ct: 2 / dt (half points), 4 / dt (columns)
    double inv_dth2, inv_2dth;  // USER mode scalings
    // source term (inhomogeneous variant): time factors of the pass's steps
    // times dt, sf[4s .. 4s+3] = dt f(t_n), dt f(t_n + dt/2) (re, im) of its step s
    double sf[4 * kMaxPassSteps];
};

// Tile order of the single-grid passes of two and three steps.  Dispatch: tile = workgroup
// x waves + wave, strips fastest; workgroups go round-robin over the 8 XCDs.
// XCD strips: each XCD takes one contiguous run of strips (its 1/8) in every
// theta chunk, so neighbouring strips (which share halo columns and 128-byte
// lines) and the chunks of a strip (which share the radial tables) meet in
// one L2; strips fastest within the XCD.
constexpr int kTileOrderDispatch = 0, kTileOrderXcdStrip = 1;

struct StepArgs {
    const double2* u_in;     // state: [Phi, Pi][nth][pitch]
    double2* u_out;
    const double* rad;       // [kNumSRad][2][pitch] (KERR)
    const double* ang;       // [nth][kNumAng]      (KERR)
    const double* uci;       // [kNumUser][nth][pitch] (USER, integer positions)
    const double* uch;       // [kNumUser][nth][pitch] (USER, half positions)
    const ExtPoint* ext;     // [n_ext]
    double2* series;         // n_ext samples of the input Phi, or nullptr
    double2* win;            // one-step pass: copy of the input state; two steps: the intermediate state; or nullptr
    double2* series_mid;     // passes of more steps: samples of Phi after the first step (then the second), or nullptr
    const double2* src_i;    // source profile at the integer positions, [nth][pitch], or nullptr
    const double2* src_h;    // source profile at the half positions, [nth][pitch]
    StepScalars k;
};

// One member of a batched launch (device-resident descriptor).
struct BatchMember {
    double2* u[2];           // the member's two state buffers
    const double* rad;       // its radial and angular tables (KERR)
    const double* ang;
    const ExtPoint* ext;     // its extraction points (k.n_ext of them), and the index of the
    int64_t ext_off;         // first among all members' points
    StepScalars k;           // its launch scalars (rows shared by all members)
    int32_t tile_begin[kMaxPassSteps];  // its first tile in the work list of the passes of 1, 2, 3 steps
    int32_t strips[kMaxPassSteps];      // its strips in these passes
};

// Where a batched launch of m steps puts the samples of the inputs of its
// steps: a row of all members' points each, or nullptr.
struct BatchSeries {
    double2* row[kMaxPassSteps];
};

// One extraction point of a batched evolution: the member's two state
// buffers (the current one is selected by the batch parity) and its point.
struct BatchExtPoint {
    const double2* u[2];
    int32_t pitch, pad;
    ExtPoint e;
};

// Mode sum at observers: up to kMaxModes modes and kMaxObservers points.
constexpr int kMaxModes = 64;
constexpr int kMaxObservers = 64;
struct AssembleArgs {
    int32_t n_modes, n_obs;
    int32_t m[kMaxModes];
    double phi[kMaxObservers], r3[kMaxObservers];
};

// Scalar launch parameters of the adjoint kernel.
struct AdjScalars {
    int32_t nr, nth, pitch, sigma;
    int32_t rows, n_strips, n_chunks, zero;  // zero: always 0 (an opaque row offset of LDS reads)
    int64_t plane;                           // nth * pitch: offset of the Pi plane in a state
    int32_t n_ext;                           // extraction points (fused transposed extraction)
    int32_t keep;                            // 1: lam_out and the tangent step's state with ordinary stores
                                             // (selects the kernel instance)
    double hdt, qdt, kap_h, kap_i;           // as in StepScalars
};

struct AdjArgs {
    const double2* nu_in;    // lambda^{m+1}, [Phi, Pi][nth][pitch]
    const double2* u_in;     // u^m
    double2* lam_out;        // lambda^m
    const double* rad;       // [kNumSRad][2][pitch]
    const double* rad_da;    // d/da of rad
    const double* ang;       // [nth][kNumAng]
    double* slots;           // [n_strips * n_chunks] spin-gradient partial sums (accumulated)
    const ExtPoint* ext;     // [n_ext] extraction points
    const double* gsample;   // gradient of the output state's sample, 2 doubles per point, or nullptr
    AdjScalars k;
};

// What a grid's tables are built from; d, t: the stages' factors of the two
// kinds of position (0: columns, 1: half points), see Stage.
struct TableArgs {
    double a, rmin, dr, dth, d[2], t[2];
    int32_t nr, nth, pitch, s, m;
};
// x_tab [2][pitch]: r - r_+ at the positions; rad [kNumSRad][2][pitch] (both
// nullptr: not built); ang [nth][kNumAng]; *failed = 1 if a position has no r.
hipError_t launch_tables(const TableArgs& a, double* x_tab, double* rad, double* ang, int* failed, hipStream_t s);
hipError_t launch_tables_da(const TableArgs& a, const double* x_tab, double* da, hipStream_t s);

// Launchers (lw_kernels.hip, adjoint_kernels.hip).  All return the
// hipError_t of the launch.
// 1, 2 or (Kerr coefficients) 3 steps in one pass; k.n_strips
// counted in strip_cols(steps)-column strips.
hipError_t launch_pass(const StepArgs& a, int steps, bool kerr, int waves_per_block, hipStream_t s);
// Small grids (ntheta <= kMaxBlockRows, Kerr coefficients): k.bsteps steps in
// one launch, each workgroup holding k.bcols columns x all rows in LDS
// (a.series: samples of the launch's input states, rows k.row0 + s).
constexpr int kMaxBlockRows = 64;
constexpr int kMaxBlockExt = 8;
constexpr int kMaxBlockSteps = 31;  // (64 columns - 2) / 2
hipError_t launch_block(const StepArgs& a, hipStream_t s);
// Tile pass (Kerr coefficients): k.bsteps steps in one launch on register
// tiles of `cols` (16, 32 or 64) columns, `rows` (1 to 3) rows a lane and
// `waves` wavefronts a workgroup (at most 16 with one row a lane, 8 with more).  A
// tile of one row a lane may hold all rows of the grid; otherwise the grid
// has more rows than a tile and a tile more than 2 x bsteps.  a.series as for
// launch_block, at most kMaxBlockExt points.
struct TileShape {
    int cols = 0, rows = 0, waves = 0;
};
hipError_t launch_tile(const StepArgs& a, const TileShape& t, hipStream_t s);
// Strips and theta tiles of a tile pass of `steps` steps; false if the shape
// does not apply.
bool tile_grid(const TileShape& t, int nr, int nth, int steps, int* n_strips, int* n_chunks);
// The same for adjoint steps, cotangents only: a.nu_in = lambda^{m+steps} ->
// a.lam_out = lambda^m, adding row g_row - s of gser ([rows][a.k.n_ext], or
// nullptr) after step s.
struct AdjTileArgs {
    int32_t steps, n_strips, n_chunks, pad;
    int64_t g_row;
};
struct AdjArgs;
hipError_t launch_adjoint_tile(const AdjArgs& a, const double2* gser, int64_t g_row, int steps, const TileShape& t,
                               hipStream_t s);
// Zero n ints (a fill kernel: usable where a memset node is not).
hipError_t launch_zero_ints(int* p, int n, hipStream_t s);
// steps per launch: 1, 2 or 3 (the work list of tile_begin[steps - 1]).
// keep: the members' next states with ordinary stores (StepScalars::keep).
// series: rows to sample (one point of a member per tile).
hipError_t launch_batch(const BatchMember* members, int n_members, int total_tiles, int parity, int n_blocks,
                        int waves_per_block, int steps, bool keep, const BatchSeries& series, hipStream_t s);
// Both planes of a state between the caller's arrays and the pitched layout.
hipError_t launch_import(const double2* phi, const double2* pi, double2* u, int nr, int nth, int pitch,
                         hipStream_t s);
hipError_t launch_export(const double2* u, double2* phi, double2* pi, int nr, int nth, int pitch, hipStream_t s);
hipError_t launch_extract(const double2* u, int pitch, const ExtPoint* pts, int n, double2* out, hipStream_t s);
hipError_t launch_batch_extract(const BatchExtPoint* pts, int n, int parity, double2* out, hipStream_t s);
hipError_t launch_assemble(const AssembleArgs& a, int64_t n_samples, const double2* samples, double2* psi,
                           hipStream_t s);
hipError_t launch_nonfinite(const double2* u, int nr, int nth, int pitch, int* flag, hipStream_t s);
// Records `step` in *first (if still 0) when the state holds a non-finite value.
hipError_t launch_nonfinite_step(const double2* u, int nr, int nth, int pitch, long long* first, int64_t step,
                                 hipStream_t s);
// Adjoint kernel variants: cotangents only (u_in, rad_da and slots are not
// read); with the spin gradient recomputed from u^m = u_in; with the spin
// gradient as the dot product of nu with T_m = u_in, the stored tangent.
enum class AdjMode { kCotangent, kSpin, kTangentDot };
// Their fused transposed extraction takes at most kRowHits points at a grid point.
constexpr int kRowHits = 3;
hipError_t launch_adjoint(const AdjArgs& a, int waves_per_block, AdjMode mode, hipStream_t s);
// Two cotangent adjoint steps: nu_in = lambda^{m+2} -> lam_out = lambda^m
// (k.n_strips counted in kStripCols2-column strips); a.gsample is the sample
// gradient added to lambda^{m+1}, gsample_b the one added to lambda^m.  With
// a.u_in = T_{m+1} and tan_b = T_m (stored tangents) the kernel also adds the
// spin gradient's dot products of both steps to a.slots.
hipError_t launch_adjoint2(const AdjArgs& a, const double* gsample_b, const double2* tan_b, int waves_per_block,
                           hipStream_t s);
// One step u_in -> u_out that also writes T = (dA/da) u_in to t_out (tiles of
// a.k: kStripCols-column strips, a.k.rows rows; a.rad_da the a-derivative tables).
hipError_t launch_tangent(const double2* u_in, double2* u_out, double2* t_out, const AdjArgs& a, int waves_per_block,
                          hipStream_t s);
// One step of the state and of its a-derivative v (u_in, v_in -> u_out,
// v_out; tiles as launch_tangent), with the samples of u_in and v_in at the
// first a.k.n_ext extraction points (at most one per tile; series_u/v may be
// nullptr).
hipError_t launch_spin_tangent(const double2* u_in, const double2* v_in, double2* u_out, double2* v_out,
                               double2* series_u, double2* series_v, const AdjArgs& a, int waves_per_block,
                               hipStream_t s);
// *out += sum Re(conj(g_i) t_i) over count complex values (stream order).
hipError_t launch_series_dot(const double2* g, const double2* t, int64_t count, double* out, hipStream_t s);
hipError_t launch_extract_adjoint(double2* lam, int pitch, const ExtPoint* pts, int n, const double2* g,
                                  hipStream_t s);
hipError_t launch_reduce_slots(const double* slots, int n, double* out, hipStream_t s);
hipError_t launch_zero_radial_boundary(double2* u, int nr, int nth, int pitch, hipStream_t s);
hipError_t launch_pitch_copy(const double* src, double* dst, int rows, int cols, int pitch, hipStream_t s);

}  // namespace teuk
