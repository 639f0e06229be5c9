// Device-side building blocks shared by the forward step kernel
// (lw_kernels.hip) and the adjoint step kernel (adjoint_kernels.hip):
// complex helpers, cross-lane moves, the coefficient reconstruction of
// Eq. (1) from the 1-D radial and angular tables, and the pieces of S and D.
#pragma once

#include "internal.hpp"

namespace teuk {
namespace {

struct cd {
    double re, im;
};

__device__ __forceinline__ cd cadd(cd a, cd b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cd csub(cd a, cd b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cd cscale(double s, cd a) { return {s * a.re, s * a.im}; }

// Cross-lane moves: lane L receives the value held by lane L+1 / lane L-1,
// as two 32-bit DPP wavefront shifts (wave_shl:1 / wave_shr:1).  The edge
// lanes (63 and 0) receive 0; their results are never stored.
constexpr int kDppWaveShl1 = 0x130;
constexpr int kDppWaveShr1 = 0x138;

// bound_ctrl: a lane whose source lane does not exist reads 0, so the
// destination needs no initialisation.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double from_right(double v) { return dpp_move<kDppWaveShl1>(v); }
__device__ __forceinline__ double from_left(double v) { return dpp_move<kDppWaveShr1>(v); }
__device__ __forceinline__ cd from_right(cd v) { return {from_right(v.re), from_right(v.im)}; }
__device__ __forceinline__ cd from_left(cd v) { return {from_left(v.re), from_left(v.im)}; }

struct Ang {
    double sn2, cs, cotp, pd;
};

// Typed pointers for the tile sweep: state in global memory (address space
// 1) and the coefficient tables, read-only for a launch, in the constant
// address space (4), so that wavefront-uniform table reads become scalar
// loads even where the pointers come from a descriptor in memory.
typedef double v2d __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) v2d* gin_t;
typedef __attribute__((address_space(1))) v2d* gout_t;
typedef const __attribute__((address_space(4))) double* ctab_t;
typedef const __attribute__((address_space(4))) ExtPoint* cext_t;

__device__ __forceinline__ Ang load_ang(ctab_t ang, int nth, int j) {
    (void)nth;
    const size_t o = (size_t)j * kNumAng;
    Ang G;
    G.sn2 = ang[o + A_SN2];
    G.cs = ang[o + A_CS];
    G.cotp = ang[o + A_COTP];
    G.pd = ang[o + A_PD];
    return G;
}

__device__ __forceinline__ Ang load_ang(const double* ang, int nth, int j) {
    (void)nth;
    const size_t o = (size_t)j * kNumAng;
    Ang G;
    G.sn2 = ang[o + A_SN2];
    G.cs = ang[o + A_CS];
    G.cotp = ang[o + A_COTP];
    G.pd = ang[o + A_PD];
    return G;
}

// 1/Sigma and 1/Sigma^2 at one (position, row).
struct Sig {
    double isig, inv;
};

// Workgroups are dispatched round-robin over the 8 XCDs; map them so that
// each XCD (own L2) receives a contiguous range of tiles, i.e. neighbouring
// strips whose halo columns overlap.  Used by the adjoint kernels (measured
// slightly faster with it); the forward passes take dispatch order or, from 64
// strips on, runs of strips (kTileOrder*).
__device__ __forceinline__ int xcd_block(int b, int nb) {
    constexpr int X = 8;
    const int x = b % X, idx = b / X, per = nb / X, rem = nb % X;
    return x * per + min(x, rem) + idx;
}

// Loads always read a valid (clamped) address, so the load itself is
// unconditional and stays in flight until it is needed.
__device__ __forceinline__ cd ld(const double2* __restrict__ p, size_t o) {
    const double2 v = p[o];
    return {v.x, v.y};
}

__device__ __forceinline__ cd ld(gin_t p, size_t o) {
    const v2d v = p[o];
    return {v.x, v.y};
}

// Streaming store of one complex value (16 B, one dwordx4 per lane): the
// value is not read again by this launch and, for a window slot, not soon.
__device__ __forceinline__ void st(double2* p, size_t o, cd v) {
    v2d w;
    w.x = v.re;
    w.y = v.im;
    __builtin_nontemporal_store(w, reinterpret_cast<v2d*>(p + o));
}

__device__ __forceinline__ void st(gout_t p, size_t o, cd v) {
    v2d w;
    w.x = v.re;
    w.y = v.im;
    __builtin_nontemporal_store(w, p + o);
}

// Store of a state the next launch reads.  KEEP: an ordinary store, whose
// line stays in the device's last-level cache, so the next launch reads it
// from there when the states fit (the host picks the kernel instance);
// otherwise streaming, which leaves the cache to the input.  The choice is
// made at compile time: with a run-time branch between the two, the
// compiler merges them into one store to the same address and drops the
// non-temporal hint.
template <int KEEP>
__device__ __forceinline__ void st_state(double2* p, size_t o, cd v) {
    if constexpr (KEEP) {
        v2d w;
        w.x = v.re;
        w.y = v.im;
        *reinterpret_cast<v2d*>(p + o) = w;
    } else {
        st(p, o, v);
    }
}

template <int KEEP>
__device__ __forceinline__ void st_state(gout_t p, size_t o, cd v) {
    if constexpr (KEEP) {
        v2d w;
        w.x = v.re;
        w.y = v.im;
        p[o] = w;
    } else {
        st(p, o, v);
    }
}

// Row access through buffer resources.  A resource describes one row of one
// plane: its base address sits in scalar registers and each lane addresses
// its column by a fixed byte offset, so moving to another row costs scalar
// arithmetic only.  The hardware checks every lane's offset against the
// resource's size and drops a store that falls outside it: a lane that must
// not write gets the offset kOffNone, so stores need no branch on the lane
// mask, and the compiler's waits on the memory counter, which count every
// store on every path, stay as loose as the loads allow.
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
constexpr int kRsrcWord3 = 0x00020000;      // raw buffer, 32-bit data format
constexpr uint32_t kOffNone = 0x80000000u;  // past the end of any row (at most 2^24 columns, 256 MiB)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(gin_t row, int32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)row, (short)0, bytes, kRsrcWord3);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const double2* row, int32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double2*>(row), (short)0, bytes, kRsrcWord3);
}

__device__ __forceinline__ cd ld_row(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    const v2d v = __builtin_bit_cast(v2d, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    return {v.x, v.y};
}

// KEEP as in st_state: 0 streaming (non-temporal), 1 an ordinary store.
template <int KEEP>
__device__ __forceinline__ void st_row(__amdgpu_buffer_rsrc_t r, uint32_t off, cd v) {
    v2d w;
    w.x = v.re;
    w.y = v.im;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, w), r, off, 0, KEEP ? 0 : 2);
}

// Before a lane reads what other lanes of its wavefront wrote to LDS.  LDS
// operations of a wavefront are done in order, so nothing is waited for; it
// keeps the compiler, which sees one lane, from moving the reads up.
__device__ __forceinline__ void wave_lds_handover() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// sched_barrier mask: all classes the scheduler may move across, scalar
// memory not among them.
constexpr int kAllButScalarLoads = 0x3FF;

template <int V>
struct Const {
    static constexpr int value = V;
};

// ---- the two stages of a step -------------------------------------------
//
// Coefficients of one stage at one (position, row) with the step's factors
// folded in.  Stage 1 works on sums over the two columns of a half point,
// stage 2 on sums over the two halves of a column, so no average is halved:
// with U, V the sums of Phi, Pi, H = 2 h_Phi and HQ = 2 h_Pi,
//   half points:      b, c by dt/dr;   ct, a2, a1, v0 by dt/2
//   integer columns:  b, c by dt/2dr;  ct, a2, a1, v0 by dt/4
// wp, wm = a2 +- a1 are the weights of the theta differences to the next and
// from the previous row, A2 f'' + A1 f' = wp (f_{t+1} - f_t) - wm (f_t - f_{t-1}).
struct Stage {
    double b, cr, ci, tr, ti, wm, wp, vr, vi;
};

struct SRad {
    double rho2, a2d, b, k0, k1, k2, k3, tr, ti0, ti1, dl2, vr, vi;
};

template <class F>
__device__ __forceinline__ SRad srad_of(F f) {
    SRad R;
    R.rho2 = f(S_RHO2);
    R.a2d = f(S_A2D);
    R.b = f(S_B);
    R.k0 = f(S_K0);
    R.k1 = f(S_K1);
    R.k2 = f(S_K2);
    R.k3 = f(S_K3);
    R.tr = f(S_TR);
    R.ti0 = f(S_TI0);
    R.ti1 = f(S_TI1);
    R.dl2 = f(S_DL2);
    R.vr = f(S_VR);
    R.vi = f(S_VI);
    return R;
}

// 1/Sigma and 1/Sigma^2: the hardware reciprocal square root (about 23
// correct bits) and one cubic step, y <- y + y e (1/2 + 3/8 e) with e = 1 - x
// y^2, whose error is 5/16 e^3.
__device__ __forceinline__ Sig ssigma(const SRad& R, const Ang& G) {
    const double x = fma(-R.a2d, G.sn2, R.rho2);
    const double y = __builtin_amdgcn_rsq(x);
    const double t = x * y;
    const double e = fma(-t, y, 1.0);
    const double ye = y * e;
    const double z = fma(ye, fma(0.375, e, 0.5), y);
    return {z, z * z};
}

// kap: 1 over the factor of ct (c has the imaginary part -b ct_i).
__device__ __forceinline__ Stage stage_coef(const SRad& R, const Ang& G, Sig s, double kap) {
    Stage k;
    k.b = R.b * s.isig;
    k.tr = R.tr * s.inv;
    k.ti = fma(R.ti1, G.cs, R.ti0) * s.inv;
    const double c1 = fma(-R.k2, G.sn2, R.k1);
    const double c0 = fma(-R.k3, s.isig, fma(-c1, s.inv, R.k0));
    k.cr = c0 * s.inv;
    const double bt = k.b * k.ti;
    k.ci = -kap * bt;
    const double a2 = R.dl2 * s.inv;
    k.wp = fma(a2, G.cotp, a2);
    k.wm = fma(-a2, G.cotp, a2);
    k.vr = fma(R.dl2, G.pd, R.vr) * s.inv;
    k.vi = R.vi * s.inv;
    return k;
}

// sd, st: the factors of (b, c) and of the rest.
__device__ __forceinline__ Stage user_stage(ctab_t u, int nth, int pitch, int j, int pos, double inv_dth2,
                                            double inv_2dth, double sd, double st) {
    auto f = [&](int k) { return u[((size_t)k * nth + j) * pitch + pos]; };
    Stage k;
    k.b = f(U_B) * sd;
    k.cr = f(U_CRE) * sd;
    k.ci = f(U_CIM) * sd;
    k.tr = f(U_CTRE) * st;
    k.ti = f(U_CTIM) * st;
    const double a2 = f(U_A2) * inv_dth2 * st, a1 = f(U_A1) * inv_2dth * st;
    k.wp = a2 + a1;
    k.wm = a2 - a1;
    k.vr = f(U_V0RE) * st;
    k.vi = f(U_V0IM) * st;
    return k;
}

// H = 2 h_Phi = U + dt/2 V - b dp.
__device__ __forceinline__ cd stage1_phi(double b, double hdt, cd U, cd V, cd dp) {
    return {fma(-b, dp.re, fma(hdt, V.re, U.re)), fma(-b, dp.im, fma(hdt, V.im, U.im))};
}

__device__ __forceinline__ cd fma_real(double w, cd x, cd y) { return {fma(w, x.re, y.re), fma(w, x.im, y.im)}; }

// The increment of 2 h_Pi over V but for its terms of the neighbour rows:
// -c dp + b dq - ct V - v0 U.  Increments are summed on their own and added
// to the value once, so that they round at their own size.
__device__ __forceinline__ cd stage1_inc0(const Stage& k, cd U, cd V, cd dp, cd dq) {
    double r = k.b * dq.re, i = k.b * dq.im;
    r = fma(-k.cr, dp.re, r);
    i = fma(-k.cr, dp.im, i);
    r = fma(k.ci, dp.im, r);
    i = fma(-k.ci, dp.re, i);
    r = fma(-k.tr, V.re, r);
    i = fma(-k.tr, V.im, i);
    r = fma(k.ti, V.im, r);
    i = fma(-k.ti, V.re, i);
    r = fma(-k.vr, U.re, r);
    i = fma(-k.vr, U.im, i);
    r = fma(k.vi, U.im, r);
    i = fma(-k.vi, U.re, i);
    return {r, i};
}

// The same with the previous row's term, -wm (U_t - U_{t-1}).
__device__ __forceinline__ cd stage1_inc(const Stage& k, cd U, cd V, cd dp, cd dq, cd dU) {
    return fma_real(-k.wm, dU, stage1_inc0(k, U, V, dp, dq));
}

// The part of stage 2's Pi increment of the row itself, -c D - v0 S, with S, D
// the sum and difference of H at the two halves.
__device__ __forceinline__ cd stage2_early0(const Stage& k, cd S, cd D) {
    double r = -k.cr * D.re, i = -k.cr * D.im;
    r = fma(k.ci, D.im, r);
    i = fma(-k.ci, D.re, i);
    r = fma(-k.vr, S.re, r);
    i = fma(-k.vr, S.im, i);
    r = fma(k.vi, S.im, r);
    i = fma(-k.vi, S.re, i);
    return {r, i};
}

// What is known when a row arrives: the same with -wm (S_t - S_{t-1}).
__device__ __forceinline__ cd stage2_early(const Stage& k, cd S, cd D, cd dS) {
    return fma_real(-k.wm, dS, stage2_early0(k, S, D));
}

// The rest, once the next row is there: b DQ - ct SQ + wp (S_{t+1} - S_t),
// with SQ, DQ the sum and difference of HQ at the two halves.
__device__ __forceinline__ cd stage2_late(double b, double tr, double ti, double wp, cd SQ, cd DQ, cd dSn) {
    double r = b * DQ.re, i = b * DQ.im;
    r = fma(-tr, SQ.re, r);
    i = fma(-tr, SQ.im, i);
    r = fma(ti, SQ.im, r);
    i = fma(-ti, SQ.re, i);
    r = fma(wp, dSn.re, r);
    i = fma(wp, dSn.im, i);
    return {r, i};
}

}  // namespace
}  // namespace teuk
