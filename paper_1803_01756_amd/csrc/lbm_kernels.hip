// HIP kernels (gfx950 / CDNA4) of the pseudopotential MRT lattice Boltzmann
// step with the coupled RK4 temperature update, arXiv:1803.01756 Section 2.
//
// Fused step layout.  Populations are structure-of-arrays planes
// [9][rows][pitch] of deviations d_i = f_i - w_i rho_ref (x fastest, pitch a
// multiple of 64), temperature a plane [rows][pitch] of T - T_ref.  Only the
// fluid rows are stored.  The buffers hold post-collision values, so a step
// pulls f_i(x) = f*_i(x - e_i), or f*_opp(i)(x) where x - e_i is a plate
// (half-way bounce-back), and writes f*(x) in place of its own node into the
// other buffer of the A-B pair.
//
// A workgroup takes a tile of up to seg_rows rows of a strip of 54 columns:
// kWaves waves of kRows consecutive rows each hold those rows and a halo of
// five rows on either side, one column per lane (lane l holds column
// strip*54 - 5 + l, periodic in x).  On all rows of the tile
//   A  pulls the row and computes rho, j, psi(rho, T),
//   B  computes the forces, u and, on its own rows, the MRT collision,
//   C..F evaluate the RK4 stages h1..h4,
// each stage on one row less at either end than the one before.  Neighbour
// columns come from the adjacent lanes through DPP wave shifts (a stage loses
// one valid lane per side, hence the 5-column halo), neighbour rows from the
// wave's own registers or, at its first and last row, through LDS with one
// barrier per stage.
//
// What bounds it (us per step, FP32): on a small grid (128 x 32, 5.5) the
// chain of stages of one workgroup, some 3.5 us, and the launch; on a middling
// one (2048 x 256, 15) that and the halo's arithmetic; on 8192 x 512 (85) the
// memory traffic: the same tiles with the arithmetic taken out take 76, with
// the loads and stores taken out 52, with either one alone 54 to 59.  A wave
// marching over a segment row by row, 10 halo iterations each, took 17.8, 31
// and 93 (FP64 2048 x 256 51 for 28 now, 8192 x 512 199 to 270 for 190).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "lbm_internal.h"

namespace lbmk {
namespace {

constexpr uint32_t kFreezeT = 1u, kSinglePhase = 2u, kEosCS = 32u, kPhaseProps = 128u,
                   kTopMixed = 256u;

// ---- lane shifts (DPP wave_shr:1 / wave_shl:1) ---------------------------
// at_xm(v): the value lane l-1 holds (column x-1); at_xp: lane l+1 (x+1).  The
// edge lanes (which lie in the halo) read 0.
__device__ __forceinline__ int dpp_shr1(int v) {
    return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true);
}
__device__ __forceinline__ int dpp_shl1(int v) {
    return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true);
}
__device__ __forceinline__ float at_xm(float v) { return __int_as_float(dpp_shr1(__float_as_int(v))); }
__device__ __forceinline__ float at_xp(float v) { return __int_as_float(dpp_shl1(__float_as_int(v))); }
__device__ __forceinline__ double at_xm(double v) {
    int2 w = *reinterpret_cast<int2*>(&v);
    w.x = dpp_shr1(w.x);
    w.y = dpp_shr1(w.y);
    return *reinterpret_cast<double*>(&w);
}
__device__ __forceinline__ double at_xp(double v) {
    int2 w = *reinterpret_cast<int2*>(&v);
    w.x = dpp_shl1(w.x);
    w.y = dpp_shl1(w.y);
    return *reinterpret_cast<double*>(&w);
}

// A row value at x kept as the centre c, the x-sum a = v(x+1) + v(x-1), the
// x-difference d = v(x+1) - v(x-1) and e = 4 c + a: every nine-point stencil
// of the step (Eq. 9 force, Eq. 16 gradient, Laplacian and divergence) uses
// only these per row, computed once when the row is produced.  In twelfths
// and sixths (N, C, S: the rows above, at and below)
//   12 d/dx = 4 d_C + d_N + d_S,   12 d/dy = e_N - e_S,
//    6 lap  = e_N + e_S + 4 a_C - 20 c_C.
template <class R>
struct Tri {
    R c, a, d, e;
};
template <class R>
__device__ __forceinline__ Tri<R> tri_of(R v, R m, R p) {
    Tri<R> t;
    t.c = v;
    t.a = p + m;
    t.d = p - m;
    t.e = (R)4 * v + t.a;
    return t;
}
template <class R>
__device__ __forceinline__ Tri<R> tri(R v) {
    return tri_of(v, at_xm(v), at_xp(v));
}
template <class R>
__device__ __forceinline__ Tri<R> tri_const(R v) {
    return tri_of(v, v, v);
}
template <class R>
__device__ __forceinline__ R dx12(const Tri<R>& S, const Tri<R>& C, const Tri<R>& N) {
    return (R)4 * C.d + (N.d + S.d);
}
template <class R>
__device__ __forceinline__ R dy12(const Tri<R>& S, const Tri<R>& N) {
    return N.e - S.e;
}

// ---- raw buffer access ------------------------------------------------------
// The planes are addressed through buffer resources: a wave-uniform byte
// offset (plane and row, scalar register) plus a per-lane byte offset (the
// column), so a load or store needs no per-lane 64-bit address arithmetic.
// num_records is the buffer size, so an access outside it reads 0 / is
// dropped by the hardware range check.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr int kBufWord3 = 0x00020000;  // gfx9 raw-buffer format word

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, kBufWord3);
}
__device__ __forceinline__ float bload(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, float) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}
__device__ __forceinline__ double bload(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, double) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
}
__device__ __forceinline__ void bstore(float v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)voff, (int)soff, 0);
}
__device__ __forceinline__ void bstore(double v, __amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)voff, (int)soff, 0);
}

// ---- rows -----------------------------------------------------------------
struct RowK {
    bool fluid;   // stored fluid row
    bool bb_lo;   // the row below is a plate (bounce-back of e_y = +1 links)
    bool bb_hi;   // the row above is a plate
    int sr;       // stored row index
};
__device__ __forceinline__ RowK row_info(int y, const Grid& g) {
    RowK r;
    if (g.periodic_y) {
        int yy = y % g.Ny;
        if (yy < 0) yy += g.Ny;
        r.fluid = true;
        r.bb_lo = r.bb_hi = false;
        r.sr = yy;
        return r;
    }
    r.fluid = (y >= 1 && y <= g.Ny - 2);
    r.bb_lo = (y == 1);
    r.bb_hi = (y == g.Ny - 2);
    r.sr = y - 1;
    return r;
}

// Pull of Eq. 12 for one stored row: f_i(x) = f*_i(x - e_i) or, across a
// plate, f*_opp(i)(x).  Velocity order of Eq. 2: 0 rest, 1 +x, 2 +y, 3 -x,
// 4 -y, 5 (+,+), 6 (-,+), 7 (-,-), 8 (+,-).
template <class S>
__device__ __forceinline__ void pull_row(const S* __restrict__ f, const Grid& g, const RowK& r,
                                         unsigned x, unsigned xm, unsigned xp, S d[9]) {
    const unsigned P = g.plane, pitch = (unsigned)g.pitch;
    const unsigned rc = (unsigned)r.sr * pitch;
    unsigned rdn, rup;
    if (g.periodic_y) {
        int a = r.sr - 1, b = r.sr + 1;
        if (a < 0) a += g.rows;
        if (b >= g.rows) b -= g.rows;
        rdn = (unsigned)a * pitch;
        rup = (unsigned)b * pitch;
    } else {
        rdn = rc - pitch;
        rup = rc + pitch;
    }
    const unsigned o0 = rc + x;
    const unsigned o1 = P + rc + xm;
    const unsigned o3 = 3 * P + rc + xp;
    const unsigned o2 = r.bb_lo ? 4 * P + rc + x : 2 * P + rdn + x;
    const unsigned o5 = r.bb_lo ? 7 * P + rc + x : 5 * P + rdn + xm;
    const unsigned o6 = r.bb_lo ? 8 * P + rc + x : 6 * P + rdn + xp;
    const unsigned o4 = r.bb_hi ? 2 * P + rc + x : 4 * P + rup + x;
    const unsigned o7 = r.bb_hi ? 5 * P + rc + x : 7 * P + rup + xp;
    const unsigned o8 = r.bb_hi ? 6 * P + rc + x : 8 * P + rup + xm;
    d[0] = f[o0];
    d[1] = f[o1];
    d[2] = f[o2];
    d[3] = f[o3];
    d[4] = f[o4];
    d[5] = f[o5];
    d[6] = f[o6];
    d[7] = f[o7];
    d[8] = f[o8];
}

// The same pull through a buffer resource.  vx, vm, vp: byte offsets of the
// lane's columns x, x-1, x+1; the uniform scalar offset carries the buffer's
// offset from the resource base (fb) plus the plane and row.
template <class S>
__device__ __forceinline__ void pull_row_buf(__amdgpu_buffer_rsrc_t f, const Grid& g,
                                             const RowK& r, unsigned fb, unsigned vx,
                                             unsigned vm, unsigned vp, S d[9]) {
    const unsigned P = g.plane * (unsigned)sizeof(S), pitch = (unsigned)g.pitch * sizeof(S);
    const unsigned rc = fb + (unsigned)r.sr * pitch;
    unsigned rdn, rup;
    if (g.periodic_y) {
        int a = r.sr - 1, b = r.sr + 1;
        if (a < 0) a += g.rows;
        if (b >= g.rows) b -= g.rows;
        rdn = fb + (unsigned)a * pitch;
        rup = fb + (unsigned)b * pitch;
    } else {
        rdn = rc - pitch;
        rup = rc + pitch;
    }
    const S t = S(0);
    d[0] = bload(f, vx, rc, t);
    d[1] = bload(f, vm, P + rc, t);
    d[3] = bload(f, vp, 3 * P + rc, t);
    if (r.bb_lo) {
        d[2] = bload(f, vx, 4 * P + rc, t);
        d[5] = bload(f, vx, 7 * P + rc, t);
        d[6] = bload(f, vx, 8 * P + rc, t);
    } else {
        d[2] = bload(f, vx, 2 * P + rdn, t);
        d[5] = bload(f, vm, 5 * P + rdn, t);
        d[6] = bload(f, vp, 6 * P + rdn, t);
    }
    if (r.bb_hi) {
        d[4] = bload(f, vx, 2 * P + rc, t);
        d[7] = bload(f, vx, 5 * P + rc, t);
        d[8] = bload(f, vx, 6 * P + rc, t);
    } else {
        d[4] = bload(f, vx, 4 * P + rup, t);
        d[7] = bload(f, vp, 7 * P + rup, t);
        d[8] = bload(f, vm, 8 * P + rup, t);
    }
}

// ---- arithmetic helpers -------------------------------------------------------
// FP32: the hardware reciprocal and square root (about 1 ulp) replace the
// IEEE division / correctly rounded square root sequences.  FP64 (the FP64
// storage build) keeps IEEE division and sqrt.
__device__ __forceinline__ float rcp_r(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_r(double x) { return 1.0 / x; }
__device__ __forceinline__ float sqrt_r(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double sqrt_r(double x) { return sqrt(x); }

// v held to [0, 1]
__device__ __forceinline__ float clamp01(float v) { return __builtin_amdgcn_fmed3f(v, 0.0f, 1.0f); }
__device__ __forceinline__ double clamp01(double v) { return fmin(fmax(v, 0.0), 1.0); }

// FP64 reciprocal square root from the FP32 hardware estimate (relative error
// ~1e-7) refined by Newton steps, each squaring the error: two steps reach
// ~1 ulp of FP64 (the FP64 build), one step ~1e-14 relative, far below what
// FP32 storage resolves (the FP32 builds).
template <int kSteps>
__device__ __forceinline__ double rsqrt_d(double x) {
    double y = (double)__builtin_amdgcn_rsqf((float)x);
    const double h = 0.5 * x;
#pragma unroll
    for (int i = 0; i < kSteps; ++i) y = y * fma(-h, y * y, 1.5);
    return y;
}

// Eqs. 10-11: psi = sqrt(2 (P_EOS(rho, T) - rho/3) / G), clamped at 0.
// FP64 throughout: the Shan-Chen force is a difference of neighbouring psi
// values and the FP32 rounding of psi itself would be of the order of that
// difference in a nearly uniform vapour.  With s = 1 + k (1 - sqrt(T/Tc)),
// D = 1 + 2 b rho - b^2 rho^2 the argument is the quotient N / Q,
//   N = (2/G) rho [R T D - (a s^2 rho + D/3) (1 - b rho)],  Q = (1 - b rho) D,
// and psi = |N| rsqrt(N Q): one reciprocal square root in place of a
// division and a square root.
// kF32: sqrt(T/Tc) in FP32 (its rounding enters phi as a smooth relative
// error, not a neighbour difference); the FP64 build takes it in FP64.
// The Carnahan-Starling option (flag kEosCS), e = b rho / 4:
//   P = rho R T (1 + e + e^2 - e^3) / (1 - e)^3 - a rho^2, Q = (1 - e)^3.
// kExt: the build that also serves the optional features (here the
// Carnahan-Starling EOS); the plain build leaves their code out.
// clamped: set when the argument is not positive (psi is then 0), the event
// the step counts per owned node.
template <bool kF32, bool kExt = true>
__device__ __forceinline__ double psi_eos(double rho, double T, const Phys& k, bool& clamped) {
    constexpr int kNewton = kF32 ? 1 : 2;
    double N, Q;
    if (kExt && (k.flags & kEosCS)) {
        const double e = 0.25 * k.b * rho, o = 1.0 - e;
        Q = o * o * o;
        N = k.R * T * (1.0 + e * (1.0 + e * (1.0 - e))) - (k.a * rho + 1.0 / 3.0) * Q;
    } else {
        const double x = T * k.inv_Tc;
        const double st = kF32 ? (double)__builtin_amdgcn_sqrtf((float)x) : x * rsqrt_d<2>(x);
        const double s = 1.0 + k.kappa * (1.0 - st);
        const double br = k.b * rho;
        const double omb = 1.0 - br;
        const double D = 1.0 + br * (2.0 - br);
        Q = omb * D;
        N = k.R * T * D - (k.a * (s * s) * rho + D * (1.0 / 3.0)) * omb;
    }
    N = k.two_inv_G * rho * N;
    const double arg = N * Q;  // the sign of N / Q
    clamped = !(arg > 0.0);
    // 0 where clamped, by a mask: the pair of v_cndmask_b32 a double's select
    // compiles to costs some 45 cycles on gfx950 (two in a row that read VCC),
    // one v_cndmask and two v_and 10
    int keep = clamped ? 0 : -1;
    asm("" : "+v"(keep));
    int2 w = __builtin_bit_cast(int2, fabs(N) * rsqrt_d<kNewton>(arg));
    w.x &= keep;
    w.y &= keep;
    return __builtin_bit_cast(double, w);
}

// Eq. 9 + Eq. 14 in one sum, per unit of the node's psi: the solid rows carry
// the effective potential psi_w G_w / G, so -G sum_i w_i phi(x + e_i) e_i
// times psi(x) is F_m + F_ads.
__device__ __forceinline__ void pair_force(const Tri<double>& pS, const Tri<double>& pC,
                                           const Tri<double>& pN, double negG12, double& ax,
                                           double& ay) {
    ax = negG12 * dx12(pS, pC, pN);
    ay = negG12 * dy12(pS, pN);
}

// Eq. 14 alone on the first / last fluid row, per unit of psi: the three
// links crossing a plate carry weight 1/3 + 2/12 = 1/2.
__device__ __forceinline__ double wall_adhesion_y(const RowK& r, const Phys& k) {
    double f = 0.0;
    if (r.bb_lo) f += 0.5 * k.Gw_psiw;
    if (r.bb_hi) f -= 0.5 * k.Gw_psiw;
    return f;
}

template <class R>
__device__ __forceinline__ const PhysR<R>& pr(const Phys& k);
template <>
__device__ __forceinline__ const PhysR<float>& pr<float>(const Phys& k) { return k.rf; }
template <>
__device__ __forceinline__ const PhysR<double>& pr<double>(const Phys& k) { return k.rd; }

// MRT collision, Eqs. 6-8, on deviations: m'_k = m_k - rho_ref (M w)_k.
// f* = M^-1 [m - Lambda (m - m_eq) + (I - Lambda/2) S] written out by the
// symmetry of the moments, with s_e = s_zeta (Eq. 3), so that the transform
// pair needs no nine moments (some 70 operations for 140): with
//   Q = [3 s_e rho u^2 + (1 - s_e/2) (6 u.F + 12 theta |F_m|^2 / (psi^2 (1/s_e - 1/2)))] / 36
// the even moments but the stresses give
//   each axis b = (1 - s_e) axis/4 + (s_e/9) drho + Q,    axis = d_1 + .. + d_4,
//   each diag c = (1 - s_e) diag/4 + (s_e/36) drho + Q,   diag = d_5 + .. + d_8,
//   rest      drho - 4 (b + c)  (the mass, to rounding);
// the x-odd moments (m*_3 = m_3 + F_x for any rate: the velocity holds half
// the force), with e_1 = d_1 - d_3 and e_5 the x-difference of the diagonals,
//   diag  +- X,  X = [s_q e_1 + (3 - 2 s_q) e_5 + F_x] / 12,
//   axis  +- (j_x + F_x - 4 X) / 2  (the momentum, to rounding),
// likewise in y, and the stresses m_7, m_8 a quarter of their relaxed value.
// Mass and momentum are closed by differences because coefficients rounded
// one by one would make them drift by some 3e-8 a step.
// Returns the post-collision deviations in d (overwritten); th: |F_m|^2 / psi^2.
template <class R>
__device__ __forceinline__ void collide(R d[9], R drho, R rho, R jx, R jy, R ux, R uy, R Fx, R Fy,
                                        R th, R sv, const PhysR<R>& c) {
    const R s13 = d[1] + d[3], s24 = d[2] + d[4], s57 = d[5] + d[7], s68 = d[6] + d[8];
    const R p57 = d[5] - d[7], p68 = d[6] - d[8];
    const R x1 = d[1] - d[3], x5 = p57 - p68, y1 = d[2] - d[4], y5 = p57 + p68;
    const R xx = ux * ux, yy = uy * uy;
    const R fx = ux * Fx, fy = uy * Fy;
    const R q = c.q_th * th + (c.q_F * (fx + fy) + c.q_u * (rho * (xx + yy)));
    const R t = c.se36 * drho + q;
    const R b0 = c.se4 * (s13 + s24) + (c.se12 * drho + t);
    const R c0 = c.se4 * (s57 + s68) + t;
    const R X5 = c.xc * x1 + (c.xd * x5 + Fx * ((R)1 / 12));
    const R Y5 = c.xc * y1 + (c.xd * y5 + Fy * ((R)1 / 12));
    const R X1 = (jx + Fx) - (R)4 * X5, Y1 = (jy + Fy) - (R)4 * Y5;
    // m* = m + S + s_v (m_eq - m - S/2)
    const R m7 = s13 - s24, m8 = s57 - s68;
    const R S7 = fx - fy, S8 = ux * Fy + uy * Fx;
    const R z7 = sv * (rho * (xx - yy) - (m7 + S7)) + ((R)2 * S7 + m7);
    const R z8 = sv * (rho * (ux * uy) - ((R)0.5 * S8 + m8)) + (S8 + m8);
    const R bp = b0 + (R)0.25 * z7, bm = b0 - (R)0.25 * z7;
    const R cp = c0 + (R)0.25 * z8, cm = c0 - (R)0.25 * z8;
    const R dp = X5 + Y5, dm = Y5 - X5;
    d[0] = drho - (R)4 * (b0 + c0);
    d[1] = bp + (R)0.5 * X1;
    d[3] = bp - (R)0.5 * X1;
    d[2] = bm + (R)0.5 * Y1;
    d[4] = bm - (R)0.5 * Y1;
    d[5] = cp + dp;
    d[7] = cp - dp;
    d[6] = cm + dm;
    d[8] = cm - dm;
}

// Per-row coefficients of K(T) (Eq. 16) with rho(n), u(n) frozen:
//   K = -(u . grad T) + q3 lap T - q1 T - q2 sqrt(T),
// using T (dP/dT)_rho = (A - B2) T + B1 sqrt(T), A = rho R / (1 - b rho),
// B1 = a k (1 + k) rho^2 / (sqrt(Tc) D), B2 = a k^2 rho^2 / (Tc D),
// D = 1 + 2 b rho - b^2 rho^2, and c = 1 / (rho C_v):
//   q1 = c div(u) (A - B2), q2 = c div(u) B1, q3 = c lambda.
// FP32 build: sqrt(T) is taken to second order about the row's T(n),
// sqrt(T) = s + (T - T_n)/(2 s) - (T - T_n)^2 / (8 s^3), s = sqrt(T_n), which
// turns the last two terms into -Q1 T - Q0 + q4 (T - T_n)^2 with
// Q1 = q1 + q2/(2 s), Q0 = q2 s / 2, q4 = q2 / (8 s^3) and needs one
// reciprocal square root per row instead of one square root per stage; with
// T = T_ref + t (stored deviation) the constant becomes Q0 + Q1 T_ref.  An RK
// stage moves T by some 1e-4 of it (1e-2 beside a plate in the first steps):
// to first order alone those steps leave T off by 6e-8.  The FP64 build keeps
// the exact sqrt.
// The stencils come in twelfths and sixths (see Tri), so the coefficients are
// kept as ux / 12, uy / 12 and q3 / 6, and in the FP32 build the centre's
// share of the Laplacian, 20 q3 / 6, is added to q1.
template <class R>
struct Coef {
    R ux, uy, q1, q2, q3, q4;
};
// dv12: 12 div(u).  lam6, glx, gly, inv_cv: a sixth of the conductivity at the
// node, its gradient and 1/C_v (constants unless lambda and C_v depend on the
// phase).  The conduction term [lambda lap T + grad(lambda).grad(T)] / (rho
// C_v) is carried as q3 lap T plus a shift of the advecting velocity by
// -grad(lambda) / (rho C_v).  amax > 0: where the diffusivity
// lambda / (rho C_v) exceeds amax the whole conduction term is scaled by
// amax over it (a departure from Eq. 17 that keeps the explicit RK4 of the
// conduction term inside its stability bound in thin vapour).
template <class R>
__device__ __forceinline__ Coef<R> heat_coef(R rho, R ux, R uy, R dv12, R Tn, R T_ref,
                                             const PhysR<R>& pc, bool cs, bool props,
                                             R lam6, R glx, R gly, R inv_cv, R amax) {
    R A, B, c;  // A = T-coefficient over rho C_v, B = rho / (C_v D)
    if (cs) {
        // Carnahan-Starling: T (dP/dT)_rho = rho R Z(e) T, no sqrt(T) term
        // (rkB1 = rkB2 = 0); inv = 1 / ((1 - e)^3 rho)
        const R e = (R)0.25 * pc.b * rho, o = (R)1 - e, o3 = o * o * o;
        const R inv = rcp_r(o3 * rho);
        A = rho * ((R)1 + e * ((R)1 + e * ((R)1 - e))) * inv;
        B = 0;
        c = inv_cv * (o3 * inv);
    } else {
        const R br = pc.b * rho;
        const R omb = (R)1 - br;
        const R D = (R)1 + br * ((R)2 - br);
        const R oD = omb * D;
        const R inv = rcp_r(oD * rho);  // 1 / ((1 - b rho) D rho)
        const R ri = rho * inv;
        A = D * ri;
        B = rho * (omb * ri);
        c = inv_cv * (oD * inv);
    }
    Coef<R> q;
    R cg = c;  // 1 / (rho C_v) as the conduction term sees it
    q.q3 = c * lam6;
    if (amax > (R)0 && q.q3 > amax * ((R)1 / 6)) {
        q.q3 = amax * ((R)1 / 6);
        cg = q.q3 * rcp_r(lam6);
    }
    q.ux = (props ? ux - cg * glx : ux) * ((R)1 / 12);
    q.uy = (props ? uy - cg * gly : uy) * ((R)1 / 12);
    const R dc = dv12 * ((R)1 / 12) * inv_cv;
    q.q1 = dc * (pc.rkA * A - pc.rkB2 * B);
    q.q2 = dc * (pc.rkB1 * B);
    if (sizeof(R) == 4) {
        const R rs = (R)__builtin_amdgcn_rsqf((float)Tn);  // 1 / sqrt(T_n)
        const R h = (R)0.5 * q.q2;
        q.q4 = (R)0.25 * h * (rs * (rs * rs));
        q.q1 = h * rs + q.q1;                // Q1
        q.q2 = h * (Tn * rs) + q.q1 * T_ref; // Q0 + Q1 T_ref
        q.q1 = (R)20 * q.q3 + q.q1;
    }
    return q;
}

// K(T) on the stage field (deviations tS, tC, tN of rows y-1, y, y+1), in the
// FP32 build without its q4 term (zero at the first stage; `bend` adds it).
template <class R>
__device__ __forceinline__ R heat_rhs(const Tri<R>& tS, const Tri<R>& tC, const Tri<R>& tN,
                                      const Coef<R>& q, R T_ref) {
    const R ring = (R)4 * tC.a + (tN.e + tS.e);
    const R tx = dx12(tS, tC, tN), ty = dy12(tS, tN);
    if (sizeof(R) == 4) return ((q.q3 * ring - q.q1 * tC.c) - q.ux * tx) - (q.uy * ty + q.q2);
    const R Tabs = T_ref + tC.c;
    const R adv_cond = q.q3 * (ring - (R)20 * tC.c) - (q.ux * tx + q.uy * ty);
    return adv_cond - q.q1 * Tabs - q.q2 * sqrt_r(Tabs);
}

template <class R>
__device__ __forceinline__ R bend(R h, const Coef<R>& q, R t, R tn) {
    if (sizeof(R) == 8) return h;
    const R dt = t - tn;
    return q.q4 * (dt * dt) + h;
}

// 12 times the divergence of u at row y from rows y-1 (S), y (C), y+1 (N)
template <class R>
__device__ __forceinline__ R div12_u(const Tri<R>& xS, const Tri<R>& xC, const Tri<R>& xN,
                                     const Tri<R>& yS, const Tri<R>& yN) {
    return dx12(xS, xC, xN) + dy12(yS, yN);
}

template <class S>
struct RealOf;
template <>
struct RealOf<float> {
    using T = float;
};
template <>
struct RealOf<double> {
    using T = double;
};

// sin(2 pi n / period): the part of a turn past the nearest whole number of
// periods (exact: one fma), folded to a quarter turn either way, and the
// Taylor series there (up to x^21 / 21!; the next term is below 2e-18).  A
// call of sin() took half a microsecond of the one wave that evaluates it, and
// the whole workgroup waits for that wave.  Beyond 2^53 turns n / period is no
// longer known to a turn and the first reduction leaves some over; the second
// (exact, and nothing below half a turn) keeps the series to its range.
__device__ double sin_of_period(long long n, double period, double inv_period) {
    const double t = (double)n;
    double a = __builtin_fma(-__builtin_rint(t * inv_period), period, t) * inv_period;
    a -= __builtin_rint(a);
    if (fabs(a) > 0.25) a = copysign(0.5, a) - a;
    const double x = a * 6.283185307179586, z = x * x;
    double p = 1.0 / 51090942171709440000.0;
    p = __builtin_fma(p, z, -1.0 / 121645100408832000.0);
    p = __builtin_fma(p, z, 1.0 / 355687428096000.0);
    p = __builtin_fma(p, z, -1.0 / 1307674368000.0);
    p = __builtin_fma(p, z, 1.0 / 6227020800.0);
    p = __builtin_fma(p, z, -1.0 / 39916800.0);
    p = __builtin_fma(p, z, 1.0 / 362880.0);
    p = __builtin_fma(p, z, -1.0 / 5040.0);
    p = __builtin_fma(p, z, 1.0 / 120.0);
    p = __builtin_fma(p, z, -1.0 / 6.0);
    return __builtin_fma(p * z, x, x);
}

// Open ends: the inlet density at time level n, the vapour-branch root of
// P_EOS(rho, T_in) = p0 (1 + p_amp sin(2 pi n / p_period)) (constant
// p0 (1 + p_amp) when p_period <= 0).  Cleared of its denominators the
// equation is a polynomial in e = b rho (RK: (1 - e) D; CS: e = b rho / 4,
// (1 - e)^3) whose sign is that of P - target.  Safeguarded Newton from rho_v
// inside (0, rho_sp), rho_sp the vapour spinodal; a step below 1e-9 of e is the
// last (the next would be of its square).  Every lane takes the same number of
// iterations (4 to 6), so a channel gets the same bits alone and in a batch.
// It is the step's longest chain before the first barrier: with the quotients
// and sin() it took 5 us of 15.7 (1600 x 48).
__device__ double inlet_density(const Phys& k, long long n) {
    const double p = k.p_period > 0.0
        ? k.p0 * (1.0 + k.p_amp * sin_of_period(n, k.p_period, k.inv_p_period))
        : k.p0 * (1.0 + k.p_amp);
    const double A = k.in_A, B = k.in_B;
    double c1, c2, c3, c4 = 0.0, c5 = 0.0;
    if (k.flags & kEosCS) {
        c1 = A + 3.0 * p;
        c2 = A - B - 3.0 * p;
        c3 = A + 3.0 * B + p;
        c4 = -(A + 3.0 * B);
        c5 = B;
    } else {
        c1 = A - p;
        c2 = 2.0 * A - B + 3.0 * p;
        c3 = B - A - p;
    }
    double lo = 0.0, hi = k.rho_sp * k.in_e, e = k.rho_v * k.in_e;
    for (int it = 0; it < 60; ++it) {
        const double F = __builtin_fma(__builtin_fma(__builtin_fma(__builtin_fma(__builtin_fma(
                             c5, e, c4), e, c3), e, c2), e, c1), e, -p);
        const double dF = __builtin_fma(__builtin_fma(__builtin_fma(__builtin_fma(
                              5.0 * c5, e, 4.0 * c4), e, 3.0 * c3), e, 2.0 * c2), e, c1);
        if (F < 0.0) lo = e; else hi = e;
        double y = __builtin_amdgcn_rcp(dF);
        y = __builtin_fma(__builtin_fma(-dF, y, 1.0), y, y);
        double en = __builtin_fma(-F, y, e);
        if (fabs(en - e) <= 1e-9 * e) return en * k.in_rho;
        if (!(en > lo && en < hi)) en = 0.5 * (lo + hi);
        e = en;
    }
    return e * k.in_rho;
}

// Zou-He on an open end (zero transverse velocity, prescribed density), in
// deviations d_i = f_i - w_i rho_ref (the rho_ref parts cancel): with
// J = rho u_x from the known populations, the inlet (x = 0) rebuilds d1, d5,
// d8, the outlet (x = Nx-1, density rho_v) d3, d6, d7.  A corner node (next
// to a plate) takes the velocity form with u = 0 (J = 0).
template <class R>
__device__ __forceinline__ void zou_he(R d[9], bool at_in, bool at_out, double rho_in,
                                       const Phys& k, bool corner) {
    const R dd = (R)0.5 * (d[2] - d[4]);
    if (at_in) {
        R J = (R)(rho_in - k.rho_ref) - (d[0] + d[2] + d[4] + (R)2 * (d[3] + d[6] + d[7]));
        if (corner) J = 0;
        d[1] = d[3] + J * ((R)2 / 3);
        d[5] = d[7] - dd + J * ((R)1 / 6);
        d[8] = d[6] + dd + J * ((R)1 / 6);
    }
    if (at_out) {
        R J = (R)(k.rho_ref - k.rho_v) + (d[0] + d[2] + d[4] + (R)2 * (d[1] + d[5] + d[8]));
        if (corner) J = 0;
        d[3] = d[1] - J * ((R)2 / 3);
        d[7] = d[5] + dd - J * ((R)1 / 6);
        d[6] = d[8] - dd - J * ((R)1 / 6);
    }
}

// Oscillating drive at time level n, evaluated on the device so that a channel
// run alone and inside a batch sees the same bits.
__device__ __forceinline__ double drive_at(const Phys& k, long long n) {
    return k.period > 0.0 ? k.g_osc * sin_of_period(n, k.period, k.inv_period) : 0.0;
}

// Add a wave's health word (see step_tile) to the counters: stat[0] gains
// the number of lanes (node columns of the wave's rows) that read a non-finite
// value, stat[1] the clamped Eq. 10 arguments.  Called by every lane of the
// wave; the sums and the atomics run only when some lane counted anything.
__device__ __forceinline__ void flush_health(unsigned long long* stat, unsigned health) {
    if (__builtin_amdgcn_ballot_w64(health != 0u) == 0ull) return;
    const unsigned long long bad = __builtin_amdgcn_ballot_w64((health >> 31) != 0u);
    unsigned clamp = health & 0x7fffffffu;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) clamp += __shfl_xor(clamp, off, 64);
    if ((threadIdx.x & (kLanes - 1)) == 0) {
        if (bad) atomicAdd(&stat[0], (unsigned long long)__builtin_popcountll(bad));
        if (clamp) atomicAdd(&stat[1], (unsigned long long)clamp);
    }
}

// ---- the step -------------------------------------------------------------------
// Rows a wave hands to the waves below [0] and above [1] it, stage by stage.
template <class R, int kWaves, bool kExt>
struct TileLds {
    double psi[kWaves][2][kLanes];
    R tn[kWaves][2][kLanes];
    R ux[kWaves][2][kLanes], uy[kWaves][2][kLanes];
    R st[3][kWaves][2][kLanes];
    R lam[kExt ? kWaves : 1][2][kLanes];
    R drive;
};

// One workgroup's tile of a step: strip `strip`, rows seg * seg_rows up.
// kExt compiles in the optional features (held and reservoir frames, the
// Carnahan-Starling EOS, open ends and plate temperature ramps,
// phase-dependent conductivity and heat capacity, the Sec. 3.2 plates); the
// plain instantiation is used whenever none is set.
template <class S, bool kMX, bool kExt, int kRows, int kWaves>
__device__ __forceinline__ void step_tile(const Grid& g, const Phys& k, const Bufs<S>& B,
                                          long long n, int strip, int seg,
                                          TileLds<typename RealOf<S>::T, kWaves, kExt>& L) {
    using R = typename RealOf<S>::T;
    const int lane = threadIdx.x & (kLanes - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // lane column and its periodic neighbours
    int cx = strip * kOwned - kHalo + lane;
    if (g.Nx >= kLanes) {  // at most one turn: -kHalo <= cx < Nx + kLanes
        cx += cx < 0 ? g.Nx : (cx >= g.Nx ? -g.Nx : 0);
    } else {
        cx %= g.Nx;
        if (cx < 0) cx += g.Nx;
    }
    const unsigned x = (unsigned)cx;
    const unsigned xm = (unsigned)(cx == 0 ? g.Nx - 1 : cx - 1);
    const unsigned xp = (unsigned)(cx == g.Nx - 1 ? 0 : cx + 1);
    const int own_w = min(kOwned, g.Nx - strip * kOwned);
    const bool own_lane = lane >= kHalo && lane < kHalo + own_w;
    // Lanes that store post-collision populations.  The collision is exact
    // on every lane but the outermost one of each side (its force needs psi
    // one column past the wave), so a wave holds its neighbours' first four
    // columns exactly.  A boundary between two strips that would split a
    // 64-byte chunk of a row into a part of at most four columns and the
    // rest is moved so that one wave writes the whole chunk: a row store then
    // makes fewer partial-chunk write requests, and every column is still
    // written by exactly one wave.  Rows start on 64-byte boundaries.  T(n+1)
    // is exact on the owned lanes only and keeps them.
    const int c0 = strip * kOwned;
    auto moved = [&](const int b, const int b_next) {
        constexpr int cpc = 64 / (int)sizeof(S), kMove = kHalo - 1;
        const int r = b % cpc;
        if (r == 0) return b;
        if (r <= kMove) return b - r;
        if (cpc - r <= kMove && b + (cpc - r) <= b_next) return b + (cpc - r);
        return b;
    };
    const int st_lo = strip > 0 ? moved(c0, c0 + own_w) : 0;
    const int st_hi = strip + 1 < g.n_strips ? moved(c0 + kOwned, min(c0 + 2 * kOwned, g.Nx))
                                             : c0 + own_w;
    const bool store_lane = c0 - kHalo + lane >= st_lo && c0 - kHalo + lane < st_hi;

    // The frame of a box: the outermost columns, and in a periodic box the
    // outermost rows.  FRAME_T holds its temperature (the RK right-hand
    // sides are zeroed there); FRAME_RHO makes it a reservoir at rest
    // (rho = rho_frame, u = 0, post-collision populations the rest
    // equilibrium of rho_frame).
    const bool edge_col = cx == 0 || cx == g.Nx - 1;
    auto on_frame = [&](const RowK& r) {
        return edge_col || (g.periodic_y && (r.sr == 0 || r.sr == g.rows - 1));
    };
    // Open ends (OPEN_X): the inlet column holds T = T_in (the outlet column
    // T = T_out when it is held), stencils past the ends see the end
    // column's own value (zero-gradient ghost), and the plates may carry a
    // temperature linear in x.
    const bool open_x = kExt && g.open_x != 0;
    const bool at_in = open_x && cx == 0, at_out = open_x && cx == g.Nx - 1;
    const bool out_held = at_out && k.hold_out != 0;
    auto held = [&](const RowK& r) {
        return (kExt && g.frame_t && on_frame(r)) || at_in || out_held;
    };
    auto trix = [&](auto v) {
        if (!open_x) return tri(v);
        auto m = at_xm(v), p = at_xp(v);
        if (at_in) m = v;
        if (at_out) p = v;
        return tri_of(v, m, p);
    };
    // The constants of the FP32 arithmetic.  Where a wave has registers to
    // spare (one row each, the build with the optional features) they are
    // kept in vector registers from the start: read from the kernel arguments
    // where they are used, each group waits for the scalar cache in every
    // stage of every wave (200 x 200: 9.4 us per step, so 8.2).  The plain build
    // would lose its second workgroup per CU (1111 x 77: 10.5 and 13.1 us).
    PhysR<R> kr = pr<R>(k);
    if (kExt && kRows == 1 && sizeof(R) == 4) {
        R* kv = reinterpret_cast<R*>(&kr);
#pragma unroll
        for (int i = 0; i < (int)(sizeof(kr) / sizeof(R)); ++i) asm("" : "+v"(kv[i]));
    }
    const R T_ref = kr.T_ref, dTw = kr.dT_wall;
    const bool ramp = kExt && k.wall_ramp != 0;
    const R dTw_x = ramp ? (R)(k.dT_wall + (k.dT_w_end - k.dT_wall) * (double)cx / (double)(g.Nx - 1))
                         : dTw;
    const bool frame_rho = kExt && g.frame_rho != 0;
    const bool props = kExt && (k.flags & kPhaseProps) != 0;
    const bool eos_cs = kExt && (k.flags & kEosCS) != 0;
    const bool freezeT = (k.flags & kFreezeT) != 0;
    const bool single = (k.flags & kSinglePhase) != 0;
    // Sec. 3.2 plates (TOP_MIXED): the bottom plate holds its own
    // temperature; the top plate holds T_w on the cold columns and elsewhere
    // mirrors the fluid row below it, stage by stage (zero normal gradient at
    // the half-way wall): `top` is what a temperature stencil of row r sees
    // above it, given the row above (N) and the row itself (C).
    const bool top_mixed = kExt && (k.flags & kTopMixed) != 0;
    const bool adiab = top_mixed && !(cx >= k.cold_x0 && cx < k.cold_x1);
    auto top = [&](const RowK& r, R N, R C) {
        return (kExt && top_mixed && r.bb_hi) ? (adiab ? C : dTw) : N;
    };

    // One buffer resource covers every buffer of the step (they share one
    // allocation); the lane's byte offset is its column, the uniform scalar
    // offset the buffer, plane and row.
    const unsigned esz = (unsigned)sizeof(S);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(B.base, B.span);
    const unsigned vx = x * esz, vm = xm * esz, vp = xp * esz, vlo = x * 4u;
    const unsigned rowb = (unsigned)g.pitch * esz, rowb_lo = (unsigned)g.pitch * 4u;
    const unsigned P = g.plane * esz;

    const int ya = g.y_first + seg * g.seg_rows;  // the tile's own rows
    const int yb = min(ya + g.seg_rows, g.y_first + g.rows);
    const int y0 = ya - kHalo + w * kRows;        // lattice row of the wave's row 0
    const int wS = max(w - 1, 0), wN = min(w + 1, kWaves - 1);
    // waves past the upper halo end here (a barrier waits for running waves)
    if (y0 >= yb + kHalo) return;

    // The wave's rows.  Rows past the tile's upper halo and plate rows are
    // not fluid; they load the first stored row (unused).
    RowK rk[kRows];
    S raw[kRows][9], rawT[kRows];
    float rawlo[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        rk[r] = row_info(y0 + r, g);
        if (y0 + r >= yb + kHalo) rk[r].fluid = false;
        const RowK rS = rk[r].fluid ? rk[r] : row_info(g.y_first, g);
        pull_row_buf<S>(rb, g, rS, B.fin, vx, vm, vp, raw[r]);
        rawT[r] = bload(rb, vx, B.Tin + (unsigned)rS.sr * rowb, S(0));
        rawlo[r] = kMX ? bload(rb, vlo, B.lo_in + (unsigned)rS.sr * rowb_lo, 0.0f) : 0.0f;
    }
    // the inlet density only where the strip holds the inlet column; the
    // drive by the first wave alone, which starts first and whose rows are
    // halo (by the last wave, 0.7 us later, everyone waited for it)
    const double rho_in = (open_x && __builtin_amdgcn_ballot_w64(at_in)) ? inlet_density(k, n) : 0.0;
    if (w == 0) L.drive = (R)drive_at(k, n);
    // health of the owned nodes (the state at level n), in one register:
    // bits 0-30 count the Eq. 10 arguments clamped to psi = 0 (at most one for
    // each of the lane's kRows rows), bit 31 is set once the lane has read a
    // non-finite rho or T
    unsigned health = 0;

    // ------------- A: pull, rho, j, psi ---------------------------------
    R d[kRows][9], rho[kRows], drho[kRows], jx[kRows], jy[kRows], tn[kRows];
    double psi[kRows], drd_[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        if (rk[r].fluid) {
            R* dc = d[r];
#pragma unroll
            for (int q = 0; q < 9; ++q) dc[q] = (R)raw[r][q];
            if (open_x) zou_he<R>(dc, at_in, at_out, rho_in, k, rk[r].bb_lo || rk[r].bb_hi);
            double drd;
            if (kMX) {
                drd = (double)dc[0] + (double)(R)rawlo[r];
#pragma unroll
                for (int q = 1; q < 9; ++q) drd += (double)dc[q];
            } else {
                R s = ((dc[0] + dc[1]) + (dc[2] + dc[3])) +
                      ((dc[4] + dc[5]) + (dc[6] + dc[7])) + dc[8];
                drd = (double)s;
            }
            jx[r] = (dc[1] - dc[3]) + ((dc[5] - dc[7]) - (dc[6] - dc[8]));
            jy[r] = (dc[2] - dc[4]) + ((dc[5] - dc[7]) + (dc[6] - dc[8]));
            if (frame_rho && on_frame(rk[r])) {
                drd = k.rho_frame - k.rho_ref;
                jx[r] = jy[r] = 0;
            }
            drho[r] = (R)drd;
            drd_[r] = drd;
            const double rho_d = k.rho_ref + drd;
            rho[r] = (R)rho_d;
            tn[r] = (R)rawT[r];
            const double Td = k.T_ref + (double)tn[r];
            bool clamped;
            psi[r] = psi_eos<sizeof(S) == 4, kExt>(rho_d, Td, k, clamped);
        } else {  // a plate row (or one that nothing reads)
            psi[r] = k.psi_wall_eff;
            tn[r] = (top_mixed && y0 + r <= 0) ? (R)k.dT_w_bot : dTw_x;
        }
    }
    L.psi[w][0][lane] = psi[0];
    L.psi[w][1][lane] = psi[kRows - 1];
    L.tn[w][0][lane] = tn[0];
    L.tn[w][1][lane] = tn[kRows - 1];
    __syncthreads();
    // ------------- B: forces, u, collision ------------------------------
    const R drive = L.drive;
    R ux[kRows], uy[kRows], lam[kRows];
    {
        Tri<double> pS = trix(L.psi[wS][1][lane]), pC = trix(psi[0]), pN;
        const double psi_up = L.psi[wN][0][lane];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int y = y0 + r;
            const RowK& rB = rk[r];
            pN = trix(r + 1 < kRows ? psi[r + 1 < kRows ? r + 1 : r] : psi_up);
            if (rB.fluid && y >= ya - 4 && y < yb + 4) {
                // force per unit of psi: F_m + F_ads (ax, ay), F_m alone (ax, am)
                double ax = 0.0, ay = 0.0, am = 0.0;
                if (!single) {
                    pair_force(pS, pC, pN, k.negG12, ax, ay);
                    am = ay;
                    if (rB.bb_lo || rB.bb_hi) am -= wall_adhesion_y(rB, k);
                } else {
                    ay = wall_adhesion_y(rB, k);
                }
                const R rh = rho[r];
                const R drv = rh - kr.rho_v;
                const R Fx = (R)(pC.c * ax) + (rh * drive + drv * kr.g_x);
                const R Fy = (R)(pC.c * ay) + drv * kr.g_y;
                const R rinv = rcp_r(rh);
                R u = (jx[r] + (R)0.5 * Fx) * rinv;
                R v = (jy[r] + (R)0.5 * Fy) * rinv;
                const bool resB = frame_rho && on_frame(rB);
                if (resB) u = v = 0;
                ux[r] = u;
                uy[r] = v;
                // Eq. 5 with a clamped fraction
                const R fr = clamp01((rh - kr.rho_g) * kr.inv_drho);
                if (props) lam[r] = (R)k.lambda + (R)(k.lam_l - k.lambda) * fr;
                if (y >= ya && y < yb) {
                    // Eq. 8 theta term uses |F_m|^2 / psi^2 of the fluid-fluid force
                    R th = 0;
                    if (!single && pC.c > 0.0) th = (R)(ax * ax + am * am);
                    const R sv = rcp_r(kr.tau_g + fr * kr.dtau);
                    R* dn = d[r];
                    collide<R>(dn, drho[r], rh, jx[r], jy[r], u, v, Fx, Fy, th, sv, kr);
                    if (resB) {
                        const double dr = k.rho_frame - k.rho_ref;
#pragma unroll
                        for (int q = 0; q < 9; ++q)
                            dn[q] = (R)((q == 0 ? 4.0 / 9 : (q < 5 ? 1.0 / 9 : 1.0 / 36)) * dr);
                    }
                    if (store_lane) {
                        // health of the node (state at level n): psi is 0
                        // exactly when Eq. 10 was clamped (a NaN too)
                        health += pC.c == 0.0 ? 1u : 0u;
                        if (!(__builtin_isfinite(rh) && __builtin_isfinite(tn[r])))
                            health |= 0x80000000u;
                        const unsigned so = B.fout + (unsigned)rB.sr * rowb;
                        if (kMX) {
                            // rest population takes whatever keeps sum_i d_i
                            // equal to the pre-collision deviation density
                            // (FP64), as (hi, lo)
                            double rest = drd_[r];
#pragma unroll
                            for (int q = 1; q < 9; ++q) rest -= (double)(S)dn[q];
                            const float hi = (float)rest;
                            bstore((S)hi, rb, vx, so);
                            bstore((float)(rest - (double)hi), rb, vlo,
                                   B.lo_out + (unsigned)rB.sr * rowb_lo);
                        } else {
                            bstore((S)dn[0], rb, vx, so);
                        }
#pragma unroll
                        for (int q = 1; q < 9; ++q) bstore((S)dn[q], rb, vx, q * P + so);
                    }
                }
            } else if (!rB.fluid) {  // solid nodes: u = 0, gas values
                ux[r] = uy[r] = 0;
                lam[r] = (R)k.lambda;
            }
            pS = pC;
            pC = pN;
        }
    }
    if (freezeT) {
        flush_health(B.stat, health);
        return;
    }
    L.ux[w][0][lane] = ux[0];
    L.ux[w][1][lane] = ux[kRows - 1];
    L.uy[w][0][lane] = uy[0];
    L.uy[w][1][lane] = uy[kRows - 1];
    if (kExt) {
        L.lam[w][0][lane] = lam[0];
        L.lam[w][1][lane] = lam[kRows - 1];
    }
    __syncthreads();
    // ------------- C: div u, coefficients, h1 ---------------------------
    R t[kRows], acc[kRows];
    Coef<R> cf[kRows];
    {
        Tri<R> xS = trix(L.ux[wS][1][lane]), xC = trix(ux[0]), xN;
        Tri<R> yS = trix(L.uy[wS][1][lane]), yC = trix(uy[0]), yN;
        Tri<R> tS = trix(L.tn[wS][1][lane]), tC = trix(tn[0]), tN;
        Tri<R> lS = tri_const<R>(0), lC = lS, lN = lS;
        if (props) {
            lS = trix(L.lam[kExt ? wS : 0][1][lane]);
            lC = trix(lam[0]);
        }
        const R x_up = L.ux[wN][0][lane], y_up = L.uy[wN][0][lane], t_up = L.tn[wN][0][lane];
        const R l_up = kExt ? L.lam[kExt ? wN : 0][0][lane] : (R)0;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int y = y0 + r, rn = r + 1 < kRows ? r + 1 : r;
            xN = trix(r + 1 < kRows ? ux[rn] : x_up);
            yN = trix(r + 1 < kRows ? uy[rn] : y_up);
            tN = trix(top(rk[r], r + 1 < kRows ? tn[rn] : t_up, tn[r]));
            if (props) lN = trix(r + 1 < kRows ? lam[rn] : l_up);
            t[r] = tn[r];
            if (rk[r].fluid && y >= ya - 3 && y < yb + 3) {
                const R dv = div12_u<R>(xS, xC, xN, yS, yN);
                R lam6 = kr.lam6, glx = 0, gly = 0, inv_cv = kr.inv_Cv;
                if (props) {
                    lam6 = lC.c * ((R)1 / 6);
                    glx = dx12(lS, lC, lN) * ((R)1 / 12);
                    gly = dy12(lS, lN) * ((R)1 / 12);
                    const R fr = clamp01((rho[r] - kr.rho_g) * kr.inv_drho);
                    inv_cv = rcp_r((R)(1.0 / k.inv_Cv) + (R)(k.cv_l - 1.0 / k.inv_Cv) * fr);
                }
                cf[r] = heat_coef<R>(rho[r], xC.c, yC.c, dv, T_ref + tC.c, T_ref, kr, eos_cs,
                                     props, lam6, glx, gly, inv_cv,
                                     kExt ? (R)k.alpha_max : (R)0);
                R h1 = heat_rhs<R>(tS, tC, tN, cf[r], T_ref);
                if (held(rk[r])) h1 = 0;
                acc[r] = h1;
                t[r] = tn[r] + (R)0.5 * h1;
            }
            xS = xC;
            xC = xN;
            yS = yC;
            yC = yN;
            tS = tC;
            tC = tN;
            lS = lC;
            lC = lN;
        }
    }
    // ------------- D, E: h2, h3 ------------------------------------------
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        L.st[s][w][0][lane] = t[0];
        L.st[s][w][1][lane] = t[kRows - 1];
        __syncthreads();
        const int reach = 2 - s;
        Tri<R> tS = trix(L.st[s][wS][1][lane]), tC = trix(t[0]), tN;
        const R t_up = L.st[s][wN][0][lane];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int y = y0 + r, rn = r + 1 < kRows ? r + 1 : r;
            tN = trix(top(rk[r], r + 1 < kRows ? t[rn] : t_up, t[r]));
            if (rk[r].fluid && y >= ya - reach && y < yb + reach) {
                R h = bend(heat_rhs<R>(tS, tC, tN, cf[r], T_ref), cf[r], tC.c, tn[r]);
                if (held(rk[r])) h = 0;
                acc[r] += (R)2 * h;
                t[r] = s == 0 ? tn[r] + (R)0.5 * h : tn[r] + h;
            }
            tS = tC;
            tC = tN;
        }
    }
    // ------------- F: h4, T(n+1) -------------------------------------------
    L.st[2][w][0][lane] = t[0];
    L.st[2][w][1][lane] = t[kRows - 1];
    __syncthreads();
    {
        Tri<R> tS = trix(L.st[2][wS][1][lane]), tC = trix(t[0]), tN;
        const R t_up = L.st[2][wN][0][lane];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int y = y0 + r, rn = r + 1 < kRows ? r + 1 : r;
            tN = trix(top(rk[r], r + 1 < kRows ? t[rn] : t_up, t[r]));
            if (rk[r].fluid && y >= ya && y < yb) {
                R h4 = bend(heat_rhs<R>(tS, tC, tN, cf[r], T_ref), cf[r], tC.c, tn[r]);
                if (held(rk[r])) h4 = 0;
                const R tnew = tn[r] + (acc[r] + h4) * ((R)1 / 6);
                if (own_lane) bstore((S)tnew, rb, vx, B.Tout + (unsigned)rk[r].sr * rowb);
            }
            tS = tC;
            tC = tN;
        }
    }
    flush_health(B.stat, health);
}

// Reads one word of every 64-byte line of the step's constants, so that the
// lines come into the scalar cache together at the start: read where they are
// needed, each costs a trip to memory in its turn, some 13 in all (0.2 to
// 0.5 us of every launch).  A batch's slots do not fit that cache together,
// and the same reads there cost 1.5 %.
template <size_t kBytes>
__device__ __forceinline__ void touch_kernarg() {
    const auto* p =
        (const __attribute__((address_space(4))) unsigned*)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int n = (int)((kBytes + 63) / 64);
    unsigned v[n];
#pragma unroll
    for (int i = 0; i < n; ++i) v[i] = p[16 * i];
#pragma unroll
    for (int i = 0; i < n; ++i) asm volatile("" ::"s"(v[i]));
}

template <class S, bool kMX, bool kExt, int kRows, int kWaves, int kPerSimd>
__global__ __launch_bounds__(kLanes* kWaves) __attribute__((amdgpu_waves_per_eu(kPerSimd)))
void step_kernel(Grid g, Phys k, Bufs<S> B, long long n) {
    touch_kernarg<sizeof(Grid) + sizeof(Phys) + sizeof(Bufs<S>) + sizeof(n)>();
    __shared__ TileLds<typename RealOf<S>::T, kWaves, kExt> L;
    int strip, seg;
    if (!tile_of_block(g, blockIdx.x, blockIdx.x & 7, n & 1, strip, seg)) return;  // whole workgroups only
    step_tile<S, kMX, kExt, kRows, kWaves>(g, k, B, n, strip, seg, L);
}

// Step i of a chunk over a batch of channels.  The slot of a block is found by
// a binary search over the slots' first blocks (multiples of eight, so that a
// slot's blocks meet the XCDs as those of a channel alone do).
template <bool kExt, int kRows, int kWaves, int kPerSimd>
__global__ __launch_bounds__(kLanes* kWaves) __attribute__((amdgpu_waves_per_eu(kPerSimd)))
void step_batched_kernel(const Slot* __restrict__ slots, int n_slots, int step_i) {
    __shared__ TileLds<float, kWaves, kExt> L;
    const int block = batch_block(blockIdx.x, gridDim.x, step_i);
    int lo = 0, hi = n_slots - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (slots[mid].block_begin <= block) lo = mid; else hi = mid - 1;
    }
    const Slot& sl = slots[lo];
    if (step_i >= sl.steps_left) return;
    // local copies: the buffer stores of the step may alias the table as far
    // as the compiler can tell, which would force reloads
    const Grid g = sl.g;
    const Phys k = sl.k;
    const long long n = sl.n0 + step_i;
    int strip, seg;
    if (!tile_of_block(g, block - sl.block_begin, blockIdx.x & 7, false, strip, seg)) return;
    Bufs<float> B;
    B.base = sl.mem;
    B.span = sl.span;
    const int a = (sl.cur_f + step_i) & 1;
    B.fin = sl.off_f[a];
    B.fout = sl.off_f[a ^ 1];
    B.lo_in = B.lo_out = 0;
    B.stat = sl.stat;
    if (sl.k.flags & kFreezeT) {
        B.Tin = B.Tout = sl.off_T[sl.cur_T];
    } else {
        const int t = (sl.cur_T + step_i) & 1;
        B.Tin = sl.off_T[t];
        B.Tout = sl.off_T[t ^ 1];
    }
    step_tile<float, false, kExt, kRows, kWaves>(g, k, B, n, strip, seg, L);
}

// ---- moments ----------------------------------------------------------------
// a node of a FRAME_RHO reservoir (y counts the plate rows)
__device__ __forceinline__ bool reservoir_node(const Grid& g, int cx, int y) {
    return g.frame_rho &&
           (cx == 0 || cx == g.Nx - 1 || (g.periodic_y && (y == 0 || y == g.Ny - 1)));
}

// The read-out's arithmetic per node, shared by the read-out and the
// one-pass reduction, so that both see bitwise the same node values.
struct NodeState {
    double rho, psi, jx, jy, T;  // rho = 0 and j = 0 on plate rows
    bool fluid;
};

// rho, psi, j and T of node (cx, y) (y counts the plate rows) at time level
// n_t from the stored post-collision state.
template <class S, bool kMX>
__device__ __forceinline__ NodeState node_state(const Grid& g, const Phys& k,
                                                const S* __restrict__ f,
                                                const float* __restrict__ f0lo,
                                                const S* __restrict__ T, int cx, int y,
                                                long long n_t) {
    NodeState o;
    const RowK r = row_info(y, g);
    o.fluid = r.fluid;
    if (!r.fluid) {
        o.psi = k.psi_wall_eff;
        o.jx = o.jy = 0.0;
        o.rho = 0.0;
        o.T = k.T_ref + (k.wall_ramp ? k.dT_wall + (k.dT_w_end - k.dT_wall) * (double)cx /
                                                       (double)(g.Nx - 1)
                         : ((k.flags & kTopMixed) && y == 0) ? k.dT_w_bot
                                                             : k.dT_wall);
        return o;
    }
    const unsigned x = (unsigned)cx;
    const unsigned xm = (unsigned)(cx == 0 ? g.Nx - 1 : cx - 1);
    const unsigned xp = (unsigned)(cx == g.Nx - 1 ? 0 : cx + 1);
    S d[9];
    pull_row<S>(f, g, r, x, xm, xp, d);
    if (g.open_x && (cx == 0 || cx == g.Nx - 1)) {
        using R = typename RealOf<S>::T;
        R dr_[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) dr_[q] = (R)d[q];
        zou_he<R>(dr_, cx == 0, cx == g.Nx - 1, cx == 0 ? inlet_density(k, n_t) : 0.0, k,
                  r.bb_lo || r.bb_hi);
#pragma unroll
        for (int q = 0; q < 9; ++q) d[q] = (S)dr_[q];
    }
    double dr = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) dr += (double)d[q];
    if (kMX) dr += (double)f0lo[(unsigned)r.sr * (unsigned)g.pitch + x];
    const bool res = reservoir_node(g, cx, y);
    if (res) dr = k.rho_frame - k.rho_ref;
    o.rho = k.rho_ref + dr;
    o.T = k.T_ref + (double)T[(unsigned)r.sr * (unsigned)g.pitch + x];
    bool clamped;
    o.psi = psi_eos<sizeof(S) == 4>(o.rho, o.T, k, clamped);
    o.jx = ((double)d[1] - (double)d[3]) + ((double)d[5] - (double)d[6]) +
           ((double)d[8] - (double)d[7]);
    o.jy = ((double)d[2] - (double)d[4]) + ((double)d[5] + (double)d[6]) -
           ((double)d[7] + (double)d[8]);
    if (res) o.jx = o.jy = 0.0;
    return o;
}

// u of a fluid node (Eq. 13) from its rho and j and the psi of the rows
// below (pS), at (pC) and above (pN) it, each as centre / x-sum / x-difference.
__device__ __forceinline__ void node_velocity(const Grid& g, const Phys& k, int cx, int y,
                                              const Tri<double>& pS, const Tri<double>& pC,
                                              const Tri<double>& pN, double rho, double jx,
                                              double jy, long long n_t, double& ux,
                                              double& uy) {
    const RowK r = row_info(y, g);
    double ax = 0.0, ay = 0.0;
    if (!(k.flags & kSinglePhase))
        pair_force(pS, pC, pN, k.negG12, ax, ay);
    else
        ay = wall_adhesion_y(r, k);
    const double Fx = pC.c * ax + (rho * drive_at(k, n_t) + (rho - k.rho_v) * k.g_x);
    const double Fy = pC.c * ay + (rho - k.rho_v) * k.g_y;
    ux = (jx + 0.5 * Fx) / rho;
    uy = (jy + 0.5 * Fy) / rho;
    if (reservoir_node(g, cx, y)) ux = uy = 0.0;
}

// the x-neighbours the read-out uses: periodic, or past an open end the end
// column itself
__device__ __forceinline__ int read_xm(const Grid& g, int cx) {
    return cx == 0 ? (g.open_x ? 0 : g.Nx - 1) : cx - 1;
}
__device__ __forceinline__ int read_xp(const Grid& g, int cx) {
    return cx == g.Nx - 1 ? (g.open_x ? cx : 0) : cx + 1;
}

// rho, u and T of every node.  A workgroup takes 64 columns of 4 x kReadRows
// rows: each wave evaluates its own kReadRows rows (kept in registers but for
// psi), the ring of one node around the block goes round in one more
// evaluation by the first threads, and u follows from the psi in LDS.  The
// outputs may be device memory or, for small results (ReadoutPlan), pinned host
// memory: a wave's stores of 64 consecutive doubles cross the link at 44 GB/s at
// 2.5 MB, 54 at 17, 56 at 134 (the link's rate), and one launch that writes the
// host arrays (13 us for 128 x 32) stands for a clearing, two passes over the
// nodes with psi and j between them in memory, and five copies (95 us).
// Non-finite nodes are counted per workgroup into bad[], every entry written
// on each launch, and the step's counters go along into words[]: both pinned
// host memory, so that the read-out needs no copy of its own for them.
constexpr int kReadRows = 2;
constexpr int kReadW = 64, kReadH = 4 * kReadRows;

template <class S, bool kMX>
__global__ __launch_bounds__(256) void moments_kernel(Grid g, Phys k, const S* __restrict__ f,
                                                      const float* __restrict__ f0lo,
                                                      const S* __restrict__ T, Moments out,
                                                      long long n_t,
                                                      const unsigned long long* __restrict__ stat,
                                                      Readout ro) {
    __shared__ double psi_t[kReadH + 2][kReadW + 2];
    __shared__ unsigned cnt[4];
    const int tiles_x = (g.Nx + kReadW - 1) / kReadW;
    const int x0 = ((int)blockIdx.x % tiles_x) * kReadW, y0 = ((int)blockIdx.x / tiles_x) * kReadH;
    const int tx = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (blockIdx.x == 0 && threadIdx.x < kStepWords) ro.words[threadIdx.x] = stat[threadIdx.x];
    const int cx = x0 + tx;
    NodeState o[kReadRows];
    unsigned bad = 0;
#pragma unroll
    for (int i = 0; i < kReadRows; ++i) {
        const int ey = wv * kReadRows + i, y = y0 + ey;
        const bool in = cx < g.Nx && y < g.Ny;
        if (in) {
            o[i] = node_state<S, kMX>(g, k, f, f0lo, T, cx, y, n_t);
            psi_t[ey + 1][tx + 1] = o[i].psi;
        }
        bad += __popcll(__ballot(in && o[i].fluid &&
                                 !(__builtin_isfinite(o[i].rho) && __builtin_isfinite(o[i].T))));
    }
    if (tx == 0) cnt[wv] = bad;
    // the ring; past the last column or row of the grid the block's own
    // entries there are the ring's (periodic image or, past an open end, the
    // end column itself); entries that no node reads are left unset
    {
        constexpr int kRow = kReadW + 2, kRing = 2 * kRow + 2 * kReadH;
        static_assert(kRing <= 256, "one ring node per thread");
        const int t = threadIdx.x;
        int ex, ey;
        if (t < 2 * kRow) {
            ey = t < kRow ? 0 : kReadH + 1;
            ex = t < kRow ? t : t - kRow;
        } else {
            ey = 1 + ((t - 2 * kRow) >> 1);
            ex = (t & 1) ? kReadW + 1 : 0;
        }
        // the ring's far side moves in to the grid's last column and row
        if (ex == kReadW + 1) ex = min(ex, g.Nx - x0 + 1);
        if (ey == kReadH + 1) ey = min(ey, g.Ny - y0 + 1);
        int rx = x0 - 1 + ex, y = y0 - 1 + ey;
        if (rx < 0) rx = read_xm(g, 0);
        else if (rx >= g.Nx) rx = rx == g.Nx ? read_xp(g, g.Nx - 1) : -1;
        if (g.periodic_y) y = y < 0 ? y + g.Ny : (y >= g.Ny ? (y == g.Ny ? 0 : -1) : y);
        else if (y >= g.Ny) y = -1;
        if (t < kRing && rx >= 0 && y >= 0)
            psi_t[ey][ex] = node_state<S, kMX>(g, k, f, f0lo, T, rx, y, n_t).psi;
    }
    __syncthreads();
    if (threadIdx.x == 0) ro.bad[blockIdx.x] = (cnt[0] + cnt[1]) + (cnt[2] + cnt[3]);
    if (cx >= g.Nx) return;
#pragma unroll
    for (int i = 0; i < kReadRows; ++i) {
        const int ey = wv * kReadRows + i, y = y0 + ey;
        if (y >= g.Ny) return;
        double ux = 0.0, uy = 0.0;
        if (o[i].fluid) {
            auto row3 = [&](int e) {
                return tri_of(psi_t[e][tx + 1], psi_t[e][tx], psi_t[e][tx + 2]);
            };
            node_velocity(g, k, cx, y, row3(ey), row3(ey + 1), row3(ey + 2), o[i].rho, o[i].jx,
                          o[i].jy, n_t, ux, uy);
        }
        const size_t at = (size_t)y * g.Nx + cx;
        if (out.rho) out.rho[at] = o[i].rho;
        if (out.ux) out.ux[at] = ux;
        if (out.uy) out.uy[at] = uy;
        if (out.T) out.T[at] = o[i].T;
    }
}

// ---- initial state ----------------------------------------------------------
// Buffers hold post-collision values, so the start state is the field that
// the first pull turns into f_i(x, 0) = w_i rho0(x): d*_i(z) = w_i (rho0(z + e_i)
// - rho_ref), or w_i (rho0(z) - rho_ref) where z + e_i is a plate.
template <class S, bool kMX>
__global__ __launch_bounds__(256) void init_kernel(Grid g, Phys k, const double* __restrict__ rho0,
                                                   S* __restrict__ f, float* __restrict__ f0lo,
                                                   S* __restrict__ T) {
    const int n = g.rows * g.Nx;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int sr = i / g.Nx, cx = i - sr * g.Nx;
    const int y = sr + g.y_first;
    const int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    const int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    const double w[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                         1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
    const unsigned o = (unsigned)sr * (unsigned)g.pitch + (unsigned)cx;
    for (int q = 0; q < 9; ++q) {
        int tx = cx + ex[q];
        tx = tx < 0 ? tx + g.Nx : (tx >= g.Nx ? tx - g.Nx : tx);
        int ty = y + ey[q];
        bool solid = false;
        if (g.periodic_y) {
            ty = ty < 0 ? ty + g.Ny : (ty >= g.Ny ? ty - g.Ny : ty);
        } else {
            solid = (ty == 0 || ty == g.Ny - 1);
        }
        const double r = solid ? rho0[y * g.Nx + cx] : rho0[ty * g.Nx + tx];
        const double v = w[q] * (r - k.rho_ref);
        if (kMX && q == 0) {
            const float hi = (float)v;
            f[o] = (S)hi;
            f0lo[o] = (float)(v - (double)hi);
        } else {
            f[q * g.plane + o] = (S)v;
        }
    }
    // T = T_0 = T_ref, T_w on a held frame node, T_in on an open inlet,
    // T_out on a held open outlet
    const bool held = g.frame_t && (cx == 0 || cx == g.Nx - 1 ||
                                    (g.periodic_y && (y == 0 || y == g.Ny - 1)));
    T[o] = (g.open_x && cx == 0)
               ? (S)k.dT_in
               : ((g.open_x && k.hold_out && cx == g.Nx - 1) ? (S)k.dT_out
                                                             : (held ? (S)k.dT_wall : (S)0));
}

// ---- deterministic FP64 reduction ------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__global__ __launch_bounds__(256) void reduce_pass1(const double* __restrict__ rho,
                                                    const double* __restrict__ ux,
                                                    const double* __restrict__ uy,
                                                    const double* __restrict__ T, int n,
                                                    double Cv, double* __restrict__ partials) {
    double s[5] = {0, 0, 0, 0, 0};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const double r = rho[i], a = ux[i], b = uy[i], t = T[i];
        if (!(isfinite(r) && isfinite(a) && isfinite(b) && isfinite(t))) {
            s[4] += 1.0;
            continue;
        }
        s[0] += r;
        s[1] += r * a;
        s[2] += r * b;
        s[3] += r * Cv * t;
    }
    __shared__ double red[4][5];
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const double t = wave_sum(s[q]);
        if (ln == 0) red[wv][q] = t;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        const int q = threadIdx.x;
        partials[blockIdx.x * 5 + q] = ((red[0][q] + red[1][q]) + (red[2][q] + red[3][q]));
    }
}

__global__ __launch_bounds__(64) void reduce_pass2(const double* __restrict__ partials, int nb,
                                                   double* __restrict__ out) {
    if (threadIdx.x < 5) {
        double s = 0.0;
        for (int b = 0; b < nb; ++b) s += partials[b * 5 + threadIdx.x];
        out[threadIdx.x] = s;
    }
}

// ---- one-pass reduction from the state (allocation-free entry point) ------
// A block takes tiles of 64 columns x 4 rows in a fixed order (tile
// blockIdx.x, then every gridDim.x-th).  For a tile it evaluates psi on the
// tile and its one-node ring into LDS (66 x 6 nodes, the ring recomputed),
// then every node of the tile its u from its own state and the psi of its
// neighbours, and adds rho, rho u_x, rho u_y, rho C_v T and the non-finite
// count in FP64.  Block totals go to part[5 * blockIdx.x + q] (every entry
// written, nothing needs clearing); reduce_pass2 sums them in block order.
constexpr int kTileW = 64, kTileH = 4;
constexpr int kRingW = kTileW + 2, kRingH = kTileH + 2;

template <class S, bool kMX>
__global__ __launch_bounds__(256) void reduce_state_kernel(Grid g, Phys k,
                                                           const S* __restrict__ f,
                                                           const float* __restrict__ f0lo,
                                                           const S* __restrict__ T, double Cv,
                                                           long long n_t,
                                                           double* __restrict__ part) {
    __shared__ double psi_t[kRingH][kRingW];
    const int tiles_x = (g.Nx + kTileW - 1) / kTileW;
    const int tiles = tiles_x * ((g.Ny + kTileH - 1) / kTileH);
    const int tx = threadIdx.x & (kTileW - 1), ty = threadIdx.x >> 6;
    double s[5] = {0, 0, 0, 0, 0};
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int x0 = (t % tiles_x) * kTileW, y0 = (t / tiles_x) * kTileH;
        __syncthreads();  // the previous tile's readers are done
        for (int e = threadIdx.x; e < kRingW * kRingH; e += blockDim.x) {
            const int ex = e % kRingW, ey = e / kRingW;
            // ring columns map as the read-out's neighbours do (periodic or
            // the end column past an open end); entries no node reads are
            // left unset
            int cx = x0 - 1 + ex;
            if (cx < 0) cx = read_xm(g, 0);
            else if (cx >= g.Nx) cx = cx == g.Nx ? read_xp(g, g.Nx - 1) : -1;
            int y = y0 - 1 + ey;
            if (g.periodic_y) y = y < 0 ? y + g.Ny : (y >= g.Ny ? y - g.Ny : y);
            else if (y < 0 || y >= g.Ny) y = -1;
            if (cx >= 0 && y >= 0 && y < g.Ny)
                psi_t[ey][ex] = node_state<S, kMX>(g, k, f, f0lo, T, cx, y, n_t).psi;
        }
        __syncthreads();
        const int cx = x0 + tx, y = y0 + ty;
        if (cx < g.Nx && y < g.Ny) {
            const NodeState o = node_state<S, kMX>(g, k, f, f0lo, T, cx, y, n_t);
            if (o.fluid) {
                auto row3 = [&](int ey) {
                    return tri_of(psi_t[ey][tx + 1], psi_t[ey][tx], psi_t[ey][tx + 2]);
                };
                double ux, uy;
                node_velocity(g, k, cx, y, row3(ty), row3(ty + 1), row3(ty + 2), o.rho, o.jx,
                              o.jy, n_t, ux, uy);
                if (!(isfinite(o.rho) && isfinite(ux) && isfinite(uy) && isfinite(o.T))) {
                    s[4] += 1.0;
                } else {
                    s[0] += o.rho;
                    s[1] += o.rho * ux;
                    s[2] += o.rho * uy;
                    s[3] += o.rho * Cv * o.T;
                }
            }
        }
    }
    __shared__ double red[4][5];
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const double v = wave_sum(s[q]);
        if (ln == 0) red[wv][q] = v;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        const int q = threadIdx.x;
        part[blockIdx.x * 5 + q] = ((red[0][q] + red[1][q]) + (red[2][q] + red[3][q]));
    }
}

inline int blocks_for(int n, int bs) { return (n + bs - 1) / bs; }

// ---- plain copy for the bandwidth probe -----------------------------------
// One 16-byte vector per thread, streaming (non-temporal) loads and stores:
// the fastest of the plain copy forms measured on MI355X (grid-stride loops
// with 2k-128k blocks, unrolled by 1 and 4, with and without the
// non-temporal hint), so the probe is a fair ceiling for the step kernel.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void copy_kernel(const f32x4* __restrict__ src,
                                                   f32x4* __restrict__ dst, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) __builtin_nontemporal_store(__builtin_nontemporal_load(&src[i]), &dst[i]);
}

}  // namespace

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
    const size_t n = bytes / 16;
    const size_t blocks = (n + 255) / 256;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffu) return hipErrorInvalidValue;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                       static_cast<const f32x4*>(src), static_cast<f32x4*>(dst), n);
    return hipGetLastError();
}

bool needs_ext(const Grid& g, const Phys& k) {
    return g.frame_t || g.frame_rho || g.open_x || k.wall_ramp || k.alpha_max > 0.0 ||
           (k.flags & (kEosCS | kPhaseProps | kTopMixed));
}

template <class S, bool kMX, bool kExt, int kTile>
static hipError_t launch_tile(const Grid& g, const Phys& k, const Bufs<S>& b, int64_t n,
                              hipStream_t s) {
    constexpr TileShape t = kTiles[kTile];
    hipLaunchKernelGGL((step_kernel<S, kMX, kExt, t.rows, t.waves, (kExt && t.per_simd > 4) ? 4 : t.per_simd>),
                       dim3(g.n_blocks), dim3(kLanes * t.waves), 0, s, g, k, b, (long long)n);
    return hipGetLastError();
}
template <class S, bool kMX, bool kExt>
static hipError_t step_impl(const Grid& g, const Phys& k, const Bufs<S>& b, int64_t n,
                            hipStream_t s) {
    if constexpr (sizeof(S) == 8) {
        if (g.tile == kTileFlat64) return launch_tile<S, kMX, kExt, kTileFlat64>(g, k, b, n, s);
        if (g.tile == kTileMid64) return launch_tile<S, kMX, kExt, kTileMid64>(g, k, b, n, s);
        if (g.tile == kTileTall64) return launch_tile<S, kMX, kExt, kTileTall64>(g, k, b, n, s);
    } else {
        if (g.tile == kTileFlat) return launch_tile<S, kMX, kExt, kTileFlat>(g, k, b, n, s);
        if (g.tile == kTileMid) return launch_tile<S, kMX, kExt, kTileMid>(g, k, b, n, s);
        constexpr int tall = kMX ? kTileTallMX : kTileTall;
        if (g.tile == tall) return launch_tile<S, kMX, kExt, tall>(g, k, b, n, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_step_f32(const Grid& g, const Phys& k, const Bufs<float>& b, bool mass_exact,
                           int64_t n, hipStream_t s) {
    const bool ext = needs_ext(g, k);
    if (mass_exact)
        return ext ? step_impl<float, true, true>(g, k, b, n, s)
                   : step_impl<float, true, false>(g, k, b, n, s);
    return ext ? step_impl<float, false, true>(g, k, b, n, s)
               : step_impl<float, false, false>(g, k, b, n, s);
}
hipError_t launch_step_f64(const Grid& g, const Phys& k, const Bufs<double>& b, int64_t n,
                           hipStream_t s) {
    return needs_ext(g, k) ? step_impl<double, false, true>(g, k, b, n, s)
                           : step_impl<double, false, false>(g, k, b, n, s);
}

template <bool kExt, int kTile>
static hipError_t launch_tile_batched(const Slot* slots, int n_slots, int total_blocks, int step_i,
                                      hipStream_t s) {
    constexpr TileShape t = kTiles[kTile];
    hipLaunchKernelGGL((step_batched_kernel<kExt, t.rows, t.waves, (kExt && t.per_simd > 4) ? 4 : t.per_simd>),
                       dim3(total_blocks), dim3(kLanes * t.waves), 0, s, slots, n_slots, step_i);
    return hipGetLastError();
}
template <bool kExt>
static hipError_t batched_impl(const Slot* slots, int n_slots, int total_blocks, int tile,
                               int step_i, hipStream_t s) {
    if (tile == kTileFlat)
        return launch_tile_batched<kExt, kTileFlat>(slots, n_slots, total_blocks, step_i, s);
    if (tile == kTileMid)
        return launch_tile_batched<kExt, kTileMid>(slots, n_slots, total_blocks, step_i, s);
    if (tile == kTileTall)
        return launch_tile_batched<kExt, kTileTall>(slots, n_slots, total_blocks, step_i, s);
    return hipErrorInvalidValue;
}
hipError_t launch_step_batched(const Slot* slots, int n_slots, int total_blocks, int tile,
                               int step_i, bool ext, hipStream_t s) {
    if (total_blocks <= 0 || n_slots <= 0) return hipSuccess;
    return ext ? batched_impl<true>(slots, n_slots, total_blocks, tile, step_i, s)
               : batched_impl<false>(slots, n_slots, total_blocks, tile, step_i, s);
}

int readout_blocks(int Nx, int Ny) {
    return ((Nx + kReadW - 1) / kReadW) * ((Ny + kReadH - 1) / kReadH);
}

template <class S, bool kMX>
static hipError_t moments_impl(const Grid& g, const Phys& k, const S* f, const float* f0lo,
                               const S* T, const Moments& out, int64_t n_t,
                               const unsigned long long* stat, const Readout& ro,
                               hipStream_t s) {
    hipLaunchKernelGGL((moments_kernel<S, kMX>), dim3(readout_blocks(g.Nx, g.Ny)), dim3(256), 0, s,
                       g, k, f, f0lo, T, out, (long long)n_t, stat, ro);
    return hipGetLastError();
}

hipError_t launch_moments_f32(const Grid& g, const Phys& k, const float* f, const float* f0lo,
                              const float* T, const Moments& out, int64_t n,
                              const unsigned long long* stat, const Readout& ro, hipStream_t s) {
    if (f0lo) return moments_impl<float, true>(g, k, f, f0lo, T, out, n, stat, ro, s);
    return moments_impl<float, false>(g, k, f, nullptr, T, out, n, stat, ro, s);
}
hipError_t launch_moments_f64(const Grid& g, const Phys& k, const double* f, const double* T,
                              const Moments& out, int64_t n, const unsigned long long* stat,
                              const Readout& ro, hipStream_t s) {
    return moments_impl<double, false>(g, k, f, nullptr, T, out, n, stat, ro, s);
}

hipError_t launch_init_f32(const Grid& g, const Phys& k, const double* rho0, float* f,
                           float* f0lo, float* T, hipStream_t s) {
    const int n = g.rows * g.Nx;
    if (f0lo)
        hipLaunchKernelGGL((init_kernel<float, true>), dim3(blocks_for(n, 256)), dim3(256), 0, s,
                           g, k, rho0, f, f0lo, T);
    else
        hipLaunchKernelGGL((init_kernel<float, false>), dim3(blocks_for(n, 256)), dim3(256), 0, s,
                           g, k, rho0, f, f0lo, T);
    return hipGetLastError();
}
hipError_t launch_init_f64(const Grid& g, const Phys& k, const double* rho0, double* f,
                           double* T, hipStream_t s) {
    const int n = g.rows * g.Nx;
    hipLaunchKernelGGL((init_kernel<double, false>), dim3(blocks_for(n, 256)), dim3(256), 0, s,
                       g, k, rho0, f, (float*)nullptr, T);
    return hipGetLastError();
}

// ---- allocation-free reduction: file-scope scratch -------------------------
// Block partials of reduce_state_kernel for callers that cannot allocate:
// kStaticReduceBlocks x 5 doubles (40 KiB) per GPU, held until the process
// ends.  Host code never uses the array's name as an address: each device's
// copy is resolved once with hipGetSymbolAddress (that device current) and
// the resolved pointer is passed to the kernels.
static __device__ __align__(256) double scratch[kStaticReduceBlocks * 5];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// this device's copy of `scratch` (resolved on its first use)
hipError_t scratch_on_current_device(double** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *out = static_cast<double*>(g_scratch_ptr[dev]);
    return hipSuccess;
}

template <class S, bool kMX>
hipError_t reduce_state_impl(const Grid& g, const Phys& k, const S* f, const float* f0lo,
                             const S* T, double Cv, int64_t n_t, double* out_dev,
                             hipStream_t s) {
    double* part = nullptr;
    hipError_t e = scratch_on_current_device(&part);
    if (e != hipSuccess) return e;
    const long long tiles = (long long)((g.Nx + kTileW - 1) / kTileW) *
                            ((g.Ny + kTileH - 1) / kTileH);
    const int nb = (int)std::min<long long>(tiles, kStaticReduceBlocks);
    hipLaunchKernelGGL((reduce_state_kernel<S, kMX>), dim3(nb), dim3(kTileW * kTileH), 0, s, g,
                       k, f, f0lo, T, Cv, (long long)n_t, part);
    hipLaunchKernelGGL(reduce_pass2, dim3(1), dim3(64), 0, s, (const double*)part, nb, out_dev);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_reduce_state_f32(const Grid& g, const Phys& k, const float* f,
                                   const float* f0lo, const float* T, double Cv, int64_t n_t,
                                   double* out_dev, hipStream_t s) {
    if (f0lo) return reduce_state_impl<float, true>(g, k, f, f0lo, T, Cv, n_t, out_dev, s);
    return reduce_state_impl<float, false>(g, k, f, nullptr, T, Cv, n_t, out_dev, s);
}
hipError_t launch_reduce_state_f64(const Grid& g, const Phys& k, const double* f, const double* T,
                                   double Cv, int64_t n_t, double* out_dev, hipStream_t s) {
    return reduce_state_impl<double, false>(g, k, f, nullptr, T, Cv, n_t, out_dev, s);
}

hipError_t launch_reduce(const double* rho, const double* ux, const double* uy, const double* T,
                         int n, double Cv, double* partials, double* out, hipStream_t s) {
    hipLaunchKernelGGL(reduce_pass1, dim3(kReduceBlocks), dim3(256), 0, s, rho, ux, uy, T, n, Cv,
                       partials);
    hipLaunchKernelGGL(reduce_pass2, dim3(1), dim3(64), 0, s, (const double*)partials,
                       kReduceBlocks, out);
    return hipGetLastError();
}

}  // namespace lbmk
