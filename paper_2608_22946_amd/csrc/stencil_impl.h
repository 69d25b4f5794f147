// Implementation of the stencil kernels and their launcher templates, included by the
// translation units that instantiate them (stencil.hip: FP32 operands; stencil_fp64.hip: FP64;
// stencil_mixed.hip: the FP16-stored operands of the mixed-precision cycle).
// Matrix-free 27-point IOFD level operator and its fused variants.
//
// Row i of H_mu = L - mu M (mu = 1 for A_l, 1 + i sigma for B_l; Sec. 2.2 and
// eq. shifted-iofd-levels) is, with a = alpha(eta*_i), kappa_i = omega ell / c_i:
//   ell^2 (H v)_i = sum_j sum_d w_j(i_j, d_j) T(d_perp) v_{i+d} - mu kappa_i^2 sum_d Mw(|d|_1) v_{i+d}
// with the stretched second-difference weights w_j (eq. pml-second-difference),
// transverse weights T = a4, a5/4, (1-a4-a5)/4 and mass weights
// Mw = a1, a2/6, a3/12, (1-a1-a2-a3)/8.  Where no stretching is present the row
// collapses to the shell form (eq. iofd-shell-form, eq. iofd-shell-coefficients).
//
// Work decomposition (CDNA wave64): one wavefront covers 64 consecutive x nodes
// of one y row; lanes 1..62 produce outputs, lanes 0 and 63 only supply the x
// halo.  x neighbours come from DPP wave shifts (no LDS), the y neighbours are
// the rows y-1 and y+1 loaded by the same lane, and the wave marches in z over a
// chunk of planes keeping per-plane partial sums in registers, so each input
// value is fetched from HBM once (plus L2-resident halo re-reads).  Workgroups
// of 4 waves cover 4 adjacent rows; the block index is remapped so that each of
// the 8 XCDs walks a contiguous range of tiles and shares halos in its own L2.
// Per-node coefficients are evaluated on the fly from the velocity: one
// reciprocal, the clamped interpolation coordinate and five cubic polynomials
// read from an LDS copy of the table, so the only per-node data read besides
// the operand is the FP32 velocity.
//
// What bounds it.  On a large level the memory path of the march: halving the vector instructions
// of its interior rows (124 -> 56 per plane) left the apply at 352^3 where it was (242 -> 246 us),
// one, two or three planes in flight measure the same, and without its stores the same loads
// take 108 us (67 us with one row load instead of three) of the 231 us that they take with
// them; a linear stream of the same arrays takes 140 us.  On a coarse level, which the cache
// holds, the instructions and the latency of a launch: there the shorter code is the gain (2h
// level of a 352^3 grid: J2 42.2 -> 37.8 us, apply 32.0 -> 30.2 us; 4h: 12.5 -> 10.6 us,
// 10.2 -> 8.4 us).  Measured and not kept: four rows a wavefront in registers (190 us for the
// loads and stores alone, but 148 registers: apply 237 us, 2h apply 42 us), rows shared by
// eight wavefronts through LDS with one barrier a plane (187 us alone, apply 260 us).
#pragma once

#include <algorithm>
#include <type_traits>

#include "helm_internal.h"

namespace helm {
namespace {

template <typename R>
struct Z {
    R r, i;
};

template <typename R>
__device__ __forceinline__ Z<R> zadd(Z<R> a, Z<R> b) { return {a.r + b.r, a.i + b.i}; }
template <typename R>
__device__ __forceinline__ Z<R> zsub(Z<R> a, Z<R> b) { return {a.r - b.r, a.i - b.i}; }
template <typename R>
__device__ __forceinline__ Z<R> zscale(R s, Z<R> a) { return {s * a.r, s * a.i}; }
template <typename R>
__device__ __forceinline__ Z<R> zmul(Z<R> a, Z<R> b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
template <typename R>
__device__ __forceinline__ Z<R> zfma(Z<R> a, Z<R> b, Z<R> acc) {  // acc + a*b
    return {acc.r + a.r * b.r - a.i * b.i, acc.i + a.r * b.i + a.i * b.r};
}
template <typename R>
__device__ __forceinline__ Z<R> zdiv(Z<R> a, Z<R> d) {
    R inv = R(1) / (d.r * d.r + d.i * d.i);
    return {(a.r * d.r + a.i * d.i) * inv, (a.i * d.r - a.r * d.i) * inv};
}

// value from the lane holding x-1 (wave_shr:1) and from the lane holding x+1 (wave_shl:1)
// (lanes without a source read 0 by bound_ctrl, so the shift folds into the addition that uses it)
__device__ __forceinline__ float from_left(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ double from_left(double v) {
    long long b = __double_as_longlong(v);
    int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), 0x138, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x138, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double from_right(double v) {
    long long b = __double_as_longlong(v);
    int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), 0x130, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x130, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <typename R>
__device__ __forceinline__ Z<R> zleft(Z<R> v) { return {from_left(v.r), from_left(v.i)}; }
template <typename R>
__device__ __forceinline__ Z<R> zright(Z<R> v) { return {from_right(v.r), from_right(v.i)}; }

template <typename R, typename T>
__device__ __forceinline__ Z<R> ld(const T *p, long long i) {
    T v = p[i];
    return {(R)v.re, (R)v.im};
}

// FP16-stored operands (c16): true value = stored value / (f qs), see helm_internal.h
template <typename R, typename T>
__device__ __forceinline__ Z<R> dq(T v, R inv) {
    Z<R> o = {(R)v.re, (R)v.im};
    if (is_half<T>()) {
        o.r *= inv;
        o.i *= inv;
    }
    return o;
}
template <typename T, typename R>
__device__ __forceinline__ T qz(Z<R> v, R s) { return to_stored<T, R>(v.r, v.i, s); }
struct Scales {
    Scale x, g, b, y;
};

__device__ __forceinline__ float recip(float c) { return __builtin_amdgcn_rcpf(c); }
__device__ __forceinline__ double recip(double c) { return 1.0 / c; }

// Interpolation coordinate and the five coefficient functions at a node
// (eq. iofd-clamped-coordinate); the table holds, per interval, the monomial
// coefficients of the cubic Hermite interpolant in the local variable t.
template <typename R>
struct Coef {
    R a1, a2, a3, a4, a5, k2;
};

template <typename R>
__device__ __forceinline__ void locate(const LevelArgs<R> &L, float c, R &kappa, int &k, R &t) {
    kappa = L.omega_ell * recip((R)c);
    R eta = kappa * (R)0.15915494309189533577;   // 1 / (2 pi)
    eta = eta < (R)0.4 ? eta : (R)0.4;
    R u = eta * L.inv_deta;
    k = (int)u;
    k = k < L.K - 1 ? k : L.K - 1;
    k = k > 0 ? k : 0;
    t = u - (R)k;
}

template <typename R>
__device__ __forceinline__ R horner(const R *p, R t) { return ((p[3] * t + p[2]) * t + p[1]) * t + p[0]; }
template <typename R>
__device__ __forceinline__ R horner5(const R *p, R t) {
    return ((((p[5] * t + p[4]) * t + p[3]) * t + p[2]) * t + p[1]) * t + p[0];
}

// FP32 levels read the scaled coordinate s = omega ell K / (0.4 * 2 pi c) per node instead of
// c (LevelArgs::s): the same interval and local coordinate as `locate`, and kappa = s kap_s.
template <typename R>
constexpr bool scaled_coordinate() { return sizeof(R) == sizeof(float); }

template <typename R>
__device__ __forceinline__ void locate_s(const LevelArgs<R> &L, float s, R &kappa, int &k, R &t) {
    kappa = (R)s * L.kap_s;
    const R u = (R)s < (R)L.K ? (R)s : (R)L.K;   // eta* clamped at 0.4
    k = (int)u;
    k = k < L.K - 1 ? k : L.K - 1;
    t = u - (R)k;
}

// the five coefficient functions and kappa^2 at a node; v is the per-node value the level
// stores (s on FP32 levels, the velocity c on FP64 ones)
template <typename R>
__device__ __forceinline__ Coef<R> coef_at(const LevelArgs<R> &L, const R *stab, float v) {
    R kappa, t;
    int k;
    if (scaled_coordinate<R>())
        locate_s(L, v, kappa, k, t);
    else
        locate(L, v, kappa, k, t);
    // stab holds the intervals kb .. kb + nk - 1 (the level's window)
    k = k < L.kb ? L.kb : (k > L.kb + L.nk - 1 ? L.kb + L.nk - 1 : k);
    const R *p = stab + (k - L.kb) * 20;
    Coef<R> o;
    o.a1 = horner(p + 0, t);
    o.a2 = horner(p + 4, t);
    o.a3 = horner(p + 8, t);
    o.a4 = horner(p + 12, t);
    o.a5 = horner(p + 16, t);
    o.k2 = kappa * kappa;
    return o;
}

// Coefficients of one row as the march uses them, all times ell^-2: mass weights m0..m3 =
// (a1, a2 / 6, a3 / 12, (1 - a1 - a2 - a3) / 8), the transverse functions a4, a5 and
// q = 1 - a4 - a5, and kappa^2.
template <typename R>
struct RowCoef {
    R m0, m1, m2, m3, a4, a5, q, k2;
};

// A table piece in LDS is read with 16-byte loads (ds_read_b128; the pieces are multiples of 16 B
// from an aligned base): 24 floats of a node's quintics take 6 loads instead of 12.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <int N>
__device__ __forceinline__ void lds_read(const float *p, float (&o)[N]) {
    static_assert(N % 4 == 0, "whole 16-byte loads");
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        const f32x4 v = reinterpret_cast<const f32x4 *>(p)[i];
        o[4 * i] = v.x; o[4 * i + 1] = v.y; o[4 * i + 2] = v.z; o[4 * i + 3] = v.w;
    }
}
template <int N>
__device__ __forceinline__ void lds_read(const double *p, double (&o)[N]) {
    static_assert(N % 2 == 0, "whole 16-byte loads");
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        const f64x2 v = reinterpret_cast<const f64x2 *>(p)[i];
        o[2 * i] = v.x; o[2 * i + 1] = v.y;
    }
}
// byte offset of table piece k (a small whole number held in a float) in a window that starts at
// piece `first`: one multiply-add and a conversion (an integer multiply is quarter rate)
__device__ __forceinline__ unsigned piece_offset(float k, float first, float bytes) {
    return (unsigned)((k - first) * bytes);
}

// RowCoef from the level's scaled table (LDS copy `etab`); v as in coef_at
__device__ __forceinline__ RowCoef<float> row_coef(const LevelArgs<float> &L, const float *etab, float v) {
    const float u = fminf(v, (float)L.K);   // eta* clamped at 0.4
    // the window holds every interval a node of the level reaches
    const float k = __builtin_amdgcn_fmed3f(truncf(u), (float)L.kb, (float)(L.kb + L.nk - 1));
    const float t = u - k;
    float c[20];
    lds_read(reinterpret_cast<const float *>(reinterpret_cast<const char *>(etab) +
                                             piece_offset(k, (float)L.kb, 80.0f)), c);
    RowCoef<float> o;
    o.m0 = horner(c, t);
    o.m1 = horner(c + 4, t);
    o.m2 = horner(c + 8, t);
    o.a4 = horner(c + 12, t);
    o.a5 = horner(c + 16, t);
    o.m3 = 0.125f * (L.inv_ell2 - o.m0) - 0.75f * o.m1 - 1.5f * o.m2;
    o.q = L.inv_ell2 - o.a4 - o.a5;
    const float kappa = v * L.kap_s;
    o.k2 = kappa * kappa;
    return o;
}
__device__ __forceinline__ RowCoef<double> row_coef(const LevelArgs<double> &L, const double *etab, float v) {
    double kappa, t;
    int k;
    locate(L, v, kappa, k, t);
    k = k < L.kb ? L.kb : (k > L.kb + L.nk - 1 ? L.kb + L.nk - 1 : k);
    double c[20];
    lds_read(etab + (k - L.kb) * 20, c);
    RowCoef<double> o;
    o.m0 = horner(c, t);
    o.m1 = horner(c + 4, t);
    o.m2 = horner(c + 8, t);
    o.a4 = horner(c + 12, t);
    o.a5 = horner(c + 16, t);
    o.m3 = 0.125 * (L.inv_ell2 - o.m0) - 0.75 * o.m1 - 1.5 * o.m2;
    o.q = L.inv_ell2 - o.a4 - o.a5;
    o.k2 = kappa * kappa;
    return o;
}

// unshifted shell coefficients C_0..C_3 (times ell^-2) at a node of an FP32 level from the quintic
// table (LDS copy `ctab`): interval min(floor(s), K), the last one unbounded in t
__device__ __forceinline__ void shell_coef(const LevelArgs<float> &L, const float *ctab, float s, float (&C)[4]) {
    const float k = __builtin_amdgcn_fmed3f(truncf(s), (float)L.cb, (float)(L.cb + L.nck - 1));
    const float t = s - k;
    float c[24];
    lds_read(reinterpret_cast<const float *>(reinterpret_cast<const char *>(ctab) +
                                             piece_offset(k, (float)L.cb, 96.0f)), c);
#pragma unroll
    for (int m = 0; m < 4; ++m) C[m] = horner5(c + 6 * m, t);
}
__device__ __forceinline__ void shell_coef(const LevelArgs<double> &, const double *, float, double (&)[4]) {}
// 1 / C_0: the row's D^-1 where it is free of stretching.  The reciprocal instruction, accurate to a unit in the
// last place, and one Newton step.
__device__ __forceinline__ float shell_dinv(const LevelArgs<float> &L, const float *ctab, float s) {
    const float k = __builtin_amdgcn_fmed3f(truncf(s), (float)L.cb, (float)(L.cb + L.nck - 1));
    const char *p = reinterpret_cast<const char *>(ctab) + piece_offset(k, (float)L.cb, 96.0f);
    const f32x4 a = reinterpret_cast<const f32x4 *>(p)[0];
    const f32x2 b = reinterpret_cast<const f32x2 *>(p)[2];
    const float c[6] = {a.x, a.y, a.z, a.w, b.x, b.y};
    const float d = horner5(c, s - k), r = __builtin_amdgcn_rcpf(d);
    return fmaf(fmaf(-d, r, 1.0f), r, r);
}
__device__ __forceinline__ double shell_dinv(const LevelArgs<double> &, const double *, float) { return 0; }

// per-node value a level's coefficient evaluation reads
template <typename R>
__device__ __forceinline__ const float *node_values(const LevelArgs<R> &L) {
    return scaled_coordinate<R>() ? L.s : L.c;
}

// diagonal entry ell^2 D = a4 (wxc + wyc + wzc) - mu kappa^2 a1
template <typename R, bool SHIFT>
__device__ __forceinline__ Z<R> diag_of(const LevelArgs<R> &L, R a1, R a4, R k2, Z<R> wsum) {
    Z<R> d = zscale(a4, wsum);
    d.r -= k2 * a1;
    if (SHIFT) d.i -= L.sigma * k2 * a1;
    return zscale(L.inv_ell2, d);
}

template <typename R>
struct Plane {
    Z<R> p0, p1, p2;   // centre, 4 in-plane face neighbours, 4 in-plane corners
    Z<R> ea, eb;       // x/y stiffness partials (tensor form only)
    Z<R> gc;           // right-hand side at the centre (residual / sweep modes)
    Z<R> dc;           // D^-1 at the centre (sweep), omega D^-1 (fused Jacobi)
    Z<R> bc;           // base value at the centre (fused Jacobi + base)
    float cc;          // per-node value at the centre (s on FP32 levels, c on FP64 ones)
};

// w . (l, c, r) with complex weights
template <typename R>
__device__ __forceinline__ Z<R> wdot(const Z<R> (&w)[3], Z<R> l, Z<R> c, Z<R> r) {
    return zfma(w[2], r, zfma(w[1], c, zmul(w[0], l)));
}
// 2 a - b
template <typename R>
__device__ __forceinline__ Z<R> twice_less(Z<R> a, Z<R> b) { return {(R)2 * a.r - b.r, (R)2 * a.i - b.i}; }

// In-plane partial sums of one z plane from the rows y-1 (a), y (b), y+1 (c)
// at this lane's x; x neighbours come from the adjacent lanes.  XI / YI: the
// x / y stretching of this wave is the identity (weights -1, 2, -1).
template <typename R, bool XI, bool YI>
__device__ __forceinline__ void plane_partials(Z<R> a, Z<R> b, Z<R> c, const Z<R> (&wx)[3], const Z<R> (&wy)[3],
                                               Plane<R> &P) {
    const Z<R> col = zadd(a, c);
    P.p0 = b;
    if constexpr (XI && YI) {
        P.p1 = zadd(zadd(col, zleft(b)), zright(b));
        P.p2 = zadd(zleft(col), zright(col));
    } else if constexpr (YI) {   // x stretched, -1, 2, -1 along y
        const Z<R> bL = zleft(b), bR = zright(b), colL = zleft(col), colR = zright(col);
        const Z<R> rs0 = zadd(bL, bR);
        P.p1 = zadd(col, rs0);
        P.p2 = zadd(colL, colR);
        P.ea = zadd(wdot(wx, bL, b, bR), twice_less(b, col));
        P.eb = zadd(wdot(wx, colL, col, colR), twice_less(rs0, P.p2));
    } else {
        const Z<R> rsm = zadd(zleft(a), zright(a)), rsp = zadd(zleft(c), zright(c));
        const Z<R> bL = zleft(b), bR = zright(b);
        const Z<R> rs0 = zadd(bL, bR);
        P.p1 = zadd(col, rs0);
        P.p2 = zadd(rsm, rsp);
        if constexpr (XI) {      // -1, 2, -1 along x, y stretched
            P.ea = zadd(wdot(wy, a, b, c), twice_less(b, rs0));
            P.eb = zadd(wdot(wy, rsm, rs0, rsp), twice_less(col, P.p2));
        } else {
            P.ea = zadd(wdot(wx, bL, b, bR), wdot(wy, a, b, c));
            P.eb = zadd(wdot(wx, zleft(col), col, zright(col)), wdot(wy, rsm, rs0, rsp));
        }
    }
}

// sum_m C_m S_m over the shell sums S_m of the 1 / 6 / 12 / 8 neighbours
template <typename R>
__device__ __forceinline__ Z<R> shell_sum(const R (&C)[4], const Z<R> (&S)[4]) {
    return {C[0] * S[0].r + C[1] * S[1].r + C[2] * S[2].r + C[3] * S[3].r,
            C[0] * S[0].i + C[1] * S[1].i + C[2] * S[2].i + C[3] * S[3].i};
}

// H v at the centre of plane "o" from planes m (z-1), o (z), p (z+1); the row's coefficients
// come from the per-node value o.cc (s or c).  Rows free of stretching take the shell form
// (eq. iofd-shell-form): the unshifted ones of an FP32 level from the quintic table (one
// Horner per coefficient), the others from alpha_1..alpha_5 (eq. iofd-shell-coefficients);
// rows in the PML take the tensor-product form.  INNER: the row is known to be free of
// stretching; otherwise zint says whether z is, and wzp holds the plane's z weights.
template <typename R, bool XYI, bool SHIFT, bool INNER>
__device__ __forceinline__ Z<R> row_value(const LevelArgs<R> &L, const R *etab, const R *ctab, const Plane<R> &m,
                                          const Plane<R> &o, const Plane<R> &p, bool zint, const R *wzp) {
    const Z<R> s0 = zadd(m.p0, p.p0), s1 = zadd(m.p1, p.p1), s2 = zadd(m.p2, p.p2);
    const Z<R> S[4] = {o.p0, zadd(o.p1, s0), zadd(o.p2, s1), s2};
    if (INNER || (XYI && zint)) {
        if constexpr (scaled_coordinate<R>() && !SHIFT) {
            R C[4];
            shell_coef(L, ctab, o.cc, C);
            return shell_sum(C, S);
        } else {
            // C_m = stiffness_m - mu kappa^2 mass_m
            const RowCoef<R> f = row_coef(L, etab, o.cc);
            const R M[4] = {f.m0, f.m1, f.m2, f.m3};
            const R C[4] = {(R)6 * f.a4 - f.k2 * f.m0, (f.a5 - f.a4) - f.k2 * f.m1,
                            (R)0.5 * (f.q - f.a5) - f.k2 * f.m2, (R)-0.75 * f.q - f.k2 * f.m3};
            Z<R> out = shell_sum(C, S);
            if (SHIFT) {   // - i sigma kappa^2 sum_m mass_m S_m
                const R sk = L.sigma * f.k2;
                const Z<R> mass = shell_sum(M, S);
                out.r += sk * mass.i;
                out.i -= sk * mass.r;
            }
            return out;
        }
    }
    const RowCoef<R> f = row_coef(L, etab, o.cc);
    const R M[4] = {f.m0, f.m1, f.m2, f.m3};
    const Z<R> mass = shell_sum(M, S);
    // the x/y parts A0, A1, A2 of the transverse weights a4, a5 / 4, q / 4
    Z<R> A0, A1, A2;
    if constexpr (XYI) {   // unit x/y stretching: ea = 4 P0 - P1, eb = 2 P1 - 2 P2
        A0 = {(R)4 * o.p0.r - o.p1.r, (R)4 * o.p0.i - o.p1.i};
        A1 = {(R)2 * (o.p1.r - o.p2.r) + ((R)4 * s0.r - s1.r), (R)2 * (o.p1.i - o.p2.i) + ((R)4 * s0.i - s1.i)};
        A2 = {(R)2 * (s1.r - s2.r), (R)2 * (s1.i - s2.i)};
    } else {
        A0 = o.ea;
        A1 = zadd(o.eb, zadd(m.ea, p.ea));
        A2 = zadd(m.eb, p.eb);
    }
    if (zint) {   // -1, 2, -1 along z
        A0 = zadd(A0, twice_less(o.p0, s0));
        A1 = zadd(A1, twice_less(o.p1, s1));
        A2 = zadd(A2, twice_less(o.p2, s2));
    } else {
        const Z<R> wz[3] = {{wzp[0], wzp[1]}, {wzp[2], wzp[3]}, {wzp[4], wzp[5]}};
        A0 = zadd(A0, wdot(wz, m.p0, o.p0, p.p0));
        A1 = zadd(A1, wdot(wz, m.p1, o.p1, p.p1));
        A2 = zadd(A2, wdot(wz, m.p2, o.p2, p.p2));
    }
    const R t1 = (R)0.25 * f.a5, t2 = (R)0.25 * f.q;
    Z<R> out = {f.a4 * A0.r + t1 * A1.r + t2 * A2.r - f.k2 * mass.r,
                f.a4 * A0.i + t1 * A1.i + t2 * A2.i - f.k2 * mass.i};
    if (SHIFT) {   // - i sigma kappa^2 mass
        const R sk = L.sigma * f.k2;
        out.r += sk * mass.i;
        out.i -= sk * mass.r;
    }
    return out;
}

__device__ __forceinline__ void block_reduce_store(double v, double *dst) {
    // wavefront sum (DPP), then across the workgroup's waves through LDS
    v = wave_sum_f64(v);
    __shared__ double red[kWavesY];
    int w = threadIdx.y, l = threadIdx.x;
    if (l == 0) red[w] = v;
    __syncthreads();
    if (w == 0 && l == 0) {
        double s = 0;
        for (int i = 0; i < kWavesY; ++i) s += red[i];
        partial_store(dst, s);
        stores_done();
    }
}

// Last-block epilogue of a stencil with fused ||y||^2: beta, state reset.
__device__ void norm_epilogue(const RedBuf &rb, int nblocks, KState *st) {
    constexpr int nt = 64 * kWavesY;   // threads of a stencil workgroup
    static_assert((nt & (nt - 1)) == 0, "the tree sum needs a power-of-two workgroup");
    __shared__ bool last;
    __shared__ double red[nt];
    const int tid = threadIdx.x + 64 * threadIdx.y;
    if (tid == 0) last = take_ticket(rb.counter, nblocks);
    __syncthreads();
    if (!last) return;
    double s = 0;
#pragma unroll 8
    for (int b = tid; b < nblocks; b += nt) s += partial_load(rb.partials + b);
    red[tid] = s;
    __syncthreads();
    for (int off = nt / 2; off > 0; off >>= 1) {
        if (tid < off) red[tid] += red[tid + off];
        __syncthreads();
    }
    if (tid == 0) {
        double beta = sqrt(red[0]);
        st->beta = beta;
        st->scale = (beta > 0.0) ? 1.0 / beta : 0.0;
        st->vs0 = st->scale;
        st->kk = 0;
        st->breakdown = 0;
        st->nonfinite = !(beta == beta && beta < 1e300);
        for (int j = 0; j <= kMMax; ++j) st->g[j][0] = st->g[j][1] = 0.0;
        st->g[0][0] = beta;
        reset_ticket(rb.counter);
    }
}

// Loads and stores go through a buffer descriptor of the plane (scalar registers) with the row's
// offset in a scalar register and the lane's byte offset in the row in a vector register, so that
// no address arithmetic runs on the vector unit.  Stores of lanes without an output are dropped
// by the descriptor's bound (their offset is kNoStore) instead of by a branch.
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kNoStore = 0xffffff00u;   // past every plane (at most 4097^2 nodes of 16 B)
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_buf(const T *plane, unsigned nodes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(plane), 0, nodes * (unsigned)sizeof(T), 0x00020000);
}
template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t b, unsigned lane_off, unsigned row_off) {
    if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, lane_off, row_off, 0));
    else if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, lane_off, row_off, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(b, lane_off, row_off, 0));
}
// A store at `off` + `row_off` of the buffer.  A 16-byte store takes its offset from the vector register alone
// (split_row): with the row's part in a scalar register the compiler puts no wait state before the next
// vector write to the data registers, which a store of more than 8 bytes reads late (the fused norm's
// squares, formed in the same registers, reached memory in place of the imaginary part).  Two 8-byte stores
// instead, each with half of every 16 bytes, cost the FP64 kernels 6 to 12% (352^3, depth 40: apply 466
// and 415 us, residual 563 and 531, J2 631 and 589).
template <typename T>
constexpr bool split_row() { return sizeof(T) <= 8; }
template <int HINT = 0, typename T>   // HINT 2: non-temporal
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t b, unsigned off, unsigned row_off, T v) {
    if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, off, row_off, HINT);
    else if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, off, row_off, HINT);
    else
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, off, 0, HINT);   // row_off: 0
}
// lane and row offsets of the stores of a row (nodes lx of the lane, r0 of the row); lanes without an output: kNoStore
template <typename T>
__device__ __forceinline__ void row_store_offsets(bool out, bool scalar_row, unsigned lx, unsigned r0, unsigned &off,
                                                  unsigned &row_off) {
    const bool split = split_row<T>() && scalar_row;
    off = out ? (split ? lx : r0 + lx) * (unsigned)sizeof(T) : kNoStore;
    row_off = split ? r0 * (unsigned)sizeof(T) : 0u;
}

// The unshifted fused Jacobi of an FP32 level forms D^-1 = 1 / C_0 of the rows of its inner tiles from
// the per-node values: 4 bytes a node of each row instead of 8 more (fine level at 352^3: 355 -> 331 us).
// The shifted ones keep the stored D^-1: theirs is complex, and their levels fit in the cache.
template <typename R>
constexpr bool own_dinv(int mode, bool shifted) {
    return scaled_coordinate<R>() && !shifted && mode == M_JAC2;
}

// modes whose result may be stored past the caches (a second store in the others costs registers)
constexpr bool may_stream(int mode, bool norm) { return mode == M_APPLY || (mode == M_RESID && !norm); }

// One wavefront: rows y-1, y, y+1 at 64 consecutive x, marching planes z0..z1-1.
// Every load reads an in-bounds node (indices clamped to the grid) and
// boundary / out-of-box values are masked to zero afterwards, so the loads
// carry no branches; the per-lane byte offsets inside a plane are fixed and the
// plane base is wave-uniform (scalar registers).  INNER: every plane and row the wave reads
// lies inside the box and every row it forms is free of stretching, so nothing is masked
// and one coefficient form remains; most waves of a large level are of this kind.
template <typename R, typename TX, typename TG, typename TY, int MODE, bool SHIFT, bool NORM, bool XI, bool YI,
          bool INNER>
__device__ __forceinline__ void march(const LevelArgs<R> &L, const R *etab, const R *ctab, const TX *__restrict__ x,
                                      const TG *__restrict__ g, const TY *__restrict__ base, TY *__restrict__ y,
                                      R omegaJ, const R (&mul)[4], int xg, int yg, int z0, int z1, bool out_lane,
                                      double &nrm, bool stream, int Z0 = 0) {
    static_assert(!INNER || (XI && YI), "inner tiles have no stretching");
    // mul: multipliers of the c16 operands (x, g, base loads; y store), 1 for the others
    const R mx = mul[0], mg = mul[1], mb = mul[2], my = mul[3];
    constexpr bool JAC = (MODE == M_JAC2 || MODE == M_JAC2_ADD);
    constexpr bool RESTRICT = (MODE == M_RESID_R);
    constexpr bool NEED_G = (MODE != M_APPLY);
    constexpr bool OWN_D = INNER && own_dinv<R>(MODE, SHIFT);
    const bool x_int = (xg >= 1 && xg <= L.nx - 1);
    const int xc = min(max(xg, 0), L.nx);
    const MarchRows rows = march_rows(yg, L.ny);
    // node offsets: of the lane in a row (vector), of the three rows in a plane (scalar where the
    // wavefront has one row)
    const unsigned lx = (unsigned)xc, r0 = (unsigned)(rows.c * (int)L.sx), rm = (unsigned)(rows.m * (int)L.sx),
                   rp = (unsigned)(rows.p * (int)L.sx);
    auto load_row = [&](const auto *p, unsigned ro) {
        using E = std::remove_const_t<std::remove_reference_t<decltype(*p)>>;
        if constexpr (XI)
            return buf_load<E>(plane_buf(p, (unsigned)L.sy), lx * (unsigned)sizeof(E), ro * (unsigned)sizeof(E));
        else
            return buf_load<E>(plane_buf(p, (unsigned)L.sy), (ro + lx) * (unsigned)sizeof(E), 0);
    };
    const bool rm_ok = x_int && (yg - 1 >= 1);
    const bool r0_ok = x_int && (yg >= 1) && (yg <= L.ny - 1);
    const bool rp_ok = x_int && (yg + 1 <= L.ny - 1);

    Z<R> wx[3] = {{0, 0}, {0, 0}, {0, 0}}, wy[3] = {{0, 0}, {0, 0}, {0, 0}};
    if constexpr (!XI) {
        const R *w = L.wx + 6 * xc;
        wx[0] = {w[0], w[1]}; wx[1] = {w[2], w[3]}; wx[2] = {w[4], w[5]};
    }
    if constexpr (!YI) {
        const R *v = L.wy + 6 * rows.c;
        wy[0] = {v[0], v[1]}; wy[1] = {v[2], v[3]}; wy[2] = {v[4], v[5]};
    }
    const Z<R> zero = {0, 0};

    // Raw loads of one plane.
    using DT = cplx<R>;
    struct Raw {
        TX va, vb, vc;     // operand rows (not in the Jacobi modes)
        TG ga, gb, gc;     // right-hand side rows (Jacobi modes; gb alone in the others)
        DT da, db, dc;     // D^-1 rows (Jacobi modes; db alone in the sweep mode)
        float ca, cp;      // per-node values of the other rows (where D^-1 is formed from them)
        TY bb;             // base at the centre (fused Jacobi + base)
        float cb;          // per-node coefficient value at the centre
    };
    constexpr bool SWEEP = (MODE == M_JSWEEP);
    const DT *dinv = reinterpret_cast<const DT *>(L.dinv[SHIFT ? 1 : 0]);
    // Planes past the tile's last plane z1 are re-read from z1 (a cache hit):
    // the prefetch is then issued unconditionally, which keeps the count of
    // outstanding loads the same on every path through the loop, so waiting
    // for one plane never waits for the planes issued after it.
    const int zlast = min(z1, L.nz);
    const float *vnode = node_values(L);
    const unsigned sy = (unsigned)L.sy;   // (N + 1)^2 nodes of a plane, at most 4097^2
    auto issue = [&](int zp, Raw &r) {
        const unsigned long long po = (unsigned long long)(unsigned)min(max(zp, 0), zlast) * sy;
        auto row = [&](const auto *p, unsigned ro) { return load_row(p + po, ro); };
        if constexpr (!JAC) {
            r.va = row(x, rm);
            r.vb = row(x, r0);
            r.vc = row(x, rp);
            if constexpr (NEED_G) r.gb = row(g, r0);
            if constexpr (SWEEP) r.db = row(dinv, r0);
        } else {
            r.ga = row(g, rm);
            r.gb = row(g, r0);
            r.gc = row(g, rp);
            if constexpr (OWN_D) {
                r.ca = row(vnode, rm);
                r.cp = row(vnode, rp);
            } else {
                r.da = row(dinv, rm);
                r.db = row(dinv, r0);
                r.dc = row(dinv, rp);
            }
            if constexpr (MODE == M_JAC2_ADD) r.bb = row(base, r0);
        }
        r.cb = row(vnode, r0);
    };
    // mask boundary / out-of-box values and form the plane partials
    auto finish = [&](int zp, const Raw &r, Plane<R> &P) {
        Z<R> a, b, c;
        if constexpr (!JAC) {
            a = dq<R>(r.va, mx);
            b = dq<R>(r.vb, mx);
            c = dq<R>(r.vc, mx);
            if constexpr (NEED_G) P.gc = dq<R>(r.gb, mg);
        } else if constexpr (OWN_D) {
            // fused two-sweep Jacobi: the operand is y1 = omega D^-1 g at every loaded node
            a = zscale(omegaJ * shell_dinv(L, ctab, r.ca), dq<R>(r.ga, mg));
            b = zscale(omegaJ * shell_dinv(L, ctab, r.cb), dq<R>(r.gb, mg));
            c = zscale(omegaJ * shell_dinv(L, ctab, r.cp), dq<R>(r.gc, mg));
        } else {
            P.dc = zscale(omegaJ, Z<R>{r.db.re, r.db.im});
            a = zmul(zscale(omegaJ, Z<R>{r.da.re, r.da.im}), dq<R>(r.ga, mg));
            b = zmul(P.dc, dq<R>(r.gb, mg));
            c = zmul(zscale(omegaJ, Z<R>{r.dc.re, r.dc.im}), dq<R>(r.gc, mg));
        }
        if constexpr (!INNER) {
            const bool zok = (zp >= 1 && zp <= L.nz - 1);
            if (!(zok && rm_ok)) a = zero;
            if (!(zok && r0_ok)) b = zero;
            if (!(zok && rp_ok)) c = zero;
        }
        P.cc = r.cb;
        if constexpr (JAC) P.gc = dq<R>(r.gb, mg);
        if constexpr (SWEEP) P.dc = Z<R>{r.db.re, r.db.im};
        if constexpr (MODE == M_JAC2_ADD) P.bc = dq<R>(r.bb, mb);
        plane_partials<R, XI, YI>(a, b, c, wx, wy, P);
    };

    const bool yint = (yg >= 1 && yg <= L.ny - 1);
    // M_RESID_R: x/z-restricted residual rows w[coarse z][fine y][coarse x]
    const int nxc = L.nx >> 1, nzc = L.nz >> 1;
    const long long wsx = nxc + 1, wsy = (long long)(L.ny + 1) * wsx;
    const int lane = threadIdx.x;
    const bool rstore = RESTRICT && (lane & 1) && lane >= 3 && lane <= 61 && yint && (xg >> 1) >= 1 && (xg >> 1) <= nxc - 1;
    Z<R> rcur = zero;
    unsigned store_off, store_row;
    row_store_offsets<TY>(out_lane, XI, lx, r0, store_off, store_row);
    // output plane z from planes m, o, p
    auto emit = [&](int z, const Plane<R> &m, const Plane<R> &o, const Plane<R> &p) {
        const bool zint = INNER || (z >= L.loz && z <= L.hiz);
        // A row of the boundary is not formed but masked below.  Besides the work that this saves on thin
        // levels, the branch keeps the compiler from drawing one plane's table reads into the next: without
        // it the residual, the sweep and the fused restriction spill 20 to 55 registers at four wavefronts
        // a SIMD, and the fused Jacobi takes 136.  With and without it, z depth 8: fused Jacobi at 352^3 366
        // and 398 us, three sweeps 897 and 974, restriction at 208^3 74 and 88, residual at 208^3 70 and 75.
        const bool interior = INNER || (r0_ok && z >= 1 && z <= L.nz - 1);
        Z<R> Hv = zero;
        if (interior) Hv = row_value<R, XI && YI, SHIFT, INNER>(L, etab, ctab, m, o, p, zint, L.wz + 6 * z);
        Z<R> res;
        if constexpr (MODE == M_APPLY) {
            res = Hv;
        } else if constexpr (MODE == M_RESID || RESTRICT) {
            res = zsub(o.gc, Hv);
        } else if constexpr (SWEEP) {
            res = zadd(o.p0, zscale(omegaJ, zmul(o.dc, zsub(o.gc, Hv))));
        } else {
            // y1 + omega D^-1 (g - H y1).  With omega D^-1 g = y1 this is 2 y1 - omega D^-1 H y1, which does not
            // keep g but takes the rounding of y1 in full, where the residual form damps it: 8.3e-8 of the
            // result at 176^3 for 7.1e-8, 9.0e-8 for 7.5e-8 in a layered medium, in the same time.
            const Z<R> r = zsub(o.gc, Hv);
            Z<R> d;
            if constexpr (OWN_D)
                d = zscale(omegaJ * shell_dinv(L, ctab, o.cc), r);
            else
                d = zmul(o.dc, r);
            res = zadd(o.p0, d);
        }
        if constexpr (!INNER) {
            // the condition again: kept over the row, `interior` spills five registers of the restriction
            if (!(r0_ok && z >= 1 && z <= L.nz - 1)) res = zero;
        }
        if constexpr (RESTRICT) {
            // full weighting along x (this lane's fine x is even on the storing
            // lanes) and along z (running sums over the coarse planes), stored per
            // fine row; the y weights follow in a second pass
            const Z<R> rl = zleft(res), rr = zright(res);
            const Z<R> rx = {(R)0.25 * (rl.r + rr.r) + (R)0.5 * res.r, (R)0.25 * (rl.i + rr.i) + (R)0.5 * res.i};
            if (z & 1) {   // odd fine plane: completes coarse plane (z-1)/2, starts (z+1)/2
                rcur.r += (R)0.25 * rx.r;
                rcur.i += (R)0.25 * rx.i;
                const int Zc = (z - 1) >> 1;
                if (rstore && z >= 2 * Z0 + 1 && Zc >= 1 && Zc <= nzc - 1)
                    y[(long long)Zc * wsy + (long long)yg * wsx + (xg >> 1)] = qz<TY>(rcur, my);
                rcur = {(R)0.25 * rx.r, (R)0.25 * rx.i};
            } else {
                rcur.r += (R)0.5 * rx.r;
                rcur.i += (R)0.5 * rx.i;
            }
        } else {
            if constexpr (MODE == M_JAC2_ADD) {
                res.r += o.bc.r;
                res.i += o.bc.i;
            }
            const auto yb = plane_buf(y + (unsigned long long)(unsigned)z * sy, sy);
            if (may_stream(MODE, NORM) && stream)
                buf_store<2>(yb, store_off, store_row, qz<TY>(res, my));
            else
                buf_store(yb, store_off, store_row, qz<TY>(res, my));
            if constexpr (NORM) {
                if (out_lane) nrm += (double)res.r * (double)res.r + (double)res.i * (double)res.i;
            }
        }
    };

    // The first three planes are loaded at once; then two planes of loads stay in flight: a
    // step issues plane z+3, forms the output of plane z, then turns the already-arrived plane
    // z+2 into partial sums.  Plane slots rotate with period 3 and load buffers with period 2.
    Plane<R> P0, P1, P2;
    Raw ra, rb;
    {
        Raw rc;
        issue(z0 - 1, ra);
        issue(z0, rb);
        issue(z0 + 1, rc);
        finish(z0 - 1, ra, P0);
        finish(z0, rb, P1);
        issue(z0 + 2, rb);
        finish(z0 + 1, rc, P2);
    }
    auto step = [&](int z, const Plane<R> &m, const Plane<R> &o, const Plane<R> &p, Plane<R> &slot,
                    const Raw &arrived, Raw &next) -> bool {
        issue(z + 3, next);
        emit(z, m, o, p);
        if (z + 1 >= z1) return false;
        finish(z + 2, arrived, slot);   // slot (held plane z-1) now holds plane z+2
        return true;
    };
    for (int z = z0;; z += 6) {
        if (!step(z, P0, P1, P2, P0, rb, ra)) break;
        if (!step(z + 1, P1, P2, P0, P1, ra, rb)) break;
        if (!step(z + 2, P2, P0, P1, P2, rb, ra)) break;
        if (!step(z + 3, P0, P1, P2, P0, ra, rb)) break;
        if (!step(z + 4, P1, P2, P0, P1, rb, ra)) break;
        if (!step(z + 5, P2, P0, P1, P2, ra, rb)) break;
    }
}

// Wavefronts a SIMD: four in single precision (128 registers; no kernel spills), two of up to 256 in double.
template <typename R>
constexpr int waves_per_simd() {
    return sizeof(R) == sizeof(float) ? 4 : 1;
}

// Whether a kernel has the INNER variant: FP32 sweeps, fused Jacobi and shifted operators.  The unshifted FP32
// apply and residuals run on the fine level, where the memory path bounds them and waves of two speeds cost
// more than the shorter code gives (352^3, with and without it: apply 246 and 239 us, residual 308 and 299,
// restricted 295 and 288; the unshifted 2h apply takes 29 us either way).  In FP64 it changes nothing (352^3
// at the best depths: apply 419 and 421 us, residual 532 and 531, J2 589 and 587; S_h at 208^3 724 and 723).
template <typename R>
constexpr bool has_inner(int mode, bool shifted) {
    return sizeof(R) == sizeof(float) && (shifted || !(mode == M_APPLY || mode == M_RESID || mode == M_RESID_R));
}

template <typename R, typename TX, typename TG, typename TY, int MODE, bool SHIFT, bool NORM, int PART>
__global__ void __launch_bounds__(64 * kWavesY, waves_per_simd<R>())
k_stencil(LevelArgs<R> L, const TX *__restrict__ x, const TG *__restrict__ g, const TY *__restrict__ base,
          TY *__restrict__ y, R omegaJ, TileMap M, RedBuf rb, KState *st, Scales sc, Batch bt) {
    // XCD-aware order of (tile, slot) pairs: block b runs on XCD b % 8; each XCD takes a
    // contiguous range of u = tile * slots + slot, so the slots of one tile run back to
    // back on one XCD and share the tile's per-node values and D^-1 through its L2.
    const int nb = gridDim.x, b = blockIdx.x;
    const int per = nb / 8, rem = nb % 8, xcd = b % 8, idx = b / 8;
    const int u = (xcd < rem) ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
    const int sl = u % bt.n;   // batched right-hand side: its own vectors, state and partials
    int t = u / bt.n;
    const int tile = t;
    if (slot_off(bt, sl)) return;
    {
        const long long nn = (long long)(L.nz + 1) * L.sy;
        x = slot_ptr(x, nn, sl);
        g = slot_ptr(g, nn, sl);
        base = slot_ptr(base, nn, sl);
        // M_RESID_R writes the x/z-restricted rows [coarse z][fine y][coarse x]
        y = slot_ptr(y, MODE == M_RESID_R ? (long long)((L.nz >> 1) + 1) * (L.ny + 1) * ((L.nx >> 1) + 1) : nn, sl);
        st = slot_ptr(st, 1, sl);
        rb = slot_rb(rb, bt, sl);
        sc.x = slot_scale(sc.x, sl);
        sc.g = slot_scale(sc.g, sl);
        sc.b = slot_scale(sc.b, sl);
        sc.y = slot_scale(sc.y, sl);
    }
    const R mul[4] = {load_mul<R, TX>(sc.x), load_mul<R, TG>(sc.g), load_mul<R, TY>(sc.b), store_mul<R, TY>(sc.y)};
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    R *etab = reinterpret_cast<R *>(smem_raw);   // alpha pieces, then (FP32) the shell quintics
    R *ctab = etab + 20 * L.nk;
    const int tid = threadIdx.x + 64 * threadIdx.y;
    // the level's window of table intervals only (at 4h almost every node is in the clamped one)
    for (int i = tid; i < L.nk * 20; i += 64 * kWavesY) etab[i] = L.etab[L.kb * 20 + i];
    if (scaled_coordinate<R>())
        for (int i = tid; i < L.nck * 24; i += 64 * kWavesY) ctab[i] = L.ctab[L.cb * 24 + i];
    __syncthreads();

    // the wavefront's tile, rows and chunk: in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.y);
    int xt, yt, zc;
    bool edge = false;
    if (PART == 1) {
        xt = t % M.nxi;
        t /= M.nxi;
        yt = M.yt_lo + t % M.nyi;
        zc = t / M.nyi;
    } else if (PART == 2) {
        // per chunk of planes the edge blocks, then the inner tiles of the rows PART 1 leaves
        const int per_z = M.neb + (M.nyt - M.nyi) * M.nxi;
        zc = t / per_z;
        int v = t - zc * per_z;
        edge = v < M.neb;
        xt = 0;
        yt = v;
        if (!edge) {
            v -= M.neb;
            xt = v % M.nxi;
            yt = v / M.nxi;
            if (yt >= M.yt_lo) yt += M.nyi;
        }
    } else if (MODE == M_RESID_R) {
        // no edge tiles: two divisions instead of four (32^3 to 132 x 40 x 48: 1 to 2% of the call)
        xt = t % M.nxi;
        t /= M.nxi;
        yt = t % M.nyt;
        zc = t / M.nyt;
    } else {
        // the blocks of neighbouring tiles follow each other, so that they run together and the cache
        // merges the sectors that two of them write: per `rows` groups of rows one edge block, then
        // their inner tiles, x fastest
        const int ne = M.strip ? 1 : 0, unit = ne + M.rows * M.nxi;
        const int per_z = M.neb + M.nyt * M.nxi;   // the last unit of a chunk may be shorter
        zc = t / per_z;
        int v = t - zc * per_z;
        const int q = v / unit;
        v -= q * unit;
        edge = v < ne;
        v -= ne;
        xt = edge ? 0 : v % M.nxi;
        yt = edge ? q : q * M.rows + v / M.nxi;
    }
    const int lane = threadIdx.x;
    const int yg = yt * kWavesY + wave;   // the row (edge tiles: the group of rows)
    // rows yg - 1 .. yg + 1 inside the box and row yg free of stretching (hd = 1: all three)
    constexpr int hd = own_dinv<R>(MODE, SHIFT) ? 1 : 0;
    const bool y_inner = yg >= max(L.loy + hd, 2) && yg <= min(L.hiy - hd, L.ny - 2);
    // planes za - 1 .. zb + 1 inside the box and planes za .. zb free of stretching (hd = 1: all)
    auto z_inner = [&](int za, int zb) { return za >= max(L.loz + hd, 2) && zb <= min(L.hiz - hd, L.nz - 2); };
    if (MODE == M_RESID_R) {
        // Fused residual + full weighting, first pass: x tiles of 60 fine columns
        // (lanes 0..63 hold x = 60 xt - 1 .. 60 xt + 62; the residual is valid on
        // lanes 1..62, so the odd lanes 3..61 hold the 30 coarse columns whose
        // three fine neighbours are all valid); z chunks of M.tz coarse planes,
        // marching fine planes 2 Z0 - 1 .. 2 Z1 - 1 (one odd plane shared with
        // the next chunk).
        const int xg = 60 * xt - 1 + lane;
        const int xa = max(1, 60 * xt), xb = min(60 * xt + 61, L.nx - 1);
        const bool xi = (xa > xb) || (xa >= L.lox && xb <= L.hix);
        const int Z0 = zc * M.tz, Z1 = min(Z0 + M.tz, L.nz >> 1);
        double nrm = 0.0;
        if (yg <= L.ny) {
            const bool yi = (yg >= L.loy && yg <= L.hiy) || yg < 1 || yg > L.ny - 1;
            const int za = 2 * Z0 - 1, zb = 2 * Z1;
            // lanes 1..63 read columns 60 xt .. 60 xt + 62
            const bool inner = has_inner<R>(MODE, SHIFT) && xi && y_inner && z_inner(za, zb - 1) && xt >= 1 && 60 * xt + 62 <= L.nx - 1;
#define HELM_MARCH_R(XI, YI, IN)                                                                                     \
    march<R, TX, TG, TY, MODE, SHIFT, false, XI, YI, IN>(L, etab, ctab, x, g, base, y, omegaJ, mul, xg, yg, za, zb, \
                                                         false, nrm, false, Z0)
            if (inner)
                HELM_MARCH_R(true, true, true);
            else if (xi && yi)
                HELM_MARCH_R(true, true, false);
            else if (xi)
                HELM_MARCH_R(true, false, false);
            else if (yi)
                HELM_MARCH_R(false, true, false);
            else
                HELM_MARCH_R(false, false, false);
#undef HELM_MARCH_R
        }
        return;
    }
    const int z0 = zc * M.tz;
    const int z1 = min(z0 + M.tz, L.nz + 1);
    double nrm = 0.0;
    int xg, yl = yg;                      // the lane's column and row
    bool out, xi, yi, x_inner = false;    // x_inner: every column an output lane reads lies inside the box
    bool rows_here = yg <= L.ny;
    if (edge) {
        // rows of 2 (strip + 2) lanes: x = -1 .. strip, then nx - strip .. nx + 1; the first and last lane
        // of each strip only supply the halo
        const int ls = M.strip + 2, sub = lane / (2 * ls), j = lane - sub * 2 * ls, half = j >= ls ? 1 : 0;
        const int i = j - half * ls, ya = yg * M.rows;
        yl = ya + sub;
        xg = half ? L.nx - M.strip + i : i - 1;
        out = i >= 1 && i <= M.strip && yl <= L.ny;
        xi = false;
        yi = ya >= L.loy && ya + M.rows - 1 <= L.hiy;
        rows_here = ya <= L.ny;
    } else {
        if (M.strip) {
            xg = M.strip - 1 + xt * kTileX + lane;
            out = lane >= 1 && lane <= kTileX && xg <= L.nx - M.strip;
            xi = true;             // columns strip - 1 .. nx - strip + 1
            x_inner = !hd || (L.lox <= M.strip - 1 && L.hix >= L.nx - M.strip + 1);
        } else {
            xg = xt * kTileX - 1 + lane;
            out = lane >= 1 && lane <= kTileX && xg <= L.nx;
            const int xa = max(1, xt * kTileX), xb = min(xt * kTileX + kTileX - 1, L.nx - 1);
            xi = (xa > xb) || (xa >= L.lox && xb <= L.hix);
            x_inner = xi && xt * kTileX - 1 >= max(1, hd * L.lox) && xt * kTileX + kTileX <= min(L.nx - 1, hd ? L.hix : L.nx);
        }
        yi = (yg >= L.loy && yg <= L.hiy) || yg < 1 || yg > L.ny - 1;
    }
#define HELM_MARCH(XI, YI, IN, YG)                                                                                   \
    march<R, TX, TG, TY, MODE, SHIFT, NORM, XI, YI, IN>(L, etab, ctab, x, g, base, y, omegaJ, mul, xg, YG, z0, z1,  \
                                                        out, nrm, M.stream != 0)
    if (!rows_here)
        ;
    else if (has_inner<R>(MODE, SHIFT) && x_inner && y_inner && z_inner(z0, z1 - 1))
        HELM_MARCH(true, true, true, yg);
    else if (xi && yi)
        HELM_MARCH(true, true, false, yg);
    else if (PART == 1)   // inner rows: no stretching
        ;
    else if (xi)
        HELM_MARCH(true, false, false, yg);
    else if (yi)
        HELM_MARCH(false, true, false, yl);
    else
        HELM_MARCH(false, false, false, yl);
#undef HELM_MARCH
    if (NORM) {
        block_reduce_store(nrm, rb.partials + M.block_offset + tile);
        norm_epilogue(rb, M.total_blocks, st);
    }
}

// Amplitude correction Q_h (eq. q-operator): row i takes the shell weights of its own node
// (from beta at the fine-grid eta*) on its interior neighbours, with no stretching and no
// ell^-2.  One wavefront per row y at 64 consecutive x (outputs on lanes 1..62, neighbours
// x -+ 1 through DPP), marching kQZ planes in z: every plane gives its in-plane shell sums of
// the interior values, S0 (centre), S1 (four faces) and S2 (four corners), and output plane z
// takes Q0 S0(z) + Q1 (S1(z) + S0(z-+1)) + Q2 (S2(z) + S1(z-+1)) + Q3 S2(z-+1).  The loads of
// plane p + 1 are issued before plane p is summed.
constexpr int kQZ = 16, kQX = 62;

template <typename R>
struct QSums {
    Z<R> s0, s1, s2;
};

template <typename R, typename TI, typename TO>
__global__ void __launch_bounds__(256) k_qapply(LevelArgs<R> L, const TI *__restrict__ x, TO *__restrict__ y,
                                               Batch bt) {
    const int sl = blockIdx.z;   // batched right-hand side
    if (slot_off(bt, sl)) return;
    const long long nn = (long long)(L.nz + 1) * L.sy;
    x = slot_ptr(x, nn, sl);
    y = slot_ptr(y, nn, sl);
    extern __shared__ unsigned char smem_raw[];
    R *btab = reinterpret_cast<R *>(smem_raw);
    for (int i = threadIdx.x + 64 * threadIdx.y; i < L.K * 12; i += 256) btab[i] = L.btab[i];
    __syncthreads();
    const int ntx = (L.nx + kQX) / kQX;   // x tiles covering nodes 0..nx
    const int xt = blockIdx.x % ntx, yt = blockIdx.x / ntx;
    const int lane = threadIdx.x, yg = yt * 4 + threadIdx.y;
    const int xg = xt * kQX - 1 + lane;
    if (yg > L.ny) return;   // whole wavefronts leave; no barrier follows
    const int z0 = blockIdx.y * kQZ, z1 = min(z0 + kQZ, L.nz + 1);
    const bool x_int = xg >= 1 && xg <= L.nx - 1;
    const bool out_lane = lane >= 1 && lane <= kQX && xg <= L.nx;
    const int xc = min(max(xg, 0), L.nx);
    const int ym = max(yg - 1, 0), yp = min(yg + 1, L.ny);
    const bool rm_ok = x_int && yg - 1 >= 1, r0_ok = x_int && yg >= 1 && yg <= L.ny - 1, rp_ok = x_int && yg + 1 <= L.ny - 1;
    const long long om = (long long)ym * L.sx + xc, o0 = (long long)yg * L.sx + xc, op = (long long)yp * L.sx + xc;
    const Z<R> zero = {0, 0};
    struct Raw {
        TI a, b, c;
    };
    auto issue = [&](int p, Raw &r) {
        const long long base = (long long)min(max(p, 0), L.nz) * L.sy;
        r.a = x[base + om];
        r.b = x[base + o0];
        r.c = x[base + op];
    };
    auto sums = [&](int p, const Raw &r) {
        const bool zok = p >= 1 && p <= L.nz - 1;
        const Z<R> a = (zok && rm_ok) ? Z<R>{(R)r.a.re, (R)r.a.im} : zero;
        const Z<R> b = (zok && r0_ok) ? Z<R>{(R)r.b.re, (R)r.b.im} : zero;
        const Z<R> c = (zok && rp_ok) ? Z<R>{(R)r.c.re, (R)r.c.im} : zero;
        const Z<R> col = zadd(a, c);
        QSums<R> q;
        q.s0 = b;
        q.s1 = zadd(col, zadd(zleft(b), zright(b)));
        q.s2 = zadd(zleft(col), zright(col));
        return q;
    };
    auto emit = [&](int z, const QSums<R> &m, const QSums<R> &o, const QSums<R> &p) {
        if (!out_lane || z < z0 || z >= z1) return;
        Z<R> acc = zero;
        if (r0_ok && z >= 1 && z <= L.nz - 1) {
            R kappa, t;
            int k;
            locate(L, L.c[(long long)z * L.sy + o0], kappa, k, t);
            const R *bp = btab + k * 12;
            const R b1 = horner(bp, t), b2 = horner(bp + 4, t), b3 = horner(bp + 8, t);
            const R Q[4] = {b1, b2 * (R)(1.0 / 6), b3 * (R)(1.0 / 12), ((R)1 - b1 - b2 - b3) * (R)0.125};
            acc = zscale(Q[0], o.s0);
            acc = zadd(acc, zscale(Q[1], zadd(o.s1, zadd(m.s0, p.s0))));
            acc = zadd(acc, zscale(Q[2], zadd(o.s2, zadd(m.s1, p.s1))));
            acc = zadd(acc, zscale(Q[3], zadd(m.s2, p.s2)));
        }
        TO v;
        v.re = acc.r;
        v.im = acc.i;
        y[(long long)z * L.sy + o0] = v;
    };
    // window of plane sums: m (z - 1), o (z), p (z + 1); output plane z after plane z + 1 is summed
    Raw ra, rb;
    issue(z0 - 1, ra);
    issue(z0, rb);
    QSums<R> m = sums(z0 - 1, ra);
    issue(z0 + 1, ra);
    QSums<R> o = sums(z0, rb);
    for (int z = z0; z < z1; z += 2) {
        issue(z + 2, rb);
        const QSums<R> p = sums(z + 1, ra);   // plane z + 1 (issued one step earlier)
        emit(z, m, o, p);
        m = o;
        o = p;
        if (z + 1 >= z1) break;
        issue(z + 3, ra);
        const QSums<R> p2 = sums(z + 2, rb);
        emit(z + 1, m, o, p2);
        m = o;
        o = p2;
    }
}

// y = diag(H) x (test and diagnostics hook)
template <typename R, typename T, bool SHIFT>
__global__ void __launch_bounds__(256) k_diag(LevelArgs<R> L, const T *__restrict__ x, T *__restrict__ y) {
    extern __shared__ unsigned char smem_raw[];
    R *stab = reinterpret_cast<R *>(smem_raw);
    for (int i = threadIdx.x; i < L.nk * 20; i += blockDim.x) stab[i] = L.atab[L.kb * 20 + i];
    __syncthreads();
    const long long nn = (long long)(L.nz + 1) * L.sy;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < nn; i += (long long)gridDim.x * blockDim.x) {
        const int xi = (int)(i % L.sx);
        const int yi = (int)((i / L.sx) % (L.ny + 1));
        const int zi = (int)(i / L.sy);
        Z<R> r = {0, 0};
        if (xi >= 1 && xi <= L.nx - 1 && yi >= 1 && yi <= L.ny - 1 && zi >= 1 && zi <= L.nz - 1) {
            Coef<R> cf = coef_at(L, stab, node_values(L)[i]);
            Z<R> ws = {L.wx[6 * xi + 2] + L.wy[6 * yi + 2] + L.wz[6 * zi + 2],
                       L.wx[6 * xi + 3] + L.wy[6 * yi + 3] + L.wz[6 * zi + 3]};
            r = zmul(diag_of<R, SHIFT>(L, cf.a1, cf.a4, cf.k2, ws), ld<R>(x, i));
        }
        T o;
        o.re = r.r;
        o.im = r.i;
        y[i] = o;
    }
}

// one Jacobi sweep from zero: y = omega D^-1 g (eq. jacobi-map with n_J = 1)
template <typename R, typename T>
__global__ void __launch_bounds__(256) k_jac1(const R *__restrict__ dinv, const T *__restrict__ g, T *__restrict__ y,
                                              long long nn, R omegaJ, Batch bt) {
    if (slot_off(bt, blockIdx.y)) return;
    g = slot_ptr(g, nn, blockIdx.y);
    y = slot_ptr(y, nn, blockIdx.y);
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < nn; i += (long long)gridDim.x * blockDim.x) {
        const Z<R> r = zscale(omegaJ, zmul(Z<R>{dinv[2 * i], dinv[2 * i + 1]}, ld<R>(g, i)));
        T o;
        o.re = r.r;
        o.im = r.i;
        y[i] = o;
    }
}

// D^-1 at every node of a level (zero on the boundary): the diagonal depends
// only on the velocity, the stretching and the shift, so the Jacobi kernels
// read it instead of evaluating the coefficients of every neighbour row.
template <typename R, bool SHIFT>
__global__ void __launch_bounds__(256) k_dinv(LevelArgs<R> L, R *__restrict__ out) {
    extern __shared__ unsigned char smem_raw[];
    R *stab = reinterpret_cast<R *>(smem_raw);
    for (int i = threadIdx.x; i < L.nk * 20; i += blockDim.x) stab[i] = L.atab[L.kb * 20 + i];
    __syncthreads();
    const long long nn = (long long)(L.nz + 1) * L.sy;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < nn; i += (long long)gridDim.x * blockDim.x) {
        const int xi = (int)(i % L.sx);
        const int yi = (int)((i / L.sx) % (L.ny + 1));
        const int zi = (int)(i / L.sy);
        Z<R> r = {0, 0};
        if (xi >= 1 && xi <= L.nx - 1 && yi >= 1 && yi <= L.ny - 1 && zi >= 1 && zi <= L.nz - 1) {
            Coef<R> cf = coef_at(L, stab, node_values(L)[i]);
            Z<R> ws = {L.wx[6 * xi + 2] + L.wy[6 * yi + 2] + L.wz[6 * zi + 2],
                       L.wx[6 * xi + 3] + L.wy[6 * yi + 3] + L.wz[6 * zi + 3]};
            r = zdiv(Z<R>{1, 0}, diag_of<R, SHIFT>(L, cf.a1, cf.a4, cf.k2, ws));
        }
        out[2 * i] = r.r;
        out[2 * i + 1] = r.i;
    }
}

int pick_tz(int ntx, int nty, int nz1) {
    long long work = (long long)ntx * nty * nz1;
    long long tz = (work + 4095) / 4096;
    if (tz < 4) tz = 4;
    if (tz > 64) tz = 64;
    return (int)tz;
}

// Modes each operand-type combination is built for: all of them for FP32 / FP64 operands;
// for FP16-stored ones (HELM_MIXED) only those the mixed-precision cycle uses, without the
// fused norm: the V-cycle's first Jacobi y = J(B, q) (c32 -> c16), the fused residual +
// restriction and the residual from y (c16 x), the bottom basis steps and the V-cycle's
// last Jacobi + base (all c16), and K_2h's A_2h Z (c16 -> c32).
template <typename TX, typename TG, typename TY>
constexpr bool mode_built(int mode, bool shifted, bool norm) {
    constexpr bool hx = is_half<TX>(), hg = is_half<TG>(), hy = is_half<TY>();
    if (!hx && !hg && !hy) return true;
    if (norm) return false;
    if (!hx && !hg && hy) return mode == M_JAC2 && shifted;
    if (hx && hg && hy) return (mode == M_JAC2 || mode == M_APPLY || mode == M_JAC2_ADD) && shifted;
    if (hx && !hg && !hy) return mode == M_RESID_R && shifted;
    if (hx && !hg && hy) return mode == M_RESID && shifted;
    if (hx && hg && !hy) return mode == M_APPLY && !shifted;
    return false;
}

}  // namespace

template <typename R, typename TX, typename TG, typename TY, int PART>
hipError_t launch_stencil_part(const LevelArgs<R> &L, const StencilCall &c, const RedBuf &rb, const TileMap &M,
                               int blocks, hipStream_t s) {
    const dim3 blk(64, kWavesY);
    const size_t shm = sizeof(R) * (L.nk * 20 + (scaled_coordinate<R>() ? L.nck * 24 : 0));
    const TX *x = (const TX *)c.x;
    const TG *g = (const TG *)c.g;
    const TY *base = (const TY *)c.base;
    TY *y = (TY *)c.y;
    const R om = (R)c.omegaJ;
    const Scales sc = {c.sx, c.sg, c.sb, c.sy};
    const Batch &bt = cur_batch();
#define HELM_LAUNCH(MODE, SH, NRM)                                                                                  \
    do {                                                                                                            \
        if constexpr (mode_built<TX, TG, TY>(MODE, SH, NRM))                                                        \
            hipLaunchKernelGGL((k_stencil<R, TX, TG, TY, MODE, SH, NRM, PART>), dim3(blocks * bt.n), blk, shm, s, L, \
                               x, g, base, y, om, M, rb, c.st, sc, bt);                                             \
        else                                                                                                        \
            return hipErrorInvalidValue;                                                                            \
    } while (0)
    if (c.norm) {
        if (c.mode != M_RESID) return hipErrorInvalidValue;
        if (c.shifted)
            HELM_LAUNCH(M_RESID, true, true);
        else
            HELM_LAUNCH(M_RESID, false, true);
        return hipGetLastError();
    }
    switch (c.mode) {
    case M_APPLY:
        if (c.shifted) HELM_LAUNCH(M_APPLY, true, false); else HELM_LAUNCH(M_APPLY, false, false);
        break;
    case M_RESID:
        if (c.shifted) HELM_LAUNCH(M_RESID, true, false); else HELM_LAUNCH(M_RESID, false, false);
        break;
    case M_JSWEEP:
        if (c.shifted) HELM_LAUNCH(M_JSWEEP, true, false); else HELM_LAUNCH(M_JSWEEP, false, false);
        break;
    case M_JAC2:
        if (c.shifted) HELM_LAUNCH(M_JAC2, true, false); else HELM_LAUNCH(M_JAC2, false, false);
        break;
    case M_JAC2_ADD:
        if (c.shifted) HELM_LAUNCH(M_JAC2_ADD, true, false); else HELM_LAUNCH(M_JAC2_ADD, false, false);
        break;
    case M_RESID_R:
        if constexpr (PART == 0) {
            if (c.shifted) HELM_LAUNCH(M_RESID_R, true, false); else HELM_LAUNCH(M_RESID_R, false, false);
        } else {
            return hipErrorInvalidValue;
        }
        break;
    default:
        return hipErrorInvalidValue;
    }
#undef HELM_LAUNCH
    return hipGetLastError();
}

template <typename R, typename TX, typename TG, typename TY>
hipError_t launch_stencil(const LevelArgs<R> &L, const StencilCall &c, const RedBuf &rb, hipStream_t s) {
    if (scaled_coordinate<R>() && (!L.s || !L.ctab)) return hipErrorInvalidValue;   // FP32 levels read s
    // the Jacobi modes read the stored D^-1 of the operator
    if ((c.mode == M_JSWEEP || c.mode == M_JAC2 || c.mode == M_JAC2_ADD) && !L.dinv[c.shifted ? 1 : 0])
        return hipErrorInvalidValue;
    if (c.mode == M_RESID_R) {
        if (c.norm) return hipErrorInvalidValue;
        const int depth = L.tz_restrict > 0 ? L.tz_restrict : restrict_depth(L.nx, L.ny, L.nz, cur_batch().n);
        const TileMap M = restrict_tiles(L.nx, L.ny, L.nz, depth);
        return launch_stencil_part<R, TX, TG, TY, 0>(L, c, rb, M, M.total_blocks, s);
    }
    const int fam = (c.mode == M_JAC2 || c.mode == M_JAC2_ADD) ? 1 : 0;
    const int tz = L.tz[fam] > 0 ? L.tz[fam] : pick_tz(ceil_div(L.nx + 1, kTileX), ceil_div(L.ny + 1, kWavesY), L.nz + 1);
    TileMap M = make_tiles(L.nx, L.ny, L.nz, L.lox, L.hix, tz);
    if (c.norm && M.total_blocks > rb.cap) return hipErrorInvalidValue;   // a partial a block
    M.stream = c.stream;
    if (L.split[fam] && M.strip) {
        // groups of four rows all inside [loy, hiy]
        M.yt_lo = ceil_div(L.loy, kWavesY);
        M.nyi = std::max(0, (L.hiy + 1) / kWavesY - M.yt_lo);
        const int bi = M.nxi * M.nyi * ceil_div(L.nz + 1, tz), bb = M.total_blocks - bi;
        if (bi > 0 && bb > 0) {
            const hipError_t e = launch_stencil_part<R, TX, TG, TY, 2>(L, c, rb, M, bb, s);
            if (e != hipSuccess) return e;
            M.block_offset = bb;
            return launch_stencil_part<R, TX, TG, TY, 1>(L, c, rb, M, bi, s);
        }
        M.yt_lo = M.nyi = 0;
    }
    return launch_stencil_part<R, TX, TG, TY, 0>(L, c, rb, M, M.total_blocks, s);
}

}  // namespace helm
