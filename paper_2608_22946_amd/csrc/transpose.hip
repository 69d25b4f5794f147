// Transposed level operators A^T, B^T (adjoint solves and products), optionally as a residual.
//
// Every row takes its coefficients at its own node, so the transpose gathers: output k sums, over its
// 27 neighbours i, row i's coefficient for the offset k - i times x_i.  The coefficients of a row
// multiply fixed shapes (the shells, or the 1-D second differences times transverse shells), so
// each node first forms the products of its coefficients with x (once), and the outputs are
// plain sums of those products along x, y and z:
//   free of stretching (eq. iofd-shell-form), u_m = C_m(i) x_i, E v = v(x-1) + v(x+1):
//     A0 = u0 + E u1, A1 = u1 + E u2, A2 = u2 + E u3 within a row;
//     same plane: A0 + (A1 of rows y -+ 1); planes z -+ 1: A1 + (A2 of rows y -+ 1).
//   stretched: with t_n = T_n x (T = a4, a5 / 4, q / 4), m_n = mu kappa^2 M_n x and the x difference
//   D of the transposed weights: P = t0 + E t1, Q = t1 + E t2, U_n = D t_n - m_n - E m_(n+1);
//     same plane: U0 + (wy0 + wz0) P + rows (U1 + wy P + wz0 Q);
//     planes z -+ 1: U1 + wy0 Q + rows (U2 + wy Q) + wz (P + rows Q).
//
// A wavefront owns one row of 64 columns (62 outputs) and marches in z; x neighbours come by DPP, and
// what a row passes to its neighbours (two complex numbers a lane, four where y or z is stretched)
// goes through LDS: twelve rows a block, ten of them with outputs, one barrier a plane.  So x and
// the velocity are read 1.2 times and the coefficients evaluated 1.2 times a node.  As in the forward
// stencils the edge tiles hold both x-PML strips of a row where these fit in 30 columns, and every
// other tile is free of x stretching; the form along y and z is chosen plane by plane.
//
// What bounds it: the LDS (five 16-byte reads a node for the coefficients, three to six accesses for the
// exchange) and the vector unit about equally, then the imbalance of the stretched blocks, which
// take about twice the time of the others.  A^T at 216^3 145 -> 86 us in FP32 and 264 -> 189 us in
// FP64, at 352^3 457 -> 290 and 840 -> 610 us, at 64^3 40 -> 11 and 47 -> 18 us, against a block of
// 64 x 4 outputs that staged nine values a node in LDS and read 27 neighbours' terms from there.
// Measured and not kept: eight rows a block (96 us at 216^3) and sixteen (104 us: one block a CU), the
// quintic table of the shell coefficients (six reads a node: 290 -> 295 us at 352^3), and
// contiguous ranges of blocks a XCD (310 us; the XCDs with the z-PML chunks finish last).
#include "stencil_impl.h"

namespace helm {
namespace {

// Twelve rows a block, two blocks a CU (24 wavefronts of up to 80 registers).  FP64 rows hold twice the
// LDS (8 KB): one exchange buffer and two barriers a plane instead of two buffers and one.
constexpr int kRowsT = 12;
template <typename R>
constexpr int kBufT = sizeof(R) == sizeof(float) ? 2 : 1;
constexpr int kStripT = 30;

template <typename R>
__device__ __forceinline__ Z<R> both(Z<R> c, Z<R> v) { return zadd(zadd(c, zleft(v)), zright(v)); }   // c + E v

// axis_w(a + d, -d), d = -1, 0, 1: weight of the neighbour row a + d for output a
template <typename R>
__device__ __forceinline__ void weights_t(const R *w, int a, int n, Z<R> (&o)[3]) {
    const bool in = a >= 1 && a <= n - 1;
    const int c = min(max(a, 1), n - 1);
#pragma unroll
    for (int d = -1; d <= 1; ++d) {
        const R *p = w + 6 * (c + d) + 2 * (1 - d);
        o[d + 1] = in ? Z<R>{p[0], p[1]} : Z<R>{0, 0};
    }
}

// what a lane of a row passes to the rows beside it
template <typename R, int N>
struct alignas(16) RowOut {
    Z<R> v[N];
};

// a row's products with its stretched coefficients, combined along x
template <typename R>
struct Terms {
    Z<R> P, Q, U0, U1, U2;
};
template <typename R, bool SHIFT, bool XI>
__device__ __forceinline__ Terms<R> terms(const LevelArgs<R> &L, const R *etab, float c, Z<R> xv, const Z<R> (&Wx)[3]) {
    const RowCoef<R> f = row_coef(L, etab, c);
    const Z<R> t0 = zscale(f.a4, xv), t1 = zscale((R)0.25 * f.a5, xv), t2 = zscale((R)0.25 * f.q, xv);
    Z<R> kx = zscale(f.k2, xv);
    if (SHIFT) kx = {kx.r - L.sigma * kx.i, kx.i + L.sigma * kx.r};
    const Z<R> m0 = zscale(f.m0, kx), m1 = zscale(f.m1, kx), m2 = zscale(f.m2, kx), m3 = zscale(f.m3, kx);
    Terms<R> o;
    if constexpr (XI) {   // D t = 2 t - E t
        const Z<R> e1 = zadd(zleft(t1), zright(t1)), e2 = zadd(zleft(t2), zright(t2));
        o.P = zadd(t0, e1);
        o.Q = zadd(t1, e2);
        o.U0 = both(twice_less(t0, m0), Z<R>{-(t0.r + m1.r), -(t0.i + m1.i)});
        o.U1 = zsub(both(twice_less(t1, m1), Z<R>{-m2.r, -m2.i}), e1);
        o.U2 = zsub(both(twice_less(t2, m2), Z<R>{-m3.r, -m3.i}), e2);
    } else {
        const Z<R> l1 = zleft(t1), q1 = zright(t1), l2 = zleft(t2), q2 = zright(t2);
        o.P = zadd(zadd(t0, l1), q1);
        o.Q = zadd(zadd(t1, l2), q2);
        o.U0 = zsub(wdot(Wx, zleft(t0), t0, zright(t0)), both(m0, m1));
        o.U1 = zsub(wdot(Wx, l1, t1, q1), both(m1, m2));
        o.U2 = zsub(wdot(Wx, l2, t2, q2), both(m2, m3));
    }
    return o;
}

template <typename R, typename TX, typename TG, typename TY, bool SHIFT, bool RESID, bool XI>
__device__ __forceinline__ void march_t(const LevelArgs<R> &L, const R *etab, const TX *__restrict__ x,
                                        const TG *__restrict__ g, TY *__restrict__ y, unsigned char *xch, int X, int Y,
                                        bool out_lane, bool yin, int Zb, int Ze) {
    constexpr int W = kRowsT;
    const int lane = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const unsigned sy = (unsigned)L.sy;
    const int xc = min(max(X, 0), L.nx), yc = min(max(Y, 0), L.ny);
    const unsigned lx = (unsigned)xc, r0 = (unsigned)(yc * (int)L.sx);
    const bool inxy = X >= 1 && X <= L.nx - 1 && Y >= 1 && Y <= L.ny - 1;
    const float *vnode = node_values(L);
    Z<R> Wx[3];
    if constexpr (!XI) weights_t(L.wx, X, L.nx, Wx);
    struct Raw {
        TX x;
        TG g;
        float c;
    };
    auto issue = [&](int p, Raw &r) {   // plane p of x, plane p - 1 of g; clamped to the grid
        const unsigned long long po = (unsigned long long)(unsigned)min(max(p, 0), L.nz) * sy;
        r.x = buf_load<TX>(plane_buf(x + po, sy), lx * (unsigned)sizeof(TX), r0 * (unsigned)sizeof(TX));
        r.c = buf_load<float>(plane_buf(vnode + po, sy), lx * 4u, r0 * 4u);
        if constexpr (RESID) {
            const unsigned long long pg = (unsigned long long)(unsigned)min(max(p - 1, 0), L.nz) * sy;
            r.g = buf_load<TG>(plane_buf(g + pg, sy), lx * (unsigned)sizeof(TG), r0 * (unsigned)sizeof(TG));
        }
    };
    unsigned store_off, store_row;
    row_store_offsets<TY>(out_lane, true, lx, r0, store_off, store_row);
    Z<R> acc0 = {0, 0}, acc1 = {0, 0}, acc2 = {0, 0};   // sums of the outputs in planes p - 1, p, p + 1
    const int here = wave * 64 + lane;
    // the first and last row have no outputs
    const int up = min(wave + 1, W - 1) * 64 + lane, dn = max(wave - 1, 0) * 64 + lane;
    auto exchange = [&](auto *buf, const auto &o, auto &a, auto &b) {
        if (kBufT<R> == 1) __syncthreads();   // the other rows have read the plane before
        buf[here] = o;
        __syncthreads();
        a = buf[dn];
        b = buf[up];
    };
    auto plane = [&](int p, const Raw &r, unsigned char *xb) {
        Z<R> xv = {(R)r.x.re, (R)r.x.im};
        if (!(inxy && p >= 1 && p <= L.nz - 1)) xv = {0, 0};   // rows exist at interior nodes only
        if (yin && p >= L.loz && p <= L.hiz) {
            // free of stretching in y and z: what goes to the planes z -+ 1 of a row also goes to its
            // neighbours in the plane
            RowOut<R, 2> o, a, b;
            Z<R> own;
            if constexpr (XI) {
                const RowCoef<R> f = row_coef(L, etab, r.c);
                const R M[4] = {f.m0, f.m1, f.m2, f.m3};
                const R C[4] = {(R)6 * f.a4 - f.k2 * f.m0, (f.a5 - f.a4) - f.k2 * f.m1,
                                (R)0.5 * (f.q - f.a5) - f.k2 * f.m2, (R)-0.75 * f.q - f.k2 * f.m3};
                const R sk = L.sigma * f.k2;
                const Z<R> ix = {sk * xv.i, -(sk * xv.r)};   // - i sigma kappa^2 x
                Z<R> u[4];
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    u[m] = SHIFT ? Z<R>{C[m] * xv.r + M[m] * ix.r, C[m] * xv.i + M[m] * ix.i} : zscale(C[m], xv);
                own = both(u[0], u[1]);
                o.v[0] = both(u[1], u[2]);
                o.v[1] = both(u[2], u[3]);
            } else {
                const Terms<R> t = terms<R, SHIFT, false>(L, etab, r.c, xv, Wx);
                own = {t.U0.r + (R)4 * t.P.r, t.U0.i + (R)4 * t.P.i};
                o.v[0] = {t.U1.r + (R)2 * t.Q.r - t.P.r, t.U1.i + (R)2 * t.Q.i - t.P.i};
                o.v[1] = {t.U2.r - (R)2 * t.Q.r, t.U2.i - (R)2 * t.Q.i};
            }
            exchange(reinterpret_cast<RowOut<R, 2> *>(xb), o, a, b);
            acc1 = zadd(acc1, zadd(own, zadd(a.v[0], b.v[0])));
            acc2 = zadd(o.v[0], zadd(a.v[1], b.v[1]));
            acc0 = zadd(acc0, acc2);
        } else {
            const Terms<R> t = terms<R, SHIFT, XI>(L, etab, r.c, xv, Wx);
            RowOut<R, 4> a, b;
            exchange(reinterpret_cast<RowOut<R, 4> *>(xb), RowOut<R, 4>{{t.P, t.Q, t.U1, t.U2}}, a, b);
            Z<R> Wy[3];
            weights_t(L.wy, Y, L.ny, Wy);
            const R *w = L.wz + 6 * min(max(p, 0), L.nz);   // x is zero on planes without rows
            const Z<R> wm = {w[0], w[1]}, w0 = {w[2], w[3]}, wp = {w[4], w[5]};
            const Z<R> qs = zadd(a.v[1], b.v[1]);
            Z<R> s = zadd(t.U0, zadd(a.v[2], b.v[2]));
            s = zfma(zadd(Wy[1], w0), t.P, s);
            s = zfma(w0, qs, s);
            s = zfma(Wy[0], a.v[0], s);
            s = zfma(Wy[2], b.v[0], s);
            Z<R> c = zadd(t.U1, zadd(a.v[3], b.v[3]));
            c = zfma(Wy[1], t.Q, c);
            c = zfma(Wy[0], a.v[1], c);
            c = zfma(Wy[2], b.v[1], c);
            const Z<R> d = zadd(t.P, qs);
            acc1 = zadd(acc1, s);
            acc0 = zadd(acc0, zfma(wm, d, c));
            acc2 = zfma(wp, d, c);
        }
        const int z = p - 1;   // its three planes of rows are in
        if (z >= Zb) {
            Z<R> v = acc0;
            if constexpr (RESID) v = {(R)r.g.re - v.r, (R)r.g.im - v.i};
            if (!(inxy && z >= 1 && z <= L.nz - 1)) v = {0, 0};
            buf_store(plane_buf(y + (unsigned long long)(unsigned)z * sy, sy), store_off, store_row,
                      TY{(decltype(TY{}.re))v.r, (decltype(TY{}.re))v.i});
        }
        acc0 = acc1;
        acc1 = acc2;
    };
    // planes Zb - 1 .. Ze, two of them in flight
    Raw ra, rb;
    issue(Zb - 1, ra);
    issue(Zb, rb);
    for (int p = Zb - 1; p <= Ze; p += 2) {
        const Raw ca = ra;
        issue(p + 2, ra);
        plane(p, ca, xch);
        if (p + 1 > Ze) break;
        const Raw cb = rb;
        issue(p + 3, rb);
        plane(p + 1, cb, xch + (kBufT<R> - 1) * sizeof(RowOut<R, 4>) * W * 64);
    }
}

template <typename R, typename TX, typename TG, typename TY, bool SHIFT, bool RESID>
__global__ void __launch_bounds__(64 * kRowsT) k_apply_t(LevelArgs<R> L, const TX *__restrict__ x,
                                                           const TG *__restrict__ g, TY *__restrict__ y, int edge,
                                                           int tz) {
    constexpr int W = kRowsT;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    R *etab = reinterpret_cast<R *>(smem_raw + sizeof(RowOut<R, 4>) * kBufT<R> * W * 64);
    const int tid = threadIdx.x + 64 * threadIdx.y;
    for (int i = tid; i < L.nk * 20; i += 64 * W) etab[i] = L.etab[L.kb * 20 + i];
    __syncthreads();
    const int lane = threadIdx.x, bx = blockIdx.x;
    const int Y0 = blockIdx.y * (W - 2);                                  // first output row
    const int Y = Y0 - 1 + __builtin_amdgcn_readfirstlane(threadIdx.y);   // this wavefront's row
    const int Zb = blockIdx.z * tz, Ze = min(Zb + tz, L.nz + 1);
    const bool edge_tile = edge && bx == 0;
    const int X0 = edge ? kStripT + (bx - 1) * kTileX : bx * kTileX;   // first output column
    int X = X0 - 1 + lane;
    bool out = lane >= 1 && lane <= kTileX && X <= (edge ? L.nx - kStripT : L.nx);
    if (edge_tile) {   // lanes 0..31: columns -1..30, lanes 32..63: nx - 30..nx + 1
        X = lane < 32 ? lane - 1 : L.nx + 1 - (63 - lane);
        out = (lane & 31) != 0 && (lane & 31) != 31;
    }
    out = out && threadIdx.y >= 1 && threadIdx.y <= W - 2 && Y <= L.ny;
    // every column (row) that the block holds free of stretching
    const bool xin = !edge_tile && X0 - 1 >= L.lox && min(X0 + kTileX, edge ? L.nx - kStripT + 1 : L.nx) <= L.hix;
    const bool yin = Y0 - 1 >= L.loy && Y0 + W - 2 <= L.hiy;
    if (xin)
        march_t<R, TX, TG, TY, SHIFT, RESID, true>(L, etab, x, g, y, smem_raw, X, Y, out, yin, Zb, Ze);
    else
        march_t<R, TX, TG, TY, SHIFT, RESID, false>(L, etab, x, g, y, smem_raw, X, Y, out, yin, Zb, Ze);
}

}  // namespace

template <typename R, typename TX, typename TG, typename TY>
hipError_t launch_apply_t(const LevelArgs<R> &L, int shifted, const TX *x, const TG *g, TY *y, hipStream_t s) {
    constexpr int W = kRowsT;
    // both strips in one tile where they hold all x stretching (the inner tiles read from column 29 on)
    const int edge = L.nx + 1 >= 2 * kStripT + 1 && L.lox <= kStripT - 1 && L.hix >= L.nx - kStripT + 1;
    const int nxt = edge ? 1 + ceil_div(L.nx + 1 - 2 * kStripT, kTileX) : ceil_div(L.nx + 1, kTileX);
    const int nyt = ceil_div(L.ny + 1, W - 2);
    // chunks of 4 to 32 planes (a chunk reads two planes more than it writes), four blocks a CU: with two
    // the stretched blocks finish last (216^3: 96 us for 86), with eight the chunks are short (92 us)
    const int chunks = std::max(1, ceil_div(1024, nxt * nyt));
    const int tz = std::min(32, std::max(4, ceil_div(L.nz + 1, chunks)));
    const dim3 grid(nxt, nyt, ceil_div(L.nz + 1, tz)), blk(64, W);
    const size_t shm = sizeof(RowOut<R, 4>) * kBufT<R> * W * 64 + sizeof(R) * L.nk * 20;
#define HELM_AT(SH, RS) hipLaunchKernelGGL((k_apply_t<R, TX, TG, TY, SH, RS>), grid, blk, shm, s, L, x, g, y, edge, tz)
    if (g) {
        if (shifted) HELM_AT(true, true); else HELM_AT(false, true);
    } else {
        if (shifted) HELM_AT(true, false); else HELM_AT(false, false);
    }
#undef HELM_AT
    return hipGetLastError();
}

template hipError_t launch_apply_t<float, c32, c32, c32>(const LevelArgs<float> &, int, const c32 *, const c32 *,
                                                         c32 *, hipStream_t);
template hipError_t launch_apply_t<double, c64, c64, c64>(const LevelArgs<double> &, int, const c64 *, const c64 *,
                                                          c64 *, hipStream_t);

}  // namespace helm
