// Fourth-order central path (section 2.6: central schemes for the convective
// terms of smooth problems and for the viscous terms; the scheme of the
// central Taylor-Green benchmark of section 6.1) on separable meshes of
// uniform spacing:
//   convection in conservative form, R_c -= sum_d D_d(F_d,c) / h_d;
//   viscous and heat-flux terms in expanded form: with g_ab = d_b u_a,
//   mu~ = mu(T)/Re and kappa = mu(T)/((gamma-1) M^2 Pr Re),
//     d_b tau_ab = sum_b d_b mu~ (g_ab + g_ba) - (2/3) d_a mu~ div
//                + mu~ [sum_b d_bb u_a + sum_b d_b(g_ba) - (2/3) sum_b d_a(g_bb)],
//     energy     = sum_ab g_ab tau_ab + sum_a u_a d_b tau_ab
//                + sum_b (d_b kappa d_b T + kappa d_bb T);
//   pure second derivatives (d_bb, and d_b(g_bb)) with the second-derivative
//   operator, mixed ones d_b(g_ba), a != b, as the first derivative of the
//   first derivative (outer index as written), d_b mu~ and d_b kappa as
//   first derivatives of their node values.
//
// Two storage strategies for the same arithmetic (section 6.1, "low memory
// intensity algorithms"):
//   StoreSome: in 3D nothing is stored between the state and the residual where
//     every stencil is centred (k_c_resid_zm); near non-periodic ends, on small
//     bounded grids (zm_pays), and in 1D and 2D, only the velocity gradients g_ab
//     are (one pointwise pass) and everything else is recomputed inside the
//     residual kernel;
//   store-all: every derivative goes to its own work array in its own pass
//     (flux derivatives, first derivatives of u, T, mu~, kappa, second and
//     mixed derivatives), and a pointwise pass assembles them, the practice
//     the paper compares against.
// Both store the residual; the pointwise finish kernel applies the RK update
// (a pass that reads neighbouring states cannot update the state in place), but
// for whole steps on fully periodic 3D grids, which go through copies of the
// state: there k_c_resid_zm updates.
#include <type_traits>

#include "point.hpp"
#include "stencil.hpp"

namespace osbli {
namespace {

// Node mapping of the central kernels: tiles of kBX x kBY columns, each
// taken plane by plane, numbered with the plane fastest; the linear block id
// b is remapped to item (b % 8) * per + b / 8, so each of the eight XCDs
// (one L2 each) walks one contiguous run of items and the blocks it holds at
// once cover neighbouring planes of the same tile: the z-neighbours of the
// five-point operators are read through that XCD's L2.
struct ColTiles {
    int tx, ty, nz, per, nt;
};

inline ColTiles col_tiles(const Grid &g) {
    ColTiles T;
    T.tx = (int)((g.n[0] + kBX - 1) / kBX);
    T.ty = (int)((g.n[1] + kBY - 1) / kBY);
    T.nz = (int)g.n[2];
    T.nt = T.tx * T.ty * T.nz;
    T.per = (T.nt + 7) / 8;
    return T;
}

__device__ __forceinline__ bool node_of_col_thread(const Grid &g, const ColTiles &T, int64_t (&idx)[3]) {
    const int L = (int)(blockIdx.x % 8) * T.per + (int)(blockIdx.x / 8);
    if (L >= T.nt) return false;
    const int k = L % T.nz, t = L / T.nz;
    idx[0] = (int64_t)(t % T.tx) * kBX + threadIdx.x;
    idx[1] = (int64_t)(t / T.tx) * kBY + threadIdx.y;
    idx[2] = k;
    return idx[0] < g.n[0] && idx[1] < g.n[1];
}

// the five-node operator window of line position p: the nodes q0 .. q0 + 4
// and the row r of the operator (-1: the centred interior / periodic stencil,
// 0, 1: the closures at the start, 3, 4: those at the end)
struct Win {
    int64_t q0;
    int r;
};

__device__ __forceinline__ Win window(int64_t p, int64_t N, bool periodic) {
    if (periodic || (p >= 2 && p <= N - 3)) return Win{p - 2, -1};
    if (p < 2) return Win{0, (int)p};
    return Win{N - 5, (int)(p - (N - 5))};
}

// first derivative per unit index from the window values f[0..4]
__device__ __forceinline__ double d1w(const double (&f)[5], int r) {
    if (r < 0) return (2.0 / 3.0) * (f[3] - f[1]) - (1.0 / 12.0) * (f[4] - f[0]);
    if (r == 0) return (-25.0 * f[0] + 48.0 * f[1] - 36.0 * f[2] + 16.0 * f[3] - 3.0 * f[4]) / 12.0;
    if (r == 1) return (-3.0 * f[0] - 10.0 * f[1] + 18.0 * f[2] - 6.0 * f[3] + f[4]) / 12.0;
    if (r == 3) return (-f[0] + 6.0 * f[1] - 18.0 * f[2] + 10.0 * f[3] + 3.0 * f[4]) / 12.0;
    return (3.0 * f[0] - 16.0 * f[1] + 36.0 * f[2] - 48.0 * f[3] + 25.0 * f[4]) / 12.0;
}

// second derivative per unit index from the window values, on differences
// from the centre (interior) or from the boundary node (closures)
__device__ __forceinline__ double d2w(const double (&f)[5], int r) {
    if (r < 0) {
        const double c = f[2];
        return (4.0 / 3.0) * ((f[3] - c) + (f[1] - c)) - (1.0 / 12.0) * ((f[4] - c) + (f[0] - c));
    }
    double d1, d2, d3, d4;
    if (r <= 1) {
        d1 = f[1] - f[0], d2 = f[2] - f[0], d3 = f[3] - f[0], d4 = f[4] - f[0];
    } else {
        d1 = f[3] - f[4], d2 = f[2] - f[4], d3 = f[1] - f[4], d4 = f[0] - f[4];
    }
    if (r == 0 || r == 4) return (-104.0 * d1 + 114.0 * d2 - 56.0 * d3 + 11.0 * d4) * (1.0 / 12.0);
    return (-20.0 * d1 + 6.0 * d2 + 4.0 * d3 - d4) * (1.0 / 12.0);
}

// node values of one extended node: the flux F_d along e_d (NC values) and
// the viscous primitives u_0..u_{ND-1}, T, mu~, kappa
template <int ND>
struct CNode {
    double F[ND + 2];
    double v[ND + 3];
};

template <int ND, bool VISC>
__device__ __forceinline__ void cnode(const double *__restrict__ U, int64_t e, int64_t cs, const Phys &ph, int d,
                                      CNode<ND> &o) {
    constexpr int NC = ND + 2;
    double q[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) q[c] = U[e + c * cs];
    const double ri = rcp64(q[0]);
    double ke = 0.0;
#pragma unroll
    for (int m = 0; m < ND; ++m) ke += q[1 + m] * q[1 + m];
    const double p = ph.gm1 * (q[ND + 1] - 0.5 * ke * ri);
    const double un = q[1 + d] * ri;
    o.F[0] = q[1 + d];
#pragma unroll
    for (int m = 0; m < ND; ++m) o.F[1 + m] = q[1 + m] * un + (m == d ? p : 0.0);
    o.F[ND + 1] = (q[ND + 1] + p) * un;
    if (VISC) {
#pragma unroll
        for (int m = 0; m < ND; ++m) o.v[m] = q[1 + m] * ri;
        const double T = ph.gamma * ph.M2 * p * ri;
        const double mu = viscosity(ph, T);
        o.v[ND] = T;
        o.v[ND + 1] = mu * ph.mu_re;
        o.v[ND + 2] = mu * ph.kheat;
    }
}

// velocity primitives only (gradient pass)
template <int ND>
__device__ __forceinline__ void cvel(const double *__restrict__ U, int64_t e, int64_t cs, double (&u)[ND]) {
    const double ri = rcp64(U[e]);
#pragma unroll
    for (int m = 0; m < ND; ++m) u[m] = U[e + (1 + m) * cs] * ri;
}

// the five window nodes of direction d around interior node idx (extended
// indices: the periodic stencil reads the ghost copies)
template <int ND>
__device__ __forceinline__ void window_ext(const Grid &g, const int64_t (&idx)[3], int d, Win &w, int64_t (&e)[5]) {
    const int64_t p = idx[d];
    w = window(p, g.n[d], g.periodic[d] != 0);
    const int64_t e0 = ext_index(g, idx[0], idx[1], idx[2]);
#pragma unroll
    for (int k = 0; k < 5; ++k) e[k] = e0 + (w.q0 + k - p) * g.es[d];
}

// the five window nodes of direction d in the interior layout (periodic:
// wrapped indices)
__device__ __forceinline__ void window_int(const Grid &g, const int64_t (&idx)[3], int d, Win &w, int64_t (&ci)[5]) {
    const int64_t p = idx[d], N = g.n[d];
    w = window(p, N, g.periodic[d] != 0);
    const int64_t c0 = int_index(g, idx[0], idx[1], idx[2]) - p * g.is[d];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        int64_t q = w.q0 + k;
        q = q < 0 ? q + N : (q >= N ? q - N : q);
        ci[k] = c0 + q * g.is[d];
    }
}

// whether every stencil of a node is the centred one
__device__ __forceinline__ bool centred(const Grid &g, int64_t x, int64_t y, int64_t z) {
    return (g.periodic[0] || (x >= 2 && x <= g.n[0] - 3)) && (g.periodic[1] || (y >= 2 && y <= g.n[1] - 3)) &&
           (g.periodic[2] || (z >= 2 && z <= g.n[2] - 3));
}

// ---------------------------------------------------------------- StoreSome
// pass 1: velocity gradients g_ab = (1/h_b) D_b u_a, stored [(a ND + b)][node]
// (ends: only near non-periodic ends, the nodes whose gradients the second pass
// reads for the nodes that the z-marching pass leaves out: its windows there
// stay within five nodes of the end)
template <int ND>
__global__ void __launch_bounds__(256) k_c_grad(const double *__restrict__ U, double *__restrict__ Gs, Grid g,
                                                Metrics m, ColTiles T, int ends) {
    int64_t idx[3];
    if (!node_of_col_thread(g, T, idx)) return;
    if (ends) {
        bool near = false;
#pragma unroll
        for (int d = 0; d < ND; ++d) near |= !g.periodic[d] && (idx[d] < 5 || idx[d] >= g.n[d] - 5);
        if (!near) return;
    }
    const int64_t ci = int_index(g, idx[0], idx[1], idx[2]);
    const int64_t cs = g.enpts;
#pragma unroll
    for (int b = 0; b < ND; ++b) {
        Win w;
        int64_t e[5];
        window_ext<ND>(g, idx, b, w, e);
        double f[ND][5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            double u[ND];
            cvel<ND>(U, e[k], cs, u);
#pragma unroll
            for (int a = 0; a < ND; ++a) f[a][k] = u[a];
        }
        const double ih = m.invh[b][idx[b]];
#pragma unroll
        for (int a = 0; a < ND; ++a) Gs[(a * ND + b) * g.nint + ci] = ih * d1w(f[a], w.r);
    }
}

// the expanded viscous terms of one node from its derivatives
template <int ND>
struct VTerms {
    double G[ND][ND];    // g_ab
    double dT[ND], dmu[ND], dka[ND];
    double s2u[ND][ND];  // d_bb u_a
    double s2T[ND];      // d_bb T
    double X[ND][ND];    // d_b(g_ba), a != b
    double Y[ND][ND];    // d_a(g_bb), a != b
    double u[ND], mu, ka;
};

template <int ND>
__device__ __forceinline__ void visc_assemble(const VTerms<ND> &t, double (&R)[ND + 2]) {
    double div = 0.0;
#pragma unroll
    for (int a = 0; a < ND; ++a) div += t.G[a][a];
    double work = 0.0;
#pragma unroll
    for (int a = 0; a < ND; ++a) {
        double first = -(2.0 / 3.0) * t.dmu[a] * div, second = 0.0;
#pragma unroll
        for (int b = 0; b < ND; ++b) {
            first += t.dmu[b] * (t.G[a][b] + t.G[b][a]);
            second += t.s2u[a][b];
            second += a == b ? t.s2u[b][b] : t.X[a][b];
            second -= (2.0 / 3.0) * (a == b ? t.s2u[b][a] : t.Y[a][b]);
        }
        const double dtau = first + t.mu * second;
#pragma unroll
        for (int b = 0; b < ND; ++b) {
            const double tau = t.mu * (t.G[a][b] + t.G[b][a] - (a == b ? (2.0 / 3.0) * div : 0.0));
            work += t.G[a][b] * tau;
        }
        work += t.u[a] * dtau;
        R[1 + a] += dtau;
    }
    double heat = 0.0;
#pragma unroll
    for (int b = 0; b < ND; ++b) heat += t.dka[b] * t.dT[b] + t.ka * t.s2T[b];
    R[ND + 1] += work + heat;
}

// pass 2 (ends: the nodes that the z-marching pass leaves out): convection and
// the viscous terms from the stored velocity gradients
// and everything recomputed locally, stored as the residual (the state is
// not updated here: neighbouring nodes still read it)
template <int ND, bool VISC>
__global__ void __launch_bounds__(256)
k_c_resid(const double *__restrict__ U, const double *__restrict__ Gs, Grid g, Phys ph, Metrics m,
          double *__restrict__ Rout, ColTiles T, int ends) {
    constexpr int NC = ND + 2;
    int64_t idx[3];
    if (!node_of_col_thread(g, T, idx)) return;
    if (ends && centred(g, idx[0], idx[1], idx[2])) return;
    const int64_t ci = int_index(g, idx[0], idx[1], idx[2]);
    const int64_t cs = g.enpts;
    double R[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) R[c] = 0.0;
    VTerms<ND> t;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        Win w;
        int64_t e[5];
        window_ext<ND>(g, idx, d, w, e);
        double F[NC][5], V[ND + 3][5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            CNode<ND> o;
            cnode<ND, VISC>(U, e[k], cs, ph, d, o);
#pragma unroll
            for (int c = 0; c < NC; ++c) F[c][k] = o.F[c];
            if (VISC) {
#pragma unroll
                for (int v = 0; v < ND + 3; ++v) V[v][k] = o.v[v];
            }
        }
        const double ih = m.invh[d][idx[d]];
#pragma unroll
        for (int c = 0; c < NC; ++c) R[c] -= ih * d1w(F[c], w.r);
        if (VISC) {
            const double ih2 = ih * ih;
            t.dT[d] = ih * d1w(V[ND], w.r);
            t.dmu[d] = ih * d1w(V[ND + 1], w.r);
            t.dka[d] = ih * d1w(V[ND + 2], w.r);
#pragma unroll
            for (int a = 0; a < ND; ++a) t.s2u[a][d] = ih2 * d2w(V[a], w.r);
            t.s2T[d] = ih2 * d2w(V[ND], w.r);
            if (d == 0) {
                // the node itself sits at window row p - q0
                const int rc = (int)(idx[0] - w.q0);
#pragma unroll
                for (int a = 0; a < ND; ++a) t.u[a] = V[a][rc];
                t.mu = V[ND + 1][rc];
                t.ka = V[ND + 2][rc];
            }
        }
    }
    if (VISC) {
#pragma unroll
        for (int a = 0; a < ND; ++a)
#pragma unroll
            for (int b = 0; b < ND; ++b) t.G[a][b] = Gs[(a * ND + b) * g.nint + ci];
#pragma unroll
        for (int b = 0; b < ND; ++b) {
            // along b: g_ba (a != b) for d_b(g_ba), and along b of g_aa for d_b(g_aa) = Y[b][a]
            Win w;
            int64_t cw[5];
            window_int(g, idx, b, w, cw);
            const double ih = m.invh[b][idx[b]];
#pragma unroll
            for (int a = 0; a < ND; ++a) {
                if (a == b) continue;
                double f[5], h[5];
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    f[k] = Gs[(b * ND + a) * g.nint + cw[k]];
                    h[k] = Gs[(a * ND + a) * g.nint + cw[k]];
                }
                t.X[a][b] = ih * d1w(f, w.r);
                t.Y[b][a] = ih * d1w(h, w.r);
            }
        }
        visc_assemble<ND>(t, R);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) Rout[c * g.nint + ci] = R[c];
}

// ---------------------------------------------------------------- 3D, z-marching
// The residual in one pass from the state alone, for nodes whose stencils are
// all centred (periodic directions, or two nodes from an end).  There the
// mixed derivatives commute, d_b(g_ba) = d_a(g_bb), so the twelve that the
// expanded form asks for are six, and none needs stored gradients: d_x d_y
// comes from the plane, d_x d_z and d_y d_z as the z derivative of in-plane
// gradients that each column keeps for five planes.
// A block owns a kCX x kCY tile of columns and marches zrun planes; a node's
// primitives are computed once, into an LDS ring of three planes with a
// two-node halo (72 KB: two blocks per CU, so that one works at the other's
// barriers; with Sutherland's law 81 KB and one), from where its x and y
// neighbours read them; the z neighbours' are a register window.  Bytes: read U,
// write the residual, 80 a node.  The node-per-thread passes (gradients stored,
// every node's primitives computed fifteen times, 75 values fetched per node
// through the caches) took 1.17 + 0.36 ms at 192^3, this one 0.29 ms (with
// Sutherland's law, which cost them no more, 0.38).  Nodes near a non-periodic end
// are left to those passes.
constexpr int kCX = 32, kCY = 8, kCHX = kCX + 4, kCHY = kCY + 4;
constexpr int kCHalo = 4 * kCHX + 4 * kCY;
static_assert(kCHalo <= kCX * kCY, "one halo position per thread");
constexpr int kCZ = 64;       // the longest run of planes
// blocks that run at a time.  Runs planned for two blocks per CU with Sutherland's
// law, which has one: 48^3 23 us, 15 as planned now; 96^3 54 and 44; 128^3 102 and
// 89; from 192^3 on alike.
constexpr int c_slots(bool suth) { return suth ? 256 : 512; }

struct ZTiles {
    int tx, ty, nt, per, zrun;
};

inline ZTiles z_tiles(const Grid &g, bool suth) {
    ZTiles T;
    T.tx = (int)((g.n[0] + kCX - 1) / kCX);
    T.ty = (int)((g.n[1] + kCY - 1) / kCY);
    T.zrun = plane_run((int64_t)T.tx * T.ty, g.n[2], kCZ, c_slots(suth));
    T.nt = T.tx * T.ty * (int)((g.n[2] + T.zrun - 1) / T.zrun);
    T.per = (T.nt + kXcds - 1) / kXcds;
    return T;
}

__device__ __forceinline__ double d1c(double m2, double m1, double p1, double p2) {
    return (2.0 / 3.0) * (p1 - m1) - (1.0 / 12.0) * (p2 - m2);
}
__device__ __forceinline__ double d2c(double m2, double m1, double c, double p1, double p2) {
    return (4.0 / 3.0) * ((p1 - c) + (m1 - c)) - (1.0 / 12.0) * ((p2 - c) + (m2 - c));
}

// what a node gives its neighbours' stencils: rho, u, v, w, p, rho E + p, T and
// (Sutherland) mu
constexpr int kCV = 8;
template <bool VISC, bool SUTH>
__device__ __forceinline__ void cprim(const double (&u)[5], const Phys &ph, double (&o)[kCV]) {
    const double ri = rcp64(u[0]);
    double ke = 0.0;
    o[0] = u[0];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[1 + a] = u[1 + a] * ri;
        ke += u[1 + a] * u[1 + a];
    }
    const double p = ph.gm1 * (u[4] - 0.5 * ke * ri);
    o[4] = p;
    o[5] = u[4] + p;
    o[6] = VISC ? ph.gamma * ph.M2 * p * ri : 0.0;
    o[7] = SUTH ? viscosity(ph, o[6]) : 1.0;
}

// STEP: the node's Runge-Kutta update instead of its residual, into another
// copy of the state (Rout: that copy): 0.40 ms at 192^3, the residual and the
// pointwise finish 0.29 + 0.21 (Sutherland's law 0.49).  With constant viscosity it
// spills 17 registers (the residual form 10) to have two blocks on a CU.
template <bool VISC, bool SUTH, bool STEP>
__global__ void __launch_bounds__(kCX * kCY, c_slots(SUTH) / 256)
k_c_resid_zm(const double *__restrict__ U, Grid g, Phys ph, Metrics m, double *__restrict__ Rout, ZTiles T,
             double *__restrict__ dU, RkStage rs, double dt) {
    constexpr int NV = !VISC ? 6 : (SUTH ? 8 : 7);  // values that neighbours read
    __shared__ double ring[3][NV][kCHY][kCHX];
    const int L = (int)(blockIdx.x % kXcds) * T.per + (int)(blockIdx.x / kXcds);
    if (L >= T.nt) return;  // block-uniform
    const int bx = L % T.tx, by = (L / T.tx) % T.ty, bz = L / (T.tx * T.ty);
    const int64_t Nx = g.n[0], Ny = g.n[1];
    const int64_t x0 = (int64_t)bx * kCX, y0 = (int64_t)by * kCY, x = x0 + threadIdx.x, y = y0 + threadIdx.y;
    const int64_t z0 = (int64_t)bz * T.zrun, z1 = z0 + T.zrun < g.n[2] ? z0 + T.zrun : g.n[2];
    const bool own = x < Nx && y < Ny;
    // columns beyond the grid hold its last ghost nodes: such values reach only
    // unused stencil slots
    const int64_t ecol = ext_index(g, x < Nx + 2 ? x : Nx + 2, y < Ny + 2 ? y : Ny + 2, 0);
    // the thread's halo position: two rows above and below the tile, two columns
    // either side
    const int h = threadIdx.y * kCX + threadIdx.x;
    const bool hal = h < kCHalo;
    int hx = 0, hy = 0;
    if (h < 4 * kCHX) {
        const int r = h / kCHX;
        hx = h - r * kCHX;
        hy = r < 2 ? r : kCY + r;
    } else if (hal) {
        const int r = h - 4 * kCHX, s = r & 3;
        hy = 2 + (r >> 2);
        hx = s < 2 ? s : kCX + s;
    }
    const int64_t gx = x0 - 2 + hx, gy = y0 - 2 + hy;
    const int64_t hcol = hal ? ext_index(g, gx > Nx + 2 ? Nx + 2 : gx, gy > Ny + 2 ? Ny + 2 : gy, 0) : ecol;
    const int64_t cs = g.enpts, sz = g.es[2], n = g.nint;
    auto load = [&](int64_t e, double (&u)[5]) {
#pragma unroll
        for (int c = 0; c < 5; ++c) u[c] = U[e + c * cs];
    };
    const double ihx = own ? m.invh[0][x] : 0.0, ihy = own ? m.invh[1][y] : 0.0;
    const int cx = threadIdx.x + 2, cy = threadIdx.y + 2;
    const int64_t col = x + y * g.is[1];
    // the column's values and its in-plane gradients d_x u, d_x w, d_y v, d_y w at
    // planes p-4 .. p of the plane p staged last; states of plane p + 1
    double w[5][kCV], gw[5][4], ou[5], hu[5];
    load(ecol + (z0 - 2) * sz, ou);
    load(hcol + (z0 - 2) * sz, hu);
    int slot = 0;  // ring slot of plane p; its centre plane p - 2 is in the slot after it
#pragma unroll 1
    for (int64_t p = z0 - 2; p < z1 + 2; ++p) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int v = 0; v < NV; ++v) w[k][v] = w[k + 1][v];
            if (VISC) {
#pragma unroll
                for (int v = 0; v < 4; ++v) gw[k][v] = gw[k + 1][v];
            }
        }
        cprim<VISC, SUTH>(ou, ph, w[4]);
        slot = slot == 2 ? 0 : slot + 1;
        __syncthreads();  // the slot's old plane is no longer read
        if (hal) {
            double f[kCV];
            cprim<VISC, SUTH>(hu, ph, f);
#pragma unroll
            for (int v = 0; v < NV; ++v) ring[slot][v][hy][hx] = f[v];
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) ring[slot][v][cy][cx] = w[4][v];
        const int64_t pn = p + 1 < z1 + 2 ? p + 1 : p;  // at most the second ghost plane
        load(ecol + pn * sz, ou);
        load(hcol + pn * sz, hu);
        __syncthreads();
        if (VISC) {
            auto gx_of = [&](int v) {
                return ihx * d1c(ring[slot][v][cy][cx - 2], ring[slot][v][cy][cx - 1], ring[slot][v][cy][cx + 1],
                                 ring[slot][v][cy][cx + 2]);
            };
            auto gy_of = [&](int v) {
                return ihy * d1c(ring[slot][v][cy - 2][cx], ring[slot][v][cy - 1][cx], ring[slot][v][cy + 1][cx],
                                 ring[slot][v][cy + 2][cx]);
            };
            gw[4][0] = gx_of(1);
            gw[4][1] = gx_of(3);
            gw[4][2] = gy_of(2);
            gw[4][3] = gy_of(3);
        }
        const int64_t z = p - 2;
        if (z < z0 || !own || !centred(g, x, y, z)) continue;  // the barriers are above
        double(&P)[NV][kCHY][kCHX] = ring[slot == 2 ? 0 : slot + 1];
        double R[5], second[3] = {0.0, 0.0, 0.0}, dmu[3] = {0.0, 0.0, 0.0}, heat = 0.0;
#pragma unroll
        for (int c = 0; c < 5; ++c) R[c] = 0.0;
        const double mu = SUTH ? w[2][7] : 1.0;
        // one direction's terms from the four neighbours' values
        auto direction = [&](auto dc, const double (&f)[4][NV], double ih) {
            constexpr int d = decltype(dc)::value;
            double F[4][5];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double un = f[k][1 + d], md = f[k][0] * un;
                F[k][0] = md;
#pragma unroll
                for (int a = 0; a < 3; ++a) F[k][1 + a] = md * f[k][1 + a] + (a == d ? f[k][4] : 0.0);
                F[k][4] = f[k][5] * un;
            }
#pragma unroll
            for (int c = 0; c < 5; ++c) R[c] -= ih * d1c(F[0][c], F[1][c], F[2][c], F[3][c]);
            if (VISC) {
                const double ih2 = ih * ih;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    // d_dd u_a; along its own direction also the (1 - 2/3) d_aa u_a
                    const double s = ih2 * d2c(f[0][1 + a], f[1][1 + a], w[2][1 + a], f[2][1 + a], f[3][1 + a]);
                    second[a] += a == d ? (4.0 / 3.0) * s : s;
                }
                heat += (mu * ph.kheat) * (ih2 * d2c(f[0][6], f[1][6], w[2][6], f[2][6], f[3][6]));
                if constexpr (SUTH) {
                    const double dm = ih * d1c(f[0][7], f[1][7], f[2][7], f[3][7]);
                    dmu[d] = dm * ph.mu_re;
                    heat += (dm * ph.kheat) * (ih * d1c(f[0][6], f[1][6], f[2][6], f[3][6]));
                }
            }
        };
        {
            double f[4][NV];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k][v] = P[v][cy][cx + (k < 2 ? k - 2 : k - 1)];
            direction(std::integral_constant<int, 0>{}, f, ihx);
        }
        {
            double f[4][NV];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k][v] = P[v][cy + (k < 2 ? k - 2 : k - 1)][cx];
            direction(std::integral_constant<int, 1>{}, f, ihy);
        }
        const double ihz = uniform_at(m.invh[2], z);
        {
            double f[4][NV];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k][v] = w[k < 2 ? k : k + 1][v];
            direction(std::integral_constant<int, 2>{}, f, ihz);
        }
        if (VISC) {
            // (1/3) d_a d_b u_b, b != a, into component a: d_x d_y of u and v from
            // the plane, the others along z from the gradient window
            auto dxy = [&](int v) {
                double r[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int yy = cy + (k < 2 ? k - 2 : k - 1);
                    r[k] = d1c(P[v][yy][cx - 2], P[v][yy][cx - 1], P[v][yy][cx + 1], P[v][yy][cx + 2]);
                }
                return (ihx * ihy) * d1c(r[0], r[1], r[2], r[3]);
            };
            auto dz = [&](int v) { return ihz * d1c(gw[0][v], gw[1][v], gw[3][v], gw[4][v]); };
            second[0] += (1.0 / 3.0) * (dxy(2) + dz(1));
            second[1] += (1.0 / 3.0) * (dxy(1) + dz(3));
            second[2] += (1.0 / 3.0) * (dz(0) + dz(2));
            double G[3][3];
            G[0][0] = gw[2][0];
            G[0][1] = ihy * d1c(P[1][cy - 2][cx], P[1][cy - 1][cx], P[1][cy + 1][cx], P[1][cy + 2][cx]);
            G[1][0] = ihx * d1c(P[2][cy][cx - 2], P[2][cy][cx - 1], P[2][cy][cx + 1], P[2][cy][cx + 2]);
            G[1][1] = gw[2][2];
            G[2][0] = gw[2][1];
            G[2][1] = gw[2][3];
#pragma unroll
            for (int a = 0; a < 3; ++a) G[a][2] = ihz * d1c(w[0][1 + a], w[1][1 + a], w[3][1 + a], w[4][1 + a]);
            const double div = G[0][0] + G[1][1] + G[2][2], mt = mu * ph.mu_re;
            double work = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                double dtau = mt * second[a];
                if (SUTH) {
                    dtau -= (2.0 / 3.0) * dmu[a] * div;
#pragma unroll
                    for (int b = 0; b < 3; ++b) dtau += dmu[b] * (G[a][b] + G[b][a]);
                }
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    work += G[a][b] * (mt * (G[a][b] + G[b][a] - (a == b ? (2.0 / 3.0) * div : 0.0)));
                work += w[2][1 + a] * dtau;
                R[1 + a] += dtau;
            }
            R[4] += work + heat;
        }
        if (STEP) {
            const unsigned ci = 8u * (unsigned)col, e0 = 8u * (unsigned)ecol;
            const int64_t pd = z * g.is[2], ed = z * sz;
            // the residual is complete here: sunk into the branches below, its
            // operands stay live to the last of them and are spilled
#pragma unroll
            for (int c = 0; c < 5; ++c) asm volatile("" : "+v"(R[c]));
            double d0[5], u0[5];
#pragma unroll
            for (int c = 0; c < 5; ++c) d0[c] = rs.first ? 0.0 : at32(dU + (c * n + pd), ci);
#pragma unroll
            for (int c = 0; c < 5; ++c) u0[c] = at32(U + (c * cs + ed), e0);
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                const double du = (rs.first ? 0.0 : rs.A * d0[c]) + dt * R[c];
                if (!rs.last) at32(dU + (c * n + pd), ci) = du;
                at32(Rout + (c * cs + ed), e0) = u0[c] + rs.B * du;
            }
        } else {
            const int64_t ci = col + z * g.is[2];
#pragma unroll
            for (int c = 0; c < 5; ++c) Rout[c * n + ci] = R[c];
        }
    }
}

// ---------------------------------------------------------------- store-all
// Work arrays (interior layout, [array][node]):
//   F   ND * NC          (1/h_d) D_d F_d,c
//   G   (ND + 3) * ND    (1/h_b) D_b of u_a, T, mu~, kappa
//   S   (ND + 1) * ND    (1/h_b^2) D2_b of u_a, T
//   X   ND * ND          d_b(g_ba), a != b
//   Y   ND * ND          d_a(g_bb), a != b
struct CWork {
    double *F, *G, *S, *X, *Y;
};

template <int ND, bool VISC>
__global__ void __launch_bounds__(256)
k_cb_first(const double *__restrict__ U, CWork W, Grid g, Phys ph, Metrics m, ColTiles T) {
    constexpr int NC = ND + 2;
    int64_t idx[3];
    if (!node_of_col_thread(g, T, idx)) return;
    const int64_t ci = int_index(g, idx[0], idx[1], idx[2]);
    const int64_t cs = g.enpts;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        Win w;
        int64_t e[5];
        window_ext<ND>(g, idx, d, w, e);
        double F[NC][5], V[ND + 3][5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            CNode<ND> o;
            cnode<ND, VISC>(U, e[k], cs, ph, d, o);
#pragma unroll
            for (int c = 0; c < NC; ++c) F[c][k] = o.F[c];
            if (VISC) {
#pragma unroll
                for (int v = 0; v < ND + 3; ++v) V[v][k] = o.v[v];
            }
        }
        const double ih = m.invh[d][idx[d]];
#pragma unroll
        for (int c = 0; c < NC; ++c) W.F[(d * NC + c) * g.nint + ci] = ih * d1w(F[c], w.r);
        if (VISC) {
#pragma unroll
            for (int v = 0; v < ND + 3; ++v) W.G[(v * ND + d) * g.nint + ci] = ih * d1w(V[v], w.r);
        }
    }
}

template <int ND>
__global__ void __launch_bounds__(256)
k_cb_second(const double *__restrict__ U, CWork W, Grid g, Phys ph, Metrics m, ColTiles T) {
    int64_t idx[3];
    if (!node_of_col_thread(g, T, idx)) return;
    const int64_t ci = int_index(g, idx[0], idx[1], idx[2]);
    const int64_t cs = g.enpts;
#pragma unroll
    for (int b = 0; b < ND; ++b) {
        Win w;
        int64_t e[5];
        window_ext<ND>(g, idx, b, w, e);
        double V[ND + 1][5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            CNode<ND> o;
            cnode<ND, true>(U, e[k], cs, ph, b, o);
#pragma unroll
            for (int v = 0; v < ND + 1; ++v) V[v][k] = o.v[v];
        }
        const double ih = m.invh[b][idx[b]];
#pragma unroll
        for (int v = 0; v < ND + 1; ++v) W.S[(v * ND + b) * g.nint + ci] = ih * ih * d2w(V[v], w.r);
        Win wi;
        int64_t cw[5];
        window_int(g, idx, b, wi, cw);
#pragma unroll
        for (int a = 0; a < ND; ++a) {
            if (a == b) continue;
            double f[5], h[5];
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                f[k] = W.G[(b * ND + a) * g.nint + cw[k]];   // g_ba along b
                h[k] = W.G[(a * ND + a) * g.nint + cw[k]];   // g_aa along b
            }
            W.X[(a * ND + b) * g.nint + ci] = ih * d1w(f, wi.r);
            W.Y[(b * ND + a) * g.nint + ci] = ih * d1w(h, wi.r);
        }
    }
}

template <int ND, bool VISC>
__global__ void __launch_bounds__(256)
k_cb_assemble(const double *__restrict__ U, CWork W, Grid g, Phys ph, double *__restrict__ Rout, ColTiles T) {
    constexpr int NC = ND + 2;
    int64_t idx[3];
    if (!node_of_col_thread(g, T, idx)) return;
    const int64_t ci = int_index(g, idx[0], idx[1], idx[2]);
    const int64_t e0 = ext_index(g, idx[0], idx[1], idx[2]);
    double R[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        double s = 0.0;
#pragma unroll
        for (int d = 0; d < ND; ++d) s += W.F[(d * NC + c) * g.nint + ci];
        R[c] = -s;
    }
    if (VISC) {
        VTerms<ND> t;
        CNode<ND> o;
        cnode<ND, true>(U, e0, g.enpts, ph, 0, o);
#pragma unroll
        for (int a = 0; a < ND; ++a) t.u[a] = o.v[a];
        t.mu = o.v[ND + 1];
        t.ka = o.v[ND + 2];
#pragma unroll
        for (int a = 0; a < ND; ++a)
#pragma unroll
            for (int b = 0; b < ND; ++b) {
                t.G[a][b] = W.G[(a * ND + b) * g.nint + ci];
                t.s2u[a][b] = W.S[(a * ND + b) * g.nint + ci];
                t.X[a][b] = a == b ? 0.0 : W.X[(a * ND + b) * g.nint + ci];
                t.Y[a][b] = a == b ? 0.0 : W.Y[(a * ND + b) * g.nint + ci];
            }
#pragma unroll
        for (int b = 0; b < ND; ++b) {
            t.dT[b] = W.G[(ND * ND + b) * g.nint + ci];
            t.dmu[b] = W.G[((ND + 1) * ND + b) * g.nint + ci];
            t.dka[b] = W.G[((ND + 2) * ND + b) * g.nint + ci];
            t.s2T[b] = W.S[(ND * ND + b) * g.nint + ci];
        }
        visc_assemble<ND>(t, R);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) Rout[c * g.nint + ci] = R[c];
}

inline size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

// Whether the z-marching pass is worth its company near bounded ends.  There the
// node passes run too, and wherever a block of 64 x 4 nodes holds one such node
// they cost almost what they cost for all of it: ends in x take every block of a
// row of up to 128 nodes.  ends: the share of such blocks; lanes: the node
// passes' threads, which their time goes by (0.16 to 0.21 ns each, inviscid
// 0.05).  The march saves about the rest of that time less 0.3 of it, and its
// launch and the blocks that only look cost some 30 us (inviscid 10).  Residuals,
// both ways (march, node passes) in us: 32^3 bounded in x 43 and 24, in z 31 and
// 20; 64^3 in z 43 and 53, in y and z 59 and 52; 96^3 in x 248 and 202, in y 104
// and 182; 144^3 in x 594 and 774; inviscid 64^3 in z 22 and 16, 96^3 in y 37 and
// 54, 144^3 in x 165 and 146, 256^3 in x 688 and 822.
inline bool zm_pays(const Grid &g, bool visc) {
    if (g.periodic[0] && g.periodic[1] && g.periodic[2]) return true;
    const int64_t bx = (g.n[0] + kBX - 1) / kBX, by = (g.n[1] + kBY - 1) / kBY;
    auto inner = [&](int d, int64_t blocks, int64_t two) {
        return g.periodic[d] ? blocks : (blocks > two ? blocks - two : 0);
    };
    const double lanes = (double)(bx * kBX) * (double)g.n[1] * (double)g.n[2];
    const double ends = 1.0 - (double)(inner(0, bx, 2) * inner(1, by, 2) * inner(2, g.n[2], 4)) /
                                  ((double)(bx * by) * (double)g.n[2]);
    return visc ? lanes * (0.85 - ends) >= 2e5 : lanes * (0.64 - ends) >= 3e5;
}

template <bool VISC, bool STEP>
void launch_zm(const Grid &g, const Phys &ph, const Metrics &m, const double *U, double *out, double *dU, RkStage rs,
               double dt, hipStream_t s) {
    const bool suth = VISC && ph.sutherland;
    const ZTiles Z = z_tiles(g, suth);
    const dim3 zb((unsigned)(Z.per * kXcds)), zs(kCX, kCY);
    if (suth)
        hipLaunchKernelGGL((k_c_resid_zm<VISC, VISC, STEP>), zb, zs, 0, s, U, g, ph, m, out, Z, dU, rs, dt);
    else
        hipLaunchKernelGGL((k_c_resid_zm<VISC, false, STEP>), zb, zs, 0, s, U, g, ph, m, out, Z, dU, rs, dt);
}

template <int ND, bool VISC>
hipError_t central_nd(const Grid &g, const Phys &ph, const Metrics &m, const double *U, double *Gs, void *work,
                      double *R, hipStream_t s) {
    const ColTiles T = col_tiles(g);
    const dim3 nb((unsigned)(8 * T.per)), bs(kBX, kBY);
    if (!work) {
        if constexpr (ND == 3)
            if (zm_pays(g, VISC)) {
                launch_zm<VISC, false>(g, ph, m, U, R, nullptr, RkStage{0.0, 0.0, 1, 1}, 0.0, s);
                if (!(g.periodic[0] && g.periodic[1] && g.periodic[2])) {
                    if (VISC) hipLaunchKernelGGL((k_c_grad<ND>), nb, bs, 0, s, U, Gs, g, m, T, 1);
                    hipLaunchKernelGGL((k_c_resid<ND, VISC>), nb, bs, 0, s, U, Gs, g, ph, m, R, T, 1);
                }
                return hipGetLastError();
            }
        if (VISC) hipLaunchKernelGGL((k_c_grad<ND>), nb, bs, 0, s, U, Gs, g, m, T, 0);
        hipLaunchKernelGGL((k_c_resid<ND, VISC>), nb, bs, 0, s, U, Gs, g, ph, m, R, T, 0);
        return hipGetLastError();
    }
    constexpr int NC = ND + 2;
    const size_t a = sizeof(double) * g.nint;
    char *w = static_cast<char *>(work);
    CWork W;
    W.F = reinterpret_cast<double *>(w);
    w += al256(a * ND * NC);
    W.G = reinterpret_cast<double *>(w);
    w += al256(a * (ND + 3) * ND);
    W.S = reinterpret_cast<double *>(w);
    w += al256(a * (ND + 1) * ND);
    W.X = reinterpret_cast<double *>(w);
    w += al256(a * ND * ND);
    W.Y = reinterpret_cast<double *>(w);
    hipLaunchKernelGGL((k_cb_first<ND, VISC>), nb, bs, 0, s, U, W, g, ph, m, T);
    if (VISC) hipLaunchKernelGGL((k_cb_second<ND>), nb, bs, 0, s, U, W, g, ph, m, T);
    hipLaunchKernelGGL((k_cb_assemble<ND, VISC>), nb, bs, 0, s, U, W, g, ph, R, T);
    return hipGetLastError();
}

}  // namespace

size_t central_work_bytes(const Grid &g, bool viscous) {
    const size_t a = sizeof(double) * g.nint;
    const int nd = g.nd, nc = g.nc;
    size_t b = al256(a * nd * nc);
    if (viscous) b += al256(a * (nd + 3) * nd) + al256(a * (nd + 1) * nd) + 2 * al256(a * nd * nd);
    return b;
}

hipError_t launch_central(const Grid &g, const Phys &ph, const Metrics &m, const double *U, double *Gs, void *work,
                          double *R, hipStream_t s) {
    const bool v = ph.viscous != 0;
    switch (g.nd) {
        case 1: return v ? central_nd<1, true>(g, ph, m, U, Gs, work, R, s) : central_nd<1, false>(g, ph, m, U, Gs, work, R, s);
        case 2: return v ? central_nd<2, true>(g, ph, m, U, Gs, work, R, s) : central_nd<2, false>(g, ph, m, U, Gs, work, R, s);
        default: return v ? central_nd<3, true>(g, ph, m, U, Gs, work, R, s) : central_nd<3, false>(g, ph, m, U, Gs, work, R, s);
    }
}

hipError_t launch_central_step(const Grid &g, const Phys &ph, const Metrics &m, const double *Uin, double *Uout,
                               double *dU, RkStage rs, double dt, hipStream_t s) {
    if (ph.viscous) launch_zm<true, true>(g, ph, m, Uin, Uout, dU, rs, dt, s);
    else launch_zm<false, true>(g, ph, m, Uin, Uout, dU, rs, dt, s);
    return hipGetLastError();
}

}  // namespace osbli
