// One Runge-Kutta stage of an inviscid 1D or 2D problem in one pass: the
// convective fluxes of every direction, the 2N update and the boundary
// conditions, from one copy of the state into another (shared by the
// single-grid and the batched launches).
//
// A pass of its own per sweep, update and ghost direction costs a small grid
// its launches (18 a step) and a large one its traffic (320 bytes per point
// and stage in 2D, where 128 are needed); and the marching y sweep of a
// 256 x 256 grid is 128 waves of nine serial fluxes.  Here a block owns a tile
// of nodes, finishes its points once into LDS (three-node halo), evaluates
// the interfaces of x and then of y one per lane, and takes each node's flux
// differences, its update and its ghost copies from LDS.  A block reads nodes
// that its neighbours own, so the new state goes to another buffer.
//
// Tiles of at most 32 x 7 nodes: 33 x 7 interfaces along x and 32 x 8 along y,
// one per thread in either direction (1.09 times the interfaces of a whole
// grid, 1.14 times the lanes); 36 KB of LDS and 168 registers, so three blocks
// per CU.  Tall tiles repeat fewer interfaces but leave waves idle: per stage
// of 1024 x 1024, 512 x 512 and 256 x 256 seven rows take 81, 31 and 18 us,
// eleven (six wave tasks on four waves) 92, 34 and 21, fifteen (eight tasks
// on four waves, two blocks per CU) 96, 40 and 22, five 98, 36 and 17.
// Bound: FP64 VALU, as the sweeps.
#pragma once

#include "sweep.hpp"

namespace osbli {
namespace cf {

template <int ND>
struct StageTile {
    static constexpr int X = ND == 1 ? 255 : 32, Y = ND == 1 ? 1 : 7;  // largest tile
    static constexpr int HY = ND == 1 ? 0 : kGhost;                     // halo rows per side
    static constexpr int PX = X + 2 * kGhost, PY = Y + 2 * HY;
    static constexpr int F = ND == 1 ? X + 1 : X * (Y + 1);             // interface slots of one direction
    static_assert(ND == 1 || (X + 1) * Y <= F, "both directions fit the flux slots");
    static_assert(F <= 256, "one interface per thread and direction, one node per thread");
};

template <int ND>
struct StageLds {
    double pt[ND + 5][StageTile<ND>::PY * StageTile<ND>::PX];  // U[0..nc), 1/rho, p, a
    double fl[ND + 2][StageTile<ND>::F];
};

// ghost copies of line position q: ne positions from e0 on (periodic images,
// or the three extrapolated layers of a boundary node)
struct Images {
    int64_t e0;
    int ne;
};
__device__ __forceinline__ Images images_of(int64_t q, int64_t N, int kind0, int kind1) {
    if (kind0 == OSBLI_PERIODIC) {  // periodic directions hold at least six nodes: at most one image
        if (q < kGhost) return Images{q + N, 1};
        if (q >= N - kGhost) return Images{q - N, 1};
    } else {
        if (q == 0 && kind0 == OSBLI_EXTRAPOLATE) return Images{-kGhost, kGhost};
        if (q == N - 1 && kind1 == OSBLI_EXTRAPOLATE) return Images{N, kGhost};
    }
    return Images{0, 0};
}

// characteristic (or routed) flux of one interface along DIR of a separable
// mesh, from the point slots s0, s0 + st, .. of the tile
template <int ND, int DIR, int SCHEME, bool MIX, bool ROUTE, bool JOINT>
__device__ __forceinline__ void stage_flux(const StageLds<ND> &sm, int s0, int st, const Phys &ph, bool cheap,
                                           double (&F)[ND + 2]) {
    constexpr int NC = ND + 2, NT = ND - 1;
    Loc<ND> P[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int s = s0 + k * st;
        P[k].r = sm.pt[0][s];
        P[k].mn = sm.pt[1 + DIR][s];
        if (NT >= 1) P[k].mt[0] = sm.pt[1 + Axes<ND, DIR>::T1][s];
        P[k].E = sm.pt[ND + 1][s];
        P[k].ri = sm.pt[NC][s];
        P[k].p = sm.pt[NC + 1][s];
        P[k].a = sm.pt[NC + 2][s];
        P[k].hu = P[k].mn * (0.5 * P[k].ri);
    }
    double Fr, Fn, Ft[2], FE;
    if (ROUTE && cheap) {
        if (MIX) cheap_flux_mixed<ND>(P, ph, Fr, Fn, Ft, FE);
        else cheap_flux<ND>(P, ph, Fr, Fn, Ft, FE);
    } else {
        // routed forms: full flux in FP64 (as in the sweeps)
        if (MIX && !ROUTE) char_flux_mixed<ND, SCHEME>(P, ph, Fr, Fn, Ft, FE);
        else char_flux<ND, SCHEME, JOINT>(P, ph, Fr, Fn, Ft, FE);
    }
    F[0] = Fr;
    F[1 + DIR] = Fn;
    if (NT >= 1) F[1 + Axes<ND, DIR>::T1] = Ft[0];
    F[NC - 1] = FE;
}

// a node's flux difference over two slots; the product is rounded by itself
// (the empty asm keeps the compiler from contracting it into the sum over the
// directions), so that a stage gives the bits of the separate sweeps
template <int NC, class Lds>
__device__ __forceinline__ void flux_difference(const Lds &sm, int a, int b, double ih, double (&v)[NC]) {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        v[k] = -ih * (sm.fl[k][b] - sm.fl[k][a]);
        asm volatile("" : "+v"(v[k]));
    }
}

// The work of one block of 256 threads: the nodes [x0, x0 + nx) x [y0, y0 +
// ny), nx <= StageTile::X, ny <= StageTile::Y.  XJOINT: one cut test for both
// sides of a split along x, as the marching x sweep of rows under 64
// interfaces has it (the lanes-along-x sweep of longer rows tests per side),
// so that the bits are the sweeps'.  Block-uniform arguments; every thread
// calls it.
template <int ND, int SCHEME, bool MIX, bool ROUTE, bool XJOINT>
__device__ __forceinline__ void stage_tile(const double *__restrict__ Uin, double *__restrict__ Uout,
                                           double *__restrict__ dU, const Grid &g, const Phys &ph,
                                           const double *const (&invh)[3], const uint8_t *const (&mask)[3],
                                           const int (&bc)[3][2], const RkStage &rs, double dt, int64_t x0,
                                           int64_t y0, int nx, int ny, unsigned *flags, StageLds<ND> &sm) {
    using T = StageTile<ND>;
    constexpr int NC = ND + 2;
    constexpr int DY = ND == 1 ? 0 : 1;
    const int tid = threadIdx.x;
    const int64_t cs = g.enpts;
    bool bad = false;
    // points of the tile and its halo (no corners: no stencil reads them)
    const int wx = nx + 2 * kGhost, np = wx * (ny + 2 * T::HY);
    for (int e = tid; e < np; e += 256) {
        const int r = e / wx, c = e - r * wx;
        if (ND == 2 && (c < kGhost || c >= nx + kGhost) && (r < kGhost || r >= ny + kGhost)) continue;
        const int64_t src = ext_index(g, x0 - kGhost + c, y0 - T::HY + r, 0);
        Pt<ND> w;
#pragma unroll
        for (int k = 0; k < NC; ++k) w.U[k] = Uin[src + k * cs];
        finish_point<ND>(ph, w, bad);
        const int s = r * T::PX + c;
#pragma unroll
        for (int k = 0; k < NC; ++k) sm.pt[k][s] = w.U[k];
        sm.pt[NC][s] = w.ri;
        sm.pt[NC + 1][s] = w.p;
        sm.pt[NC + 2][s] = w.a;
    }
    __syncthreads();
    // interfaces outside the line count as smooth (as in the sweeps)
    auto routed = [&](const uint8_t *mk, int64_t at, int64_t st, int64_t p, int64_t N) {
        auto ml = [&](int o) { return (p + o < -1 || p + o > N - 1) ? true : mk[at + o * st] != 0; };
        return ml(0) && (ph.dilate < 1 || (ml(-1) && ml(1))) && (ph.dilate < 2 || (ml(-2) && ml(2)));
    };
    if (tid < (nx + 1) * ny) {
        const int r = tid / (nx + 1), c = tid - r * (nx + 1);
        bool cheap = false;
        if (ROUTE) {
            const int64_t p = x0 + c - 1;
            cheap = routed(mask[0], (y0 + r) * (g.n[0] + 1) + p + 1, 1, p, g.n[0]);
        }
        double F[NC];
        stage_flux<ND, 0, SCHEME, MIX, ROUTE, XJOINT>(sm, (r + T::HY) * T::PX + c, 1, ph, cheap, F);
#pragma unroll
        for (int k = 0; k < NC; ++k) sm.fl[k][tid] = F[k];
    }
    __syncthreads();
    // the thread's node: its x flux difference, then the flux slots are free
    const int r = tid / nx, c = tid - r * nx;
    const int64_t x = x0 + c, y = y0 + r;
    double R[NC];
    if (r < ny) {
        const int f = r * (nx + 1) + c;
        flux_difference<NC>(sm, f, f + 1, invh[0][x], R);
    }
    if constexpr (ND == 2) {
        __syncthreads();
        if (r <= ny) {
            bool cheap = false;
            if (ROUTE) {
                const int64_t p = y - 1;
                cheap = routed(mask[1], y * g.n[0] + x, g.n[0], p, g.n[1]);
            }
            double F[NC];
            stage_flux<ND, DY, SCHEME, MIX, ROUTE, true>(sm, r * T::PX + c + kGhost, T::PX, ph, cheap, F);
#pragma unroll
            for (int k = 0; k < NC; ++k) sm.fl[k][tid] = F[k];
        }
        __syncthreads();
    }
    if (r < ny) {
        if constexpr (ND == 2) {
            double v[NC];
            flux_difference<NC>(sm, tid, tid + nx, invh[1][y], v);
#pragma unroll
            for (int k = 0; k < NC; ++k) R[k] += v[k];
        }
        const int64_t ci = int_index(g, x, y, 0);
        const int s = (r + T::HY) * T::PX + c + kGhost;
        double u[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const double du = (rs.first ? 0.0 : rs.A * dU[k * g.nint + ci]) + dt * R[k];
            if (!rs.last) dU[k * g.nint + ci] = du;
            u[k] = sm.pt[k][s] + rs.B * du;
        }
        auto put = [&](int64_t px, int64_t py) {
            const int64_t o = ext_index(g, px, py, 0);
#pragma unroll
            for (int k = 0; k < NC; ++k) Uout[o + k * cs] = u[k];
        };
        const Images ix = images_of(x, g.n[0], bc[0][0], bc[0][1]);
        const Images iy = ND == 2 ? images_of(y, g.n[1], bc[1][0], bc[1][1]) : Images{0, 0};
        put(x, y);
        for (int a = 0; a < ix.ne; ++a) put(ix.e0 + a, y);
        for (int b = 0; b < iy.ne; ++b) {
            put(x, iy.e0 + b);
            for (int a = 0; a < ix.ne; ++a) put(ix.e0 + a, iy.e0 + b);
        }
    }
    if (bad) atomicOr(flags, kFlagNonPhys);
}

}  // namespace cf

constexpr int kStageSlots = 3;  // tiles per CU

// Tiling of one grid: nx x ny tiles of at most tx x ty nodes, split evenly.
struct StageTiles {
    int tx, ty;
    int64_t nx, ny;
};

inline StageTiles stage_tiles(const Grid &g) {
    const bool one = g.nd == 1;
    const int mx = one ? cf::StageTile<1>::X : cf::StageTile<2>::X, my = one ? 1 : cf::StageTile<2>::Y;
    StageTiles t;
    t.nx = (g.n[0] + mx - 1) / mx;
    t.tx = (int)((g.n[0] + t.nx - 1) / t.nx);
    t.nx = (g.n[0] + t.tx - 1) / t.tx;
    t.ny = (g.n[1] + my - 1) / my;
    t.ty = (int)((g.n[1] + t.ny - 1) / t.ny);
    t.ny = (g.n[1] + t.ty - 1) / t.ty;
    return t;
}

}  // namespace osbli
