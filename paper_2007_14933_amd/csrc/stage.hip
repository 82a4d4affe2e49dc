// Single-grid launches of the one-pass Runge-Kutta stage (stage.hpp):
// inviscid 1D and 2D problems on separable meshes with periodic or
// extrapolated ends, the schemes with six-point stencils.
#include "stage.hpp"

namespace osbli {
namespace {
using namespace cf;

struct StageArgs {
    const double *invh[3];
    const uint8_t *mask[3];
    int bc[3][2];
};

// tiles are numbered x fastest and placed as one contiguous run per XCD, so
// that neighbouring tiles read their halos through one L2
template <int ND, int SCHEME, bool MIX, bool ROUTE, bool XS>
__global__ void __launch_bounds__(256, kStageSlots)
k_stage(const double *__restrict__ Uin, double *__restrict__ Uout, double *__restrict__ dU, Grid g, Phys ph,
        StageArgs a, RkStage rs, double dt, int tx, int ty, int nx, int ntiles, int per, unsigned *flags) {
    __shared__ StageLds<ND> sm;
    const int L = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (L >= ntiles) return;  // block-uniform
    const int by = L / nx, bx = L - by * nx;
    const int64_t x0 = (int64_t)bx * tx, y0 = (int64_t)by * ty;
    const int wx = (int)(g.n[0] - x0 < tx ? g.n[0] - x0 : tx), wy = (int)(g.n[1] - y0 < ty ? g.n[1] - y0 : ty);
    stage_tile<ND, SCHEME, MIX, ROUTE, XS>(Uin, Uout, dU, g, ph, a.invh, a.mask, a.bc, rs, dt, x0, y0, wx, wy, flags,
                                       sm);
}

template <int ND, int SCHEME, bool MIX, bool ROUTE, bool XS>
hipError_t launch_one(const Grid &g, const Phys &ph, const StageArgs &a, const double *Uin, double *Uout, double *dU,
                      const RkStage &rs, double dt, unsigned *flags, hipStream_t s) {
    const StageTiles t = stage_tiles(g);
    const int nt = (int)(t.nx * t.ny), per = (nt + 7) / 8;
    hipLaunchKernelGGL((k_stage<ND, SCHEME, MIX, ROUTE, XS>), dim3((unsigned)(8 * per)), dim3(256), 0, s, Uin, Uout, dU,
                       g, ph, a, rs, dt, t.tx, t.ty, (int)t.nx, nt, per, flags);
    return hipGetLastError();
}

template <int SCHEME, bool MIX, bool ROUTE>
hipError_t launch_nd(const Grid &g, const Phys &ph, const StageArgs &a, const double *Uin, double *Uout, double *dU,
                     const RkStage &rs, double dt, unsigned *flags, hipStream_t s) {
    // the other schemes reconstruct side by side everywhere
    if constexpr (SCHEME == OSBLI_WENOZ5 || SCHEME == OSBLI_TENO5)
        if (g.n[0] + 1 < 64)
            return g.nd == 1 ? launch_one<1, SCHEME, MIX, ROUTE, true>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s)
                             : launch_one<2, SCHEME, MIX, ROUTE, true>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s);
    return g.nd == 1 ? launch_one<1, SCHEME, MIX, ROUTE, false>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s)
                     : launch_one<2, SCHEME, MIX, ROUTE, false>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s);
}

}  // namespace

bool stage_supported(const Grid &g, const osbli_params &p) {
    if (g.nd > 2 || (p.mesh == OSBLI_MESH_GENERAL && g.nd == 2) || p.Re > 0.0) return false;
    if (p.scheme == OSBLI_CENTRAL4 || p.scheme == OSBLI_WENOZ7) return false;
    // the precision form without routing keeps the sweeps: its FP32 arithmetic
    // is contracted differently here, a change of 1e-7 of the state's jumps
    if (p.form == OSBLI_FORM_MIXED && !p.sensor) return false;
    // the pass needs a second and a third copy of the state: bounded
    if (g.nint > kStageMaxNodes) return false;
    for (int d = 0; d < g.nd; ++d)
        for (int s = 0; s < 2; ++s)
            if (p.bc_kind[d][s] != OSBLI_PERIODIC && p.bc_kind[d][s] != OSBLI_EXTRAPOLATE) return false;
    return true;
}

hipError_t launch_stage(const Grid &g, const Phys &ph, const Metrics &m, const osbli_params &p, const double *Uin,
                        double *Uout, double *dU, uint8_t *const mask[3], bool route, const RkStage &rs, double dt,
                        unsigned *flags, hipStream_t s) {
    StageArgs a;
    for (int d = 0; d < 3; ++d) {
        a.invh[d] = m.invh[d];
        a.mask[d] = mask[d];
        for (int k = 0; k < 2; ++k) a.bc[d][k] = p.bc_kind[d][k];
    }
    const bool mix = ph.mixed != 0;
    switch (ph.scheme) {
        case OSBLI_WENOZ5: return launch_nd<OSBLI_WENOZ5, false, false>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s);
        case OSBLI_TENO5:
            if (route)
                return mix ? launch_nd<OSBLI_TENO5, true, true>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s)
                           : launch_nd<OSBLI_TENO5, false, true>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s);
            return launch_nd<OSBLI_TENO5, false, false>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s);
        case OSBLI_TENO6: return launch_nd<OSBLI_TENO6, false, false>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s);
        case OSBLI_WENOJS5: return launch_nd<OSBLI_WENOJS5, false, false>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s);
        case OSBLI_WENOZ3: return launch_nd<OSBLI_WENOZ3, false, false>(g, ph, a, Uin, Uout, dU, rs, dt, flags, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace osbli
