// Learned shock sensor (not in the paper; the paper names sensor-switched
// hybrids of central and shock-capturing fluxes as hard to design by hand):
//   - sensor features of an interface and the TENO "all stencils kept" label
//     (training data made by the method itself);
//   - a 10 -> 32 -> 32 -> 1 network (ReLU, ReLU, sigmoid) with bfloat16
//     weights: FP32 training forward / backward, a deterministic gradient
//     reduction and Adam on FP32 master weights;
//   - inference on the matrix cores (bf16 MFMA, FP32 accumulation), 64
//     interfaces per wave, producing per-interface routing masks.
#include "charflux.hpp"
#include "sensor.hpp"

namespace osbli {
namespace {
using namespace cf;
using namespace sn;

// features + label of every interface of direction DIR (TENO5 labels)
template <int ND, int DIR>
__global__ void __launch_bounds__(256)
k_labels(const double *__restrict__ U, Grid g, Phys ph, float *__restrict__ feat, uint8_t *__restrict__ lab) {
    const IfaceGrid I = iface_grid(g, DIR);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= I.total) return;
    int64_t q[3];
    q[0] = t % I.E[0];
    q[1] = (t / I.E[0]) % I.E[1];
    q[2] = t / (I.E[0] * I.E[1]);
    q[DIR] -= 1;  // interface position p in [-1, N-1]
    const int64_t st = g.es[DIR], cs = g.enpts;
    const int64_t e0 = ext_index(g, q[0], q[1], q[2]) - 2 * st;
    float f[kIn];
    features<ND, DIR>(U, e0, st, cs, ph, f);
#pragma unroll
    for (int m = 0; m < kIn; ++m) feat[t * kIn + m] = f[m];
    Loc<ND> P[6];
    constexpr int T1 = (DIR + 1) % ND, T2 = (DIR + 2) % ND;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        Pt<ND> w;
#pragma unroll
        for (int c = 0; c < ND + 2; ++c) w.U[c] = U[e0 + k * st + c * cs];
        bool bad = false;
        finish_point<ND>(ph, w, bad);
        P[k].r = w.U[0];
        P[k].mn = w.U[1 + DIR];
        P[k].mt[0] = ND >= 2 ? w.U[1 + T1] : 0.0;
        P[k].mt[1] = ND >= 3 ? w.U[1 + T2] : 0.0;
        P[k].E = w.U[ND + 1];
        P[k].p = w.p;
        P[k].a = w.a;
        P[k].ri = w.ri;
        P[k].hu = P[k].mn * (0.5 * w.ri);
    }
    bool kept = true;
    double Fr, Fn, Ft[2], FE;
    char_flux<ND, OSBLI_TENO5>(P, ph, Fr, Fn, Ft, FE, &kept);
    lab[t] = kept ? 1 : 0;
}

// ------------------------------------------------------ FP32 training pass
struct Fwd {
    float a1[kH], a2[kH], z;
};

__device__ __forceinline__ void fwd_fp32(const float (&x)[kIn], const float *W, Fwd &o) {
#pragma unroll
    for (int j = 0; j < kH; ++j) {
        float s = W[oB1 + j];
#pragma unroll
        for (int k = 0; k < kIn; ++k) s += x[k] * W[oW1 + k * kH + j];
        o.a1[j] = s;
    }
#pragma unroll
    for (int j = 0; j < kH; ++j) {
        float s = W[oB2 + j];
#pragma unroll
        for (int k = 0; k < kH; ++k) s += fmaxf(o.a1[k], 0.0f) * W[oW2 + k * kH + j];
        o.a2[j] = s;
    }
    float z = W[oB3];
#pragma unroll
    for (int j = 0; j < kH; ++j) z += fmaxf(o.a2[j], 0.0f) * W[oW3 + j];
    o.z = z;
}

// Gradient of the mean class-weighted BCE.  A training batch (512 samples) is
// far too small to fill the chip, so the pass is a latency chain and the work
// is spread as thin as the network allows: a block takes kMB = 16 samples with
// 16 threads each, two hidden units of every layer per thread (one wave per 64
// samples, each thread running a whole network, left 8 waves on the chip:
// 111 us per call on a batch of 512 with its reduction, this form 10 us).  Blocks stride over the sample
// tiles, at most kMaxBlk of them, so the partial records stay small.
// A sample's forward and backward values are one record in LDS; every entry
// of the gradient is the sum over the samples of a product of two record
// entries (biases and loss: with the constant 1), FP64 products and sums.
constexpr int kMB = 16;
constexpr int kMaxBlk = 1024;
constexpr int kW2S = kH + 1;  // LDS row stride of W2: rows and columns are read without bank conflicts
// record offsets: x, relu(a1), d1, relu(a2), d2, dz, loss term, 1
constexpr int rX = 0, rH1 = rX + kIn, rD1 = rH1 + kH, rH2 = rD1 + kH, rD2 = rH2 + kH, rDz = rD2 + kH, rL = rDz + 1,
              rOne = rL + 1, kRec = rOne + 1;
static_assert(kRec % 2 == 1, "odd record stride: the samples of a wave start in different banks");
constexpr int kPerThread = (kNPad + 255) / 256;

// the two record entries whose product, summed over the samples, is entry e of the gradient
__device__ __forceinline__ void grad_entry(int e, int &a, int &b) {
    if (e < oB1) a = rX + e / kH, b = rD1 + e % kH;
    else if (e < oW2) a = rOne, b = rD1 + e - oB1;
    else if (e < oB2) a = rH1 + (e - oW2) / kH, b = rD2 + (e - oW2) % kH;
    else if (e < oW3) a = rOne, b = rD2 + e - oB2;
    else if (e < oB3) a = rDz, b = rH2 + e - oW3;
    else a = rOne, b = e == oB3 ? rDz : rL;
}

__global__ void __launch_bounds__(256)
k_mlp_grad(const float *__restrict__ X, const uint8_t *__restrict__ y, int64_t n, const uint16_t *__restrict__ w,
           float wneg, float inv_n, double *__restrict__ partial) {
    __shared__ float W1[kIn * kH], W2[kH * kW2S], B1[kH], B2[kH], W3[kH];
    __shared__ float rec[kMB][kRec];
    const int tid = threadIdx.x;
    for (int e = tid; e < kIn * kH; e += 256) W1[e] = bf2f(w[oW1 + e]);
    for (int e = tid; e < kH * kH; e += 256) W2[(e / kH) * kW2S + e % kH] = bf2f(w[oW2 + e]);
    if (tid < kH) {
        B1[tid] = bf2f(w[oB1 + tid]);
        B2[tid] = bf2f(w[oB2 + tid]);
        W3[tid] = bf2f(w[oW3 + tid]);
    }
    const float b3 = bf2f(w[oB3]);
    int ea[kPerThread], eb[kPerThread];
    double acc[kPerThread];
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        const int e = tid + 256 * i;
        grad_entry(e < kNPad ? e : kNPad - 1, ea[i], eb[i]);
        acc[i] = 0.0;
    }
    __syncthreads();
    // sample sl of the tile, hidden units u and u + 16; a sample's sixteen
    // threads lie in one wave
    const int sl = tid >> 4, u = tid & 15;
    float *const r = rec[sl];
    for (int64_t s0 = (int64_t)blockIdx.x * kMB; s0 < n; s0 += (int64_t)gridDim.x * kMB) {
        const int64_t s = s0 + sl;
        const bool valid = s < n;
        if (u < kIn) r[rX + u] = valid ? X[s * kIn + u] : 0.0f;
        if (u == 15) r[rOne] = 1.0f;
        const float yv = valid ? (float)y[s] : 0.0f;
        wave_sync();
        float a1[2], a2[2], d2[2], g1[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            a1[h] = B1[u + 16 * h];
#pragma unroll
            for (int k = 0; k < kIn; ++k) a1[h] = fmaf(r[rX + k], W1[k * kH + u + 16 * h], a1[h]);
            r[rH1 + u + 16 * h] = fmaxf(a1[h], 0.0f);
        }
        wave_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            a2[h] = B2[u + 16 * h];
#pragma unroll
            for (int k = 0; k < kH; ++k) a2[h] = fmaf(r[rH1 + k], W2[k * kW2S + u + 16 * h], a2[h]);
        }
        float z = fmaxf(a2[0], 0.0f) * W3[u] + fmaxf(a2[1], 0.0f) * W3[u + 16];
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) z += __shfl_xor(z, off, 64);
        z += b3;
        const float wt = valid ? (yv > 0.5f ? 1.0f : wneg) : 0.0f;
        // sigmoid and the loss term in FP64 (float expf would carry its own
        // rounding into every gradient)
        const double zd = z, ex = exp(-fabs(zd));
        const double sig = (zd >= 0.0 ? 1.0 : ex) / (1.0 + ex);
        const float dz = (float)(wt * (sig - yv) * inv_n);
        if (u == 0) {
            r[rDz] = dz;
            r[rL] = (float)(wt * ((fmax(zd, 0.0) + log1p(ex)) - yv * zd) * inv_n);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            d2[h] = a2[h] > 0.0f ? dz * W3[u + 16 * h] : 0.0f;
            r[rD2 + u + 16 * h] = d2[h];
            r[rH2 + u + 16 * h] = fmaxf(a2[h], 0.0f);
        }
        wave_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            g1[h] = 0.0f;
#pragma unroll
            for (int j = 0; j < kH; ++j) g1[h] = fmaf(r[rD2 + j], W2[(u + 16 * h) * kW2S + j], g1[h]);
            r[rD1 + u + 16 * h] = a1[h] > 0.0f ? g1[h] : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < kMB; ++t)
#pragma unroll
            for (int i = 0; i < kPerThread; ++i) acc[i] = fma((double)rec[t][ea[i]], (double)rec[t][eb[i]], acc[i]);
        __syncthreads();
    }
    double *out = partial + (int64_t)blockIdx.x * kNPad;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
        if (tid + 256 * i < kNPad) out[tid + 256 * i] = acc[i];
}

// fixed-order sum of the block partials -> gradient (1441) and loss: 32
// entries per block, eight threads each over every eighth partial
__global__ void __launch_bounds__(256)
k_mlp_reduce(const double *__restrict__ partial, int nblk, float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ double part[8][32];
    const int el = threadIdx.x & 31, q = threadIdx.x >> 5;
    const int e = blockIdx.x * 32 + el;
    double acc = 0.0;
    if (e < kNPad)
#pragma unroll 4
        for (int b = q; b < nblk; b += 8) acc += partial[(int64_t)b * kNPad + e];
    part[q][el] = acc;
    __syncthreads();
    if (q != 0 || e >= kNPad) return;
#pragma unroll
    for (int k = 1; k < 8; ++k) acc += part[k][el];
    if (e < kNP) grad[e] = (float)acc;
    else if (loss) *loss = (float)acc;
}

__global__ void k_mlp_adam(float *__restrict__ master, uint16_t *__restrict__ w, const float *__restrict__ grad,
                           float *__restrict__ m, float *__restrict__ v, float lr, float b1, float b2, float eps,
                           float c1, float c2) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= kNP) return;
    const float g = grad[e];
    const float mm = b1 * m[e] + (1.0f - b1) * g;
    const float vv = b2 * v[e] + (1.0f - b2) * g * g;
    m[e] = mm;
    v[e] = vv;
    const float th = master[e] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    master[e] = th;
    w[e] = f2bf(th);
}

__global__ void k_mlp_fwd_fp32(const float *__restrict__ X, int64_t n, const uint16_t *__restrict__ w,
                               float *__restrict__ z) {
    __shared__ float W[kNP];
    for (int e = threadIdx.x; e < kNP; e += blockDim.x) W[e] = bf2f(w[e]);
    __syncthreads();
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    float x[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) x[k] = X[s * kIn + k];
    Fwd o;
    fwd_fp32(x, W, o);
    z[s] = o.z;
}

// ------------------------------------------------------ MFMA inference
__global__ void __launch_bounds__(256)
k_mlp_fwd_mfma(const float *__restrict__ X, int64_t n, const uint16_t *__restrict__ w, float *__restrict__ z) {
    const int lane = threadIdx.x & 63;
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t sc = s < n ? s : n - 1;
    float x[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) x[k] = X[sc * kIn + k];
    MlpFrag F;
    load_frag(w, lane, F);
    const float zz = mlp_mfma(x, F, lane);
    if (s < n) z[s] = zz;
}

// routing mask of every interface of direction DIR: 1 when the network's
// logit reaches zcut (P(smooth) >= threshold)
template <int ND, int DIR>
__global__ void __launch_bounds__(256)
k_sensor(const double *__restrict__ U, Grid g, Phys ph, const uint16_t *__restrict__ w, float zcut,
         uint8_t *__restrict__ mask) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    sensor_item<ND, DIR>(U, g, ph, w, zcut, mask, t);
}

template <int ND>
hipError_t labels_nd(const Grid &g, const Phys &ph, const double *U, int d, float *feat, uint8_t *lab,
                     hipStream_t s) {
    const IfaceGrid I = iface_grid(g, d);
    const unsigned nb = (unsigned)((I.total + 255) / 256);
    if (d == 0) hipLaunchKernelGGL((k_labels<ND, 0>), dim3(nb), dim3(256), 0, s, U, g, ph, feat, lab);
    else if (d == 1) hipLaunchKernelGGL((k_labels<ND, (ND >= 2 ? 1 : 0)>), dim3(nb), dim3(256), 0, s, U, g, ph, feat, lab);
    else hipLaunchKernelGGL((k_labels<ND, (ND >= 3 ? 2 : 0)>), dim3(nb), dim3(256), 0, s, U, g, ph, feat, lab);
    return hipGetLastError();
}

// y and z directions: each wave marches a segment of interfaces along 64
// neighbouring lines (sensor_line)
template <int ND, int DIR>
__global__ void __launch_bounds__(256)
k_sensor_line(const double *__restrict__ U, Grid g, Phys ph, const uint16_t *__restrict__ w, float zcut,
              uint8_t *__restrict__ mask, int64_t seg, int64_t nseg) {
    constexpr int O1 = DIR == 0 ? 1 : 0;
    constexpr int O2 = DIR == 2 ? 1 : 2;
    const int64_t lines = g.n[O1] * g.n[O2];
    const int64_t wpl = (lines + 63) >> 6;
    const int64_t gw = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t sg = gw / wpl;
    if (sg >= nseg) return;  // wave-uniform
    const int64_t line0 = (gw - sg * wpl) << 6;
    const int64_t NI = g.n[DIR] + 1;
    const int64_t iq0 = sg * seg, iq1 = iq0 + seg < NI ? iq0 + seg : NI;
    const int lane = threadIdx.x & 63;
    MlpFrag F;
    load_frag(w, lane, F);
    sensor_line<ND, DIR>(U, g, ph, F, zcut, mask, line0, iq0, iq1);
}

// x direction, rows of >= 64 interfaces: 64 interfaces per wave with the
// points staged once (sensor_x_lanes)
template <int ND>
__global__ void __launch_bounds__(256)
k_sensor_xl(const double *__restrict__ U, Grid g, Phys ph, const uint16_t *__restrict__ w, float zcut,
            uint8_t *__restrict__ mask, int64_t totalJ) {
    __shared__ SxLds<ND> sp[4];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t gw = (int64_t)blockIdx.x * (blockDim.x >> 6) + wv;
    const int64_t J0 = gw * 64;
    if (J0 >= totalJ) return;  // wave-uniform
    const int lane = threadIdx.x & 63;
    MlpFrag F;
    load_frag(w, lane, F);
    sensor_x_lanes<ND>(U, g, ph, F, zcut, mask, J0, totalJ, sp[wv]);
}

template <int ND>
hipError_t sensor_nd(const Grid &g, const Phys &ph, const double *U, int d, const uint16_t *w, float zcut,
                     uint8_t *mask, hipStream_t s) {
    const IfaceGrid I = iface_grid(g, d);
    if (d == 0 && g.n[0] + 1 >= 64) {
        const int64_t waves = (I.total + 63) / 64;
        const unsigned nb = (unsigned)((waves + 3) / 4);
        hipLaunchKernelGGL((k_sensor_xl<ND>), dim3(nb), dim3(256), 0, s, U, g, ph, w, zcut, mask, I.total);
        return hipGetLastError();
    }
    if (d == 0 || ND == 1) {
        const unsigned nb = (unsigned)((I.total + 255) / 256);
        hipLaunchKernelGGL((k_sensor<ND, 0>), dim3(nb), dim3(256), 0, s, U, g, ph, w, zcut, mask);
        return hipGetLastError();
    }
    const int o1 = 0, o2 = d == 2 ? 1 : 2;  // lines of the y and z directions run along x
    const int64_t lines = g.n[o1] * g.n[o2], NI = g.n[d] + 1;
    // about 2^19 lanes (the network's cost per interface does not shrink with
    // longer segments, so parallelism is worth more than the shared prologue)
    int64_t seg = (NI * lines + (int64_t(1) << 19) - 1) >> 19;
    seg = seg < 2 ? 2 : (seg > NI ? NI : seg);
    const int64_t nseg = (NI + seg - 1) / seg;
    const int64_t waves = ((lines + 63) / 64) * nseg;
    const unsigned nb = (unsigned)((waves + 3) / 4);
    if (d == 1)
        hipLaunchKernelGGL((k_sensor_line<ND, (ND >= 2 ? 1 : 0)>), dim3(nb), dim3(256), 0, s, U, g, ph, w, zcut, mask,
                           seg, nseg);
    else
        hipLaunchKernelGGL((k_sensor_line<ND, (ND >= 3 ? 2 : 0)>), dim3(nb), dim3(256), 0, s, U, g, ph, w, zcut, mask,
                           seg, nseg);
    return hipGetLastError();
}

// number of nonzero bytes (integer atomics: order independent)
__global__ void k_count_u8(const uint8_t *__restrict__ a, int64_t n, unsigned long long *out) {
    unsigned long long c = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        c += a[i] != 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(out, c);
}

}  // namespace

hipError_t launch_count_u8(const uint8_t *a, int64_t n, unsigned long long *out, hipStream_t s) {
    int64_t nb = (n + 255) / 256;
    if (nb > 1024) nb = 1024;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_count_u8, dim3((unsigned)nb), dim3(256), 0, s, a, n, out);
    return hipGetLastError();
}

int64_t iface_count(const Grid &g, int d) { return iface_grid(g, d).total; }

hipError_t launch_labels(const Grid &g, const Phys &ph, const double *U, int d, float *feat, uint8_t *lab,
                         hipStream_t s) {
    switch (g.nd) {
        case 1: return labels_nd<1>(g, ph, U, d, feat, lab, s);
        case 2: return labels_nd<2>(g, ph, U, d, feat, lab, s);
        default: return labels_nd<3>(g, ph, U, d, feat, lab, s);
    }
}

hipError_t launch_sensor(const Grid &g, const Phys &ph, const double *U, int d, const uint16_t *w, float zcut,
                         uint8_t *mask, hipStream_t s) {
    switch (g.nd) {
        case 1: return sensor_nd<1>(g, ph, U, d, w, zcut, mask, s);
        case 2: return sensor_nd<2>(g, ph, U, d, w, zcut, mask, s);
        default: return sensor_nd<3>(g, ph, U, d, w, zcut, mask, s);
    }
}

static int64_t mlp_blocks(int64_t n) {
    const int64_t tiles = (n + kMB - 1) / kMB;
    return tiles < kMaxBlk ? tiles : kMaxBlk;
}

// (eight bytes more than the records: the caller's buffer may be aligned to four)
size_t mlp_workspace_bytes(int64_t n) { return (size_t)mlp_blocks(n) * kNPad * sizeof(double) + sizeof(double); }

hipError_t launch_mlp_grad(const float *X, const uint8_t *y, int64_t n, const uint16_t *w, float wneg, float *grad,
                           float *loss, void *workspace, hipStream_t s) {
    const int64_t nblk = mlp_blocks(n);
    double *partial = reinterpret_cast<double *>((reinterpret_cast<uintptr_t>(workspace) + 7) & ~uintptr_t(7));
    hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)nblk), dim3(256), 0, s, X, y, n, w, wneg, 1.0f / (float)n, partial);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((kNPad + 31) / 32), dim3(256), 0, s, partial, (int)nblk, grad, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float *master, uint16_t *w, const float *grad, float *m, float *v, int64_t t, float lr,
                           float b1, float b2, float eps, hipStream_t s) {
    const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_mlp_adam, dim3((kNP + 255) / 256), dim3(256), 0, s, master, w, grad, m, v, lr, b1, b2,
                       eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const float *X, int64_t n, const uint16_t *w, float *z, int inference,
                              hipStream_t s) {
    const unsigned nb = (unsigned)((n + 255) / 256);
    if (inference) hipLaunchKernelGGL(k_mlp_fwd_mfma, dim3(nb), dim3(256), 0, s, X, n, w, z);
    else hipLaunchKernelGGL(k_mlp_fwd_fp32, dim3(nb), dim3(256), 0, s, X, n, w, z);
    return hipGetLastError();
}

}  // namespace osbli
