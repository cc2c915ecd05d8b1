// sensor_impl.h -- continuum-breakdown sensor, its training, and the
// kinetic/fluid hybrid step (device templates).
//
// Sensor.  Per cell ten features of the local state and its gradients
//   x = [ln rho, u/sqrt(T) (3), ln T, lambda |grad rho|/rho,
//        lambda |grad u_b|/sqrt(T) (3), lambda |grad T|/T],  lambda = tau sqrt(T),
// gradients by central differences over face-neighbour values (the mean of
// the four leaves across a FINER face) with centre distances h, 3h/4 (FINER),
// 3h/2 (COARSER); a domain face uses the cell's own value at distance h.
// The network 10-64-64-1 (exact GELU) maps standardised features to a logit;
// a cell is kinetic iff the logit is > 0 (probability > 1/2).  Inference runs
// on the matrix cores: each wave pushes 16 cells through
// v_mfma_f32_16x16x16_bf16 (BF16 weights and activations, FP32 accumulation).
//
// Training.  FP32 master weights; forward and backward pass in FP32 and the
// weight gradients' sums over samples in FP64, tiles of 16 samples on the
// matrix cores in a fixed order (deterministic), then Adam.  Loss:
// class-weighted binary cross-entropy on the logit.
//
// Hybrid step (paper: kinetic and continuum cells on one adaptive mesh).  A
// frozen mask per step: kinetic cells run the fused DVM step unchanged;
// fluid cells carry only U = (rho, rho u, E) (the moments buffer) and advance
//   U' = U - dt/h sum_faces (H_out(Mt(U)) + H_in(g_nb)),
// H the half-range flux sums w sum_{+-xi.n > 0} (xi.n) psi g of the discrete
// velocity set, g_nb = f (kinetic neighbour, summed over its half row) or
// Mt(U_nb) (fluid neighbour, from separable 1D sums of its Maxwellian
// tables: O(N) per face instead of O(N^3)).  Fluid cells next to kinetic
// cells (and cells turning kinetic) write Mt(U) into the state buffer first,
// so the kinetic transport reads them as ordinary rows.
#pragma once

#include "step_impl.h"

namespace dvm {
namespace impl {

// parameter block of the network (floats)
constexpr int kIn = 10, kHid = 64;
constexpr int kW1 = 0, kB1 = kW1 + kHid * kIn, kW2 = kB1 + kHid, kB2 = kW2 + kHid * kHid, kW3 = kB2 + kHid;
constexpr int kB3 = kW3 + kHid, kMean = kB3 + 1, kStd = kMean + kIn, kParams = kStd + kIn;
constexpr int kWeights = kMean;
static_assert(kParams == 4949 && kWeights == 4929, "parameter block layout");

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// ---------------------------------------------------------------------------
// features
// ---------------------------------------------------------------------------

struct FeatArgs {
    const double *mom;   // [5][n]
    const DevCell *cells;
    int64_t n;
    double h0;
    int tau_mode;
    double tau_or_kn;
};

__device__ inline void prim5(const double *mom, int64_t n, int64_t c, double q[5]) {
    const double rho = mom[c];
    const double ux = mom[n + c] / rho, uy = mom[2 * n + c] / rho, uz = mom[3 * n + c] / rho;
    q[0] = rho;
    q[1] = ux;
    q[2] = uy;
    q[3] = uz;
    q[4] = (2.0 * mom[4 * n + c] / rho - ((ux * ux + uy * uy) + uz * uz)) / 3.0;
}

// features of cell c (FP64)
__device__ inline void cell_features(const FeatArgs &a, int64_t c, double x[10]) {
    const DevCell &cell = a.cells[c];
    const double h = a.h0 / double(1 << cell.level);
    double q[5];
    prim5(a.mom, a.n, c, q);
    double g2[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        double qs[2][5], ds[2];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int f = 2 * b + side;
            const int ty = cell.type[f];
            ds[side] = h;
            if (ty == DVM_FACE_SAME || ty == DVM_FACE_COARSER) {
                prim5(a.mom, a.n, cell.nbr[f][0], qs[side]);
                if (ty == DVM_FACE_COARSER) ds[side] = 1.5 * h;
            } else if (ty == DVM_FACE_FINER) {
                double t[4][5];
                for (int k = 0; k < 4; ++k) prim5(a.mom, a.n, cell.nbr[f][k], t[k]);
                for (int v = 0; v < 5; ++v) qs[side][v] = 0.25 * (((t[0][v] + t[1][v]) + t[2][v]) + t[3][v]);
                ds[side] = 0.75 * h;
            } else {
                for (int v = 0; v < 5; ++v) qs[side][v] = q[v];
            }
        }
        for (int v = 0; v < 5; ++v) {
            const double d = (qs[1][v] - qs[0][v]) / (ds[0] + ds[1]);
            g2[v] += d * d;
        }
    }
    const double rho = q[0], T = q[4], sT = sqrt(T);
    const double tau = a.tau_mode == DVM_TAU_HS ? a.tau_or_kn / (rho * sT) : a.tau_or_kn;
    const double lam = tau * sT;
    x[0] = log(rho);
    x[1] = q[1] / sT;
    x[2] = q[2] / sT;
    x[3] = q[3] / sT;
    x[4] = log(T);
    x[5] = lam * sqrt(g2[0]) / rho;
    x[6] = lam * sqrt(g2[1]) / sT;
    x[7] = lam * sqrt(g2[2]) / sT;
    x[8] = lam * sqrt(g2[3]) / sT;
    x[9] = lam * sqrt(g2[4]) / T;
}

__global__ __launch_bounds__(256) void k_features(FeatArgs a, float *x) {
    const int64_t c = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (c >= a.n) return;
    double f[10];
    cell_features(a, c, f);
    for (int k = 0; k < 10; ++k) x[c * 10 + k] = float(f[k]);
}

// ---------------------------------------------------------------------------
// labels: r = |f - Mt|_2 / |Mt|_2 per cell, Mt of the cell's own moments
// ---------------------------------------------------------------------------

template <typename F, int NH, int T>
__global__ __launch_bounds__(T) void k_labels(const F *f, float *r, VelGrid g) {
    using L = Lane<NH, T>;
    constexpr int S = L::S;
    constexpr int64_t NV = 8 * L::B;
    __shared__ StepSmem<F, NH, T> sm;
    const L ln;
    const int64_t c = blockIdx.x;
    const F *row = f + c * NV;
    F fo[8][S];
    double m[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < S; ++q) {
#pragma unroll
        for (int o = 0; o < 8; ++o) fo[o][q] = ln.ok(q) ? row[o * L::B + ln.slot(q)] : F(0);
        if (!ln.ok(q)) continue;
        int a3[3];
        ln.axes(q, a3[0], a3[1], a3[2]);
        const double xa = (a3[0] + 0.5) * g.dv[0], ya = (a3[1] + 0.5) * g.dv[1], za = (a3[2] + 0.5) * g.dv[2];
        double s0, sx, sy, sz;
        octant_sums<F, S>(fo, q, s0, sx, sy, sz);
        m[0] += s0;
        m[1] += xa * sx;
        m[2] += ya * sy;
        m[3] += za * sz;
        m[4] += 0.5 * (xa * xa + ya * ya + za * za) * s0;
    }
    block_sum<T, 5>(m, sm.red);
    const double w = g.w;
    const double rho = w * m[0];
    const double u[3] = {w * m[1] / rho, w * m[2] / rho, w * m[3] / rho};
    const double Tt = (2.0 * w * m[4] / rho - (u[0] * u[0] + u[1] * u[1] + u[2] * u[2])) / 3.0;
    maxwell_tables<F, NH, T>(sm.mx, rho, u, Tt, 1.0, g);
    double s2[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < S; ++q) {
        if (!ln.ok(q)) continue;
        int a3[3];
        ln.axes(q, a3[0], a3[1], a3[2]);
        double G[3][2], P[3][2];
        for (int b = 0; b < 3; ++b) {
            G[b][0] = sm.mx.tab[b][NH - 1 - a3[b]][0];
            G[b][1] = sm.mx.tab[b][NH + a3[b]][0];
            P[b][0] = sm.mx.tab[b][NH - 1 - a3[b]][1];
            P[b][1] = sm.mx.tab[b][NH + a3[b]][1];
        }
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            const int ox = o >> 2, oy = (o >> 1) & 1, oz = o & 1;
            const double M = (G[0][ox] * G[1][oy]) * G[2][oz] * ((P[0][ox] + P[1][oy]) + P[2][oz]);
            const double d = double(fo[o][q]) - M;
            s2[0] += d * d;
            s2[1] += M * M;
        }
    }
    block_sum<T, 2>(s2, sm.red);
    if (threadIdx.x == 0) r[c] = float(sqrt(s2[0] / s2[1]));
}

// ---------------------------------------------------------------------------
// the network: FP32 reference forward, BF16 matrix-core forward
// ---------------------------------------------------------------------------

// one sample, FP32, weights in LDS
__device__ inline float mlp_logit32(const float *w, const float *xr) {
    float xs[kIn];
    for (int k = 0; k < kIn; ++k) xs[k] = (xr[k] - w[kMean + k]) / w[kStd + k];
    float h1[kHid];
    for (int j = 0; j < kHid; ++j) {
        float z = w[kB1 + j];
        for (int k = 0; k < kIn; ++k) z += w[kW1 + j * kIn + k] * xs[k];
        h1[j] = gelu_f(z);
    }
    float out = w[kB3];
    for (int j = 0; j < kHid; ++j) {
        float z = w[kB2 + j];
        for (int k = 0; k < kHid; ++k) z += w[kW2 + j * kHid + k] * h1[k];
        out += w[kW3 + j] * gelu_f(z);
    }
    return out;
}

__global__ __launch_bounds__(256) void k_mlp_fwd32(const float *P, const float *x, int64_t n, float *z) {
    __shared__ float w[kParams];
    for (int i = threadIdx.x; i < kParams; i += 256) w[i] = P[i];
    __syncthreads();
    const int64_t s = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (s >= n) return;
    z[s] = mlp_logit32(w, x + s * kIn);
}

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ short to_bf16(float v) {
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    u += 0x7fffu + ((u >> 16) & 1u);
    return short(u >> 16);
}

// One column of both hidden layers per lane (column 16 w + l % 16 in wave w of
// four) in the matrix cores' B layout, BF16, read once per workgroup straight
// from the parameter block; the output layer's weights of the columns
// l % 16 + 16 n.  Four-byte alignment of P is enough.
struct NetCols {
    bf16x4 b1, b2[4];
    float c1, c2, w3[4], b3;
};
__device__ __forceinline__ NetCols load_cols(const float *P) {
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4, j = 16 * (threadIdx.x >> 6) + li;
    NetCols W;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int k = 4 * lg + t;
        W.b1[t] = to_bf16(k < kIn ? P[kW1 + j * kIn + k] : 0.0f);
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        float v[4];
        __builtin_memcpy(v, P + kW2 + j * kHid + kb * 16 + 4 * lg, sizeof v);
#pragma unroll
        for (int t = 0; t < 4; ++t) W.b2[kb][t] = to_bf16(v[t]);
    }
    W.c1 = P[kB1 + j];
    W.c2 = P[kB2 + j];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) W.w3[nb] = P[kW3 + nb * 16 + li];
    W.b3 = P[kB3];
    return W;
}

// LDS of a tile of 16 rows.  The row strides keep 8-byte alignment and put
// rows on different banks.
struct NetSmem {
    __align__(8) short h1[16][kHid + 8];  // BF16 activations, the next layer's A rows
    float h2[16][kHid + 4];
};

// Logits of 16 rows by a workgroup of four waves on the matrix cores, each
// wave 16 columns of both hidden layers.  Operand layout of
// v_mfma_f32_16x16x16_bf16 for lane l: A[i = l % 16][k = 4 (l / 16) + 0..3],
// B[k = 4 (l / 16) + 0..3][j = l % 16], result D[i = 4 (l / 16) + v][j = l % 16],
// v = 0..3.  Hidden activations go through LDS to turn the result layout into
// the next layer's A layout.  xs: standardised features in BF16 (columns
// >= 10 zero), written before a barrier; every thread of row threadIdx.x / 16
// receives that row's logit.  Two barriers.
__device__ __forceinline__ float net_tile(const NetCols &W, const short (*xs)[16], NetSmem &sm) {
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4, j = 16 * (threadIdx.x >> 6) + li;
    const bf16x4 a = *reinterpret_cast<const bf16x4 *>(&xs[li][4 * lg]);
    f32x4 d = {0.f, 0.f, 0.f, 0.f};
    d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, W.b1, d, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) sm.h1[4 * lg + v][j] = to_bf16(gelu_f(d[v] + W.c1));
    __syncthreads();
    d = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
        d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
            *reinterpret_cast<const bf16x4 *>(&sm.h1[li][kb * 16 + 4 * lg]), W.b2[kb], d, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) sm.h2[4 * lg + v][j] = gelu_f(d[v] + W.c2);
    __syncthreads();
    float z = 0.0f;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) z = __builtin_fmaf(W.w3[nb], sm.h2[threadIdx.x >> 4][nb * 16 + li], z);
    return row_sum32(z) + W.b3;
}

// Logits of raw feature rows x[n][10] on the matrix cores, 16 rows at a time
// per workgroup (tile b, b + gridDim.x, ...).
__global__ __launch_bounds__(256) void k_mlp_fwd_mfma(const float *P, const float *x, int64_t n, float *z) {
    __shared__ __align__(8) short xs[16][16];
    __shared__ NetSmem sm;
    const int r = threadIdx.x >> 4, k = threadIdx.x & 15;
    const NetCols W = load_cols(P);
    const float mean = k < kIn ? P[kMean + k] : 0.0f, sd = k < kIn ? P[kStd + k] : 1.0f;
    for (int64_t r0 = int64_t(blockIdx.x) * 16; r0 < n; r0 += int64_t(gridDim.x) * 16) {
        const int64_t s = r0 + r;
        xs[r][k] = to_bf16((k < kIn && s < n) ? (x[s * kIn + k] - mean) / sd : 0.0f);
        __syncthreads();
        const float v = net_tile(W, xs, sm);
        if (k == 0 && s < n) z[s] = v;
    }
}

// Feature `lane` of cell c by a row of 16 lanes, lane f < 6 at face f (the
// same operations in the same order as cell_features, so the same bits).
__device__ __forceinline__ double cell_feature_row(const FeatArgs &a, int64_t c) {
    const int j = threadIdx.x & 15;
    const DevCell &cell = a.cells[c];
    const int ty = j < 6 ? cell.type[j] : 0;
    const bool finer = ty == DVM_FACE_FINER, one = ty == DVM_FACE_SAME || ty == DVM_FACE_COARSER;
    const bool nbr = j < 6 && (finer || one);
    const double h = a.h0 / double(1 << cell.level);
    double q[5], qs[5];
    prim5(a.mom, a.n, c, q);
    prim5(a.mom, a.n, nbr ? cell.nbr[j][0] : c, qs);
    if (j < 6 && finer) {
        double t[3][5];
        for (int k = 0; k < 3; ++k) prim5(a.mom, a.n, cell.nbr[j][k + 1], t[k]);
        for (int v = 0; v < 5; ++v) qs[v] = 0.25 * (((qs[v] + t[0][v]) + t[1][v]) + t[2][v]);
    }
    double ds = h;
    if (nbr && ty == DVM_FACE_COARSER) ds = 1.5 * h;
    if (nbr && finer) ds = 0.75 * h;
    const double dd = ds + dpp_f64<0xb1>(ds);
    double g2[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        const double d = (dpp_f64<0xb1>(qs[v]) - qs[v]) / dd;  // even lanes: side 1 - side 0 of axis lane / 2
        const double d0 = dpp_f64<0x150>(d), d1 = dpp_f64<0x152>(d), d2 = dpp_f64<0x154>(d);  // row_newbcast
        g2[v] = __builtin_fma(d2, d2, __builtin_fma(d1, d1, d0 * d0));
    }
    const double rho = q[0], T = q[4], sT = sqrt(T);
    const double tau = a.tau_mode == DVM_TAU_HS ? a.tau_or_kn / (rho * sT) : a.tau_or_kn;
    const double lam = tau * sT;
    const double g = j == 5 ? g2[0] : j == 6 ? g2[1] : j == 7 ? g2[2] : j == 8 ? g2[3] : g2[4];
    const double num = j < 5 ? (j == 1 ? q[1] : j == 2 ? q[2] : q[3]) : lam * sqrt(g);
    const double den = j == 5 ? rho : j == 9 ? T : sT;
    const double lg = log(j == 0 ? rho : T);
    return j == 0 || j == 4 ? lg : num / den;
}

// The sensor: features of CELLS cells per workgroup of four waves, then the
// network on the matrix cores (P != nullptr) or the largest gradient-length
// Knudsen number against kappa.  mask = 1: kinetic.  CELLS = 256: one thread
// per cell.  CELLS = 16: 16 lanes per cell, one at each face: a small mesh is
// bound by the latency of one tile (neighbours, FP64 divisions, the layers),
// and this form has a sixth of the chain and 16 times the wavefronts.  16^3
// cells with the network: 8.9 us a call against 27.4 with CELLS = 256;
// one-wave workgroups of 16 cells with the weights staged in LDS took 15.0.  A cell's result does not
// depend on CELLS.
template <int CELLS>
__global__ __launch_bounds__(256) void k_sensor(FeatArgs a, const float *P, double kappa, uint8_t *mask,
                                                float *score) {
    static_assert(CELLS == 16 || CELLS == 256, "cells per workgroup");
    __shared__ __align__(8) short xs[CELLS][16];
    __shared__ NetSmem sm;
    const int64_t c0 = int64_t(blockIdx.x) * CELLS;
    NetCols W{};
    if (P) W = load_cols(P);
    const auto write = [&](int64_t c, float v) {
        if (score) score[c] = P ? 1.0f / (1.0f + expf(-v)) : v;
        mask[c] = P ? uint8_t(v > 0.0f) : uint8_t(double(v) > kappa);
    };
    if constexpr (CELLS == 16) {
        const int r = threadIdx.x >> 4, k = threadIdx.x & 15;
        const int64_t c = c0 + r;
        const float mean = P && k < kIn ? P[kMean + k] : 0.0f, sd = P && k < kIn ? P[kStd + k] : 1.0f;
        const double f = cell_feature_row(a, c < a.n ? c : a.n - 1);
        if (P) {
            xs[r][k] = to_bf16(k < kIn ? (float(f) - mean) / sd : 0.0f);
        } else {
            const double f6 = dpp_f64<0x156>(f), f7 = dpp_f64<0x157>(f), f8 = dpp_f64<0x158>(f),
                         f9 = dpp_f64<0x159>(f);
            double g = dpp_f64<0x155>(f);
            g = f6 > g ? f6 : g;
            g = f7 > g ? f7 : g;
            g = f8 > g ? f8 : g;
            g = f9 > g ? f9 : g;
            if (k == 0 && c < a.n) write(c, float(g));
        }
    } else {
        const int64_t c = c0 + threadIdx.x;
        double f[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        if (c < a.n) cell_features(a, c, f);
        if (P) {
#pragma unroll
            for (int k = 0; k < 16; ++k)
                xs[threadIdx.x][k] =
                    to_bf16((k < kIn && c < a.n) ? (float(f[k < kIn ? k : 0]) - P[kMean + k]) / P[kStd + k] : 0.0f);
        } else if (c < a.n) {
            double g = f[5];
            for (int k = 6; k < 10; ++k) g = f[k] > g ? f[k] : g;
            write(c, float(g));
        }
    }
    if (!P) return;
    __syncthreads();
#pragma nounroll
    for (int t = 0; t < CELLS / 16; ++t) {
        const float v = net_tile(W, xs + 16 * t, sm);
        const int64_t c = c0 + 16 * t + (threadIdx.x >> 4);
        if ((threadIdx.x & 15) == 0 && c < a.n) write(c, v);
    }
}

// ---------------------------------------------------------------------------
// training
// ---------------------------------------------------------------------------

typedef double f64x4 __attribute__((ext_vector_type(4)));

// one weight of Adam with bias correction; c1 = 1 - beta1^t, c2 = 1 - beta2^t
struct AdamArgs {
    float *P, *m, *v;  // P NULL: the gradient only
    float lr, c1, c2;
};
__device__ __forceinline__ void adam_one(const AdamArgs &a, int i, float g) {
    const float mi = 0.9f * a.m[i] + 0.1f * g;
    const float vi = 0.999f * a.v[i] + 0.001f * g * g;
    a.m[i] = mi;
    a.v[i] = vi;
    a.P[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + 1e-8f);
}

// Forward, backward and weight-gradient sums of tiles of 16 samples, one tile
// at a time per workgroup of four waves (tile b, b + gridDim.x, ...); wave w
// owns columns 16 w .. 16 w + 15 of both hidden layers.  All three 64-wide
// contractions run on the matrix cores at the precision of the scalar code
// they replace: the layers and the back-propagated deltas in FP32
// (v_mfma_f32_16x16x4_f32), the gradient sums over samples in FP64
// (v_mfma_f64_16x16x4_f64: products of two FP32 values are exact there).
// Operand layouts for lane l, g = l / 16: A[l % 16][g], B[g][l % 16]; results:
// FP32 D[4 g + v][l % 16], FP64 D[g + 4 v][l % 16].  The sums start from the
// bias and take the inputs in index order, one fused multiply-add each, as a
// scalar loop does.
// part[block][kWeights]: the block's gradient sums; loss_part[block].
// Bound: the latency of one tile (LDS round trips between the layers, erff and
// expf), so as many workgroups as tiles up to kTrainBlocks.  A train step of
// 4,096 samples: 2,053 us with one thread per sample, its activations in a
// record in memory and one thread per weight summing over the samples; 19.7 us
// with the two launches here.
__global__ __launch_bounds__(256) void k_train_tiles(const float *P, const float *x, const float *y, int64_t n,
                                                     float pos_weight, double *part, double *loss_part) {
    constexpr int LD = kHid + 4;  // LDS row stride: 16-byte aligned rows on different banks
    __shared__ __align__(16) float xs[16][16], h1[16][LD], h2[16][LD], d1[16][LD], d2[16][LD];
    __shared__ float w3s[kHid], dz[16];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, g = lane >> 4;
    const int j = 16 * wv + li;  // this lane's column
    // the weights this lane multiplies by, kept for every tile
    float b1w[3], b2w[16], b2t[16];
#pragma unroll
    for (int t = 0; t < 3; ++t) b1w[t] = 4 * t + g < kIn ? P[kW1 + j * kIn + 4 * t + g] : 0.0f;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        b2w[t] = P[kW2 + j * kHid + 4 * t + g];
        b2t[t] = P[kW2 + (4 * t + g) * kHid + j];
    }
    const float bias1 = P[kB1 + j], bias2 = P[kB2 + j], w3 = P[kW3 + j], b3 = P[kB3];
    if (tid < kHid) w3s[tid] = P[kW3 + tid];
    f64x4 a1 = {0, 0, 0, 0}, a2[4];  // gradient sums: w1 and b1 (column kIn), w2
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) a2[nb] = f64x4{0, 0, 0, 0};
    double av = 0.0, loss = 0.0;  // threads 0..63: b2; 64..127: w3; 128: b3
    for (int64_t s0 = int64_t(blockIdx.x) * 16; s0 < n; s0 += int64_t(gridDim.x) * 16) {
        const int nr = int(min(int64_t(16), n - s0));
        {
            const int r = tid >> 4, k = tid & 15;  // column kIn: one, for the bias gradients
            float v = 0.0f;
            if (r < nr) v = k < kIn ? (x[(s0 + r) * kIn + k] - P[kMean + k]) / P[kStd + k] : k == kIn ? 1.0f : 0.0f;
            xs[r][k] = v;
        }
        __syncthreads();
        f32x4 z = {bias1, bias1, bias1, bias1};
#pragma unroll
        for (int t = 0; t < 3; ++t)
            z = __builtin_amdgcn_mfma_f32_16x16x4f32(4 * t + g < kIn ? xs[li][4 * t + g] : 0.0f, b1w[t], z, 0, 0, 0);
        float g1[4], g2[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            g1[v] = gelu_d(z[v]);
            h1[4 * g + v][j] = 4 * g + v < nr ? gelu_f(z[v]) : 0.0f;
        }
        __syncthreads();
        z = f32x4{bias2, bias2, bias2, bias2};
#pragma unroll
        for (int t = 0; t < 16; ++t) z = __builtin_amdgcn_mfma_f32_16x16x4f32(h1[li][4 * t + g], b2w[t], z, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            g2[v] = gelu_d(z[v]);
            h2[4 * g + v][j] = 4 * g + v < nr ? gelu_f(z[v]) : 0.0f;
        }
        __syncthreads();
        if (tid < 16) {
            float d = 0.0f;
            if (tid < nr) {
                float zz = b3;
#pragma unroll 16
                for (int k = 0; k < kHid; ++k) zz += w3s[k] * h2[tid][k];
                const float yy = y[s0 + tid];
                const float wt = yy > 0.5f ? pos_weight : 1.0f;
                const float ez = expf(-fabsf(zz));
                const float sig = zz >= 0.0f ? 1.0f / (1.0f + ez) : ez / (1.0f + ez);
                loss += double(wt) * (double(fmaxf(zz, 0.0f)) - double(zz) * yy + log1p(double(ez)));
                d = wt * (sig - yy) / float(n);
            }
            dz[tid] = d;
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v)  // rows beyond the batch: zero, whatever the weights are
            d2[4 * g + v][j] = 4 * g + v < nr ? dz[4 * g + v] * w3 * g2[v] : 0.0f;
        __syncthreads();
        z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 16; ++t) z = __builtin_amdgcn_mfma_f32_16x16x4f32(d2[li][4 * t + g], b2t[t], z, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) d1[4 * g + v][j] = 4 * g + v < nr ? z[v] * g1[v] : 0.0f;
        // d1's columns of a wave are read by that wave only; the rows of the
        // other arrays are complete since the last barrier
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int r = 4 * t + g;
            const double e2 = d2[r][j], e1 = d1[r][j];
            a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(e1, double(xs[r][li]), a1, 0, 0, 0);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                a2[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(e2, double(h1[r][16 * nb + li]), a2[nb], 0, 0, 0);
        }
        if (tid < 64) {
            for (int r = 0; r < 16; ++r) av += double(d2[r][tid]);
        } else if (tid < 128) {
            for (int r = 0; r < 16; ++r) av += double(dz[r]) * double(h2[r][tid - 64]);
        } else if (tid == 128) {
            for (int r = 0; r < 16; ++r) av += double(dz[r]);
        }
        __syncthreads();
    }
    double *out = part + int64_t(blockIdx.x) * kWeights;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = 16 * wv + g + 4 * v;
        if (li < kIn) out[kW1 + row * kIn + li] = a1[v];
        else if (li == kIn) out[kB1 + row] = a1[v];
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) out[kW2 + row * kHid + 16 * nb + li] = a2[nb][v];
    }
    if (tid < 64) out[kB2 + tid] = av;
    else if (tid < 128) out[kW3 + tid - 64] = av;
    else if (tid == 128) out[kB3] = av;
    if (tid < 64) {
        const double t = wave_sum(tid < 16 ? loss : 0.0);
        if (tid == 0) loss_part[blockIdx.x] = t;
    }
}

// gradient = sum of the blocks' sums in a fixed order (four interleaved
// partial sums per weight, so that 64 weights a workgroup keep their loads
// coalesced and four times the lanes busy), the mean loss, and the Adam update
// of the weight where one is asked for
__global__ __launch_bounds__(256) void k_train_reduce(const double *part, const double *loss_part, int nb, int64_t n,
                                                      float *grad, double *loss, AdamArgs adam) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int i = int(blockIdx.x) * 64 + lane;
    double s = 0.0;
    if (i < kWeights) {
#pragma unroll 8
        for (int b = q; b < nb; b += 4) s += part[int64_t(b) * kWeights + i];
    }
    red[q][lane] = s;
    if (blockIdx.x == 0 && q == 3) {
        double l = 0.0;
        for (int b = lane; b < nb; b += 64) l += loss_part[b];
        l = wave_sum(l);
        if (lane == 0) *loss = l / double(n);
    }
    __syncthreads();
    if (q == 0 && i < kWeights) {
        const float gr = float((red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]));
        grad[i] = gr;
        if (adam.P) adam_one(adam, i, gr);
    }
}

__global__ __launch_bounds__(256) void k_adam(AdamArgs a, const float *grad) {
    const int i = int(blockIdx.x) * 256 + threadIdx.x;
    if (i < kWeights) adam_one(a, i, grad[i]);
}

// standardisation statistics of a feature set (FP64, fixed order)
__global__ __launch_bounds__(256) void k_norm_stats(const float *x, int64_t n, float *P) {
    __shared__ double red[4 * 2];
    const int k = blockIdx.x;  // feature
    double s[2] = {0.0, 0.0};
    for (int64_t i = threadIdx.x; i < n; i += 256) s[0] += double(x[i * kIn + k]);
    double v1[1] = {s[0]};
    block_sum<256, 1>(v1, red);
    const double mean = v1[0] / double(n);
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double d = double(x[i * kIn + k]) - mean;
        s[1] += d * d;
    }
    double v2[1] = {s[1]};
    block_sum<256, 1>(v2, red);
    if (threadIdx.x == 0) {
        const double sd = sqrt(v2[0] / double(n));
        P[kMean + k] = float(mean);
        P[kStd + k] = float(sd > 1e-6 ? sd : 1e-6);
    }
}

// ---------------------------------------------------------------------------
// hybrid step
// ---------------------------------------------------------------------------

// per axis: full A[3], B[3]; + half A[4], B[4]; - half A[4], B[4]; then rho, u[3], T
constexpr int kFluxRec = 71;

struct HybArgs {
    const uint8_t *mask;  // effective mask (1 kinetic)
    uint8_t *prev;        // mask of the previous hybrid step
    uint8_t *rows;        // bit 0: write Mt(U) into the state buffer before the step;
                          // bit 1 + f: a kinetic cell with a fluid neighbour across face f
    double *flux;         // [n][kFluxRec] separable sums of fluid cells' Maxwellians
    double *face;         // [n][6][5] outgoing half-range fluxes of kinetic cells next to fluid ones
    int32_t closed;       // fluid-fluid faces: continuous half-range integrals (erf form)
    int32_t pad;
};

// mask | (cell touches a non-periodic domain face): those cells stay kinetic
__global__ __launch_bounds__(64) void k_mask_eff(const uint8_t *in, uint8_t *out, const DevCell *cells, int64_t n) {
    const int64_t c = int64_t(blockIdx.x) * 64 + threadIdx.x;
    if (c >= n) return;
    uint8_t m = in[c] ? 1 : 0;
    for (int f = 0; f < 6; ++f) m |= uint8_t(cells[c].type[f] >= DVM_FACE_INFLOW);
    out[c] = m;
}

// The cells' preparation, 16 lanes per cell and four cells per one-wave
// workgroup.  Lanes f < 6 look over face f: the cells whose state buffer row
// must hold Mt(U) this step are flagged (fluid cells next to a kinetic one,
// cells turning kinetic), and so are the faces of kinetic cells next to a
// fluid one (the step kernel reads that one byte instead of its neighbours'
// masks); the previous mask is updated.  Fluid cells get the separable sums of their
// Maxwellian (the construction of maxwell_solve): a lane per velocity node for
// the tables and their sums, every lane the 5 x 6 elimination, a lane per
// half-axis sum of the record.  Bound by latency: with a thread per cell the
// same took 20.7 us on 16^3 cells x 8^3 nodes (64 wavefronts, 48 exponentials
// and 100 divisions in one chain), 6.8 now.
__global__ __launch_bounds__(64) void k_fluid_state(StepArgs a, HybArgs h) {
    __shared__ double2 tab[4][3][24];  // (g, 1 + d.phi part) per node; axis 0 carries C
    const int r = threadIdx.x >> 4, j = threadIdx.x & 15;
    const int64_t n = a.n_cells, cr = int64_t(blockIdx.x) * 4 + r, c = cr < n ? cr : n - 1;
    const int m = h.mask[c], pm = h.prev[c];
    const DevCell &cell = a.cells[c];
    double U[5];
#pragma unroll
    for (int x = 0; x < 5; ++x) U[x] = a.mom[x * n + c];
    bool kin_nb = false, fluid_nb = false;
    if (j < 6) {
        const int ty = cell.type[j];
        const int k = ty == DVM_FACE_FINER ? 4 : (ty == DVM_FACE_SAME || ty == DVM_FACE_COARSER) ? 1 : 0;
        for (int q = 0; q < k; ++q) {
            const bool kin = h.mask[cell.nbr[j][q]] != 0;
            kin_nb |= kin;
            fluid_nb |= !kin;
        }
    }
    const bool any_kin = (__ballot(kin_nb) >> (16 * r)) & 0xffff;
    const int fluid_faces = int(__ballot(fluid_nb) >> (16 * r)) & 0x3f;
    if (j == 0 && cr < n) {
        h.rows[c] = uint8_t(((m == 0 && any_kin) || (m == 1 && pm == 0)) | (m == 1 ? fluid_faces << 1 : 0));
        h.prev[c] = uint8_t(m);
    }
    const double rho = U[0];
    const double u[3] = {U[1] / rho, U[2] / rho, U[3] / rho};
    const double Tt = (2.0 * U[4] / rho - ((u[0] * u[0] + u[1] * u[1]) + u[2] * u[2])) / 3.0;
    bool act = cr < n && !m;
    if (act && (!(rho > 0.0) || !(Tt > 0.0))) {
        if (j == 0) *a.flag = 1;
        act = false;
    }
    if (!__any(act)) return;
    const double sT = sqrt(Tt);
    const int nh = a.g.nh, N = 2 * nh;
    double S[15], ck[3][2], gk[3][2];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        double p[5];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int k = j + 16 * s;
            ck[b][s] = ((double(k - nh) + 0.5) * a.g.dv[b] - u[b]) / sT;
            gk[b][s] = 0.0;
            if (s == 0 || N > 16) gk[b][s] = k < N ? exp(-0.5 * ck[b][s] * ck[b][s]) : 0.0;
            double t = gk[b][s];
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                p[q] = s == 0 ? t : p[q] + t;
                t *= ck[b][s];
            }
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) S[5 * b + q] = row_sum(p[q]) * a.g.dv[b];
    }
    const double x2 = 6.283185307179586476925286766559 * Tt;
    const double C = rho / (x2 * sqrt(x2)), n32 = rho / C;
    double A[5][6], d[5];
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int l = i; l < 5; ++l) A[i][l] = A[l][i] = gram_entry(i, l, &S[0], &S[5], &S[10]);
#pragma unroll
    for (int i = 0; i < 5; ++i) A[i][5] = (i == 0 ? 1.0 : i == 4 ? 3.0 : 0.0) * n32 - A[i][0];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            if (i == k) continue;
            const double t = A[i][k] / A[k][k];
#pragma unroll
            for (int l = k + 1; l < 6; ++l) A[i][l] -= t * A[k][l];
        }
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) d[i] = A[i][5] / A[i][i];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int k = j + 16 * s;
            const double cc = ck[b][s];
            if (k < N)
                tab[r][b][k] = double2{b == 0 ? gk[b][s] * C : gk[b][s],
                                       (b == 0 ? 1.0 + d[0] : 0.0) + d[1 + b] * cc + d[4] * cc * cc};
        }
    __syncthreads();
    if (!act) return;
    // lane (half, polynomial on or off, power): 16 sums over the nodes of one
    // half of an axis; the whole-axis sums are those of the two halves
    double *R = h.flux + c * kFluxRec;
    const int neg = j >> 3, pol = (j >> 2) & 1, pw = j & 3;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        double acc = 0.0;
        for (int i = 0; i < nh; ++i) {
            const int k = neg ? i : nh + i;
            const double xi = (double(k - nh) + 0.5) * a.g.dv[b];
            const double2 t = tab[r][b][k];
            const double x1 = pw > 0 ? xi : 1.0, x2 = pw > 1 ? xi : 1.0, x3 = pw > 2 ? xi : 1.0;
            acc += ((x1 * x2) * x3 * t.x) * (pol ? t.y : 1.0);
        }
        const double both = acc + dpp_f64<0x128>(acc);  // row_ror:8
        R[b * 22 + 6 + j] = acc;
        if (!neg && pw < 3) R[b * 22 + 3 * pol + pw] = both;
    }
    // the primitive state of U itself (the closed-form fluxes)
    if (j < 5) R[66 + j] = j == 0 ? rho : j == 1 ? u[0] : j == 2 ? u[1] : j == 3 ? u[2] : Tt;
}

// Mt(U) rows of the flagged cells (one workgroup per cell, others exit).
template <typename F, int NH, int T>
__global__ __launch_bounds__(T) void k_hybrid_rows(StepArgs a, HybArgs h) {
    constexpr int64_t NV = 8 * NH * NH * NH;
    __shared__ MaxwellSmem<F, NH> sm;
    const int64_t c = blockIdx.x, n = a.n_cells;
    if (!(h.rows[c] & 1)) return;
    const double rho = a.mom[c];
    const double u[3] = {a.mom[n + c] / rho, a.mom[2 * n + c] / rho, a.mom[3 * n + c] / rho};
    const double Tt = (2.0 * a.mom[4 * n + c] / rho - (u[0] * u[0] + u[1] * u[1] + u[2] * u[2])) / 3.0;
    if (!(rho > 0.0) || !(Tt > 0.0)) {
        if (threadIdx.x == 0) *a.flag = 1;
        return;
    }
    maxwell_tables<F, NH, T>(sm, rho, u, Tt, 1.0, a.g);
    F zero[8][Lane<NH, T>::S];
    for (int q = 0; q < Lane<NH, T>::S; ++q)
        for (int o = 0; o < 8; ++o) zero[o][q] = F(0);
    const Rsrc out = rsrc(static_cast<const F *>(a.f_in) + c * NV, uint32_t(NV * sizeof(F)));
    relax_store<F, NH, T, false>(sm, zero, F(0), out);
}

// sum over the tensor grid of prod_a xi_a^p[a] Mt, the normal axis b summed
// over one half (hs = 6: positive, 14: negative), the others over all nodes
__device__ __forceinline__ double sep_moment(const double *R, int b, int hs, int px, int py, int pz) {
    const double *X = R, *Y = R + 22, *Z = R + 44;
    const double Ax = b == 0 ? X[hs + px] : X[px], Bx = b == 0 ? X[hs + 4 + px] : X[3 + px];
    const double Ay = b == 1 ? Y[hs + py] : Y[py], By = b == 1 ? Y[hs + 4 + py] : Y[3 + py];
    const double Az = b == 2 ? Z[hs + pz] : Z[pz], Bz = b == 2 ? Z[hs + 4 + pz] : Z[3 + pz];
    return Bx * Ay * Az + Ax * By * Az + Ax * Ay * Bz;
}

// w sum over one half (normal axis b) of xi_b psi Mt, psi = (1, xi, |xi|^2/2)
__device__ __forceinline__ void sep_flux(const double *R, int b, int hs, double w, double out[5]) {
    const int px = b == 0, py = b == 1, pz = b == 2;
    out[0] = w * sep_moment(R, b, hs, px, py, pz);
    out[1] = w * sep_moment(R, b, hs, px + 1, py, pz);
    out[2] = w * sep_moment(R, b, hs, px, py + 1, pz);
    out[3] = w * sep_moment(R, b, hs, px, py, pz + 1);
    out[4] = 0.5 * w *
             ((sep_moment(R, b, hs, px + 2, py, pz) + sep_moment(R, b, hs, px, py + 2, pz)) +
              sep_moment(R, b, hs, px, py, pz + 2));
}

// Kinetic cells next to fluid ones: the half-range flux of their own f
// through each such face (listed in one byte: reading types, neighbours and
// their masks here was a chain of loads per face), w sum_{leaving} xi_b psi f (signed xi_b), before
// the transport overwrites f.
struct HybHook {
    HybArgs h;
    // moments of the values leaving through face FACE of cell c (FACE < 0:
    // face `face`, uniform).  Up to three rounds a thread one code serves the
    // six faces and picks the octants by selects: with a copy per face the
    // cells next to fluid ones spent their time fetching instructions (hybrid
    // channel, 26,100 cells x 12^3 nodes FP32: 233 -> 177 us with the sensor,
    // 193 with a cell's divisions in full; 262,144 cells x 8^3: 597 -> 540, 592).
    // At nine rounds (24^3 FP32) the selects cost more: 719 us with copies, 775
    // without.
    template <int FACE, typename F, int NH, int T>
    __device__ __forceinline__ void face_flux(const StepArgs &a, int64_t c, int face, const Regs<F, NH, T> &fo,
                                              double *red) const {
        using L = Lane<NH, T>;
        constexpr int S = L::S;
        const int f = FACE < 0 ? face : FACE, b = f >> 1, side = f & 1;
        const L ln;
        // For a round the four leaving octants share |xi| and the sign along
        // b; only the signs along the other two axes (p, r) change.  So the
        // five moments need three sums of the stored values, formed in the
        // storage precision and widened once: S (all four), Sp and Sr (signed
        // by the sign along p and along r).
        const int p = b == 0 ? 1 : 0, r = b == 2 ? 1 : 2;
        const double sg = side ? 1.0 : -1.0;
        double v[5] = {0, 0, 0, 0, 0};  // density, along b, p, r, energy
#pragma unroll
        for (int q = 0; q < S; ++q) {
            if (!ln.ok(q)) continue;
            F s0 = F(0), sp = F(0), sr = F(0);
#pragma unroll
            for (int o = 0; o < 8; ++o) {
                const bool leaves = ((o >> (2 - b)) & 1) == side;
                if (FACE >= 0 && !leaves) continue;
                const F x = leaves ? fo[o][q] : F(0);
                s0 += x;
                sp += (o >> (2 - p)) & 1 ? x : -x;
                sr += (o >> (2 - r)) & 1 ? x : -x;
            }
            int a3[3];
            ln.axes(q, a3[0], a3[1], a3[2]);
            const double ax = (a3[0] + 0.5) * a.g.dv[0], ay = (a3[1] + 0.5) * a.g.dv[1],
                         az = (a3[2] + 0.5) * a.g.dv[2];
            const double S0 = double(s0), Sp = double(sp), Sr = double(sr);
            const double xb = sg * (b == 0 ? ax : b == 1 ? ay : az);  // xi . e_b of the leaving values
            v[0] += xb * S0;
            v[1] += xb * xb * S0;
            v[2] += xb * (b == 0 ? ay : ax) * Sp;
            v[3] += xb * (b == 2 ? ay : az) * Sr;
            v[4] += 0.5 * xb * ((ax * ax + ay * ay) + az * az) * S0;
        }
        block_sum<T, 5>(v, red);
        if (threadIdx.x == 0) {
            double *out = h.face + (c * 6 + f) * 5;
            out[0] = a.g.w * v[0];
            out[1 + b] = a.g.w * v[1];
            out[1 + p] = a.g.w * v[2];
            out[1 + r] = a.g.w * v[3];
            out[4] = a.g.w * v[4];
        }
    }
    template <typename F, int NH, int T>
    __device__ __forceinline__ void apply(const StepArgs &a, int64_t c, const Regs<F, NH, T> &fo, double *red) const {
        const uint32_t faces = h.rows[c] >> 1;  // written by k_fluid_state
#pragma nounroll
        for (int f = 0; f < 6; ++f) {
            if (!((faces >> f) & 1)) continue;
            if constexpr (Lane<NH, T>::S <= 3) {
                face_flux<-1, F, NH, T>(a, c, f, fo, red);
            } else {
                switch (f) {
                case 0: face_flux<0, F, NH, T>(a, c, f, fo, red); break;
                case 1: face_flux<1, F, NH, T>(a, c, f, fo, red); break;
                case 2: face_flux<2, F, NH, T>(a, c, f, fo, red); break;
                case 3: face_flux<3, F, NH, T>(a, c, f, fo, red); break;
                case 4: face_flux<4, F, NH, T>(a, c, f, fo, red); break;
                default: face_flux<5, F, NH, T>(a, c, f, fo, red); break;
                }
            }
        }
    }
};

// Kinetic cells (fluid cells: k_fluid_update), in the XCD-aware cell order
// of the plain step.  A kinetic cell with no fluid face neighbour has nothing
// to record and runs exactly the plain step's code (the reduced code when it
// has no FINER or WALL face); one next to a fluid cell runs the full code with
// the interface-flux hook.  All three compute the same step, bitwise.  One
// kernel holds them all: at 24^3 FP32 the hook's copies make it spill 53 of its
// 168 registers (208 B a lane), where the plain step's 155 fit.
template <typename F, int NH, int T, int WPE, int FENCE, bool NT>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(WPE, 8))) void k_step_hybrid(StepArgs a,
                                                                                               HybArgs h) {
    __shared__ StepSmem<F, NH, T> sm;
    const int64_t c = remap_cell(blockIdx.x, gridDim.x, a.xcd_log2);
    if (!h.mask[c]) return;
    // one byte, written by k_fluid_state: the faces with a fluid neighbour
    if (h.rows[c] >> 1) {
        const HybHook hook{h};
        step_cell<F, NH, T, FENCE, NT, false, false, HybHook>(a, c, sm, hook);
    } else if (needs_correction(a.cells, c)) {
        step_cell<F, NH, T, FENCE, NT, false, false>(a, c, sm);
    } else {
        step_cell<F, NH, T, FENCE, NT, false, true>(a, c, sm);
    }
}

// Half-range flux of the continuous Maxwellian of (rho, u, T) = P[0..4]
// through a face with normal e_b: the integral over xi_b > 0 (pos) or < 0 of
// xi_b (1, xi, |xi|^2 / 2) M.  With xi_b = u_b + sqrt(T) t, t standard
// normal, the half-space is t > -s (pos) or t < -s, s = u_b / sqrt(T); its
// probability is q = erfc(-+s / sqrt 2) / 2 and the truncated moments of t
// follow from phi(s) = exp(-s^2/2) / sqrt(2 pi): E[t] = +-phi,
// E[t^2] = q -+ s phi, E[t^3] = +-(s^2 + 2) phi.  The transverse axes are
// full Gaussians (mean u_a, variance T).
__device__ __forceinline__ void closed_flux(const double *P, int b, bool pos, double out[5]) {
    const double rho = P[0], T = P[4], sd = sqrt(T);
    const double ub = P[1 + b], s = ub / sd;
    const double sg = pos ? 1.0 : -1.0;
    const double q = 0.5 * erfc(-sg * s * 0.70710678118654752440);
    const double ph = exp(-0.5 * s * s) * 0.39894228040143267794;
    const double m1 = ub * q + sg * sd * ph;
    const double m2 = (ub * ub + T) * q + sg * ub * sd * ph;
    const double m3 = (ub * ub + 3.0 * T) * ub * q + sg * (ub * ub + 2.0 * T) * sd * ph;
    double tr = 0.0;
    for (int x = 0; x < 3; ++x) {
        if (x == b) {
            out[1 + x] = rho * m2;
        } else {
            out[1 + x] = rho * P[1 + x] * m1;
            tr += P[1 + x] * P[1 + x] + T;
        }
    }
    out[0] = rho * m1;
    out[4] = 0.5 * rho * (m3 + m1 * tr);
}

// Signed flux sum of face f of fluid cell c (H_out + H_in, averaged over the
// leaves of a FINER face).
__device__ __forceinline__ void fluid_face(const StepArgs &a, const HybArgs &h, const DevCell &cell, int64_t c, int f,
                                           double term[5]) {
    const double w = a.g.w;
    const int b = f >> 1, side = f & 1;
    const double sg = side ? 1.0 : -1.0;  // outward normal along b
    const int nk = cell.type[f] == DVM_FACE_FINER ? 4 : 1;
    double hout[5];
    sep_flux(h.flux + c * kFluxRec, b, side ? 6 : 14, w, hout);
    if (h.closed) {
        // per neighbour: closed-form fluxes on both sides of a fluid-fluid
        // face, the discrete ones where the neighbour is kinetic
        double cout[5], s[5] = {0, 0, 0, 0, 0};
        closed_flux(h.flux + c * kFluxRec + 66, b, side == 1, cout);
        for (int k = 0; k < nk; ++k) {
            const int64_t nb = cell.nbr[f][k];
            double t[5];
            if (h.mask[nb] == 0) {
                closed_flux(h.flux + nb * kFluxRec + 66, b, side == 0, t);
                for (int x = 0; x < 5; ++x) s[x] += cout[x] + t[x];
            } else {
                const double *q = h.face + (nb * 6 + (f ^ 1)) * 5;
                for (int x = 0; x < 5; ++x) s[x] += hout[x] + q[x];
            }
        }
        for (int x = 0; x < 5; ++x) term[x] = sg * (s[x] / double(nk));
        return;
    }
    double hin[5] = {0, 0, 0, 0, 0};
    for (int k = 0; k < nk; ++k) {
        const int64_t nb = cell.nbr[f][k];
        double t[5];
        if (h.mask[nb] == 0) {
            sep_flux(h.flux + nb * kFluxRec, b, side ? 14 : 6, w, t);
        } else {
            const double *q = h.face + (nb * 6 + (f ^ 1)) * 5;  // leaving nb towards c
            for (int x = 0; x < 5; ++x) t[x] = q[x];
        }
        for (int x = 0; x < 5; ++x) hin[x] += t[x];
    }
    for (int x = 0; x < 5; ++x) term[x] = sg * (hout[x] + hin[x] / double(nk));
}

// Fluid cells: U' = U - dt/h sum_faces (H_out + H_in).  Eight lanes per cell
// and eight cells per one-wave workgroup: lane f < 6 takes face f, then lane
// x < 5 adds the six faces' terms of moment x in face order.  With a thread
// per cell the six faces' chains of dependent loads ran one after another:
// 16.8 us on 16^3 cells, 4.4 now.
__global__ __launch_bounds__(64) void k_fluid_update(StepArgs a, HybArgs h) {
    __shared__ double terms[8][6][5];
    const int r = threadIdx.x >> 3, f = threadIdx.x & 7;
    const int64_t n = a.n_cells, cr = int64_t(blockIdx.x) * 8 + r, c = cr < n ? cr : n - 1;
    const bool act = cr < n && !h.mask[c];
    if (!__any(act)) return;
    const DevCell &cell = a.cells[c];
    if (act && f < 6) fluid_face(a, h, cell, c, f, terms[r][f]);
    __syncthreads();
    double U = 0.0;
    if (act && f < 5) {
        double acc = 0.0;
        for (int e = 0; e < 6; ++e) acc += terms[r][e][f];
        const double hc = a.h0 / double(1 << cell.level);
        U = a.mom[f * n + c] - a.dt / hc * acc;
        a.mom[f * n + c] = U;
    }
    const double U0 = __shfl(U, 0, 8), U1 = __shfl(U, 1, 8), U2 = __shfl(U, 2, 8), U3 = __shfl(U, 3, 8),
                 U4 = __shfl(U, 4, 8);
    const double k2 = (U1 * U1 + U2 * U2 + U3 * U3) / U0;
    if (act && f == 0 && (!(U0 > 0.0) || !(2.0 * U4 - k2 > 0.0))) *a.flag = 1;
}

// After hybrid steps the f rows of fluid cells are stale and their state is
// the conserved moments U: copy U over what was recomputed from f.
__global__ __launch_bounds__(256) void k_fluid_moments(const uint8_t *mask, const double *mom, double *out,
                                                       int64_t n) {
    const int64_t c = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (c >= n || mask[c]) return;
    for (int x = 0; x < 5; ++x) out[x * n + c] = mom[x * n + c];
}

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------

template <typename F>
hipError_t labels_dispatch(const void *f, float *r, int64_t n, const VelGrid &g, hipStream_t st) {
    const F *p = static_cast<const F *>(f);
    const dim3 grid{unsigned(n), 1, 1};
    switch (g.nh) {
    case 2: hipLaunchKernelGGL((k_labels<F, 2, 64>), grid, dim3(64), 0, st, p, r, g); break;
    case 4: hipLaunchKernelGGL((k_labels<F, 4, 64>), grid, dim3(64), 0, st, p, r, g); break;
    case 6: hipLaunchKernelGGL((k_labels<F, 6, 256>), grid, dim3(256), 0, st, p, r, g); break;
    case 8: hipLaunchKernelGGL((k_labels<F, 8, 256>), grid, dim3(256), 0, st, p, r, g); break;
    case 12: hipLaunchKernelGGL((k_labels<F, 12, 576>), grid, dim3(576), 0, st, p, r, g); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename F>
hipError_t hybrid_dispatch(const StepArgs &a, const HybArgs &h, hipStream_t st) {
    const dim3 grid{unsigned(a.n_cells), 1, 1}, g4{unsigned((a.n_cells + 3) / 4), 1, 1},
        g8{unsigned((a.n_cells + 7) / 8), 1, 1};
    hipLaunchKernelGGL(k_fluid_state, g4, dim3(64), 0, st, a, h);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
#define DVM_HYB(NH, T, W, FN)                                                                      \
    case NH:                                                                                       \
        hipLaunchKernelGGL((k_hybrid_rows<F, NH, T>), grid, dim3(T), 0, st, a, h);               \
        e = hipGetLastError();                                                                     \
        if (e != hipSuccess) return e;                                                             \
        hipLaunchKernelGGL((k_step_hybrid<F, NH, T, W, FN, true>), grid, dim3(T), 0, st, a, h); \
        break;
    switch (a.g.nh) {
        DVM_HYB(2, 64, 4, 0)
        DVM_HYB(4, 64, 5, 0)
        DVM_HYB(6, 256, 6, 0)
        DVM_HYB(8, 256, 5, 0)
    case 12:
        // FP64 rows do not fit the registers of 192 threads at three waves per
        // SIMD (394 spilled): the plain step's wide shape.  Channel, 8,000
        // cells: 857 -> 582 us with the sensor (a quarter more at five waves, 134
        // spilled).
        if constexpr (std::is_same<F, double>::value) {
            switch (a.g.nh) { DVM_HYB(12, 576, 3, 0) }
        } else {
            switch (a.g.nh) { DVM_HYB(12, 192, 3, 1) }
        }
        break;
    default: return hipErrorInvalidValue;
    }
#undef DVM_HYB
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fluid_update, g8, dim3(64), 0, st, a, h);
    return hipGetLastError();
}

}  // namespace impl
}  // namespace dvm
