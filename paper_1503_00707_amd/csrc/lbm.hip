// lbm.hip -- the lattice Boltzmann subset (section 4): D3Q19 / D3Q27 on the
// same octree, finite-volume upwind transport of eq. (2) for each lattice
// vector, then BGK relaxation toward the second-order equilibrium
//   f_eq = w rho (1 + c.u / cs^2 + (c.u)^2 / (2 cs^4) - |u|^2 / (2 cs^2)),  cs^2 = 1/3.
// With 19 or 27 values per cell a whole cell fits in one thread's registers:
// one thread per cell, f stored population-major ([q][cell]) so that the
// lanes of a wave read 64 consecutive cells of one population (coalesced),
// and the upwind neighbours' values are gathers served mostly by L2 (cells
// in Morton order).  Algorithmic traffic: read f once, write f once,
// 2 Q sizeof(F) bytes per cell, plus the 32-byte cell record.
#include <hip/hip_runtime.h>

#include "step_impl.h"

namespace dvm {
namespace {

// lattice vectors in canonical 3^3 order (kx, ky, kz in 0..2, c = k - 1),
// the 8 corners left out for D3Q19
template <int Q>
struct Lattice {
    int c[Q][3];
    double w[Q];
    constexpr Lattice() : c(), w() {
        int q = 0;
        for (int kx = 0; kx < 3; ++kx)
            for (int ky = 0; ky < 3; ++ky)
                for (int kz = 0; kz < 3; ++kz) {
                    const int c2 = (kx - 1) * (kx - 1) + (ky - 1) * (ky - 1) + (kz - 1) * (kz - 1);
                    if (Q == 19 && c2 == 3) continue;
                    c[q][0] = kx - 1;
                    c[q][1] = ky - 1;
                    c[q][2] = kz - 1;
                    w[q] = Q == 27 ? (c2 == 0 ? 8.0 / 27 : c2 == 1 ? 2.0 / 27 : c2 == 2 ? 1.0 / 54 : 1.0 / 216)
                                   : (c2 == 0 ? 1.0 / 3 : c2 == 1 ? 1.0 / 18 : 1.0 / 36);
                    ++q;
                }
    }
};

template <int Q>
__device__ constexpr Lattice<Q> kLat{};

// the populations that enter through face f, ascending, five bits each
template <int Q>
constexpr uint64_t face_populations(int f) {
    constexpr Lattice<Q> lat{};
    uint64_t code = 0;
    int k = 0;
    for (int q = 0; q < Q; ++q)
        if (lat.c[q][f >> 1] == (f & 1 ? -1 : 1)) code |= uint64_t(q) << (5 * k++);
    return code;
}

// a value from lane `src` of the wave
__device__ __forceinline__ float lane_value(float v, int src) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src << 2, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double lane_value(double v, int src) { return impl::shfl_f64(v, src); }

__device__ __forceinline__ int face_kind(uint32_t meta, int f) { return int((meta >> (3 * f)) & 7u); }

// One cell per thread.  What bounds it: the address units, which take some 20
// cycles for each gather of 64 scattered values.  A regular cell needs 19 + 30
// reads (D3Q19); a FINER face adds four reads for each of its populations, and
// done where they occur nearly every wave of the 996,150-cell octree (15 % of
// the cells have FINER faces) issues them for every face with a few lanes
// active.  So the workgroup lists its FINER faces first and its threads form
// the means of whole lists of them into LDS (kFineCap faces; a workgroup with
// more of them forms each in its own lane), and a neighbour among the wave's
// own 64 cells (about two thirds of them, in Morton order) is read from that
// lane's registers.  D3Q19 FP32 on that octree: 95 -> 45 us a step, 248 MB past
// the L2 at 5.8 TB/s (a copy of that size reaches 7.0 TB/s here).
// BUF: the state fits 32-bit byte offsets, so every access is a raw buffer
// access (per-lane 32-bit cell offset, the population's base as a scalar
// offset) instead of a 64-bit address per lane.
constexpr int kFineCap = 256;
// FINE: the mesh has FINER faces; without, no list is made.
template <typename F, int Q, bool BUF, bool FINE>
__global__ __launch_bounds__(256) void k_lbm(LbmArgs a) {
    constexpr int NF = Q == 19 ? 5 : 9;  // populations that enter through a face
    __shared__ F mean[NF][kFineCap];     // [population of the face, ascending][listed face]
    __shared__ int2 list[kFineCap];      // first leaf list entry, face
    __shared__ int n_fine[4];
    const int64_t n = a.n;
    const int64_t c = int64_t(impl::remap_cell(blockIdx.x, gridDim.x, a.xcd_log2)) * 256 + threadIdx.x;
    const F *fi = static_cast<const F *>(a.f_in);
    F *fo = static_cast<F *>(a.f_out);
    const uint32_t bytes = BUF ? uint32_t(uint64_t(Q) * uint64_t(a.n) * sizeof(F)) : 0u;
    const impl::Rsrc ri = impl::rsrc(fi, bytes), ro = impl::rsrc(fo, bytes);
    auto ld = [&](int q, int64_t idx) -> F {
        if constexpr (BUF)
            return impl::bld<F>(ri, uint32_t(idx) * uint32_t(sizeof(F)), uint32_t(q) * uint32_t(a.n) * uint32_t(sizeof(F)));
        else
            return fi[q * a.n + idx];
    };
    auto ldv = [&](int64_t at) -> F {  // the same with the population in the lane's own offset
        if constexpr (BUF) return impl::bld<F>(ri, uint32_t(at) * uint32_t(sizeof(F)), 0u);
        else return fi[at];
    };
    LbmCell rec{};
    if (c < n) rec = a.cells[c];
    // on a mesh without level jumps the own values are in flight with the record
    // (32^3 cells, D3Q19 FP32: 6.1 -> 5.8 us a step); with jumps they follow the
    // list, since held across it they cost more registers than latency (996,150
    // cells: 49 against 45 us)
    F fs[Q], acc[Q];
    if constexpr (!FINE) {
#pragma unroll
        for (int q = 0; q < Q; ++q) fs[q] = ld(q, min(c, n - 1));
    }
    // the one upwind cell per face; the cell itself at an OUTFLOW face (zero
    // gradient) and at a FINER one, whose mean replaces what is read there
    int32_t up[6];
    bool fine[6];
    int my_fine = 0;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int kind = face_kind(rec.meta, f);
        fine[f] = kind == DVM_FACE_FINER;
        my_fine += fine[f];
        up[f] = kind == DVM_FACE_SAME || kind == DVM_FACE_COARSER ? rec.nb[f] : int32_t(c);
    }
    // this lane's place in the workgroup's list of FINER faces
    int at = my_fine, total = 0;
    if constexpr (FINE) {
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(at, off, 64);
            if (lane >= off) at += v;
        }
        if (lane == 63) n_fine[wv] = at;
        at -= my_fine;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            at += w < wv ? n_fine[w] : 0;
            total += n_fine[w];
        }
    }
    const bool listed = total <= kFineCap;
    if (FINE && total > 0 && listed) {  // uniform
        int k = at, t = rec.fine;
#pragma unroll
        for (int f = 0; f < 6; ++f)
            if (fine[f]) {
                list[k++] = int2{t, f};
                t += 4;  // tuples of four follow each other in face order
            }
        __syncthreads();
        for (int e = threadIdx.x; e < total; e += 256) {
            const int f = list[e].y;
            const int32_t *t4 = a.fine + list[e].x;
            const int32_t t0 = t4[0], t1 = t4[1], t2 = t4[2], t3 = t4[3];
            uint64_t code = 0;
#pragma unroll
            for (int g = 0; g < 6; ++g) code = f == g ? face_populations<Q>(g) : code;
#pragma unroll
            for (int k2 = 0; k2 < NF; ++k2) {
                const int64_t q = int64_t((code >> (5 * k2)) & 31u) * n;
                mean[k2][e] = F(0.25) * ((ldv(q + t0) + ldv(q + t1)) + (ldv(q + t2) + ldv(q + t3)));
            }
        }
        __syncthreads();
    }
    if (c >= n) return;
    const double h = a.h0 / double(1u << (rec.meta >> 24));
    const F r = F(a.dt / h);
    if constexpr (FINE) {
#pragma unroll
        for (int q = 0; q < Q; ++q) fs[q] = ld(q, c);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q] = F(0);
    const int32_t *t = a.fine + rec.fine;
    // Upwind values along axis b: a neighbour among the wave's own cells from
    // that lane's registers, the others' read.  Without level jumps these reads
    // are an axis ahead, the first axis' in flight with the own values: where
    // the state stays in the Infinity Cache their latency showed (100^3 cells
    // D3Q19 FP32: 32.4 us a step with every neighbour read, 35.1 with the reads
    // after the exchange, 31.8 now; 85^3 FP64 37.4, 41.4, 38.1; 128^3 FP64 154.8,
    // 146.0, 144.9).  With jumps the registers are not there.
    F ua[FINE ? 1 : 3][Q];
    const auto others = [&](int b, F *u) {
#pragma unroll
        for (int f = 2 * b; f < 2 * b + 2; ++f)
            if ((up[f] ^ int32_t(c)) >> 6) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (kLat<Q>.c[q][b] == (f & 1 ? -1 : 1)) u[q] = ld(q, up[f]);
            }
    };
    if constexpr (!FINE) others(0, ua[0]);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        F *u = ua[FINE ? 0 : b];
        if constexpr (!FINE)
            if (b < 2) others(b + 1, ua[b + 1]);
#pragma unroll
        for (int f = 2 * b; f < 2 * b + 2; ++f) {
            const bool own = !((up[f] ^ int32_t(c)) >> 6);
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (kLat<Q>.c[q][b] == (f & 1 ? -1 : 1)) {
                    const F w = lane_value(fs[q], up[f] & 63);
                    u[q] = FINE || own ? w : u[q];
                }
        }
        if constexpr (FINE) others(b, u);
#pragma unroll
        for (int f = 2 * b; f < 2 * b + 2; ++f) {
            if (!FINE || !fine[f]) continue;
            int k = 0;
            if (listed) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (kLat<Q>.c[q][b] == (f & 1 ? -1 : 1)) u[q] = mean[k++][at];
                ++at;
            } else {
                const int32_t t0 = t[0], t1 = t[1], t2 = t[2], t3 = t[3];
                t += 4;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (kLat<Q>.c[q][b] == (f & 1 ? -1 : 1))
                        u[q] = F(0.25) * ((ld(q, t0) + ld(q, t1)) + (ld(q, t2) + ld(q, t3)));
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (kLat<Q>.c[q][b] != 0) acc[q] += fs[q] - u[q];
        if constexpr (!FINE) asm volatile("" ::: "memory");  // no further ahead than one axis
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) fs[q] = fs[q] - r * acc[q];
    double rho = 0.0, mx = 0.0, my = 0.0, mz = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const double v = double(fs[q]);
        rho += v;
        mx += double(kLat<Q>.c[q][0]) * v;
        my += double(kLat<Q>.c[q][1]) * v;
        mz += double(kLat<Q>.c[q][2]) * v;
    }
    if (!(rho > 0.0)) *a.flag = 1;
    const double ux = mx / rho, uy = my / rho, uz = mz / rho;
    const double uu = ux * ux + uy * uy + uz * uz;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const double cu = kLat<Q>.c[q][0] * ux + kLat<Q>.c[q][1] * uy + kLat<Q>.c[q][2] * uz;
        const double feq = kLat<Q>.w[q] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu);
        const double v = double(fs[q]);
        const double out = a.euler ? v + a.relax * (feq - v) : feq + (v - feq) * a.relax;
        if constexpr (BUF)
            impl::bst<F, 0>(ro, uint32_t(c) * uint32_t(sizeof(F)), uint32_t(q) * uint32_t(n) * uint32_t(sizeof(F)), F(out));
        else
            fo[q * n + c] = F(out);
    }
}

// moments (rho, rho u, E = sum |c|^2 f / 2) of every cell, and the cell's
// volume-weighted contribution summed per block (first stage of the global sums)
template <typename F, int Q>
__global__ __launch_bounds__(256) void k_lbm_moments(const F *f, const LbmCell *cells, int64_t n, double h0,
                                                     double *mom, double *partials) {
    __shared__ double red[4 * 5];
    const int64_t c = int64_t(blockIdx.x) * 256 + threadIdx.x;
    double v[5] = {0, 0, 0, 0, 0};
    if (c < n) {
        double m[5] = {0, 0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const double x = double(f[q * n + c]);
            const int cx = kLat<Q>.c[q][0], cy = kLat<Q>.c[q][1], cz = kLat<Q>.c[q][2];
            m[0] += x;
            m[1] += cx * x;
            m[2] += cy * x;
            m[3] += cz * x;
            m[4] += 0.5 * double(cx * cx + cy * cy + cz * cz) * x;
        }
        for (int k = 0; k < 5; ++k) mom[k * n + c] = m[k];
        const double h = h0 / double(1u << (cells[c].meta >> 24));
        for (int k = 0; k < 5; ++k) v[k] = h * h * h * m[k];
    }
    impl::block_sum<256, 5>(v, red);
    if (threadIdx.x == 0)
        for (int k = 0; k < 5; ++k) partials[blockIdx.x * 5 + k] = v[k];
}

__global__ __launch_bounds__(256) void k_lbm_sums(const double *partials, int nb, double *out) {
    __shared__ double red[4 * 5];
    double v[5] = {0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < nb; b += 256)
        for (int k = 0; k < 5; ++k) v[k] += partials[b * 5 + k];
    impl::block_sum<256, 5>(v, red);
    if (threadIdx.x == 0)
        for (int k = 0; k < 5; ++k) out[k] = v[k];
}

// f_eq of (rho, u) per cell: prim [4][n]
template <typename F, int Q>
__global__ __launch_bounds__(256) void k_lbm_init(const double *prim, F *f, int64_t n, int *flag) {
    const int64_t c = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (c >= n) return;
    const double rho = prim[c], ux = prim[n + c], uy = prim[2 * n + c], uz = prim[3 * n + c];
    if (!(rho > 0.0)) *flag = 1;
    const double uu = ux * ux + uy * uy + uz * uz;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const double cu = kLat<Q>.c[q][0] * ux + kLat<Q>.c[q][1] * uy + kLat<Q>.c[q][2] * uz;
        f[q * n + c] = F(kLat<Q>.w[q] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu));
    }
}

// population-major [Q][n] <-> canonical [n][27] (corners zero for D3Q19): the
// rows of kCanonCells cells are turned in LDS so that both sides of the copy
// run over consecutive addresses (the odd row length of 27 spreads a
// population's column over the banks); D3Q19 FP32 on 996,150 cells: 311 us with
// each thread writing its cell's row, 35 us
constexpr int kCanonCells = 128;
template <typename F, int Q>
__global__ __launch_bounds__(256) void k_lbm_canon(const F *src, F *dst, int64_t n, int to_canon) {
    __shared__ F tile[kCanonCells * 27];
    const int64_t c0 = int64_t(blockIdx.x) * kCanonCells;
    const int nc = int(min(int64_t(kCanonCells), n - c0));
    const int cl = threadIdx.x & (kCanonCells - 1), half = threadIdx.x / kCanonCells;
    if (to_canon) {
        if (Q < 27)
            for (int i = threadIdx.x; i < kCanonCells * 27; i += 256) tile[i] = F(0);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int k = (kLat<Q>.c[q][0] + 1) * 9 + (kLat<Q>.c[q][1] + 1) * 3 + (kLat<Q>.c[q][2] + 1);
            if ((q & 1) == half && cl < nc) tile[cl * 27 + k] = src[q * n + c0 + cl];
        }
        __syncthreads();
        for (int i = threadIdx.x; i < nc * 27; i += 256) dst[c0 * 27 + i] = tile[i];
    } else {
        for (int i = threadIdx.x; i < nc * 27; i += 256) tile[i] = src[c0 * 27 + i];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int k = (kLat<Q>.c[q][0] + 1) * 9 + (kLat<Q>.c[q][1] + 1) * 3 + (kLat<Q>.c[q][2] + 1);
            if ((q & 1) == half && cl < nc) dst[q * n + c0 + cl] = tile[cl * 27 + k];
        }
    }
}

template <typename F, int Q>
hipError_t run(const char *what, const LbmArgs &a, const void *p0, void *p1, double *p2, double *p3, int64_t n,
               double h0, int flagmode, hipStream_t st) {
    const dim3 g{unsigned((n + 255) / 256), 1, 1}, blk{256, 1, 1};
    switch (what[0]) {
    case 's':
        if (uint64_t(Q) * uint64_t(n) * sizeof(F) < (uint64_t(1) << 32)) {
            if (a.any_fine) hipLaunchKernelGGL((k_lbm<F, Q, true, true>), g, blk, 0, st, a);
            else hipLaunchKernelGGL((k_lbm<F, Q, true, false>), g, blk, 0, st, a);
        } else {
            if (a.any_fine) hipLaunchKernelGGL((k_lbm<F, Q, false, true>), g, blk, 0, st, a);
            else hipLaunchKernelGGL((k_lbm<F, Q, false, false>), g, blk, 0, st, a);
        }
        break;
    case 'm':
        hipLaunchKernelGGL((k_lbm_moments<F, Q>), g, blk, 0, st, static_cast<const F *>(p0), a.cells, n, h0, p2, p3);
        break;
    case 'i':
        hipLaunchKernelGGL((k_lbm_init<F, Q>), g, blk, 0, st, static_cast<const double *>(p0), static_cast<F *>(p1),
                           n, a.flag);
        break;
    default:
        hipLaunchKernelGGL((k_lbm_canon<F, Q>), dim3(unsigned((n + kCanonCells - 1) / kCanonCells)), blk, 0, st,
                           static_cast<const F *>(p0), static_cast<F *>(p1), n, flagmode);
        break;
    }
    return hipGetLastError();
}

template <int Q>
hipError_t run_prec(bool fp64, const char *what, const LbmArgs &a, const void *p0, void *p1, double *p2, double *p3,
                    int64_t n, double h0, int flagmode, hipStream_t st) {
    return fp64 ? run<double, Q>(what, a, p0, p1, p2, p3, n, h0, flagmode, st)
                : run<float, Q>(what, a, p0, p1, p2, p3, n, h0, flagmode, st);
}

hipError_t dispatch(int q, bool fp64, const char *what, const LbmArgs &a, const void *p0, void *p1, double *p2,
                    double *p3, int64_t n, double h0, int flagmode, hipStream_t st) {
    if (q == 19) return run_prec<19>(fp64, what, a, p0, p1, p2, p3, n, h0, flagmode, st);
    if (q == 27) return run_prec<27>(fp64, what, a, p0, p1, p2, p3, n, h0, flagmode, st);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_lbm_step(int q, bool fp64, const LbmArgs &a, hipStream_t st) {
    return dispatch(q, fp64, "step", a, nullptr, nullptr, nullptr, nullptr, a.n, a.h0, 0, st);
}

hipError_t launch_lbm_moments(int q, bool fp64, const void *f, const LbmCell *cells, int64_t n, double h0,
                              double *mom, double *partials, double *sums, hipStream_t st) {
    LbmArgs a{};
    a.cells = cells;
    hipError_t e = dispatch(q, fp64, "moments", a, f, nullptr, mom, partials, n, h0, 0, st);
    if (e != hipSuccess || !sums) return e;
    hipLaunchKernelGGL(k_lbm_sums, dim3(1), dim3(256), 0, st, partials, int((n + 255) / 256), sums);
    return hipGetLastError();
}

hipError_t launch_lbm_init(int q, bool fp64, const double *prim, void *f, int64_t n, int *flag, hipStream_t st) {
    LbmArgs a{};
    a.flag = flag;
    return dispatch(q, fp64, "init", a, prim, f, nullptr, nullptr, n, 0.0, 0, st);
}

hipError_t launch_lbm_canon(int q, bool fp64, const void *src, void *dst, int64_t n, bool to_canon, hipStream_t st) {
    LbmArgs a{};
    return dispatch(q, fp64, "canon", a, src, dst, nullptr, nullptr, n, 0.0, to_canon ? 1 : 0, st);
}

}  // namespace dvm
