// korobov.hip -- the Boltzmann collision integral on Korobov lattice nodes
// (section 3.2, eqs. 3-6) applied in place to the post-transport state:
//   B_i = sum_k W f_j            (eq. 4, collision frequency)
//   C_i = sum_k W f_l f_m        (eq. 5, inverse-collision integral)
//   I_i = -f_i P_i B_i + C_i     (eq. 6, conservative correction)
//   f'_i = f_i + (dt / Kn) I_i,  W = V_box |xi_j - xi_i| / p.
// The trials are the same for every cell.  A workgroup takes a tile of CELLS
// cells whose rows sit in LDS node-major ([node][cell]), so the gather of one
// node for all cells of the tile is one contiguous vector read.  The LDS gathers
// bound it (three of every trial, two thirds of their cycles bank conflicts, took
// 931 us for 16^3 cells, 8^3 nodes, p = 1021 in FP64; 355 us now), so no trial
// gathers what it need not:
//   C runs over lists of the trials that have a gain term (61 % of them at 8^3),
//     the nodes ordered by the length of their list so that the 64 nodes of a
//     wave end together; an entry carries the two node indices and
//     n = |k_j - k_i|^2 in grid units, W = w0 dv sqrt(n) a lookup in LDS;
//   B is linear in f with coefficients that no cell changes, a dense matrix on
//     the small grids (two trials per entry at 8^3 and p = 1021): FP64 matrix
//     cores, 16 nodes x the tile's cells at a time.  On 12^3 nodes the matrix is
//     sparse and its product costs more than the gathers, which stay.
// The lists and the nodes' rows are arranged on the host so that the lanes whose
// reads are served together mostly start on different bank groups (korobov.cpp):
// 1.6 cycles per 16 lanes at 8^3 and p = 1021 against 3 and more in lattice
// order; without the arrangement the same kernel takes 576 us.
// The five coefficients of P solve the conservation system in the scaled basis
// (1, xi/v, |xi|^2/v^2), v = the grid's half width (the span of eq. 6's (1, xi,
// |xi|^2): the same P), assembled from FP64 workgroup sums.
// The paper's own kernel runs one thread block per velocity node over all
// cells, f stored velocity-major and transposed for the correction; here the
// tables stream through L2 once per tile and f is never transposed.
// Not free of scratch: the solve's 5 x 5 arrays lie there, and the shapes of
// eight cells a thread spill some 30 of 128 registers (384 B a lane).
#include <hip/hip_runtime.h>

#include "step_impl.h"

namespace dvm {
namespace impl {
namespace {

template <int NH>
__device__ __forceinline__ void node_velocity(int v, const VelGrid &g, double xi[3]) {
    constexpr int B = NH * NH * NH;
    const int o = v / B, s = v % B;
    const int ax = s / (NH * NH), ay = (s / NH) % NH, az = s % NH;
    xi[0] = ((o >> 2) ? 1.0 : -1.0) * (ax + 0.5) * g.dv[0];
    xi[1] = (((o >> 1) & 1) ? 1.0 : -1.0) * (ay + 0.5) * g.dv[1];
    xi[2] = ((o & 1) ? 1.0 : -1.0) * (az + 0.5) * g.dv[2];
}

// Gauss elimination with partial pivoting of a 5x5 system (one thread)
__device__ inline bool solve5(double A[5][5], double r[5], double x[5]) {
    for (int c = 0; c < 5; ++c) {
        int piv = c;
        for (int q = c + 1; q < 5; ++q)
            if (fabs(A[q][c]) > fabs(A[piv][c])) piv = q;
        if (A[piv][c] == 0.0) return false;
        if (piv != c) {
            for (int k = 0; k < 5; ++k) {
                const double t = A[c][k];
                A[c][k] = A[piv][k];
                A[piv][k] = t;
            }
            const double t = r[c];
            r[c] = r[piv];
            r[piv] = t;
        }
        for (int q = c + 1; q < 5; ++q) {
            const double m = A[q][c] / A[c][c];
            for (int k = c; k < 5; ++k) A[q][k] -= m * A[c][k];
            r[q] -= m * r[c];
        }
    }
    for (int q = 4; q >= 0; --q) {
        double s = r[q];
        for (int k = q + 1; k < 5; ++k) s -= A[q][k] * x[k];
        x[q] = s / A[q][q];
    }
    return true;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// NV nodes in R rounds of NV / R threads, G groups of such threads with CPT cells
// of the tile each.  MAT: B by the matrix product (one round).
template <typename F, int NH, int R, int G, int CPT, bool MAT, int WPE>
__global__ __launch_bounds__(8 * NH * NH * NH / R * G) __attribute__((amdgpu_waves_per_eu(WPE, 8))) void k_korobov(
    KorArgs a) {
    constexpr int NV = 8 * NH * NH * NH, NT = NV / R, T = NT * G, CELLS = G * CPT, NWN = NT / 64;
    constexpr int NW = 3 * (2 * NH - 1) * (2 * NH - 1) + 1;
    static_assert(NV % R == 0 && NT % 64 == 0, "whole nodes per thread, whole waves");
    static_assert(!MAT || (R == 1 && CELLS <= 16), "one round, one tile of columns");
    // a node's row of the tile, padded to an odd number of 16-byte groups: rows
    // whose nodes differ modulo 16 start on different bank groups (the lists are
    // arranged for that).  Rows of one group (FP32, four cells) take three all the
    // same: 512 cells x 12^3 nodes 355 us, 371 with rows of one, 100 x 8^3 177
    // against 183
    constexpr int RS = (CELLS * int(sizeof(F)) / 16 % 2 ? CELLS + 32 / int(sizeof(F)) : CELLS + 16 / int(sizeof(F)));
    constexpr int RB = CELLS + 2;
    constexpr size_t kTile = size_t(NV) * RS * sizeof(F), kB = MAT ? size_t(NV) * RB * 8 : 0;
    __shared__ __align__(16) char tile[kTile > kB ? kTile : kB];
    __shared__ double Wn[NW];
    __shared__ double red[(T / 64) * CPT * 20];
    __shared__ double dco[CELLS][5];
    F *fs = reinterpret_cast<F *>(tile);
    double *bs = reinterpret_cast<double *>(tile);  // B, once the tile has been read
    F *f = static_cast<F *>(a.f);
    const int64_t c0 = int64_t(blockIdx.x) * CELLS;
    const int nc = int(min(int64_t(CELLS), a.n_cells - c0));
    for (int e = threadIdx.x; e < NV * CELLS; e += T) {
        const int c = e / NV, v = e % NV;
        fs[a.row[v] * RS + c] = c < nc ? f[(c0 + c) * NV + v] : F(0);
    }
    const double wd = a.w0 * a.g.dv[0];
    for (int q = threadIdx.x; q < NW; q += T) Wn[q] = wd * sqrt(double(q));
    __syncthreads();
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int t = threadIdx.x % NT, cg = (threadIdx.x / NT) * CPT;  // node slot, first cell
    int node[R], row[R];
    double b[R][CPT], cc[R][CPT];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        node[r] = a.node[t + r * NT];
        row[r] = a.row[node[r]];
#pragma unroll
        for (int c = 0; c < CPT; ++c) b[r][c] = cc[r][c] = 0.0;
    }
    // eq. 5: each list entry once per tile, applied to every cell of it; four
    // entries are in flight while the four before them are used
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int wave = __builtin_amdgcn_readfirstlane((t >> 6) + r * NWN);
        const int len = a.gain_len[wave];
        const uint64_t *tab = a.gain + a.gain_at[wave] + lane;
        uint64_t e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = tab[k * 64];
        for (int k0 = 0; k0 < len; k0 += 4) {
            tab += 4 * 64;  // (the table ends with one entry group more)
            uint64_t next[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) next[k] = tab[k * 64];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int l = int(e[k] & 0xFFFFu), m = int((e[k] >> 16) & 0xFFFFu);
                const double W = Wn[int(e[k] >> 32)];
                F fl[CPT], fm[CPT];
                __builtin_memcpy(fl, fs + l * RS + cg, sizeof fl);
                __builtin_memcpy(fm, fs + m * RS + cg, sizeof fm);
#pragma unroll
                for (int c = 0; c < CPT; ++c) cc[r][c] += W * double(fl[c]) * double(fm[c]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) e[k] = next[k];
        }
    }
    // eq. 4
    F fv[R][CPT];
#pragma unroll
    for (int r = 0; r < R; ++r) __builtin_memcpy(fv[r], fs + row[r] * RS + cg, sizeof fv[r]);
    if constexpr (MAT) {
        // lane l, g = l / 16: A[l % 16][g], B[g][l % 16], result D[g + 4 v][l % 16];
        // a row block's coefficients lie in that order, two steps of the
        // contraction a load
        constexpr int NB = NV / 16, PER = (NB + T / 64 - 1) / (T / 64);
        static_assert(NB % PER == 0, "whole row blocks per wave");
        const int li = lane & 15, g = lane >> 4;
        const bool on = wid * PER < NB;
        const double2 *A = reinterpret_cast<const double2 *>(a.freq) + size_t(wid) * PER * (NV / 8) * 64 + lane;
        f64x4 acc[PER];
#pragma unroll
        for (int x = 0; x < PER; ++x) acc[x] = f64x4{0, 0, 0, 0};
        if (on) {
#pragma unroll 4
            for (int s = 0; s < NV / 8; ++s) {
                const double f0 = li < CELLS ? double(fs[(8 * s + g) * RS + li]) : 0.0;
                const double f1 = li < CELLS ? double(fs[(8 * s + 4 + g) * RS + li]) : 0.0;
#pragma unroll
                for (int x = 0; x < PER; ++x) {
                    const double2 w = A[(size_t(x) * (NV / 8) + s) * 64];
                    acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.x, f0, acc[x], 0, 0, 0);
                    acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.y, f1, acc[x], 0, 0, 0);
                }
            }
        }
        __syncthreads();  // every wave has read the tile
        if (on && li < CELLS) {
#pragma unroll
            for (int x = 0; x < PER; ++x)
#pragma unroll
                for (int v = 0; v < 4; ++v) bs[((wid * PER + x) * 16 + g + 4 * v) * RB + li] = acc[x][v];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < CPT; ++c) b[0][c] = bs[t * RB + cg + c];
    } else {
        for (int k = 0; k < a.p; ++k) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t e = a.pair[size_t(k) * NV + r * NT + t];
                F fj[CPT];
                __builtin_memcpy(fj, fs + int(e & 0xFFFFu) * RS + cg, sizeof fj);
                const double W = Wn[int(e >> 16)];
#pragma unroll
                for (int c = 0; c < CPT; ++c) b[r][c] += W * double(fj[c]);
            }
        }
    }
    // eq. 6: per cell the 5x5 conservation system in the scaled basis
    const double iv = 1.0 / a.vmax;
    double psi[R][5];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        double xi[3];
        node_velocity<NH>(node[r], a.g, xi);
        psi[r][0] = 1.0;
        psi[r][1] = xi[0] * iv;
        psi[r][2] = xi[1] * iv;
        psi[r][3] = xi[2] * iv;
        psi[r][4] = (xi[0] * xi[0] + xi[1] * xi[1] + xi[2] * xi[2]) * iv * iv;
    }
    // per cell 20 sums (15 of the symmetric matrix, 5 of the right side):
    // wave sums into LDS, then one barrier, the wave totals, and one thread
    // per cell solves its system
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        double s[20];
#pragma unroll
        for (int q = 0; q < 20; ++q) s[q] = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double fb = double(fv[r][c]) * b[r][c];
            const double rr = cc[r][c] - fb;
            int q = 0;
#pragma unroll
            for (int x = 0; x < 5; ++x)
#pragma unroll
                for (int y = x; y < 5; ++y) s[q++] += psi[r][x] * psi[r][y] * fb;
#pragma unroll
            for (int x = 0; x < 5; ++x) s[15 + x] += psi[r][x] * rr;
        }
#pragma unroll
        for (int q = 0; q < 20; ++q) {
            const double x = wave_sum(s[q]);
            if (lane == 0) red[(wid * CPT + c) * 20 + q] = x;
        }
    }
    __syncthreads();
    if (threadIdx.x < CELLS && int(threadIdx.x) < nc) {
        const int c = threadIdx.x, w0 = c / CPT * NWN;
        double sm[20];
        for (int q = 0; q < 20; ++q) {
            double x = 0.0;
            for (int w = 0; w < NWN; ++w) x += red[((w0 + w) * CPT + c % CPT) * 20 + q];
            sm[q] = x;
        }
        double A[5][5], rv[5], d[5] = {0, 0, 0, 0, 0};
        int q = 0;
        for (int x = 0; x < 5; ++x)
            for (int y = x; y < 5; ++y) A[x][y] = A[y][x] = sm[q++];
        for (int x = 0; x < 5; ++x) rv[x] = sm[15 + x];
        if (!solve5(A, rv, d)) *a.flag = 1;
        for (int x = 0; x < 5; ++x) dco[c][x] = d[x];
    }
    __syncthreads();
    // the new rows back into the tile, for whole-line stores
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const double d0 = dco[cg + c][0], d1 = dco[cg + c][1], d2 = dco[cg + c][2], d3 = dco[cg + c][3],
                     d4 = dco[cg + c][4];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double P = 1.0 + d0 + (d1 * psi[r][1] + d2 * psi[r][2] + d3 * psi[r][3]) + d4 * psi[r][4];
            const double x = double(fv[r][c]);
            const double I = -x * P * b[r][c] + cc[r][c];
            fs[row[r] * RS + cg + c] = F(x + a.dt_kn * I);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NV * nc; e += T) {
        const int c = e / NV, v = e % NV;
        f[(c0 + c) * NV + v] = fs[a.row[v] * RS + c];
    }
}

}  // namespace
}  // namespace impl

// Cells per tile: 16 where the tiles still cover three quarters of the compute
// units, so that the lists and the matrix are read once for more cells; fewer
// below, down to 4, so that a small mesh spreads (8^3 nodes, FP64: 2,028 cells,
// p = 1021 in tiles of 8, 498 -> 228 us; 100 cells in tiles of 4, 522 -> 170 us).
template <typename F, int NH, int R, int G, int CPT, bool MAT, int WPE>
static hipError_t run(const KorArgs &a, hipStream_t st) {
    constexpr int CELLS = G * CPT;
    hipLaunchKernelGGL((impl::k_korobov<F, NH, R, G, CPT, MAT, WPE>), dim3(unsigned((a.n_cells + CELLS - 1) / CELLS)),
                       dim3(8 * NH * NH * NH / R * G), 0, st, a);
    return hipGetLastError();
}

template <typename F>
static hipError_t korobov_dispatch(const KorArgs &a, hipStream_t st) {
    const int64_t tiles16 = (a.n_cells + 15) / 16;
    const bool mat = a.freq != nullptr;
    switch (a.g.nh) {
    case 2:
        if (!mat) return run<F, 2, 1, 2, 4, false, 3>(a, st);
        return tiles16 >= 256 ? run<F, 2, 1, 4, 4, true, 3>(a, st) : run<F, 2, 1, 2, 4, true, 3>(a, st);
    case 4:
        if (!mat) return tiles16 >= 192 ? run<F, 4, 1, 2, 8, false, 4>(a, st) : run<F, 4, 1, 1, 4, false, 3>(a, st);
        if (tiles16 >= 192) return run<F, 4, 1, 2, 8, true, 4>(a, st);
        return tiles16 >= 96 ? run<F, 4, 1, 1, 8, true, 3>(a, st) : run<F, 4, 1, 1, 4, true, 3>(a, st);
    case 6: return run<F, 6, 3, 1, 4, false, 3>(a, st);
    default: return hipErrorInvalidValue;
    }
}

bool korobov_supported(int nh) { return nh == 2 || nh == 4 || nh == 6; }

hipError_t launch_korobov(bool fp64, const KorArgs &a, hipStream_t st) {
    return fp64 ? korobov_dispatch<double>(a, st) : korobov_dispatch<float>(a, st);
}

}  // namespace dvm
