// korobov.cpp -- host side of the Boltzmann collision integral on Korobov
// lattice nodes (section 3.2, eqs. 3-6): the lattice generator, the per-node
// trial tables shared by every cell (eqs. 3-5: "the same for all points of
// [physical] space"), their export for tests.
//
// Tables.  For velocity node i (canonical index) and trial k = 0..p-1 of a
// p-point rank-1 Korobov lattice in 5 dimensions (generator a):
//   q_d = (k a^d + s_d(i)) mod p,  s_d(i) = (i + 1) c_d mod p,
//   c_d = (2654435761 mod p)(d + 1) mod p,                       d = 0..4,
//   partner node j_b = floor((q_b + 1/2) N_b / p)                 b = 0, 1, 2,
//   direction cos(theta) = 1 - 2 (q_3 + 1/2)/p,  phi = 2 pi (q_4 + 1/2)/p,
//   post-collision velocities c +- (|g|/2) n, c = (xi_i + xi_j)/2, g = xi_j - xi_i,
//   each in the node whose velocity cell holds it (none: the trial has no
//   gain term).  Node velocities are lo + (k + 1/2) d per axis, FP64.
// The device's form of them is korobov_plan's, in its own velocity order
// (internal octant-major index).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "solver_impl.h"

using namespace dvm;

namespace {

bool prime(int64_t p) {
    if (p < 2) return false;
    for (int64_t q = 2; q * q <= p; ++q)
        if (p % q == 0) return false;
    return true;
}

// P_2 figure of merit of the 5-dimensional lattice of generator a; factor(z)
// that of a coordinate z / p
template <class Factor>
double p2_merit(int64_t p, int64_t a, const Factor &factor) {
    int64_t step[5], z[5] = {0, 0, 0, 0, 0};
    step[0] = 1;
    for (int d = 1; d < 5; ++d) step[d] = step[d - 1] * a % p;
    double sum = 0.0;
    for (int64_t k = 0; k < p; ++k) {
        double prod = 1.0;
        for (int d = 0; d < 5; ++d) {
            prod *= factor(z[d]);
            z[d] += step[d];
            if (z[d] >= p) z[d] -= p;
        }
        sum += prod;
    }
    return sum / double(p) - 1.0;
}

template <class Factor>
int64_t best_generator(int64_t p, const Factor &factor) {
    int64_t best = -1;
    double best_v = 0.0;
    for (int64_t a = 2; a < p; ++a) {
        const double v = p2_merit(p, a, factor);
        // a, -a, 1/a, -1/a (mod p) span the same lattice up to the order and
        // sign of coordinates: equal merit; the first of a tie wins
        if (best < 0 || v < best_v - 1e-9 * std::fabs(best_v)) {
            best = a;
            best_v = v;
        }
    }
    return best;
}

// internal (octant-major) index of canonical node (kx, ky, kz)
int64_t internal_of(int nh, int kx, int ky, int kz) {
    const int sx = kx >= nh, sy = ky >= nh, sz = kz >= nh;
    const int ax = sx ? kx - nh : nh - 1 - kx, ay = sy ? ky - nh : nh - 1 - ky, az = sz ? kz - nh : nh - 1 - kz;
    const int64_t B = int64_t(nh) * nh * nh;
    return int64_t((sx << 2) | (sy << 1) | sz) * B + (int64_t(ax) * nh + ay) * nh + az;
}

}  // namespace

namespace dvm {

int64_t korobov_generator(int64_t p) {
    if (!prime(p) || p < 5 || p >= (int64_t(1) << 31)) return -1;
    const double two_pi2 = 2.0 * M_PI * M_PI;
    const auto factor = [&](int64_t z) {
        const double x = double(z) / double(p);
        return 1.0 + two_pi2 * (x * x - x + 1.0 / 6.0);
    };
    if (p > (int64_t(1) << 20)) return best_generator(p, factor);
    std::vector<double> table(static_cast<size_t>(p));
    for (int64_t z = 0; z < p; ++z) table[size_t(z)] = factor(z);
    return best_generator(p, [&](int64_t z) { return table[size_t(z)]; });
}

// canonical-index tables [i][k] (j, l, m; -1 for no gain term)
void korobov_tables(int n, double vmax, int64_t p, int64_t a, std::vector<int32_t> &J, std::vector<int32_t> &L,
                    std::vector<int32_t> &M) {
    const int64_t nv = int64_t(n) * n * n;
    J.assign(size_t(nv * p), 0);
    L.assign(size_t(nv * p), -1);
    M.assign(size_t(nv * p), -1);
    const double lo = -vmax, d = (vmax - lo) / n;
    std::vector<double> x(static_cast<size_t>(n));
    for (int k = 0; k < n; ++k) x[size_t(k)] = lo + (k + 0.5) * d;
    int64_t ap[5], c[5];
    ap[0] = 1;
    for (int e = 1; e < 5; ++e) ap[e] = ap[e - 1] * a % p;
    for (int e = 0; e < 5; ++e) c[e] = (int64_t(2654435761ll % p) * (e + 1)) % p;
    // what depends on one lattice coordinate alone, once per value of it
    std::vector<int64_t> ka(static_cast<size_t>(5 * p));   // k a^e mod p
    std::vector<int> jq(static_cast<size_t>(p));           // partner's axis index
    std::vector<double> ctv(static_cast<size_t>(p)), stv(static_cast<size_t>(p)), cv(static_cast<size_t>(p)),
        sv(static_cast<size_t>(p));
    for (int64_t q = 0; q < p; ++q) {
        for (int e = 0; e < 5; ++e) ka[size_t(e * p + q)] = q * ap[e] % p;
        jq[size_t(q)] = int(((2 * q + 1) * n) / (2 * p));
        const double ct = 1.0 - 2.0 * ((double(q) + 0.5) / double(p)), ph = 2.0 * M_PI * ((double(q) + 0.5) / double(p));
        ctv[size_t(q)] = ct;
        stv[size_t(q)] = std::sqrt(std::fmax(0.0, 1.0 - ct * ct));
        cv[size_t(q)] = std::cos(ph);
        sv[size_t(q)] = std::sin(ph);
    }
    auto cell_of = [&](double v) -> int {
        const double t = (v - lo) / d;
        return t >= 0.0 && t < double(n) ? int(t) : -1;
    };
    for (int64_t i = 0; i < nv; ++i) {
        const int ix = int(i / (int64_t(n) * n)), iy = int((i / n) % n), iz = int(i % n);
        const double xi[3] = {x[size_t(ix)], x[size_t(iy)], x[size_t(iz)]};
        int64_t s[5];
        for (int e = 0; e < 5; ++e) s[e] = ((i + 1) % p) * c[e] % p;
        for (int64_t k = 0; k < p; ++k) {
            int64_t q[5];
            for (int e = 0; e < 5; ++e) {
                q[e] = ka[size_t(e * p + k)] + s[e];
                if (q[e] >= p) q[e] -= p;
            }
            int jb[3];
            for (int b = 0; b < 3; ++b) jb[b] = jq[size_t(q[b])];
            const double xs[3] = {x[size_t(jb[0])], x[size_t(jb[1])], x[size_t(jb[2])]};
            const double gx = xs[0] - xi[0], gy = xs[1] - xi[1], gz = xs[2] - xi[2];
            const double gg = std::sqrt(gx * gx + gy * gy + gz * gz);
            const double st = stv[size_t(q[3])];
            const double nn[3] = {st * cv[size_t(q[4])], st * sv[size_t(q[4])], ctv[size_t(q[3])]};
            int l1[3], l2[3];
            bool ok = true;
            for (int b = 0; b < 3; ++b) {
                const double cb = 0.5 * (xi[b] + xs[b]);
                l1[b] = cell_of(cb + 0.5 * gg * nn[b]);
                l2[b] = cell_of(cb - 0.5 * gg * nn[b]);
                ok = ok && l1[b] >= 0 && l2[b] >= 0;
            }
            const size_t e = size_t(i * p + k);
            J[e] = int32_t((int64_t(jb[0]) * n + jb[1]) * n + jb[2]);
            if (ok) {
                L[e] = int32_t((int64_t(l1[0]) * n + l1[1]) * n + l1[2]);
                M[e] = int32_t((int64_t(l2[0]) * n + l2[1]) * n + l2[2]);
            }
        }
    }
}

namespace {

struct Entry {
    uint16_t x, y;  // rows that a list entry gathers
    uint32_t d2;
};

// The lanes of a wave whose 16-byte LDS reads are served together: 0-3, 12-15,
// 20-23, 24-27; the others of the first 32; the same of the last 32 (lists
// arranged for 16 consecutive lanes run slower than unarranged ones).
inline int phase_lane(int phase, int t) {
    static const uint8_t first[2][16] = {{0, 1, 2, 3, 12, 13, 14, 15, 20, 21, 22, 23, 24, 25, 26, 27},
                                         {4, 5, 6, 7, 8, 9, 10, 11, 16, 17, 18, 19, 28, 29, 30, 31}};
    return (phase >> 1) * 32 + first[phase & 1][t];
}

// Order the lists of 16 lanes that are served together so that the rows
// gathered in one step start on different LDS bank groups: rows lie an odd
// number of 16-byte groups apart, so that 16 rows are free of conflicts when
// their indices differ modulo 16.  Greedy: each lane takes, among the residues
// (of x, of y) that no other lane has in this step, one it has most of.  Steps
// beyond a lane's list get entries of weight 0 on free residues.
// PAIR: the lists of partners, one row an entry (x = y).
template <bool PAIR>
void arrange(const std::vector<Entry> *lists, int64_t len, std::vector<Entry> *out) {
    // entries left of residue r, with the smaller residue first among equals,
    // as one number: (left << 4) + 15 - r
    struct Lane {
        std::vector<Entry> e;                          // sorted by residue pair
        int64_t row[16], col[PAIR ? 1 : 256];          // of x; of y under each x
        int32_t next[PAIR ? 16 : 256];
        uint32_t rows, cols[16];                       // which of them are left
    };
    constexpr size_t NB = PAIR ? 16 : 256;
    const auto bucket = [](const Entry &e) { return PAIR ? size_t(e.x & 15) : size_t((e.x & 15) * 16 + (e.y & 15)); };
    std::vector<Lane> lane(16);
    for (int t = 0; t < 16; ++t) {
        Lane &z = lane[size_t(t)];
        int32_t at[NB + 1] = {0};
        for (const Entry &e : lists[t]) at[bucket(e) + 1]++;
        z.rows = 0;
        for (int r = 0; r < 16; ++r) {
            z.row[r] = 15 - r;
            z.cols[r] = 0;
        }
        for (size_t q = 0; q < NB; ++q) {
            const size_t x = PAIR ? q : q >> 4;
            const int64_t left = at[q + 1];
            z.row[x] += left * 16;
            if constexpr (!PAIR) z.col[q] = left * 16 + 15 - int64_t(q & 15);
            if (left) {
                z.rows |= 1u << x;
                if (!PAIR) z.cols[x] |= 1u << (q & 15);
            }
            at[q + 1] += at[q];
            z.next[q] = at[q];
        }
        z.e.resize(lists[t].size());
        for (const Entry &e : lists[t]) z.e[size_t(at[bucket(e)]++)] = e;
        out[t].clear();
        out[t].reserve(size_t(len));
    }
    // the residue of which a lane has most, among those in `of`
    const auto most = [](uint32_t of, const int64_t *key) {
        int64_t best = -1;
        for (; of; of &= of - 1) best = std::max(best, key[__builtin_ctz(of)]);
        return best < 0 ? -1 : int(15 - (best & 15));
    };
    for (int64_t k = 0; k < len; ++k) {
        uint32_t ux = 0, uy = 0;
        for (int q = 0; q < 16; ++q) {
            const int t = int((q + k) & 15);
            Lane &z = lane[size_t(t)];
            Entry take{0, 0, 0};
            if (k < int64_t(lists[t].size())) {
                int x = -1, y = -1;
                for (uint32_t of = z.rows & ~ux; of && y < 0;) {
                    x = most(of, z.row);
                    of &= ~(1u << x);
                    y = PAIR ? x : most(z.cols[x] & ~uy, z.col + (PAIR ? 0 : 16 * x));
                }
                if (y < 0) {  // no pair is free: any that is left
                    x = __builtin_ctz(z.rows);
                    const uint32_t of = z.cols[x] & ~uy;
                    y = PAIR ? x : __builtin_ctz(of ? of : z.cols[x]);
                }
                const int b = PAIR ? x : 16 * x + y;
                if constexpr (!PAIR)
                    if ((z.col[b] -= 16) < 16) z.cols[x] &= ~(1u << y);
                if ((z.row[x] -= 16) < 16) z.rows &= ~(1u << x);
                take = z.e[size_t(z.next[b]++)];
            } else {
                take.x = uint16_t(ux == 0xffffu ? 0 : __builtin_ctz(~ux));
                take.y = uint16_t(uy == 0xffffu ? 0 : __builtin_ctz(~uy));
            }
            ux |= 1u << (take.x & 15);
            uy |= 1u << (take.y & 15);
            out[t].push_back(take);
        }
    }
}

}  // namespace

// Device form: the nodes sorted by decreasing number of trials with a gain
// term (slots); per 64 slots the lists of those trials side by side, as long as
// the longest of the 64 rounded up to four, each 16 of them arranged against
// bank conflicts; the frequency's matrix, or the partner lists, in slot order.
void korobov_plan(int nh, double vmax, const std::vector<int32_t> &J, const std::vector<int32_t> &L,
                  const std::vector<int32_t> &M, int64_t p, KorPlan &out) {
    const int n = 2 * nh;
    const int64_t nv = int64_t(n) * n * n;
    std::vector<int32_t> to_int(static_cast<size_t>(nv));
    for (int kx = 0; kx < n; ++kx)
        for (int ky = 0; ky < n; ++ky)
            for (int kz = 0; kz < n; ++kz)
                to_int[size_t((int64_t(kx) * n + ky) * n + kz)] = int32_t(internal_of(nh, kx, ky, kz));
    // |k_j - k_i|^2 in node units: |xi_j - xi_i| = dv sqrt(n) on the cubic grid
    std::vector<int32_t> axis(static_cast<size_t>(3 * nv));
    for (int64_t i = 0; i < nv; ++i) {
        axis[size_t(3 * i)] = int32_t(i / (n * n));
        axis[size_t(3 * i + 1)] = int32_t((i / n) % n);
        axis[size_t(3 * i + 2)] = int32_t(i % n);
    }
    const auto dist2 = [&](int64_t i, int64_t j) {
        const int32_t *a = &axis[size_t(3 * i)], *b = &axis[size_t(3 * j)];
        const int32_t dx = b[0] - a[0], dy = b[1] - a[1], dz = b[2] - a[2];
        return uint32_t(dx * dx + dy * dy + dz * dz);
    };
    std::vector<int32_t> count(static_cast<size_t>(nv)), slot(static_cast<size_t>(nv));  // slot s holds canonical node slot[s]
    for (int64_t i = 0; i < nv; ++i) {
        slot[size_t(i)] = int32_t(i);
        for (int64_t k = 0; k < p; ++k) count[size_t(i)] += L[size_t(i * p + k)] >= 0;
    }
    std::stable_sort(slot.begin(), slot.end(), [&](int32_t x, int32_t y) { return count[size_t(x)] > count[size_t(y)]; });
    // LDS row of each (canonical) node: nodes by how often the lists gather them,
    // dealt to the 16 residues in turn there and back, so that every residue has
    // its share (slow velocities are gathered most, and neighbours in any plain
    // order of the nodes)
    std::vector<int32_t> often(static_cast<size_t>(nv)), by(static_cast<size_t>(nv)), row(static_cast<size_t>(nv));
    for (int64_t e = 0; e < nv * p; ++e)
        if (L[size_t(e)] >= 0) {
            often[size_t(L[size_t(e)])]++;
            often[size_t(M[size_t(e)])]++;
        }
    for (int64_t i = 0; i < nv; ++i) by[size_t(i)] = int32_t(i);
    std::stable_sort(by.begin(), by.end(), [&](int32_t x, int32_t y) { return often[size_t(x)] > often[size_t(y)]; });
    for (int64_t q = 0; q < nv; ++q)
        row[size_t(by[size_t(q)])] = int32_t((q / 16) * 16 + ((q / 16) % 2 ? 15 - q % 16 : q % 16));
    const size_t groups = size_t(nv / 64);
    std::vector<int32_t> len(groups), at(groups);
    size_t entries = 0;
    for (size_t g = 0; g < groups; ++g) {
        len[g] = (count[size_t(slot[64 * g])] + 3) / 4 * 4;
        at[g] = int32_t(entries);
        entries += size_t(len[g]) * 64;
    }
    entries += 4 * 64;  // the kernel reads one group of four ahead
    out.matrix = korobov_matrix(nh, p);
    size_t o = 0;
    const auto take = [&](size_t bytes) {
        const size_t x = o;
        o += align256(bytes);
        return x;
    };
    out.node = take(size_t(nv) * 4);
    out.row = take(size_t(nv) * 4);
    out.gain_len = take(groups * 4);
    out.gain_at = take(groups * 4);
    out.gain = take(entries * 8);
    out.freq = take(out.matrix ? size_t(nv) * size_t(nv) * 8 : 0);
    out.pair = take(out.matrix ? 0 : size_t(p) * size_t(nv) * 4);
    out.host.assign(o, 0);
    int32_t *node = reinterpret_cast<int32_t *>(out.host.data() + out.node);
    int32_t *rows = reinterpret_cast<int32_t *>(out.host.data() + out.row);
    for (int64_t s = 0; s < nv; ++s) node[s] = to_int[size_t(slot[size_t(s)])];
    for (int64_t i = 0; i < nv; ++i) rows[to_int[size_t(i)]] = row[size_t(i)];
    std::copy(len.begin(), len.end(), reinterpret_cast<int32_t *>(out.host.data() + out.gain_len));
    std::copy(at.begin(), at.end(), reinterpret_cast<int32_t *>(out.host.data() + out.gain_at));
    uint64_t *gain = reinterpret_cast<uint64_t *>(out.host.data() + out.gain);
    double *freq = reinterpret_cast<double *>(out.host.data() + out.freq);
    uint32_t *pair = reinterpret_cast<uint32_t *>(out.host.data() + out.pair);
    const double wd = 8.0 * vmax * vmax * vmax / double(p) * (2.0 * vmax / n);
    std::vector<Entry> list[16], put[16];
    for (int64_t q = 0; q < nv / 16; ++q) {
        const size_t g = size_t(q / 4);
        const auto slot_of = [&](int t) { return int64_t(64 * g) + phase_lane(int(q % 4), t); };
        for (int t = 0; t < 16; ++t) {
            const int64_t s = slot_of(t), i = slot[size_t(s)];
            list[t].clear();
            for (int64_t k = 0; k < p; ++k) {
                const size_t e = size_t(i * p + k);
                const uint32_t d2 = dist2(i, J[e]);
                if (L[e] >= 0)
                    list[t].push_back(Entry{uint16_t(row[size_t(L[e])]), uint16_t(row[size_t(M[e])]), d2});
                if (out.matrix) {
                    // row block s / 16, pair of steps j / 8, lane 16 (j % 4) + s % 16, step (j / 4) % 2 of the pair
                    const uint64_t j = uint64_t(row[size_t(J[e])]);
                    freq[((size_t(s / 16) * size_t(nv / 8) + j / 8) * 64 + 16 * (j % 4) + uint64_t(s % 16)) * 2 +
                         (j / 4) % 2] += wd * std::sqrt(double(d2));
                }
            }
        }
        arrange<false>(list, len[g], put);
        for (int64_t k = 0; k < len[g]; ++k)
            for (int t = 0; t < 16; ++t) {
                const Entry &e = put[t][size_t(k)];
                gain[size_t(at[g]) + size_t(k * 64 + slot_of(t) % 64)] =
                    uint64_t(e.x) | (uint64_t(e.y) << 16) | (uint64_t(e.d2) << 32);
            }
        if (out.matrix) continue;
        for (int t = 0; t < 16; ++t) {
            const int64_t i = slot[size_t(slot_of(t))];
            list[t].clear();
            for (int64_t k = 0; k < p; ++k) {
                const int32_t j = J[size_t(i * p + k)];
                const uint16_t r = uint16_t(row[size_t(j)]);
                list[t].push_back(Entry{r, r, dist2(i, j)});
            }
        }
        arrange<true>(list, p, put);
        for (int64_t k = 0; k < p; ++k)
            for (int t = 0; t < 16; ++t) {
                const Entry &e = put[t][size_t(k)];
                pair[size_t(k * nv + slot_of(t))] = uint32_t(e.x) | (e.d2 << 16);
            }
    }
}

}  // namespace dvm

extern "C" {

int dvm_korobov_generator(int64_t p, int64_t *a) {
    clear_error();
    if (!a) return fail(DVM_ERR_ARG, "null argument");
    *a = korobov_generator(p);
    if (*a < 0) return fail(DVM_ERR_ARG, "p = %lld must be a prime in [5, 2^31)", (long long)p);
    return DVM_OK;
}

int dvm_korobov_tables(int32_t nv, double vmax, int64_t p, int64_t a, int32_t *j, int32_t *l, int32_t *m) {
    clear_error();
    if (!j || !l || !m) return fail(DVM_ERR_ARG, "null argument");
    if (nv < 2 || nv > 256 || !(vmax > 0)) return fail(DVM_ERR_ARG, "bad velocity grid");
    if (!prime(p) || p < 5 || p >= (int64_t(1) << 31) || a < 1 || a >= p)
        return fail(DVM_ERR_ARG, "p must be a prime in [5, 2^31) and 1 <= a < p");
    std::vector<int32_t> J, L, M;
    korobov_tables(nv, vmax, p, a, J, L, M);
    std::copy(J.begin(), J.end(), j);
    std::copy(L.begin(), L.end(), l);
    std::copy(M.begin(), M.end(), m);
    return DVM_OK;
}

}  // extern "C"
