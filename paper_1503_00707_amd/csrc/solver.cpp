// solver.cpp -- host side of the solver: argument checks, buffer layout,
// kernel launches on the caller's stream.  Holds no device memory of its own:
// every buffer is bound by the caller (dvm_bind).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

#include "solver_impl.h"

using namespace dvm;

namespace {
// The FP64 default at 24^3 nodes, shape (192, 21): the regular cells with 192
// threads at two waves per SIMD in one launch and the others with 576 at five
// in a second.  Regular cells hold three times the loads in flight per wave
// that way (27,000 of them: 2,014 -> 1,578 us); the correction pass over the
// four rows behind a FINER face wants the wide workgroup (30,400 cells, 16 %
// with such faces: one launch at 576 threads 2,614 us, at 192 threads 4 %
// more, two launches 2,351).  FP32 keeps one launch: 420,251 cells 12.5 ms
// against 14.0.
bool two_shapes(const dvm_solver *s, const StepConfig &cfg) {
    return has_two_shapes(s) && is_two_shapes(cfg.threads, cfg.wpe);
}

// two launches (reduced kernel over the regular cells, full kernel over the
// rest) instead of one: first order, kernels compiled
bool use_split(const dvm_solver *s, const StepConfig &cfg) {
    return s->split && !s->muscl && s->n_reg > 0 &&
           (two_shapes(s, cfg) || have_regular_kernel(s->nh, cfg.threads, cfg.wpe)) &&
           have_kernel(s->nh, s->cfg_irr.threads, s->cfg_irr.wpe);
}

// the regular cells (at least one) in shape cfg's reduced kernel, the others in
// shape irr
hipError_t launch_pair(const dvm_solver *s, const StepArgs &a, const StepConfig &cfg, ShapeId irr, hipStream_t st) {
    StepConfig c = cfg;  // stores and grouping as chosen; each launch its own shape
    c.regular = 1;
    StepArgs part = a;
    part.sel = s->sel();
    part.n_sel = s->n_reg;
    hipError_t e = launch_step(s->fp64, part, c, st);
    if (e != hipSuccess || s->n == s->n_reg) return e;
    c.regular = 0;
    c.threads = irr.threads;
    c.wpe = irr.wpe;
    part.sel = s->sel() + s->n_reg;
    part.n_sel = s->n - s->n_reg;
    return launch_step(s->fp64, part, c, st);
}
}  // namespace

void dvm::default_grouping(StepConfig &c, const dvm_solver *s, int64_t n, double state_bytes) {
    const int nh = s->nh;
    // Consecutive cells share upwind rows, so each XCD takes runs of them.
    // Group 1 / 64 on 30,400 cells FP64: 16^3 nodes 700 / 565 us, 12^3 329 /
    // 294, 8^3 101 / 83; FP32 8^3, 243,200 cells: 421 / 365.  24^3 nodes: runs
    // of 32, by time alone (FP32, 420,251 cells, 512 / 128 / 32 / 8: 12.51 /
    // 12.37 / 12.31 / 12.73 ms, though the shorter runs read more past the L2:
    // 996,150 cells 122 GB at 512, 138 at 32; 3,800 cells, 512 / 16: 175 / 141
    // us; FP64, 30,400 cells, 64 / 32: 2,340 / 2,317 us).  A round over the
    // XCDs has to fit the mesh: at most n / 8 (4,200 meshes of 40 to 4,000
    // cells, all grids: 6 % faster than without runs, 4 % of them slower by more
    // than 1.5 %; n / 16 and n / 32 worse).  Below 100 cells every cell has a
    // compute unit, and runs gain 1 % or lose up to 10: none.  FP64 24^3 in one
    // launch of few rounds over the compute units: 64 (512 to 1,536 cells, 900
    // meshes: 32 takes 2 % less on average, but up to 30 % more).
    const bool few = has_two_shapes(s) && !runs_as_pair(s) && n >= 512;
    int64_t g = n < 100 ? 1 : nh == 12 && !few ? 32 : 64;
    g = std::min(g, std::max<int64_t>(1, n / 8));
    c.xcd_group = 1;
    while (2 * c.xcd_group <= g) c.xcd_group *= 2;
    // Stores: non-temporal once the two state buffers exceed the 256 MB Infinity
    // Cache.  Below that plain ones leave the next step its rows there, but what
    // they write back is paid for when other states step in between.  One state
    // over and over, non-temporal / plain, then three in turn, us: FP64 16^3,
    // 3,800 cells, 84 / 75; FP32 12^3, 12,167 cells, 56.4 / 47.8, 56.2 / 60.3;
    // 24^3, 1,728 cells, 57.7 / 52.0, 58.0 / 61.9; 16^3, 5,832 cells, 50.6 /
    // 46.5, 51.1 / 55.5; FP64 24^3, 818 cells, 93.4 / 87.6, 94.5 / 102.1.  The
    // last two had non-temporal stores at every size and keep them (in turn they
    // were up to 6 % slower without; FP64 24^3 below 40 MiB is not: 343 cells
    // 30.5 / 28.0).  FP32 from 12^3 on is also better off with them where a
    // buffer is less than the XCDs' L2s (24^3, 343 cells of 18 MB, 18.4 / 19.7;
    // 12^3, 1,320 of 9 MB, 12.6 / 14.0).
    const double mb = state_bytes / double(1 << 20);
    c.nt_store = mb > 128.0 || (s->fp64 ? nh == 12 && mb > 40.0 : nh == 8 || (nh >= 6 && mb < 24.0));
}

// On few cells the pair costs more than it gives: two launches one after the
// other, neither of which fills the card (one launch at 576 threads / the pair,
// us; 27 cells between walls 19 / 35, 209 cells with jumps 31.5 / 49.4, 581: 57
// / 64, 1,057: 100 / 96, 1,452 between walls 112 / 121, 1,583: 147 / 142, 2,255:
// 214 / 197).  Without other cells there is no second launch: 216 cells 20.0 /
// 21.0, 343: 32.7 / 27.9.  The one launch holds five waves per EU where there is
// more than a workgroup for each compute unit (729 cells between walls 60.7 us
// against 63.5, 27 cells 16.9 against 16.7).
bool dvm::runs_as_pair(const dvm_solver *s) {
    return s->n_reg > 0 && s->n > (s->n_reg == s->n ? 256 : 1536);
}

hipError_t dvm::launch_shape(const dvm_solver *s, const StepArgs &a, const StepConfig &cfg, hipStream_t st) {
    if (!two_shapes(s, cfg)) return launch_step(s->fp64, a, cfg, st);
    if (runs_as_pair(s)) return launch_pair(s, a, cfg, ShapeId{576, 51}, st);
    StepConfig one = cfg;
    one.threads = kOneShape.threads;
    one.wpe = s->n > 256 ? 51 : kOneShape.wpe;
    return launch_step(s->fp64, a, one, st);
}

StepArgs dvm::solver_step_args(const dvm_solver *s, double dt) {
    StepArgs a{};
    a.mom = s->mom;
    a.cells = s->tables;
    a.ghost_in = s->gin();
    a.wall_m1 = s->m1();
    a.wall_den = s->den();
    a.flag = s->flag();
    a.n_cells = s->n;
    a.dt = dt;
    a.h0 = s->m->h0;
    a.dt_h0 = dt / s->m->h0;
    a.g = s->g;
    // the Korobov collision runs as its own kernel after a transport-only step
    a.collision = s->korobov() ? DVM_COLL_OFF : s->p.collision;
    a.tau_mode = s->p.tau_mode;
    a.tau_or_kn = s->p.tau_or_kn;
    a.xcd_log2 = 0;
    while ((1 << (a.xcd_log2 + 1)) <= s->cfg.xcd_group) ++a.xcd_log2;
    a.muscl = s->muscl ? 1 : 0;
    return a;
}

hipError_t dvm::solver_state_replaced(dvm_solver *s, hipStream_t st) {
    hipError_t e = solver_reset_hybrid(s, st);
    if (e == hipSuccess) e = launch_moments(s->fp64, s->f[s->cur], s->mom, s->n, s->g, st);
    s->hybrid_fluid = false;
    return e;
}

double dvm::solver_max_speed_sum(const dvm_solver *s) {
    double r = 0.0;
    for (int b = 0; b < 3; ++b) r += (s->nh - 0.5) * s->g.dv[b];
    return r;
}

extern "C" {

int dvm_create_solver(const dvm_mesh *m, const dvm_params *p, dvm_solver **out) {
    clear_error();
    if (!m || !p || !out) return fail(DVM_ERR_ARG, "null argument");
    *out = nullptr;
    if (p->nv < 2 || p->nv % 2) return fail(DVM_ERR_UNSUPPORTED, "nv = %d: the device path needs an even N", p->nv);
    for (int b = 0; b < 3; ++b)
        if (!(p->vmax[b] > 0)) return fail(DVM_ERR_ARG, "vmax[%d] must be > 0", b);
    if (p->precision != DVM_PREC_FP64 && p->precision != DVM_PREC_FP32) return fail(DVM_ERR_ARG, "bad precision");
    if (p->scheme != DVM_SCHEME_UPWIND1 && p->scheme != DVM_SCHEME_MUSCL) return fail(DVM_ERR_ARG, "bad scheme");
    if (p->collision < DVM_COLL_EXP || p->collision > DVM_COLL_KOROBOV) return fail(DVM_ERR_ARG, "bad collision mode");
    if (p->tau_mode != DVM_TAU_CONST && p->tau_mode != DVM_TAU_HS) return fail(DVM_ERR_ARG, "bad tau mode");
    if (p->fluid_flux != DVM_FLUX_GRID && p->fluid_flux != DVM_FLUX_CLOSED) return fail(DVM_ERR_ARG, "bad fluid_flux");
    if (p->collision != DVM_COLL_OFF && !(p->tau_or_kn > 0)) return fail(DVM_ERR_ARG, "tau_or_kn must be > 0");
    const bool fp64 = p->precision == DVM_PREC_FP64;
    const int nh = p->nv / 2;
    const int thr = default_threads(fp64, nh);
    if (!thr) return fail(DVM_ERR_UNSUPPORTED, "no device kernel for N = %d (have 4, 8, 12, 16, 24)", p->nv);
    int64_t kor_a = 0;
    if (p->collision == DVM_COLL_KOROBOV) {
        if (!korobov_supported(nh)) return fail(DVM_ERR_UNSUPPORTED, "Korobov collision kernel for N = 4, 8, 12 only");
        if (p->hybrid) return fail(DVM_ERR_UNSUPPORTED, "the hybrid step relaxes with BGK");
        if (p->vmax[0] != p->vmax[1] || p->vmax[0] != p->vmax[2])
            return fail(DVM_ERR_UNSUPPORTED, "Korobov collision on a cubic velocity box only");
        const int64_t gen = korobov_generator(p->korobov_p);
        if (gen < 0) return fail(DVM_ERR_ARG, "korobov_p = %d must be a prime in [5, 2^31)", p->korobov_p);
        kor_a = p->korobov_a ? p->korobov_a : gen;
        if (kor_a < 1 || kor_a >= p->korobov_p) return fail(DVM_ERR_ARG, "korobov_a must be in [1, p)");
    }
    dvm_solver *s = new (std::nothrow) dvm_solver();
    if (!s) return fail(DVM_ERR_ARG, "out of host memory");
    s->m = m;
    s->p = *p;
    s->fp64 = fp64;
    s->nh = nh;
    s->nv = int64_t(p->nv) * p->nv * p->nv;
    s->n = int64_t(m->cells.size());
    s->g.nh = nh;
    s->g.w = 1.0;
    for (int b = 0; b < 3; ++b) {
        s->g.dv[b] = 2.0 * p->vmax[b] / p->nv;
        s->g.w *= s->g.dv[b];
    }
    // measured defaults per (precision, N); dvm_tune_set overrides them
    s->cfg.threads = thr;
    s->cfg.wpe = 0;
    if (nh == 12 && !fp64) {
        s->cfg.threads = 192;
        s->cfg.wpe = 31;
    }
    if ((nh == 6 || nh == 8) && !fp64) {
        // 12^3 and 16^3: per-cell fixed work (reductions, the Maxwellian
        // system) dominates, and two waves per cell keep more cells in flight
        s->cfg.threads = 128;
        s->cfg.wpe = nh == 6 ? 60 : 50;
    }
    if (nh == 12 && fp64) {
        const ShapeId d = p->scheme == DVM_SCHEME_MUSCL ? kOneShape : kTwoShapes;
        s->cfg.threads = d.threads;
        s->cfg.wpe = d.wpe;
    }
    if (m->device_tables) {
        // no solid leaves: domain faces are the only INFLOW / WALL faces
        for (int f = 0; f < 6; ++f) {
            s->has_inflow |= m->bc[f] == DVM_BC_INFLOW;
            s->has_wall |= m->bc[f] == DVM_BC_WALL;
        }
    } else {
        s->has_inflow = m->n_faces[DVM_FACE_INFLOW] > 0;
        s->has_wall = m->n_faces[DVM_FACE_WALL] > 0;
    }
    const size_t fs = fp64 ? 8 : 4;
    s->f_bytes = align256(size_t(s->n) * size_t(s->nv) * fs);
    s->mom_bytes = align256(size_t(5) * size_t(s->n) * 8);
    s->tab_bytes = align256(size_t(s->n) * sizeof(DevCell));
    size_t o = 0;
    s->off_gin = o;  o += align256(size_t(s->nv) * fs);
    s->off_m1 = o;   o += align256(size_t(s->nv) * fs);
    s->off_den = o;  o += align256(6 * 8);
    s->off_flag = o; o += 256;
    s->off_part = o; o += align256(size_t(kPartials) * 5 * 8);
    s->off_sums = o; o += 256;
    s->muscl = p->scheme == DVM_SCHEME_MUSCL;
    s->off_kor = o;
    if (p->collision == DVM_COLL_KOROBOV) {
        s->kor_p = p->korobov_p;
        s->kor_a = kor_a;
        std::vector<int32_t> J, L, M;
        korobov_tables(p->nv, p->vmax[0], s->kor_p, s->kor_a, J, L, M);
        korobov_plan(nh, p->vmax[0], J, L, M, s->kor_p, s->kor);
        o += align256(s->kor.host.size());
    }
    s->hybrid = p->hybrid != 0;
    s->off_hyb = o;
    if (s->hybrid)
        o += 3 * align256(size_t(s->n)) + align256(size_t(s->n) * kFluxRecord * 8) +
             align256(size_t(s->n) * kFaceRecord * 8);
    // selection list: regular cells (no FINER or WALL face) first, then the rest
    s->off_sel = o;  o += align256(size_t(s->n) * 4);
    if (!m->device_tables) s->sel_host.reserve(size_t(s->n));
    for (int pass = 0; pass < 2 && !m->device_tables; ++pass)
        for (int64_t c = 0; c < s->n; ++c) {
            const DevCell &d = m->table[size_t(c)];
            bool irregular = false;
            for (int f = 0; f < 6; ++f) irregular |= d.type[f] == DVM_FACE_FINER || d.type[f] == DVM_FACE_WALL;
            if (irregular == (pass == 1)) s->sel_host.push_back(uint32_t(c));
            if (pass == 0 && !irregular) ++s->n_reg;
        }
    default_grouping(s->cfg, s, s->n, s->state_bytes());
    // the second launch's shape: one with a full kernel, which the pair has not
    s->cfg_irr = s->cfg;
    if (two_shapes(s, s->cfg)) {
        s->cfg_irr.threads = kOneShape.threads;
        s->cfg_irr.wpe = kOneShape.wpe;
    }
    s->ws_bytes = o;
    *out = s;
    return DVM_OK;
}

int dvm_buffer_sizes(const dvm_solver *s, dvm_sizes *out) {
    clear_error();
    if (!s || !out) return fail(DVM_ERR_ARG, "null argument");
    out->f_bytes = s->f_bytes;
    out->moments_bytes = s->mom_bytes;
    out->tables_bytes = s->tab_bytes;
    out->ws_bytes = s->ws_bytes;
    out->n_cells = s->n;
    out->nv_total = s->nv;
    return DVM_OK;
}

int dvm_bind(dvm_solver *s, void *f_a, void *f_b, double *moments, void *tables, void *ws) {
    clear_error();
    if (!s) return fail(DVM_ERR_ARG, "null solver");
    void *ptrs[5] = {f_a, f_b, moments, tables, ws};
    for (void *q : ptrs) {
        if (!q) return fail(DVM_ERR_WORKSPACE, "a buffer is NULL");
        if (reinterpret_cast<uintptr_t>(q) & 255) return fail(DVM_ERR_ARG, "buffers must be 256-byte aligned");
    }
    if (f_a == f_b) return fail(DVM_ERR_ARG, "the two state buffers must differ");
    s->f[0] = f_a;
    s->f[1] = f_b;
    s->cur = 0;
    s->mom = moments;
    s->tables = static_cast<DevCell *>(tables);
    s->ws = static_cast<char *>(ws);
    s->uploaded = false;
    s->tables_pending = false;
    s->steps = 0;
    return DVM_OK;
}

int dvm_upload(dvm_solver *s, void *stream) {
    clear_error();
    if (!s || !s->ws) return fail(DVM_ERR_WORKSPACE, "solver not bound");
    hipStream_t st = S(stream);
    const bool dev_tab = s->m->device_tables;
    hipError_t e = hipSuccess;
    if (!dev_tab) {
        e = hipMemcpyAsync(s->tables, s->m->table.data(), s->m->table.size() * sizeof(DevCell),
                           hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(tables)");
    }
    e = hipMemsetAsync(s->ws, 0, s->ws_bytes, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemsetAsync(ws)");
    if (!dev_tab) {
        e = hipMemcpyAsync(s->ws + s->off_sel, s->sel_host.data(), s->sel_host.size() * 4, hipMemcpyHostToDevice,
                           st);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(selection)");
    }
    InitArgs a{};
    a.prim = nullptr;
    a.n = 1;
    a.g = s->g;
    a.flag = s->flag();
    a.mom = nullptr;
    if (s->has_inflow) {
        for (int k = 0; k < 5; ++k) a.prim0[k] = s->p.inflow[k];
        a.f_out = s->gin();
        e = launch_init(s->fp64, a, st);
        if (e != hipSuccess) return hip_fail(e, "inflow ghost");
    }
    if (s->has_wall) {
        const double pw[5] = {1.0, 0.0, 0.0, 0.0, s->p.t_wall};
        for (int k = 0; k < 5; ++k) a.prim0[k] = pw[k];
        a.f_out = s->m1();
        e = launch_init(s->fp64, a, st);
        if (e != hipSuccess) return hip_fail(e, "wall Maxwellian");
        e = launch_wall_den(s->fp64, s->m1(), s->den(), s->g, st);
        if (e != hipSuccess) return hip_fail(e, "wall denominators");
    }
    if (s->korobov()) {
        e = hipMemcpyAsync(s->ws + s->off_kor, s->kor.host.data(), s->kor.host.size(), hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return hip_fail(e, "Korobov table");
    }
    e = solver_reset_hybrid(s, st);
    if (e != hipSuccess) return hip_fail(e, "hybrid masks");
    s->hybrid_fluid = false;
    {
        int dev = 0;
        e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&s->n_cu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return hip_fail(e, "device attributes");
    }
    // the host table must stay valid until the copy has been consumed
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    // a device-table mesh is ready once dvm_adapt_tables has built its tables
    s->uploaded = !dev_tab;
    s->tables_pending = dev_tab;
    return DVM_OK;
}

int dvm_init_maxwellian(dvm_solver *s, const double *prim, void *stream) {
    clear_error();
    if (!s || !prim) return fail(DVM_ERR_ARG, "null argument");
    if (!s->uploaded) return fail(DVM_ERR_WORKSPACE, "call dvm_upload first");
    InitArgs a{};
    a.prim = prim;
    a.n = s->n;
    a.g = s->g;
    a.flag = s->flag();
    a.mom = s->mom;
    s->cur = 0;
    a.f_out = s->f[0];
    hipError_t e = launch_init(s->fp64, a, S(stream));
    if (e != hipSuccess) return hip_fail(e, "init");
    e = solver_reset_hybrid(s, S(stream));
    if (e != hipSuccess) return hip_fail(e, "hybrid masks");
    s->hybrid_fluid = false;
    s->steps = 0;
    return DVM_OK;
}

int dvm_dt(const dvm_solver *s, double cfl, double *dt) {
    clear_error();
    if (!s || !dt) return fail(DVM_ERR_ARG, "null argument");
    if (!(cfl > 0)) return fail(DVM_ERR_ARG, "cfl must be > 0");
    *dt = cfl * s->m->h_min / solver_max_speed_sum(s);
    return DVM_OK;
}

int dvm_step(dvm_solver *s, int32_t n_steps, double dt, double cfl, void *stream) {
    clear_error();
    if (!s) return fail(DVM_ERR_ARG, "null solver");
    if (!s->uploaded) return fail(DVM_ERR_WORKSPACE, "call dvm_upload first");
    if (n_steps < 0) return fail(DVM_ERR_ARG, "n_steps < 0");
    if (s->hybrid_fluid)
        return fail(DVM_ERR_UNSUPPORTED, "fluid cells hold no f: continue with dvm_hybrid_step (an all-ones mask "
                                         "turns every cell kinetic)");
    if (!(dt > 0)) {
        int rc = dvm_dt(s, cfl, &dt);
        if (rc) return rc;
    }
    StepArgs a = solver_step_args(s, dt);
    hipStream_t st = S(stream);
    hipError_t e = hipSuccess;
    for (int it = 0; it < n_steps; ++it) {
        a.f_in = s->f[s->cur];
        a.f_out = s->f[s->cur ^ 1];
        e = use_split(s, s->cfg) ? launch_pair(s, a, s->cfg, ShapeId{s->cfg_irr.threads, s->cfg_irr.wpe}, st)
                                 : launch_shape(s, a, s->cfg, st);
        if (e != hipSuccess) return hip_fail(e, "step");
        if (s->korobov()) {
            KorArgs k{};
            k.f = a.f_out;
            const char *plan = s->ws + s->off_kor;
            k.node = reinterpret_cast<const int32_t *>(plan + s->kor.node);
            k.row = reinterpret_cast<const int32_t *>(plan + s->kor.row);
            k.gain_len = reinterpret_cast<const int32_t *>(plan + s->kor.gain_len);
            k.gain_at = reinterpret_cast<const int32_t *>(plan + s->kor.gain_at);
            k.gain = reinterpret_cast<const uint64_t *>(plan + s->kor.gain);
            k.freq = s->kor.matrix ? reinterpret_cast<const double *>(plan + s->kor.freq) : nullptr;
            k.pair = reinterpret_cast<const uint32_t *>(plan + s->kor.pair);
            k.n_cells = s->n;
            k.p = int(s->kor_p);
            k.w0 = 8.0 * s->p.vmax[0] * s->p.vmax[0] * s->p.vmax[0] / double(s->kor_p);
            k.dt_kn = dt / s->p.tau_or_kn;
            k.vmax = s->p.vmax[0];
            k.g = s->g;
            k.flag = s->flag();
            e = launch_korobov(s->fp64, k, st);
            if (e != hipSuccess) return hip_fail(e, "Korobov collision");
        }
        s->cur ^= 1;
        s->steps++;
        if (s->p.check_every > 0 && s->steps % s->p.check_every == 0) {
            e = launch_global_sums(s->mom, s->tables, s->n, s->m->h0, s->partials(), kPartials, s->sums(), st);
            if (e != hipSuccess) return hip_fail(e, "global sums");
        }
    }
    return DVM_OK;
}

int dvm_global_sums(dvm_solver *s, void *stream) {
    clear_error();
    if (!s) return fail(DVM_ERR_ARG, "null solver");
    if (!s->uploaded) return fail(DVM_ERR_WORKSPACE, "call dvm_upload first");
    hipError_t e = launch_global_sums(s->mom, s->tables, s->n, s->m->h0, s->partials(), kPartials, s->sums(), S(stream));
    if (e != hipSuccess) return hip_fail(e, "global sums");
    return DVM_OK;
}

int dvm_current_f(const dvm_solver *s, void **f) {
    clear_error();
    if (!s || !f) return fail(DVM_ERR_ARG, "null argument");
    *f = s->f[s->cur];
    return DVM_OK;
}

int dvm_moments(dvm_solver *s, double *out, void *stream) {
    clear_error();
    if (!s || !out) return fail(DVM_ERR_ARG, "null argument");
    if (!s->f[0]) return fail(DVM_ERR_WORKSPACE, "solver not bound");
    if (s->hybrid_fluid && out == s->mom)
        return fail(DVM_ERR_ARG, "after hybrid steps the moments buffer holds the fluid cells' state: pass "
                                 "another output buffer");
    hipError_t e = launch_moments(s->fp64, s->f[s->cur], out, s->n, s->g, S(stream));
    // fluid cells of a hybrid step carry only their conserved moments
    if (e == hipSuccess) e = solver_fluid_moments(s, out, S(stream));
    if (e != hipSuccess) return hip_fail(e, "moments");
    return DVM_OK;
}

int dvm_check(dvm_solver *s, void *stream, dvm_diag *out) {
    clear_error();
    if (!s || !out) return fail(DVM_ERR_ARG, "null argument");
    if (!s->uploaded) return fail(DVM_ERR_WORKSPACE, "call dvm_upload first");
    hipStream_t st = S(stream);
    hipError_t e = launch_global_sums(s->mom, s->tables, s->n, s->m->h0, s->partials(), kPartials, s->sums(), st);
    if (e != hipSuccess) return hip_fail(e, "global sums");
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    int flag = 0;
    e = hipMemcpy(out->sums, s->sums(), 5 * sizeof(double), hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(&flag, s->flag(), sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpy(diag)");
    out->nonphysical = flag != 0;
    out->steps = s->steps;
    if (flag) return fail(DVM_ERR_NONPHYSICAL, "a cell reached rho <= 0, T <= 0 or NaN");
    return DVM_OK;
}

int dvm_f_to_canonical(const dvm_solver *s, const void *f_internal, void *f_canon, void *stream) {
    clear_error();
    if (!s || !f_internal || !f_canon) return fail(DVM_ERR_ARG, "null argument");
    hipError_t e = launch_to_canonical(s->fp64, true, f_internal, f_canon, s->n, s->nh, S(stream));
    if (e != hipSuccess) return hip_fail(e, "to_canonical");
    return DVM_OK;
}

int dvm_f_from_canonical(dvm_solver *s, const void *f_canon, void *f_internal, void *stream) {
    clear_error();
    if (!s || !f_internal || !f_canon) return fail(DVM_ERR_ARG, "null argument");
    hipError_t e = launch_to_canonical(s->fp64, false, f_canon, f_internal, s->n, s->nh, S(stream));
    if (e != hipSuccess) return hip_fail(e, "from_canonical");
    if (f_internal == s->f[s->cur] && s->uploaded) {
        // the buffer holds a new state: its moments, fresh hybrid masks
        e = launch_moments(s->fp64, f_internal, s->mom, s->n, s->g, S(stream));
        if (e != hipSuccess) return hip_fail(e, "moments");
        e = solver_reset_hybrid(s, S(stream));
        if (e != hipSuccess) return hip_fail(e, "hybrid masks");
        s->hybrid_fluid = false;
    }
    return DVM_OK;
}

int dvm_tune_shapes(const dvm_solver *s, int32_t *threads, int32_t *wpe, int32_t cap, int32_t *n) {
    clear_error();
    if (!s || !n || (cap > 0 && (!threads || !wpe))) return fail(DVM_ERR_ARG, "null argument");
    int t[64], w[64];
    const int total = list_shapes(s, t, w, 64);
    for (int k = 0; k < total && k < cap && k < 64; ++k) {
        threads[k] = t[k];
        wpe[k] = w[k];
    }
    *n = total;
    return DVM_OK;
}

int dvm_tune_set(dvm_solver *s, int32_t threads, int32_t wpe, int32_t xcd_group, int32_t nt_store) {
    clear_error();
    if (!s) return fail(DVM_ERR_ARG, "null solver");
    if (xcd_group < 1 || xcd_group > 4096 || (xcd_group & (xcd_group - 1)))
        return fail(DVM_ERR_ARG, "xcd_group must be a power of two in [1, 4096]");
    if (!have_shape(s, threads, wpe))
        return fail(DVM_ERR_UNSUPPORTED, "no step kernel with %d threads, wpe %d for N = %d", threads, wpe, 2 * s->nh);
    s->cfg.threads = threads;
    s->cfg.wpe = wpe;
    s->cfg.xcd_group = xcd_group;
    s->cfg.nt_store = nt_store != 0;
    s->cfg_default = false;
    return DVM_OK;
}

int dvm_tune_get(const dvm_solver *s, int32_t *threads, int32_t *wpe, int32_t *xcd_group, int32_t *nt_store) {
    clear_error();
    if (!s || !threads || !wpe || !xcd_group || !nt_store) return fail(DVM_ERR_ARG, "null argument");
    *threads = s->cfg.threads;
    *wpe = s->cfg.wpe;
    *xcd_group = s->cfg.xcd_group;
    *nt_store = s->cfg.nt_store;
    return DVM_OK;
}

int dvm_tune_split(dvm_solver *s, int32_t enable, int32_t threads_irr, int32_t wpe_irr, int32_t *previous) {
    clear_error();
    if (!s) return fail(DVM_ERR_ARG, "null solver");
    if (previous) *previous = s->split ? 1 : 0;
    if (enable < 0) return DVM_OK;
    if (threads_irr > 0) {
        if (!have_kernel(s->nh, threads_irr, wpe_irr))
            return fail(DVM_ERR_UNSUPPORTED, "no step kernel with %d threads, wpe %d for N = %d", threads_irr, wpe_irr,
                        2 * s->nh);
        s->cfg_irr.threads = threads_irr;
        s->cfg_irr.wpe = wpe_irr;
    }
    s->split = enable != 0;
    return DVM_OK;
}

void dvm_destroy_solver(dvm_solver *s) { delete s; }

}  // extern "C"
