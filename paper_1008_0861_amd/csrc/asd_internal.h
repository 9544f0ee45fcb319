// Host-side internals of libasd (grid handle, sweep configurations).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/asd.h"
#include "../../include/asd_extra.h"
#include "asd_device.h"
#include "asd_launch.h"

// Launch shape of one sweep: waves per line (wpl, the solve's), lines per
// workgroup, segments per line (power of two), the compiled per-lane
// capacity MMAX, io (1 or 2): staging and stores run on io times the
// solve's waves, and the tile body (face slots, or cell slots with io = 1).
struct SweepCfg {
    int wpl = 1, lpw = 1, P = 2, mmax = 1, io = 1;
    int variant = asd::SWEEP_FACE_SLOTS;
    int lpl = 64;  // lanes of a wave per line: 64, or 32 (two lines per wave; face body, batches only)
    int nthreads() const { return lpl * wpl * io * lpw; }
};

// gfx950: 160 KiB of LDS per workgroup; keep 2 KiB for static shared data.
static constexpr size_t kLdsLimit = 160 * 1024 - 2048;

inline int pow2_floor(int v) {
    int p = 1;
    while (p * 2 <= v) p *= 2;
    return p;
}

inline int ilog2(int v) {
    int l = 0;
    while ((1 << (l + 1)) <= v) ++l;
    return l;
}

// LDS layout and bytes of a sweep launch (slot rows of the lpw lines and the
// interface-exchange buffers) for either tile body.
inline asd::TileLayout sweep_layout(int es, int ndim, int n, const SweepCfg& c, bool tw = false) {
    return c.variant == asd::SWEEP_CELL_SLOTS
               ? asd::tile_layout_cell(es, ndim, n, c.lpw, c.nthreads(), c.wpl, ilog2(c.P), c.mmax)
               : asd::tile_layout(es, n, c.lpw, c.nthreads(), c.wpl, ilog2(c.P), c.mmax, c.lpl, tw);
}
inline size_t sweep_lds(int es, int ndim, int n, const SweepCfg& c, bool tw = false) {
    return (size_t)sweep_layout(es, ndim, n, c, tw).total;
}

inline int sweep_threads_cap(int es, int mmax, int variant = asd::SWEEP_FACE_SLOTS) {
    return variant == asd::SWEEP_CELL_SLOTS ? asd::sweep_cell_max_threads(es, mmax) : asd::sweep_max_threads(es, mmax);
}

// Fill *out for a line of n cells.  want_wpl / want_lpw: 0 = heuristic.
// Returns false if no configuration fits.
inline bool choose_sweep_cfg_wpl(int es, int ndim, int n, bool chi, int wpl, int want_lpw, SweepCfg* out, int io = 1,
                                 int variant = asd::SWEEP_FACE_SLOTS);

inline bool choose_sweep_cfg(int es, int ndim, int n, bool chi, int want_wpl, int want_lpw, SweepCfg* out,
                             int io = 1, int variant = asd::SWEEP_FACE_SLOTS) {
    if (want_wpl > 0) return choose_sweep_cfg_wpl(es, ndim, n, chi, want_wpl, want_lpw, out, io, variant);
    // heuristic: the fewest waves per line that keep <= pref cells per lane;
    // otherwise the feasible shape with the fewest cells per lane
    const int pref = es == 8 ? 8 : 16;
    SweepCfg best;
    bool found = false;
    for (int wpl = 1; wpl <= 16; wpl *= 2) {
        SweepCfg c;
        if (!choose_sweep_cfg_wpl(es, ndim, n, chi, wpl, want_lpw, &c, 1, variant)) continue;
        if (c.mmax <= pref) {
            *out = c;
            return true;
        }
        if (!found || c.mmax < best.mmax) {
            best = c;
            found = true;
        }
    }
    if (found) *out = best;
    return found;
}

inline bool choose_sweep_cfg_wpl(int es, int ndim, int n, bool chi, int wpl, int want_lpw, SweepCfg* out, int io,
                                 int variant) {
    if (wpl < 1 || wpl > 16 || (wpl & (wpl - 1))) return false;
    if (io != 1 && io != 2) return false;
    if (variant != asd::SWEEP_FACE_SLOTS && variant != asd::SWEEP_CELL_SLOTS) return false;
    if (variant == asd::SWEEP_CELL_SLOTS && io != 1) return false;
    const int P = std::min(64 * wpl, pow2_floor(n));
    const int m = (n + P - 1) / P;
    int mmax = 1;
    while (mmax < m) mmax *= 2;
    if (mmax > 16) return false;
    const int cap = sweep_threads_cap(es, mmax, variant);
    const int tpl = 64 * wpl * io;  // threads per line
    if (tpl > cap) return false;
    SweepCfg c;
    c.wpl = wpl;
    c.P = P;
    c.mmax = mmax;
    c.io = io;
    c.variant = variant;
    c.lpw = want_lpw > 0 ? want_lpw : std::max(1, 256 / (64 * wpl));
    while (c.lpw > 1 && (tpl * c.lpw > cap || sweep_lds(es, ndim, n, c) > kLdsLimit)) c.lpw /= 2;
    if (tpl * c.lpw > cap) return false;
    if (sweep_lds(es, ndim, n, c) > kLdsLimit) return false;
    *out = c;
    return true;
}

// The launch shape of the two-solve launches (SWEEP_TWICE) for shape c:
// the face body with as many lines per workgroup as its LDS slots (twice as
// large) and its register budget allow.  False: it does not fit.
inline bool twice_cfg(int es, int ndim, int n, SweepCfg c, SweepCfg* out) {
    c.variant = asd::SWEEP_FACE_SLOTS;
    c.io = 1;
    const int cap = asd::sweep_twice_max_threads(es, c.mmax);
    while (c.lpw > 1 && (c.nthreads() > cap || sweep_lds(es, ndim, n, c, true) > kLdsLimit)) c.lpw /= 2;
    if (c.nthreads() > cap || sweep_lds(es, ndim, n, c, true) > kLdsLimit) return false;
    *out = c;
    return true;
}

// Lines that the workgroups on one CU hold at a time in shape c, by their LDS
// (160 KiB per CU in units of 1280 bytes; the reduction's static share added).
inline int resident_lines(int es, int ndim, int n, const SweepCfg& c) {
    const size_t unit = 1280, tile = (sweep_lds(es, ndim, n, c) + 384 + unit - 1) / unit * unit;
    return (int)(160 * 1024 / tile) * c.lpw;
}

// Default launch shape of a sweep of `lines` lines of n cells.  Each choice
// is the measured best over sizes (us per step, all sweeps alike).  units(l) is
// the number of lines of the busiest of the 256 CUs with l lines per workgroup.
// - Lines per workgroup: pieces of at most 16 bytes in the transposed store
//   (longer ones leave CUs idle or one workgroup per CU: FP32 1024^2 16.6 with
//   4 lines, 18.9 with 8), fewer where that keeps more CUs busy: l grows while
//   it costs at most a third more (FP32 256^2 7.0 with 1 line, 7.4 with 4), on
//   FP32 lines of more than 1024 cells less than that for the fourth (1536^2
//   39.0 with 2 lines, 41.0 with 4; 1792^2 41.4, 38.4).  FP64 lines of up to 512
//   cells take pieces of 32 bytes (432 x 1649 26.5, 28.0; 500 x 777 20.8, 22.0).
// - Rows that start on half lines of the cache (64 bytes) keep short pieces
//   together: at most 2 lines (FP32 2000^2 49.1, 53.3 with 4; 1904^2 46.1, 48.2),
//   and so do rows one element short of that (x sweep of 1936 x 1935 23, 28).
//   Rows that start anywhere need whole pieces, up to two thirds more load:
//   FP32 1403^2 35.8 with 4 lines, 47.9 with 2; 1210^2 33.3, 38.1.
// - FP32 body, above 1024 cells: cell slots while a CU holds six lines of them, or
//   all that it gets (1392^2 28.4 with 2 lines, face slots 33.7; 1536^2, four
//   lines, 49.6 and 39.1; 1344^2 with 4 lines per workgroup, four lines, 38.5 and
//   33.8), unless its last lines then leave it a third empty (2000 x 1200, eight
//   lines and six held, 39.9 and 36.2); on up to 1024 always (1024^2 16.6 against
//   19.1).
// - Waves per line: at most 8 cells per lane with cell slots up to 1024 cells, 16
//   above and with face slots.
// - FP64, up to 1024 cells: cell slots, on two waves from 7 of a lane's 8 cells up
//   (1024^2 22.0, face slots 27.0; 960^2 26.3, 29.5; 768^2 30.0, 24.6) or with at
//   most a line per CU (600 x 60 11.4, 11.8); on one wave while a CU holds all its
//   lines (512^2 12.7; 500 x 3000, twelve lines and eight held, 55.6, face 53.2).
// - FP64, 1025 to 2048: four waves and one line (1400^2 50.6, two waves and two
//   lines 66.1), but two and two where rows start off the half lines (1403^2
//   67.8, 83.2; 1100^2 52.1, 62.1) or every lane is nearly full, a CU has more than
//   two lines and none more for it (1920^2 78.0, 81.5; 1999 x 512 29.9, 28.2).  Longer lines: four waves (3000 x 300 40.5, eight
//   waves 47.3), eight where there is at most a line per CU (3000 x 100 25.0, 23.9), but for
//   the two-solve launches (256 x 4096 33.8, eight waves 40.5).
// - 3-D: FP32 cell slots and 4 lines (256^3 261, face slots 299; 200^3 142,
//   162), but face slots for lines of 65 to 127 cells, which leave part of a
//   lane's two cells empty (100^3 34.8, cell slots 36.4; 110^3 35.7, 37.8), and
//   8 lines for the two-solve launches of the 4-step scheme (293, 299); FP64 face
//   slots (200^3 290, 312).
// - The two-solve launches (twice) of lines of 1025 to 2048 cells take four waves,
//   whose second solve finds its registers: FP64 one line (1536^2 106, two waves
//   and two lines 129; 1403^2 100, 116), FP32 two (1536^2 63.7, 77.8 with two waves
//   and four lines; 1200^2 45.6, 52.9 with two and two), but for rows off the half
//   lines above 1420 cells (1500^2 68.8, 66.6; 1700^2 79.4, 70.4) or where that
//   spares no CU a line (937 x 1403 37.3, 35.3).
// - FP32 with T = 0 walls keeps face slots: cell slots are faster (500^2 18.8,
//   15.6), but the energy drifts more (against 64-bit arithmetic, 100 steps: 64^2
//   1.4e-7, face slots 2e-8; 234^2 3.3e-8, 6e-9; only at 1024^2 less).
// - FP32 grids of fewer than 2^18 cells keep face slots and one wave per line,
//   with two staging and storing (256^2 7.9; cell slots 7.0, one staging wave 8.5,
//   four lines per workgroup 9.1).  Both bodies are as far from 64-bit
//   arithmetic there, but round differently (energies 1e-8 apart): the default
//   keeps its results, the tuner takes cell slots.
inline bool default_sweep_cfg(int es, int ndim, int n, int64_t lines, bool chi, bool twice, bool walls, SweepCfg* out) {
    const bool keep = es == 4 && ndim == 2 && (walls || (int64_t)n * lines < (1 << 18));
    auto units = [&](int64_t l) { return (lines + 256 * l - 1) / (256 * l) * l; };
    int lpw = 1, wpl = 0, io = 1, body = asd::SWEEP_FACE_SLOTS;
    for (int l = 2; l <= (es == 4 || (ndim == 2 && n <= 512) ? 4 : 2); l *= 2)
        if (3 * units(l) <= 4 * units(1)) lpw = l;
    // lines of cell slots that a CU holds in this shape
    auto cell_lines = [&](int w, int l) {
        SweepCfg c;
        return choose_sweep_cfg_wpl(es, ndim, n, chi, w, l, &c, 1, asd::SWEEP_CELL_SLOTS) && c.lpw == l ? resident_lines(es, ndim, n, c) : 0;
    };
    const int64_t row = lines * es % 128;  // of the transposed output
    const bool aligned = row % 64 == 0;
    if (ndim == 3) {
        if (es == 4 && n <= 512) {
            wpl = 1;
            if (twice) lpw *= 2;
            else if (n <= 64 || n >= 128) body = asd::SWEEP_CELL_SLOTS;
        }
    } else if (keep && n <= 1024) {
        wpl = 1;
        io = n >= 128 ? 2 : 1;
        lpw = std::max(lpw, io);
    } else if (n <= 1024) {
        wpl = n <= 512 ? 1 : 2;
        if (es == 4 || n >= 7 * 128 || lines <= 256 || (n <= 512 && cell_lines(wpl, lpw) >= units(lpw))) body = asd::SWEEP_CELL_SLOTS;
    } else if (es == 8) {
        const bool two = aligned ? n > 14 * 128 && lines > 512 && units(2) == units(1) : lpw == 2;
        wpl = n < 2048 && two && !twice ? 2 : n <= 2048 || lines > 256 || twice ? 4 : 0;
        lpw = wpl == 2 ? 2 : 1;
    } else if (n <= 2048) {
        wpl = 2;
        if (twice && (aligned || (n <= 1420 && units(2) < units(4)))) {
            wpl = 4;
            lpw = 2;
        } else if (!aligned && (row % 64 != 60 || twice)) {
            if (3 * units(4) <= 5 * units(1)) lpw = 4;
        } else if (lpw == 4 && (row != 0 || 3 * units(4) == 4 * units(1))) {
            lpw = 2;
        }
        const int64_t u = units(lpw), held = twice ? 0 : cell_lines(wpl, lpw);
        if (held >= std::min<int64_t>(6, u) && (held >= u || 3 * ((u + held - 1) / held) * held <= 4 * u))
            body = asd::SWEEP_CELL_SLOTS;
    } else {
        wpl = 4;
    }
    if (keep) body = asd::SWEEP_FACE_SLOTS;
    for (; wpl > 0 && wpl <= 16; wpl *= 2)
        if (choose_sweep_cfg_wpl(es, ndim, n, chi, wpl, lpw, out, io, body)) return true;
    return choose_sweep_cfg(es, ndim, n, chi, 0, 0, out);
}

// Whether a 2-D sweep stores line-contiguous and transposes afterwards, and
// its shape then.  A transposed store writes pieces of at most 16 bytes of
// each output row; on a grid beyond the L2s they reach memory unmerged
// (8192^2 FP32, 8-byte pieces: 4.4 bytes written per byte), the sooner if the
// rows do not start on cache lines.  The line-contiguous store needs one line
// per workgroup only (several workgroups per CU, whose load and solve phases
// overlap), and the transpose costs two more passes over the state.  us per
// step, transposed store / line-contiguous and transpose:
//   FP32 1700^2 42 / 47, 2048^2 38 / 46, 2500^2 115 / 88, 3000^2 141 / 106,
//   4096^2 185 / 168, 8192^2 1250 / 800; FP64 1500^2 71 / 68, 1700^2 87 / 81,
//   2048^2 75 / 81, 2500^2 310 / 191, 4096^2 538 / 380.
inline bool default_split(int es, int ndim, int n, int nt, bool walls, SweepCfg* out) {
    const bool cell = es == 4 && n < 4096 && !walls;  // 3000^2 106 against 111, 4096^2 177 against 168
    bool ok = false;
    for (int wpl = 4; wpl <= 16 && !ok; wpl *= 2)
        ok = choose_sweep_cfg_wpl(es, ndim, n, false, wpl, 1, out, 1, cell ? asd::SWEEP_CELL_SLOTS : asd::SWEEP_FACE_SLOTS);
    if (!ok || ndim != 2) return false;
    const int64_t bytes = (int64_t)n * nt * es;
    const bool rows_aligned = ((int64_t)nt * es) % 128 == 0;
    return bytes > (rows_aligned ? (int64_t)32 << 20 : (int64_t)16 << 20);
}

// One captured step loop, keyed on what the capture baked in.
struct GraphEntry {
    hipGraphExec_t exec = nullptr;
    int kind = 0;  // 1 = semi-implicit, 2 = explicit
    double dt = 0.0;
    int nsteps = 0;
    double* energy = nullptr;
    double* series = nullptr;
    uint64_t last_use = 0;
};
static constexpr int kGraphCacheEntries = 4;
// ASD_GRAPHS_AUTO captures calls of at least this many steps; shorter calls
// launch directly (a graph launch starts its first kernel several
// microseconds later than a direct launch, more than the host-side launch
// cost of a short call)
static constexpr int kGraphMinSteps = 64;
static constexpr int kAuxEvents = 5;

struct asd_grid_s {
    asd_desc d{};
    hipStream_t st = nullptr;
    char* ws = nullptr;
    size_t ws_bytes = 0;
    int64_t N = 0;
    size_t es = 4;
    void* T = nullptr;
    void* b[3] = {nullptr, nullptr, nullptr};
    void* chi = nullptr;
    void* src = nullptr;       // source Q (optional), natural layout
    bool ws_inited = false;
    bool coef_valid = false;   // face coefficients computed for coef_dt
    double coef_dt = 0.0;
    void* tmp[2] = {nullptr, nullptr};
    char* coef[3][3] = {};     // [sweep][alpha, beta_t1, beta_t2], sweep's input layout
    double* ring = nullptr;    // reduction partials: ring_slots + 1 slots of max_blocks (sum, min, max)
    int ring_slots = 2;
    int64_t max_blocks = 0;
    unsigned* flags = nullptr;
    double* stats = nullptr;
    SweepCfg cfg[3];
    // 2-D sweeps whose transposed store would be made of pieces too short to
    // meet in the L2: stored line-contiguous in shape split_cfg, then transposed
    bool split[3] = {false, false, false};
    SweepCfg split_cfg[3];
    // graph cache of step loops: a few captured loops, least recently used
    // replaced first; graph_valid = false marks every entry stale (fields,
    // coefficients or launch shapes changed)
    int graph_mode = ASD_GRAPHS_AUTO;  // ASD_GRAPHS_OFF / _AUTO / _ALWAYS
    bool graph_valid = false;
    GraphEntry graphs[kGraphCacheEntries];
    uint64_t graph_clock = 0;
    // the adjoint's second stream (recomputation beside the reverse pass)
    // and its events; created by the first adjoint call that needs them
    hipStream_t aux = nullptr;
    hipEvent_t aux_ev[kAuxEvents] = {};
};

// whether a step call of nsteps steps replays a captured graph (only on a
// non-default stream)
inline bool graphs_for(asd_grid_s* g, int nsteps) {
    if (!g->st || nsteps < 2) return false;
    return g->graph_mode == ASD_GRAPHS_ALWAYS || (g->graph_mode == ASD_GRAPHS_AUTO && nsteps >= kGraphMinSteps);
}

// capi.cpp
int asd_fail(int code, const char* fmt, ...);
int validate_desc(const asd_desc* d);
size_t grid_workspace_bytes(const asd_desc* desc);  // desc validated
// Fill a grid handle over a workspace (desc validated; no device work).
int init_grid_in_place(asd_grid_s* g, const asd_desc* desc, void* dev_ws, size_t ws_bytes, void* stream);
int check_dt(asd_grid g, double dt, bool explicit_scheme);
// Sweep mode bits (the rhs_mode argument of fill_sweep_params / enqueue_sweep).
enum : int {
    SWEEP_SOLVE_ONLY = 1,   // right-hand side = U (no transverse term)
    SWEEP_KEEP_LAYOUT = 2,  // output in the input layout
    SWEEP_SOURCE = 4,       // dt Q joins the right-hand side (input in the natural layout)
    SWEEP_REDUCE_INPUT = 8, // the reduction (red) sums the input state instead of the output
    SWEEP_TWICE = 16,       // the 4-step scheme's two solves of a direction in one launch
};

template <typename T>
int fill_sweep_params(asd_grid g, int d, const void* in, void* out, int rhs_mode, const SweepCfg& c,
                      asd::SweepParams<T>* P);
bool set_default_cfg(asd_grid_s* g, int q);
// Whether axis q stores line-contiguous by default, and the shape it does that
// in (2-D; filled whether or not).
bool default_line_cfg(asd_grid_s* g, int q, SweepCfg* out);
// What one step of a grid launches: per axis the shape and the store, and for
// the 4-step scheme whether a direction's two solves share a launch (twice) or
// take one each (two).
struct StepPlan {
    SweepCfg cfg[3];
    bool split[3] = {false, false, false};  // line-contiguous store, then a transpose
    bool twice = false, two = false;
};
// The plan with launch shapes cfg[], or line[] on the axes with split[].  The
// two solves share a launch when the coefficients are those of the step (not
// chi(T), whose second solve has its own), every axis has the face body with
// io = 1 and the larger tile fits on every axis (with fewer lines per workgroup
// than the shape says, where it must); two launches need both spare states, so
// that they store transposed.
StepPlan step_plan(asd_grid g, const SweepCfg* cfg, const SweepCfg* line, const bool* split);
inline StepPlan step_plan(asd_grid g) { return step_plan(g, g->cfg, g->split_cfg, g->split); }
// Direction d of a step: in -> out, by way of spare where the plan takes two
// launches or a transpose (spare is then not in or out; out may be in).
// mode: SWEEP_SOURCE, SWEEP_REDUCE_INPUT.  coef: chi(T)'s coefficients from
// each launch's input first.
int enqueue_direction(asd_grid g, const StepPlan& plan, int d, double dt, const void* in, void* spare, void* out,
                      int mode, const asd::ReduceParams& red, int* nblocks_out, bool coef);
int check_fields(asd_grid g, bool need_T);
int prepare(asd_grid g, double dt);  // dt > 0: face coefficients for dt
int64_t layout_stride(const asd_grid g, int L, int a);
asd::ReduceParams no_reduce();
// Per-step outputs of a step loop (each nullable): energies, FP64[nsteps+1];
// series of (energy, min T, max T), FP64[3 (nsteps+1)].
struct StepOut {
    double* energy = nullptr;
    double* series = nullptr;
    bool any() const { return energy || series; }
    const double* e0() const { return energy ? energy : series; }  // energy of the initial state
};
// Fold of count consecutive reductions into entries first .. first+count-1 of out.
asd::FoldParams make_fold(asd_grid g, const double* partials, int nblocks, int count, const StepOut& out, int first);
inline double* ring_slot(asd_grid g, int i) { return g->ring + (size_t)i * g->max_blocks * 3; }
// out2 (nullable): the output also written in the input layout (sweeps
// whose output layout is transposed).
int enqueue_sweep(asd_grid g, int d, double dt, const void* in, void* out, int rhs_mode,
                  const asd::ReduceParams& red, const SweepCfg* cfg,
                  int* nblocks_out, void* out2 = nullptr);
int enqueue_si_loop(asd_grid g, double dt, int nsteps, const StepOut& out);
int enqueue_explicit_loop(asd_grid g, double dt, int nsteps, const StepOut& out);
int enqueue_permute_2d(asd_grid g, const void* in, void* out, bool a_to_b);
int enqueue_explicit(asd_grid g, double dt, const void* src, void* dst, const asd::ReduceParams& red,
                     int* nblocks_out);
int enqueue_copy(asd_grid g, const void* src, void* dst);
int enqueue_reduce(asd_grid g, const void* x, const StepOut& out, asd::FoldParams* fold);
int enqueue_fold(asd_grid g, const asd::FoldParams& f);
// graph.cpp
int run_si_graph(asd_grid g, double dt, int nsteps, const StepOut& out);
int run_explicit_graph(asd_grid g, double dt, int nsteps, const StepOut& out);
