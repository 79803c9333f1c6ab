// capi.hip -- host side of the C ABI declared in include/flipmc.h.
//
// Validates parameters, lays the system out in the caller's device buffer,
// fills the device descriptor (SysDev) and enqueues the kernels of
// kernels.hip on the caller's stream.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <limits>
#include <string>
#include <utility>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "engine.h"
#include "flipmc.h"

using namespace flipmc;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

}  // namespace

namespace flipmc {

int api_error(int code, const char* msg)
{
    g_err = msg;
    return code;
}

size_t device_lds_limit()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 163840;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
        v <= 0) {
        (void)hipGetLastError();
        return 163840;
    }
    return (size_t)v;
}

}  // namespace flipmc

namespace {

// A named range on the host timeline of a profiler that records roctx
// markers (rocprofv3 --marker-trace): one per API call that enqueues work,
// one per launch of sweeps or events inside it.
struct TraceRange {
    explicit TraceRange(const char* what) { roctxRangePushA(what); }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange&) = delete;
    TraceRange& operator=(const TraceRange&) = delete;
};

#define HIPCHK(x)                                                                       \
    do {                                                                                \
        hipError_t e_ = (x);                                                            \
        if (e_ != hipSuccess) return fail(MC_EDEVICE, "%s: %s", #x, hipGetErrorString(e_)); \
    } while (0)

// Side of the rigid triangle: the minimum of WCA + FENE (Eq. 1 + Eq. 2) of a
// sigma_ij = 1 bond, found by Newton's method on the slope.
double bond_star()
{
    auto slope = [](double x) {
        return -48.0 * std::pow(x, -13.0) + 24.0 * std::pow(x, -7.0) +
               30.0 * x / (1.0 - x * x / 2.25);
    };
    auto curvature = [](double x) {
        const double d = 1.0 - x * x / 2.25;
        return 624.0 * std::pow(x, -14.0) - 168.0 * std::pow(x, -8.0) +
               30.0 / d + 30.0 * x * (2.0 * x / 2.25) / (d * d);
    };
    double x = 0.96;
    for (int it = 0; it < 100; ++it) {
        const double nx = x - slope(x) / curvature(x);
        if (nx == x) break;
        x = nx;
    }
    return x;
}

struct Geometry {
    double L, bond, radius, reach;
    uint32_t k, nc, ncell;
    bool resident;
    uint32_t near_cap;    // molecules listed near a cell
    bool team;            // standalone sweeps run on the multi-workgroup engine
    uint32_t team_blocks;    // the workgroups it launches alone, the most it takes in a batch
    bool lists;              // the multi-workgroup engine has the cell lists in LDS
    uint32_t wave_fit;       // cells that its workgroups have room for with one per wave
    uint32_t team_waves;     // waves with a cell each when it runs alone
    size_t lds;              // LDS of the one-workgroup engine
    double sweep_cost;    // modelled cycles of one sweep on one workgroup
    // Modelled cycles of a sweep on nb workgroups with a cell per wave (waves) or
    // per workgroup.
    double spread_cycles(uint32_t M, uint32_t nb, bool waves) const;
    // Whether the buffer has the multi-workgroup engine's arrays.
    bool team_arrays() const { return !resident || team || team_blocks >= 2; }
};

// The critical path of one sweep of the resident kernel, as the choice of the
// decomposition has always taken it (the same parameters keep the same cells,
// and with them the same chain): k^3 colour phases; in each, the busiest wave
// builds the neighbour list of each of its cells and runs the cell's trials one
// after another.
double cost_estimate(uint32_t M, double L, double reach, uint32_t k, uint32_t nc)
{
    const double ncell = (double)nc * nc * nc;
    const double per_cell = (double)M / ncell;
    const double w = L / nc;
    const double na3 = std::pow((double)(nc / k), 3.0);
    const double cells_per_wave = std::ceil(na3 / kWaves);
    const double span = std::min((double)nc, 2.0 * (k - 1) + 1.0);
    const double stencil = std::min((double)M, span * span * span * per_cell);
    const double region = 0.75 * std::pow(w + 2.0 * reach, 3.0) * (double)M / (L * L * L);
    const double listed = std::min(stencil, region);
    const double t_list = 300.0 + 20.0 * stencil;
    const double t_trial = 1800.0 + 12.0 * listed;
    return (double)k * k * k * (cells_per_wave * (t_list + std::max(1.0, per_cell) * t_trial) + 300.0);
}

// Cycles of a sweep on one workgroup, for the sizes of time slices and the
// choice of the engine.  Fitted to 216 (k = 3, n_c = 6), 512 and 1000 (k = 2,
// n_c = 4) and 1728 (n_c = 6) molecules in LDS: 195, 180, 313 and 565 us (by now
// 185, 171, 302 and 549).
double sweep_cycles(uint32_t M, uint32_t k, uint32_t nc)
{
    const double per_cell = std::max(1.0, (double)M / ((double)nc * nc * nc));
    const double cells_per_wave = std::ceil(std::pow((double)(nc / k), 3.0) / kWaves);
    return (double)k * k * k * (cells_per_wave * (6000.0 + 4800.0 * per_cell) + 6000.0);
}

// The same for the multi-workgroup engine on nb workgroups with a cell each:
// a workgroup's waves list the neighbourhood together and evaluate kWaves trials
// at once, of which the decisions use those up to the first accepted one
// (measured: 3.5 rounds for 16 trials at T = 0.75, 2.3 for 8 at T = 1.1); cells
// wait for their neighbours at every colour and all workgroups three times a
// sweep.
double team_cycles(uint32_t M, uint32_t k, uint32_t nc, uint32_t nb)
{
    const double per_cell = std::max(1.0, (double)M / ((double)nc * nc * nc));
    const double rounds = std::ceil(std::pow((double)(nc / k), 3.0) / nb), colours = (double)k * k * k;
    return colours * rounds * (9000.0 + 4750.0 * (1.0 + per_cell / 6.2)) + (nb > 1 ? colours * 9000.0 + 45000.0 : 10000.0);
}

// With a cell per wave on nb workgroups of `waves` such waves: longer, but at a
// quarter of the work, so a full device moves more molecules.  With at most a
// wave on each SIMD a round is 7 % shorter (2197 molecules, 27 cells of a colour:
// 290 us a sweep on 4 workgroups, 271 on 7).
double waves_cycles(uint32_t M, uint32_t k, uint32_t nc, uint32_t nb, uint32_t waves)
{
    const double per_cell = std::max(1.0, (double)M / ((double)nc * nc * nc));
    const double cells = std::pow((double)(nc / k), 3.0) / nb;  // of a workgroup
    const double rounds = std::ceil(cells / waves), colours = (double)k * k * k, pace = cells <= 4.0 ? 0.93 : 1.0;
    return colours * (rounds * (9000.0 + 4800.0 * per_cell) * pace + 8000.0) + 45000.0;
}

// Initial milliseconds per modelled cycle of the engine classes (one
// workgroup with the state in LDS, in HBM; the multi-workgroup engine with a cell
// per workgroup, with a cell per wave) in FP32 and in FP64, relative to the FP32
// LDS class; a batch then measures its own.  Measured alone at T = 1.5, 216 - 27000
// molecules: FP32 LDS 0.84 - 1.05, HBM 0.74 - 0.91, a cell per workgroup 0.7 - 1.1,
// per wave 0.85 - 1.3; FP64 1.1 - 1.5, 1.1 - 1.4, 1.0 - 1.5, 0.85 - 1.2.  (With one
// set for both, 1.0, 1.0, 1.1, 1.4, a batch never tried what it took for slow: 100
// FP64 systems of 2197 molecules stayed on one workgroup each, 29 ms for 20 sweeps,
// 20 on two.)
constexpr double kCycleRatio[2][4] = {{1.0, 0.85, 1.0, 1.1}, {1.4, 1.25, 1.35, 1.0}};

double Geometry::spread_cycles(uint32_t M, uint32_t nb, bool waves) const
{
    return waves ? waves_cycles(M, k, nc, nb, wave_fit) : team_cycles(M, k, nc, nb);
}

// Whether the multi-workgroup engine on nb workgroups is modelled at least
// 25 % faster than the system's own engine on one workgroup, with ms_one and
// ms_multi the milliseconds per modelled cycle of the two (always on several,
// for a system beyond one workgroup's LDS).
bool spread_pays(const Geometry& g, uint32_t M, uint32_t nb, bool waves, double ms_one, double ms_multi)
{
    return (!g.resident && nb > 1) || g.sweep_cost * ms_one >= 1.25 * g.spread_cycles(M, nb, waves) * ms_multi;
}

int geometry(const mc_params* p, Geometry* g)
{
    if (!p) return fail(MC_EINVAL, "null parameters");
    if (p->n_molecules < 1 || p->n_molecules > (uint32_t)kMaxMolecules)
        return fail(MC_EINVAL, "n_molecules must be in [1, %d]", kMaxMolecules);
    if (p->precision != MC_FP64 && p->precision != MC_FP32_DE)
        return fail(MC_EINVAL, "precision must be MC_FP64 or MC_FP32_DE");
    if (!(p->density > 0) || !(p->temperature > 0))
        return fail(MC_EINVAL, "density and temperature must be positive");
    for (int i = 0; i < 3; ++i)
        if (!(p->sigma[i] > 0)) return fail(MC_EINVAL, "sigma must be positive");
    if (!(p->p_flip >= 0) || !(p->p_translate >= 0) || p->p_flip + p->p_translate > 1.0)
        return fail(MC_EINVAL, "move probabilities out of range");
    if (!(p->max_displacement >= 0) || !(p->max_rotation >= 0))
        return fail(MC_EINVAL, "step sizes must be non-negative");
    if (!(p->gofr_dr > 0)) return fail(MC_EINVAL, "gofr_dr must be positive");
    if (!(p->fs_q >= 0) || !(p->fs_q_cm >= 0)) return fail(MC_EINVAL, "fs_q and fs_q_cm must be >= 0");
    g->L = std::cbrt(3.0 * (double)p->n_molecules / p->density);
    g->bond = p->bond_length > 0 ? p->bond_length : bond_star();
    g->radius = g->bond / std::sqrt(3.0);
    const double smax = std::max(p->sigma[0], std::max(p->sigma[1], p->sigma[2]));
    const double rcmax = std::pow(2.0, 1.0 / 6.0) * smax;
    g->reach = rcmax + 2.0 * g->radius;
    // Pair terms are formed from the nearest image of the two centres plus the
    // site offsets.  That is the nearest image of every interacting site pair
    // only when no molecule reaches another through two images: L >= 2 reach.
    if (g->L < 2.0 * (g->reach + 2.0 * p->max_displacement))
        return fail(MC_EGEOM, "box side %.4f below twice the interaction reach %.4f (minimum image)",
                    g->L, g->reach + 2.0 * p->max_displacement);
    uint32_t k = p->colours_per_axis, nc = p->cells_per_side;
    if (k == 0 && nc == 0) {
        double best = std::numeric_limits<double>::infinity();
        for (uint32_t kk = 2; kk <= 3; ++kk) {
            uint32_t n = (uint32_t)std::floor((kk - 1) * g->L / g->reach);
            n -= n % kk;
            while (n >= 2 && std::pow((double)n, 3.0) > 65535.0) n -= kk;
            if (n < 2 || n < kk) continue;
            const double c = cost_estimate(p->n_molecules, g->L, g->reach, kk, n);
            if (c < best) {
                best = c;
                k = kk;
                nc = n;
            }
        }
        if (k == 0) return fail(MC_EGEOM, "no checkerboard fits a box of side %.4f", g->L);
    } else if (k == 0 || nc == 0) {
        return fail(MC_EINVAL, "give both colours_per_axis and cells_per_side, or neither");
    }
    if (k < 2 || k > 3) return fail(MC_EGEOM, "colours_per_axis must be 2 or 3");
    if (nc < 2 || nc % k != 0) return fail(MC_EGEOM, "cells_per_side must be a multiple of k >= 2");
    if ((double)(k - 1) * (g->L / (double)nc) < g->reach)
        return fail(MC_EGEOM, "(k-1) * cell width %.5f is below the interaction reach %.5f",
                    (double)(k - 1) * g->L / nc, g->reach);
    const double ncell = (double)nc * nc * nc;
    if (ncell > 65535.0) return fail(MC_EGEOM, "too many cells (%u per side)", nc);
    g->k = k;
    g->nc = nc;
    g->ncell = nc * nc * nc;
    const bool fp64 = p->precision == MC_FP64;
    const size_t limit = device_lds_limit();
    // the near list: what a cell of this width meets at this density with a
    // fifth to spare, in steps of 64; fewer where that keeps the state in LDS
    {
        const double w = g->L / nc, R = g->reach;
        const double region = w * w * w + 6.0 * w * w * R + 3.0 * M_PI * w * R * R + 4.0 / 3.0 * M_PI * R * R * R;
        const double need = std::min((double)p->n_molecules, 1.2 * region * p->density / 3.0 + 16.0);
        g->near_cap = kNearMin;
        while (g->near_cap < kNearMax && g->near_cap < need) g->near_cap += 64;
        while (g->near_cap > kNearMin &&
               lds_layout(fp64, true, p->n_molecules, g->ncell, g->near_cap).total > limit &&
               lds_layout(fp64, true, p->n_molecules, g->ncell, kNearMin).total <= limit)
            g->near_cap -= 64;
    }
    const LdsLayout res = lds_layout(fp64, true, p->n_molecules, g->ncell, g->near_cap);
    g->resident = res.total <= limit && !(p->flags & MC_FLAG_HBM_STATE);
    g->lds = g->resident ? res.total : lds_layout(fp64, false, p->n_molecules, g->ncell, g->near_cap).total;
    const bool one_wg = (p->flags & MC_FLAG_SINGLE_WORKGROUP) || p->workgroups == 1;
    g->lists = spread_layout(fp64, true, p->n_molecules, g->ncell, g->near_cap, 0).total <= limit;
    g->wave_fit = 0;
    while (g->wave_fit < (uint32_t)cell_threads(fp64, g->lists) / 64u &&
           spread_layout(fp64, g->lists, p->n_molecules, g->ncell, g->near_cap, g->wave_fit + 1).total <= limit)
        ++g->wave_fit;
    g->team_waves = 0;
    g->team = false;
    g->team_blocks = 1;
    // the model is fitted to the LDS state; with the state in HBM a sweep on
    // one workgroup takes about 1.3 times as long (measured 1.1 - 1.4 over
    // 2197 - 27000 molecules)
    g->sweep_cost = sweep_cycles(p->n_molecules, k, nc) * (g->resident ? 1.0 : 1.3);
    if (!one_wg) {
        // one workgroup per cell of a colour, as many as the device holds.  A
        // system whose state fits one workgroup's LDS runs alone on the
        // multi-workgroup engine too when that is modelled faster or when the
        // caller asks for a workgroup count; otherwise it keeps the count for a
        // batch, which may move it there when compute units are idle
        uint32_t maxb = 0;
        const hipError_t e = spread_max_blocks(&maxb);
        if (e != hipSuccess || maxb == 0) {
            (void)hipGetLastError();
        } else {
            const uint32_t na = nc / k, nact = na * na * na;
            const uint32_t most = p->workgroups ? std::min(p->workgroups, maxb) : maxb;
            const double* ratio = kCycleRatio[fp64];
            g->team_blocks = std::min(nact, most);
            g->team = !g->resident || (p->workgroups >= 2 && g->team_blocks >= 2) ||
                      spread_pays(*g, p->n_molecules, g->team_blocks, false, ratio[0], ratio[2]);
            // With several cells for each workgroup of a colour, a cell per wave
            // where that is modelled less than 15 % slower: its time hardly
            // depends on how many trials are accepted, that of a cell per
            // workgroup does (27000 molecules on 256, FP32: T = 0.75 214 and 217 us
            // a sweep, T = 3 235 and 217, steps a tenth as long 296 and 225; FP64
            // 306 - 398 and 239 - 245).
            const double margin = nact > g->team_blocks ? 0.85 : 1.0;
            if (g->wave_fit && margin * ratio[3] * g->spread_cycles(p->n_molecules, g->team_blocks, true) <
                                   ratio[2] * g->spread_cycles(p->n_molecules, g->team_blocks, false))
                g->team_waves = std::min(g->wave_fit, (nact + g->team_blocks - 1) / g->team_blocks);
        }
    }
    return MC_OK;
}

// Modelled cycles of a time slice of max_moves moves of the 1000-molecule
// reference system (k = 2, n_c = 4) on one workgroup.
double slice_time(uint64_t max_moves)
{
    static const double ref = sweep_cycles(1000, 2, 4);
    return (double)max_moves / 1000.0 * ref;
}

// Milliseconds per modelled cycle on an idle device: a sweep of the
// 1000-molecule reference (k = 2, n_c = 4) takes about 0.3 ms on one
// workgroup with the state in LDS.
double ms_per_model_cycle()
{
    return 0.31 / slice_time(1000);
}

// Times (in falling order) put on n workgroups, each on the one that is done
// first: the time at which the last is done, and which took each.
double longest_first(const std::vector<double>& times, uint32_t n, std::vector<uint32_t>* taken)
{
    std::vector<std::pair<double, uint32_t>> done;
    for (uint32_t w = 0; w < n; ++w) done.emplace_back(0.0, w);  // a heap as it is
    if (taken) taken->clear();
    double end = 0.0;
    for (const double t : times) {
        std::pop_heap(done.begin(), done.end(), std::greater<>());
        done.back().first += t;
        end = std::max(end, done.back().first);
        if (taken) taken->push_back(done.back().second);
        std::push_heap(done.begin(), done.end(), std::greater<>());
    }
    return end;
}

// Workgroups of the multi-workgroup event kernel for M molecules, 1 =
// single-workgroup events.  256 molecules are 16 units; a total energy of 200
// takes 44 us on one workgroup and 43 on several, of 255 49 and 45, of 300 61 and
// 45, of 1000 207 and 39.
uint32_t event_blocks(uint32_t M)
{
    if (M < 256) return 1;
    return std::min(256u, (event_units(M).count() + kWaves - 1) / kWaves);
}

// Systems below this size take scheduled re-sums and C_2 samples inside a
// batch's sweep kernel.
constexpr uint32_t kInlineBelow = 2048;

struct BufLayout {
    size_t sys, stats, com, quat, types, u0, kref, esamp, dsamp, gall, ginter, c2, c2s;
    size_t img, r0, o0, fs, fscm, mom;
    size_t props, gpart, gsite, gcell, gcellid, glist, gcnt, gecell, gbar, total;
};

size_t al(size_t x) { return (x + 255) & ~size_t(255); }

BufLayout buf_layout(const mc_params* p, const Geometry& g)
{
    BufLayout b{};
    const size_t M = p->n_molecules;
    size_t o = 0;
    b.sys = o;    o = al(o + sizeof(SysDev));
    // what the reading calls want lies together, so that each takes one copy:
    // the observables, and on to the configuration
    b.stats = o;  o = al(o + sizeof(Stats));
    b.gall = o;   o = al(o + kGofrBins * sizeof(uint64_t));
    b.ginter = o; o = al(o + kGofrBins * sizeof(uint64_t));
    b.c2 = o;     o = al(o + kC2Max * sizeof(double));
    b.c2s = o;    o = al(o + kC2Max * sizeof(uint64_t));
    b.fs = o;     o = al(o + kC2Max * sizeof(double));
    b.fscm = o;   o = al(o + kC2Max * sizeof(double));
    b.mom = o;    o = al(o + 4 * kC2Max * sizeof(double));
    b.com = o;    o = al(o + 3 * M * sizeof(double));
    b.quat = o;   o = al(o + 4 * M * sizeof(double));
    b.types = o;  o = al(o + M * sizeof(uint32_t));
    b.u0 = o;     o = al(o + 3 * M * sizeof(double));
    b.kref = o;   o = al(o + M);
    b.esamp = o;  o = al(o + size_t(p->max_samples) * sizeof(double));
    b.dsamp = o;  o = al(o + size_t(p->max_samples) * sizeof(double));
    b.img = o;    o = al(o + 3 * M * sizeof(int32_t));
    b.r0 = o;     o = al(o + 3 * M * sizeof(double));
    b.o0 = o;     o = al(o + 9 * M * sizeof(double));
    b.props = o;  o = al(o + M * 48);
    b.gpart = o;  o = al(o + max_units((uint32_t)M) * sizeof(double));
    if (g.team_arrays()) {
        const bool fp64 = p->precision == MC_FP64;
        b.gsite = o;   o = al(o + M * std::max(3 * site_bytes(fp64), mol_bytes(fp64)));
        b.gcell = o;   o = al(o + (size_t(g.ncell) + 1) * sizeof(uint32_t));
        b.gcellid = o; o = al(o + M * sizeof(uint16_t));
        b.glist = o;   o = al(o + M * sizeof(uint16_t));
        b.gcnt = o;    o = al(o + 2 * size_t(g.ncell) * sizeof(uint32_t));
        b.gecell = o;  o = al(o + size_t(g.ncell) * sizeof(double));
        b.gbar = o;    o = al(o + kBarWords * sizeof(uint32_t));
    }
    b.total = o;
    return b;
}

}  // namespace

struct mc_system {
    mc_params p;
    Geometry g;
    BufLayout lay;
    SysDev host;
    SysDev* dev;
    uint8_t* buf;
    hipStream_t stream;
    uint64_t sweep;   // host mirror of the device sweep counter
    uint64_t origin;  // host mirror of the observable origin
    mc_batch* batch;
    // launch timing (mc_timing_enable)
    bool timing;
    std::vector<hipEvent_t> ev_pool;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_sweep, ev_event;
};

// Slices of the systems on the multi-workgroup engine that one run of all
// remaining sweeps enqueues (they end at event sweeps).  A run ends with its
// slowest system, so few slices a run leave compute units idle at each end, and
// each slice has its tables: 600 sweeps of 24 and 64 systems of 125 - 8000
// molecules with a re-sum every 20 take 218 and 318 ms with 4, 147 and 224 with 16,
// 147 and 222 with 64.
constexpr uint32_t kRounds = 16;

struct mc_batch {
    uint32_t max_slots;
    uint32_t precision;
    hipStream_t stream;
    std::vector<mc_system*> sys;
    std::vector<uint64_t> remaining;
    Slot* dev_slots[2];   // per parity: [resident | non-resident | events] x max_slots
    Slot* host_slots[2];
    hipEvent_t copied[2];
    bool pending[2];
    int parity;
    // systems on the multi-workgroup engine: one launch per run on stream2,
    // overlapping the batch stream's launches
    hipStream_t stream2;              // caller's second stream (or the batch stream)
    hipEvent_t go, done;              // stream2 waits for go (stream), stream for done (stream2)
    // systems on one workgroup with the state in HBM: their launch on stream3
    // (a third caller stream) runs beside the LDS class's launch on stream;
    // nullptr = after it on stream
    hipStream_t stream3;
    hipEvent_t go3, done3;            // stream3 waits for go3 (stream), stream for done3 (stream3)
    SpreadSlot* dev_spread[2];        // per parity: [systems | (events as Slot)] x max_slots
    SpreadSlot* host_spread[2];       // staging of kRounds tables of ncu systems
    Slot* dev_ev2[2];
    Slot* host_ev2[2];
    hipEvent_t copied2[2];
    bool pending2[2];
    uint32_t spread_max;              // workgroups of one launch of it that the device holds
    uint32_t ncu;                     // compute units of the device
    uint32_t wg_limit;                // compute units the batch's runs use at once
    uint32_t turn;                    // where the next run starts taking systems when
                                      // there are more than wg_limit
    // slice calibration per engine class (one workgroup with the state in LDS,
    // one workgroup with the state in HBM, multi-workgroup with a cell per
    // workgroup, with a cell per wave): milliseconds per
    // modelled cycle, learnt from the timed launches of earlier runs
    double ms_per_cycle[4];
    double pred[4];                   // modelled cycles of the class's last launch (0: none)
    hipEvent_t t_beg[4], t_end[4];
};

namespace {

// A system inside a batch is advanced on the batch's stream: wait for it
// before reading the system's state on its own stream.
int sync_owner(mc_system* s)
{
    if (s->batch) HIPCHK(hipStreamSynchronize(s->batch->stream));
    return MC_OK;
}

int upload_desc(mc_system* s)
{
    HIPCHK(hipMemcpyAsync(s->dev, &s->host, sizeof(SysDev), hipMemcpyHostToDevice, s->stream));
    HIPCHK(hipStreamSynchronize(s->stream));
    return MC_OK;
}

hipEvent_t take_event(mc_system* s)
{
    if (!s->ev_pool.empty()) {
        hipEvent_t e = s->ev_pool.back();
        s->ev_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// Record a start event when timing is on (nullptr otherwise).
hipEvent_t timing_start(mc_system* s)
{
    if (!s->timing) return nullptr;
    hipEvent_t a = take_event(s);
    if (a && hipEventRecord(a, s->stream) != hipSuccess) return nullptr;
    return a;
}

void timing_stop(mc_system* s, hipEvent_t a, bool sweep_kernel)
{
    if (!a) return;
    hipEvent_t b = take_event(s);
    if (!b || hipEventRecord(b, s->stream) != hipSuccess) return;
    (sweep_kernel ? s->ev_sweep : s->ev_event).emplace_back(a, b);
}

constexpr uint32_t kOverPairs = kFlagResumSet | kFlagResumReport | kFlagResumPeriodic | kFlagGofr;

// The part of event work `flags` of a system that goes to the multi-workgroup
// event kernel, and in *units the energies it leaves.  A scheduled re-sum
// follows sweeps, whose cell lists are still there (but not the LDS engine's):
// above 8192 molecules they save more than the shorter ranges of a wave cost
// (27000 molecules: 0.5 ms over all pairs).
PartSlot part_slot(const mc_system* s, uint32_t flags, uint32_t first, uint32_t* units)
{
    const uint32_t M = s->p.n_molecules;
    PartSlot p{s->dev, flags, first, event_blocks(M), 0u};
    const int span = (int)std::ceil((std::sqrt(s->host.reach2) + 2.0 * 1.7320508075688772 * s->host.dmax + 1e-9) /
                                    s->host.w);
    const uint32_t planes = 2u * (uint32_t)span + 1u;
    if (M > 8192 && !(flags & (kFlagResumSet | kFlagResumReport)) && s->host.g_cell && planes <= s->host.nc &&
        planes <= kMaxPlanes)
        p.span = (uint32_t)span;
    *units = p.span ? (M + 63u) / 64u * planes : event_units(M).count();
    return p;
}

int launch_events_one(mc_system* s, uint32_t flags)
{
    TraceRange tr((flags & (kFlagResumSet | kFlagResumReport | kFlagResumPeriodic)) ? "flipmc events: FP64 re-sum"
                                                                                    : "flipmc events");
    Slot one{};
    one.sys = s->dev;
    one.flags = flags;
    hipEvent_t t0 = timing_start(s);
    if (event_blocks(s->p.n_molecules) > 1 && (flags & kOverPairs)) {
        // the re-sum and g(r) frame over all pairs on many workgroups, then the rest
        PartList pl{};
        pl.s[0] = part_slot(s, flags, 0u, &one.pad);
        pl.n = 1;
        HIPCHK(launch_event_parts(pl, pl.s[0].count, s->stream));
        one.flags = flags | kFlagParts;
    }
    HIPCHK(launch_events(nullptr, one, 1, s->stream));
    timing_stop(s, t0, false);
    return MC_OK;
}

bool is_c2_time(uint64_t t)
{
    if (t == 0) return false;
    while (t % 10 == 0) t /= 10;
    return t == 1 || t == 2 || t == 5;
}

// Event work due right after sweep `sweep` of system s.
uint32_t events_at(const mc_system* s, uint64_t sweep)
{
    uint32_t f = 0;
    const mc_params& p = s->p;
    if (p.resum_interval && sweep % p.resum_interval == 0) f |= kFlagResumPeriodic;
    const uint64_t t = sweep - s->origin;
    if (p.gofr_interval && t >= p.obs_start && t % p.gofr_interval == 0) f |= kFlagGofr;
    if (is_c2_time(t)) f |= kFlagC2;
    return f;
}

// First sweep after s->sweep at which some event work is due (only g(r)
// frames when the sweep kernel takes the re-sums and C_2 samples itself).
uint64_t next_event(const mc_system* s, bool gofr_only = false)
{
    const mc_params& p = s->p;
    const uint64_t now = s->sweep;
    uint64_t best = UINT64_MAX;
    if (p.resum_interval && !gofr_only)
        best = std::min(best, (now / p.resum_interval + 1) * p.resum_interval);
    const uint64_t t = now - s->origin;
    if (p.gofr_interval) {
        uint64_t n = (t / p.gofr_interval + 1) * p.gofr_interval;
        if (n < p.obs_start) n = ((p.obs_start + p.gofr_interval - 1) / p.gofr_interval) * p.gofr_interval;
        best = std::min(best, s->origin + n);
    }
    for (uint64_t dec = 1; !gofr_only && dec <= (uint64_t)1e18; dec *= 10) {
        bool found = false;
        for (uint64_t m : {1ull, 2ull, 5ull}) {
            if (m * dec > t) {
                best = std::min(best, s->origin + m * dec);
                found = true;
                break;
            }
        }
        if (found) break;
    }
    return best;
}

constexpr uint64_t kMaxSweepsPerLaunch = 1u << 16;
// Workgroups that share a system are those that find room when the launch starts
// (join_crew), for the whole launch, so a launch beside other work is kept short:
// 0.1 s and more of sweeps, against some 20 us for the next launch.
constexpr uint64_t kCrewSweeps = 1024;

// Zero a system's barrier words with a kernel, not a memset: mc_sweep stays
// free of memset nodes for callers that capture it into a graph.
__global__ void k_zero_counter(uint32_t* c)
{
    for (int i = threadIdx.x; i < kBarWords; i += blockDim.x) c[i] = 0u;
}

// The kernel of systems with a cell per wave (waves) or per workgroup, whose cell
// lists all fit its LDS or not.
SpreadMode spread_mode(bool waves, bool lists)
{
    return waves ? (lists ? kSpreadWaves : kSpreadCrewWaves) : (lists ? kSpreadTeam : kSpreadCrew);
}

// Enqueue n sweeps of one system, split at event sweeps.
int advance(mc_system* s, uint64_t n)
{
    Slot one{};
    one.sys = s->dev;
    while (n > 0) {
        // at most kMaxSweepsPerLaunch sweeps per launch (a bounded kernel time)
        const uint64_t chunk = std::min<uint64_t>({n, next_event(s) - s->sweep,
                                                   s->g.team && s->g.team_blocks >= 2 ? kCrewSweeps : kMaxSweepsPerLaunch});
        one.n_sweeps = chunk;
        one.flags = 0;
        TraceRange tr(s->g.team ? "flipmc sweeps: multi-workgroup launch" : "flipmc sweeps: one-workgroup launch");
        if (s->g.team && s->g.team_blocks >= 2) {
            hipLaunchKernelGGL(k_zero_counter, dim3(1), dim3(64), 0, s->stream, s->host.g_bar);
            HIPCHK(hipGetLastError());
        }
        hipEvent_t t0 = timing_start(s);
        if (s->g.team) {
            SpreadSlot sl{};
            sl.sys = s->dev;
            sl.n_sweeps = chunk;
            sl.first_block = 0;
            sl.n_blocks = s->g.team_blocks;
            sl.waves = s->g.team_waves;
            const size_t lds = spread_layout(s->p.precision == MC_FP64, s->g.lists, s->p.n_molecules, s->g.ncell,
                                             s->g.near_cap, sl.waves).total;
            HIPCHK(launch_spread(s->p.precision == MC_FP64, spread_mode(sl.waves, s->g.lists), nullptr, 1, sl,
                                 s->g.team_blocks, lds, s->stream));
        }
        else
            HIPCHK(launch_sweeps(s->p.precision == MC_FP64, s->g.resident, nullptr, one, 1,
                                 s->g.lds, s->stream));
        timing_stop(s, t0, true);
        s->sweep += chunk;
        n -= chunk;
        const uint32_t f = events_at(s, s->sweep);
        if (f) {
            const int rc = launch_events_one(s, f);
            if (rc) return rc;
        }
    }
    return MC_OK;
}

// A copy of the system's buffer from its statistics up to byte `to` (a system of
// 1000 molecules took 70 us for its configuration in four copies, each with a wait
// of its own).
int read_block(mc_system* s, size_t to, std::vector<uint8_t>* out, Stats* st)
{
    if (int rc = sync_owner(s)) return rc;
    out->resize(to - s->lay.stats);
    HIPCHK(hipMemcpyAsync(out->data(), s->buf + s->lay.stats, out->size(), hipMemcpyDeviceToHost, s->stream));
    HIPCHK(hipStreamSynchronize(s->stream));
    std::memcpy(st, out->data(), sizeof(Stats));
    if (st->fault)
        return fail(MC_EDEVICE, "a workgroup barrier of the multi-workgroup engine timed out: "
                                "the system's state is invalid");
    return MC_OK;
}

int read_stats(mc_system* s, Stats* st)
{
    std::vector<uint8_t> raw;
    return read_block(s, s->lay.stats + sizeof(Stats), &raw, st);
}

int write_stats(mc_system* s, const Stats* st)
{
    HIPCHK(hipMemcpyAsync(s->host.stats, st, sizeof(Stats), hipMemcpyHostToDevice, s->stream));
    HIPCHK(hipStreamSynchronize(s->stream));
    return MC_OK;
}

int upload_state(mc_system* s, const double* com, const double* quat, const uint8_t* types)
{
    const size_t M = s->p.n_molecules;
    std::vector<double> c(3 * M), q(4 * M);
    std::vector<uint32_t> t(M);
    for (size_t m = 0; m < M; ++m) {
        for (int a = 0; a < 3; ++a) c[a * M + m] = com[3 * m + a];
        double nrm = 0;
        for (int a = 0; a < 4; ++a) nrm += quat[4 * m + a] * quat[4 * m + a];
        if (!(std::fabs(nrm - 1.0) < 1e-6))
            return fail(MC_EINVAL, "quaternion of molecule %zu is not a unit quaternion", m);
        for (int a = 0; a < 4; ++a) q[a * M + m] = quat[4 * m + a];
        const uint8_t a0 = types[3 * m], a1 = types[3 * m + 1], a2 = types[3 * m + 2];
        if (a0 > 2 || a1 > 2 || a2 > 2 || a0 == a1 || a0 == a2 || a1 == a2)
            return fail(MC_EINVAL, "types of molecule %zu are not a permutation of A, B, C", m);
        t[m] = (uint32_t)a0 | ((uint32_t)a1 << 8) | ((uint32_t)a2 << 16);
    }
    HIPCHK(hipMemcpyAsync(s->host.com, c.data(), c.size() * sizeof(double), hipMemcpyHostToDevice, s->stream));
    HIPCHK(hipMemcpyAsync(s->host.quat, q.data(), q.size() * sizeof(double), hipMemcpyHostToDevice, s->stream));
    HIPCHK(hipMemcpyAsync(s->host.types, t.data(), t.size() * sizeof(uint32_t), hipMemcpyHostToDevice, s->stream));
    HIPCHK(hipStreamSynchronize(s->stream));
    return MC_OK;
}

// The event work over many workgroups of several systems: one launch per
// kPartSlots systems, each system on its own event_blocks() workgroups.
hipError_t launch_parts_of(const std::vector<std::pair<mc_system*, uint32_t>>& parts,
                                  hipStream_t stream)
{
    for (size_t i0 = 0; i0 < parts.size(); i0 += kPartSlots) {
        PartList pl{};
        uint32_t blocks = 0;
        for (size_t i = i0; i < std::min(parts.size(), i0 + kPartSlots); ++i) {
            uint32_t units;
            pl.s[pl.n] = part_slot(parts[i].first, parts[i].second, blocks, &units);
            blocks += pl.s[pl.n++].count;
        }
        const hipError_t e = launch_event_parts(pl, blocks, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

extern "C" {

const char* mc_last_error(void) { return g_err.c_str(); }

void mc_params_default(mc_params* p)
{
    if (!p) return;
    std::memset(p, 0, sizeof *p);
    p->n_molecules = 1000;
    p->precision = MC_FP64;
    p->density = 1.2;
    p->temperature = 3.0;
    p->sigma[0] = 0.9;
    p->sigma[1] = 1.0;
    p->sigma[2] = 1.1;
    p->bond_length = 0.0;
    p->p_flip = 0.2;
    p->p_translate = 0.4;
    p->max_displacement = 0.1;
    p->max_rotation = 0.2;
    p->seed = 1;
    p->colours_per_axis = 0;
    p->cells_per_side = 0;
    p->resum_interval = 100;
    p->obs_interval = 10;
    p->gofr_interval = 100;
    p->obs_start = 0;
    p->max_samples = 4096;
    p->gofr_dr = 0.02;
    p->barrier_polls = 0;
    p->fs_q = 7.4;     // first peak of the site structure factor (Sec. III.B)
    p->fs_q_cm = 5.1;  // first peak of the centres' structure factor
    p->workgroups = 0;
}

int mc_geometry(const mc_params* p, double* box, uint32_t* k, uint32_t* nc)
{
    Geometry g;
    const int rc = geometry(p, &g);
    if (rc) return rc;
    if (box) *box = g.L;
    if (k) *k = g.k;
    if (nc) *nc = g.nc;
    return MC_OK;
}

int mc_placement(const mc_params* p, int* resident, size_t* lds_bytes)
{
    Geometry g;
    const int rc = geometry(p, &g);
    if (rc) return rc;
    if (resident) *resident = g.resident ? 1 : 0;
    if (lds_bytes) *lds_bytes = g.lds;
    return MC_OK;
}

int mc_engine(const mc_params* p, int* engine, uint32_t* workgroups)
{
    Geometry g;
    const int rc = geometry(p, &g);
    if (rc) return rc;
    if (engine) *engine = g.team ? MC_ENGINE_SPREAD : (g.resident ? MC_ENGINE_LDS : MC_ENGINE_HBM);
    if (workgroups) *workgroups = g.team ? g.team_blocks : 1u;
    return MC_OK;
}

int mc_required_bytes(const mc_params* p, size_t* bytes)
{
    Geometry g;
    const int rc = geometry(p, &g);
    if (rc) return rc;
    if (!bytes) return fail(MC_EINVAL, "null output");
    *bytes = buf_layout(p, g).total;
    return MC_OK;
}

int mc_init_system(const mc_params* p, const double* com, const double* quat, const uint8_t* types,
                   void* device_buf, size_t buf_bytes, void* hip_stream, mc_system** out)
{
    if (!out) return fail(MC_EINVAL, "null output handle");
    *out = nullptr;
    Geometry g;
    int rc = geometry(p, &g);
    if (rc) return rc;
    const bool lattice = !com && !quat && !types;
    if (!lattice && !(com && quat && types))
        return fail(MC_EINVAL, "give com, quat and types together, or none of them");
    if (lattice) {
        uint32_t n = 1;
        while ((n + 1) * (n + 1) * (n + 1) <= p->n_molecules) ++n;
        if (n * n * n != p->n_molecules)
            return fail(MC_EINVAL, "lattice start needs n_molecules = n^3 (got %u)", p->n_molecules);
    }
    if (!device_buf) return fail(MC_EINVAL, "null device buffer");
    if (((uintptr_t)device_buf & 255u) != 0) return fail(MC_EINVAL, "device buffer must be 256-byte aligned");
    const BufLayout lay = buf_layout(p, g);
    if (buf_bytes < lay.total)
        return fail(MC_ENOMEM, "device buffer of %zu bytes, %zu needed", buf_bytes, lay.total);

    mc_system* s = new mc_system();
    s->p = *p;
    s->g = g;
    s->lay = lay;
    s->buf = (uint8_t*)device_buf;
    s->stream = (hipStream_t)hip_stream;
    s->sweep = 0;
    s->batch = nullptr;
    s->timing = false;
    SysDev& D = s->host;
    std::memset(&D, 0, sizeof D);
    uint8_t* b = s->buf;
    D.M = p->n_molecules;
    D.k = g.k;
    D.nc = g.nc;
    D.ncell = g.ncell;
    D.precision = p->precision;
    D.resident = g.resident ? 1u : 0u;
    D.seed_lo = (uint32_t)p->seed;
    D.seed_hi = (uint32_t)(p->seed >> 32);
    D.L = g.L;
    D.w = g.L / (double)g.nc;
    D.T = p->temperature;
    D.p_flip = p->p_flip;
    D.p_ft = p->p_flip + p->p_translate;
    D.dmax = p->max_displacement;
    D.rot_max = p->max_rotation;
    const double reach = g.reach * (1.0 + 1e-9);
    D.reach2 = reach * reach;
    D.radius = g.radius;
    D.rc2_factor = std::cbrt(2.0);
    const double body[9] = {g.radius, 0.0, 0.0, -0.5 * g.radius, 0.5 * g.bond, 0.0,
                            -0.5 * g.radius, -0.5 * g.bond, 0.0};
    std::memcpy(D.body, body, sizeof body);
    for (int i = 0; i < 3; ++i) D.sigma[i] = p->sigma[i];
    D.resum_interval = p->resum_interval;
    D.obs_interval = p->obs_interval;
    D.gofr_interval = p->gofr_interval;
    D.obs_start = p->obs_start;
    D.max_samples = p->max_samples;
    const double rmax = std::min(0.5 * g.L, 5.0);
    uint32_t nb = (uint32_t)std::floor(rmax / p->gofr_dr + 1e-6);
    if (nb > (uint32_t)kGofrBins) nb = kGofrBins;
    D.gofr_nbins = nb;
    D.gofr_dr = p->gofr_dr;
    D.barrier_polls = p->barrier_polls ? p->barrier_polls : (1u << 23);
    D.near_cap = g.near_cap;
    D.gofr_rmax = rmax;
    D.lds_bytes = (uint32_t)g.lds;
    D.com = (double*)(b + lay.com);
    D.quat = (double*)(b + lay.quat);
    D.types = (uint32_t*)(b + lay.types);
    D.u0 = (double*)(b + lay.u0);
    D.kref = (uint8_t*)(b + lay.kref);
    D.stats = (Stats*)(b + lay.stats);
    D.e_samples = (double*)(b + lay.esamp);
    D.drift_samples = (double*)(b + lay.dsamp);
    D.gofr_all = (uint64_t*)(b + lay.gall);
    D.gofr_inter = (uint64_t*)(b + lay.ginter);
    D.c2 = (double*)(b + lay.c2);
    D.c2_sweep = (uint64_t*)(b + lay.c2s);
    D.img = (int32_t*)(b + lay.img);
    D.r0 = (double*)(b + lay.r0);
    D.o0 = (double*)(b + lay.o0);
    D.fs = (double*)(b + lay.fs);
    D.fs_cm = (double*)(b + lay.fscm);
    D.mom = (double*)(b + lay.mom);
    D.fs_q = p->fs_q;
    D.fs_q_cm = p->fs_q_cm;
    D.props = (void*)(b + lay.props);
    D.g_part = (double*)(b + lay.gpart);
    if (g.team_arrays()) {
        D.g_site = (void*)(b + lay.gsite);
        D.g_cell = (uint32_t*)(b + lay.gcell);
        D.g_cellid = (uint16_t*)(b + lay.gcellid);
        D.g_list = (uint16_t*)(b + lay.glist);
        D.g_cnt = (uint32_t*)(b + lay.gcnt);
        D.g_ecell = (double*)(b + lay.gecell);
        D.g_bar = (uint32_t*)(b + lay.gbar);
    }
    s->dev = (SysDev*)(b + lay.sys);

    auto bail = [&](int code) {
        delete s;
        return code;
    };
    hipError_t e = hipMemsetAsync(device_buf, 0, lay.total, s->stream);
    if (e != hipSuccess) return bail(fail(MC_EDEVICE, "hipMemsetAsync: %s", hipGetErrorString(e)));
    if ((rc = upload_desc(s))) return bail(rc);
    if (lattice) {
        e = launch_init_lattice(s->dev, p->n_molecules, s->stream);
        if (e != hipSuccess) return bail(fail(MC_EDEVICE, "lattice kernel: %s", hipGetErrorString(e)));
    } else if ((rc = upload_state(s, com, quat, types))) {
        return bail(rc);
    }
    s->origin = 0;
    if ((rc = launch_events_one(s, kFlagResumSet | kFlagObsReset))) return bail(rc);
    Stats st;
    if ((rc = read_stats(s, &st))) return bail(rc);
    if (!std::isfinite(st.e_acc))
        return bail(fail(MC_ENONFINITE, "initial energy is not finite (overlapping sites)"));
    *out = s;
    return MC_OK;
}

int mc_sweep(mc_system* s, uint64_t n)
{
    TraceRange tr("mc_sweep");
    if (!s) return fail(MC_EINVAL, "null system");
    if (s->batch) return fail(MC_EBUSY, "system is in a batch");
    return advance(s, n);
}

int mc_energy(mc_system* s, double* e_total, double* e_per_molecule, double* drift)
{
    TraceRange tr("mc_energy");
    if (!s) return fail(MC_EINVAL, "null system");
    if (s->batch) return fail(MC_EBUSY, "system is in a batch");
    int rc = launch_events_one(s, kFlagResumReport);
    if (rc) return rc;
    Stats st;
    if ((rc = read_stats(s, &st))) return rc;
    if (e_total) *e_total = st.e_resum;
    if (e_per_molecule) *e_per_molecule = st.e_resum / (double)s->p.n_molecules;
    if (drift) *drift = st.e_acc - st.e_resum;
    if (!std::isfinite(st.e_resum)) return fail(MC_ENONFINITE, "energy is not finite");
    return MC_OK;
}

namespace {

// Eq. (3): g(r) = counts / (frames N rho (4 pi / 3) (r_{b+1}^3 - r_b^3)) with
// N = 3 M sites, rho = N / L^3 and the exact shell volume of bin b.
void gofr_normalise(const mc_system* s, mc_obs* o)
{
    const double N = 3.0 * (double)s->p.n_molecules;
    const double rho = N / (s->g.L * s->g.L * s->g.L);
    const double frames = (double)o->n_gofr_frames;
    const double dr = o->gofr_dr;
    for (uint32_t b = 0; b < o->gofr_nbins && frames > 0.0; ++b) {
        const double r0 = dr * (double)b, r1 = dr * (double)(b + 1);
        const double shell = 4.0 * M_PI / 3.0 * (r1 * r1 * r1 - r0 * r0 * r0);
        const double ideal = frames * N * rho * shell;
        o->gofr_norm_all[b] = (double)o->gofr_all[b] / ideal;
        o->gofr_norm_inter[b] = (double)o->gofr_inter[b] / ideal;
    }
}

}  // namespace

int mc_observables(mc_system* s, mc_obs* o)
{
    if (!s || !o) return fail(MC_EINVAL, "null argument");
    Stats st;
    std::vector<uint8_t> raw;
    if (int rc = read_block(s, s->lay.com, &raw, &st)) return rc;
    const uint8_t* at = raw.data() - s->lay.stats;
    std::memset(o, 0, sizeof *o);
    o->sweep = st.sweep;
    for (int i = 0; i < 3; ++i) {
        o->attempts[i] = st.attempts[i];
        o->accepts[i] = st.accepts[i];
    }
    o->exits = st.exits;
    o->pair_terms = st.pair_terms;
    o->pair_tests = st.pair_tests;
    o->near_overflows = st.near_overflows;
    o->e_acc = st.e_acc;
    o->e_resum = st.e_resum;
    o->drift = st.drift;
    o->max_abs_drift = st.max_abs_drift;
    o->resum_sweep = st.resum_sweep;
    o->n_energy_samples = st.n_e;
    o->n_drift_samples = st.n_drift;
    o->energy_sum = st.e_sum;
    o->energy_sumsq = st.e_sumsq;
    o->n_gofr_frames = st.n_gofr;
    o->gofr_nbins = s->host.gofr_nbins;
    o->gofr_dr = s->host.gofr_dr;
    o->gofr_rmax = s->host.gofr_rmax;
    o->n_c2 = st.n_c2;
    const BufLayout& l = s->lay;
    std::memcpy(o->gofr_all, at + l.gall, sizeof o->gofr_all);
    std::memcpy(o->gofr_inter, at + l.ginter, sizeof o->gofr_inter);
    std::memcpy(o->c2, at + l.c2, sizeof o->c2);
    std::memcpy(o->fs, at + l.fs, sizeof o->fs);
    std::memcpy(o->fs_cm, at + l.fscm, sizeof o->fs_cm);
    std::memcpy(o->c2_sq, at + l.mom, sizeof o->c2_sq);
    std::memcpy(o->fs_cm_sq, at + l.mom + kC2Max * sizeof(double), sizeof o->fs_cm_sq);
    std::memcpy(o->c2_fs_cm, at + l.mom + 2 * kC2Max * sizeof(double), sizeof o->c2_fs_cm);
    std::memcpy(o->fs_sq, at + l.mom + 3 * kC2Max * sizeof(double), sizeof o->fs_sq);
    std::memcpy(o->c2_sweep, at + l.c2s, sizeof o->c2_sweep);
    gofr_normalise(s, o);
    return MC_OK;
}

int mc_samples(mc_system* s, double* energy, double* drift, size_t cap, size_t* n_energy,
               size_t* n_drift)
{
    if (!s) return fail(MC_EINVAL, "null system");
    Stats st;
    int rc = read_stats(s, &st);
    if (rc) return rc;
    const size_t ne = std::min<size_t>({(size_t)st.n_e, (size_t)s->p.max_samples, cap});
    const size_t nd = std::min<size_t>({(size_t)st.n_drift, (size_t)s->p.max_samples, cap});
    if (energy && ne)
        HIPCHK(hipMemcpyAsync(energy, s->host.e_samples, ne * sizeof(double), hipMemcpyDeviceToHost, s->stream));
    if (drift && nd)
        HIPCHK(hipMemcpyAsync(drift, s->host.drift_samples, nd * sizeof(double), hipMemcpyDeviceToHost, s->stream));
    HIPCHK(hipStreamSynchronize(s->stream));
    if (n_energy) *n_energy = ne;
    if (n_drift) *n_drift = nd;
    return MC_OK;
}

int mc_reset_observables(mc_system* s)
{
    if (!s) return fail(MC_EINVAL, "null system");
    if (s->batch) return fail(MC_EBUSY, "system is in a batch");
    s->origin = s->sweep;
    return launch_events_one(s, kFlagObsReset);
}

int mc_get_state(mc_system* s, double* com, double* quat, uint8_t* types, uint64_t* sweep,
                 double* e_acc)
{
    if (!s) return fail(MC_EINVAL, "null system");
    const size_t M = s->p.n_molecules;
    Stats st;
    std::vector<uint8_t> raw;
    if (int rc = read_block(s, s->lay.types + M * sizeof(uint32_t), &raw, &st)) return rc;
    const uint8_t* at = raw.data() - s->lay.stats;
    const double* c = (const double*)(at + s->lay.com);
    const double* q = (const double*)(at + s->lay.quat);
    const uint32_t* t = (const uint32_t*)(at + s->lay.types);
    for (size_t m = 0; m < M; ++m) {
        if (com)
            for (int a = 0; a < 3; ++a) com[3 * m + a] = c[a * M + m];
        if (quat)
            for (int a = 0; a < 4; ++a) quat[4 * m + a] = q[a * M + m];
        if (types)
            for (int a = 0; a < 3; ++a) types[3 * m + a] = (uint8_t)((t[m] >> (8 * a)) & 0xFFu);
    }
    if (sweep) *sweep = st.sweep;
    if (e_acc) *e_acc = st.e_acc;
    return MC_OK;
}

int mc_set_state(mc_system* s, const double* com, const double* quat, const uint8_t* types,
                 uint64_t sweep, double e_acc)
{
    if (!s || !com || !quat || !types) return fail(MC_EINVAL, "null argument");
    if (s->batch) return fail(MC_EBUSY, "system is in a batch");
    int rc = upload_state(s, com, quat, types);
    if (rc) return rc;
    // the new state has crossed no periodic images yet
    HIPCHK(hipMemsetAsync(s->host.img, 0, 3 * sizeof(int32_t) * s->p.n_molecules, s->stream));
    Stats st;
    if ((rc = read_stats(s, &st))) return rc;
    st.sweep = sweep;
    st.e_acc = std::isnan(e_acc) ? 0.0 : e_acc;
    if (sweep < s->origin) {
        st.obs_origin = sweep;
        s->origin = sweep;
    }
    if ((rc = write_stats(s, &st))) return rc;
    s->sweep = sweep;
    if (std::isnan(e_acc)) {
        if ((rc = launch_events_one(s, kFlagResumSet))) return rc;
        if ((rc = read_stats(s, &st))) return rc;
        if (!std::isfinite(st.e_acc)) return fail(MC_ENONFINITE, "energy of the new state is not finite");
    }
    return MC_OK;
}

int mc_decision_log(mc_system* s, void* device_records, size_t capacity)
{
    if (!s) return fail(MC_EINVAL, "null system");
    if (s->batch) return fail(MC_EBUSY, "system is in a batch");
    Stats st;
    int rc = read_stats(s, &st);
    if (rc) return rc;
    s->host.log = device_records;
    s->host.log_sweep0 = st.sweep;
    s->host.log_sweeps = device_records ? capacity / s->p.n_molecules : 0;
    return upload_desc(s);
}

int mc_timing_enable(mc_system* s, int enable)
{
    if (!s) return fail(MC_EINVAL, "null system");
    HIPCHK(hipStreamSynchronize(s->stream));
    for (auto& pr : s->ev_sweep) { s->ev_pool.push_back(pr.first); s->ev_pool.push_back(pr.second); }
    for (auto& pr : s->ev_event) { s->ev_pool.push_back(pr.first); s->ev_pool.push_back(pr.second); }
    s->ev_sweep.clear();
    s->ev_event.clear();
    s->timing = enable != 0;
    return MC_OK;
}

int mc_timing_read(mc_system* s, double* sweep_ms, uint64_t* sweep_launches, double* event_ms,
                   uint64_t* event_launches)
{
    if (!s) return fail(MC_EINVAL, "null system");
    HIPCHK(hipStreamSynchronize(s->stream));
    double t[2] = {0.0, 0.0};
    const std::vector<std::pair<hipEvent_t, hipEvent_t>>* v[2] = {&s->ev_sweep, &s->ev_event};
    for (int i = 0; i < 2; ++i)
        for (auto& pr : *v[i]) {
            float ms = 0.f;
            HIPCHK(hipEventElapsedTime(&ms, pr.first, pr.second));
            t[i] += ms;
        }
    if (sweep_ms) *sweep_ms = t[0];
    if (sweep_launches) *sweep_launches = s->ev_sweep.size();
    if (event_ms) *event_ms = t[1];
    if (event_launches) *event_launches = s->ev_event.size();
    return MC_OK;
}

void mc_destroy(mc_system* s)
{
    if (!s) return;
    // no kernel of the system may still run when the caller frees its buffer:
    // wait for its own stream and, inside a batch, for the batch's streams
    (void)hipStreamSynchronize(s->stream);
    if (s->batch) {
        (void)hipStreamSynchronize(s->batch->stream);
        if (s->batch->stream2) (void)hipStreamSynchronize(s->batch->stream2);
        if (s->batch->stream3) (void)hipStreamSynchronize(s->batch->stream3);
    }
    for (auto& pr : s->ev_sweep) { s->ev_pool.push_back(pr.first); s->ev_pool.push_back(pr.second); }
    for (auto& pr : s->ev_event) { s->ev_pool.push_back(pr.first); s->ev_pool.push_back(pr.second); }
    for (hipEvent_t e : s->ev_pool) (void)hipEventDestroy(e);
    if (s->batch) {
        mc_batch* b = s->batch;
        for (size_t i = 0; i < b->sys.size(); ++i)
            if (b->sys[i] == s) b->sys[i] = nullptr;
    }
    delete s;
}

// ------------------------------------------------- analysis of several runs --

namespace {

// First time the samples c[0..n) fall to `level`: linear in ln t between the
// two samples around the crossing; NaN when they never do.
double crossing_time(const uint64_t* t, const double* c, uint32_t n, double level)
{
    for (uint32_t j = 1; j < n; ++j) {
        if (c[j] <= level && level < c[j - 1]) {
            const double x0 = std::log((double)t[j - 1]), x1 = std::log((double)t[j]);
            return std::exp(x0 + (x1 - x0) * (c[j - 1] - level) / (c[j - 1] - c[j]));
        }
    }
    return std::numeric_limits<double>::quiet_NaN();
}

}  // namespace

namespace {

// mc_dynamics and mcf_dynamics: sites = particles of F_s per molecule (the
// susceptibility of F_s counts n M of them).
int dynamics_of(const mc_obs* runs, size_t n_runs, uint32_t n_molecules, uint32_t sites, mc_dyn* out)
{
    if (!runs || !out || n_runs == 0 || n_molecules == 0 || sites == 0) return fail(MC_EINVAL, "bad arguments");
    std::memset(out, 0, sizeof *out);
    const uint32_t n = runs[0].n_c2;
    if (n > MC_C2_MAX) return fail(MC_EINVAL, "n_c2 above %d", MC_C2_MAX);
    for (size_t r = 1; r < n_runs; ++r) {
        if (runs[r].n_c2 != n) return fail(MC_EINVAL, "run %zu has %u samples, run 0 %u", r, runs[r].n_c2, n);
        for (uint32_t j = 0; j < n; ++j)
            if (runs[r].c2_sweep[j] != runs[0].c2_sweep[j])
                return fail(MC_EINVAL, "run %zu samples other sweeps than run 0", r);
    }
    out->n_times = n;
    out->n_runs = (uint32_t)n_runs;
    const double R = (double)n_runs, M = (double)n_molecules;
    for (uint32_t j = 0; j < n; ++j) {
        out->t[j] = runs[0].c2_sweep[j];
        double m[3] = {0, 0, 0}, m2[3] = {0, 0, 0}, sq[3] = {0, 0, 0}, cross = 0.0;
        for (size_t r = 0; r < n_runs; ++r) {
            const mc_obs& o = runs[r];
            const double v[3] = {o.c2[j], o.fs[j], o.fs_cm[j]};
            const double q[3] = {o.c2_sq[j], o.fs_sq[j], o.fs_cm_sq[j]};
            for (int a = 0; a < 3; ++a) {
                m[a] += v[a];
                m2[a] += v[a] * v[a];
                sq[a] += q[a];
            }
            cross += o.c2_fs_cm[j];
        }
        double chi[3], self[3];
        const double npart[3] = {M, (double)sites * M, M};
        for (int a = 0; a < 3; ++a) {
            m[a] /= R;
            chi[a] = npart[a] * (m2[a] / R - m[a] * m[a]);
            self[a] = sq[a] / R - m[a] * m[a];
        }
        out->c2[j] = m[0]; out->fs[j] = m[1]; out->fs_cm[j] = m[2];
        out->chi4_c2[j] = chi[0]; out->chi4_fs[j] = chi[1]; out->chi4_fs_cm[j] = chi[2];
        out->chi4s_c2[j] = self[0]; out->chi4s_fs[j] = self[1]; out->chi4s_fs_cm[j] = self[2];
        out->rho[j] = (cross / R - m[0] * m[2]) / std::sqrt(self[0] * self[2]);
    }
    const double e1 = std::exp(-1.0);
    out->tau_c2 = crossing_time(out->t, out->c2, n, e1);
    out->tau_fs = crossing_time(out->t, out->fs, n, e1);
    out->tau_fs_cm = crossing_time(out->t, out->fs_cm, n, e1);
    return MC_OK;
}

}  // namespace

int mc_dynamics(const mc_obs* runs, size_t n_runs, uint32_t n_molecules, mc_dyn* out)
{
    return dynamics_of(runs, n_runs, n_molecules, 3u, out);
}

int mcf_dynamics(const mc_obs* runs, size_t n_runs, uint32_t n_molecules, uint32_t atoms_per_molecule,
                 mc_dyn* out)
{
    if (atoms_per_molecule < 3 || atoms_per_molecule > 4) return fail(MC_EINVAL, "atoms_per_molecule must be 3 or 4");
    return dynamics_of(runs, n_runs, n_molecules, atoms_per_molecule, out);
}

// ------------------------------------------------------------------ batches --

namespace {

// The batch's device slot tables in the caller's buffer, double-buffered:
// per parity [resident | non-resident | events] x max_slots Slots, max_slots
// SpreadSlots, max_slots Slots of the multi-workgroup engine's events.
struct BatchLayout {
    size_t slots[2], spread[2], ev2[2], total;
};

BatchLayout batch_layout(uint32_t max_slots)
{
    BatchLayout l{};
    size_t o = 0;
    for (int i = 0; i < 2; ++i) {
        l.slots[i] = o;  o = al(o + 3 * sizeof(Slot) * max_slots);
        l.spread[i] = o; o = al(o + sizeof(SpreadSlot) * max_slots);
        l.ev2[i] = o;    o = al(o + sizeof(Slot) * max_slots);
    }
    l.total = o;
    return l;
}

constexpr uint32_t kMaxBatchSlots = 1u << 16;

}  // namespace

int mc_batch_required_bytes(uint32_t max_slots, size_t* bytes)
{
    if (!bytes || max_slots == 0 || max_slots > kMaxBatchSlots)
        return fail(MC_EINVAL, "max_slots must be in [1, %u] and bytes non-null", kMaxBatchSlots);
    *bytes = batch_layout(max_slots).total;
    return MC_OK;
}

int mc_batch_create(uint32_t max_slots, uint32_t precision, void* device_buf, size_t buf_bytes,
                    void* hip_stream, void* hip_stream_aux, mc_batch** out)
{
    if (!out) return fail(MC_EINVAL, "null output handle");
    *out = nullptr;
    if (max_slots == 0 || max_slots > kMaxBatchSlots)
        return fail(MC_EINVAL, "max_slots must be in [1, %u]", kMaxBatchSlots);
    if (precision != MC_FP64 && precision != MC_FP32_DE) return fail(MC_EINVAL, "bad precision");
    if (!device_buf) return fail(MC_EINVAL, "null device buffer");
    if (((uintptr_t)device_buf & 255u) != 0) return fail(MC_EINVAL, "device buffer must be 256-byte aligned");
    const BatchLayout lay = batch_layout(max_slots);
    if (buf_bytes < lay.total)
        return fail(MC_ENOMEM, "device buffer of %zu bytes, %zu needed", buf_bytes, lay.total);
    mc_batch* b = new mc_batch();
    b->max_slots = max_slots;
    b->precision = precision;
    b->stream = (hipStream_t)hip_stream;
    b->sys.assign(max_slots, nullptr);
    b->remaining.assign(max_slots, 0);
    b->parity = 0;
    b->stream2 = nullptr;
    b->go = b->done = nullptr;
    b->stream3 = nullptr;
    b->go3 = b->done3 = nullptr;
    b->spread_max = 0;
    b->ncu = 1;
    b->wg_limit = 0;
    b->turn = 0;
    for (int c = 0; c < 4; ++c) {
        b->ms_per_cycle[c] = ms_per_model_cycle() * kCycleRatio[precision == MC_FP64][c];
        b->pred[c] = 0.0;
        b->t_beg[c] = b->t_end[c] = nullptr;
    }
    for (int i = 0; i < 2; ++i) {
        b->dev_slots[i] = nullptr;
        b->host_slots[i] = nullptr;
        b->pending[i] = false;
        b->copied[i] = nullptr;
        b->dev_spread[i] = nullptr;
        b->host_spread[i] = nullptr;
        b->dev_ev2[i] = nullptr;
        b->host_ev2[i] = nullptr;
        b->copied2[i] = nullptr;
        b->pending2[i] = false;
    }
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        mc_batch_destroy(b);
        return fail(MC_EDEVICE, "could not query the device");
    }
    const size_t table = std::min(max_slots, (uint32_t)std::max(1, ncu));  // systems on several workgroups
    uint8_t* dbuf = (uint8_t*)device_buf;
    for (int i = 0; i < 2; ++i) {
        // slot tables: one per residency class, double-buffered; the device
        // copies in the caller's buffer, their pinned host staging owned here
        b->dev_slots[i] = (Slot*)(dbuf + lay.slots[i]);
        b->dev_spread[i] = (SpreadSlot*)(dbuf + lay.spread[i]);
        b->dev_ev2[i] = (Slot*)(dbuf + lay.ev2[i]);
        if (hipHostMalloc((void**)&b->host_slots[i], 3 * sizeof(Slot) * max_slots, hipHostMallocDefault) != hipSuccess ||
            hipEventCreateWithFlags(&b->copied[i], hipEventDisableTiming) != hipSuccess ||
            hipHostMalloc((void**)&b->host_spread[i], sizeof(SpreadSlot) * kRounds * table, hipHostMallocDefault) != hipSuccess ||
            hipHostMalloc((void**)&b->host_ev2[i], sizeof(Slot) * kRounds * table, hipHostMallocDefault) != hipSuccess ||
            hipEventCreateWithFlags(&b->copied2[i], hipEventDisableTiming) != hipSuccess) {
            mc_batch_destroy(b);
            return fail(MC_EDEVICE, "could not allocate the host staging of the slot tables");
        }
    }
    for (int c = 0; c < 4; ++c)
        if (hipEventCreate(&b->t_beg[c]) != hipSuccess || hipEventCreate(&b->t_end[c]) != hipSuccess) {
            mc_batch_destroy(b);
            return fail(MC_EDEVICE, "could not create the timing events");
        }
    b->stream2 = hip_stream_aux ? (hipStream_t)hip_stream_aux : b->stream;
    if (hipEventCreateWithFlags(&b->go, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&b->done, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&b->go3, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&b->done3, hipEventDisableTiming) != hipSuccess) {
        mc_batch_destroy(b);
        return fail(MC_EDEVICE, "could not create the stream events");
    }
    if (spread_max_blocks(&b->spread_max) != hipSuccess) {
        (void)hipGetLastError();
        b->spread_max = 0;
    }
    b->ncu = (uint32_t)ncu;
    b->wg_limit = (uint32_t)ncu;
    {
        // the first launch of a kernel carries one-time set-up costs: run the
        // sweep kernels once here with no system, so the batch's timing of its
        // own launches (its engine calibration) does not see them
        const bool fp64 = precision == MC_FP64;
        Slot none{};
        SpreadSlot snone{};
        hipError_t e = launch_sweeps(fp64, true, nullptr, none, 1, 0, b->stream, true);
        if (e == hipSuccess) e = launch_sweeps(fp64, false, nullptr, none, 1, 0, b->stream, true);
        for (const SpreadMode m : {kSpreadTeam, kSpreadWaves, kSpreadCrew, kSpreadCrewWaves})
            if (e == hipSuccess && b->spread_max >= 2) e = launch_spread(fp64, m, nullptr, 0, snone, 1, 0, b->stream);
        if (e != hipSuccess) {
            mc_batch_destroy(b);
            return fail(MC_EDEVICE, "warm-up launch: %s", hipGetErrorString(e));
        }
    }
    *out = b;
    return MC_OK;
}

int mc_batch_add(mc_batch* b, mc_system* s, uint64_t n_sweeps, uint32_t* slot)
{
    if (!b || !s) return fail(MC_EINVAL, "null argument");
    if (s->batch) return fail(MC_EINVAL, "system is already in a batch");
    if (s->p.precision != b->precision) return fail(MC_EINVAL, "precision differs from the batch's");
    for (uint32_t i = 0; i < b->max_slots; ++i) {
        if (!b->sys[i]) {
            b->sys[i] = s;
            b->remaining[i] = n_sweeps;
            s->batch = b;
            if (slot) *slot = i;
            return MC_OK;
        }
    }
    return fail(MC_EBUSY, "no free slot");
}

int mc_batch_set_workgroups(mc_batch* b, uint32_t max_workgroups)
{
    if (!b) return fail(MC_EINVAL, "null batch");
    b->wg_limit = max_workgroups ? max_workgroups : b->ncu;
    return MC_OK;
}

int mc_batch_set_hbm_stream(mc_batch* b, void* hip_stream)
{
    if (!b) return fail(MC_EINVAL, "null batch");
    // the previous run's launch on the old stream was joined into the batch
    // stream, so later work there already follows it
    b->stream3 = (hipStream_t)hip_stream == b->stream ? nullptr : (hipStream_t)hip_stream;
    return MC_OK;
}

int mc_batch_run(mc_batch* b, uint64_t max_moves_per_slot, uint32_t* n_launched)
{
    TraceRange tr("mc_batch_run");
    if (!b) return fail(MC_EINVAL, "null batch");
    const int par = b->parity;
    b->parity ^= 1;
    if (b->pending[par]) {
        HIPCHK(hipEventSynchronize(b->copied[par]));
        b->pending[par] = false;
    }
    if (b->pending2[par]) {
        HIPCHK(hipEventSynchronize(b->copied2[par]));
        b->pending2[par] = false;
    }
    Slot* hs = b->host_slots[par];
    const uint32_t S = b->max_slots;
    const bool fp64 = b->precision == MC_FP64;

    // calibration from the launches of the last run that have finished
    for (int c = 0; c < 4; ++c) {
        if (b->pred[c] <= 0.0) continue;
        if (hipEventQuery(b->t_end[c]) != hipSuccess) {
            (void)hipGetLastError();  // not finished: no sample
            continue;
        }
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, b->t_beg[c], b->t_end[c]) == hipSuccess && ms > 0.f) {
            const double f = b->ms_per_cycle[c];
            const double r = std::min(4.0 * f, std::max(0.25 * f, (double)ms / b->pred[c]));
            b->ms_per_cycle[c] = 0.5 * f + 0.5 * r;
        }
        (void)hipGetLastError();
        b->pred[c] = 0.0;
    }
    // every launch of a run is sized to the time the reference system takes
    // for max_moves_per_slot moves
    double t_slice = slice_time(max_moves_per_slot) * ms_per_model_cycle();
    double pred[4] = {0.0, 0.0, 0.0, 0.0};

    // Engine of every system for this run.  Each system needs one workgroup;
    // the workgroups left over (up to the batch's limit) go to systems that can
    // run on the multi-workgroup engine (below).  The engines make the same
    // decisions, so a system may change engine from run to run.
    std::vector<uint32_t> active;
    for (uint32_t i = 0; i < S; ++i)
        if (b->sys[i] && b->remaining[i] != 0) active.push_back(i);
    // More systems than workgroups at once: a run takes whole rounds of them
    // (the largest multiple of the limit), the systems in turn from run to
    // run, so that no run ends with a partly filled round of workgroups
    if (b->wg_limit && active.size() > b->wg_limit) {
        const size_t A = active.size(), m = (A / b->wg_limit) * b->wg_limit;
        std::vector<uint32_t> chosen;
        chosen.reserve(m);
        for (size_t i = 0; i < m; ++i) chosen.push_back(active[(b->turn + i) % A]);
        b->turn = (uint32_t)((b->turn + m) % A);
        std::sort(chosen.begin(), chosen.end());
        active.swap(chosen);
    }
    // A run of all remaining sweeps: the earliest end T that the engines' models
    // allow.  Within T a system takes its own engine's one workgroup, or the
    // way on several that costs the fewest workgroups times time; the systems
    // on one workgroup with their state in LDS share as many workgroups as their
    // times fill, one after another (a system each left the compute units of the
    // short ones idle: 40 sweeps of 256 replicas of 216 - 1728 molecules took 24.4 ms,
    // the longest of them, with 12.6 ms of work per compute unit; 50 sweeps of 24
    // systems of 125 - 8000 molecules 22 ms instead of 13, with the greedy division
    // that the time slices below keep, whose lengths come out alike anyway).
    std::vector<uint32_t> nblk(S, 0);
    std::vector<char> by_wave(S, 0);
    uint32_t lds_blocks = S;  // workgroups of the systems on one with the state in LDS
    const bool whole = max_moves_per_slot == 0 && b->spread_max >= 2 && b->stream2 != b->stream &&
                       !active.empty() && b->wg_limit >= 2;
    if (whole) {
        struct Option {
            double time;
            uint32_t nb;
            char wave;
        };
        std::vector<std::vector<Option>> opts(active.size());
        double hi = 0.0, lo = 0.0;
        for (size_t x = 0; x < active.size(); ++x) {
            const mc_system* s = b->sys[active[x]];
            const double rem = (double)b->remaining[active[x]];
            const double one = rem * s->g.sweep_cost * b->ms_per_cycle[s->g.resident ? 0 : 1];
            opts[x].push_back(Option{one, 0u, 0});
            hi = std::max(hi, one);
            lo += one;
            if (!s->g.team_arrays()) continue;
            const uint32_t na = s->g.nc / s->g.k, nact = na * na * na, M = s->p.n_molecules;
            for (const char w : {0, 1}) {
                const uint32_t cells = w ? s->g.wave_fit : 1u;  // of a workgroup at once
                if (w && cells < 2) continue;
                uint32_t last = 0;
                auto offer = [&](uint32_t n) {
                    const uint32_t nb = std::min(s->g.team_blocks, n);
                    if (nb == last) return;
                    last = nb;
                    const double t = rem * s->g.spread_cycles(M, nb, w) * b->ms_per_cycle[w ? 3 : 2];
                    // (the model is off by about that much, see kCycleRatio)
                    if (t < 0.9 * one) opts[x].push_back(Option{t, nb, w});
                };
                for (uint32_t r = (nact + cells - 1) / cells; r >= 1; r = std::min(r - 1, std::max(r / 2, 8u)))
                    offer((nact + cells * r - 1) / (cells * r));
                if (cells > 4u) offer((nact + 3u) / 4u);  // a wave for each SIMD
            }
        }
        // The workgroups of a launch go to the XCDs in turn, whether a compute unit
        // is free there or not, so a launch takes as many as a whole number of
        // turns has (all 256 in three launches left some waiting for a whole
        // system: 30 sweeps of 100 systems of 500 - 8000 molecules took 34.7 ms,
        // 21.2 so).
        constexpr uint32_t kXcds = 8;
        auto turns = [&](uint32_t n) { return (n + kXcds - 1) / kXcds * kXcds; };
        std::vector<uint32_t> pick(active.size(), 0), narrow(active.size(), 0), best, order;
        std::vector<double> times;
        uint32_t room = 0, best_room = 0;  // for the systems on one workgroup with their state in LDS
        // whether all can end by T, with the options into pick
        auto fits = [&](double T) {
            // each system's option of the least workgroups times time, and where
            // those are too many for the device, the narrowest for those that give
            // back most
            uint32_t count[3] = {0, 0, 0};  // a cell per workgroup, per wave, one with the state in HBM
            double area = 0.0;
            auto add = [&](size_t x, uint32_t o, int sign) {
                const Option& p = opts[x][o];
                if (p.nb) count[(int)p.wave] += (uint32_t)(sign * (int)p.nb);
                else if (b->sys[active[x]]->g.resident) area += sign * p.time;
                else count[2] += (uint32_t)sign;
            };
            order.clear();
            for (size_t x = 0; x < active.size(); ++x) {
                double least = std::numeric_limits<double>::infinity();
                uint32_t fewest = 0;
                for (uint32_t o = 0; o < opts[x].size(); ++o) {
                    const Option& p = opts[x][o];
                    if (p.time > T) continue;
                    const uint32_t n = std::max(p.nb, 1u);
                    const double a = p.time * n;
                    if (a < least) {
                        least = a;
                        pick[x] = o;
                    }
                    if (!fewest || n < fewest) {
                        fewest = n;
                        narrow[x] = o;
                    }
                }
                if (!fewest) return false;
                add(x, pick[x], 1);
                if (narrow[x] != pick[x]) order.push_back((uint32_t)x);
            }
            auto gain = [&](uint32_t x) { return opts[x][pick[x]].nb - std::max(opts[x][narrow[x]].nb, 1u); };
            std::sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return gain(x) > gain(y); });
            for (size_t next = 0;;) {
                const uint32_t held = count[0] + count[1] + count[2];
                const uint32_t taken = turns(count[0]) + turns(count[1]) + turns(count[2]);
                room = held < b->wg_limit && taken < b->ncu ? std::min(b->wg_limit - held, b->ncu - taken) : 0u;
                if (held <= b->wg_limit && taken <= b->ncu && area <= T * room) {
                    times.clear();
                    for (size_t x = 0; x < active.size(); ++x)
                        if (!opts[x][pick[x]].nb && b->sys[active[x]]->g.resident) times.push_back(opts[x][pick[x]].time);
                    std::sort(times.begin(), times.end(), std::greater<>());
                    if (times.empty() ||
                        longest_first(times, std::min(room, (uint32_t)times.size()), nullptr) <= 1.001 * T)
                        return true;
                }
                if (next == order.size()) return false;
                const uint32_t x = order[next++];
                add(x, pick[x], -1);
                add(x, narrow[x], 1);
                pick[x] = narrow[x];
            }
        };
        lo /= (double)b->wg_limit * 16.0;
        if (fits(hi)) {
            best = pick;
            best_room = room;
            for (int step = 0; step < 16; ++step) {
                const double T = std::sqrt(lo * hi);
                if (fits(T)) {
                    hi = T;
                    best = pick;
                    best_room = room;
                } else {
                    lo = T;
                }
            }
            lds_blocks = best_room;
            for (size_t x = 0; x < active.size(); ++x) {
                const Option& p = opts[x][best[x]];
                nblk[active[x]] = p.nb;
                by_wave[active[x]] = p.wave;
            }
        }
    }
    // Time slices: the spare compute units go to the systems that would otherwise finish
    // last: the one with the longest modelled time for its remaining sweeps
    // takes workgroups until one of its rounds of cells per colour is saved, and
    // so on while any are left.  (In proportion to the remaining work, a share
    // that saves no round is lost, and one slow system holds up the run.)  With
    // its workgroups a system has a cell per workgroup or a cell per wave,
    // whichever is modelled faster.
    if (b->spread_max >= 2 && !whole) {
        struct Cand {
            double time;  // of the remaining sweeps on nb workgroups (0: its own engine's one)
            uint32_t slot, nb;
        };
        auto later = [](const Cand& a, const Cand& b) {
            return a.time < b.time || (a.time == b.time && a.slot > b.slot);
        };
        std::vector<Cand> heap;
        uint32_t left = b->wg_limit > active.size() ? b->wg_limit - (uint32_t)active.size() : 0u;
        uint32_t held = 0;
        for (uint32_t i : active) {
            const mc_system* s = b->sys[i];
            const double one = s->g.sweep_cost * b->ms_per_cycle[s->g.resident ? 0 : 1];
            if (s->g.team_arrays()) heap.push_back(Cand{(double)b->remaining[i] * one, i, 0u});
        }
        std::make_heap(heap.begin(), heap.end(), later);
        while (!heap.empty()) {
            std::pop_heap(heap.begin(), heap.end(), later);
            Cand c = heap.back();
            heap.pop_back();
            const mc_system* s = b->sys[c.slot];
            const uint32_t na = s->g.nc / s->g.k, nact = na * na * na, M = s->p.n_molecules, most = s->g.team_blocks;
            const double ms_one = b->ms_per_cycle[s->g.resident ? 0 : 1];
            // the fewest workgroups that save a round of one of the ways, and pay
            uint32_t want = 0;
            char wave = 0;
            double time = c.time;
            for (uint32_t nb = c.nb; nb < most && !want;) {
                uint32_t next = most;
                for (const uint32_t cells : {1u, s->g.wave_fit}) {  // of a workgroup at once
                    if (cells == 0u) continue;
                    const uint32_t rounds = nb ? (nact + cells * nb - 1) / (cells * nb) : nact + 1u;
                    if (rounds > 1) next = std::min(next, (nact + cells * (rounds - 1) - 1) / (cells * (rounds - 1)));
                }
                nb = std::min(most, std::max(nb + 1, next));
                for (const char w : {0, 1}) {
                    if (w && s->g.wave_fit < 2) continue;
                    const double ms = b->ms_per_cycle[w ? 3 : 2];
                    const double t = (double)b->remaining[c.slot] * s->g.spread_cycles(M, nb, w) * ms;
                    if (t < time && (c.nb || spread_pays(s->g, M, nb, w, ms_one, ms))) {
                        want = nb;
                        wave = w;
                        time = t;
                    }
                }
            }
            const uint32_t more = want - std::max(c.nb, 1u);
            if (!want || more > left || held + want - c.nb > b->spread_max) continue;  // as fast as it gets
            left -= more;
            held += want - c.nb;
            nblk[c.slot] = c.nb = want;
            by_wave[c.slot] = wave;
            c.time = time;
            heap.push_back(c);
            std::push_heap(heap.begin(), heap.end(), later);
        }
        // The two ways are two launches, the second beside the first on the third
        // stream.  Where that is taken (systems on one workgroup with their state
        // in HBM) or missing, a second one would start when the first has ended
        // and double the slice: one job of 125 molecules with a cell per
        // workgroup made slices of 54 ms out of 31 (a stream of 200 jobs:
        // 2.74e8 moves/s, 3.1 - 3.2e8 with one way).  Then all that have several
        // workgroups have a cell per wave, and the others stay on their one.  (A
        // system whose cell lists do not fit LDS has no other way; with one of
        // those both stay.)
        bool busy3 = !b->stream3 || b->stream2 == b->stream, movable = true;
        uint32_t by[2] = {0, 0};
        for (uint32_t i : active) {
            const mc_system* s = b->sys[i];
            if (nblk[i]) ++by[(int)by_wave[i]];
            else busy3 = busy3 || !s->g.resident;
            movable = movable && (!nblk[i] || s->g.resident || s->g.wave_fit >= 2);
        }
        if (busy3 && by[0] && by[1] && movable)
            for (uint32_t i : active) {
                const mc_system* s = b->sys[i];
                if (!nblk[i] || by_wave[i]) continue;
                by_wave[i] = s->g.wave_fit >= 2 &&
                             spread_pays(s->g, s->p.n_molecules, nblk[i], true, b->ms_per_cycle[0], b->ms_per_cycle[3]);
                if (!by_wave[i]) nblk[i] = 0;
            }
    }
    // More workgroups than compute units (the device's, not the batch's limit):
    // they take turns within the run, so each gets its part of the slice, and
    // what a launch then takes is mostly the others' time and no sample of its
    // own.  Taken as one, the class whose workgroups started first kept its 31 ms,
    // and the others' slices shrank to what was left: of 1024 jobs with 256 on the
    // multi-workgroup engine those in LDS had 3 ms of 46 (a stream of 2000 jobs: the
    // median job done after 16.6 s).
    uint32_t wanted = 0;
    for (uint32_t i : active) wanted += std::max(nblk[i], 1u);
    const bool crowded = max_moves_per_slot && wanted > b->ncu;
    if (crowded) t_slice *= (double)b->ncu / (double)wanted;
    uint32_t n[3] = {0, 0, 0};
    size_t lds[2] = {0, 0};
    // the O(M^2) event work of large systems goes to the event kernel over
    // many workgroups, whatever engine ran the sweeps
    std::vector<std::pair<mc_system*, uint32_t>> parts1;
    std::vector<std::pair<double, Slot>> ones;  // modelled cycles, entry
    // some system on one workgroup stops at a g(r) frame: those on several then
    // stop at theirs too, so that the next run has work for all compute units
    bool ones_left = false;
    std::vector<char> stopped(S, 0);
    auto event_slot = [&](mc_system* s, uint32_t f, std::vector<std::pair<mc_system*, uint32_t>>& parts) {
        Slot ev{};
        ev.sys = s->dev;
        ev.flags = f;
        // (many small systems fill the device with a workgroup each: 20 sweeps with
        // five g(r) frames of 128 systems of 300, 1000 and 1900 molecules take 6.1,
        // 12.4 and 24.5 ms so, 6.0, 10.5 and 19.0 on many workgroups; of 160, 6.3,
        // 12.5 and 30.5, and 6.8, 11.7 and 27.6; of 224, 6.4, 12.7 and 31.5, and
        // 7.4, 13.5 and 32.2)
        const uint32_t M = s->p.n_molecules;
        if ((M >= kInlineBelow || active.size() <= 128) && event_blocks(M) > 1 && (f & kOverPairs)) {
            parts.emplace_back(s, f);
            (void)part_slot(s, f, 0u, &ev.pad);
            ev.flags = f | kFlagParts;
        }
        return ev;
    };
    for (uint32_t i : active) {
        if (nblk[i]) continue;
        mc_system* s = b->sys[i];
        // a system on one workgroup whose events fit the one-workgroup event
        // kernel takes its scheduled re-sums and C_2 samples inside the sweep
        // kernel: its slice stops only at g(r) frames
        const bool inl = s->p.n_molecules < kInlineBelow;
        uint64_t k = std::min<uint64_t>(b->remaining[i], next_event(s, inl) - s->sweep);
        const int cls = s->g.resident ? 0 : 1;
        if (max_moves_per_slot) {
            // equal time slices: the time of max_moves_per_slot moves of the
            // 1000-molecule reference, in sweeps of this system
            const double cap = t_slice / (b->ms_per_cycle[cls] * s->g.sweep_cost);
            k = std::min<uint64_t>(k, std::max<uint64_t>(1, (uint64_t)cap));
        }
        Slot sl{};
        sl.sys = s->dev;
        sl.n_sweeps = k;
        sl.flags = inl ? kFlagInline : 0u;
        if (cls == 0) {
            ones.emplace_back((double)k * s->g.sweep_cost, sl);
        } else {
            pred[cls] = std::max(pred[cls], (double)k * s->g.sweep_cost);
            hs[cls * S + n[cls]++] = sl;
        }
        lds[cls] = std::max(lds[cls], s->g.lds);
        b->remaining[i] -= k;
        s->sweep += k;
        const uint32_t f = events_at(s, s->sweep) & (inl ? ~(kFlagResumPeriodic | kFlagC2) : ~0u);
        if (f) hs[2 * S + n[2]++] = event_slot(s, f, parts1);
        ones_left = ones_left || b->remaining[i] != 0;
    }
    // the longest first, each on the workgroup that is done first
    n[0] = (uint32_t)ones.size();
    {
        const uint32_t blocks = std::min(lds_blocks, n[0]);
        if (blocks < n[0])
            std::stable_sort(ones.begin(), ones.end(), [](const auto& x, const auto& y) { return x.first > y.first; });
        std::vector<double> times;
        for (const auto& x : ones) times.push_back(x.first);
        std::vector<uint32_t> taken, tail(blocks);
        if (blocks) pred[0] = longest_first(times, blocks, &taken);
        uint32_t more = blocks;
        for (uint32_t x = 0; x < n[0]; ++x) {
            // the first `blocks` entries start a workgroup each
            const uint32_t at = x < blocks ? x : more++;
            hs[at] = ones[x].second;
            if (x >= blocks) hs[tail[taken[x]]].pad = at + 1u;
            tail[taken[x]] = at;
        }
    }

    // A slice of every system on the multi-workgroup engine: those with a cell
    // per workgroup in one launch, those with a cell per wave in another, beside
    // it on the third stream where that is free, then the event work of both.
    std::vector<uint32_t> several;
    for (uint32_t i : active)
        if (nblk[i]) several.push_back(i);
    const size_t table = std::min(S, b->ncu);
    bool team_runs = false, wave_runs = false;
    auto spread_round = [&](uint32_t round) -> int {
        SpreadSlot* hsp = b->host_spread[par] + round * table;
        Slot* hev = b->host_ev2[par] + round * table;
        std::vector<std::pair<mc_system*, uint32_t>> parts;
        std::vector<SpreadSlot> by[2];
        uint32_t blocks[2] = {0, 0}, ne = 0;
        size_t need[2] = {0, 0}, crew_need[2] = {0, 0};
        double cycles[2] = {0.0, 0.0};
        bool lists[2] = {true, true};  // the cell lists of all systems fit the LDS
        for (uint32_t i : several) {
            mc_system* s = b->sys[i];
            uint64_t k = std::min<uint64_t>({b->remaining[i], next_event(s) - s->sweep, kCrewSweeps});
            if (k == 0 || (ones_left && stopped[i])) continue;
            const int w = by_wave[i];
            const double unit = s->g.spread_cycles(s->p.n_molecules, nblk[i], w);  // modelled cycles of a sweep
            if (max_moves_per_slot) {
                const double q = t_slice / (b->ms_per_cycle[2 + w] * unit);
                k = std::min<uint64_t>(k, std::max<uint64_t>(1, (uint64_t)q));
            }
            cycles[w] = std::max(cycles[w], (double)k * unit);
            SpreadSlot sl{};
            sl.sys = s->dev;
            sl.n_sweeps = k;
            sl.first_block = blocks[w];
            sl.n_blocks = nblk[i];
            sl.waves = w ? s->g.wave_fit : 0u;
            by[w].push_back(sl);
            blocks[w] += nblk[i];
            need[w] = std::max(need[w], spread_layout(fp64, s->g.lists, s->p.n_molecules, s->g.ncell, s->g.near_cap,
                                                      sl.waves).total);
            lists[w] = lists[w] && s->g.lists;
            crew_need[w] = std::max(crew_need[w], spread_layout(fp64, false, s->p.n_molecules, s->g.ncell,
                                                                s->g.near_cap, sl.waves).total);
            b->remaining[i] -= k;
            s->sweep += k;
            if (const uint32_t f = events_at(s, s->sweep)) {
                hev[ne++] = event_slot(s, f, parts);
                stopped[i] = stopped[i] || (f & kFlagGofr);
            }
        }
        const uint32_t nt = (uint32_t)by[0].size(), nw = (uint32_t)by[1].size();
        if (nt + nw == 0) return MC_OK;
        team_runs = team_runs || nt;
        wave_runs = wave_runs || nw;
        std::copy(by[0].begin(), by[0].end(), hsp);
        std::copy(by[1].begin(), by[1].end(), hsp + nt);
        const hipStream_t st = b->stream2;
        HIPCHK(hipMemcpyAsync(b->dev_spread[par], hsp, sizeof(SpreadSlot) * (nt + nw), hipMemcpyHostToDevice, st));
        if (ne) HIPCHK(hipMemcpyAsync(b->dev_ev2[par], hev, sizeof(Slot) * ne, hipMemcpyHostToDevice, st));
        HIPCHK(hipEventRecord(b->copied2[par], st));
        b->pending2[par] = true;
        const SpreadSlot none{};
        HIPCHK(launch_zero_barriers(b->dev_spread[par], nt + nw, st));
        const bool beside = nt && nw && b->stream3 && !n[1];
        const hipStream_t st_of[2] = {st, beside ? b->stream3 : st};
        if (beside) {
            HIPCHK(hipEventRecord(b->go3, st));
            HIPCHK(hipStreamWaitEvent(b->stream3, b->go3, 0));
        }
        for (int w = 1; w >= 0; --w) {
            if (by[w].empty()) continue;
            const SpreadMode mode = spread_mode(w, lists[w]);
            const bool sample = !crowded && cycles[w] > pred[2 + w];  // the longest slice is the run's sample
            if (sample) HIPCHK(hipEventRecord(b->t_beg[2 + w], st_of[w]));
            HIPCHK(launch_spread(fp64, mode, b->dev_spread[par] + (w ? nt : 0u), (uint32_t)by[w].size(), none, blocks[w],
                                 lists[w] ? need[w] : crew_need[w], st_of[w]));
            if (sample) {
                HIPCHK(hipEventRecord(b->t_end[2 + w], st_of[w]));
                b->pred[2 + w] = pred[2 + w] = cycles[w];
            }
            if (w && beside) HIPCHK(hipEventRecord(b->done3, st_of[w]));
        }
        if (beside) HIPCHK(hipStreamWaitEvent(st, b->done3, 0));
        HIPCHK(launch_parts_of(parts, st));
        const Slot none2{};
        if (ne) HIPCHK(launch_events(b->dev_ev2[par], none2, ne, st));
        return MC_OK;
    };
    if (!several.empty()) {
        HIPCHK(hipEventRecord(b->go, b->stream));
        HIPCHK(hipStreamWaitEvent(b->stream2, b->go, 0));
        if (const int rc = spread_round(0)) return rc;
    }

    if (n[0] + n[1] + n[2]) {
        HIPCHK(hipMemcpyAsync(b->dev_slots[par], hs, 3 * sizeof(Slot) * S, hipMemcpyHostToDevice,
                              b->stream));
        HIPCHK(hipEventRecord(b->copied[par], b->stream));
        b->pending[par] = true;
        Slot none{};
        // with a third stream the HBM class's launch runs beside the LDS
        // class's (each on its own compute units) instead of after it; the
        // events below follow both
        const bool side = n[0] && n[1] && b->stream3;
        if (side) {
            HIPCHK(hipEventRecord(b->go3, b->stream));
            HIPCHK(hipStreamWaitEvent(b->stream3, b->go3, 0));
        }
        for (int cls = 0; cls < 2; ++cls)
            if (n[cls]) {
                hipStream_t st = cls == 1 && side ? b->stream3 : b->stream;
                HIPCHK(hipEventRecord(b->t_beg[cls], st));
                HIPCHK(launch_sweeps(fp64, cls == 0, b->dev_slots[par] + cls * S, none,
                                     cls == 0 ? std::min(n[0], lds_blocks) : n[cls], lds[cls], st, true));
                HIPCHK(hipEventRecord(b->t_end[cls], st));
                b->pred[cls] = crowded ? 0.0 : pred[cls];
            }
        if (side) {
            HIPCHK(hipEventRecord(b->done3, b->stream3));
            HIPCHK(hipStreamWaitEvent(b->stream, b->done3, 0));
        }
        HIPCHK(launch_parts_of(parts1, b->stream));
        if (n[2]) HIPCHK(launch_events(b->dev_slots[par] + 2 * S, none, n[2], b->stream));
    }
    // later work on the batch stream (the next run, poll, reads) follows the
    // multi-workgroup launch
    if (!several.empty()) {
        // all remaining sweeps: the slices between these systems' event sweeps
        // one after another, beside the others' launch
        for (uint32_t r = 1; r < kRounds && !max_moves_per_slot && b->stream2 != b->stream; ++r)
            if (const int rc = spread_round(r)) return rc;
        HIPCHK(hipEventRecord(b->done, b->stream2));
        HIPCHK(hipStreamWaitEvent(b->stream, b->done, 0));
    }
    if (n_launched) *n_launched = (n[0] ? 1u : 0u) + (n[1] ? 1u : 0u) + (team_runs ? 1u : 0u) + (wave_runs ? 1u : 0u);
    return MC_OK;
}

int mc_batch_poll(mc_batch* b, uint32_t* slots, mc_system** systems, size_t cap, size_t* n)
{
    if (!b) return fail(MC_EINVAL, "null batch");
    HIPCHK(hipStreamSynchronize(b->stream));
    size_t k = 0;
    for (uint32_t i = 0; i < b->max_slots && k < cap; ++i) {
        mc_system* s = b->sys[i];
        if (!s || b->remaining[i] != 0) continue;
        if (slots) slots[k] = i;
        if (systems) systems[k] = s;
        s->batch = nullptr;
        b->sys[i] = nullptr;
        ++k;
    }
    if (n) *n = k;
    return MC_OK;
}

int mc_batch_cancel(mc_batch* b, uint32_t slot)
{
    if (!b || slot >= b->max_slots || !b->sys[slot]) return fail(MC_EINVAL, "no such slot");
    HIPCHK(hipStreamSynchronize(b->stream));
    b->sys[slot]->batch = nullptr;
    b->sys[slot] = nullptr;
    b->remaining[slot] = 0;
    return MC_OK;
}

void mc_batch_destroy(mc_batch* b)
{
    if (!b) return;
    (void)hipStreamSynchronize(b->stream);
    for (auto* s : b->sys)
        if (s) s->batch = nullptr;
    if (b->stream2) (void)hipStreamSynchronize(b->stream2);
    if (b->stream3) (void)hipStreamSynchronize(b->stream3);
    for (int i = 0; i < 2; ++i) {
        if (b->host_slots[i]) (void)hipHostFree(b->host_slots[i]);
        if (b->copied[i]) (void)hipEventDestroy(b->copied[i]);
        if (b->host_spread[i]) (void)hipHostFree(b->host_spread[i]);
        if (b->host_ev2[i]) (void)hipHostFree(b->host_ev2[i]);
        if (b->copied2[i]) (void)hipEventDestroy(b->copied2[i]);
    }
    for (int c = 0; c < 4; ++c) {
        if (b->t_beg[c]) (void)hipEventDestroy(b->t_beg[c]);
        if (b->t_end[c]) (void)hipEventDestroy(b->t_end[c]);
    }
    if (b->go) (void)hipEventDestroy(b->go);
    if (b->done) (void)hipEventDestroy(b->done);
    if (b->go3) (void)hipEventDestroy(b->go3);
    if (b->done3) (void)hipEventDestroy(b->done3);
    delete b;
}

}  // extern "C"
