// engine.h -- device-side data layout of the flip Monte Carlo engine.
//
// A system either has one workgroup of 512 threads (8 wave64s) -- when its state
// fits the workgroup's LDS ("resident") centres of mass, site offsets and cell
// lists stay there for the whole launch, else in HBM, where the same code reads
// them through global pointers -- or shares several workgroups, each with the
// neighbourhood of the cell it works on in LDS and the state in HBM.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace flipmc {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxSeg = 64;        // stencil row segments per cell (k <= 3: <= 50)
constexpr int kGofrBins = 256;
constexpr int kGofrQueue = 128;  // per-wave queue of molecule pairs of a g(r) frame
constexpr int kC2Max = 32;
constexpr int kMaxMolecules = 65535;  // indices are stored as u16 in cell lists
// Molecules near a cell that an engine lists: a system has as many places as
// its cells need (near_cap, set by the host), the same in every engine, so that
// all take the same cells for too full.
constexpr uint32_t kNearMin = 192, kNearMax = 320;
constexpr int kNearSlots = kNearMin / 64;  // list entries per lane in registers
// The single-workgroup event kernel copies centres, quaternions and types of
// systems up to this size into LDS for its O(M^2) loops (larger systems use
// the multi-workgroup event kernel).
constexpr uint32_t kEventStage = 2047;
constexpr size_t kEventStageBytes = size_t(kEventStage) * (7 * sizeof(double) + sizeof(uint32_t));

// The units of the event work over all pairs of M molecules (a wave's each):
// blocks of 64 molecules, each against `splits` ranges of the other half, of 32
// molecules or more.  That allows (M / 64)^2 units: 16 of 256 molecules, 225 of
// 1000; from 2900 on there are about 2048, two waves for each of the 1024 SIMDs.
struct EventUnits {
    uint32_t blocks, splits;
    __host__ __device__ uint32_t count() const { return blocks * splits; }
};
__host__ __device__ inline EventUnits event_units(uint32_t M)
{
    EventUnits u;
    u.blocks = (M + 63u) / 64u;
    const uint32_t most = M / 64u ? M / 64u : 1u, want = 2048u / u.blocks ? 2048u / u.blocks : 1u;
    u.splits = want < most ? want : most;
    return u;
}
// Planes of cells that a re-sum from the cell lists may take as units.
constexpr uint32_t kMaxPlanes = 5;
__host__ __device__ inline uint32_t max_units(uint32_t M)
{
    const uint32_t a = event_units(M).count(), b = (M + 63u) / 64u * kMaxPlanes;
    return a > b ? a : b;
}

// Work of the event kernel (Slot::flags).
enum : uint32_t {
    kFlagResumSet = 1u,       // re-sum E and take it as the accumulated energy
    kFlagResumReport = 2u,    // re-sum E and store it as e_resum / drift
    kFlagObsReset = 4u,       // take the current state as the C_2 reference / time origin
    kFlagResumPeriodic = 8u,  // scheduled re-sum: also record the drift sample
    kFlagGofr = 16u,          // accumulate one g(r) frame
    kFlagC2 = 32u,            // record one C_2 sample
    kFlagParts = 64u,         // the re-sum and the g(r) frame were done by the
                              // multi-workgroup event kernel: sum its unit
                              // energies (Slot::pad of them), count the frame
    kFlagInline = 128u,       // (a sweep slot) the scheduled re-sums and C_2
                              // samples of its sweeps are taken by the sweep
                              // kernel itself, as the event kernel takes them
};

// Device accumulators of one system.
struct Stats {
    uint64_t sweep;          // sweeps done (keys the random numbers)
    uint64_t obs_origin;     // sweep at the last observable reset
    double e_acc;            // E_0 + sum of accepted dE
    double e_resum;          // last FP64 re-sum
    double drift;            // e_acc - e_resum at that re-sum
    double max_abs_drift;    // over re-sums after the first window
    uint64_t resum_sweep;
    uint64_t n_resum;
    uint64_t attempts[3];
    uint64_t accepts[3];
    uint64_t exits;
    uint64_t pair_terms;
    uint64_t pair_tests;
    uint64_t near_overflows;  // cells whose near list overflowed (every stencil molecule evaluated)
    double e_sum;
    double e_sumsq;
    uint32_t n_e;
    uint32_t n_drift;
    uint32_t n_gofr;
    uint32_t n_c2;
    uint32_t fault;          // nonzero: a workgroup barrier of the multi-workgroup engine timed out
    uint32_t pad;
};

// Everything a workgroup needs about its system; lives in the system's device
// buffer and is written by the host.
struct SysDev {
    uint32_t M, k, nc, ncell;
    uint32_t precision, resident, seed_lo, seed_hi;
    double L, w, T, p_flip, p_ft, dmax, rot_max, reach2, radius, rc2_factor;
    double body[9];      // body-frame site offsets, row s = site s
    double sigma[3];     // diameters of types A, B, C
    uint32_t resum_interval, obs_interval, gofr_interval, obs_start;
    uint32_t max_samples, gofr_nbins, lds_bytes, barrier_polls;
    uint32_t near_cap, pad1;
    double gofr_dr, gofr_rmax;
    double fs_q, fs_q_cm;  // wavenumbers of F_s (sites) and F_s^cm (centres)
    // state
    double* com;         // SoA [3][M]
    double* quat;        // SoA [4][M], (w, x, y, z)
    uint32_t* types;     // [M]: byte s = type of site s
    double* u0;          // SoA [3][M] C_2 reference orientation
    uint8_t* kref;       // [M] site index followed by C_2
    Stats* stats;
    double* e_samples;
    double* drift_samples;
    uint64_t* gofr_all;
    uint64_t* gofr_inter;
    double* c2;
    uint64_t* c2_sweep;
    int32_t* img;        // SoA [3][M] periodic images crossed by accepted translations
    double* r0;          // SoA [3][M] unwrapped centres at the observable origin
    double* o0;          // SoA [9][M] site offsets at the observable origin
    double* fs;          // [kC2Max] F_s(q, t) at the C_2 sample sweeps
    double* fs_cm;       // [kC2Max] F_s^cm(q, t) at the same sweeps
    double* mom;         // [4][kC2Max] per-particle moments at the same sweeps
    // HBM copies of the work arrays of non-resident systems
    void* g_site;        // Real4 [3M]: offset xyz + sigma of the site's type, or molecule records [M]
    uint32_t* g_cell;    // [ncell + 1] cell starts
    uint16_t* g_cellid;  // [M]
    uint16_t* g_list;    // [M] molecules sorted by cell, ascending inside a cell
    void* props;         // [M] proposals of the current sweep (48 bytes each)
    uint32_t* g_cnt;     // [2 * ncell] cell counts and fill cursors (multi-workgroup engine)
    double* g_part;      // [max_units(M)] unit energies of a re-sum
    double* g_ecell;     // [ncell] accepted dE of each cell in the current sweep (HBM state)
    uint32_t* g_bar;     // [kBarWords] barrier counter and crew of the system's workgroups (multi-workgroup engine)
    // decision log
    void* log;
    uint64_t log_sweep0;
    uint64_t log_sweeps;
};

struct Slot {
    SysDev* sys;
    uint64_t n_sweeps;
    uint32_t flags;
    uint32_t pad;  // of a sweep: 1 + the entry the workgroup takes next, 0 for none; of events: see kFlagParts
};

struct MoveRecord {   // mirrors mc_move_record
    double delta_e;
    double scale;
    double t_log_u;
    uint64_t sweep;
    uint32_t molecule;
    uint8_t move, accepted, exited, axis;
    uint32_t pair_terms;
    uint32_t pad;
};
static_assert(sizeof(MoveRecord) == 48, "record layout");

// Per-wave LDS work areas: the molecules near the current cell, the
// survivors of a trial's prune, the trial in flight.
__host__ __device__ constexpr size_t site_bytes(bool fp64) { return fp64 ? 32 : 16; }
__host__ __device__ constexpr size_t mol_bytes(bool fp64) { return fp64 ? 128 : 64; }  // record of a molecule (multi-workgroup engine)
__host__ __device__ constexpr size_t trial_bytes(bool fp64) { return fp64 ? 272 : 160; }
__host__ __device__ constexpr size_t record_bytes(bool fp64) { return fp64 ? 304 : 208; }  // a trial with its proposal
constexpr size_t kSumBytes = 24;  // an evaluated trial
constexpr size_t kPropBytes = 48;  // a proposal

__host__ __device__ inline size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

// LDS carve-up, shared by the host (launch size) and the kernel (pointers).
struct LdsLayout {
    size_t surv, seglo, segoff, near, misc, trial;
    size_t com, site, cell, cellid, list, ecell, total;
};

__host__ __device__ inline LdsLayout lds_layout(bool fp64, bool resident, uint32_t M,
                                                 uint32_t ncell, uint32_t near_cap)
{
    LdsLayout l{};
    size_t o = 0;
    l.surv = o;   o = align16(o + kWaves * size_t(near_cap) * sizeof(uint16_t));
    l.seglo = o;  o = align16(o + kWaves * kMaxSeg * sizeof(uint16_t));
    l.segoff = o; o = align16(o + kWaves * kMaxSeg * sizeof(uint16_t));
    l.near = o;   o = align16(o + kWaves * size_t(near_cap) * 8);
    l.misc = o;   o = align16(o + 16 * sizeof(double));
    l.trial = o;  o = align16(o + kWaves * trial_bytes(fp64));
    if (resident) {
        l.com = o;    o = align16(o + 3 * size_t(M) * sizeof(double));
        l.site = o;   o = align16(o + 3 * size_t(M) * site_bytes(fp64));
        l.cell = o;   o = align16(o + (size_t(ncell) + 1) * sizeof(uint32_t));
        l.cellid = o; o = align16(o + size_t(M) * sizeof(uint16_t));
        l.list = o;   o = align16(o + size_t(M) * sizeof(uint16_t));
        l.ecell = o;  o = align16(o + size_t(ncell) * sizeof(double));
    }
    l.total = o;
    return l;
}

// Multi-workgroup ("spread") engine: a workgroup takes a cell of the current
// colour, stages the cell's neighbourhood (up to near_cap molecules) in its LDS
// and its waves share the cell's trials; or each of the first `waves` waves of a
// workgroup takes and stages a cell of its own.

// Threads of a workgroup whose waves have a cell each.  A wave of 512 threads has
// 256 registers, of which FP64 trials spill 280 values and FP32 160: 20 sweeps of
// 20 systems of 8000 molecules take 23.3 ms in FP64 so, 12.3 with half the waves
// and twice the registers.  FP32 gains more by the second wave of a SIMD (64
// workgroups, 8000 molecules), but not with the lists in the buffer (50000
// molecules 365 us a sweep, 312 with 256 threads).
__host__ __device__ constexpr int cell_threads(bool fp64, bool lists) { return fp64 || !lists ? kThreads / 2 : kThreads; }
constexpr int kBarWords = 272;   // words of SysDev::g_bar

// LDS of one of its workgroups: the lists of the system's cells too where they
// fit (lists), which are put together over the place of the staged cells.
struct SpreadLayout {
    size_t com, site, own, near, surv, seg, trial;  // from the start, or from each wave's
    size_t wave;                                    // bytes of a wave that has a cell
    size_t sums, cnt, misc, cell, list, total;
};

__host__ __device__ inline SpreadLayout spread_layout(bool fp64, bool lists, uint32_t M, uint32_t ncell,
                                                      uint32_t near_cap, uint32_t waves)
{
    SpreadLayout l{};
    const size_t N = near_cap;
    size_t o = 0;
    l.com = o;   o = align16(o + 3 * N * sizeof(double));     // staged centres
    l.site = o;  o = align16(o + 3 * N * site_bytes(fp64));   // staged sites
    l.own = o;   o = align16(o + N * sizeof(uint16_t));       // slot of each cell molecule
    l.near = o;  o = align16(o + N * 8);                      // near list
    l.surv = o;  o = align16(o + (waves ? 1 : kWaves) * N * sizeof(uint16_t));  // survivors, per wave
    l.seg = o;   o = align16(o + 2 * size_t(kMaxSeg) * sizeof(uint16_t));       // stencil segments
    l.trial = o; o = align16(o + (waves ? 1 : 64) * record_bytes(fp64));  // the trial, or the next of the cell
    l.wave = o;
    if (waves) o = waves * l.wave;
    l.sums = o;  o = align16(o + 2 * kWaves * kSumBytes);  // evaluated trials, by turns
    l.cnt = o;   o = align16(o + 2 * kWaves * sizeof(uint32_t));
    if (lists && o < size_t(M) * sizeof(uint16_t)) o = align16(size_t(M) * sizeof(uint16_t));
    // (the proposals of 512 molecules leave from there too)
    if (o < kThreads * kPropBytes) o = kThreads * kPropBytes;
    l.misc = o;  o = align16(o + 16 * sizeof(double));
    if (lists) {
        l.cell = o; o = align16(o + (size_t(ncell) + 1) * sizeof(uint32_t));
        l.list = o; o = align16(o + size_t(M) * sizeof(uint16_t));
    }
    l.total = o;
    return l;
}

// Kernel launchers (kernels.hip).  inline_events: the sweep kernel takes the
// scheduled re-sums and C_2 samples of slots flagged kFlagInline.
hipError_t launch_sweeps(bool fp64, bool resident, const Slot* dev_slots, const Slot& one,
                         uint32_t n_blocks, size_t lds_bytes, hipStream_t stream,
                         bool inline_events = false);
hipError_t launch_events(const Slot* dev_slots, const Slot& one, uint32_t n_blocks,
                         hipStream_t stream);
hipError_t launch_init_lattice(SysDev* dev_sys, uint32_t M, hipStream_t stream);
// One system of a multi-workgroup launch: its workgroups and sweeps.
struct SpreadSlot {
    SysDev* sys;
    uint64_t n_sweeps;
    uint32_t first_block, n_blocks;
    uint32_t waves, pad;  // waves of a workgroup with a cell each, 0: a cell per workgroup
};

// Launch of the multi-workgroup engine over n_blocks workgroups: the systems of
// dev_slots[0 .. n_slots) (device array), or `one` when dev_slots is null, with
// a cell per workgroup or a cell per wave (SpreadSlot::waves) and the cell lists
// in LDS or in the systems' buffers (crew), and the LDS that the largest needs (spread_layout).  The workgroups of each system synchronise
// among themselves only (each system's g_bar must be zero at launch; one
// workgroup alone does not use it).
enum SpreadMode { kSpreadTeam, kSpreadWaves, kSpreadCrew, kSpreadCrewWaves };
hipError_t launch_spread(bool fp64, SpreadMode mode, const SpreadSlot* dev_slots, uint32_t n_slots,
                         const SpreadSlot& one, uint32_t n_blocks, size_t lds, hipStream_t stream);
// Zero the barrier words of the systems of dev_slots[0 .. n_slots).
hipError_t launch_zero_barriers(const SpreadSlot* dev_slots, uint32_t n_slots, hipStream_t stream);
// Workgroups of the spread kernel that the current device holds at once.
hipError_t spread_max_blocks(uint32_t* n_blocks);
// The systems of one launch of the event work over many workgroups, passed by
// value (no table in memory): system i owns workgroups [first, first + count),
// whose waves take its units in turn.
struct PartSlot {
    SysDev* sys;
    uint32_t flags, first, count;
    uint32_t span;  // re-sum from the cell lists, so many cells each way (0: all pairs)
};
constexpr uint32_t kPartSlots = 128;
struct PartList {
    PartSlot s[kPartSlots];
    uint32_t n;
};
// The part over all pairs of the events of list.s[0 .. n) (re-sum unit energies
// into g_part, g(r) frame into the histograms), n_blocks = the sum of their
// counts; follow with launch_events(flags | kFlagParts, pad = units).
hipError_t launch_event_parts(const PartList& list, uint32_t n_blocks, hipStream_t stream);

// Record msg as the calling thread's last error (mc_last_error) and return code.
int api_error(int code, const char* msg);

}  // namespace flipmc
