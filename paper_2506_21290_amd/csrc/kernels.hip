// kernels.hip -- gfx950 kernels of the flip Monte Carlo engine.
//
// Method (Simon, Barrat & Berthier, Sec. II): Metropolis sweeps over rigid
// triangular A/B/C molecules with the site-site WCA potential (Eq. 1), mixing
// translations, rotations and the intramolecular flip of Sec. II.B.
//
// A sweep is a checkerboard over a randomly shifted cubic cell grid: the k^3
// colours run one after another, and the molecules of a cell are tried in
// ascending index.  Cells of one colour are at least (k-1) cells apart, farther
// than any two molecules can interact, so they never race.  Proposals of all
// molecules of a sweep are drawn in parallel before its first colour.  Inside a
// trial the 64 lanes of a wave share the energy difference: the molecules near
// the cell (listed once per cell) are pruned against the trial molecule's
// centre, every site of the survivors takes a lane and is evaluated against the
// moved sites before and after the move, and a DPP reduction in FP64 gives dE in
// a fixed order.
//
// Two engines run that, with the same near lists, the same sums and so the same
// bits:
//   k_sweeps: one workgroup of 8 wave64s owns one system for the whole launch
//     (state in LDS where it fits), each wave runs cells of the colour from
//     trial to trial.  A batch of as many systems as compute units.
//   k_spread: a workgroup per cell of a colour, its 8 waves evaluating the next
//     8 trials of the cell at once; one system, or few, on the whole device.
// What bounds both is the chain of dependent trials in a cell; a wave issues an
// instruction about every eighth cycle, a trial has some 550, two waves fill a
// SIMD.  FP32: 1000 molecules (T = 0.75) 302 us a sweep with k_sweeps, 134 - 140
// with k_spread on 8 compute units; 8000 (T = 1.1) 2650 on one, 203 with a cell per
// wave on 32, 123 - 127 on 125; 27000 (T = 2) 225 with a cell per wave on 256.
//
// The random numbers are Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11)
// keyed by the seed and counted by (molecule, sweep low, sweep high, tag), so a
// run is reproducible regardless of how systems are batched.
#include <type_traits>

#include "engine.h"
#include "wave.h"

namespace flipmc {
namespace {

// Sum over the workgroup in a fixed order (identical bits in every thread).
__device__ double block_sum(double v, double* red)
{
    const int lane = threadIdx.x & 63, wave = wave_index();
    v = wave_sum(v);
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < kWaves; ++i) t += red[i];
    __syncthreads();
    return t;
}

__device__ __forceinline__ void block_excl_scan(uint32_t* a, uint32_t n, uint32_t* scratch)
{
    block_excl_scan_t<kThreads>(a, n, scratch);
}

// --------------------------------------------------------------- geometry --

__device__ __forceinline__ double wrap(double x, double L) { return x - L * floor(x / L); }

__device__ __forceinline__ double min_image(double d, double L, double invL)
{
    return d - L * rint(d * invL);
}

__device__ __forceinline__ int cell_axis(double x, double h, double L, double w, int nc)
{
    const double g = wrap(x - h, L);
    int c = (int)floor(g / w);
    c = c < 0 ? 0 : c;
    return c >= nc ? nc - 1 : c;
}

__device__ __forceinline__ void rotation(double qw, double qx, double qy, double qz, double r[9])
{
    r[0] = 1.0 - 2.0 * (qy * qy + qz * qz);
    r[1] = 2.0 * (qx * qy - qw * qz);
    r[2] = 2.0 * (qx * qz + qw * qy);
    r[3] = 2.0 * (qx * qy + qw * qz);
    r[4] = 1.0 - 2.0 * (qx * qx + qz * qz);
    r[5] = 2.0 * (qy * qz - qw * qx);
    r[6] = 2.0 * (qx * qz - qw * qy);
    r[7] = 2.0 * (qy * qz + qw * qx);
    r[8] = 1.0 - 2.0 * (qx * qx + qy * qy);
}

// Shifted WCA of Eq. (1) written as (2 (s/r)^6 - 1)^2, given s^2 and r^2.
__device__ __forceinline__ float pair_u(float s2, float r2)
{
    const float x = s2 * __builtin_amdgcn_rcpf(r2);
    const float x3 = x * x * x;
    const float t = fmaf(2.0f, x3, -1.0f);
    return t * t;
}
__device__ __forceinline__ double pair_u(double s2, double r2)
{
    // 1 / r2: the hardware estimate refined by two Newton steps (within an
    // ulp or two of the quotient; r2 is a normal number here)
    double y = __builtin_amdgcn_rcp(r2);
    y = fma(fma(-r2, y, 1.0), y, y);
    y = fma(fma(-r2, y, 1.0), y, y);
    const double x = s2 * y;
    const double x3 = x * x * x;
    const double t = fma(2.0, x3, -1.0);
    return t * t;
}

// Body-frame coordinate a of site s of the equilateral triangle.
template <class Cx>
__device__ __forceinline__ double body_at(const Cx& C, uint32_t s, int a)
{
    if (a == 0) return s == 0 ? C.bR : -0.5 * C.bR;
    if (a == 1) return s == 0 ? 0.0 : (s == 1 ? C.bH : -C.bH);
    return 0.0;
}

// Diameter of type t, from the 3-entry table in LDS (filled at kernel entry);
// a table lookup keeps the per-system constants out of dynamically indexed
// memory.
template <class Cx>
__device__ __forceinline__ double sigma_of(const Cx& C, uint32_t t)
{
    return C.misc[1 + t];
}

// ------------------------------------------------------------- per system --

// Everything a workgroup needs, copied from the system descriptor at kernel
// entry (before any store, so the copies are scalar loads kept in SGPRs) plus
// the LDS or HBM addresses of the work arrays.
// Where the work arrays are: in device memory, in LDS, or either (the event
// kernels, which stage what fits).
// The multi-workgroup engine has its positions in records of device memory and
// the cell lists in LDS (kMemTeam) or in device memory too (kMemCrew).
enum : int { kMemHbm = 0, kMemLds = 1, kMemAny = 2, kMemTeam = 3, kMemCrew = 4 };
constexpr bool has_records(int mem) { return mem == kMemTeam || mem == kMemCrew; }

// A molecule as the multi-workgroup engine keeps it during a launch: centre,
// site offsets and types in one aligned piece.  A workgroup fetches some 400 of
// them per cell, each from a place of its own, and pays for whole 128-byte
// lines: with separate arrays of x, y, z and sites that was 243 KB per cell at
// 1000 molecules, 8.6k cycles; this is 27 KB.
template <typename Real>
struct alignas(64) MolRec {
    double c[3];
    Real o[9];       // offset of site s at 3 s
    uint32_t types;  // byte s = type of site s
};
static_assert(sizeof(MolRec<float>) == 64 && sizeof(MolRec<double>) == 128, "molecule record");
template <typename Real>
constexpr uint32_t mol_used()  // bytes of it that hold anything
{
    return 3 * sizeof(double) + 9 * sizeof(Real) + sizeof(uint32_t);
}
// Site t with its diameter.
template <typename Cx, typename Real>
__device__ __forceinline__ R4<Real> mol_site(const Cx& C, const MolRec<Real>& m, int t)
{
    const uint32_t ty = (m.types >> (8 * t)) & 0xFFu;
    return R4<Real>{m.o[3 * t], m.o[3 * t + 1], m.o[3 * t + 2],
                    (Real)(ty == 0u ? C.sig0 : (ty == 1u ? C.sig1 : C.sig2))};
}
static_assert(sizeof(MolRec<float>) == mol_bytes(false) && sizeof(MolRec<double>) == mol_bytes(true),
              "molecule record");

template <typename Real, int kMem>
struct Ctx {
    template <typename T>
    using Work = std::conditional_t<kMem == kMemAny, T, std::conditional_t<kMem == kMemLds, Lds<T>, Global<T>>>;
    template <typename T>
    using Index = std::conditional_t<kMem == kMemTeam, Lds<T>, Work<T>>;
    template <typename T>
    using Dev = std::conditional_t<kMem == kMemAny, T, Global<T>>;
    uint32_t M, k, nc, ncell, seed_lo, seed_hi;
    uint32_t resum_interval, obs_interval, gofr_interval, obs_start, max_samples, gofr_nbins;
    double L, invL, w, T, p_flip, p_ft, dmax, rot_max, reach2, radius, rc2_factor;
    double bR, bH;            // body frame: site 0 at (bR, 0, 0), sites 1, 2 at (-bR/2, +-bH, 0)
    double sig0, sig1, sig2;  // diameters of types A, B, C
    double gofr_dr, gofr_rmax;
    double fs_q, fs_q_cm;
    Dev<double>* gcom;
    Dev<double>* quat;
    Dev<uint32_t>* types;
    double* u0;
    uint8_t* kref;
    Dev<int32_t>* img;
    double* r0;
    double* o0;
    double* fs;
    double* fs_cm;
    double* mom;
    Stats* stats;
    double* e_samples;
    double* drift_samples;
    uint64_t* gofr_all;
    uint64_t* gofr_inter;
    double* c2;
    uint64_t* c2_sweep;
    MoveRecord* log;
    uint64_t log_sweep0, log_sweeps;
    double* gpart;
    // work arrays (LDS when resident)
    Work<double>* com;
    Work<R4<Real>>* site;
    Global<MolRec<Real>>* rec;
    Index<uint32_t>* cellb;
    Work<uint16_t>* cellid;
    Index<uint16_t>* list;
    double* red;
    Work<double>* ecell;  // accepted dE of each cell in the current sweep
    const double* off;  // FP64 site offsets [9][M] computed up front (event kernel), or null
    uint32_t* bins;
    double* misc;
};

// Data that several workgroups of the multi-workgroup engine read or write
// inside a launch (a molecule changes hands from sweep to sweep) goes past the caches of the XCDs, which do not follow each other:
// loads and stores at agent scope, and 16-byte loads with the same cache bits
// (sc1).  A barrier then only waits for a workgroup's own stores; writing back
// and invalidating the L2 for it took 5k cycles more per barrier with 125
// workgroups, 10k with 256.
template <typename T>
__device__ __forceinline__ T agent_load(const Global<T>* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(Global<T>* p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
using Words = uint32_t __attribute__((ext_vector_type(4)));
constexpr int kAgentScope = 16;  // sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t agent_buffer(const void* p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void agent_put_words(__amdgpu_buffer_rsrc_t b, uint32_t byte, Words v)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, b, (int)byte, 0, kAgentScope);
}
__device__ __forceinline__ Words agent_words(__amdgpu_buffer_rsrc_t b, uint32_t byte)
{
    return (Words)__builtin_amdgcn_raw_buffer_load_b128(b, (int)byte, 0, kAgentScope);
}

// A record of whole 16-byte words, the first kBytes of it.
template <typename T, uint32_t kBytes = sizeof(T)>
__device__ __forceinline__ T agent_record(__amdgpu_buffer_rsrc_t b, uint32_t index)
{
    union {
        Words w[(sizeof(T) + 15) / 16];
        T v;
    } u;
#pragma unroll
    for (uint32_t i = 0; i < (kBytes + 15u) / 16u; ++i) u.w[i] = agent_words(b, index * (uint32_t)sizeof(T) + 16u * i);
    return u.v;
}

// Proposal of one molecule for the current sweep.  All proposals of a sweep
// are drawn at its start by the whole workgroup (they depend only on the
// molecule's own state, which no earlier trial of the sweep can change) and
// kept in HBM; a wave loads those of a cell when it reaches the cell.
struct alignas(16) PropRec {
    uint32_t kind;  // move | exited << 4 | axis << 8
    uint32_t pad;
    double thr;     // T ln u_acc
    double a0, a1, a2, a3;  // translation: displacement a0..a2; rotation: new quaternion
};
static_assert(sizeof(PropRec) == 48, "proposal record");

__device__ __forceinline__ PropRec load_prop(const Global<PropRec>* p)
{
    return PropRec{p->kind, 0u, p->thr, p->a0, p->a1, p->a2, p->a3};
}
__device__ __forceinline__ void store_prop(Global<PropRec>* p, const PropRec& v)
{
    p->kind = v.kind; p->thr = v.thr;
    p->a0 = v.a0; p->a1 = v.a1; p->a2 = v.a2; p->a3 = v.a3;
}

// Site records through pointers of any address space.
template <typename P>
__device__ __forceinline__ auto load_site(P p)
{
    return R4<std::decay_t<decltype(p->x + p->x)>>{p->x, p->y, p->z, p->w};
}
template <typename P, typename Real>
__device__ __forceinline__ void store_site(P p, const R4<Real>& v)
{
    p->x = v.x; p->y = v.y; p->z = v.z; p->w = v.w;
}

template <typename Real, int kMem>
__device__ PropRec propose(const Ctx<Real, kMem>& C, uint32_t m, uint64_t sweep, double hx,
                           double hy, double hz, int cx, int cy, int cz)
{
    PropRec p;
    const uint32_t slo = (uint32_t)sweep, shi = (uint32_t)(sweep >> 32);
    const U4 b0 = philox10(m, slo, shi, 0u, C.seed_lo, C.seed_hi);
    const U4 b1 = philox10(m, slo, shi, 1u, C.seed_lo, C.seed_hi);
    const double uacc = unit_53(b0.x, b0.y), ut = unit_open(b0.z);
    const double p0 = unit_open(b1.x), p1 = unit_open(b1.y), p2 = unit_open(b1.z);
    p.thr = C.T * log(uacc);
    const uint32_t move = ut < C.p_flip ? 2u : (ut < C.p_ft ? 0u : 1u);
    uint32_t exited = 0, axis = 255;
    const uint32_t M = C.M;
    p.pad = 0;
    p.a0 = p.a1 = p.a2 = p.a3 = 0.0;
    if (move == 0u) {
        double c0, c1, c2;
        if constexpr (has_records(kMem)) {
            c0 = agent_load(&C.rec[m].c[0]); c1 = agent_load(&C.rec[m].c[1]); c2 = agent_load(&C.rec[m].c[2]);
        } else {
            c0 = C.com[m]; c1 = C.com[M + m]; c2 = C.com[2 * M + m];
        }
        p.a0 = C.dmax * (2.0 * p0 - 1.0);
        p.a1 = C.dmax * (2.0 * p1 - 1.0);
        p.a2 = C.dmax * (2.0 * p2 - 1.0);
        const int nc = (int)C.nc;
        exited = (cell_axis(wrap(c0 + p.a0, C.L), hx, C.L, C.w, nc) != cx) ||
                 (cell_axis(wrap(c1 + p.a1, C.L), hy, C.L, C.w, nc) != cy) ||
                 (cell_axis(wrap(c2 + p.a2, C.L), hz, C.L, C.w, nc) != cz);
    } else if (move == 1u) {
        const double z = 2.0 * p0 - 1.0;
        const double phi = kTwoPi * p1;
        const double st = sqrt(1.0 - z * z);
        const double nx = st * cos(phi), ny = st * sin(phi), nz = z;
        const double th = C.rot_max * (2.0 * p2 - 1.0);
        const double ch = cos(0.5 * th), sh = sin(0.5 * th);
        const double dw = ch, dx = nx * sh, dy = ny * sh, dz = nz * sh;
        double qw, qx, qy, qz;
        if constexpr (has_records(kMem)) {
            qw = agent_load(&C.quat[m]); qx = agent_load(&C.quat[M + m]);
            qy = agent_load(&C.quat[2 * M + m]); qz = agent_load(&C.quat[3 * M + m]);
        } else {
            qw = C.quat[m]; qx = C.quat[M + m]; qy = C.quat[2 * M + m]; qz = C.quat[3 * M + m];
        }
        const double rw = dw * qw - dx * qx - dy * qy - dz * qz;
        const double rx = dw * qx + dx * qw + dy * qz - dz * qy;
        const double ry = dw * qy - dx * qz + dy * qw + dz * qx;
        const double rz = dw * qz + dx * qy - dy * qx + dz * qw;
        const double nrm = sqrt(rw * rw + rx * rx + ry * ry + rz * rz);
        p.a0 = rw / nrm; p.a1 = rx / nrm; p.a2 = ry / nrm; p.a3 = rz / nrm;
    } else {
        int a = (int)(3.0 * p0);
        axis = (uint32_t)(a > 2 ? 2 : a);
    }
    p.kind = move | (exited << 4) | (axis << 8);
    return p;
}

// Proposals of every molecule for this sweep (after the cell build).
template <typename Real, int kMem>
__device__ void propose_all(const Ctx<Real, kMem>& C, Global<PropRec>* props, uint64_t sweep, double hx,
                            double hy, double hz)
{
    const int nc = (int)C.nc;
    for (uint32_t m = threadIdx.x; m < C.M; m += kThreads) {
        const int cid = C.cellid[m];
        const int cx = cid % nc, cy = (cid / nc) % nc, cz = cid / (nc * nc);
        store_prop(props + m, propose(C, m, sweep, hx, hy, hz, cx, cy, cz));
    }
}

template <typename Real, int kMem>
__device__ __forceinline__ void store_sites_from_quat(const Ctx<Real, kMem>& C, uint32_t m)
{
    const uint32_t M = C.M;
    double r[9];
    rotation(C.quat[m], C.quat[M + m], C.quat[2 * M + m], C.quat[3 * M + m], r);
    const uint32_t ty = C.types[m];
    if constexpr (has_records(kMem)) {
#pragma unroll
        for (int a = 0; a < 3; ++a) agent_store(&C.rec[m].c[a], (double)C.com[a * M + m]);
        agent_store(&C.rec[m].types, ty);
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        R4<Real> v;
        v.x = (Real)(r[0] * body_at(C, s, 0) + r[1] * body_at(C, s, 1) + r[2] * body_at(C, s, 2));
        v.y = (Real)(r[3] * body_at(C, s, 0) + r[4] * body_at(C, s, 1) + r[5] * body_at(C, s, 2));
        v.z = (Real)(r[6] * body_at(C, s, 0) + r[7] * body_at(C, s, 1) + r[8] * body_at(C, s, 2));
        if constexpr (has_records(kMem)) {
            agent_store(&C.rec[m].o[3 * s], v.x);
            agent_store(&C.rec[m].o[3 * s + 1], v.y);
            agent_store(&C.rec[m].o[3 * s + 2], v.z);
        } else {
            v.w = (Real)sigma_of(C, (ty >> (8 * s)) & 0xFFu);
            store_site(C.site + 3 * m + s, v);
        }
    }
}

// FP64 offsets of molecule m straight from its quaternion, plus site sigmas.
template <typename Real, int kMem>
__device__ __forceinline__ void offsets_f64(const Ctx<Real, kMem>& C, uint32_t m, double o[9],
                                            double sg[3])
{
    const uint32_t M = C.M;
    if (C.off) {
#pragma unroll
        for (int i = 0; i < 9; ++i) o[i] = C.off[i * M + m];
    } else {
        double r[9];
        rotation(C.quat[m], C.quat[M + m], C.quat[2 * M + m], C.quat[3 * M + m], r);
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int a = 0; a < 3; ++a)
                o[3 * s + a] = r[3 * a] * body_at(C, s, 0) + r[3 * a + 1] * body_at(C, s, 1) +
                               r[3 * a + 2] * body_at(C, s, 2);
    }
    const uint32_t ty = C.types[m];
#pragma unroll
    for (int s = 0; s < 3; ++s) sg[s] = sigma_of(C, (ty >> (8 * s)) & 0xFFu);
}

// The event work over all pairs of molecules is cut into units that a wave
// takes: 64 molecules, one a lane, against a range of the others (EventUnits).
// Whoever takes a unit adds it up in the same order, so one workgroup and many
// give the same bits.
//
// Almost all pairs end at the distance of their centres, so the few that go on
// are queued and evaluated 64 at a time with every lane busy: evaluated where
// they were found, one of 64 lanes having one kept the others waiting in most
// iterations.  A total energy of 8000 molecules took 858 us on 16 workgroups,
// a thread per molecule.

// Pairs of a wave that passed the distance test, its `each` called with 64 of
// them (or the rest, at the end).
template <typename Each>
struct PairQueue {
    uint32_t* q;  // kGofrQueue words of LDS
    Each each;
    uint32_t n;
    __device__ __forceinline__ void drain(uint32_t upto)
    {
        while (n >= upto && n > 0u) {
            const uint32_t take = min(n, 64u), base = n - take, lane = (uint32_t)__lane_id();
            if (lane < take) each(q[base + lane] & 0xFFFFu, q[base + lane] >> 16);
            n = base;
        }
    }
    // keep: whether this lane has the pair (m, j)
    __device__ __forceinline__ void push(bool keep, uint32_t m, uint32_t j)
    {
        const uint64_t bm = __ballot(keep);
        if (bm == 0ull) return;
        if (keep) q[n + rank_below(bm)] = m | (j << 16);
        n += (uint32_t)__popcll(bm);
        wave_lds_sync();
        drain(64u);
        wave_lds_sync();
    }
};

// The pairs of unit u whose centres are nearer than the root of cut2, and some a
// little farther: the distance test is in FP32 (half the time of FP64).  The
// centres are folded into the box before they are rounded (a caller's may lie
// anywhere), which leaves a difference of two within 5 2^-24 L of its value
// along each axis (two centres, the image's shift, the results); with the
// rounding of the squares a distance is off by 6e-7 L at most, and the margin is
// 1e-6 L, or 1e-3 where that is more (boxes up to 1000).  What is added up for a
// pair is in FP64 and nothing past the cut-off.
// window: 3 x (kSpan + 64) words of LDS for the wave, where the centres that the
// 64 molecules meet next are held as floats.
constexpr uint32_t kEventSpan = 128, kInlineSpan = 32;
template <uint32_t kSpan, typename Cx, typename Queue>
__device__ __forceinline__ void unit_pairs(const Cx& C, const EventUnits& U, uint32_t u, double cut2, float* window,
                                           Queue& Q)
{
    const uint32_t M = C.M, half = M / 2;
    const uint32_t blk = u / U.splits, part = u - blk * U.splits;
    const uint32_t m = 64u * blk + (uint32_t)__lane_id();
    const uint32_t d0 = 1u + (uint32_t)((uint64_t)half * part / U.splits),
                   d1 = 1u + (uint32_t)((uint64_t)half * (part + 1u) / U.splits);
    const bool mine = m < M;
    auto folded = [&](double x) { return (float)(x - C.L * floor(x * C.invL)); };
    const float cx = mine ? folded(C.com[m]) : 0.f, cy = mine ? folded(C.com[M + m]) : 0.f,
                cz = mine ? folded(C.com[2 * M + m]) : 0.f;
    const float L = (float)C.L, invL = (float)C.invL;
    const float cut = (float)sqrt(cut2) + fmaxf(1e-3f, 1e-6f * L), lim = cut * cut;
    constexpr uint32_t kWindow = kSpan + 64u;
    const uint32_t lane = (uint32_t)__lane_id();
    for (uint32_t c0 = d0; c0 < d1; c0 += kSpan) {
        wave_lds_sync();
#pragma unroll
        for (uint32_t t = 0; t < (kWindow + 63u) / 64u; ++t) {  // the centres of 64 blk + c0 ...
            uint32_t j = 64u * blk + c0 + 64u * t + lane;
            while (j >= M) j -= M;
            const uint32_t at = 64u * t + lane;
            if (kWindow % 64u != 0u && at >= kWindow) continue;
            window[at] = folded(C.com[j]);
            window[kWindow + at] = folded(C.com[M + j]);
            window[2u * kWindow + at] = folded(C.com[2 * M + j]);
        }
        wave_lds_sync();
        const uint32_t end = min(c0 + kSpan, d1);
        for (uint32_t dj = c0; dj < end; ++dj) {
            const uint32_t at = lane + (dj - c0);
            float dx = window[at] - cx, dy = window[kWindow + at] - cy, dz = window[2u * kWindow + at] - cz;
            dx = fmaf(-L, rintf(dx * invL), dx);
            dy = fmaf(-L, rintf(dy * invL), dy);
            dz = fmaf(-L, rintf(dz * invL), dz);
            // (half way round an even number each pair comes twice)
            const bool keep = mine && !((M & 1u) == 0u && dj == half && m >= half) && dx * dx + dy * dy + dz * dz < lim;
            const uint32_t j = m + dj;
            Q.push(keep, m, j >= M ? j - M : j);
        }
    }
}

// Energy of the nine site pairs of two molecules.
template <typename Cx>
__device__ __forceinline__ double pair_energy(const Cx& C, uint32_t m, uint32_t j)
{
    const uint32_t M = C.M;
    double om[9], sm[3], oj[9], sj[3];
    offsets_f64(C, m, om, sm);
    offsets_f64(C, j, oj, sj);
    const double dx = min_image(C.com[j] - C.com[m], C.L, C.invL);
    const double dy = min_image(C.com[M + j] - C.com[M + m], C.L, C.invL);
    const double dz = min_image(C.com[2 * M + j] - C.com[2 * M + m], C.L, C.invL);
    double e = 0.0;
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const double rx = dx + oj[3 * t] - om[3 * s];
            const double ry = dy + oj[3 * t + 1] - om[3 * s + 1];
            const double rz = dz + oj[3 * t + 2] - om[3 * s + 2];
            const double r2 = rx * rx + ry * ry + rz * rz;
            const double sg = 0.5 * (sm[s] + sj[t]);
            const double s2 = sg * sg;
            if (r2 < C.rc2_factor * s2) e += pair_u(s2, r2);
        }
    return e;
}

// Eq. (1) over all pairs of sites of different molecules in FP64, unit by unit
// into C.gpart: units wave, wave + nwaves, ...  queue: the wave's words of LDS.
template <uint32_t kSpan, typename Real, int kMem>
__device__ __forceinline__ void resum_units(const Ctx<Real, kMem>& C, const EventUnits& U, uint32_t wave,
                                            uint32_t nwaves, uint32_t* queue, float* window)
{
    for (uint32_t u = wave; u < U.count(); u += nwaves) {
        double e = 0.0;
        auto each = [&](uint32_t m, uint32_t j) __attribute__((always_inline)) { e += pair_energy(C, m, j); };
        PairQueue<decltype(each)> Q{queue, each, 0u};
        unit_pairs<kSpan>(C, U, u, C.reach2, window, Q);
        Q.drain(1u);
        e = wave_sum_dpp(e);
        if (__lane_id() == 0) C.gpart[u] = e;
    }
}

// The same from the cell lists of the sweep that ended (positions that moved at
// most one step since they were made, `span` cells each way): unit u takes 64
// molecules against one plane of cells.  Requires 2 span + 1 <= n_c.
template <typename Real, int kMem>
__device__ __forceinline__ void resum_units_cells(const Ctx<Real, kMem>& C, uint32_t wave, uint32_t nwaves, int span,
                                                  uint32_t* queue)
{
    const uint32_t M = C.M, planes = 2u * (uint32_t)span + 1u;
    const int nc = (int)C.nc;
    for (uint32_t u = wave; u < (M + 63u) / 64u * planes; u += nwaves) {
        double e = 0.0;
        auto each = [&](uint32_t m, uint32_t j) __attribute__((always_inline)) { e += pair_energy(C, m, j); };
        PairQueue<decltype(each)> Q{queue, each, 0u};
        const uint32_t blk = u / planes;
        const int oz = (int)(u - blk * planes) - span;
        const uint32_t m = 64u * blk + (uint32_t)__lane_id();
        const bool mine = m < M;
        const double cx = mine ? C.com[m] : 0.0, cy = mine ? C.com[M + m] : 0.0, cz = mine ? C.com[2 * M + m] : 0.0;
        const int cid = mine ? (int)C.cellid[m] : 0;
        const int ix = cid % nc, iy = (cid / nc) % nc, iz = cid / (nc * nc);
        auto wrapped = [&](int v) { return v + (v < 0 ? nc : (v >= nc ? -nc : 0)); };
        const int z = wrapped(iz + oz);
        for (int oy = -span; oy <= span; ++oy)
            for (int ox = -span; ox <= span; ++ox) {
                const uint32_t c = (uint32_t)(wrapped(ix + ox) + nc * (wrapped(iy + oy) + nc * z));
                uint32_t p = mine ? (uint32_t)C.cellb[c] : 0u;
                const uint32_t pe = mine ? (uint32_t)C.cellb[c + 1] : 0u;
                while (__ballot(p < pe) != 0ull) {
                    bool keep = p < pe;
                    uint32_t j = 0;
                    if (keep) {
                        j = C.list[p];
                        const double dx = min_image(C.com[j] - cx, C.L, C.invL);
                        const double dy = min_image(C.com[M + j] - cy, C.L, C.invL);
                        const double dz = min_image(C.com[2 * M + j] - cz, C.L, C.invL);
                        keep = j > m && dx * dx + dy * dy + dz * dz < C.reach2;
                    }
                    Q.push(keep, m, j);
                    ++p;
                }
            }
        Q.drain(1u);
        e = wave_sum_dpp(e);
        if (__lane_id() == 0) C.gpart[u] = e;
    }
}

// Sum of the first n unit energies by the workgroup, in a fixed order.
template <typename Cx>
__device__ double sum_units(const Cx& C, uint32_t n)
{
    double e = 0.0;
    for (uint32_t u = threadIdx.x; u < n; u += kThreads) e += C.gpart[u];
    return block_sum(e, C.red);
}

__device__ __forceinline__ bool is_c2_time(uint64_t t)
{
    if (t == 0) return false;
    while (t % 10 == 0) t /= 10;
    return t == 1 || t == 2 || t == 5;
}

// sin(x) / x, with its Taylor value near 0.
__device__ __forceinline__ double sinc(double x)
{
    return x < 1e-4 ? 1.0 - x * x / 6.0 : sin(x) / x;
}

// The time correlations of one sample (Sec. III.B) and the moments of their
// per-particle contributions (Sec. V.A) that the four-point susceptibilities
// and the Pearson coefficient (Sec. V.B and V.C) are built from:
//   C_2^i    = P_2(u_i(t) . u_i(0)), u following the site that held type B
//              at the observable origin (Eq. 7, l = 2),
//   F_s^cm,i = sin(q d)/(q d) at |q| = C.fs_q_cm, d the displacement of the
//              unwrapped centre (Eq. 6 averaged over all directions of q),
//   F_s^i    = the same over each site index at |q| = C.fs_q (Eq. 5); a
//              site keeps its index through a flip, so a flip moves no site.
// Centres are unwrapped with the image counts of the accepted translations.
// d[0..6] = means of C_2^i, (C_2^i)^2, F_s^cm,i, (F_s^cm,i)^2, C_2^i F_s^cm,i
// over molecules and of F_s^i, (F_s^i)^2 over sites.
constexpr int kDyn = 7;

template <typename Real, int kMem>
__device__ void dyn_values(const Ctx<Real, kMem>& C, double d[kDyn])
{
    const uint32_t M = C.M;
    double a[kDyn];
#pragma unroll
    for (int j = 0; j < kDyn; ++j) a[j] = 0.0;
    for (uint32_t m = threadIdx.x; m < M; m += kThreads) {
        double o[9], sg[3];
        offsets_f64(C, m, o, sg);
        const int k = C.kref[m];
        double dot = 0.0;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const double okx = k == 0 ? o[x] : (k == 1 ? o[3 + x] : o[6 + x]);
            dot += (okx / C.radius) * C.u0[x * M + m];
        }
        const double c2 = 0.5 * (3.0 * dot * dot - 1.0);
        double dc[3];
#pragma unroll
        for (int x = 0; x < 3; ++x)
            dc[x] = (C.com[x * M + m] + C.L * (double)C.img[x * M + m]) - C.r0[x * M + m];
        const double fcm = sinc(C.fs_q_cm * sqrt(dc[0] * dc[0] + dc[1] * dc[1] + dc[2] * dc[2]));
        a[0] += c2; a[1] += c2 * c2; a[2] += fcm; a[3] += fcm * fcm; a[4] += c2 * fcm;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const double ex = dc[0] + (o[3 * t] - C.o0[(3 * t) * M + m]);
            const double ey = dc[1] + (o[3 * t + 1] - C.o0[(3 * t + 1) * M + m]);
            const double ez = dc[2] + (o[3 * t + 2] - C.o0[(3 * t + 2) * M + m]);
            const double f = sinc(C.fs_q * sqrt(ex * ex + ey * ey + ez * ez));
            a[5] += f; a[6] += f * f;
        }
    }
#pragma unroll
    for (int j = 0; j < kDyn; ++j) d[j] = block_sum(a[j], C.red) / ((j < 5 ? 1.0 : 3.0) * (double)M);
}

// One sample of the time correlations at the current sweep.
template <typename Real, int kMem>
__device__ void store_dyn(const Ctx<Real, kMem>& C, Stats* st, uint64_t t)
{
    double d[kDyn];
    dyn_values(C, d);
    if (threadIdx.x == 0 && st->n_c2 < kC2Max) {
        const uint32_t n = st->n_c2;
        C.c2[n] = d[0];
        C.fs_cm[n] = d[2];
        C.fs[n] = d[5];
        C.mom[n] = d[1];
        C.mom[kC2Max + n] = d[3];
        C.mom[2 * kC2Max + n] = d[4];
        C.mom[3 * kC2Max + n] = d[6];
        C.c2_sweep[n] = t;
        st->n_c2 = n + 1;
    }
}

template <typename Real, int kMem>
__device__ void reset_observables(const Ctx<Real, kMem>& C)
{
    const uint32_t M = C.M;
    for (uint32_t m = threadIdx.x; m < M; m += kThreads) {
        // F_s references: unwrapped centre and site offsets
        double o[9], sg[3];
        offsets_f64(C, m, o, sg);
#pragma unroll
        for (int i = 0; i < 9; ++i) C.o0[i * M + m] = o[i];
#pragma unroll
        for (int k = 0; k < 3; ++k) C.r0[k * M + m] = C.com[k * M + m] + C.L * (double)C.img[k * M + m];
        const uint32_t ty = C.types[m];
        int k = 0;
        for (int s = 0; s < 3; ++s)
            if (((ty >> (8 * s)) & 0xFFu) == 1u) k = s;
        C.kref[m] = (uint8_t)k;
        double r[9];
        rotation(C.quat[m], C.quat[M + m], C.quat[2 * M + m], C.quat[3 * M + m], r);
        for (int a = 0; a < 3; ++a)
            C.u0[a * M + m] = (r[3 * a] * body_at(C, k, 0) + r[3 * a + 1] * body_at(C, k, 1) +
                               r[3 * a + 2] * body_at(C, k, 2)) / C.radius;
    }
    for (uint32_t b = threadIdx.x; b < kGofrBins; b += kThreads) {
        C.gofr_all[b] = 0;
        C.gofr_inter[b] = 0;
    }
    if (threadIdx.x == 0) {
        Stats* st = C.stats;
        st->obs_origin = st->sweep;
        st->n_e = st->n_drift = st->n_gofr = st->n_c2 = 0;
        st->e_sum = st->e_sumsq = 0.0;
        st->max_abs_drift = 0.0;
    }
}

// One g(r) frame (Eq. 3 numerator): every ordered pair of distinct sites.
template <typename Real, int kMem>
__device__ void gofr_frame(const Ctx<Real, kMem>& C, const EventUnits& U, uint32_t wave, uint32_t nwaves,
                           bool shared_out, uint32_t* queue, float* window)
{
    const uint32_t M = C.M, nb = C.gofr_nbins;
    uint32_t* bintra = C.bins;  // intramolecular pairs; all = intra + inter at the end
    uint32_t* binter = C.bins + kGofrBins;
    for (uint32_t b = threadIdx.x; b < 2 * kGofrBins; b += kThreads) C.bins[b] = 0;
    __syncthreads();
    const double dr = C.gofr_dr, rmax = C.gofr_rmax;
    const double cut = rmax + 2.0 * C.radius;
    const double cut2 = cut * cut;
    const float inv_dr = (float)(1.0 / dr);
    // bin floor(sqrt(r2) / dr) in FP64; an FP32 estimate decides unless it
    // lies within 2e-4 of a bin edge (its error stays below 1e-4 up to the last bin)
    auto bin = [&](double r2) __attribute__((always_inline)) {
        const float t = sqrtf((float)r2) * inv_dr;
        const float fl = floorf(t);
        int b = (int)fl;
        if (t - fl < 2e-4f || fl + 1.0f - t < 2e-4f) b = (int)floor(sqrt(r2) / dr);
        return b;
    };
    // the nine site pairs of molecules m, j (each with its own nearest image)
    auto site_pairs = [&](uint32_t m, uint32_t j) __attribute__((always_inline)) {
        double om[9], sm[3], oj[9], sj[3];
        offsets_f64(C, m, om, sm);
        offsets_f64(C, j, oj, sj);
        const double dx = min_image(C.com[j] - C.com[m], C.L, C.invL);
        const double dy = min_image(C.com[M + j] - C.com[M + m], C.L, C.invL);
        const double dz = min_image(C.com[2 * M + j] - C.com[2 * M + m], C.L, C.invL);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const double bx = dx + oj[3 * t], by = dy + oj[3 * t + 1], bz = dz + oj[3 * t + 2];
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                // r reaches L / 2
                const double rx = min_image(bx - om[3 * s], C.L, C.invL);
                const double ry = min_image(by - om[3 * s + 1], C.L, C.invL);
                const double rz = min_image(bz - om[3 * s + 2], C.L, C.invL);
                const int b = bin(rx * rx + ry * ry + rz * rz);
                if (b >= 0 && b < (int)nb) atomicAdd(&binter[b], 2u);
            }
        }
    };
    // (the counts do not depend on the order)
    PairQueue<decltype(site_pairs)> Q{queue, site_pairs, 0u};
    for (uint32_t u = wave; u < U.count(); u += nwaves) {
        const uint32_t m = 64u * (u / U.splits) + (uint32_t)__lane_id();
        if (u % U.splits == 0u && m < M) {
            double om[9], sm[3];
            offsets_f64(C, m, om, sm);
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int t = s + 1; t < 3; ++t) {
                    const double rx = om[3 * t] - om[3 * s], ry = om[3 * t + 1] - om[3 * s + 1],
                                 rz = om[3 * t + 2] - om[3 * s + 2];
                    const int b = bin(rx * rx + ry * ry + rz * rz);
                    if (b >= 0 && b < (int)nb) atomicAdd(&bintra[b], 2u);
                }
        }
        unit_pairs<kEventSpan>(C, U, u, cut2, window, Q);
    }
    Q.drain(1u);
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < nb; b += kThreads) {
        const uint32_t all = bintra[b] + binter[b];
        if (shared_out) {  // several workgroups add into the histograms
            if (all) atomicAdd((unsigned long long*)&C.gofr_all[b], (unsigned long long)all);
            if (binter[b]) atomicAdd((unsigned long long*)&C.gofr_inter[b], (unsigned long long)binter[b]);
        } else {
            C.gofr_all[b] += all;
            C.gofr_inter[b] += binter[b];
        }
    }
    if (threadIdx.x == 0 && !shared_out) C.stats->n_gofr += 1;
}

// Ascending molecule index inside every cell of cells c0, c0 + cstep, ...,
// one wave per cell and a lane per molecule: its new place is the number of
// smaller indices in the cell.  Up to 8 cells of a wave have their loads in
// flight together; a cell of more than 64 molecules is sorted by one lane.
template <typename List, typename Starts>
__device__ void sort_cells(List list, Starts cellb, uint32_t c0, uint32_t cstep,
                           uint32_t ncell)
{
    const uint32_t lane = (uint32_t)__lane_id();
    for (uint32_t cg = c0; cg < ncell; cg += 8u * cstep) {
        uint32_t b[8], n[8], v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const uint32_t c = cg + (uint32_t)r * cstep;
            b[r] = 0;
            n[r] = 0;
            if (c < ncell) {
                b[r] = cellb[c];
                n[r] = cellb[c + 1] - b[r];
            }
            b[r] = (uint32_t)__builtin_amdgcn_readfirstlane((int)b[r]);
            n[r] = (uint32_t)__builtin_amdgcn_readfirstlane((int)n[r]);
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = lane < n[r] && n[r] <= 64u ? list[b[r] + lane] : 0xFFFFu;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (n[r] <= 1u) continue;
            if (n[r] <= 64u) {
                uint32_t rank = 0;
                for (uint32_t q = 0; q < n[r]; ++q) rank += rl_u(v[r], (int)q) < v[r] ? 1u : 0u;
                if (lane < n[r]) list[b[r] + rank] = (uint16_t)v[r];
            } else if (lane == 0) {
                const uint32_t lo = b[r], hi = b[r] + n[r];
                for (uint32_t i = lo + 1; i < hi; ++i) {
                    const uint16_t x = list[i];
                    uint32_t q = i;
                    while (q > lo && list[q - 1] > x) {
                        list[q] = list[q - 1];
                        --q;
                    }
                    list[q] = x;
                }
            }
        }
    }
}

// Cell grid of one sweep: counting sort of molecules by cell.
template <typename Real, int kMem>
__device__ void build_cells(const Ctx<Real, kMem>& C, double hx, double hy, double hz,
                            uint32_t* scratch)
{
    const uint32_t M = C.M, ncell = C.ncell;
    const int nc = (int)C.nc;
    for (uint32_t i = threadIdx.x; i <= ncell; i += kThreads) C.cellb[i] = 0;
    __syncthreads();
    for (uint32_t m = threadIdx.x; m < M; m += kThreads) {
        const int ix = cell_axis(C.com[m], hx, C.L, C.w, nc);
        const int iy = cell_axis(C.com[M + m], hy, C.L, C.w, nc);
        const int iz = cell_axis(C.com[2 * M + m], hz, C.L, C.w, nc);
        const uint32_t cid = (uint32_t)(ix + nc * (iy + nc * iz));
        C.cellid[m] = (uint16_t)cid;
        atomicAdd((uint32_t*)&C.cellb[cid + 1], 1u);
    }
    __syncthreads();
    block_excl_scan((uint32_t*)(C.cellb + 1), ncell, scratch);
    for (uint32_t m = threadIdx.x; m < M; m += kThreads) {
        const uint32_t pos = atomicAdd((uint32_t*)&C.cellb[C.cellid[m] + 1u], 1u);
        C.list[pos] = (uint16_t)m;
    }
    __syncthreads();
    sort_cells(C.list, C.cellb, wave_index(), kWaves, ncell);
    __syncthreads();
}

// Counters, kept in registers for the whole launch.
struct WaveCount {
    uint32_t att0, att1, att2, acc0, acc1, acc2, exits, overflows;
    uint64_t terms, tests;  // summed over the lanes
    double e;  // accepted dE of the current cell, in trial order
};

// A trial: the moved sites and the proposal, written by one lane and read by
// the wave that evaluates it and the lane that commits it.
template <typename Real>
struct alignas(16) TrialLds {
    R4<Real> old_site[3];  // moved sites before the move: offset from the old centre + sigma
    R4<Real> new_site[3];  // after the move: offset from the new centre + sigma
    double cm[3];          // centre of mass before the move
    Real dl[3];            // displacement of a translation, zero for the other moves
    uint32_t kind, mi;     // PropRec::kind, molecule index
    float mr[3];           // centre relative to the cell centre
    uint32_t types;        // of the molecule's sites
    double thr, a[4];      // PropRec
};
static_assert(offsetof(TrialLds<float>, kind) <= trial_bytes(false), "trial in flight (FP32)");
static_assert(offsetof(TrialLds<double>, kind) <= trial_bytes(true), "trial in flight (FP64)");
static_assert(sizeof(TrialLds<float>) == record_bytes(false) && sizeof(TrialLds<double>) == record_bytes(true),
              "trial record");

// A molecule near the current cell: its index and its centre relative to the
// cell centre (nearest image), rounded to FP16.  The coordinates only prune
// candidates (with a margin); the positions used for energies are formed from
// the FP64 centres.
struct alignas(8) NearEntry {
    uint16_t j;
    __fp16 rx, ry, rz;
};
static_assert(sizeof(NearEntry) == 8, "near-list entry");

// Per-wave LDS work areas (the near list is the workgroup's where its waves
// share a cell).
template <typename Real>
struct WaveLds {
    uint16_t* surv;       // molecules that passed the prune of the trial in flight
    uint16_t* seglo;      // neighbour row segments of the current cell
    uint16_t* segoff;
    NearEntry* near;      // molecules near the current cell
    TrialLds<Real>* tr;   // the trial in flight, or (waves that share a cell) the next 64 of the cell
    uint32_t near_cap;
};

// a / n for a < 2^16 and n < 2^8 with inv = 1.f / n: an integer division by a
// variable takes some 35 instructions.  The rounding errors of the product
// stay below the distance 0.5 / n of (a + 0.5) / n to the next integer.
__device__ __forceinline__ uint32_t small_div(uint32_t a, float inv) { return (uint32_t)(((float)a + 0.5f) * inv); }

// Axes of place v in an n x n x n block, x fastest.
__device__ __forceinline__ void split3(uint32_t v, int n, float inv, int& x, int& y, int& z)
{
    const uint32_t t = small_div(v, inv), u = small_div(t, inv);
    x = (int)(v - t * (uint32_t)n);
    y = (int)(t - u * (uint32_t)n);
    z = (int)u;
}

// Row of the stencil that this lane's segment lies in, with one or two
// segments a row: y | z << 8 from the stencil's corner.
struct StencilRows {
    int n;  // rows per axis
    uint32_t one, two;
};

template <typename Cx>
__device__ __forceinline__ StencilRows stencil_rows(const Cx& C)
{
    StencilRows w;
    w.n = (int)min(C.nc, 2u * C.k - 1u);
    const float inv = 1.f / (float)w.n;
    const uint32_t a = (uint32_t)__lane_id(), b = a >> 1;
    const uint32_t za = small_div(a, inv), zb = small_div(b, inv);
    w.one = (a - za * (uint32_t)w.n) | za << 8;
    w.two = (b - zb * (uint32_t)w.n) | zb << 8;
    return w;
}

// Neighbour cells of cell (cx, cy, cz) as row segments along x: (2r+1)^2 rows
// of 1 or 2 x-ranges (r = k - 1), those that hold molecules, in order: lane s
// has the molecules before segment s in the stencil (off) and what leads from a
// place in the stencil to one in the cell list (delta).  Writes the segment
// table too.
struct Segments {
    int n;
    uint32_t total, off, delta;
};

template <typename Real, int kMem>
__device__ __forceinline__ Segments stencil_segments(const Ctx<Real, kMem>& C, const StencilRows& rows,
                                                     int cx, int cy, int cz, uint16_t* seglo, uint16_t* segoff)
{
    const int lane = __lane_id();
    const int nc = (int)C.nc;
    const int r = (int)C.k - 1;
    const bool full = 2 * r + 1 >= nc;
    const int nrow = rows.n;
    int xa0, xb0, xa1 = 0, xb1 = -1;
    if (full) {
        xa0 = 0; xb0 = nc - 1;
    } else if (cx - r < 0) {
        xa0 = cx - r + nc; xb0 = nc - 1; xa1 = 0; xb1 = cx + r;
    } else if (cx + r >= nc) {
        xa0 = cx - r; xb0 = nc - 1; xa1 = 0; xb1 = cx + r - nc;
    } else {
        xa0 = cx - r; xb0 = cx + r;
    }
    const int nxr = xb1 >= xa1 ? 2 : 1;
    Segments g;
    uint32_t scnt = 0, lo = 0;
    if (lane < nrow * nrow * nxr) {
        const bool ixr = nxr == 2 && (lane & 1);
        const uint32_t yz = nxr == 2 ? rows.two : rows.one;
        int y = (int)(yz & 255u), z = (int)(yz >> 8);
        if (!full) {
            y += cy - r; z += cz - r;
            y += y < 0 ? nc : (y >= nc ? -nc : 0);
            z += z < 0 ? nc : (z >= nc ? -nc : 0);
        }
        const int xa = ixr ? xa1 : xa0, xb = ixr ? xb1 : xb0;
        const uint32_t rowbase = (uint32_t)(nc * (y + nc * z));
        lo = C.cellb[rowbase + xa];
        scnt = C.cellb[rowbase + xb + 1] - lo;
    }
    const uint32_t off = wave_excl_scan(scnt, &g.total);
    const uint64_t some = __ballot(scnt != 0u);
    g.n = (int)__popcll(some);
    // (a lane without one sends to one past them)
    const int to = 4 * (int)(scnt ? rank_below(some) : 63u);
    g.off = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)off);
    g.delta = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(lo - off));
    if (lane < g.n) {
        seglo[lane] = (uint16_t)(g.off + g.delta);
        segoff[lane] = (uint16_t)g.off;
    }
    wave_lds_sync();
    return g;
}

// This lane's place in the cell list, the (base + lane)-th of the stencil, or
// none past its end: the segments that start in the 64 places as bits, counted
// up to the lane's (about 25 instructions whatever the number of segments).
__device__ __forceinline__ uint32_t stencil_place(const Segments& g, uint32_t base, uint32_t none)
{
    const uint32_t lane = (uint32_t)__lane_id();
    const bool mine = lane < (uint32_t)g.n;
    const uint32_t p = g.off - base;  // >= 64: starts outside
    const uint32_t lo = wave_or_dpp(mine && p < 32u ? 1u << p : 0u);
    const uint32_t hi = wave_or_dpp(mine && p - 32u < 32u ? 1u << (p - 32u) : 0u);
    const uint32_t before = (uint32_t)__popcll(__ballot(mine && g.off < base));
    const uint64_t starts = (uint64_t)hi << 32 | lo;
    const uint32_t seg = before + rank_below(starts) + (uint32_t)((starts >> lane) & 1ull) - 1u;
    const uint32_t d = (uint32_t)__shfl((int)g.delta, (int)(seg & 63u));
    return base + lane < g.total ? base + lane + d : none;
}

// idx-th molecule of the stencil (segment table in LDS).
template <typename Real, int kMem>
__device__ __forceinline__ uint32_t stencil_molecule(const Ctx<Real, kMem>& C, const uint16_t* seglo,
                                                     const uint16_t* segoff, int nseg, uint32_t idx)
{
    int lo = 0, hi = nseg;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((uint32_t)segoff[mid] <= idx) lo = mid; else hi = mid;
    }
    return C.list[(uint32_t)seglo[lo] + (idx - (uint32_t)segoff[lo])];
}

constexpr uint32_t kNoMolecule = 0xFFFFFFFFu;

// Where a cell's trials read positions: centres as [3][stride] and site
// offsets as [3 * stride], indexed by a local molecule id (the molecule index
// itself, or the slot of a staged copy of the cell's neighbourhood).
template <typename Real, bool kLds>
struct View {
    template <typename T>
    using P = std::conditional_t<kLds, Lds<T>, Global<T>>;
    P<double>* com;
    P<R4<Real>>* sites;
    uint32_t stride;
    __device__ __forceinline__ double centre(uint32_t j, int a) const { return com[a * stride + j]; }
    __device__ __forceinline__ R4<Real> site(uint32_t j, uint32_t t) const { return load_site(sites + (3u * j + t)); }
    __device__ __forceinline__ void set_centre(uint32_t j, double x, double y, double z) const
    {
        com[j] = x; com[stride + j] = y; com[2 * stride + j] = z;
    }
    __device__ __forceinline__ void set_offset(uint32_t j, uint32_t t, const R4<Real>& v) const
    {
        auto* p = sites + (3u * j + t);
        p->x = v.x; p->y = v.y; p->z = v.z;
    }
    __device__ __forceinline__ void set_sigma(uint32_t j, uint32_t t, Real w) const { sites[3u * j + t].w = w; }
};

// The same straight from the molecule records, where a cell's neighbourhood is
// too large to be staged (commit_trial writes the records anyway).
template <typename Real>
struct RecView {
    Global<MolRec<Real>>* rec;
    const double* sigma;  // of types A, B, C
    __device__ __forceinline__ double centre(uint32_t j, int a) const { return agent_load(&rec[j].c[a]); }
    __device__ __forceinline__ R4<Real> site(uint32_t j, uint32_t t) const
    {
        const Global<MolRec<Real>>* p = rec + j;
        return R4<Real>{agent_load(&p->o[3u * t]), agent_load(&p->o[3u * t + 1u]), agent_load(&p->o[3u * t + 2u]),
                        (Real)sigma[(agent_load(&p->types) >> (8u * t)) & 0xFFu]};
    }
    __device__ __forceinline__ void set_centre(uint32_t, double, double, double) const {}
    __device__ __forceinline__ void set_offset(uint32_t, uint32_t, const R4<Real>&) const {}
    __device__ __forceinline__ void set_sigma(uint32_t, uint32_t, Real) const {}
};

// The moved sites of the trial in flight, in registers (wave-uniform).
template <typename Real>
struct Moved {
    R4<Real> o[3], n[3];
    Real dlx, dly, dlz;
    double cx, cy, cz;
};

// Pair terms of one candidate item (a site of a survivor, with the survivor's
// centre and the site's offset already loaded) with the moved sites before and
// after a move of kind kMove (0 translation, 1 rotation, 2 flip): Eq. (1)
// within each pair's cut-off.  Returns u_new - u_old (0 for an invalid item);
// sc gets u_new + u_old; terms counts the pairs inside the cut-off over the
// wave (popcounts of the compare masks).
template <int kMove, bool kLog, typename Real>
__device__ __forceinline__ Real item_terms(const Moved<Real>& mv, double L, double invL,
                                           double jx, double jy, double jz, const R4<Real>& sj,
                                           bool valid, Real rc2f, Real& sc, uint32_t& terms)
{
    const double dx = fma(-L, rint((jx - mv.cx) * invL), jx - mv.cx);
    const double dy = fma(-L, rint((jy - mv.cy) * invL), jy - mv.cy);
    const double dz = fma(-L, rint((jz - mv.cz) * invL), jz - mv.cz);
    Real px = (Real)dx + sj.x, py = (Real)dy + sj.y, pz = (Real)dz + sj.z;
    if (!valid) px = Real(1e4);
    Real d = Real(0);
    sc = Real(0);
    constexpr int kNmv = kMove == 2 ? 2 : 3;
#pragma unroll
    for (int v = 0; v < kNmv; ++v) {
        const R4<Real> o = mv.o[v];
        const Real rx = px - o.x, ry = py - o.y, rz = pz - o.z;
        const Real r2 = fma(rx, rx, fma(ry, ry, rz * rz));
        const Real sg = Real(0.5) * (o.w + sj.w);
        const Real s2 = sg * sg, rc2 = rc2f * s2;
        const bool io = r2 < rc2;
        const Real uo = io ? pair_u(s2, r2) : Real(0);
        Real r2n, s2n, rc2n;
        if (kMove == 0) {  // same offsets about the displaced centre
            const Real qx = rx - mv.dlx, qy = ry - mv.dly, qz = rz - mv.dlz;
            r2n = fma(qx, qx, fma(qy, qy, qz * qz));
            s2n = s2; rc2n = rc2;
        } else if (kMove == 1) {  // rotated offsets about the same centre
            const R4<Real> n = mv.n[v];
            const Real qx = px - n.x, qy = py - n.y, qz = pz - n.z;
            r2n = fma(qx, qx, fma(qy, qy, qz * qz));
            s2n = s2; rc2n = rc2;
        } else {  // same position, swapped type
            const Real sgn = Real(0.5) * (mv.n[v].w + sj.w);
            r2n = r2;
            s2n = sgn * sgn; rc2n = rc2f * s2n;
        }
        const bool in = r2n < rc2n;
        const Real un = in ? pair_u(s2n, r2n) : Real(0);
        d += un - uo;
        if (kLog) sc += un + uo;
        terms += (uint32_t)__popcll(__ballot(io)) + (uint32_t)__popcll(__ballot(in));
    }
    return d;
}

template <typename Real>
struct PassSum {
    Real d, s;       // sum of u_new - u_old, of u_new + u_old
    uint32_t terms;  // pairs inside the cut-off (wave total)
};

// One step of the item loop: items base + lane and base + 64 + lane (item
// 3 s + t = site t of survivor s), with the loads of both passes issued
// before any arithmetic.
template <int kMove, bool kLog, typename Real, typename Vw>
__device__ __forceinline__ PassSum<Real> item_pair_pass(const Vw& V, double L, double invL,
                                                        const uint16_t* surv, const Moved<Real>& mv,
                                                        uint32_t base, uint32_t nit, Real rc2f)
{
    const bool two = nit - base > 64u;  // wave-uniform: the second pass has items
    const uint32_t itA = base + (uint32_t)__lane_id(), itB = itA + 64u;
    const bool vA = itA < nit, vB = itB < nit;
    const uint32_t cA = vA ? itA : 0u, cB = vB ? itB : 0u;
    const uint32_t sA = cA / 3u, sB = cB / 3u;
    const uint32_t tA = cA - 3u * sA, tB = cB - 3u * sB;
    const uint32_t jA = surv[sA];
    uint32_t jB = 0;
    if (two) jB = surv[sB];
    const double xA = V.centre(jA, 0), yA = V.centre(jA, 1), zA = V.centre(jA, 2);
    const R4<Real> gA = V.site(jA, tA);
    double xB = 0.0, yB = 0.0, zB = 0.0;
    R4<Real> gB{};
    if (two) {
        xB = V.centre(jB, 0); yB = V.centre(jB, 1); zB = V.centre(jB, 2);
        gB = V.site(jB, tB);
    }
    __builtin_amdgcn_sched_barrier(0);
    Real sa = Real(0), sb = Real(0);
    uint32_t terms = 0;
    Real d = item_terms<kMove, kLog>(mv, L, invL, xA, yA, zA, gA, vA, rc2f, sa, terms);
    if (two) d += item_terms<kMove, kLog>(mv, L, invL, xB, yB, zB, gB, vB, rc2f, sb, terms);
    return PassSum<Real>{d, sa + sb, terms};
}

// Per-phase constants of the trial loop.
struct PhaseConst {
    double half_w, reach_box, step;
    float prune2;        // largest prune radius squared (3e38 when pruning is off)
    float pr_base, pr_step;  // radius = pr_base + pr_step * (own translation + same cell)
    float box_in;        // |relative centre| per axis below which an entry is in the cell
    bool prune_on;
    bool logging;
};

template <typename Real, int kMem>
__device__ __forceinline__ PhaseConst phase_const(const Ctx<Real, kMem>& C, uint64_t sweep)
{
    PhaseConst P;
    P.logging = C.log != nullptr && sweep - C.log_sweep0 < C.log_sweeps;
    P.half_w = 0.5 * C.w;
    const double reach = sqrt(C.reach2);
    P.reach_box = (reach + 1e-6) * (reach + 1e-6);
    // prune radius on the FP16 relative centres: own move + a neighbour of the
    // same cell that moved earlier in this cell + rounding
    P.step = C.dmax * 1.7320508075688772;
    const float prune_r = (float)(reach + 2.0 * P.step + 0.02);
    // the relative centres are unique images only while the list region stays
    // below half the box; otherwise every listed molecule survives the prune
    // (and FP16 keeps the rounding below the 0.02 margin only up to |r| < 16)
    const bool prune_ok = P.half_w + (double)prune_r + P.step < fmin(0.5 * C.L - 1e-3, 16.0);
    P.prune2 = prune_ok ? prune_r * prune_r : 3.0e38f;
    P.prune_on = prune_ok;
    // the margins a trial needs: its own move when it translates the
    // molecule, and the moves made earlier in this cell by molecules of the
    // cell (no other molecule within reach moves during the colour phase)
    P.pr_base = (float)(reach + 0.02);
    P.pr_step = (float)P.step;
    P.box_in = (float)(P.half_w + 0.05);
    return P;
}

// Entry idx of the near list as a lane holds it: local id, FP16-rounded
// relative centre and what an earlier move of the entry can add to the prune
// radius.
struct NearOne {
    uint32_t j;
    float x, y, z, more;
};

__device__ __forceinline__ NearOne near_one(const PhaseConst& P, const NearEntry* near, uint32_t idx, uint32_t n)
{
    NearOne r{kNoMolecule, 0.f, 0.f, 0.f, 0.f};
    if (idx < n) {
        const NearEntry e = near[idx];
        r.j = e.j;
        r.x = (float)e.rx; r.y = (float)e.ry; r.z = (float)e.rz;
    }
    const bool in_cell = fabsf(r.x) <= P.box_in && fabsf(r.y) <= P.box_in && fabsf(r.z) <= P.box_in;
    r.more = in_cell ? P.pr_step : 0.f;
    return r;
}

// The first entries of the near list (entries lane, lane + 64, ...) are held in
// registers; longer lists are read again from LDS at each trial.  FP64 trials of
// k_sweeps with the state in HBM have no registers left: ten of the twelve values
// came back from scratch memory at each trial, with three waits.  They read the
// entries from LDS, all at once (2197 molecules on one workgroup 1165 us a sweep
// held, 1050 so, 1400 803 and 705; with the state in LDS, or on the engine of
// several workgroups, held is 2 - 6 % faster).
template <typename Real, int kMem>
constexpr bool near_held() { return !(sizeof(Real) == 8 && kMem == kMemHbm); }

template <bool kHeld>
struct NearRegs {
    NearOne e[kHeld ? kNearSlots : 1];
    const NearEntry* near;
    uint32_t n;  // entries (0 after an overflow)
};

template <bool kHeld>
__device__ __forceinline__ NearRegs<kHeld> near_regs(const PhaseConst& P, const NearEntry* near, uint32_t nnear, bool overflow)
{
    NearRegs<kHeld> r;
    r.n = overflow ? 0u : nnear;
    r.near = near;
    if constexpr (kHeld) {
#pragma unroll
        for (int c = 0; c < kNearSlots; ++c) r.e[c] = near_one(P, near, (uint32_t)__lane_id() + 64u * c, r.n);
    }
    return r;
}

// Where the multi-workgroup engine stages a cell's neighbourhood (LDS of the
// workgroup): centres, sites, the molecule of each slot and the slot of each
// of the cell's own molecules.
template <typename Real>
struct StageLds {
    Lds<double>* com;     // [3][near_cap] centres
    Lds<R4<Real>>* site;  // [3 * near_cap] site offsets + sigma
    Lds<uint16_t>* own;   // slot of the cell's q-th molecule
    uint32_t* cnt;        // [2][kWaves] near molecules found by each wave
};

// Whether a molecule at (x, y, z) is within reach of the box of a cell centred
// at (bx0, by0, bz0), and its centre relative to the cell's.
template <typename Cx>
__device__ __forceinline__ bool near_box(const Cx& C, const PhaseConst& P, double x, double y, double z, double bx0,
                                         double by0, double bz0, float& fx, float& fy, float& fz)
{
    const double rx = min_image(x - bx0, C.L, C.invL);
    const double ry = min_image(y - by0, C.L, C.invL);
    const double rz = min_image(z - bz0, C.L, C.invL);
    const double ex = fmax(fabs(rx) - P.half_w, 0.0), ey = fmax(fabs(ry) - P.half_w, 0.0),
                 ez = fmax(fabs(rz) - P.half_w, 0.0);
    fx = (float)rx; fy = (float)ry; fz = (float)rz;
    return ex * ex + ey * ey + ez * ez < P.reach_box;
}

// The molecules whose centre is within reach of a cell's box, from the stencil
// segments of the cell list, into the near list in stencil order (index and
// FP16 relative centre; returns the count, sets overflow past the list's
// capacity).  By one wave, four molecules per lane at a time, the loads issued
// before any arithmetic.
template <typename Real, int kMem>
__device__ __forceinline__ uint32_t gather_near(const Ctx<Real, kMem>& C, const PhaseConst& P, const Segments& g,
                                                double bx0, double by0, double bz0, uint32_t cbeg,
                                                const WaveLds<Real>& W, bool& overflow)
{
    constexpr int kPer = 4;
    const uint32_t lane = (uint32_t)__lane_id();
    const uint32_t M = C.M;
    uint32_t nnear = 0;
    overflow = false;
    for (uint32_t b0 = 0; b0 < g.total; b0 += 64u * kPer) {
        uint32_t jj[kPer];
        double xx[kPer], yy[kPer], zz[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            jj[u] = cbeg;
            if (b0 + 64u * u < g.total) jj[u] = stencil_place(g, b0 + 64u * u, cbeg);  // (wave-uniform)
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) jj[u] = C.list[jj[u]];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            xx[u] = C.com[jj[u]];
            yy[u] = C.com[M + jj[u]];
            zz[u] = C.com[2 * M + jj[u]];
        }
        __builtin_amdgcn_sched_barrier(0);
        float fx[kPer], fy[kPer], fz[kPer];
        bool vv[kPer];
        uint64_t bm[kPer];
        uint32_t base[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            vv[u] = b0 + 64u * u + lane < g.total &&
                    near_box(C, P, xx[u], yy[u], zz[u], bx0, by0, bz0, fx[u], fy[u], fz[u]);
            bm[u] = __ballot(vv[u]);
            base[u] = nnear;
            nnear += (uint32_t)__popcll(bm[u]);
        }
        if (nnear > W.near_cap) {
            overflow = true;
            break;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (vv[u]) {
                NearEntry e;
                e.j = (uint16_t)jj[u];
                e.rx = (__fp16)fx[u]; e.ry = (__fp16)fy[u]; e.rz = (__fp16)fz[u];
                W.near[base[u] + rank_below(bm[u])] = e;
            }
        }
    }
    wave_lds_sync();
    return nnear;
}

// The same list by one wave from the molecule records, with copies of the
// molecules (centres, sites) in S, whose slots the list holds, and the slots of
// the cell's own molecules (list places cbeg .. cbeg + ccnt) in S.own.
template <typename Real, int kMem>
__device__ __forceinline__ uint32_t gather_wave(const Ctx<Real, kMem>& C, const PhaseConst& P, const Segments& g,
                                                double bx0, double by0, double bz0, uint32_t cbeg, uint32_t ccnt,
                                                __amdgpu_buffer_rsrc_t recs, const WaveLds<Real>& W,
                                                const StageLds<Real>& S, bool& overflow)
{
    constexpr int kPer = 2;
    uint32_t nnear = 0;
    overflow = false;
    for (uint32_t b0 = 0; b0 < g.total; b0 += 64u * kPer) {
        uint32_t place[kPer];
        MolRec<Real> mol[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            place[u] = cbeg;
            if (b0 + 64u * u < g.total) place[u] = stencil_place(g, b0 + 64u * u, cbeg);  // (wave-uniform)
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            mol[u] = agent_record<MolRec<Real>, mol_used<Real>()>(recs, C.list[place[u]]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            float fx, fy, fz;
            const bool vv = b0 + 64u * u + (uint32_t)__lane_id() < g.total &&
                            near_box(C, P, mol[u].c[0], mol[u].c[1], mol[u].c[2], bx0, by0, bz0, fx, fy, fz);
            const uint64_t bm = __ballot(vv);
            const uint32_t base = nnear;
            nnear += (uint32_t)__popcll(bm);
            if (nnear <= W.near_cap && vv) {
                const uint32_t slot = base + rank_below(bm);
                NearEntry e;
                e.j = (uint16_t)slot;
                e.rx = (__fp16)fx; e.ry = (__fp16)fy; e.rz = (__fp16)fz;
                W.near[slot] = e;
#pragma unroll
                for (int a = 0; a < 3; ++a) S.com[a * W.near_cap + slot] = mol[u].c[a];
#pragma unroll
                for (int t = 0; t < 3; ++t) store_site(S.site + 3 * slot + t, mol_site(C, mol[u], t));
                const uint32_t q = place[u] - cbeg;
                if (q < min(ccnt, W.near_cap)) S.own[q] = (uint16_t)slot;
            }
        }
        if (nnear > W.near_cap) {
            overflow = true;
            break;
        }
    }
    wave_lds_sync();
    return nnear;
}

// The same list by a whole workgroup, a molecule per thread at a time; the
// molecules are also copied to S (centres, sites) and the list holds their
// slots, and the cell's own molecules (list places cbeg .. cbeg + ccnt) get
// theirs in S.own.  place: list place of the thread's first one.
template <typename Real, int kMem>
__device__ __forceinline__ uint32_t gather_team(const Ctx<Real, kMem>& C, const PhaseConst& P, const Segments& g,
                                                double bx0, double by0, double bz0, uint32_t cbeg, uint32_t ccnt,
                                                uint32_t place, __amdgpu_buffer_rsrc_t recs, int wave,
                                                const WaveLds<Real>& W, const StageLds<Real>& S, bool& overflow)
{
    const uint32_t lane = (uint32_t)__lane_id();
    uint32_t nnear = 0;
    overflow = false;
    int par = 0;
    for (uint32_t b0 = 0; b0 < g.total; b0 += kThreads, par ^= 1) {
        const uint32_t at = b0 + 64u * (uint32_t)wave + lane;
        if (b0) place = stencil_place(g, b0 + 64u * (uint32_t)wave, cbeg);
        const uint32_t j = C.list[place];
        const MolRec<Real> mol = agent_record<MolRec<Real>, mol_used<Real>()>(recs, j);
        const double x = mol.c[0], y = mol.c[1], z = mol.c[2];
        __builtin_amdgcn_sched_barrier(0);
        float fx, fy, fz;
        const bool vv = at < g.total && near_box(C, P, x, y, z, bx0, by0, bz0, fx, fy, fz);
        const uint64_t bm = __ballot(vv);
        // this wave's place behind the earlier waves' finds
        if (lane == 0) S.cnt[par * kWaves + wave] = (uint32_t)__popcll(bm);
        __syncthreads();
        const uint32_t c = lane < (uint32_t)kWaves ? S.cnt[par * kWaves + lane] : 0u;
        const uint32_t inc = wave_incl_scan(c);
        const uint32_t base = nnear + (wave ? rl_u(inc, wave - 1) : 0u);
        nnear += rl_u(inc, kWaves - 1);
        if (nnear > W.near_cap) {
            overflow = true;
            break;
        }
        if (vv) {
            const uint32_t slot = base + rank_below(bm);
            NearEntry e;
            e.j = (uint16_t)slot;
            e.rx = (__fp16)fx; e.ry = (__fp16)fy; e.rz = (__fp16)fz;
            W.near[slot] = e;
            S.com[slot] = x;
            S.com[W.near_cap + slot] = y;
            S.com[2 * W.near_cap + slot] = z;
#pragma unroll
            for (int t = 0; t < 3; ++t) store_site(S.site + 3 * slot + t, mol_site(C, mol, t));
            const uint32_t q = place - cbeg;
            if (q < min(ccnt, W.near_cap)) S.own[q] = (uint16_t)slot;
        }
    }
    __syncthreads();
    return nnear;
}

// What every lane of an evaluating or deciding wave needs of the trial of lane
// l; the local id is the molecule's in the view.
struct TrialHead {
    uint32_t kind, mi, ml;
    float mrx, mry, mrz;
    double thr;
};

// A molecule's trial in one lane: proposal, centre, relative centre, sites
// and, for a rotation, the rotated offsets.
template <typename Real>
struct TrialRegs {
    TrialHead h;
    double a0, a1, a2, a3;
    double cmx, cmy, cmz;
    Real no[9];
    R4<Real> os0, os1, os2;  // the molecule's sites before its trial
    uint32_t types;          // (multi-workgroup engine)
};

// The trial of molecule mi (one lane) from the system's arrays: no trial before
// its own changes it.
template <typename Real, int kMem>
__device__ __forceinline__ void load_trial(const Ctx<Real, kMem>& C, const Global<PropRec>* props, uint32_t mi,
                                           double bx0, double by0, double bz0, TrialRegs<Real>& T)
{
    const uint32_t M = C.M;
    PropRec pr;
    if constexpr (has_records(kMem)) {
        pr = agent_record<PropRec>(agent_buffer((const void*)props, M * sizeof(PropRec)), mi);
        const MolRec<Real> mol =
            agent_record<MolRec<Real>, mol_used<Real>()>(agent_buffer((const void*)C.rec, M * sizeof(MolRec<Real>)), mi);
        T.cmx = mol.c[0]; T.cmy = mol.c[1]; T.cmz = mol.c[2];
        T.os0 = mol_site(C, mol, 0);
        T.os1 = mol_site(C, mol, 1);
        T.os2 = mol_site(C, mol, 2);
        T.types = mol.types;
    } else {
        pr = load_prop(props + mi);
        T.cmx = C.com[mi]; T.cmy = C.com[M + mi]; T.cmz = C.com[2 * M + mi];
        T.os0 = load_site(C.site + 3 * mi);
        T.os1 = load_site(C.site + 3 * mi + 1);
        T.os2 = load_site(C.site + 3 * mi + 2);
    }
    T.h.mi = T.h.ml = mi;
    T.h.kind = pr.kind;
    T.h.thr = pr.thr;
    T.a0 = pr.a0; T.a1 = pr.a1; T.a2 = pr.a2; T.a3 = pr.a3;
    T.h.mrx = (float)min_image(T.cmx - bx0, C.L, C.invL);
    T.h.mry = (float)min_image(T.cmy - by0, C.L, C.invL);
    T.h.mrz = (float)min_image(T.cmz - bz0, C.L, C.invL);
    if ((pr.kind & 15u) == 1u) {
        double rm[9];
        rotation(pr.a0, pr.a1, pr.a2, pr.a3, rm);
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const double b0 = body_at(C, s, 0), b1 = body_at(C, s, 1), b2 = body_at(C, s, 2);
            T.no[3 * s] = (Real)(rm[0] * b0 + rm[1] * b1 + rm[2] * b2);
            T.no[3 * s + 1] = (Real)(rm[3] * b0 + rm[4] * b1 + rm[5] * b2);
            T.no[3 * s + 2] = (Real)(rm[6] * b0 + rm[7] * b1 + rm[8] * b2);
        }
    }
}

// This lane's trial into its record: the moved sites (all three, or the two
// swapped ones of a flip) before and after the move.
template <typename Real>
__device__ __forceinline__ void publish_trial(const TrialRegs<Real>& T, TrialLds<Real>* tr)
{
    const uint32_t move = T.h.kind & 15u, axis = T.h.kind >> 8;
    const uint32_t a1 = (axis + 1) % 3, a2 = (axis + 2) % 3;
    if (move == 2u) {
        const R4<Real> x1 = a1 == 0u ? T.os0 : (a1 == 1u ? T.os1 : T.os2);
        const R4<Real> x2 = a2 == 0u ? T.os0 : (a2 == 1u ? T.os1 : T.os2);
        tr->old_site[0] = x1;
        tr->old_site[1] = x2;
        tr->new_site[0] = R4<Real>{x1.x, x1.y, x1.z, x2.w};
        tr->new_site[1] = R4<Real>{x2.x, x2.y, x2.z, x1.w};
    } else {
        tr->old_site[0] = T.os0;
        tr->old_site[1] = T.os1;
        tr->old_site[2] = T.os2;
        if (move == 1u) {
            tr->new_site[0] = R4<Real>{T.no[0], T.no[1], T.no[2], T.os0.w};
            tr->new_site[1] = R4<Real>{T.no[3], T.no[4], T.no[5], T.os1.w};
            tr->new_site[2] = R4<Real>{T.no[6], T.no[7], T.no[8], T.os2.w};
        }
    }
    tr->cm[0] = T.cmx; tr->cm[1] = T.cmy; tr->cm[2] = T.cmz;
    tr->dl[0] = move == 0u ? (Real)T.a0 : Real(0);
    tr->dl[1] = move == 0u ? (Real)T.a1 : Real(0);
    tr->dl[2] = move == 0u ? (Real)T.a2 : Real(0);
}

struct TrialSum {
    double de, scale;  // scale only in logged sweeps
    uint32_t terms, tests;
};
static_assert(sizeof(TrialSum) == kSumBytes, "evaluated trial");

// dE of the trial of lane i (not one that leaves its cell) against the present
// state, by the whole wave:
//   1. the moved sites are read from the trial's record;
//   2. the near list is pruned against the molecule's centre (FP32 on the
//      FP16 relative centres, with margins for the trial's own move and for
//      earlier moves of the same cell) and the survivors are compacted;
//   3. every site of every survivor takes a lane: the separation of the
//      centres is formed in FP64 with the nearest image and the site is
//      evaluated against the moved sites before and after the move (two
//      64-lane passes issued together);
//   4. a DPP reduction in FP64 gives dE in a fixed order.
// After a near-list overflow every stencil molecule is a candidate.
template <typename Real, int kMem, typename Vw>
__device__ __forceinline__ TrialSum eval_trial(const Ctx<Real, kMem>& C, const Vw& V, const PhaseConst& P,
                                               const TrialHead& T, int i, const NearRegs<near_held<Real, kMem>()>& nr, bool overflow,
                                               const Segments& g, const TrialLds<Real>* tr, const WaveLds<Real>& W)
{
    const int lane = __lane_id();
    const Real rc2f = (Real)C.rc2_factor;
    const uint32_t move = rl_u(T.kind, i) & 15u;
    const uint32_t mloc = rl_u(T.ml, i);
    // 1. the moved sites
    Moved<Real> mv;
    auto load_moved = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            mv.o[s] = tr->old_site[s];
            mv.n[s] = tr->new_site[s];
        }
        mv.cx = tr->cm[0]; mv.cy = tr->cm[1]; mv.cz = tr->cm[2];
        mv.dlx = tr->dl[0]; mv.dly = tr->dl[1]; mv.dlz = tr->dl[2];
        __builtin_amdgcn_sched_barrier(0);
    };

    Real acc = Real(0), accs = Real(0);
    TrialSum r{0.0, 0.0, 0u, 0u};
    // 3. one lane per (survivor, site), two passes at a time
    auto eval_items = [&](uint32_t nit) __attribute__((always_inline)) {
        r.tests += nit * (move == 2u ? 4u : 6u);
        for (uint32_t base = 0; base < nit; base += 128u) {
            PassSum<Real> ps;
            if (P.logging) {
                if (move == 0u)
                    ps = item_pair_pass<0, true>(V, C.L, C.invL, W.surv, mv, base, nit, rc2f);
                else if (move == 1u)
                    ps = item_pair_pass<1, true>(V, C.L, C.invL, W.surv, mv, base, nit, rc2f);
                else
                    ps = item_pair_pass<2, true>(V, C.L, C.invL, W.surv, mv, base, nit, rc2f);
            } else {
                if (move == 0u)
                    ps = item_pair_pass<0, false>(V, C.L, C.invL, W.surv, mv, base, nit, rc2f);
                else if (move == 1u)
                    ps = item_pair_pass<1, false>(V, C.L, C.invL, W.surv, mv, base, nit, rc2f);
                else
                    ps = item_pair_pass<2, false>(V, C.L, C.invL, W.surv, mv, base, nit, rc2f);
            }
            acc += ps.d;
            accs += ps.s;
            r.terms += ps.terms;
        }
    };

    // 2. prune and compact the survivors (the prune needs only the molecule's
    // relative centre, taken from the lane that holds it while that lane's
    // record is still being written); after a list overflow every stencil
    // molecule, 64 at a time.  (The two apart: with one loop for both the moved
    // sites were carried through it, which FP64 paid with spills: 1000 molecules
    // on one workgroup 447 us a sweep, 417 so, FP32 317 and 312.)
    if (!overflow) {
        uint32_t nsurv = 0;
        const float tmx = rl_f(T.mrx, i), tmy = rl_f(T.mry, i), tmz = rl_f(T.mrz, i);
        const float r_far = P.pr_base + (move == 0u ? P.pr_step : 0.f);
        auto prune = [&](const NearOne& e) __attribute__((always_inline)) {
            const float px = e.x - tmx, py = e.y - tmy, pz = e.z - tmz;
            const float rr = r_far + e.more;
            const float lim = P.prune_on ? rr * rr : P.prune2;
            const bool keep = e.j != kNoMolecule && e.j != mloc && px * px + py * py + pz * pz < lim;
            const uint64_t bm = __ballot(keep);
            if (keep) W.surv[nsurv + rank_below(bm)] = (uint16_t)e.j;
            nsurv += (uint32_t)__popcll(bm);
        };
        NearOne e[kNearSlots];
#pragma unroll
        for (int c = 0; c < kNearSlots; ++c) {
            if constexpr (near_held<Real, kMem>()) e[c] = nr.e[c];
            else e[c] = near_one(P, nr.near, (uint32_t)lane + 64u * c, nr.n);
        }
#pragma unroll
        for (int c = 0; c < kNearSlots; ++c) prune(e[c]);
        for (uint32_t b = 64u * kNearSlots; b < nr.n; b += 64u)
            prune(near_one(P, nr.near, b + (uint32_t)lane, nr.n));
        wave_lds_sync();  // the record and the survivors
        load_moved();
        if (nsurv) eval_items(3u * nsurv);
    } else {
        wave_lds_sync();  // the record
        load_moved();
        const uint32_t m = rl_u(T.mi, i);
        for (uint32_t base = 0; base < g.total; base += 64u) {
            const uint32_t idx = base + (uint32_t)lane;
            uint32_t j = kNoMolecule;
            if (idx < g.total) j = stencil_molecule(C, W.seglo, W.segoff, g.n, idx);
            const bool keep = j != kNoMolecule && j != m;
            const uint64_t bm = __ballot(keep);
            wave_lds_sync();
            if (keep) W.surv[rank_below(bm)] = (uint16_t)j;
            wave_lds_sync();
            const uint32_t nsurv = (uint32_t)__popcll(bm);
            if (nsurv) eval_items(3u * nsurv);
        }
    }
    r.de = wave_sum_dpp((double)acc);
    if (P.logging) r.scale = wave_sum_dpp((double)accs);
    return r;
}

// The accepted move of the trial of record tr, by one lane: centre, sites,
// orientation or types in the view (local id ml); by the multi-workgroup
// engine also in the molecule's record, which holds its centre and types until
// the end of the launch.
template <typename Real, int kMem, typename Vw>
__device__ __forceinline__ void commit_trial(const Ctx<Real, kMem>& C, const Vw& V,
                                             const TrialLds<Real>* tr, uint32_t kind, uint32_t mi, uint32_t ml,
                                             double a0, double a1, double a2, double a3)
{
    const uint32_t M = C.M;
    const uint32_t move = kind & 15u, axis = kind >> 8;
    if (move == 0u) {
        const double tx = tr->cm[0] + a0, ty = tr->cm[1] + a1, tz = tr->cm[2] + a2;
        // periodic images crossed (the shifts the wrap takes off)
        const double fx = floor(tx / C.L), fy = floor(ty / C.L), fz = floor(tz / C.L);
        const double nx = tx - C.L * fx, ny = ty - C.L * fy, nz = tz - C.L * fz;
        const int ix = (int)fx, iy = (int)fy, iz = (int)fz;
        V.set_centre(ml, nx, ny, nz);
        if constexpr (has_records(kMem)) {
            agent_store(&C.rec[mi].c[0], nx); agent_store(&C.rec[mi].c[1], ny); agent_store(&C.rec[mi].c[2], nz);
        }
        if (ix) atomicAdd((int32_t*)&C.img[mi], ix);
        if (iy) atomicAdd((int32_t*)&C.img[M + mi], iy);
        if (iz) atomicAdd((int32_t*)&C.img[2 * M + mi], iz);
    } else if (move == 1u) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const R4<Real> n = tr->new_site[s];
            V.set_offset(ml, s, n);
            if constexpr (has_records(kMem)) {
                agent_store(&C.rec[mi].o[3 * s], n.x);
                agent_store(&C.rec[mi].o[3 * s + 1], n.y);
                agent_store(&C.rec[mi].o[3 * s + 2], n.z);
            }
        }
        if constexpr (has_records(kMem)) {
            agent_store(&C.quat[mi], a0); agent_store(&C.quat[M + mi], a1);
            agent_store(&C.quat[2 * M + mi], a2); agent_store(&C.quat[3 * M + mi], a3);
        } else {
            C.quat[mi] = a0;
            C.quat[M + mi] = a1;
            C.quat[2 * M + mi] = a2;
            C.quat[3 * M + mi] = a3;
        }
    } else {
        const uint32_t s1 = (axis + 1) % 3, s2 = (axis + 2) % 3;
        V.set_sigma(ml, s1, tr->new_site[0].w);
        V.set_sigma(ml, s2, tr->new_site[1].w);
        uint32_t ty;
        if constexpr (has_records(kMem)) ty = tr->types;
        else ty = C.types[mi];
        const uint32_t t1 = (ty >> (8 * s1)) & 0xFFu, t2 = (ty >> (8 * s2)) & 0xFFu;
        uint32_t nt = ty & ~((0xFFu << (8 * s1)) | (0xFFu << (8 * s2)));
        nt |= (t2 << (8 * s1)) | (t1 << (8 * s2));
        if constexpr (has_records(kMem)) agent_store(&C.rec[mi].types, nt);
        else C.types[mi] = nt;
    }
}

template <typename Real, int kMem>
__device__ __forceinline__ void log_trial(const Ctx<Real, kMem>& C, const TrialHead& T, uint64_t sweep, bool exited,
                                          double de, double scale, uint32_t terms, bool accept)
{
    MoveRecord rec;
    rec.delta_e = de; rec.scale = scale; rec.t_log_u = T.thr; rec.sweep = sweep;
    rec.molecule = T.mi; rec.move = (uint8_t)(T.kind & 15u); rec.accepted = accept ? 1 : 0;
    rec.exited = exited ? 1 : 0; rec.axis = (uint8_t)(T.kind >> 8); rec.pair_terms = terms; rec.pad = 0;
    C.log[(sweep - C.log_sweep0) * C.M + T.mi] = rec;
}

// The trials of one cell (molecules list[cbeg .. cbeg + ccnt), a cell box
// centred at (bx0, by0, bz0)), in ascending order, by one wave.  Positions are
// read through V (local ids: molecule indices).  After a near-list overflow
// every stencil molecule is a candidate.
template <typename Real, int kMem, typename Vw>
__device__ void cell_trials(const Ctx<Real, kMem>& C, const Vw& V, const Global<PropRec>* props,
                            uint64_t sweep, const PhaseConst& P, uint32_t cbeg, uint32_t ccnt,
                            double bx0, double by0, double bz0, const NearRegs<near_held<Real, kMem>()>& nr, bool overflow,
                            const Segments& g, const WaveLds<Real>& W, WaveCount& wc,
                            const Lds<uint16_t>* own_slot = nullptr)
{
    const int lane = __lane_id();
    for (uint32_t q0 = 0; q0 < ccnt; q0 += 64u) {
        const uint32_t n = min(64u, ccnt - q0);
        TrialRegs<Real> T{};
        if ((uint32_t)lane < n) {
            load_trial(C, props, C.list[cbeg + q0 + lane], bx0, by0, bz0, T);
            if (own_slot) T.h.ml = own_slot[q0 + lane];
        }
        for (uint32_t q = 0; q < n; ++q) {
            const int i = (int)q;
            const uint32_t kind = rl_u(T.h.kind, i), move = kind & 15u;
            wc.att0 += move == 0u;
            wc.att1 += move == 1u;
            wc.att2 += move == 2u;
            if ((kind >> 4) & 1u) {
                wc.exits += 1;
                // (the axis of a move that exits is 255)
                if (P.logging && lane == i) log_trial(C, T.h, sweep, true, 0.0, 0.0, 0u, false);
                continue;
            }
            if (lane == i) {
                publish_trial(T, W.tr);
                if constexpr (has_records(kMem)) W.tr->types = T.types;
            }
            const TrialSum r = eval_trial(C, V, P, T.h, i, nr, overflow, g, W.tr, W);
            // Metropolis on the FP64 sum
            const double thr = rl_d(T.h.thr, i);
            const bool accept = (r.de <= 0.0) || (thr < -r.de);
            wc.terms += lane == 0 ? r.terms : 0u;
            wc.tests += lane == 0 ? r.tests : 0u;
            if (accept) {
                wc.acc0 += move == 0u;
                wc.acc1 += move == 1u;
                wc.acc2 += move == 2u;
                wc.e += r.de;
            }
            if (lane == i) {
                if (accept)
                    commit_trial(C, V, W.tr, kind, T.h.mi, T.h.ml, T.a0, T.a1, T.a2, T.a3);
                if (P.logging) log_trial(C, T.h, sweep, false, r.de, r.scale, r.terms, accept);
            }
            wave_lds_sync();
        }
    }
}

// Trials q0 .. q0 + 64 of a cell (list places cbeg ..) into the records, a lane
// each.
template <typename Real, int kMem>
__device__ __forceinline__ void load_records(const Ctx<Real, kMem>& C, const Global<PropRec>* props, uint32_t cbeg,
                                             uint32_t ccnt, uint32_t q0, double bx0, double by0, double bz0,
                                             TrialLds<Real>* recs)
{
    const uint32_t q = q0 + (uint32_t)__lane_id();
    if (q < ccnt) {
        TrialRegs<Real> T;
        load_trial(C, props, C.list[cbeg + q], bx0, by0, bz0, T);
        TrialLds<Real>* tr = recs + (q - q0);
        publish_trial(T, tr);
        tr->kind = T.h.kind; tr->mi = T.h.mi; tr->types = T.types;
        tr->mr[0] = T.h.mrx; tr->mr[1] = T.h.mry; tr->mr[2] = T.h.mrz;
        tr->thr = T.h.thr;
        tr->a[0] = T.a0; tr->a[1] = T.a1; tr->a[2] = T.a2; tr->a[3] = T.a3;
    }
}

// The trials of one cell in ascending order by a whole workgroup; the records
// of the first 64 are there.
//
// A wave issues an instruction about every eighth cycle, so a cell's chain of
// trials on one wave lasts as long as all their instructions; but only about
// one trial in six is accepted, and all before it can be evaluated on the same
// state.  Each wave evaluates one of the next kWaves trials as it would alone;
// then every wave decides them in order: those up to the first accepted one
// stand, a lane commits it, and the later ones are evaluated again.  So
// every decision is taken on the state its predecessors left, with the same
// dE.
template <bool kStaged, typename Real, int kMem, typename Vw>
__device__ __forceinline__ void team_trials(const Ctx<Real, kMem>& C, const Vw& V,
                                            const Global<PropRec>* props, uint64_t sweep, const PhaseConst& P,
                                            uint32_t cbeg, uint32_t ccnt, double bx0, double by0, double bz0,
                                            const NearRegs<near_held<Real, kMem>()>& nr, bool overflow, const Segments& g, int wave,
                                            const Lds<uint16_t>* own_slot, const WaveLds<Real>& W, TrialSum* sums,
                                            WaveCount& wc)
{
    const uint32_t lane = (uint32_t)__lane_id();
    int turn = 0;
    for (uint32_t q0 = 0; q0 < ccnt; q0 += 64u) {
        const uint32_t n = min(64u, ccnt - q0);
        const bool mine = lane < n;
        if (q0) {
            // every wave has its heads of the last 64 (a round's barriers say
            // so too, but there is none when all 64 leave the cell)
            __syncthreads();
            if (wave == 0) load_records(C, props, cbeg, ccnt, q0, bx0, by0, bz0, W.tr);
            __syncthreads();
        }
        TrialHead T{};
        if (mine) {
            const TrialLds<Real>* tr = W.tr + lane;
            T.kind = tr->kind; T.mi = tr->mi;
            T.ml = kStaged ? (uint32_t)own_slot[q0 + lane] : T.mi;
            T.mrx = tr->mr[0]; T.mry = tr->mr[1]; T.mrz = tr->mr[2];
            T.thr = tr->thr;
        }
        const uint32_t move = T.kind & 15u;
        const bool exited = mine && ((T.kind >> 4) & 1u);
        const uint64_t exits = __ballot(exited);
        if (wave == 0) {
            wc.att0 += (uint32_t)__popcll(__ballot(mine && move == 0u));
            wc.att1 += (uint32_t)__popcll(__ballot(mine && move == 1u));
            wc.att2 += (uint32_t)__popcll(__ballot(mine && move == 2u));
            wc.exits += (uint32_t)__popcll(exits);
            if (P.logging && exited) log_trial(C, T, sweep, true, 0.0, 0.0, 0u, false);
        }
        uint64_t todo = (n >= 64u ? ~0ull : (1ull << n) - 1ull) & ~exits;
        while (todo) {
            // the wave's trial: the wave-th of those left
            uint64_t left = todo;
            for (int w = 0; w < wave; ++w) left &= left - 1ull;
            TrialSum* sum = sums + turn * kWaves;
            if (left) {
                const int i = (int)__builtin_ctzll(left);
                const TrialSum r = eval_trial(C, V, P, T, i, nr, overflow, g, W.tr + i, W);
                if (lane == 0) sum[wave] = r;
            }
            __syncthreads();
            // decided in order by every wave alike
            const uint32_t rank = rank_below(todo);
            const bool in = ((todo >> lane) & 1ull) && rank < (uint32_t)kWaves;
            const uint64_t group = __ballot(in);
            const double de = sum[rank & (kWaves - 1)].de;
            const bool accept = in && ((de <= 0.0) || (T.thr < -de));
            const uint64_t acc = __ballot(accept);
            const uint64_t done = acc ? group & ((acc & (0ull - acc)) * 2ull - 1ull) : group;
            todo &= ~done;
            if (wave == 0) {
                if ((done >> lane) & 1ull) {
                    const TrialSum r = sum[rank];
                    wc.terms += r.terms;
                    wc.tests += r.tests;
                    if (P.logging) log_trial(C, T, sweep, false, r.de, r.scale, r.terms, accept);
                }
            }
            if (acc) {
                const int i = (int)__builtin_ctzll(acc);
                // a lane of the last wave commits it, wave 0 counts it
                if (wave == kWaves - 1) {
                    if ((int)lane == i) {
                        const TrialLds<Real>* tr = W.tr + i;
                        commit_trial(C, V, tr, T.kind, T.mi, T.ml, tr->a[0], tr->a[1], tr->a[2],
                                                          tr->a[3]);
                    }
                } else if (wave == 0) {
                    wc.e += rl_d(de, i);
                    const uint32_t mq = rl_u(move, i);
                    wc.acc0 += mq == 0u;
                    wc.acc1 += mq == 1u;
                    wc.acc2 += mq == 2u;
                }
                if (todo || q0 + 64u < ccnt) {
                    if (!kStaged) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    __syncthreads();
                }
            }
            turn ^= 1;
        }
    }
    __syncthreads();  // the cell's LDS areas are free again
}

// All trials of the cells of colour `col` owned by this wave of the
// single-workgroup engine: per cell, the near list from the system's own
// arrays, then the cell's trials.
template <typename Real, int kMem>
__device__ void run_phase(const Ctx<Real, kMem>& C, const Global<PropRec>* props, int col, uint64_t sweep,
                          double hx, double hy, double hz, const StencilRows& rows, const WaveLds<Real>& W,
                          WaveCount& wc)
{
    const int wave = wave_index();
    const int lane = __lane_id();
    const float invk = 1.f / (float)C.k;
    const int k = (int)C.k, nc = (int)C.nc, na = (int)small_div(C.nc, invk);
    const int nact = na * na * na;
    const float inva = 1.f / (float)na;
    int kx, ky, kz;
    split3((uint32_t)col, k, invk, kx, ky, kz);
    const PhaseConst P = phase_const(C, sweep);
    const View<Real, kMem == kMemLds> V{C.com, C.site, C.M};
    // With at most one cell per wave, the colour's cells go to the waves in
    // order of decreasing molecule count: the lower waves of each SIMD, whose
    // instructions issue first, take the larger cells, so the two waves of a
    // SIMD tend to finish together.  Otherwise wave w takes cells
    // w + kWaves ci.  Cells of a colour do not interact, so any assignment
    // gives the same results.
    const bool ranked = nact <= kWaves;
    uint32_t rank = 0;
    if (ranked) {
        uint32_t cnt = 0;
        if (lane < nact) {
            int cx, cy, cz;
            split3((uint32_t)lane, na, inva, cx, cy, cz);
            cx = kx + k * cx; cy = ky + k * cy; cz = kz + k * cz;
            const uint32_t cell = (uint32_t)(cx + nc * (cy + nc * cz));
            cnt = C.cellb[cell + 1] - C.cellb[cell];
        }
        for (int j = 0; j < nact; ++j) {
            const uint32_t cj = rl_u(cnt, j);
            rank += (cj > cnt || (cj == cnt && j < lane)) ? 1u : 0u;
        }
    }
    const int ncw = (nact + kWaves - 1) / kWaves;

    for (int ci = 0; ci < ncw; ++ci) {
        int a = wave + kWaves * ci;
        if (ranked) {
            const uint64_t bm = __ballot(lane < nact && rank == (uint32_t)wave);
            a = bm ? __ffsll((long long)bm) - 1 : nact;
        }
        if (a >= nact) continue;
        int cx, cy, cz;
        split3((uint32_t)a, na, inva, cx, cy, cz);
        cx = kx + k * cx; cy = ky + k * cy; cz = kz + k * cz;
        const uint32_t cell = (uint32_t)(cx + nc * (cy + nc * cz));
        const uint32_t cbeg = uniform(C.cellb[cell]), ccnt = uniform(C.cellb[cell + 1]) - cbeg;
        if (ccnt == 0) {
            if (__lane_id() == 0) C.ecell[cell] = 0.0;
            continue;
        }
        const double bx0 = hx + ((double)cx + 0.5) * C.w;
        const double by0 = hy + ((double)cy + 0.5) * C.w;
        const double bz0 = hz + ((double)cz + 0.5) * C.w;
        const Segments g = stencil_segments(C, rows, cx, cy, cz, W.seglo, W.segoff);
        bool overflow;
        const uint32_t nnear = gather_near(C, P, g, bx0, by0, bz0, cbeg, W, overflow);
        const auto nr = near_regs<near_held<Real, kMem>()>(P, W.near, nnear, overflow);
        wc.overflows += overflow ? 1u : 0u;
        wc.e = 0.0;
        cell_trials(C, V, props, sweep, P, cbeg, ccnt, bx0, by0, bz0, nr, overflow, g, W, wc);
        if (__lane_id() == 0) C.ecell[cell] = wc.e;
    }
}

// Fill the per-system constants of a workgroup (before any store).
template <typename Real, int kMem>
__device__ __forceinline__ void load_ctx(Ctx<Real, kMem>& C, const SysDev* __restrict__ Dp)
{
    C.M = Dp->M; C.k = Dp->k; C.nc = Dp->nc; C.ncell = Dp->ncell;
    C.seed_lo = Dp->seed_lo; C.seed_hi = Dp->seed_hi;
    C.resum_interval = Dp->resum_interval; C.obs_interval = Dp->obs_interval;
    C.gofr_interval = Dp->gofr_interval; C.obs_start = Dp->obs_start;
    C.max_samples = Dp->max_samples; C.gofr_nbins = Dp->gofr_nbins;
    C.L = Dp->L; C.invL = 1.0 / Dp->L; C.w = Dp->w; C.T = Dp->T;
    C.p_flip = Dp->p_flip; C.p_ft = Dp->p_ft; C.dmax = Dp->dmax; C.rot_max = Dp->rot_max;
    C.reach2 = Dp->reach2; C.radius = Dp->radius; C.rc2_factor = Dp->rc2_factor;
    C.bR = Dp->body[0]; C.bH = Dp->body[4];
    C.sig0 = Dp->sigma[0]; C.sig1 = Dp->sigma[1]; C.sig2 = Dp->sigma[2];
    C.gofr_dr = Dp->gofr_dr; C.gofr_rmax = Dp->gofr_rmax;
    using X = Ctx<Real, kMem>;
    C.gcom = (typename X::template Dev<double>*)Dp->com;
    C.quat = (typename X::template Dev<double>*)Dp->quat;
    C.types = (typename X::template Dev<uint32_t>*)Dp->types;
    C.img = (typename X::template Dev<int32_t>*)Dp->img;
    C.u0 = Dp->u0; C.kref = Dp->kref; C.r0 = Dp->r0; C.o0 = Dp->o0; C.fs = Dp->fs; C.fs_cm = Dp->fs_cm; C.mom = Dp->mom;
    C.fs_q = Dp->fs_q; C.fs_q_cm = Dp->fs_q_cm;
    C.stats = Dp->stats; C.e_samples = Dp->e_samples; C.drift_samples = Dp->drift_samples;
    C.gofr_all = Dp->gofr_all; C.gofr_inter = Dp->gofr_inter; C.c2 = Dp->c2;
    C.c2_sweep = Dp->c2_sweep;
    C.log = (MoveRecord*)Dp->log; C.log_sweep0 = Dp->log_sweep0; C.log_sweeps = Dp->log_sweeps;
    C.gpart = Dp->g_part;
}

// The work arrays of a system in the workgroup's LDS, or in its buffer.
template <typename Real, int kMem>
__device__ __forceinline__ void work_arrays(Ctx<Real, kMem>& C, const SysDev* __restrict__ Dp, unsigned char* smem,
                                            const LdsLayout& L)
{
    using X = Ctx<Real, kMem>;
    constexpr bool lds = kMem == kMemLds;
    C.com = (typename X::template Work<double>*)(lds ? smem + L.com : (unsigned char*)Dp->com);
    C.site = (typename X::template Work<R4<Real>>*)(lds ? smem + L.site : (unsigned char*)Dp->g_site);
    C.rec = (Global<MolRec<Real>>*)Dp->g_site;
    C.cellb = (typename X::template Index<uint32_t>*)(lds ? smem + L.cell : (unsigned char*)Dp->g_cell);
    C.cellid = (typename X::template Work<uint16_t>*)(lds ? smem + L.cellid : (unsigned char*)Dp->g_cellid);
    C.list = (typename X::template Index<uint16_t>*)(lds ? smem + L.list : (unsigned char*)Dp->g_list);
    C.ecell = (typename X::template Work<double>*)(lds ? smem + L.ecell : (unsigned char*)Dp->g_ecell);
    C.off = nullptr;
}

// The scheduled re-sum and C_2 sample of a sweep inside the batch's sweep
// kernel (not inlined: its registers stay out of the sweep loop's).  The
// context is rebuilt from the descriptor and the LDS layout the kernel uses.
template <typename Real, int kMem>
__device__ __attribute__((noinline)) void inline_events(const SysDev* __restrict__ Dp, unsigned char* smem,
                                                       uint64_t sweep, uint64_t origin, bool resum, bool c2)
{
    Ctx<Real, kMem> E;
    load_ctx(E, Dp);
    const int tid = threadIdx.x;
    const bool fp64 = sizeof(Real) == 8;
    const LdsLayout L = lds_layout(fp64, kMem == kMemLds, E.M, E.ncell, Dp->near_cap);
    E.bins = nullptr;
    E.misc = (double*)(smem + L.misc);
    E.red = E.misc + 8;
    work_arrays(E, Dp, smem, L);
    Stats* st = E.stats;
    __syncthreads();
    if (resum) {
        // (the waves' work areas are free between sweeps)
        constexpr uint32_t kWords = kGofrQueue + 3u * (kInlineSpan + 64u);
        static_assert(kWaves * kWords * 4u <= kWaves * (kNearMin * 10u + 4u * kMaxSeg), "survivors, segments, near lists");
        uint32_t* queue = (uint32_t*)(smem + L.surv) + (size_t)wave_index() * kWords;
        const EventUnits U = event_units(E.M);
        resum_units<kInlineSpan>(E, U, (uint32_t)wave_index(), kWaves, queue, (float*)(queue + kGofrQueue));
        __syncthreads();
        const double e = sum_units(E, U.count());
        if (tid == 0) {
            // re-anchor the accumulated energy: each drift sample is the
            // error of one window
            const double drift = E.misc[0] - e;
            E.misc[0] = e;
            st->e_resum = e;
            st->drift = drift;
            st->resum_sweep = sweep;
            st->n_resum += 1;
            if (st->n_drift < E.max_samples) E.drift_samples[st->n_drift] = drift;
            st->n_drift += 1;
            if (sweep > E.resum_interval && fabs(drift) > st->max_abs_drift) st->max_abs_drift = fabs(drift);
        }
        __syncthreads();
    }
    if (c2) {
        store_dyn(E, st, sweep - origin);
        __syncthreads();
    }
}

// The hot kernel: n checkerboard sweeps of every slot's system, one
// workgroup per system, with the state resident in LDS when it fits.  The
// variant with kInl also takes the scheduled re-sums and C_2 samples of slots
// flagged kFlagInline (a batch's systems); the plain one leaves them to the
// event kernel.
template <typename Real, bool kRes, bool kInl>
__device__ __forceinline__ void sweep_system(const Slot& sl, unsigned char* smem)
{
    const SysDev* __restrict__ Dp = sl.sys;
    constexpr int kMem = kRes ? kMemLds : kMemHbm;
    Ctx<Real, kMem> C;
    load_ctx(C, Dp);
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const bool fp64 = sizeof(Real) == 8;
    const LdsLayout L = lds_layout(fp64, kRes, C.M, C.ncell, Dp->near_cap);
    C.red = nullptr;
    C.bins = nullptr;
    C.misc = (double*)(smem + L.misc);
    work_arrays(C, Dp, smem, L);
    const uint32_t near_cap = Dp->near_cap;
    WaveLds<Real> W;
    W.surv = (uint16_t*)(smem + L.surv) + wave * near_cap;
    W.seglo = (uint16_t*)(smem + L.seglo) + wave * kMaxSeg;
    W.segoff = (uint16_t*)(smem + L.segoff) + wave * kMaxSeg;
    W.near = (NearEntry*)(smem + L.near) + wave * near_cap;
    W.tr = (TrialLds<Real>*)(smem + L.trial + wave * trial_bytes(fp64));  // up to TrialLds::kind
    W.near_cap = near_cap;
    Global<PropRec>* props = (Global<PropRec>*)Dp->props;
    uint32_t* uscratch = (uint32_t*)(C.misc + 8);
    const uint32_t M = C.M;

    Stats* st = C.stats;
    if (tid == 0) {
        C.misc[0] = st->e_acc;
        C.misc[1] = C.sig0;
        C.misc[2] = C.sig1;
        C.misc[3] = C.sig2;
    }
    __syncthreads();
    if (kRes)
        for (uint32_t i = tid; i < 3 * M; i += kThreads) C.com[i] = C.gcom[i];
    for (uint32_t m = tid; m < M; m += kThreads) store_sites_from_quat(C, m);
    WaveCount wc{};
    uint64_t sweep = st->sweep;
    const uint64_t origin = st->obs_origin;
    __syncthreads();

    const int ncol = (int)(C.k * C.k * C.k);
    const StencilRows rows = stencil_rows(C);
    for (uint64_t it = 0; it < sl.n_sweeps; ++it) {
        const U4 g = philox10(0xFFFFFFFFu, (uint32_t)sweep, (uint32_t)(sweep >> 32), 3u, C.seed_lo,
                              C.seed_hi);
        const double hx = C.w * unit_open(g.x), hy = C.w * unit_open(g.y),
                     hz = C.w * unit_open(g.z);
        build_cells(C, hx, hy, hz, uscratch);
        propose_all(C, props, sweep, hx, hy, hz);
        __syncthreads();
        for (int col = 0; col < ncol; ++col) {
            run_phase(C, props, col, sweep, hx, hy, hz, rows, W, wc);
            __syncthreads();
        }
        // E_acc += the sweep's dE (sweep_energy); E/M samples
        ++sweep;
        if (wave == 0) {
            const double e = C.misc[0] + sweep_energy([&](uint32_t c) { return (double)C.ecell[c]; }, C.ncell);
            if (lane == 0) C.misc[0] = e;
        }
        if (tid == 0) {
            const double e = C.misc[0];
            const uint64_t t = sweep - origin;
            if (t >= C.obs_start && C.obs_interval && t % C.obs_interval == 0) {
                const double em = e / (double)M;
                if (st->n_e < C.max_samples) C.e_samples[st->n_e] = em;
                st->n_e += 1;
                st->e_sum += em;
                st->e_sumsq += em * em;
            }
        }
        if (kInl && (sl.flags & kFlagInline)) {
            // this sweep's scheduled re-sum and C_2 sample, taken here with the
            // event kernel's routines and thread mapping (the same sums), so
            // that a slice need not end at them
            const bool resum = C.resum_interval && sweep % C.resum_interval == 0;
            const bool c2 = is_c2_time(sweep - origin);
            if (resum || c2) inline_events<Real, kMem>(Dp, smem, sweep, origin, resum, c2);
        }
    }

    // write back
    if (kRes)
        for (uint32_t i = tid; i < 3 * M; i += kThreads) C.gcom[i] = C.com[i];
    const unsigned long long terms = wave_sum_ull(wc.terms), tests = wave_sum_ull(wc.tests);
    if (lane == 0) {
        const uint64_t att[3] = {wc.att0, wc.att1, wc.att2}, acc[3] = {wc.acc0, wc.acc1, wc.acc2};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (att[i]) atomicAdd((unsigned long long*)&st->attempts[i], (unsigned long long)att[i]);
            if (acc[i]) atomicAdd((unsigned long long*)&st->accepts[i], (unsigned long long)acc[i]);
        }
        if (wc.exits) atomicAdd((unsigned long long*)&st->exits, (unsigned long long)wc.exits);
        if (terms) atomicAdd((unsigned long long*)&st->pair_terms, terms);
        if (tests) atomicAdd((unsigned long long*)&st->pair_tests, tests);
        if (wc.overflows)
            atomicAdd((unsigned long long*)&st->near_overflows, (unsigned long long)wc.overflows);
    }
    __syncthreads();
    if (tid == 0) {
        st->sweep = sweep;
        st->e_acc = C.misc[0];
    }
}

// A workgroup takes the system of table entry blockIdx.x and those that follow it
// (Slot::pad).
template <typename Real, bool kRes, bool kInl>
__global__ void __launch_bounds__(kThreads) k_sweeps(const Slot* __restrict__ slots, Slot one)
{
    extern __shared__ __align__(16) unsigned char smem[];
    for (uint32_t i = blockIdx.x;;) {
        const Slot sl = slots ? slots[i] : one;
        if (sl.sys == nullptr || sl.n_sweeps == 0) return;  // (the same for the whole workgroup)
        sweep_system<Real, kRes, kInl>(sl, smem);
        if (sl.pad == 0u) return;
        i = sl.pad - 1u;
        __syncthreads();
    }
}

// Cold work at event sweeps, straight from the HBM state in FP64: re-sum of
// the energy (and drift), a g(r) frame, a C_2 sample, observable reset.
__global__ void __launch_bounds__(kThreads) k_events(const Slot* __restrict__ slots, Slot one)
{
    __shared__ double red[kWaves];
    __shared__ double misc[16];
    __shared__ uint32_t bins[2 * kGofrBins];
    __shared__ uint32_t gqueue[kWaves * kGofrQueue];
    __shared__ float windows[kWaves * 3u * (kEventSpan + 64u)];
    extern __shared__ __align__(16) unsigned char ev_stage[];
    const Slot sl = slots ? slots[blockIdx.x] : one;
    if (sl.sys == nullptr || sl.flags == 0) return;
    Ctx<double, kMemAny> C;
    load_ctx(C, sl.sys);
    C.com = C.gcom;
    C.red = red;
    C.misc = misc;
    C.bins = bins;
    C.ecell = nullptr;
    C.off = nullptr;
    C.site = nullptr;
    C.cellb = nullptr;
    C.cellid = nullptr;
    C.list = nullptr;
    const int tid = threadIdx.x;
    uint32_t* queue = gqueue + wave_index() * kGofrQueue;
    float* window = windows + wave_index() * 3u * (kEventSpan + 64u);
    Stats* st = C.stats;
    if (tid == 0) {
        misc[1] = C.sig0;
        misc[2] = C.sig1;
        misc[3] = C.sig2;
    }
    const uint64_t sweep = st->sweep;
    const double e_acc = st->e_acc;
    const uint32_t f = sl.flags;
    const uint32_t M = C.M;
    if ((f & (kFlagResumSet | kFlagResumReport | kFlagResumPeriodic | kFlagGofr)) &&
        !(f & kFlagParts) && M <= kEventStage) {
        // the O(M^2) loops read centres, orientations and types from an LDS
        // copy (same values, same order: the same sums)
        // (with the site offsets computed once per molecule when they fit)
        double* scom = (double*)ev_stage;
        double* squat = scom + 3 * M;
        const bool pre = size_t(M) * (12 * sizeof(double) + sizeof(uint32_t)) <= kEventStageBytes;
        uint32_t* stypes = (uint32_t*)(squat + (pre ? 9 : 4) * M);
        for (uint32_t i = tid; i < 3 * M; i += kThreads) scom[i] = C.gcom[i];
        for (uint32_t i = tid; i < M; i += kThreads) stypes[i] = C.types[i];
        if (pre) {
            __syncthreads();  // sigma table (misc) before offsets_f64
            for (uint32_t m = tid; m < M; m += kThreads) {
                double o[9], sg[3];
                offsets_f64(C, m, o, sg);
#pragma unroll
                for (int i = 0; i < 9; ++i) squat[i * M + m] = o[i];
            }
            C.off = squat;
        } else {
            for (uint32_t i = tid; i < 4 * M; i += kThreads) squat[i] = C.quat[i];
            C.quat = squat;
        }
        C.com = scom;
        C.types = stypes;
    }
    __syncthreads();
    if (f & kFlagObsReset) {
        reset_observables(C);
        __syncthreads();
    }
    if (f & (kFlagResumSet | kFlagResumReport | kFlagResumPeriodic)) {
        double e;
        // (kFlagParts: the units were added up by the multi-workgroup kernel)
        uint32_t n = sl.pad;
        if (!(f & kFlagParts)) {
            const EventUnits U = event_units(M);
            resum_units<kEventSpan>(C, U, (uint32_t)wave_index(), kWaves, queue, window);
            n = U.count();
            __syncthreads();
        }
        e = sum_units(C, n);
        if (tid == 0) {
            const double acc = (f & kFlagResumSet) ? e : e_acc;
            // a set or a scheduled re-sum re-anchors the accumulated energy, so
            // each drift sample is the error of one window
            if (f & (kFlagResumSet | kFlagResumPeriodic)) st->e_acc = e;
            const double drift = acc - e;
            st->e_resum = e;
            st->drift = drift;
            st->resum_sweep = sweep;
            if (f & kFlagResumPeriodic) {
                st->n_resum += 1;
                if (st->n_drift < C.max_samples) C.drift_samples[st->n_drift] = drift;
                st->n_drift += 1;
                if (sweep > C.resum_interval && fabs(drift) > st->max_abs_drift)
                    st->max_abs_drift = fabs(drift);
            }
        }
        __syncthreads();
    }
    if (f & kFlagGofr) {
        if (f & kFlagParts) {
            if (tid == 0) st->n_gofr += 1;
        } else {
            gofr_frame(C, event_units(M), (uint32_t)wave_index(), kWaves, false, queue, window);
        }
        __syncthreads();
    }
    if (f & kFlagC2) store_dyn(C, st, sweep - st->obs_origin);
}

// ----------------------------------------------------- multi-workgroup --
//
// The spread engine advances a system with several workgroups in one launch,
// its state in HBM.  A sweep is: cell and proposal of every molecule, an equal
// share to each workgroup; the cell lists, which each workgroup puts together in
// its own LDS from the molecules' cells; then the k^3 colours.  For every cell
// the workgroup (or one wave of it) copies the neighbourhood (molecules within
// reach of the cell's box) into LDS and runs the cell's trials on the copy,
// writing each accepted move through to HBM.  All workgroups meet after each of
// the first two steps and at the end of the sweep; between colours a cell waits
// for its neighbours only.  So the decisions are those of one workgroup.
//
// What bounds it (1000 molecules, FP32, T = 0.75, cycles of a sweep on 8
// workgroups, 335k in all): rounds of side-by-side trials 130k (27 of 4.8k: 2.9k
// to evaluate, 1k until the last wave has, 0.9k to decide), waiting for
// neighbours with more rounds 60k, copying neighbourhoods 40k (1.4k of it the
// latency of the records), what a cell needs before the wait 40k, proposals and
// lists 26k.  At the start of this design, with a wave per cell on two compute
// units or one, it was 750k.

// The workgroups of one system that share its sweeps.  The launch gives it up
// to n of them, but promises nothing about when they start, and a workgroup
// that waits for one that cannot start would wait for ever.  So the crew is
// whoever is on the device: every workgroup draws a ticket, the holder of the
// first waits until all n are drawn or kCrewWait has passed (the others' places
// are taken by other work then), and the tickets drawn so far are the crew, with
// the ticket as its member's place.  A later one finds the crew closed and
// leaves.  Any number of workgroups gives the same results.
//
// The words in the system's buffer (SysDev::g_bar, zero at launch).
// Barriers count in two steps where the crew is large: 256 workgroups that add
// to one word queue for longer than the barrier takes.
enum : int { kBarCount = 0, kBarTickets = 1, kBarCrew = 2, kBarGroups = 16, kBarStride = 16 };
constexpr uint32_t kGroup = 16;  // workgroups that count together
static_assert(kBarWords >= kBarGroups + kBarStride * (int)((256 + kGroup - 1) / kGroup), "barrier words");
constexpr uint64_t kCrewWait = 100000;  // ticks of the 100 MHz clock: 1 ms

// Barrier of the crew: a counter that each workgroup raises once per barrier; a
// workgroup passes the n-th barrier when the counter reaches n x (workgroups of
// the crew).  Every wait is bounded (SysDev::barrier_polls polls, seconds by
// default): past the bound the system is marked faulted (Stats::fault) and
// sys_sync returns false, and the workgroup must leave the kernel at once.  A
// workgroup thus only goes on past a barrier when every workgroup has finished
// the work before it, and the others, which then miss its increments, time out
// too.
struct SysBarrier {
    uint32_t* count;
    uint32_t nblk;   // workgroups, and how many of them (or groups of them) raise count
    uint32_t ncount;
    uint32_t* group;  // the word of this workgroup's group, or null
    uint32_t ngroup;  // its workgroups
    uint32_t epoch;
    uint32_t polls;
};
// Every wave waits for its own stores; kFenced: some of the exchanged data lies
// in the caches (write back, invalidate), otherwise all went past them.

__device__ __forceinline__ SysBarrier crew_barrier(uint32_t* bar, uint32_t nblk, uint32_t bid, uint32_t polls)
{
    SysBarrier B{bar + kBarCount, nblk, nblk, nullptr, 0u, 0u, polls};
    if (nblk > 2u * kGroup) {
        const uint32_t g = bid / kGroup;
        B.ncount = (nblk + kGroup - 1u) / kGroup;
        B.group = bar + kBarGroups + kBarStride * g;
        B.ngroup = min(kGroup, nblk - g * kGroup);
    }
    return B;
}

// This workgroup's place in the crew and the crew's size, 0 when it has none.
// Call with the whole workgroup; `out` is two words of its LDS.
__device__ uint32_t join_crew(uint32_t* bar, uint32_t n, uint32_t polls, uint32_t* fault, uint32_t* out,
                              uint32_t* place)
{
    if (threadIdx.x == 0) {
        const uint32_t t = __hip_atomic_fetch_add(bar + kBarTickets, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t crew = 0;
        if (t == 0) {
            const uint64_t t0 = wall_clock64();
            do {
                crew = __hip_atomic_load(bar + kBarTickets, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } while (crew < n && wall_clock64() - t0 < kCrewWait);
            crew = min(crew, n);
            __hip_atomic_store(bar + kBarCrew, crew, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            // the first ticket's holder is on the device and closes the crew
            // within kCrewWait
            uint32_t spins = 0;
            const uint32_t most = max(polls, 1u << 20);
            while ((crew = __hip_atomic_load(bar + kBarCrew, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0u) {
                __builtin_amdgcn_s_sleep(1);
                if (++spins >= most) {
                    __hip_atomic_store(fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
            }
        }
        out[0] = t;
        out[1] = t < crew ? crew : 0u;
    }
    __syncthreads();
    *place = uniform(out[0]);
    const uint32_t crew = uniform(out[1]);
    __syncthreads();
    return crew;
}

// The two halves: every wave has arrived before sys_arrive's count, and what
// does not touch the other workgroups' work can be done before the wait.
template <bool kFenced>
__device__ __forceinline__ void sys_arrive(SysBarrier& B)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (B.nblk == 1) return;
    ++B.epoch;
    if (threadIdx.x == 0) {
        if (kFenced) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        bool last = true;
        if (B.group) {
            const uint32_t n =
                __hip_atomic_fetch_add(B.group, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
            last = n == B.epoch * B.ngroup;
            if (kFenced && last) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
        }
        if (last) __hip_atomic_fetch_add(B.count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <bool kFenced>
__device__ __forceinline__ bool sys_wait(SysBarrier& B, uint32_t* fault, uint32_t* flag)
{
    if (B.nblk == 1) {
        __syncthreads();
        return true;
    }
    if (threadIdx.x == 0) {
        uint32_t bad = 0;
        // the counter may wrap in a long launch: compare the signed distance
        // (the workgroups are never 2^31 increments apart)
        const uint32_t target = B.epoch * B.ncount;
        uint32_t spins = 0;
        while ((int32_t)(__hip_atomic_load(B.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) -
                         target) < 0) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins >= B.polls) {
                bad = 1;
                __hip_atomic_store(fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
        if (kFenced) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *flag = bad;
    }
    __syncthreads();
    return *flag == 0u;
}

template <bool kFenced>
__device__ __forceinline__ bool sys_sync(SysBarrier& B, uint32_t* fault, uint32_t* flag)
{
    sys_arrive<kFenced>(B);
    return sys_wait<kFenced>(B, fault, flag);
}

// The molecules of every cell, in no order, in this workgroup's LDS from the
// cell of every molecule: count, scan, fill.  base is C.cellb (ncell + 1
// words), tmp M words of LDS, both this workgroup's.
template <int kThr, typename Real>
__device__ __forceinline__ void team_fill(const Ctx<Real, kMemTeam>& C, Lds<uint16_t>* tmp, uint32_t* scratch)
{
    const uint32_t tid = threadIdx.x, M = C.M, ncell = C.ncell;
    Lds<uint32_t>* base = C.cellb;
    Lds<uint32_t>* cur = base + 1;
    // eight molecules per thread and turn: one 16-byte load, eight LDS
    // operations in flight; the cells of the first kHeld turns stay in registers
    using C8 = uint16_t __attribute__((ext_vector_type(8)));
    constexpr uint32_t kHeld = 4;
    const uint32_t M8 = M / 8u;
    const __amdgpu_buffer_rsrc_t ids = agent_buffer((const void*)C.cellid, M * sizeof(uint16_t));
    auto ids_at = [&](uint32_t i) { return __builtin_bit_cast(C8, agent_words(ids, 16u * i)); };
    C8 held[kHeld];
#pragma unroll
    for (uint32_t u = 0; u < kHeld; ++u) held[u] = ids_at(tid + u * kThr);  // (none past the end)
    auto turns = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t u = 0; u < kHeld; ++u)
            if (tid + u * kThr < M8) f(tid + u * kThr, held[u]);
        for (uint32_t i = tid + kHeld * kThr; i < M8; i += kThr) f(i, ids_at(i));
    };
    if (tid == 0) base[0] = 0u;
    for (uint32_t c = tid; c < ncell; c += kThr) cur[c] = 0u;
    const uint32_t mr = 8u * M8 + tid, cr = mr < M ? (uint32_t)agent_load(&C.cellid[mr]) : 0u;  // the last M mod 8
    __syncthreads();
    turns([&](uint32_t, C8 c) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 8; ++t) atomicAdd((uint32_t*)&cur[c[t]], 1u);
    });
    if (mr < M) atomicAdd((uint32_t*)&cur[cr], 1u);
    __syncthreads();
    block_excl_scan_t<kThr>((uint32_t*)cur, ncell, scratch);
    // a cell's cursor moves from its start to its end, which is the next start
    turns([&](uint32_t i, C8 c) __attribute__((always_inline)) {
        uint32_t at[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) at[t] = atomicAdd((uint32_t*)&cur[c[t]], 1u);
#pragma unroll
        for (int t = 0; t < 8; ++t) tmp[at[t]] = (uint16_t)(8u * i + t);
    });
    if (mr < M) tmp[atomicAdd((uint32_t*)&cur[cr], 1u)] = (uint16_t)mr;
    __syncthreads();
}

// Each of the molecules at places [p0, p1) of tmp (whole cells) to its rank
// among its cell's (ascending index), four places per thread at a time.
template <int kThr, typename Real, typename Put>
__device__ __forceinline__ void team_rank(const Ctx<Real, kMemTeam>& C, const Lds<uint16_t>* tmp, uint32_t p0,
                                          uint32_t p1, Put put)
{
    const Lds<uint32_t>* base = C.cellb;
    for (uint32_t q0 = p0 + threadIdx.x; q0 < p1; q0 += 4u * kThr) {
        uint32_t m[4], lo[4], n[4], rank[4], most = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) m[t] = tmp[min(q0 + t * kThr, p1 - 1u)];
#pragma unroll
        for (int t = 0; t < 4; ++t) lo[t] = agent_load(&C.cellid[m[t]]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t c = lo[t];
            lo[t] = base[c];
            n[t] = q0 + t * kThr < p1 ? base[c + 1] - lo[t] : 0u;
            rank[t] = 0;
            most = max(most, n[t]);
        }
        for (uint32_t q = 0; q < most; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) rank[t] += q < n[t] && (uint32_t)tmp[min(lo[t] + q, p1 - 1u)] < m[t] ? 1u : 0u;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (n[t]) put(lo[t] + rank[t], (uint16_t)m[t]);
    }
}

// The cells whose trials come before a cell's: its neighbours (the cells of the
// stencil) of lower colours.  A workgroup waits for these only, not for the
// whole colour, so one cell with many rounds holds up its neighbours and not
// the others (8000 molecules: 13k cycles of waiting per colour with a barrier).
// Cells of one colour are not neighbours, and a neighbour of a higher colour
// waits for this cell, so nothing in the stencil changes while a cell runs and
// its trials see what they see colour by colour.  Waiting only for lower
// colours, which every workgroup has behind it, cannot end in a circle.
struct CellDeps {
    uint32_t o0, o1;  // offsets of this lane's neighbours from the cell: x | y << 8 | z << 16, 255: none
};

template <typename Cx>
__device__ __forceinline__ CellDeps cell_deps(const Cx& C)
{
    const int r = (int)C.k - 1, n = 2 * r + 1;
    const float inv = 1.f / (float)n;
    auto at = [&](uint32_t i) {
        int x, y, z;
        split3(i, n, inv, x, y, z);
        return i < (uint32_t)(n * n * n) ? (uint32_t)(x | y << 8 | z << 16) : 255u;
    };
    return CellDeps{at((uint32_t)__lane_id()), at((uint32_t)__lane_id() + 64u)};
}

constexpr uint32_t kNoCell = 0xFFFFFFFFu;

// This lane's neighbours of lower colours of cell (cx, cy, cz), whose colour is
// col at (kx, ky, kz).
template <typename Cx>
__device__ __forceinline__ void cell_waits(const Cx& C, const CellDeps& D, int col, int cx, int cy, int cz, int kx,
                                           int ky, int kz, uint32_t& dep0, uint32_t& dep1)
{
    const int k = (int)C.k, nc = (int)C.nc, r = k - 1;
    auto at = [&](uint32_t o) {
        const int dx = (int)(o & 255u) - r, dy = (int)((o >> 8) & 255u) - r, dz = (int)((o >> 16) & 255u) - r;
        auto wrapped = [](int v, int n) { return v + (v < 0 ? n : (v >= n ? -n : 0)); };
        const int c = wrapped(kx + dx, k) + k * (wrapped(ky + dy, k) + k * wrapped(kz + dz, k));
        const int x = wrapped(cx + dx, nc), y = wrapped(cy + dy, nc), z = wrapped(cz + dz, nc);
        return (o & 255u) != 255u && c < col ? (uint32_t)(x + nc * (y + nc * z)) : kNoCell;
    };
    dep0 = at(D.o0);
    dep1 = at(D.o1);
}

// Waits until they have all had sweep n of the launch (bounded as sys_wait's
// wait; false past the bound).  By one wave, whose lanes hold the cells.
__device__ __forceinline__ bool wave_cells_done(const Global<uint32_t>* done, uint32_t dep0, uint32_t dep1, uint32_t n,
                                                uint32_t polls, uint32_t* fault)
{
    for (uint32_t spins = 0;;) {
        const uint32_t a = dep0 == kNoCell ? n : agent_load(done + dep0);
        const uint32_t b = dep1 == kNoCell ? n : agent_load(done + dep1);
        if (__ballot(a < n || b < n) == 0ull) return true;
        if (++spins >= polls) break;
        __builtin_amdgcn_s_sleep(1);
    }
    if (__lane_id() == 0) __hip_atomic_store(fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
}

// The same for a workgroup; wave 0's lanes hold the cells.
__device__ __forceinline__ bool cells_done(const Global<uint32_t>* done, uint32_t dep0, uint32_t dep1, uint32_t n,
                                           uint32_t polls, uint32_t* fault, uint32_t* flag)
{
    if (threadIdx.x < 64) {
        const bool ok = wave_cells_done(done, dep0, dep1, n, polls, fault);
        if (threadIdx.x == 0) *flag = ok ? 0u : 1u;
    }
    __syncthreads();
    return *flag == 0u;
}

// Up to this size each workgroup ranks all molecules itself: two a thread take
// 4k cycles, a barrier and the copy back about 5k and each further thousand
// 2k (measured at 1000 and 8000 molecules).
constexpr uint32_t kRankAlone = 2048;

// Sweeps by workgroups that take a cell of the current colour each (team_trials)
// with the cell's neighbourhood staged in LDS and the state in HBM; kMem says
// where the cell lists are (kMemTeam: in LDS, where they fit; kMemCrew: in the
// buffer).  With kCellWaves each of some of its waves takes a cell instead (two
// kernels: one with both has 10 % slower trials, from spilled registers), in
// workgroups of kThr threads (see cell_threads).  One launch can advance several
// systems: slot i owns workgroups [first_block, first_block + n_blocks) and runs
// n_sweeps sweeps; the workgroups of a system synchronise among themselves
// (sys_sync), so systems of one launch run at their own pace.
template <typename Real, int kMem, bool kCellWaves, int kThr>
__global__ void __launch_bounds__(kThr) k_spread(const SpreadSlot* __restrict__ slots,
                                                     uint32_t n_slots, SpreadSlot one)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr bool fp64 = sizeof(Real) == 8, kFenced = kMem == kMemCrew;
    SpreadSlot sl = one;
    if (slots) {
        for (uint32_t i = 0; i < n_slots; ++i) {
            const SpreadSlot t = slots[i];
            if (blockIdx.x >= t.first_block && blockIdx.x < t.first_block + t.n_blocks) {
                sl = t;
                break;
            }
        }
    }
    if (sl.sys == nullptr || sl.n_blocks == 0) return;  // a workgroup of no system
    SysDev* __restrict__ Dp = sl.sys;
    Ctx<Real, kMem> C;
    load_ctx(C, Dp);
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const uint32_t cell_waves = kCellWaves ? sl.waves : 0u;
    const SpreadLayout Y = spread_layout(fp64, kMem == kMemTeam, C.M, C.ncell, Dp->near_cap, cell_waves);
    // the staged cell is the workgroup's, or the wave's
    unsigned char* own = smem + (cell_waves ? min((uint32_t)wave, cell_waves - 1u) * Y.wave : 0u);
    StageLds<Real> S;
    S.com = (Lds<double>*)(own + Y.com);
    S.site = (Lds<R4<Real>>*)(own + Y.site);
    S.own = (Lds<uint16_t>*)(own + Y.own);
    S.cnt = (uint32_t*)(smem + Y.cnt);
    WaveLds<Real> W;
    W.near_cap = Dp->near_cap;
    W.surv = (uint16_t*)(own + Y.surv) + (cell_waves ? 0u : (uint32_t)wave * W.near_cap);
    W.seglo = (uint16_t*)(own + Y.seg);
    W.segoff = W.seglo + kMaxSeg;
    W.near = (NearEntry*)(own + Y.near);
    W.tr = (TrialLds<Real>*)(own + Y.trial);
    TrialSum* sums = (TrialSum*)(smem + Y.sums);
    C.misc = (double*)(smem + Y.misc);
    work_arrays(C, Dp, smem, LdsLayout{});
    if (kMem == kMemTeam) {
        C.cellb = (typename Ctx<Real, kMem>::template Index<uint32_t>*)(smem + Y.cell);
        C.list = (typename Ctx<Real, kMem>::template Index<uint16_t>*)(smem + Y.list);
    }
    C.red = nullptr;
    C.bins = nullptr;
    Global<uint32_t>* cnt = (Global<uint32_t>*)Dp->g_cnt;
    Global<uint32_t>* fill = cnt + C.ncell;
    Global<PropRec>* props = (Global<PropRec>*)Dp->props;
    Stats* st = C.stats;
    const uint32_t M = C.M, ncell = C.ncell;
    uint32_t* bflag = (uint32_t*)(C.misc + 14);
    uint32_t bid = 0, nblk = 1;
    if (sl.n_blocks > 1) {
        nblk = join_crew(Dp->g_bar, sl.n_blocks, Dp->barrier_polls, &st->fault, bflag, &bid);
        if (nblk == 0) return;
    }
    // this workgroup's molecules: an equal share
    const uint32_t m0 = (uint32_t)((uint64_t)M * bid / nblk), m1 = (uint32_t)((uint64_t)M * (bid + 1u) / nblk);
    const uint32_t gtid = bid * kThr + tid, GT = nblk * kThr;
    const uint32_t gw = bid * (kThr / 64) + wave, NW = nblk * (kThr / 64);
    const int k = (int)C.k, nc = (int)C.nc, na = nc / k;
    const uint32_t nact = (uint32_t)(na * na * na);
    const int ncol = k * k * k;
    const float invk = 1.f / (float)k, inva = 1.f / (float)na;
    const StencilRows rows = stencil_rows(C);

    if (tid == 0) {
        C.misc[1] = C.sig0;
        C.misc[2] = C.sig1;
        C.misc[3] = C.sig2;
        *bflag = 0u;
    }
    __syncthreads();
    for (uint32_t m = m0 + tid; m < m1; m += kThr) store_sites_from_quat(C, m);
    for (uint32_t c = gtid; c < 2 * ncell; c += GT) agent_store(&cnt[c], 0u);
    Global<uint32_t>* done = cnt;  // (kMemTeam) the last sweep of the launch each cell has had, from 1
    const CellDeps deps = cell_deps(C);
    const __amdgpu_buffer_rsrc_t recs = agent_buffer((const void*)C.rec, M * sizeof(MolRec<Real>));
    WaveCount wc{};
    double e_acc = st->e_acc;
    uint64_t sweep = st->sweep;
    const uint64_t origin = st->obs_origin;
    SysBarrier B = crew_barrier(Dp->g_bar, nblk, bid, Dp->barrier_polls);
    // at every barrier a workgroup that timed out leaves (see sys_sync)
    if (!sys_sync<kFenced>(B, &st->fault, bflag)) return;

    for (uint64_t it = 0; it < sl.n_sweeps; ++it) {
        const U4 g = philox10(0xFFFFFFFFu, (uint32_t)sweep, (uint32_t)(sweep >> 32), 3u, C.seed_lo,
                              C.seed_hi);
        const double hx = C.w * unit_open(g.x), hy = C.w * unit_open(g.y),
                     hz = C.w * unit_open(g.z);
        // cell of every molecule, counts, proposals
        // (the proposals through LDS, so that they leave in whole lines: as
        // single words past the caches they took 20 us at 27000 molecules)
        for (uint32_t b0 = m0; b0 < m1; b0 += kThr) {
            const uint32_t m = b0 + tid, n = min((uint32_t)kThr, m1 - b0);
            Lds<PropRec>* out = (Lds<PropRec>*)smem;
            if (m < m1) {
                const int ix = cell_axis(agent_load(&C.rec[m].c[0]), hx, C.L, C.w, nc);
                const int iy = cell_axis(agent_load(&C.rec[m].c[1]), hy, C.L, C.w, nc);
                const int iz = cell_axis(agent_load(&C.rec[m].c[2]), hz, C.L, C.w, nc);
                const uint32_t cid = (uint32_t)(ix + nc * (iy + nc * iz));
                agent_store(&C.cellid[m], (uint16_t)cid);
                if constexpr (kMem == kMemCrew) atomicAdd((uint32_t*)&cnt[cid], 1u);
                const PropRec pr = propose(C, m, sweep, hx, hy, hz, ix, iy, iz);
                out[tid].kind = pr.kind; out[tid].pad = 0u; out[tid].thr = pr.thr;
                out[tid].a0 = pr.a0; out[tid].a1 = pr.a1; out[tid].a2 = pr.a2; out[tid].a3 = pr.a3;
            }
            __syncthreads();
            const __amdgpu_buffer_rsrc_t pb = agent_buffer((const void*)props, M * sizeof(PropRec));
            constexpr uint32_t kW = sizeof(PropRec) / sizeof(Words);
            for (uint32_t i = tid; i < kW * n; i += kThr)
                agent_put_words(pb, b0 * (uint32_t)sizeof(PropRec) + 16u * i, ((Lds<Words>*)smem)[i]);
            __syncthreads();
        }
        if (!sys_sync<kFenced>(B, &st->fault, bflag)) return;
        if constexpr (kMem == kMemTeam) {
            Lds<uint16_t>* tmp = (Lds<uint16_t>*)smem;
            team_fill<kThr>(C, tmp, (uint32_t*)(C.misc + 8));
            Global<uint16_t>* gl = (Global<uint16_t>*)Dp->g_list;
            const bool shared = nblk > 1 && M > kRankAlone;
            if (shared) {
                // each workgroup ranks the molecules of its share of the cells
                const uint32_t c0 = (uint32_t)((uint64_t)ncell * bid / nblk),
                               c1 = (uint32_t)((uint64_t)ncell * (bid + 1u) / nblk);
                team_rank<kThr>(C, tmp, uniform(C.cellb[c0]), uniform(C.cellb[c1]),
                          [&](uint32_t at, uint16_t m) { agent_store(gl + at, m); });
                if (!sys_sync<kFenced>(B, &st->fault, bflag)) return;
                using C8 = uint16_t __attribute__((ext_vector_type(8)));
                const __amdgpu_buffer_rsrc_t gb = agent_buffer((const void*)gl, M * sizeof(uint16_t));
                for (uint32_t i = tid; i < M / 8u; i += kThr) {
                    const C8 v = __builtin_bit_cast(C8, agent_words(gb, 16u * i));
#pragma unroll
                    for (int t = 0; t < 8; ++t) C.list[8u * i + t] = v[t];
                }
                for (uint32_t i = M / 8u * 8u + tid; i < M; i += kThr) C.list[i] = agent_load(gl + i);
            } else {
                team_rank<kThr>(C, tmp, 0u, M, [&](uint32_t at, uint16_t m) { C.list[at] = m; });
            }
            __syncthreads();
            if (it + 1 == sl.n_sweeps) {  // for a scheduled re-sum after the launch
                Global<uint32_t>* gc = (Global<uint32_t>*)Dp->g_cell;
                for (uint32_t c = bid * kThr + tid; c <= ncell; c += nblk * kThr) gc[c] = C.cellb[c];
                if (!shared)
                    for (uint32_t i = bid * kThr + tid; i < M; i += nblk * kThr) gl[i] = C.list[i];
            }
        } else {
            // cell starts (exclusive scan of the counts); counts cleared for the
            // next sweep
            if (bid == 0) {
                for (uint32_t c = tid; c < ncell; c += kThr) C.cellb[c] = cnt[c];
                __syncthreads();
                block_excl_scan_t<kThr>((uint32_t*)C.cellb, ncell, (uint32_t*)(C.misc + 8));
                if (tid == 0) C.cellb[ncell] = M;
                for (uint32_t c = tid; c < ncell; c += kThr) cnt[c] = 0;
            }
            if (!sys_sync<kFenced>(B, &st->fault, bflag)) return;
            for (uint32_t m = gtid; m < M; m += GT) {
                const uint32_t c = C.cellid[m];
                C.list[C.cellb[c] + atomicAdd((uint32_t*)&fill[c], 1u)] = (uint16_t)m;
            }
            if (!sys_sync<kFenced>(B, &st->fault, bflag)) return;
            // ascending molecule index inside every cell
            sort_cells(C.list, C.cellb, gw, NW, ncell);
            for (uint32_t c = gtid; c < ncell; c += GT) fill[c] = 0;
            if (!sys_sync<kFenced>(B, &st->fault, bflag)) return;
        }

        const PhaseConst P = phase_const(C, sweep);
        const View<Real, true> V{S.com, S.site, W.near_cap};
        // What the next cell needs and the other workgroups do not change is
        // done as soon as the last cell is, before the wait for them: its
        // trials (no trial but its own changes a molecule of the cell) and the
        // list places of its neighbourhood.
        struct Cell {
            uint32_t id, beg, cnt, place, dep0, dep1;
            double bx0, by0, bz0;
            Segments sg;
        };
        auto take_cell = [&](int col, uint32_t a) __attribute__((always_inline)) {
            Cell e;
            int kx, ky, kz, cx, cy, cz;
            split3((uint32_t)col, k, invk, kx, ky, kz);
            split3(a, na, inva, cx, cy, cz);
            cx = kx + k * cx; cy = ky + k * cy; cz = kz + k * cz;
            e.id = (uint32_t)(cx + nc * (cy + nc * cz));
            e.beg = uniform(C.cellb[e.id]);
            e.cnt = uniform(C.cellb[e.id + 1]) - e.beg;
            e.bx0 = hx + ((double)cx + 0.5) * C.w;
            e.by0 = hy + ((double)cy + 0.5) * C.w;
            e.bz0 = hz + ((double)cz + 0.5) * C.w;
            if (wave == 0) cell_waits(C, deps, col, cx, cy, cz, kx, ky, kz, e.dep0, e.dep1);
            if (wave == 1) load_records(C, props, e.beg, e.cnt, 0u, e.bx0, e.by0, e.bz0, W.tr);
            e.sg = stencil_segments(C, rows, cx, cy, cz, W.seglo, W.segoff);
            e.place = stencil_place(e.sg, 64u * (uint32_t)wave, e.beg);
            return e;
        };
        if constexpr (kCellWaves) {
            // a cell per wave, each wave at its own pace (see CellDeps); colour by
            // colour where the cell lists, and with them the words that say which
            // cells are done, have their place taken (kMemCrew)
            const uint32_t workers = nblk * cell_waves;
            const uint32_t first = (uint32_t)wave < cell_waves ? bid + nblk * (uint32_t)wave : nact;
            bool ok = true;
            for (int col = 0; col < ncol && ok; ++col) {
                int kx, ky, kz;
                split3((uint32_t)col, k, invk, kx, ky, kz);
                for (uint32_t a = first; a < nact; a += workers) {
                    int cx, cy, cz;
                    split3(a, na, inva, cx, cy, cz);
                    cx = kx + k * cx; cy = ky + k * cy; cz = kz + k * cz;
                    const uint32_t cell = (uint32_t)(cx + nc * (cy + nc * cz));
                    const uint32_t cbeg = uniform(C.cellb[cell]), ccnt = uniform(C.cellb[cell + 1]) - cbeg;
                    wc.e = 0.0;
                    if (ccnt) {
                        const double bx0 = hx + ((double)cx + 0.5) * C.w;
                        const double by0 = hy + ((double)cy + 0.5) * C.w;
                        const double bz0 = hz + ((double)cz + 0.5) * C.w;
                        const Segments sg = stencil_segments(C, rows, cx, cy, cz, W.seglo, W.segoff);
                        if constexpr (kMem == kMemTeam) {
                            uint32_t dep0, dep1;
                            cell_waits(C, deps, col, cx, cy, cz, kx, ky, kz, dep0, dep1);
                            ok = wave_cells_done(done, dep0, dep1, (uint32_t)it + 1u, B.polls, &st->fault);
                            if (!ok) break;
                        }
                        bool overflow;
                        const uint32_t ns = gather_wave(C, P, sg, bx0, by0, bz0, cbeg, ccnt, recs, W, S, overflow);
                        const auto nr = near_regs<near_held<Real, kMem>()>(P, W.near, ns, overflow);
                        wc.overflows += overflow ? 1u : 0u;
                        if (overflow)
                            cell_trials(C, RecView<Real>{C.rec, C.misc + 1}, props, sweep, P, cbeg, ccnt, bx0, by0, bz0,
                                        nr, overflow, sg, W, wc);
                        else
                            cell_trials(C, V, props, sweep, P, cbeg, ccnt, bx0, by0, bz0, nr, overflow, sg, W, wc,
                                        S.own);
                    }
                    if (lane == 0) agent_store(&C.ecell[cell], wc.e);
                    if constexpr (kMem == kMemTeam) {
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // its moves are out before it is done
                        if (lane == 0) agent_store(&done[cell], (uint32_t)it + 1u);
                    }
                }
                if constexpr (kMem == kMemCrew)
                    if (!sys_sync<kFenced>(B, &st->fault, bflag)) return;
            }
            ++sweep;
            if constexpr (kMem == kMemTeam) {
                if (!ok && lane == 0) *bflag = 2u;
                sys_arrive<kFenced>(B);
                const bool all = *bflag != 2u;
                __syncthreads();  // (the wait writes the flag)
                if (!sys_wait<kFenced>(B, &st->fault, bflag) || !all) return;
            }
        } else {
        Cell e{};
        if (bid < nact) e = take_cell(0, bid);
        for (int col = 0; col < ncol; ++col) {
            for (uint32_t a = bid; a < nact; a += nblk) {
                wc.e = 0.0;
                if (e.cnt) {
                    if (kMem == kMemTeam && nblk > 1 && col > 0 &&
                        !cells_done(done, e.dep0, e.dep1, (uint32_t)it + 1u, B.polls, &st->fault, bflag))
                        return;
                    bool overflow;
                    const uint32_t ns = gather_team(C, P, e.sg, e.bx0, e.by0, e.bz0, e.beg, e.cnt, e.place, recs, wave, W, S,
                                                    overflow);
                    const auto nr = near_regs<near_held<Real, kMem>()>(P, W.near, ns, overflow);
                    if (wave == 0) wc.overflows += overflow ? 1u : 0u;
                    if (overflow)  // not staged: straight from the system's arrays
                        team_trials<false>(C, RecView<Real>{C.rec, C.misc + 1}, props, sweep, P, e.beg, e.cnt, e.bx0,
                                           e.by0, e.bz0, nr, overflow, e.sg, wave, nullptr, W, sums, wc);
                    else
                        team_trials<true>(C, V, props, sweep, P, e.beg, e.cnt, e.bx0, e.by0, e.bz0, nr, overflow, e.sg,
                                          wave, S.own, W, sums, wc);
                }
                if (tid == 0) agent_store(&C.ecell[e.id], wc.e);
                if (kMem == kMemTeam) {  // its moves are out before it is done
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    __syncthreads();
                    if (tid == 0) agent_store(&done[e.id], (uint32_t)it + 1u);
                }
                if (a + nblk < nact) e = take_cell(col, a + nblk);
            }
            if (kMem == kMemCrew || col == ncol - 1) sys_arrive<kFenced>(B);
            if (col == ncol - 1) ++sweep;
            else if (bid < nact) e = take_cell(col + 1, bid);
            if (kMem == kMemCrew || col == ncol - 1)
                if (!sys_wait<kFenced>(B, &st->fault, bflag)) return;
        }
        }
        // E_acc += the sweep's dE (sweep_energy); E/M samples (the next
        // sweep's steps touch neither)
        if (bid == 0 && wave == 0) {
            e_acc += sweep_energy([&](uint32_t c) { return agent_load(&C.ecell[c]); }, C.ncell);
        }
        if (bid == 0 && tid == 0) {
            const uint64_t t = sweep - origin;
            if (t >= C.obs_start && C.obs_interval && t % C.obs_interval == 0) {
                const double em = e_acc / (double)M;
                if (st->n_e < C.max_samples) C.e_samples[st->n_e] = em;
                st->n_e += 1;
                st->e_sum += em;
                st->e_sumsq += em * em;
            }
        }
    }

    // centres and types from the records
    for (uint32_t m = m0 + tid; m < m1; m += kThr) {
#pragma unroll
        for (int a = 0; a < 3; ++a) C.com[a * M + m] = agent_load(&C.rec[m].c[a]);
        C.types[m] = agent_load(&C.rec[m].types);
    }
    const unsigned long long terms = wave_sum_ull(wc.terms), tests = wave_sum_ull(wc.tests);
    if (lane == 0) {
        const uint64_t att[3] = {wc.att0, wc.att1, wc.att2}, acc[3] = {wc.acc0, wc.acc1, wc.acc2};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (att[i]) atomicAdd((unsigned long long*)&st->attempts[i], (unsigned long long)att[i]);
            if (acc[i]) atomicAdd((unsigned long long*)&st->accepts[i], (unsigned long long)acc[i]);
        }
        if (wc.exits) atomicAdd((unsigned long long*)&st->exits, (unsigned long long)wc.exits);
        if (terms) atomicAdd((unsigned long long*)&st->pair_terms, terms);
        if (tests) atomicAdd((unsigned long long*)&st->pair_tests, tests);
        if (wc.overflows)
            atomicAdd((unsigned long long*)&st->near_overflows, (unsigned long long)wc.overflows);
    }
    if (bid == 0 && tid == 0) {
        st->sweep = sweep;
        st->e_acc = e_acc;
    }
}

// The event work over all pairs on many workgroups: the waves of a system's
// workgroups take its units in turn, the energies go to g_part for k_events to
// sum, the g(r) counts into the histograms.
__global__ void __launch_bounds__(kThreads) k_event_parts(PartList list)
{
    // this workgroup's system: the last slot whose first workgroup is at or
    // below it (the slots are in ascending first)
    uint32_t lo = 0, hi = list.n;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (list.s[mid].first <= blockIdx.x) lo = mid; else hi = mid;
    }
    const PartSlot one = list.s[lo];
    const uint32_t bid = blockIdx.x - one.first;
    __shared__ double red[kWaves];
    __shared__ double misc[16];
    __shared__ uint32_t bins[2 * kGofrBins];
    __shared__ uint32_t gqueue[kWaves * kGofrQueue];
    __shared__ float windows[kWaves * 3u * (kEventSpan + 64u)];
    Ctx<double, kMemAny> C;
    load_ctx(C, one.sys);
    C.com = C.gcom;
    C.red = red;
    C.misc = misc;
    C.bins = bins;
    C.ecell = nullptr;
    C.off = nullptr;
    C.site = nullptr;
    C.cellb = one.sys->g_cell;
    C.cellid = one.sys->g_cellid;
    C.list = one.sys->g_list;
    if (threadIdx.x == 0) {
        misc[1] = C.sig0;
        misc[2] = C.sig1;
        misc[3] = C.sig2;
    }
    __syncthreads();
    const uint32_t f = one.flags;
    const EventUnits U = event_units(C.M);
    const uint32_t wave = bid * kWaves + (uint32_t)wave_index(), nwaves = one.count * kWaves;
    uint32_t* queue = gqueue + wave_index() * kGofrQueue;
    float* window = windows + wave_index() * 3u * (kEventSpan + 64u);
    if (f & (kFlagResumSet | kFlagResumReport | kFlagResumPeriodic)) {
        const int span = one.span;
        if (span) resum_units_cells(C, wave, nwaves, span, queue);
        else resum_units<kEventSpan>(C, U, wave, nwaves, queue, window);
    }
    if (f & kFlagGofr) gofr_frame(C, U, wave, nwaves, true, queue, window);
}

__global__ void k_init_lattice(SysDev* Dp, uint32_t n)
{
    const SysDev& D = *Dp;
    const uint32_t m = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t M = D.M;
    if (m >= M) return;
    const double a = D.L / (double)n;
    const uint32_t i = m % n, j = (m / n) % n, l = m / (n * n);
    D.com[m] = ((double)i + 0.5) * a;
    D.com[M + m] = ((double)j + 0.5) * a;
    D.com[2 * M + m] = ((double)l + 0.5) * a;
    const U4 g = philox10(m, 0xFFFFFFFFu, 0xFFFFFFFFu, 2u, D.seed_lo, D.seed_hi);
    const double u1 = unit_open(g.x), u2 = unit_open(g.y), u3 = unit_open(g.z);
    const double r1 = sqrt(1.0 - u1), r2 = sqrt(u1);
    D.quat[m] = r2 * cos(kTwoPi * u3);
    D.quat[M + m] = r1 * sin(kTwoPi * u2);
    D.quat[2 * M + m] = r1 * cos(kTwoPi * u2);
    D.quat[3 * M + m] = r2 * sin(kTwoPi * u3);
    D.types[m] = 0u | (1u << 8) | (2u << 16);
}

template <typename Real, bool kRes, bool kInl>
hipError_t launch_one(const Slot* dev_slots, const Slot& one, uint32_t n_blocks, size_t lds,
                      hipStream_t stream)
{
    static size_t configured = 0;
    if (lds > configured) {
        hipError_t e = hipFuncSetAttribute((const void*)&k_sweeps<Real, kRes, kInl>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured = lds;
    }
    hipLaunchKernelGGL((k_sweeps<Real, kRes, kInl>), dim3(n_blocks), dim3(kThreads), lds, stream,
                       dev_slots, one);
    return hipGetLastError();
}

template <typename Real, bool kInl>
hipError_t launch_res(bool resident, const Slot* dev_slots, const Slot& one, uint32_t n_blocks,
                      size_t lds, hipStream_t stream)
{
    return resident ? launch_one<Real, true, kInl>(dev_slots, one, n_blocks, lds, stream)
                    : launch_one<Real, false, kInl>(dev_slots, one, n_blocks, lds, stream);
}

}  // namespace

hipError_t launch_sweeps(bool fp64, bool resident, const Slot* dev_slots, const Slot& one, 
                         uint32_t n_blocks, size_t lds_bytes, hipStream_t stream, bool inline_events)
{
    if (fp64)
        return inline_events
                   ? launch_res<double, true>(resident, dev_slots, one, n_blocks, lds_bytes, stream)
                   : launch_res<double, false>(resident, dev_slots, one, n_blocks, lds_bytes, stream);
    return inline_events
               ? launch_res<float, true>(resident, dev_slots, one, n_blocks, lds_bytes, stream)
               : launch_res<float, false>(resident, dev_slots, one, n_blocks, lds_bytes, stream);
}

hipError_t launch_events(const Slot* dev_slots, const Slot& one, uint32_t n_blocks,
                         hipStream_t stream)
{
    static const hipError_t attr = hipFuncSetAttribute(
        (const void*)&k_events, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kEventStageBytes);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(k_events, dim3(n_blocks), dim3(kThreads), kEventStageBytes, stream,
                       dev_slots, one);
    return hipGetLastError();
}

namespace {

template <typename Real, int kMem, bool kCellWaves>
hipError_t launch_spread_t(const SpreadSlot* dev_slots, uint32_t n_slots, const SpreadSlot& one,
                           uint32_t n_blocks, size_t lds, hipStream_t stream)
{
    constexpr int kThr = kCellWaves ? cell_threads(sizeof(Real) == 8, kMem == kMemTeam) : kThreads;
    static size_t configured = 0;
    if (lds > configured) {
        const hipError_t e = hipFuncSetAttribute((const void*)&k_spread<Real, kMem, kCellWaves, kThr>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured = lds;
    }
    hipLaunchKernelGGL((k_spread<Real, kMem, kCellWaves, kThr>), dim3(n_blocks), dim3(kThr), lds, stream, dev_slots,
                       n_slots, one);
    return hipGetLastError();
}

template <typename Real>
hipError_t launch_spread_m(SpreadMode mode, const SpreadSlot* dev_slots, uint32_t n_slots, const SpreadSlot& one,
                           uint32_t n_blocks, size_t lds, hipStream_t stream)
{
    switch (mode) {
    case kSpreadWaves: return launch_spread_t<Real, kMemTeam, true>(dev_slots, n_slots, one, n_blocks, lds, stream);
    case kSpreadCrewWaves: return launch_spread_t<Real, kMemCrew, true>(dev_slots, n_slots, one, n_blocks, lds, stream);
    case kSpreadTeam: return launch_spread_t<Real, kMemTeam, false>(dev_slots, n_slots, one, n_blocks, lds, stream);
    default: return launch_spread_t<Real, kMemCrew, false>(dev_slots, n_slots, one, n_blocks, lds, stream);
    }
}

__global__ void k_zero_barriers(const SpreadSlot* __restrict__ slots, uint32_t n)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        for (int w = 0; w < kBarWords; ++w) slots[i].sys->g_bar[w] = 0u;
}

}  // namespace

hipError_t spread_max_blocks(uint32_t* n_blocks)
{
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) *n_blocks = (uint32_t)cus;
    return e;
}

hipError_t launch_spread(bool fp64, SpreadMode mode, const SpreadSlot* dev_slots, uint32_t n_slots,
                         const SpreadSlot& one, uint32_t n_blocks, size_t lds, hipStream_t stream)
{
    return fp64 ? launch_spread_m<double>(mode, dev_slots, n_slots, one, n_blocks, lds, stream)
                : launch_spread_m<float>(mode, dev_slots, n_slots, one, n_blocks, lds, stream);
}

hipError_t launch_zero_barriers(const SpreadSlot* dev_slots, uint32_t n_slots, hipStream_t stream)
{
    hipLaunchKernelGGL(k_zero_barriers, dim3((n_slots + 63) / 64), dim3(64), 0, stream, dev_slots, n_slots);
    return hipGetLastError();
}

hipError_t launch_event_parts(const PartList& list, uint32_t n_blocks, hipStream_t stream)
{
    hipLaunchKernelGGL(k_event_parts, dim3(n_blocks), dim3(kThreads), 0, stream, list);
    return hipGetLastError();
}

hipError_t launch_init_lattice(SysDev* dev_sys, uint32_t M, hipStream_t stream)
{
    uint32_t n = 1;
    while ((n + 1) * (n + 1) * (n + 1) <= M) ++n;
    hipLaunchKernelGGL(k_init_lattice, dim3((M + 255) / 256), dim3(256), 0, stream, dev_sys, n);
    return hipGetLastError();
}

}  // namespace flipmc
