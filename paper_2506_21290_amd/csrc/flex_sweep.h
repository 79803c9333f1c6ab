// flex_sweep.h -- the sweep kernel of the flexible-molecule engine (the
// paper's own model, Sec. II.A: atoms joined by FENE bonds, Eq. 2, with the
// WCA potential of Eq. 1 between every pair of atoms, intramolecular pairs
// included; and the squares and tetrahedra of Sec. VII), with the descriptor
// it reads.  Included by flex.hip, which holds the event kernels and the host
// code.
//
// A sweep attempts every atom once (a Monte Carlo timestep of N attempts,
// Sec. II.B): with probability p_flip a flip of the atom's molecule -- a
// permutation of the types of its atoms at fixed positions, one of the 180
// degree rotations of the ideal body -- otherwise a translation of the atom,
// uniform in [-d, d)^3 and confined to its cell.
//
// Execution: one workgroup of 8 wave64s per system (several systems per
// launch, a workgroup each), the positions, types and cell lists in LDS when
// they fit.  Per sweep a random shift of a cubic cell grid over the atoms, a
// counting sort into cells (ascending atom index inside each cell), the
// proposals and the neighbours of every atom, then the k^3 colours in order;
// the waves take the cells of a colour, and a wave runs its cell's attempts in
// order, several of them evaluated side by side, a row of 16 lanes per changed
// atom.
// Same-colour cells are at least (k - 1) w >= 2 D + r_c apart (D the largest
// distance two atoms of one molecule can reach, r_c the largest cut-off), so
// no two attempts of a colour touch the same pair term.  A DPP reduction in
// FP64 over each row gives dE in a fixed order.  A bond stretched to 1.5
// sigma_ij or beyond makes dE infinite: the move is rejected.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "engine.h"
#include "flipmc.h"
#include "wave.h"

namespace flipmc {
namespace {
constexpr int kFxThreads = 512;
constexpr int kFxWaves = kFxThreads / 64;
// Neighbour lists: kFxNbr entries per atom, three for each lane of a row of
// 16.  The first kFxPartners are the other atoms of its own molecule, the rest
// atoms of other molecules.  The entries have 16 bits in systems that fit LDS
// (the marks sign-extended), 32 bits in the others.
constexpr uint32_t kFxNbr = 48, kFxPartners = 3;
constexpr int kFxSlots = 6;  // atoms of the 27 cells per lane of a list build
template <bool kRes>
using FxNbr = std::conditional_t<kRes, int16_t, uint32_t>;
constexpr uint32_t kFxBuild = 8;  // atoms whose lists are put together at a time
constexpr uint32_t kFxNone = 0xFFFFFFFFu;  // no neighbour
constexpr uint32_t kFxOver = 0xFFFFFFFEu;  // entry kFxPartners of a list that did not fit
constexpr uint32_t kFxRows = 8;  // rows of one evaluation: two per 16 lanes
// static LDS of the sweep kernel: pair tables, the waves' row tasks and sums,
// scan scratch and the energy accumulator (with room to spare)
constexpr size_t kFxStaticLds = 2 * 16 * 8 + (size_t)kFxWaves * (kFxRows * (40 + 8 + 8 + 4) + kFxBuild * 64 * 2) + 512;
constexpr uint32_t kFxParts = 1024;  // workgroups of the event kernel
constexpr uint32_t kFxMany = 256;    // systems of one sweep launch (a workgroup each)

// An atom as the sweep kernel holds it: position, type, cell of the sweep.
struct alignas(16) FxAtom {
    double x, y, z;
    uint32_t type, cell;
};
static_assert(sizeof(FxAtom) == 32, "two 16-byte words");

// The proposal of an attempt (Sec. II.B).
struct alignas(8) FxProp {
    double thr;         // T ln u
    double tx, ty, tz;  // translation target before the wrap
    uint32_t kind;      // flip: rotation index; translation: kFxMove
    uint32_t cross;     // translation: bits 2 a, 2 a + 1 = periodic image crossed along axis a plus 1; kFxExit
};
constexpr uint32_t kFxMove = 255, kFxExit = 64;

// Everything a workgroup needs about one system; in the system's buffer.
struct FxDev {
    uint32_t geometry, n, M, N;
    uint32_t k, nc, ncell, nflip;
    uint32_t seed_lo, seed_hi, pad2, pad3;
    uint32_t bonded;  // bit 4 i + j: atoms i, j of a molecule are bonded
    uint32_t resum_interval, obs_interval, gofr_interval, obs_start, max_samples, gofr_nbins;
    float wide_r2;  // FxK::list_r2 of cells wider than 500
    double L, invL, w, T, p_flip, dmax, rc2f;
    double sigma[4];
    double gofr_dr, gofr_rmax, fs_q, fs_q_cm;
    // a colour's cells run side by side when sep = (k - 1) w >= 2 D + dyn_base
    // (dyn_base = r_c + 4 sqrt(3) d), D the largest atom distance inside a
    // molecule with an atom in those cells at the colour's start; always
    // when `together` is 1 (the gap covers the worst case), never when it is
    // 2 (forced one cell at a time)
    double sep, dyn_base;
    uint32_t together, pad4;
    uint8_t flips[4][4];  // new type of atom s = old type of atom flips[q][s]
    double* pos;          // SoA [3][N], wrapped into [0, L)
    uint8_t* type;        // [N]
    int32_t* img;         // SoA [3][N] periodic images crossed by accepted translations
    Stats* stats;
    double* e_samples;
    double* drift_samples;
    uint64_t* gofr_all;
    uint64_t* gofr_inter;
    double* c2;
    uint64_t* c2_sweep;
    double* fs;
    double* fs_cm;
    double* mom;          // [4][kC2Max] per-particle moments at the C_2 samples
    double* u0;           // [3][M] orientation at the observable origin
    uint8_t* kref;        // [M] atom the orientation follows
    double* r0;           // [3][N] unwrapped atoms at the origin
    double* rcm0;         // [3][M] unwrapped centres at the origin
    uint32_t* cell_start; // [ncell + 1]
    uint32_t* cell_list;  // [N] atoms sorted by cell, ascending inside a cell
    double* ecell;        // [ncell] accepted dE of each cell in the current sweep
    double* part;         // [kFxParts] partial energies of the event kernel
    FxAtom* atom;         // [N] the sweep kernel's copy of the state, or null (in LDS)
    FxProp* props;        // [N] proposals of the current sweep, in cell-list order
    void* nbr;            // [N][kFxNbr] neighbours of each atom in the current sweep
    MoveRecord* log;
    uint64_t log_sweep0, log_sweeps;
};

// The systems of one sweep launch, passed by value (2 KiB of kernel
// arguments): workgroup b runs d[b].
struct FxList {
    FxDev* d[kFxMany];
};

// The constants of the sweep kernel, copied from the system's descriptor into
// registers at the start of a launch (read through the descriptor, every
// store to LDS or memory could alias them and force a reload).
struct FxK {
    uint32_t n, N, nc, nflip, bonded, seed_lo, seed_hi, together;
    uint32_t flipw[4];  // byte s of word q: flips[q][s]
    uint32_t chgw;      // bits 4 q + s: flip q changes the type of atom s
    double L, invL, w, invw, T, p_flip, dmax, rc2f, sep, dyn_base;
    Global<int32_t>* img;
    Global<FxProp>* props;
    Global<void>* nbr;  // FxNbr [N][kFxNbr]
    float list_r2;  // neighbour lists: squared radius, (r_c + 2 sqrt(3) d)^2 with a margin
};

__device__ __forceinline__ FxK fx_const(const FxDev& D)
{
    FxK K;
    K.n = D.n; K.N = D.N; K.nc = D.nc; K.nflip = D.nflip; K.bonded = D.bonded;
    K.seed_lo = D.seed_lo; K.seed_hi = D.seed_hi;
    K.chgw = 0;
    for (int q = 0; q < 4; ++q) {
        K.flipw[q] = (uint32_t)D.flips[q][0] | ((uint32_t)D.flips[q][1] << 8) | ((uint32_t)D.flips[q][2] << 16) |
                     ((uint32_t)D.flips[q][3] << 24);
        for (uint32_t t = 0; t < 4; ++t) K.chgw |= (t < D.n && D.flips[q][t] != t ? 1u : 0u) << (4 * q + t);
    }
    K.L = D.L; K.invL = D.invL; K.w = D.w; K.invw = 1.0 / D.w;
    K.T = D.T; K.p_flip = D.p_flip; K.dmax = D.dmax; K.rc2f = D.rc2f;
    K.sep = D.sep; K.dyn_base = D.dyn_base; K.together = D.together;
    K.img = (Global<int32_t>*)D.img; K.props = (Global<FxProp>*)D.props; K.nbr = (Global<void>*)D.nbr;
    // the FP32 distances of the list build are within 1.2e-6 w of the FP64 ones:
    // coordinates up to 1.5 w from the cell's centre, rounded to 2^-24 of that,
    // their difference and its nearest image to 2^-24 of 3 w, along three axes;
    // cells wider than 500 have a margin of their own (FxDev::wide_r2, which for
    // all cells, as a scalar, makes the sweep 1 % slower)
    const double smax = fmax(fmax(D.sigma[0], D.sigma[1]), fmax(D.sigma[2], D.n > 3u ? D.sigma[3] : 0.0));
    const float r = (float)(sqrt(D.rc2f) * smax + 2.0 * 1.7320508075688772 * D.dmax) + 1e-3f;
    K.list_r2 = D.w > 500.0 ? D.wide_r2 : r * r;
    return K;
}

// Molecule of atom j.
__device__ __forceinline__ uint32_t fx_mol(uint32_t n, uint32_t j)
{
    return n == 3u ? __umulhi(j, 0x55555556u) : j >> 2;  // N <= 2^24
}

__device__ __forceinline__ double fx_mi(double d, double L, double invL) { return d - L * rint(d * invL); }
// the same with one rounding fewer (the events keep the plain form, whose
// bits the g(r) bins are defined by)
__device__ __forceinline__ double fx_mif(double d, double L, double invL) { return fma(-L, rint(d * invL), d); }

// floor(x / y), iy = 1 / y: the product is within an ulp or two of the
// quotient (below 1e3 here), so the floors agree unless it lies next to a
// whole number; only then the division is taken.
__device__ __forceinline__ double fx_floor_div(double x, double y, double iy)
{
    const double q = x * iy;
    double f = floor(q);
    if (fabs(q - rint(q)) < 1e-9) f = floor(x / y);
    return f;
}

__device__ __forceinline__ double fx_wrap(double x, double L) { return x - L * floor(x / L); }

__device__ __forceinline__ int fx_axis(double x, double h, const FxK& D)
{
    const double d = x - h;
    const double g = d - D.L * fx_floor_div(d, D.L, D.invL);
    int c = (int)fx_floor_div(g, D.w, D.invw);
    c = c < 0 ? 0 : c;
    return c >= (int)D.nc ? (int)D.nc - 1 : c;
}

__device__ __forceinline__ uint32_t fx_cell(double x, double y, double z, const double h[3], const FxK& D)
{
    const uint32_t nc = D.nc;
    return (uint32_t)fx_axis(x, h[0], D) +
           nc * ((uint32_t)fx_axis(y, h[1], D) + nc * (uint32_t)fx_axis(z, h[2], D));
}

// Eq. (1) as (2 (s/r)^6 - 1)^2 below the cut-off, FP64.  1 / r^2 is the
// hardware estimate refined by two Newton steps (within an ulp or two of the
// quotient; r^2 is a normal number for every pair inside the cut-off).
__device__ __forceinline__ double fx_wca(double s2, double r2, double rc2f)
{
    if (!(r2 < rc2f * s2)) return 0.0;
    double y = __builtin_amdgcn_rcp(r2);
    y = fma(fma(-r2, y, 1.0), y, y);
    y = fma(fma(-r2, y, 1.0), y, y);
    const double x = s2 * y;
    const double t = fma(2.0, x * x * x, -1.0);
    return t * t;
}

// Eq. (2), infinite at or beyond 1.5 sigma_ij.
__device__ __forceinline__ double fx_fene(double sig, double r2)
{
    const double lim2 = 2.25 * sig * sig;
    if (!(r2 < lim2)) return __builtin_inf();
    return -33.75 * log(1.0 - r2 / lim2);
}

// This lane's share of the counters, and the accepted dE of the wave's
// current cell in attempt order (wave-uniform, as the accepted counts).
struct FxCount {
    uint32_t att_t, att_f, acc_t, acc_f, exits;
    uint64_t terms;
    double e;
};

// A row of an evaluation: one changed atom of an attempt.
struct alignas(8) FxRow {
    double tx, ty, tz;  // target of a translation
    uint32_t atom, base, kind, pad;
};

// LDS of one wave: the rows of an evaluation and what they sum; of the workgroup: the pair diameters sigma_ij and
// their squares by 4 t_i + t_j.
struct FxWaveLds {
    FxRow* row;      // [kFxRows]
    double* sum;     // [kFxRows] dE
    double* scale;   // [kFxRows] u_new + u_old (logged sweeps)
    uint32_t* terms; // [kFxRows] pairs inside the cut-off
    void* list;      // FxNbr [kFxBuild][64] lists being built
    const double* sij;
    const double* s2ij;
};

// Where the sweep kernel keeps the state and the cell lists: the workgroup's
// LDS for systems that fit there, the system's buffer otherwise.
template <bool kRes>
struct FxView {
    template <typename T>
    using Ptr = std::conditional_t<kRes, Lds<T>, Global<T>>*;
    Ptr<FxAtom> atom;         // [N]
    Ptr<uint32_t> cell_start; // [ncell + 1]
    Ptr<uint32_t> cell_list;  // [N]
    Ptr<double> ecell;        // [ncell]
    __device__ __forceinline__ FxAtom at(uint32_t i) const
    {
        const auto* p = atom + i;
        return FxAtom{p->x, p->y, p->z, p->type, p->cell};
    }
};

struct FxLds {
    size_t atom, cstart, clist, ecell, total;
};

__host__ __device__ inline FxLds fx_lds_layout(uint32_t N, uint32_t ncell)
{
    FxLds l{};
    size_t o = 0;
    auto a16 = [](size_t x) { return (x + 15) & ~size_t(15); };
    l.atom = o;   o = a16(o + size_t(N) * sizeof(FxAtom));
    l.ecell = o;  o = a16(o + size_t(ncell) * sizeof(double));
    l.cstart = o; o = a16(o + (size_t(ncell) + 1) * sizeof(uint32_t));
    l.clist = o;  o = a16(o + size_t(N) * sizeof(uint32_t));
    l.total = o;
    return l;
}

// The 27 cells around cell (cx, cy, cz) (every cell once where they span an
// axis) as row segments along x of one or two contiguous cell ranges: lane s
// gets segment s's first place in the cell list (*lo) and the atoms before it
// in the stencil (*off).  Returns the number of segments; *total = atoms.
template <bool kRes>
__device__ __forceinline__ int fx_segments(const FxK& D, const FxView<kRes>& V, int cx, int cy, int cz, uint32_t* lo,
                                           uint32_t* off, uint32_t* total)
{
    const int lane = __lane_id();
    const int nc = (int)D.nc;
    const bool full = 3 >= nc;
    const int nrow = full ? nc : 3;
    int xa0, xb0, xa1 = 0, xb1 = -1;
    if (full) {
        xa0 = 0; xb0 = nc - 1;
    } else if (cx < 1) {
        xa0 = cx - 1 + nc; xb0 = nc - 1; xa1 = 0; xb1 = cx + 1;
    } else if (cx + 1 >= nc) {
        xa0 = cx - 1; xb0 = nc - 1; xa1 = 0; xb1 = cx + 1 - nc;
    } else {
        xa0 = cx - 1; xb0 = cx + 1;
    }
    const int nxr = xb1 >= xa1 ? 2 : 1;
    const int nseg = nrow * nrow * nxr;
    uint32_t cnt = 0;
    *lo = 0;
    if (lane < nseg) {
        const int r = nxr == 2 ? lane >> 1 : lane, ixr = nxr == 2 ? lane & 1 : 0;
        const int iz = nrow == 3 ? r / 3 : r >> 1, iy = r - nrow * iz;  // nrow is 2 or 3
        int y = full ? iy : cy - 1 + iy, z = full ? iz : cz - 1 + iz;
        y += y < 0 ? nc : (y >= nc ? -nc : 0);
        z += z < 0 ? nc : (z >= nc ? -nc : 0);
        const int xa = ixr ? xa1 : xa0, xb = ixr ? xb1 : xb0;
        const uint32_t row = (uint32_t)(nc * (y + nc * z));
        *lo = V.cell_start[row + xa];
        cnt = V.cell_start[row + xb + 1] - *lo;
    }
    *off = wave_excl_scan(cnt, total);
    return nseg;
}

template <typename T>
__device__ __forceinline__ T fx_pick(const T v[4], uint32_t i)
{
    return i == 0 ? v[0] : (i == 1 ? v[1] : (i == 2 ? v[2] : v[3]));
}

// The proposals of every atom's attempt in this sweep, at the atom's place in
// the cell list: move kind, flip rotation or translation target, the cell-exit
// test and T ln u (an atom's position changes only in its own attempt, so the
// draws do not depend on the attempts before it).  A thread per atom, before
// the first colour: drawn by the cell's wave, they were a tenth of its chain.
template <bool kRes>
__device__ __forceinline__ void fx_propose_all(const FxDev& Dv, const FxK& D, const FxView<kRes>& V, uint64_t sweep,
                                               const double h[3], bool logging, FxCount& wc)
{
    const uint32_t slo = (uint32_t)sweep, shi = (uint32_t)(sweep >> 32);
    for (uint32_t p = threadIdx.x; p < D.N; p += kFxThreads) {
        const uint32_t a = V.cell_list[p];
        const FxAtom at = V.at(a);
        const U4 b0 = philox10(a, slo, shi, 0u, D.seed_lo, D.seed_hi);
        const U4 b1 = philox10(a, slo, shi, 1u, D.seed_lo, D.seed_hi);
        const double uacc = unit_53(b0.x, b0.y), ut = unit_open(b0.z);
        const double p0 = unit_open(b1.x), p1 = unit_open(b1.y), p2 = unit_open(b1.z);
        FxProp pr;
        pr.thr = D.T * log(uacc);
        pr.kind = kFxMove;
        pr.cross = 0;
        pr.tx = pr.ty = pr.tz = 0.0;
        if (ut < D.p_flip) {
            const uint32_t q = (uint32_t)((double)D.nflip * p0);
            pr.kind = q >= D.nflip ? D.nflip - 1 : q;
            wc.att_f += 1;
        } else {
            pr.tx = at.x + D.dmax * (2.0 * p0 - 1.0);
            pr.ty = at.y + D.dmax * (2.0 * p1 - 1.0);
            pr.tz = at.z + D.dmax * (2.0 * p2 - 1.0);
            // d < L / 4: at most one image
            const double fx = fx_floor_div(pr.tx, D.L, D.invL), fy = fx_floor_div(pr.ty, D.L, D.invL),
                         fz = fx_floor_div(pr.tz, D.L, D.invL);
            pr.cross = (uint32_t)((int)fx + 1) | (uint32_t)((int)fy + 1) << 2 | (uint32_t)((int)fz + 1) << 4;
            wc.att_t += 1;
            if (fx_cell(pr.tx - D.L * fx, pr.ty - D.L * fy, pr.tz - D.L * fz, h, D) != at.cell) {
                pr.cross |= kFxExit;
                wc.exits += 1;
                if (logging) {
                    MoveRecord rec;
                    rec.delta_e = 0.0; rec.scale = 0.0; rec.t_log_u = pr.thr; rec.sweep = sweep;
                    rec.molecule = a; rec.move = MC_TRANSLATE; rec.accepted = 0; rec.exited = 1;
                    rec.axis = 255; rec.pair_terms = 0; rec.pad = 0;
                    Dv.log[(sweep - Dv.log_sweep0) * D.N + a] = rec;
                }
            }
        }
        Global<FxProp>* out = D.props + p;
        out->thr = pr.thr; out->tx = pr.tx; out->ty = pr.ty; out->tz = pr.tz;
        out->kind = pr.kind; out->cross = pr.cross;
    }
}

using W4 = uint32_t __attribute__((ext_vector_type(4)));

// Eq. (1) given whether the pair is inside the cut-off (the reciprocal as in
// fx_wca).
__device__ __forceinline__ double fx_wca_in(double s2, double r2, bool in)
{
    double y = __builtin_amdgcn_rcp(r2);
    y = fma(fma(-r2, y, 1.0), y, y);
    y = fma(fma(-r2, y, 1.0), y, y);
    const double x = s2 * y;
    const double t = fma(2.0, x * x * x, -1.0);
    return in ? t * t : 0.0;
}

// The lists of one cell's atoms (list places q0 .. q0 + cnt, cnt <= 64) from
// the atoms of the 27 cells around it, S of them per lane.  fold: nearest
// image per pair.
template <int S, bool kFold, bool kRes>
__device__ __forceinline__ void fx_cell_lists(const FxK& K, const FxView<kRes>& V, uint32_t q0, uint32_t cnt, double ox,
                                              double oy, double oz, int nseg, uint32_t delta, uint32_t off,
                                              uint32_t total, const FxWaveLds& W)
{
    const uint32_t lane = (uint32_t)__lane_id(), n = K.n;
    const float Lf = (float)K.L, iLf = (float)K.invL;
    uint32_t id[S], mj[S], sg[S];
    uint64_t have[S];  // lanes with an atom
    float x[S], y[S], z[S];
#pragma unroll
    for (int u = 0; u < S; ++u) sg[u] = 0;
    for (int t = 1; t < nseg; ++t) {  // the segment each place lies in
        const uint32_t o = rl_u(off, t);
#pragma unroll
        for (int u = 0; u < S; ++u) sg[u] += 64u * (uint32_t)u + lane >= o ? 1u : 0u;
    }
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const uint32_t idx = 64u * (uint32_t)u + lane;
        have[u] = __builtin_amdgcn_ballot_w64(idx < total);
        const uint32_t d = (uint32_t)__shfl((int)delta, (int)sg[u]);
        id[u] = V.cell_list[idx < total ? idx + d : q0];
    }
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const FxAtom A = V.at(id[u]);
        mj[u] = fx_mol(n, id[u]);
        x[u] = (float)fx_mif(A.x - ox, K.L, K.invL);
        y[u] = (float)fx_mif(A.y - oy, K.L, K.invL);
        z[u] = (float)fx_mif(A.z - oz, K.L, K.invL);
    }
    uint32_t at = 0, mol = 0;  // lane q: the cell's atom q
    float ax = 0.f, ay = 0.f, az = 0.f;
    if (lane < cnt) {
        at = V.cell_list[q0 + lane];
        const FxAtom A = V.at(at);
        mol = fx_mol(n, at);
        ax = (float)fx_mif(A.x - ox, K.L, K.invL);
        ay = (float)fx_mif(A.y - oy, K.L, K.invL);
        az = (float)fx_mif(A.z - oz, K.L, K.invL);
    }
    using T = FxNbr<kRes>;
    T* list = (T*)W.list;
    constexpr uint32_t kWords = kFxNbr * sizeof(T) / 4u, kLdsWords = 64u * sizeof(T) / 4u;  // of a list
    for (uint32_t qb = 0; qb < cnt; qb += kFxBuild) {
        // the lists in LDS: no neighbour, the partners, then the neighbours
        // compacted by ballots (those past the end share the last, spare entry)
#pragma unroll
        for (uint32_t t = 0; t < kFxBuild * kLdsWords; t += 256u)
            ((W4*)W.list)[t / 4u + lane] = W4{~0u, ~0u, ~0u, ~0u};
        wave_lds_sync();
        {
            const int q = (int)((qb + (lane >> 2)) & 63u);
            const uint32_t p = lane & 3u, a = (uint32_t)__shfl((int)at, q), m = (uint32_t)__shfl((int)mol, q);
            if (lane < 4u * kFxBuild && p + 1u < n)
                list[64u * (lane >> 2) + p] = (T)(n * m + p + (p >= a - n * m ? 1u : 0u));
        }
        wave_lds_sync();
        const uint32_t nq = min(kFxBuild, cnt - qb);
#pragma unroll 2
        for (uint32_t i = 0; i < nq; ++i) {
            const int q = (int)(qb + i);
            const float qx = rl_f(ax, q), qy = rl_f(ay, q), qz = rl_f(az, q);
            const uint32_t qm = rl_u(mol, q);
            uint32_t k = kFxPartners;
#pragma unroll
            for (int u = 0; u < S; ++u) {
                float dx = x[u] - qx, dy = y[u] - qy, dz = z[u] - qz;
                if (kFold) {
                    dx = fmaf(-Lf, rintf(dx * iLf), dx);
                    dy = fmaf(-Lf, rintf(dy * iLf), dy);
                    dz = fmaf(-Lf, rintf(dz * iLf), dz);
                }
                const uint64_t bm = __builtin_amdgcn_ballot_w64(fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < K.list_r2) &
                                    __builtin_amdgcn_ballot_w64(mj[u] != qm) & have[u];
                const uint32_t kk = __builtin_amdgcn_mbcnt_hi((uint32_t)(bm >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)bm, k));
                if (__builtin_amdgcn_inverse_ballot_w64(bm)) list[64u * i + min(kk, 63u)] = (T)id[u];
                k += (uint32_t)__popcll(bm);
            }
            if (k > kFxNbr && lane == 0u) list[64u * i + kFxPartners] = (T)kFxOver;
        }
        wave_lds_sync();
        // out, coalesced
#pragma unroll
        for (uint32_t t0 = 0; t0 < kFxBuild * kWords; t0 += 64u) {
            const uint32_t r = (t0 + lane) / kWords, e = t0 + lane - kWords * r;
            const uint32_t a = (uint32_t)__shfl((int)at, (int)((qb + r) & 63u));
            const uint32_t v = ((const uint32_t*)W.list)[kLdsWords * r + e];
            if (r < nq) ((Global<uint32_t>*)K.nbr)[(size_t)a * kWords + e] = v;
        }
        wave_lds_sync();
    }
}

// The neighbours of every atom in the current sweep: the other atoms of its
// molecule, and the atoms of other molecules within r_c + 2 sqrt(3) d of it at
// the sort (each of two atoms moves at most sqrt(3) d in the sweep, so every
// pair that comes within its cut-off is listed).  A wave per cell: the atoms
// of the 27 cells around it up to kFxSlots to a lane (relative to the cell's
// centre, FP32), tested against the cell's atoms one after another; a list
// keeps the order of the cell list.  Built once per sweep by all waves side by
// side, it takes the search (158 atoms of the 27 cells for about 18 within
// reach) out of the serial attempts: an attempt then needs a row of 16 lanes
// instead of the whole wave.  The lists are put together in LDS: stored from
// the lanes that found them, 2 bytes at a time under a branch each, the build
// of 3000 atoms' lists took 0.37 ms instead of 0.25.
template <bool kRes>
__device__ __forceinline__ void fx_build_lists(const FxK& K, const FxView<kRes>& V, const double h[3], int wave,
                                               uint32_t ncell, const FxWaveLds& W)
{
    const uint32_t nc = K.nc;
    const bool fold = nc <= 3u;  // the 27 cells span the box
    for (uint32_t cell = (uint32_t)wave; cell < ncell; cell += kFxWaves) {
        const uint32_t b = uniform(V.cell_start[cell]),
                       e = uniform(V.cell_start[cell + 1]);
        if (b >= e) continue;
        const uint32_t ix = cell % nc, iy = (cell / nc) % nc, iz = cell / (nc * nc);
        const double ox = h[0] + ((double)ix + 0.5) * K.w, oy = h[1] + ((double)iy + 0.5) * K.w,
                     oz = h[2] + ((double)iz + 0.5) * K.w;
        uint32_t lo, off, total;
        const int nseg = fx_segments(K, V, (int)ix, (int)iy, (int)iz, &lo, &off, &total);
        total = uniform(total);
        for (uint32_t q0 = b; q0 < e; q0 += 64u) {
            const uint32_t cnt = min(64u, e - q0);
            if (total > 64u * kFxSlots) {
                // too many for the lanes: the rows of these atoms walk the cells
                const uint32_t lane = (uint32_t)__lane_id();
                if (lane < cnt) {
                    const uint32_t a = V.cell_list[q0 + lane], m = fx_mol(K.n, a), sa = a - K.n * m;
                    for (uint32_t p = 0; p < kFxNbr; ++p) {
                        const uint32_t v = p + 1u < K.n ? K.n * m + p + (p >= sa ? 1u : 0u)
                                                        : (p == kFxPartners ? kFxOver : kFxNone);
                        ((Global<FxNbr<kRes>>*)K.nbr)[(size_t)a * kFxNbr + p] = (FxNbr<kRes>)v;
                    }
                }
            } else if (fold) {
                fx_cell_lists<kFxSlots, true>(K, V, q0, cnt, ox, oy, oz, nseg, lo - off, off, total, W);
            } else if (total <= 192u) {
                fx_cell_lists<3, false>(K, V, q0, cnt, ox, oy, oz, nseg, lo - off, off, total, W);
            } else if (total <= 256u) {
                fx_cell_lists<4, false>(K, V, q0, cnt, ox, oy, oz, nseg, lo - off, off, total, W);
            } else {
                fx_cell_lists<kFxSlots, false>(K, V, q0, cnt, ox, oy, oz, nseg, lo - off, off, total, W);
            }
        }
    }
}

// dE of the rows W.row[0 .. nrow), nrow <= 4 G, against the present state into
// W.sum: row r = 4 g + (lane / 16) is one changed atom of an attempt, a lane
// per listed neighbour and per partner in its molecule (three passes of 16,
// the third rarely filled).  The G evaluations of a lane are independent
// chains side by side.
template <int G, bool kLog, bool kRes>
__device__ __forceinline__ void fx_eval_rows(const FxK& K, const FxView<kRes>& V, uint32_t nrow, bool logging,
                                             const FxWaveLds& W)
{
    const uint32_t lane = (uint32_t)__lane_id(), row = lane >> 4, rl = lane & 15u;
    bool act[G], fl[G];
    uint32_t cl[G], bl[G], kl[G], perm[G], to[G], tn[G], j[G][3];
    double xo[G], yo[G], zo[G], mx[G], my[G], mz[G], de[G], sc[G];
    uint32_t terms[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t r = 4u * (uint32_t)g + row;
        act[g] = r < nrow;
        const FxRow* R = W.row + (act[g] ? r : 0u);
        mx[g] = R->tx; my[g] = R->ty; mz[g] = R->tz;
        cl[g] = R->atom; bl[g] = R->base; kl[g] = R->kind;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const Global<FxNbr<kRes>>* list = (Global<FxNbr<kRes>>*)K.nbr + (size_t)cl[g] * kFxNbr + rl;
#pragma unroll
        for (uint32_t u = 0; u < 3; ++u) j[g][u] = (uint32_t)(int32_t)list[16u * u];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const FxAtom A = V.at(cl[g]);
        xo[g] = A.x; yo[g] = A.y; zo[g] = A.z; to[g] = A.type;
        fl[g] = kl[g] != kFxMove;
        perm[g] = fx_pick(K.flipw, kl[g]);
        const uint32_t tp = V.atom[bl[g] + ((perm[g] >> (8u * (cl[g] - bl[g]))) & 3u)].type;
        tn[g] = fl[g] ? tp : to[g];
        // the displacement of a translation; none for a flip
        mx[g] = fl[g] ? 0.0 : mx[g] - xo[g];
        my[g] = fl[g] ? 0.0 : my[g] - yo[g];
        mz[g] = fl[g] ? 0.0 : mz[g] - zo[g];
        de[g] = 0.0;
        sc[g] = 0.0;
        terms[g] = 0;
        if (!act[g]) j[g][0] = j[g][1] = j[g][2] = kFxNone;
    }
    // the pairs of lane's neighbours (one per g): separations after the move
    // are those before it plus the displacement; partner lanes (bond) hold
    // atoms of the own molecule, whose type a flip may change too
    auto pass = [&](const uint32_t (&jn)[G], const bool (&valid)[G], bool inner) __attribute__((always_inline)) {
        uint32_t tj[G], tm[G];
        double dx[G], dy[G], dz[G], num[G], den[G];
        bool bond[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const FxAtom A = V.at(valid[g] ? jn[g] : cl[g]);
            dx[g] = xo[g] - A.x; dy[g] = yo[g] - A.y; dz[g] = zo[g] - A.z;
            tj[g] = tm[g] = A.type;
            bond[g] = false;
        }
        if (inner) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                bond[g] = valid[g] && jn[g] - bl[g] < K.n;
                const uint32_t sj = bond[g] ? jn[g] - bl[g] : 0u;
                const uint32_t tp = V.atom[bl[g] + ((perm[g] >> (8u * sj)) & 3u)].type;
                if (bond[g] && fl[g]) tm[g] = tp;
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            bool ok = valid[g];
            if (inner) {
                // a pair of two changed atoms counts in the row of the lower
                const uint32_t sj = jn[g] - bl[g];
                ok = ok && !(bond[g] && fl[g] && jn[g] < cl[g] && ((K.chgw >> (4u * (kl[g] & 3u) + (sj & 3u))) & 1u));
            }
            const double s2o = W.s2ij[4u * to[g] + tj[g]], s2n = W.s2ij[4u * tn[g] + tm[g]];
            const double ux = fx_mif(dx[g], K.L, K.invL), uy = fx_mif(dy[g], K.L, K.invL),
                         uz = fx_mif(dz[g], K.L, K.invL);
            const double vx = ux + mx[g], vy = uy + my[g], vz = uz + mz[g];
            const double r2o = fma(ux, ux, fma(uy, uy, uz * uz));
            const double r2n = fma(vx, vx, fma(vy, vy, vz * vz));
            const bool io = ok && r2o < K.rc2f * s2o, in = ok && r2n < K.rc2f * s2n;
            const double uo = fx_wca_in(s2o, r2o, io), un = fx_wca_in(s2n, r2n, in);
            de[g] += un - uo;
            if (kLog) sc[g] += un + uo;
            terms[g] += (io ? 1u : 0u) + (in ? 1u : 0u);
            if (inner) {
                const uint32_t sc0 = min(jn[g], cl[g]) - bl[g], sc1 = max(jn[g], cl[g]) - bl[g];
                const bool fene = ok && bond[g] && ((K.bonded >> ((4u * sc0 + sc1) & 31u)) & 1u);
                // Eq. (2): +inf at or beyond the limit, else the ratio of its
                // arguments after and before the move
                const double lo2 = 2.25 * s2o, ln2 = 2.25 * s2n;
                const bool fo = r2o < lo2, fn = r2n < ln2, fin = fene && fo && fn;
                num[g] = fin ? (ln2 - r2n) * lo2 : 1.0;
                den[g] = fin ? (lo2 - r2o) * ln2 : 1.0;
                if (fene) {
                    if (!fin) de[g] += (fn ? 0.0 : __builtin_inf()) - (fo ? 0.0 : __builtin_inf());
                    terms[g] += (fo ? 1u : 0u) + (fn ? 1u : 0u);
                    if (kLog && logging)
                        sc[g] += fx_fene(W.sij[4u * to[g] + tj[g]], r2o) + fx_fene(W.sij[4u * tn[g] + tm[g]], r2n);
                }
            }
        }
        if (inner) {
            // the change of Eq. (2) in one logarithm; the partners sit on the
            // first lanes of a row, so the second evaluation's go to lanes 8 ..
            // and one division and one logarithm serve both
            double nu = num[0], dn = den[0];
            if (G == 2) {
                const double n1 = dpp_move<0x128, 0xf>(num[G - 1]), d1 = dpp_move<0x128, 0xf>(den[G - 1]);  // row_ror:8
                nu = rl < 8u ? nu : n1;
                dn = rl < 8u ? dn : d1;
            }
            const double dl = -33.75 * log(nu / dn);
            if (G == 2) {
                de[0] += rl < 8u ? dl : 0.0;
                de[G - 1] += rl < 8u ? 0.0 : dl;
            } else {
                de[0] += dl;
            }
        }
    };
    // a list that did not fit: its row walks the 27 cells instead
    bool over[G];
    bool any_over = false, any_third = false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        over[g] = act[g] && (uint32_t)__shfl((int)j[g][0], (int)((lane & 48u) + kFxPartners)) == kFxOver;
        any_over = any_over || over[g];
        any_third = any_third || j[g][2] < kFxOver;
    }
    {
        uint32_t jn[G];
        bool ok[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            jn[g] = j[g][0];
            ok[g] = j[g][0] < kFxOver && (!over[g] || rl < kFxPartners);
        }
        pass(jn, ok, true);
#pragma unroll
        for (int g = 0; g < G; ++g) { jn[g] = j[g][1]; ok[g] = j[g][1] < kFxOver && !over[g]; }
        pass(jn, ok, false);
        if (__ballot(any_third || any_over)) {
#pragma unroll
            for (int g = 0; g < G; ++g) { jn[g] = j[g][2]; ok[g] = j[g][2] < kFxOver && !over[g]; }
            pass(jn, ok, false);
            if (__ballot(any_over)) {
                const uint32_t nc = K.nc, span = min(nc, 3u);
                for (uint32_t o = 0; o < span * span * span; ++o) {
                    uint32_t q[G], ce[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const uint32_t cid = V.atom[cl[g]].cell;
                        const uint32_t ix = cid % nc, iy = (cid / nc) % nc, iz = cid / (nc * nc);
                        const uint32_t x = (ix + nc - 1u + o % span) % nc, y = (iy + nc - 1u + (o / span) % span) % nc,
                                       z = (iz + nc - 1u + o / (span * span)) % nc;
                        const uint32_t c = x + nc * (y + nc * z);
                        q[g] = V.cell_start[c] + rl;
                        ce[g] = over[g] ? V.cell_start[c + 1] : 0u;
                    }
                    for (;;) {
                        bool more = false;
#pragma unroll
                        for (int g = 0; g < G; ++g) {
                            const bool in = q[g] < ce[g];
                            more = more || in;
                            jn[g] = in ? V.cell_list[q[g]] : cl[g];
                            ok[g] = in && jn[g] - bl[g] >= K.n;
                            q[g] += 16u;
                        }
                        if (!__ballot(more)) break;
                        pass(jn, ok, false);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const double rs = row_sum_dpp(de[g]);
        const uint32_t ts = row_sum_dpp_u(terms[g]);
        double ss = 0.0;
        if (kLog) ss = row_sum_dpp(sc[g]);
        if (rl == 15u) {
            W.sum[4u * (uint32_t)g + row] = rs;
            W.terms[4u * (uint32_t)g + row] = ts;
            if (kLog) W.scale[4u * (uint32_t)g + row] = ss;
        }
    }
}

// dE of the attempt on atom a, summed over the atoms of the 27 cells in stencil
// order by the whole wave, a lane each: the order in which E_acc was summed
// before attempts had rows.  An overlapping start has moves that change its
// energy by 1e10 and more; the last bits of their terms, up to 1e6 in all, stay in
// E_acc until the next re-sum, and with this order E_acc of such a start keeps the
// values it had.  Neither order is the more exact one, and this second evaluation
// makes the sweeps of an overlapping start 3 % longer.  Only the net change is
// tested: terms of 1e10 that cancel to less than kFxLarge enter by the sum over
// the rows, and the two sums then differ by some 1e-6.
constexpr double kFxLarge = 1e4;

__device__ __forceinline__ bool fx_in_stencil(double x, double h, uint32_t c, const FxDev& D, double m)
{
    if (D.nc <= 3u) return true;  // the three cells are the whole axis
    const double t = fx_mi(fx_wrap(x - h, D.L) - (double)c * D.w, D.L, D.invL);
    return t >= m - D.w && t <= 2.0 * D.w - m;
}

constexpr uint32_t kFxListed = 384;  // atoms of a cell's stencil that serve its molecules' other atoms too

template <bool kRes>
__device__ __attribute__((noinline)) double fx_stencil_sum(const FxDev* Dp, typename FxView<kRes>::template Ptr<FxAtom> atom,
                                                           typename FxView<kRes>::template Ptr<uint32_t> cell_start,
                                                           typename FxView<kRes>::template Ptr<uint32_t> cell_list,
                                                           uint32_t a, uint32_t kind, double tx, double ty, double tz,
                                                           double hx, double hy, double hz, uint32_t cell)
{
    const FxDev& D = *Dp;
    const FxView<kRes> V{atom, cell_start, cell_list, nullptr};
    FxK K{};
    K.nc = D.nc;
    const int lane = __lane_id();
    const uint32_t n = D.n, nc = D.nc, base = n * fx_mol(n, a);
    const bool flip = kind != kFxMove;
    const double sig[4] = {D.sigma[0], D.sigma[1], D.sigma[2], D.sigma[3]};
    double ox[4], oy[4], oz[4], nx[4], ny[4], nz[4];
    uint32_t ot[4], nt[4], changed = 0;
    for (uint32_t s = 0; s < 4; ++s) {
        const FxAtom A = V.at(base + (s < n ? s : 0u));
        ox[s] = nx[s] = A.x; oy[s] = ny[s] = A.y; oz[s] = nz[s] = A.z;
        ot[s] = nt[s] = A.type;
    }
    for (uint32_t s = 0; s < n; ++s) {
        if (flip) {
            nt[s] = fx_pick(ot, D.flips[kind][s]);
            if (nt[s] != ot[s]) changed |= 1u << s;
        } else if (base + s == a) {
            nx[s] = fx_wrap(tx, D.L); ny[s] = fx_wrap(ty, D.L); nz[s] = fx_wrap(tz, D.L);
            changed = 1u << s;
        }
    }
    double de = 0.0;
    {
        // intramolecular pairs on lanes 0 .. 5: (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
        const uint32_t i = lane < 3 ? 0u : (lane < 5 ? 1u : 2u);
        const uint32_t j = lane < 3 ? (uint32_t)lane + 1u : (lane < 5 ? (uint32_t)lane - 1u : 3u);
        if (lane < 6 && j < n && (((changed >> i) | (changed >> j)) & 1u)) {
            const double dxo = fx_mi(fx_pick(ox, i) - fx_pick(ox, j), D.L, D.invL),
                         dyo = fx_mi(fx_pick(oy, i) - fx_pick(oy, j), D.L, D.invL),
                         dzo = fx_mi(fx_pick(oz, i) - fx_pick(oz, j), D.L, D.invL);
            const double dxn = fx_mi(fx_pick(nx, i) - fx_pick(nx, j), D.L, D.invL),
                         dyn = fx_mi(fx_pick(ny, i) - fx_pick(ny, j), D.L, D.invL),
                         dzn = fx_mi(fx_pick(nz, i) - fx_pick(nz, j), D.L, D.invL);
            const double r2o = dxo * dxo + dyo * dyo + dzo * dzo, r2n = dxn * dxn + dyn * dyn + dzn * dzn;
            const double so = 0.5 * (fx_pick(sig, fx_pick(ot, i)) + fx_pick(sig, fx_pick(ot, j)));
            const double sn = 0.5 * (fx_pick(sig, fx_pick(nt, i)) + fx_pick(sig, fx_pick(nt, j)));
            de = fx_wca(sn * sn, r2n, D.rc2f) - fx_wca(so * so, r2o, D.rc2f);
            if ((D.bonded >> (4 * i + j)) & 1u) {
                const double lo2 = 2.25 * so * so, ln2 = 2.25 * sn * sn;
                if (r2o < lo2 && r2n < ln2)
                    de += -33.75 * log((1.0 - r2n / ln2) / (1.0 - r2o / lo2));
                else
                    de += (r2n < ln2 ? 0.0 : __builtin_inf()) - (r2o < lo2 ? 0.0 : __builtin_inf());
            }
        }
    }
    uint32_t lo, off, total;
    int nseg = fx_segments(K, V, (int)(cell % nc), (int)((cell / nc) % nc), (int)(cell / (nc * nc)), &lo, &off, &total);
    const bool list = total <= kFxListed;
    // an atom of another cell is served by the list of this one when every atom
    // that can reach it was sorted into the list's 27 cells
    const double m = sqrt(D.rc2f) * fmax(fmax(sig[0], sig[1]), fmax(sig[2], sig[3])) + 1.7320508075688772 * D.dmax + 1e-9;
    for (uint32_t s = 0; s < n; ++s) {
        if (!((changed >> s) & 1u)) continue;  // wave-uniform
        const uint32_t at = uniform(V.atom[base + s].cell);
        bool listed = list && at == cell;
        if (!listed && list && flip)
            listed = fx_in_stencil(fx_pick(ox, s), hx, cell % nc, D, m) &&
                     fx_in_stencil(fx_pick(oy, s), hy, (cell / nc) % nc, D, m) &&
                     fx_in_stencil(fx_pick(oz, s), hz, cell / (nc * nc), D, m);
        listed = __ballot(listed) != 0ull;  // (the same in every lane)
        const uint32_t from = listed ? cell : at;
        nseg = fx_segments(K, V, (int)(from % nc), (int)((from / nc) % nc), (int)(from / (nc * nc)), &lo, &off, &total);
        const double sos = fx_pick(sig, fx_pick(ot, s)), sns = fx_pick(sig, fx_pick(nt, s));
        for (uint32_t b = 0; b < total; b += 64u) {
            const uint32_t idx = b + (uint32_t)lane;
            uint32_t seg = 0;
            for (int t = 1; t < nseg; ++t) seg += idx >= rl_u(off, t) ? 1u : 0u;
            const uint32_t d = (uint32_t)__shfl((int)(lo - off), (int)seg);
            const uint32_t j = idx < total ? (uint32_t)V.cell_list[idx + d] : base;
            const bool valid = j - base >= n;  // not an atom of the molecule
            const FxAtom A = V.at(j);
            const double sj = fx_pick(sig, valid ? A.type : 0u);
            const double xj = valid ? A.x : 0.0, yj = valid ? A.y : 0.0, zj = valid ? A.z : 0.0;
            const double dxo = fx_mi(fx_pick(ox, s) - xj, D.L, D.invL), dyo = fx_mi(fx_pick(oy, s) - yj, D.L, D.invL),
                         dzo = fx_mi(fx_pick(oz, s) - zj, D.L, D.invL);
            const double r2o = valid ? dxo * dxo + dyo * dyo + dzo * dzo : 1e30;
            const double dxn = fx_mi(fx_pick(nx, s) - xj, D.L, D.invL), dyn = fx_mi(fx_pick(ny, s) - yj, D.L, D.invL),
                         dzn = fx_mi(fx_pick(nz, s) - zj, D.L, D.invL);
            const double r2n = flip ? r2o : (valid ? dxn * dxn + dyn * dyn + dzn * dzn : 1e30);
            const double so = 0.5 * (sos + sj), sn = 0.5 * (sns + sj);
            de += fx_wca(sn * sn, r2n, D.rc2f) - fx_wca(so * so, r2o, D.rc2f);
        }
    }
    return wave_sum_dpp(de);
}

// The attempts on up to 64 atoms of one cell (lane q holds atom q and its
// proposal), in order, by one wave.
//
// The next attempts, up to kFxRows changed atoms of them (one for a
// translation, two to four for a flip), are evaluated side by side against the
// present state, a row of 16 lanes per changed atom.  They are decided in
// order: everything up to the first accepted one stands; those after it are
// evaluated again on the state it leaves (in a cell nearly every pair of atoms
// is within reach), so every decision is taken on its predecessors' state and
// dE does not depend on how the attempts were grouped.  With 7 - 30 % accepted
// a cell of 6 atoms takes one to three evaluations of 2 us.  The chain of
// evaluations bounds the kernel (a system runs on one compute unit): a sweep
// of 1000 triangles at T = 0.75 takes 0.78 ms, of 333 tetrahedra 1.38 ms (by
// the whole wave, one attempt after another over the 27 cells' atoms, 2.80 and
// 7.4 ms; with one row per 16 lanes instead of two 0.78 and 1.61 ms).
template <bool kLog, bool kRes>
__device__ __forceinline__ void fx_run_rows(const FxDev& Dv, const FxK& K, const FxView<kRes>& V, uint32_t cnt, uint32_t at,
                                            const FxProp& pr, uint64_t sweep, const double h[3], uint32_t cell,
                                            bool logging, const FxWaveLds& W, FxCount& wc)
{
    const uint32_t lane = (uint32_t)__lane_id();
    const uint32_t n = K.n;
    const uint32_t base = n * fx_mol(n, at);
    const bool flip = pr.kind != kFxMove;
    const uint32_t chg = flip ? (K.chgw >> (4u * (pr.kind & 3u))) & 15u : 1u << (at - base);
    uint64_t live = __ballot(lane < cnt && !(pr.cross & kFxExit));
    while (live) {
        // the rows: first row of each attempt by a prefix sum
        uint32_t need = (live >> lane) & 1u ? (uint32_t)__popc(chg) : 0u;
        const uint32_t end = wave_incl_scan(need);
        const bool in = need != 0u && end <= kFxRows;
        const uint64_t win = __ballot(in);
        const uint32_t nrow = rl_u(end, 63 - __builtin_clzll(win));
        if (in) {
            uint32_t r = end - need;
#pragma unroll
            for (uint32_t t = 0; t < 4; ++t)
                if ((chg >> t) & 1u) W.row[r++] = FxRow{pr.tx, pr.ty, pr.tz, base + t, base, pr.kind, 0u};
        }
        wave_lds_sync();
        if (nrow > 4u)
            fx_eval_rows<2, kLog>(K, V, nrow, logging, W);
        else
            fx_eval_rows<1, kLog>(K, V, nrow, logging, W);
        wave_lds_sync();
        double dE = 0.0;
        const uint32_t r0 = in ? end - need : 0u;
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            const double v = W.sum[(r0 + t) & (kFxRows - 1u)];
            if (t < need) dE += v;
        }
        const bool accept = in && ((dE <= 0.0) || (pr.thr < -dE));
        const uint64_t acc = __ballot(accept);
        const uint64_t done = acc ? win & ((acc & (0ull - acc)) * 2ull - 1ull) : win;
        if ((done >> lane) & 1u) {
            uint32_t tt = 0;
            double S = 0.0;
            for (uint32_t t = 0; t < need; ++t) {
                tt += W.terms[r0 + t];
                if (kLog) S += W.scale[r0 + t];
            }
            wc.terms += tt;
            if (kLog && logging) {
                MoveRecord rec;
                rec.delta_e = dE; rec.scale = S; rec.t_log_u = pr.thr; rec.sweep = sweep;
                rec.molecule = at; rec.move = flip ? MC_FLIP : MC_TRANSLATE; rec.accepted = accept ? 1 : 0;
                rec.exited = 0; rec.axis = (uint8_t)pr.kind; rec.pair_terms = tt; rec.pad = 0;
                Dv.log[(sweep - Dv.log_sweep0) * K.N + at] = rec;
            }
        }
        live &= ~done;
        if (acc) {
            const int q = (int)__builtin_ctzll(acc);
            double de = rl_d(dE, q);
            if (fabs(de) > kFxLarge)
                de = fx_stencil_sum<kRes>(&Dv, V.atom, V.cell_start, V.cell_list, rl_u(at, q), rl_u(pr.kind, q),
                                          rl_d(pr.tx, q), rl_d(pr.ty, q), rl_d(pr.tz, q), h[0], h[1], h[2], cell);
            wc.e += de;
            if (rl_u(pr.kind, q) != kFxMove) wc.acc_f += 1; else wc.acc_t += 1;
            if ((int)lane == q) {
                if (flip) {
                    const uint32_t perm = fx_pick(K.flipw, pr.kind);
                    uint32_t t[4];
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u) t[u] = V.atom[base + (u < n ? (perm >> (8u * u)) & 3u : 0u)].type;
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u)
                        if ((chg >> u) & 1u) V.atom[base + u].type = t[u];
                } else {
                    // wrapped; the shifts are the periodic images crossed
                    const int fx = (int)(pr.cross & 3u) - 1, fy = (int)((pr.cross >> 2) & 3u) - 1,
                              fz = (int)((pr.cross >> 4) & 3u) - 1;
                    V.atom[at].x = pr.tx - K.L * (double)fx;
                    V.atom[at].y = pr.ty - K.L * (double)fy;
                    V.atom[at].z = pr.tz - K.L * (double)fz;
                    if (fx) K.img[at] += fx;
                    if (fy) K.img[K.N + at] += fy;
                    if (fz) K.img[2 * K.N + at] += fz;
                }
            }
        }
        wave_lds_sync();
    }
}

// Ascending atom index inside every cell of c0, c0 + cstep, ...: one wave per
// cell, a lane per atom whose place is the number of smaller indices (a cell
// of more than 64 atoms is sorted by one lane).
__device__ void fx_sort_cells(uint32_t* list, const uint32_t* start, uint32_t c0, uint32_t cstep,
                              uint32_t ncell)
{
    const uint32_t lane = (uint32_t)__lane_id();
    for (uint32_t c = c0; c < ncell; c += cstep) {
        const uint32_t b = uniform(start[c]), cnt = uniform(start[c + 1]) - b;
        if (cnt <= 1u) continue;
        if (cnt <= 64u) {
            const uint32_t v = lane < cnt ? list[b + lane] : 0xFFFFFFFFu;
            uint32_t rank = 0;
            for (uint32_t q = 0; q < cnt; ++q) rank += (uint32_t)__builtin_amdgcn_readlane((int)v, (int)q) < v;
            wave_lds_sync();
            if (lane < cnt) list[b + rank] = v;
        } else if (lane == 0) {
            for (uint32_t i = b + 1; i < b + cnt; ++i) {
                const uint32_t x = list[i];
                uint32_t q = i;
                while (q > b && list[q - 1] > x) {
                    list[q] = list[q - 1];
                    --q;
                }
                list[q] = x;
            }
        }
        wave_lds_sync();
    }
}

// The hot kernel: n sweeps of one system on one workgroup.  With kRes the
// atoms and cell lists live in LDS for the whole launch; otherwise the same
// code runs on arrays in the system's buffer.  Positions and types are copied
// in at the start and written back at the end.  kLog: some system of the
// launch has a decision log.
template <bool kRes, bool kLog>
__global__ void __launch_bounds__(kFxThreads) k_fx_sweeps(FxList list, uint64_t n_sweeps)
{
    FxDev* __restrict__ Dp = list.d[blockIdx.x];
    __shared__ double pair_s[16], pair_s2[16];
    __shared__ FxRow rows[kFxWaves][kFxRows];
    __shared__ uint32_t rterms[kFxWaves][kFxRows];
    __shared__ double rsum[kFxWaves][kFxRows], rscale[kLog ? kFxWaves : 1][kFxRows];
    __shared__ __align__(16) FxNbr<kRes> lists[kFxWaves][kFxBuild * 64];
    __shared__ uint32_t scratch[kFxWaves];
    __shared__ double misc[2];
    __shared__ double dmax2[kFxWaves];
    extern __shared__ __align__(16) unsigned char fx_smem[];
    const FxDev& D = *Dp;
    const FxK K = fx_const(D);
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    FxWaveLds W{rows[wave], rsum[wave], rscale[kLog ? wave : 0], rterms[wave], lists[wave], pair_s, pair_s2};
    Stats* st = D.stats;
    const uint32_t N = D.N, ncell = D.ncell, nc = D.nc, k = D.k;
    FxView<kRes> V;
    if constexpr (kRes) {
        const FxLds l = fx_lds_layout(N, ncell);
        V = FxView<kRes>{(Lds<FxAtom>*)(fx_smem + l.atom), (Lds<uint32_t>*)(fx_smem + l.cstart),
                         (Lds<uint32_t>*)(fx_smem + l.clist), (Lds<double>*)(fx_smem + l.ecell)};
    } else {
        V = FxView<kRes>{(Global<FxAtom>*)D.atom, (Global<uint32_t>*)D.cell_start, (Global<uint32_t>*)D.cell_list,
                         (Global<double>*)D.ecell};
    }
    for (uint32_t i = tid; i < N; i += kFxThreads)
    {
        auto* a = V.atom + i;
        a->x = D.pos[i]; a->y = D.pos[N + i]; a->z = D.pos[2 * N + i];
        a->type = D.type[i]; a->cell = 0u;
    }
    const uint32_t na = nc / k, nact = na * na * na;
    uint64_t sweep = st->sweep;
    const uint64_t origin = st->obs_origin;
    if (tid == 0) misc[0] = st->e_acc;
    if (tid < 16) {
        const double sg = 0.5 * (D.sigma[tid >> 2] + D.sigma[tid & 3]);
        pair_s[tid] = sg;
        pair_s2[tid] = sg * sg;
    }
    __syncthreads();
    FxCount wc{};
    for (uint64_t it = 0; it < n_sweeps; ++it) {
        const U4 g = philox10(0xFFFFFFFFu, (uint32_t)sweep, (uint32_t)(sweep >> 32), 3u, K.seed_lo, K.seed_hi);
        const double h[3] = {K.w * unit_open(g.x), K.w * unit_open(g.y), K.w * unit_open(g.z)};
        // counting sort of the atoms by cell
        for (uint32_t c = tid; c <= ncell; c += kFxThreads) V.cell_start[c] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < N; i += kFxThreads) {
            const uint32_t c = fx_cell(V.atom[i].x, V.atom[i].y, V.atom[i].z, h, K);
            V.atom[i].cell = c;
            atomicAdd((uint32_t*)&V.cell_start[c + 1], 1u);
        }
        __syncthreads();
        block_excl_scan_t<kFxThreads>((uint32_t*)(V.cell_start + 1), ncell, scratch);
        for (uint32_t i = tid; i < N; i += kFxThreads)
            V.cell_list[atomicAdd((uint32_t*)&V.cell_start[V.atom[i].cell + 1], 1u)] = i;
        __syncthreads();
        fx_sort_cells((uint32_t*)V.cell_list, (const uint32_t*)V.cell_start, (uint32_t)wave, kFxWaves, ncell);
        __syncthreads();
        const bool logging = kLog && D.log != nullptr && sweep - D.log_sweep0 < D.log_sweeps;
        fx_propose_all(D, K, V, sweep, h, logging, wc);
        fx_build_lists(K, V, h, wave, ncell, W);
        __syncthreads();
        // The cells of a colour are attempted in ascending index; they run
        // side by side when no attempt in one can reach an atom another
        // reads or writes.  Two attempted atoms of different cells are at
        // least the gap (k - 1) w apart, and their attempts can meet only
        // through pairs within r_c of their molecules' atoms: so the cells
        // cannot interact when the gap is at least 2 D_c + r_c, D_c the
        // largest atom distance inside a molecule with an atom in the
        // colour's cells at the colour's start plus 2 sqrt(3) d (each atom
        // moves at most once per sweep).  Otherwise one cell at a time, in
        // that order: the same chain either way.
        auto colour_together = [&](uint32_t kx, uint32_t ky, uint32_t kz) __attribute__((always_inline)) {
            if (K.together != 0u) return K.together == 1u;
            double d2 = 0.0;
            const uint32_t n = K.n;
            for (uint32_t ci = (uint32_t)wave; ci < nact; ci += kFxWaves) {
                const uint32_t cell = (kx + k * (ci % na)) + nc * ((ky + k * ((ci / na) % na)) +
                                                                  nc * (kz + k * (ci / (na * na))));
                const uint32_t b = V.cell_start[cell], e = V.cell_start[cell + 1];
                for (uint32_t q = b + (uint32_t)lane; q < e; q += 64u) {
                    const uint32_t base = n * fx_mol(n, V.cell_list[q]);
                    for (uint32_t i = 0; i + 1 < n; ++i)
                        for (uint32_t j = i + 1; j < n; ++j) {
                            const double dx = fx_mif(V.atom[base + i].x - V.atom[base + j].x, K.L, K.invL);
                            const double dy = fx_mif(V.atom[base + i].y - V.atom[base + j].y, K.L, K.invL);
                            const double dz = fx_mif(V.atom[base + i].z - V.atom[base + j].z, K.L, K.invL);
                            d2 = fmax(d2, dx * dx + dy * dy + dz * dz);
                        }
                }
            }
#pragma unroll
            for (int o = 32; o; o >>= 1) d2 = fmax(d2, __shfl_xor(d2, o));
            if (lane == 0) dmax2[wave] = d2;
            __syncthreads();
            double dm = 0.0;
            for (int w2 = 0; w2 < kFxWaves; ++w2) dm = fmax(dm, dmax2[w2]);
            __syncthreads();
            return K.sep >= 2.0 * sqrt(dm) + K.dyn_base;
        };
        // Cell number i of the colours in order; a wave takes number `wave` of
        // each colour and every kFxWaves-th after it.
        auto cell_of = [&](uint32_t col, uint32_t ci) __attribute__((always_inline)) {
            const uint32_t kx = col % k, ky = (col / k) % k, kz = col / (k * k);
            return (kx + k * (ci % na)) + nc * ((ky + k * ((ci / na) % na)) + nc * (kz + k * (ci / (na * na))));
        };
        const uint32_t ncol = k * k * k;
        // The lines of the wave's next cell (its proposals and the lists of its
        // molecules' atoms) are brought near while the present cell is attempted.
        uint32_t touched = 0;
        auto touch = [&](uint32_t cell) __attribute__((always_inline)) {
            const uint32_t b = V.cell_start[cell], e = V.cell_start[cell + 1];
            const uint32_t q = b + (uint32_t)(lane >> 3), s = (uint32_t)(lane >> 1) & 3u;
            if (q < e) {
                const uint32_t c = K.n * fx_mol(K.n, V.cell_list[q]) + s;
                if (s < K.n)
                    touched = (uint32_t)((Global<FxNbr<kRes>>*)K.nbr)[(size_t)c * kFxNbr + (lane & 1 ? kFxNbr - 1u : 0u)];
                else
                    touched = K.props[q].kind;
            }
        };
        // the attempts of cell `ci` of colour `col` by this wave
        auto run_cell = [&](uint32_t col, uint32_t ci) __attribute__((always_inline)) {
            const uint32_t cell = cell_of(col, ci);
            const uint32_t b = uniform(V.cell_start[cell]),
                           e = uniform(V.cell_start[cell + 1]);
            wc.e = 0.0;
            for (uint32_t q0 = b; q0 < e; q0 += 64u) {
                const uint32_t cnt = min(64u, e - q0);
                uint32_t at = 0;
                FxProp pr{};
                if ((uint32_t)lane < cnt) {
                    at = V.cell_list[q0 + lane];
                    const Global<FxProp>* in = K.props + (q0 + (uint32_t)lane);
                    pr = FxProp{in->thr, in->tx, in->ty, in->tz, in->kind, in->cross};
                }
                asm volatile("" ::"v"(touched));
                const bool last = ci + kFxWaves >= nact;
                if (!last || col + 1u < ncol) touch(last ? cell_of(col + 1u, (uint32_t)wave) : cell_of(col, ci + kFxWaves));
                fx_run_rows<kLog>(D, K, V, cnt, at, pr, sweep, h, cell, logging, W, wc);
            }
            if (lane == 0) V.ecell[cell] = wc.e;
        };
        for (uint32_t col = 0; col < ncol; ++col) {
            const uint32_t kx = col % k, ky = (col / k) % k, kz = col / (k * k);
            if (colour_together(kx, ky, kz)) {
                for (uint32_t ci = (uint32_t)wave; ci < nact; ci += kFxWaves) run_cell(col, ci);
                __syncthreads();
            } else {
                for (uint32_t ci = 0; ci < nact; ++ci) {
                    if (ci % kFxWaves == (uint32_t)wave) run_cell(col, ci);
                    __syncthreads();
                }
            }
        }
        ++sweep;
        // E_acc += the sweep's dE, the cells in a fixed order; E/M samples
        if (wave == 0) {
            const double e = misc[0] + sweep_energy([&](uint32_t c) { return (double)V.ecell[c]; }, ncell);
            if (lane == 0) misc[0] = e;
        }
        if (tid == 0) {
            const uint64_t t = sweep - origin;
            if (t >= D.obs_start && D.obs_interval && t % D.obs_interval == 0) {
                const double em = misc[0] / (double)D.M;
                if (st->n_e < D.max_samples) D.e_samples[st->n_e] = em;
                st->n_e += 1;
                st->e_sum += em;
                st->e_sumsq += em * em;
            }
        }
        __syncthreads();
    }
    {
        const uint32_t att_t = wave_sum_u(wc.att_t), att_f = wave_sum_u(wc.att_f), exits = wave_sum_u(wc.exits);
        unsigned long long terms = wc.terms;
#pragma unroll
        for (int o = 32; o; o >>= 1) terms += __shfl_xor(terms, o);
        if (lane == 0) {
            if (att_t) atomicAdd((unsigned long long*)&st->attempts[MC_TRANSLATE], (unsigned long long)att_t);
            if (att_f) atomicAdd((unsigned long long*)&st->attempts[MC_FLIP], (unsigned long long)att_f);
            if (wc.acc_t) atomicAdd((unsigned long long*)&st->accepts[MC_TRANSLATE], (unsigned long long)wc.acc_t);
            if (wc.acc_f) atomicAdd((unsigned long long*)&st->accepts[MC_FLIP], (unsigned long long)wc.acc_f);
            if (exits) atomicAdd((unsigned long long*)&st->exits, (unsigned long long)exits);
            if (terms) atomicAdd((unsigned long long*)&st->pair_terms, terms);
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < N; i += kFxThreads) {
        const FxAtom A = V.at(i);
        D.pos[i] = A.x;
        D.pos[N + i] = A.y;
        D.pos[2 * N + i] = A.z;
        D.type[i] = (uint8_t)A.type;
    }
    if (tid == 0) {
        st->sweep = sweep;
        st->e_acc = misc[0];
    }
}

}  // namespace
}  // namespace flipmc
