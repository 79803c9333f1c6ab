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
// neighbours of every atom, then the k^3 colours in order; the waves take the
// cells of a colour, and a wave runs its cell's attempts in order, up to four
// of them evaluated side by side, a row of 16 lanes per changed atom.
// Same-colour cells are at least (k - 1) w >= 2 D + r_c apart (D the largest
// distance two atoms of one molecule can reach, r_c the largest cut-off), so
// no two attempts of a colour touch the same pair term.  A DPP reduction in
// FP64 over each row gives dE in a fixed order.  A bond stretched to 1.5
// sigma_ij or beyond makes dE infinite: the move is rejected.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "engine.h"
#include "flipmc.h"
#include "wave.h"

namespace flipmc {
namespace {
constexpr int kFxThreads = 512;
constexpr int kFxWaves = kFxThreads / 64;
constexpr int kFxSeg = 64;          // stencil row segments per attempt (radius <= 2: <= 50)
constexpr uint32_t kFxNbr = 48;     // neighbours listed per atom (three lanes' worth of a 16-lane row)
constexpr uint32_t kFxListed = 65534;  // atoms a 16-bit list can index (0xFFFE, 0xFFFF are marks)
constexpr uint32_t kFxNone = 0xFFFFu;  // no neighbour
constexpr uint32_t kFxOver = 0xFFFEu;  // first entry of a list that did not fit
// static LDS of the sweep kernel: segments per wave, pair tables, scan
// scratch and the energy accumulator (with room to spare)
constexpr size_t kFxStaticLds = (size_t)kFxWaves * 2 * kFxSeg * 4 + 2 * 16 * 8 + 512;
constexpr uint32_t kFxParts = 1024;  // workgroups of the event kernel
constexpr uint32_t kFxMany = 256;    // systems of one sweep launch (a workgroup each)

// Everything a workgroup needs about one system; in the system's buffer.
struct FxDev {
    uint32_t geometry, n, M, N;
    uint32_t k, nc, ncell, nflip;
    uint32_t seed_lo, seed_hi, pad2, pad3;
    uint32_t bonded;  // bit 4 i + j: atoms i, j of a molecule are bonded
    uint32_t resum_interval, obs_interval, gofr_interval, obs_start, max_samples, gofr_nbins;
    uint32_t pad;
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
    uint32_t* cell_id;    // [N]
    double* ecell;        // [ncell] accepted dE of each cell in the current sweep
    double* part;         // [kFxParts] partial energies of the event kernel
    uint16_t* nbr;        // [N][kFxNbr] neighbours of each atom in the current sweep, or null
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
    double L, invL, w, T, p_flip, dmax, rc2f, sep, dyn_base;
    double sigma[4];
    int32_t* img;
    uint16_t* nbr;
    MoveRecord* log;
    uint64_t log_sweep0;
    uint32_t chg[4];    // bit s of word q: flip q changes the type of atom s
    float list_r2;      // neighbour lists: squared radius, (r_c + 2 sqrt(3) d)^2 with a margin
};

__device__ __forceinline__ FxK fx_const(const FxDev& D)
{
    FxK K;
    K.n = D.n; K.N = D.N; K.nc = D.nc; K.nflip = D.nflip; K.bonded = D.bonded;
    K.seed_lo = D.seed_lo; K.seed_hi = D.seed_hi;
    for (int q = 0; q < 4; ++q)
        K.flipw[q] = (uint32_t)D.flips[q][0] | ((uint32_t)D.flips[q][1] << 8) | ((uint32_t)D.flips[q][2] << 16) |
                     ((uint32_t)D.flips[q][3] << 24);
    K.L = D.L; K.invL = D.invL; K.w = D.w; K.T = D.T; K.p_flip = D.p_flip; K.dmax = D.dmax; K.rc2f = D.rc2f;
    K.sep = D.sep; K.dyn_base = D.dyn_base; K.together = D.together;
    for (int t = 0; t < 4; ++t) K.sigma[t] = D.sigma[t];
    K.img = D.img;
    K.nbr = D.nbr;
    K.log = D.log;
    K.log_sweep0 = D.log_sweep0;
    for (int q = 0; q < 4; ++q) {
        uint32_t c = 0;
        for (uint32_t t = 0; t < 4; ++t) c |= (t < D.n && D.flips[q][t] != t ? 1u : 0u) << t;
        K.chg[q] = c;
    }
    // the FP32 distances of the list build are within 1e-5 of the FP64 ones
    const double smax = fmax(fmax(D.sigma[0], D.sigma[1]), fmax(D.sigma[2], D.n > 3u ? D.sigma[3] : 0.0));
    const float r = (float)(sqrt(D.rc2f) * smax + 2.0 * 1.7320508075688772 * D.dmax) + 1e-3f;
    K.list_r2 = r * r;
    return K;
}

__device__ __forceinline__ double fx_wrap(double x, double L) { return x - L * floor(x / L); }
__device__ __forceinline__ double fx_mi(double d, double L, double invL) { return d - L * rint(d * invL); }

__device__ __forceinline__ int fx_axis(double x, double h, const FxK& D)
{
    int c = (int)floor(fx_wrap(x - h, D.L) / D.w);
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

struct FxCount {
    uint32_t att_t, att_f, acc_t, acc_f, exits;
    uint32_t terms;  // interacting pairs, this lane's share
    double e;  // accepted dE of the current cell, in attempt order
};

// Per-wave LDS: the stencil's row segments.  Per workgroup: the pair
// diameters sigma_ij and their squares by 4 t_i + t_j.
struct FxWaveLds {
    uint32_t* seglo;
    uint32_t* segoff;
    const double* sij;
    const double* s2ij;
};

// Where the sweep kernel reads and writes the state and the cell lists: the
// workgroup's LDS for systems that fit there, the system's buffer otherwise.
struct FxView {
    double* pos;          // SoA [3][N]
    uint8_t* type;        // [N]
    uint32_t* cell_start; // [ncell + 1]
    uint32_t* cell_list;  // [N]
    uint32_t* cell_id;    // [N]
    double* ecell;        // [ncell]
};

struct FxLds {
    size_t pos, type, cstart, clist, cid, ecell, total;
};

__host__ __device__ inline FxLds fx_lds_layout(uint32_t N, uint32_t ncell)
{
    FxLds l{};
    size_t o = 0;
    auto a16 = [](size_t x) { return (x + 15) & ~size_t(15); };
    l.pos = o;    o = a16(o + 3 * size_t(N) * sizeof(double));
    l.ecell = o;  o = a16(o + size_t(ncell) * sizeof(double));
    l.type = o;   o = a16(o + size_t(N));
    l.cstart = o; o = a16(o + (size_t(ncell) + 1) * sizeof(uint32_t));
    l.clist = o;  o = a16(o + size_t(N) * sizeof(uint32_t));
    l.cid = o;    o = a16(o + size_t(N) * sizeof(uint32_t));
    l.total = o;
    return l;
}

// Row segments of the cells within radius r of cell (cx, cy, cz): rows along
// x of one or two contiguous cell ranges (every cell once when the stencil
// covers the whole axis).  Returns the number of segments; *total = atoms.
__device__ __forceinline__ int fx_segments(const FxK& D, const FxView& V, int cx, int cy, int cz, int r,
                                           const FxWaveLds& W,
                           uint32_t* total)
{
    const int lane = __lane_id();
    const int nc = (int)D.nc;
    const bool full = 2 * r + 1 >= nc;
    const int nrow = full ? nc : 2 * r + 1;
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
    const int nseg = nrow * nrow * nxr;
    uint32_t cnt = 0, lo = 0;
    if (lane < nseg) {
        const int ixr = lane % nxr, iy = (lane / nxr) % nrow, iz = lane / (nxr * nrow);
        const int y = full ? iy : (cy - r + iy + nc) % nc;
        const int z = full ? iz : (cz - r + iz + nc) % nc;
        const int xa = ixr ? xa1 : xa0, xb = ixr ? xb1 : xb0;
        const uint32_t row = (uint32_t)(nc * (y + nc * z));
        lo = V.cell_start[row + xa];
        cnt = V.cell_start[row + xb + 1] - lo;
    }
    const uint32_t off = wave_excl_scan(cnt, total);
    if (lane < nseg) {
        W.seglo[lane] = lo;
        W.segoff[lane] = off;
    }
    wave_lds_sync();
    return nseg;
}

__device__ __forceinline__ uint32_t fx_stencil_atom(const FxView& V, const FxWaveLds& W, int nseg, uint32_t idx)
{
    int lo = 0, hi = nseg;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (W.segoff[mid] <= idx) lo = mid; else hi = mid;
    }
    return V.cell_list[W.seglo[lo] + (idx - W.segoff[lo])];
}

template <typename T>
__device__ __forceinline__ T fx_pick(const T v[4], uint32_t i)
{
    return i == 0 ? v[0] : (i == 1 ? v[1] : (i == 2 ? v[2] : v[3]));
}

// The proposal of the attempt on atom a (Sec. II.B): move kind, flip
// rotation or translation target, the cell-exit test and T ln u.  Drawn for
// the atoms of a cell by one lane each before the cell's attempts (an atom's
// position changes only in its own attempt, so the draws do not depend on
// the attempts before it).
struct FxProp {
    double thr;         // T ln u
    double tx, ty, tz;  // translation target before the wrap
    uint32_t kind;      // flip: rotation index; translation: 255
    uint32_t flip, exited;
};

__device__ __forceinline__ FxProp fx_propose(const FxK& D, const FxView& V, uint32_t a, uint64_t sweep,
                                             const double h[3], uint32_t cell)
{
    const uint32_t N = D.N;
    const uint32_t slo = (uint32_t)sweep, shi = (uint32_t)(sweep >> 32);
    const U4 b0 = philox10(a, slo, shi, 0u, D.seed_lo, D.seed_hi);
    const U4 b1 = philox10(a, slo, shi, 1u, D.seed_lo, D.seed_hi);
    const double uacc = unit_53(b0.x, b0.y), ut = unit_open(b0.z);
    const double p0 = unit_open(b1.x), p1 = unit_open(b1.y), p2 = unit_open(b1.z);
    FxProp pr;
    pr.thr = D.T * log(uacc);
    pr.flip = ut < D.p_flip ? 1u : 0u;
    pr.kind = 255;
    pr.exited = 0;
    pr.tx = pr.ty = pr.tz = 0.0;
    if (pr.flip) {
        uint32_t q = (uint32_t)((double)D.nflip * p0);
        pr.kind = q >= D.nflip ? D.nflip - 1 : q;
    } else {
        pr.tx = V.pos[a] + D.dmax * (2.0 * p0 - 1.0);
        pr.ty = V.pos[N + a] + D.dmax * (2.0 * p1 - 1.0);
        pr.tz = V.pos[2 * N + a] + D.dmax * (2.0 * p2 - 1.0);
        pr.exited = fx_cell(fx_wrap(pr.tx, D.L), fx_wrap(pr.ty, D.L), fx_wrap(pr.tz, D.L), h, D) != cell;
    }
    return pr;
}

// Sum over each row of 16 lanes (the row's last lane gets it) in the order of
// wave_sum_dpp's first steps.
__device__ __forceinline__ double fx_row_sum(double v)
{
    v += dpp_move<0x111, 0xf>(v);
    v += dpp_move<0x112, 0xf>(v);
    v += dpp_move<0x114, 0xf>(v);
    v += dpp_move<0x118, 0xf>(v);
    return v;
}
__device__ __forceinline__ uint32_t fx_row_sum_u(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);
    return v;
}

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

// The neighbours of every atom in the current sweep: the atoms of other
// molecules within r_c + 2 sqrt(3) d of it at the sort (each of two atoms
// moves at most sqrt(3) d in the sweep, so every pair that comes within its
// cut-off is listed).  A wave per cell: the atoms of the 27 cells around it a
// lane each (relative to the cell's centre, FP32), tested against the cell's
// atoms one after another; the list keeps the order of the cell list.  Built
// once per sweep by all waves side by side, it takes the search (158 atoms of
// the 27 cells for about 18 within reach) out of the serial attempts: an
// attempt then needs a row of 16 lanes instead of the whole wave.
__device__ __forceinline__ void fx_build_lists(const FxK& K, const FxView& V, const double h[3], int wave,
                                               uint32_t ncell, const FxWaveLds& W)
{
    const uint32_t lane = (uint32_t)__lane_id();
    const uint32_t nc = K.nc, N = K.N, n = K.n;
    const bool fold = nc <= 3u;  // the 27 cells span the box: nearest image per pair
    const float Lf = (float)K.L, iLf = (float)K.invL;
    for (uint32_t cell = (uint32_t)wave; cell < ncell; cell += kFxWaves) {
        const uint32_t b = V.cell_start[cell], e = V.cell_start[cell + 1];
        if (b >= e) continue;
        const uint32_t ix = cell % nc, iy = (cell / nc) % nc, iz = cell / (nc * nc);
        const double ox = h[0] + ((double)ix + 0.5) * K.w, oy = h[1] + ((double)iy + 0.5) * K.w,
                     oz = h[2] + ((double)iz + 0.5) * K.w;
        uint32_t total;
        const int nseg = fx_segments(K, V, (int)ix, (int)iy, (int)iz, 1, W, &total);
        for (uint32_t q0 = b; q0 < e; q0 += 64u) {
            const uint32_t cnt = min(64u, e - q0);
            uint32_t at = 0, mol = 0, have = 0;  // lane q: atom q, its molecule, neighbours found
            float ax = 0.f, ay = 0.f, az = 0.f;
            if (lane < cnt) {
                at = V.cell_list[q0 + lane];
                mol = at / n;
                ax = (float)fx_mi(V.pos[at] - ox, K.L, K.invL);
                ay = (float)fx_mi(V.pos[N + at] - oy, K.L, K.invL);
                az = (float)fx_mi(V.pos[2 * N + at] - oz, K.L, K.invL);
            }
            for (uint32_t c0 = 0; c0 < total; c0 += 192u) {
                uint32_t id[3], mj[3];
                float x[3], y[3], z[3];
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const uint32_t idx = c0 + 64u * (uint32_t)u + lane;
                    id[u] = kFxNone;
                    mj[u] = 0xFFFFFFFFu;
                    x[u] = y[u] = z[u] = 1e9f;
                    if (idx < total) {
                        const uint32_t j = fx_stencil_atom(V, W, nseg, idx);
                        id[u] = j;
                        mj[u] = j / n;
                        x[u] = (float)fx_mi(V.pos[j] - ox, K.L, K.invL);
                        y[u] = (float)fx_mi(V.pos[N + j] - oy, K.L, K.invL);
                        z[u] = (float)fx_mi(V.pos[2 * N + j] - oz, K.L, K.invL);
                    }
                }
                for (uint32_t q = 0; q < cnt; ++q) {
                    const float qx = rl_f(ax, (int)q), qy = rl_f(ay, (int)q), qz = rl_f(az, (int)q);
                    const uint32_t qm = rl_u(mol, (int)q);
                    uint16_t* out = K.nbr + (size_t)rl_u(at, (int)q) * kFxNbr;
                    uint32_t k = rl_u(have, (int)q);
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        float dx = x[u] - qx, dy = y[u] - qy, dz = z[u] - qz;
                        if (fold) {
                            dx = fmaf(-Lf, rintf(dx * iLf), dx);
                            dy = fmaf(-Lf, rintf(dy * iLf), dy);
                            dz = fmaf(-Lf, rintf(dz * iLf), dz);
                        }
                        const bool keep = fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < K.list_r2 && mj[u] != qm;
                        const uint64_t bm = __ballot(keep);
                        const uint32_t at_k = k + rank_below(bm);
                        if (keep && at_k < kFxNbr) out[at_k] = (uint16_t)id[u];
                        k += (uint32_t)__popcll(bm);
                    }
                    if (lane == q) have = k;
                }
            }
            // pad the lists; mark those that did not fit
            for (uint32_t q = 0; q < cnt; ++q) {
                uint16_t* out = K.nbr + (size_t)rl_u(at, (int)q) * kFxNbr;
                const uint32_t k = rl_u(have, (int)q);
                if (k <= kFxNbr) {
                    if (lane >= k && lane < kFxNbr) out[lane] = (uint16_t)kFxNone;
                } else if (lane == 0) {
                    out[0] = (uint16_t)kFxOver;
                }
            }
        }
    }
}

// The attempts on up to 64 atoms of one cell (lane q holds atom q and its
// proposal), in order, by one wave.
//
// Up to four attempts are evaluated side by side against the present state, a
// row of 16 lanes for each atom that changes (one for a translation, two to
// four for a flip; a flip's rows stay together): a lane per listed neighbour,
// and on the first row of an attempt a lane per pair inside the molecule.
// They are then decided in order.  An accepted attempt voids those after it in
// the group that have a changed atom among their neighbours or in their own
// molecule; the next group starts from the first void one, so every decision
// is taken on the state its predecessors left, and dE does not depend on how
// the attempts were grouped.  With 7 - 30 % accepted about three of four
// stand.  The serial chain of a cell's attempts bounds the kernel (a system
// runs on one compute unit); a group costs little more than one attempt by
// the whole wave over the 27 cells' atoms did: a sweep of 1000 triangles at
// T = 0.75 went from 2.80 to 1.22 ms, of 333 tetrahedra from 7.4 to 2.2 ms.
__device__ __forceinline__ void fx_run_rows(const FxK& K, const FxView& V, uint32_t cnt,
                                            uint32_t at, const FxProp& pr, uint64_t sweep, bool logging,
                                            const FxWaveLds& W, FxCount& wc)
{
    const uint32_t lane = (uint32_t)__lane_id(), row = lane >> 4, rl = lane & 15u;
    const uint32_t n = K.n, N = K.N;
    const uint32_t base = n * (at / n);
    const bool mine = lane < cnt;
    const uint64_t flips = __ballot(mine && pr.flip != 0u);
    const uint64_t exits = __ballot(mine && pr.exited != 0u);
    wc.att_f += (uint32_t)__popcll(flips);
    wc.att_t += cnt - (uint32_t)__popcll(flips);
    wc.exits += (uint32_t)__popcll(exits);
    if (logging && mine && pr.exited) {
        MoveRecord rec;
        rec.delta_e = 0.0; rec.scale = 0.0; rec.t_log_u = pr.thr; rec.sweep = sweep;
        rec.molecule = at; rec.move = MC_TRANSLATE; rec.accepted = 0; rec.exited = 1;
        rec.axis = 255; rec.pair_terms = 0; rec.pad = 0;
        K.log[(sweep - K.log_sweep0) * N + at] = rec;
    }
    uint64_t live = (cnt >= 64u ? ~0ull : (1ull << cnt) - 1ull) & ~exits;
    // pair (i, j) inside the molecule on row lane 0 .. 5
    const uint32_t pi = rl < 3u ? 0u : (rl < 5u ? 1u : 2u);
    const uint32_t pj = rl < 3u ? rl + 1u : (rl < 5u ? rl - 1u : 3u);
    const bool pair_lane = rl < 6u && pj < n;
    while (live) {
        // ---- form a group: byte r of rows = attempt | atom of the molecule << 6
        uint32_t rows = 0, nrow = 0, natt = 0;
        uint32_t qa[4] = {0, 0, 0, 0}, r0[5] = {0, 0, 0, 0, 0};
        {
            uint64_t left = live;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (!left || natt != (uint32_t)g) continue;
                const uint32_t q = (uint32_t)__builtin_ctzll(left);
                uint32_t chg, need;
                if ((flips >> q) & 1u) {
                    chg = fx_pick(K.chg, rl_u(pr.kind, (int)q));
                    need = (uint32_t)__popc(chg);
                } else {
                    chg = 1u << (rl_u(at, (int)q) - rl_u(base, (int)q));
                    need = 1u;
                }
                if (nrow + need > 4u) continue;
                qa[g] = q;
                r0[g] = nrow;
#pragma unroll
                for (uint32_t t = 0; t < 4; ++t)
                    if ((chg >> t) & 1u) {
                        rows |= (q | (t << 6)) << (8u * nrow);
                        ++nrow;
                    }
                r0[g + 1] = nrow;
                natt = (uint32_t)g + 1u;
                left &= left - 1ull;
            }
        }
        // ---- the lanes' atoms and neighbours
        const bool act = row < nrow;
        const uint32_t info = act ? (rows >> (8u * row)) & 0xFFu : qa[0];
        const int ql = (int)(info & 63u);
        const uint32_t bl = (uint32_t)__shfl((int)base, ql), al = (uint32_t)__shfl((int)at, ql);
        const uint32_t kl = (uint32_t)__shfl((int)pr.kind, ql);
        const bool fl = kl != 255u;
        const uint32_t cl = fl ? bl + (info >> 6) : al;
        uint32_t j[3] = {kFxNone, kFxNone, kFxNone};
        if (K.nbr != nullptr && act) {
            const uint16_t* list = K.nbr + (size_t)cl * kFxNbr;
#pragma unroll
            for (int u = 0; u < 3; ++u) j[u] = list[16u * (uint32_t)u + rl];
        }
        // rows without a list (it did not fit, or the system has none)
        const uint32_t head = K.nbr != nullptr ? (uint32_t)__shfl((int)j[0], (int)(lane & 48u)) : kFxOver;
        const bool over = act && head == kFxOver;
        const double xo = V.pos[cl], yo = V.pos[N + cl], zo = V.pos[2 * N + cl];
        const double tx = __shfl(pr.tx, ql), ty = __shfl(pr.ty, ql), tz = __shfl(pr.tz, ql);
        const double mx = fl ? 0.0 : tx - xo, my = fl ? 0.0 : ty - yo, mz = fl ? 0.0 : tz - zo;
        const uint32_t perm = fx_pick(K.flipw, kl);
        const uint32_t to = V.type[cl];
        const uint32_t tn = fl ? (uint32_t)V.type[bl + ((perm >> (8u * (cl - bl))) & 0xFFu)] : to;
        double de = 0.0, sc = 0.0;
        uint32_t terms = 0;
        // ---- pairs with other molecules: separations after a translation are
        // those before it plus the displacement
        auto eval = [&](uint32_t jn, bool valid) __attribute__((always_inline)) {
            const uint32_t jj = valid ? jn : cl;
            const double xj = V.pos[jj], yj = V.pos[N + jj], zj = V.pos[2 * N + jj];
            const uint32_t tj = V.type[jj];
            const double s2o = W.s2ij[4u * to + tj], s2n = W.s2ij[4u * tn + tj];
            const double dx = fx_mi(xo - xj, K.L, K.invL), dy = fx_mi(yo - yj, K.L, K.invL),
                         dz = fx_mi(zo - zj, K.L, K.invL);
            const double ex = dx + mx, ey = dy + my, ez = dz + mz;
            const double r2o = dx * dx + dy * dy + dz * dz;
            const double r2n = ex * ex + ey * ey + ez * ez;
            const bool io = valid && r2o < K.rc2f * s2o, in = valid && r2n < K.rc2f * s2n;
            const double uo = fx_wca_in(s2o, r2o, io), un = fx_wca_in(s2n, r2n, in);
            de += un - uo;
            if (logging) sc += un + uo;
            terms += (io ? 1u : 0u) + (in ? 1u : 0u);
        };
        if (!__ballot(over)) {
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const bool valid = j[u] < kFxOver;
                if (u && !__ballot(valid)) break;  // wave-uniform
                eval(j[u], valid);
            }
        } else {
            // the 27 cells around the cell the atom was sorted into (every
            // cell once where they span the axis), a lane per atom
            const uint32_t nc = K.nc, span = min(nc, 3u);
            const uint32_t cid = V.cell_id[cl];
            const uint32_t ix = cid % nc, iy = (cid / nc) % nc, iz = cid / (nc * nc);
            const uint32_t listed = over ? 3u : 0u;
            for (uint32_t u = 0; u < 3u; ++u) {
                const uint32_t ju = u == 0 ? j[0] : (u == 1 ? j[1] : j[2]);
                eval(ju, !listed && ju < kFxOver);
            }
            for (uint32_t o = 0; o < span * span * span; ++o) {
                const uint32_t x = (ix + nc - 1u + o % span) % nc, y = (iy + nc - 1u + (o / span) % span) % nc,
                               z = (iz + nc - 1u + o / (span * span)) % nc;
                const uint32_t c = x + nc * (y + nc * z);
                const uint32_t cb = V.cell_start[c], ce = over ? V.cell_start[c + 1] : cb;
                for (uint32_t q = cb + rl; __ballot(q < ce); q += 16u) {
                    const uint32_t ja = q < ce ? V.cell_list[q] : cl;
                    eval(ja, q < ce && ja - bl >= n);
                }
            }
        }
        // ---- pairs inside the molecule that touch a changed atom, on the
        // attempt's first row
        {
            bool first = false;
#pragma unroll
            for (int g = 0; g < 4; ++g) first = first || ((uint32_t)g < natt && row == r0[g]);
            const uint32_t chg = fl ? fx_pick(K.chg, kl) : 1u << (cl - bl);
            const bool on = first && pair_lane && (((chg >> pi) | (chg >> pj)) & 1u);
            if (on) {
                const uint32_t ai = bl + pi, aj = bl + pj;
                const double dx = fx_mi(V.pos[ai] - V.pos[aj], K.L, K.invL),
                             dy = fx_mi(V.pos[N + ai] - V.pos[N + aj], K.L, K.invL),
                             dz = fx_mi(V.pos[2 * N + ai] - V.pos[2 * N + aj], K.L, K.invL);
                const double sg = ai == cl ? 1.0 : (aj == cl ? -1.0 : 0.0);  // m is 0 for a flip
                const double ex = fma(sg, mx, dx), ey = fma(sg, my, dy), ez = fma(sg, mz, dz);
                const double r2o = dx * dx + dy * dy + dz * dz;
                const double r2n = ex * ex + ey * ey + ez * ez;
                const uint32_t oi = V.type[ai], oj = V.type[aj];
                uint32_t ni = oi, nj = oj;
                if (fl) {
                    ni = V.type[bl + ((perm >> (8u * pi)) & 0xFFu)];
                    nj = V.type[bl + ((perm >> (8u * pj)) & 0xFFu)];
                }
                const double so = W.s2ij[4u * oi + oj], sn = W.s2ij[4u * ni + nj];
                const bool io = r2o < K.rc2f * so, in = r2n < K.rc2f * sn;
                const double uo = fx_wca_in(so, r2o, io), un = fx_wca_in(sn, r2n, in);
                de += un - uo;
                if (logging) sc += un + uo;
                terms += (io ? 1u : 0u) + (in ? 1u : 0u);
                if ((K.bonded >> (4u * pi + pj)) & 1u) {
                    // the change of Eq. (2) in one logarithm: the ratio of the
                    // arguments before and after; +inf at or beyond the limit
                    const double lo2 = 2.25 * so, ln2 = 2.25 * sn;
                    const bool fo = r2o < lo2, fn = r2n < ln2;
                    if (fo && fn)
                        de += -33.75 * log(((ln2 - r2n) * lo2) / ((lo2 - r2o) * ln2));
                    else
                        de += (fn ? 0.0 : __builtin_inf()) - (fo ? 0.0 : __builtin_inf());
                    terms += (fo ? 1u : 0u) + (fn ? 1u : 0u);
                    if (logging)
                        sc += fx_fene(W.sij[4u * oi + oj], r2o) + fx_fene(W.sij[4u * ni + nj], r2n);
                }
            }
        }
        // ---- decide in order
        const double rs = fx_row_sum(de);
        double ss = 0.0;
        uint32_t ts = 0;
        if (logging) {
            ss = fx_row_sum(sc);
            ts = fx_row_sum_u(terms);
        }
        uint32_t void_rows = 0, done_rows = 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if ((uint32_t)g >= natt) break;
            const uint32_t rb = r0[g], re = r0[g + 1];
            const uint32_t rmask = ((1u << re) - 1u) & ~((1u << rb) - 1u);
            if (void_rows & rmask) break;  // evaluated on a state that has changed since
            double dE = 0.0;
            for (uint32_t r = rb; r < re; ++r) dE += rl_d(rs, (int)(16u * r + 15u));
            const int q = (int)qa[g];
            const bool flip = (flips >> q) & 1u;
            const double thr = rl_d(pr.thr, q);
            const bool accept = (dE <= 0.0) || (thr < -dE);
            done_rows |= rmask;
            live &= live - 1ull;
            if (logging) {
                double S = 0.0;
                uint32_t tt = 0;
                for (uint32_t r = rb; r < re; ++r) {
                    S += rl_d(ss, (int)(16u * r + 15u));
                    tt += rl_u(ts, (int)(16u * r + 15u));
                }
                if ((int)lane == q) {
                    MoveRecord rec;
                    rec.delta_e = dE; rec.scale = S; rec.t_log_u = thr; rec.sweep = sweep;
                    rec.molecule = at; rec.move = flip ? MC_FLIP : MC_TRANSLATE; rec.accepted = accept ? 1 : 0;
                    rec.exited = 0; rec.axis = (uint8_t)pr.kind; rec.pair_terms = tt; rec.pad = 0;
                    K.log[(sweep - K.log_sweep0) * N + at] = rec;
                }
            }
            if (!accept) continue;
            wc.e += dE;
            if (flip) wc.acc_f += 1; else wc.acc_t += 1;
            if (rl == 0u && row >= rb && row < re) {
                if (flip) {
                    V.type[cl] = (uint8_t)tn;
                } else {
                    // wrapped as fx_wrap does; the shifts are the periodic
                    // images crossed
                    const double fx = floor(tx / K.L), fy = floor(ty / K.L), fz = floor(tz / K.L);
                    V.pos[cl] = tx - K.L * fx;
                    V.pos[N + cl] = ty - K.L * fy;
                    V.pos[2 * N + cl] = tz - K.L * fz;
                    if ((int)fx) K.img[cl] += (int)fx;
                    if ((int)fy) K.img[N + cl] += (int)fy;
                    if ((int)fz) K.img[2 * N + cl] += (int)fz;
                }
            }
            if ((uint32_t)g + 1u < natt) {
                // attempts after this one that a changed atom reaches
                bool hit = over || bl == rl_u(base, q);
                for (uint32_t r = rb; r < re; ++r) {
                    const uint32_t c = rl_u(cl, (int)(16u * r));
                    hit = hit || j[0] == c || j[1] == c || j[2] == c;
                }
                const uint64_t hb = __ballot(hit && row >= re && act);
#pragma unroll
                for (uint32_t r = 0; r < 4; ++r)
                    if ((hb >> (16u * r)) & 0xFFFFull) void_rows |= 1u << r;
            }
        }
        if ((done_rows >> row) & 1u) wc.terms += terms;
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
        const uint32_t b = start[c], cnt = start[c + 1] - b;
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
// positions, types and cell lists live in LDS for the whole launch (copied in
// at the start, positions and types written back at the end); otherwise the
// same code runs on the arrays in the system's buffer.
template <bool kRes>
__global__ void __launch_bounds__(kFxThreads) k_fx_sweeps(FxList list, uint64_t n_sweeps)
{
    FxDev* __restrict__ Dp = list.d[blockIdx.x];
    __shared__ uint32_t seg[kFxWaves][2][kFxSeg];
    __shared__ double pair_s[16], pair_s2[16];
    __shared__ uint32_t scratch[kFxWaves];
    __shared__ double misc[2];
    __shared__ double dmax2[kFxWaves];
    extern __shared__ __align__(16) unsigned char fx_smem[];
    const FxDev& D = *Dp;
    const FxK K = fx_const(D);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    FxWaveLds W{seg[wave][0], seg[wave][1], pair_s, pair_s2};
    Stats* st = D.stats;
    const uint32_t N = D.N, ncell = D.ncell, nc = D.nc, k = D.k;
    FxView V{D.pos, D.type, D.cell_start, D.cell_list, D.cell_id, D.ecell};
    if (kRes) {
        const FxLds l = fx_lds_layout(N, ncell);
        V = FxView{(double*)(fx_smem + l.pos), (uint8_t*)(fx_smem + l.type), (uint32_t*)(fx_smem + l.cstart),
                   (uint32_t*)(fx_smem + l.clist), (uint32_t*)(fx_smem + l.cid), (double*)(fx_smem + l.ecell)};
        for (uint32_t i = tid; i < 3 * N; i += kFxThreads) V.pos[i] = D.pos[i];
        for (uint32_t i = tid; i < N; i += kFxThreads) V.type[i] = D.type[i];
        __syncthreads();
    }
    const uint32_t na = nc / k, nact = na * na * na;
    uint64_t sweep = st->sweep;
    const uint64_t origin = st->obs_origin;
    if (tid == 0) misc[0] = st->e_acc;
    if (tid < 16) {
        const double sg = 0.5 * (fx_pick(K.sigma, (uint32_t)tid >> 2) + fx_pick(K.sigma, (uint32_t)tid & 3u));
        pair_s[tid] = sg;
        pair_s2[tid] = sg * sg;
    }
    FxCount wc{};
    for (uint64_t it = 0; it < n_sweeps; ++it) {
        const U4 g = philox10(0xFFFFFFFFu, (uint32_t)sweep, (uint32_t)(sweep >> 32), 3u, K.seed_lo, K.seed_hi);
        const double h[3] = {K.w * unit_open(g.x), K.w * unit_open(g.y), K.w * unit_open(g.z)};
        // counting sort of the atoms by cell
        for (uint32_t c = tid; c <= ncell; c += kFxThreads) V.cell_start[c] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < N; i += kFxThreads) {
            const uint32_t c = fx_cell(V.pos[i], V.pos[N + i], V.pos[2 * N + i], h, K);
            V.cell_id[i] = c;
            atomicAdd(&V.cell_start[c + 1], 1u);
        }
        __syncthreads();
        block_excl_scan_t<kFxThreads>(V.cell_start + 1, ncell, scratch);
        for (uint32_t i = tid; i < N; i += kFxThreads)
            V.cell_list[atomicAdd(&V.cell_start[V.cell_id[i] + 1], 1u)] = i;
        __syncthreads();
        fx_sort_cells(V.cell_list, V.cell_start, (uint32_t)wave, kFxWaves, ncell);
        __syncthreads();
        if (K.nbr != nullptr) {
            fx_build_lists(K, V, h, wave, ncell, W);
            __syncthreads();
        }
        const bool logging = D.log != nullptr && sweep - D.log_sweep0 < D.log_sweeps;
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
                    const uint32_t base = n * (V.cell_list[q] / n);
                    for (uint32_t i = 0; i + 1 < n; ++i)
                        for (uint32_t j = i + 1; j < n; ++j) {
                            const double dx = fx_mi(V.pos[base + i] - V.pos[base + j], K.L, K.invL);
                            const double dy = fx_mi(V.pos[N + base + i] - V.pos[N + base + j], K.L, K.invL);
                            const double dz =
                                fx_mi(V.pos[2 * N + base + i] - V.pos[2 * N + base + j], K.L, K.invL);
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
        // the attempts of cell `ci` of a colour by this wave
        auto run_cell = [&](uint32_t kx, uint32_t ky, uint32_t kz, uint32_t ci) __attribute__((always_inline)) {
            const uint32_t cell = (kx + k * (ci % na)) + nc * ((ky + k * ((ci / na) % na)) +
                                                              nc * (kz + k * (ci / (na * na))));
            wc.e = 0.0;
            const uint32_t b = V.cell_start[cell], e = V.cell_start[cell + 1];
            if (b < e) {
                for (uint32_t q0 = b; q0 < e; q0 += 64u) {
                    const uint32_t cnt = min(64u, e - q0);
                    uint32_t at = 0;
                    FxProp pr{};
                    if ((uint32_t)lane < cnt) {
                        at = V.cell_list[q0 + lane];
                        pr = fx_propose(K, V, at, sweep, h, cell);
                    }
                    fx_run_rows(K, V, cnt, at, pr, sweep, logging, W, wc);
                }
            }
            if (lane == 0) V.ecell[cell] = wc.e;
        };
        for (uint32_t col = 0; col < k * k * k; ++col) {
            const uint32_t kx = col % k, ky = (col / k) % k, kz = col / (k * k);
            if (colour_together(kx, ky, kz)) {
                for (uint32_t ci = (uint32_t)wave; ci < nact; ci += kFxWaves) run_cell(kx, ky, kz, ci);
                __syncthreads();
            } else {
                for (uint32_t ci = 0; ci < nact; ++ci) {
                    if (ci % kFxWaves == (uint32_t)wave) run_cell(kx, ky, kz, ci);
                    __syncthreads();
                }
            }
        }
        ++sweep;
        // E_acc += the sweep's dE, the cells in a fixed order; E/M samples
        if (wave == 0) {
            const double e = misc[0] + sweep_energy(V.ecell, ncell);
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
    if (lane == 0) {
        if (wc.att_t) atomicAdd((unsigned long long*)&st->attempts[MC_TRANSLATE], (unsigned long long)wc.att_t);
        if (wc.att_f) atomicAdd((unsigned long long*)&st->attempts[MC_FLIP], (unsigned long long)wc.att_f);
        if (wc.acc_t) atomicAdd((unsigned long long*)&st->accepts[MC_TRANSLATE], (unsigned long long)wc.acc_t);
        if (wc.acc_f) atomicAdd((unsigned long long*)&st->accepts[MC_FLIP], (unsigned long long)wc.acc_f);
        if (wc.exits) atomicAdd((unsigned long long*)&st->exits, (unsigned long long)wc.exits);
    }
    {
        uint64_t t = wc.terms;
#pragma unroll
        for (int o = 32; o; o >>= 1) t += (uint64_t)__shfl_xor((unsigned long long)t, o);
        if (lane == 0 && t) atomicAdd((unsigned long long*)&st->pair_terms, (unsigned long long)t);
    }
    __syncthreads();
    if (kRes) {
        for (uint32_t i = tid; i < 3 * N; i += kFxThreads) D.pos[i] = V.pos[i];
        for (uint32_t i = tid; i < N; i += kFxThreads) D.type[i] = V.type[i];
    }
    if (tid == 0) {
        st->sweep = sweep;
        st->e_acc = misc[0];
    }
}

}  // namespace
}  // namespace flipmc
