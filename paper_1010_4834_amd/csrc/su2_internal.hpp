// su2_internal.hpp -- kernel argument block and launcher declarations shared
// by the kernels (su2_kernels.hip) and the C-ABI host code (su2_api.hip).
#pragma once

#include "su2_device.hpp"

namespace su2 {

// Arguments common to the lattice kernels (passed by value).
struct KArgs {
    const LatDesc *desc;                 // per-lattice descriptors
    const Tile *tiles;                   // (lattice, first index) work list
    int ntiles;
    int xcd_remap;
    void *links;                         // native link buffer
    DevState *st;                        // seed / sweep counter
    unsigned int *err;                   // sampler try-cap hits (&st->err)
    uint32_t *trace;                     // per-link try record or null
    unsigned long long *tries_part;      // per-tile try counts
    double *plaq_part;                   // per-sweep-slot tile plaquette sums
    int sampler;                         // 0 hybrid, 1 Creutz
    int advance;                         // heat bath: substeps of whole sweeps (advance the counter)
    int nslots;                          // series slots of the partial buffers (0: no series)
    int every;                           // series: one measured sweep per `every` sweeps (>= 1)
    int tile_links;                      // heat bath: links per tile where four lanes share a link, else 0
};

// Largest number of sites, all lattices together, at which four lanes share a
// link (k_heatbath_split; single-link launch shapes); beta the smallest coupling.
// us per substep with one and with four lanes: Kennedy-Pendleton binary64 7.9 and
// 6.1 at 8192 sites, 8.1 and 6.7 at 32768, 8.0 and 8.3 at 57344; Creutz at beta 2.3
// binary32 12.8 and 6.9 at 4096, 14.3 and 9.2 at 98304, binary64 15.1 and 8.7, 17.2
// and 15.5.  A binary32 Kennedy-Pendleton try is too short to gain (4.1 and 4.2 at
// 8192).  The smaller beta, the fewer tries there are to share: Creutz binary32
// 5.7 and 6.1 at beta 0, 7.4 and 6.8 at beta 0.2 (98304 sites), 7.5 and 7.6 at beta
// 0.3, 9.4 and 8.2 at beta 1 (131072); binary64 7.3 and 7.9 at beta 0, 9.2 and 8.7 at
// beta 0.1 (65536), 9.9 and 12.0 at beta 0.5, 13.7 and 13.7 at beta 1.5 (98304);
// Kennedy-Pendleton binary64, which has Creutz tries there, 6.4 and 6.6 at beta 0,
// 8.5 and 7.3 at beta 0.3 (4096).
constexpr long long split_sites(bool f32, bool creutz, double beta) {
    if (!creutz) return f32 || beta < 0.1 ? 0 : 1LL << 15;
    if (f32) return beta < 0.1 ? 1LL << 16 : beta < 0.5 ? 98304 : 1LL << 17;
    return beta < 0.1 ? 1LL << 15 : beta < 1.5 ? 1LL << 16 : 98304;
}

// A call's sweeps of small lattices, one workgroup per lattice with its links
// in LDS (k_small_run), and whether four lanes share a link there.
// us per substep here and as replayed launches: Kennedy-Pendleton binary32 2.1
// and 3.3 (256 sites), 2.6 and 3.7 (1024); binary64 4.3 and 5.6 (256), 4.9 and
// 5.9 (512), 6.4 and 6.0 (768); over-relaxation binary32 1.3 and 2.4, 1.6 and
// 2.8, binary64 1.6 and 2.7, 2.3 and 3.6 (256, 1024).  Creutz, whose tries are
// many, with four lanes per link 4.0 and 5.3 (binary32, 256), 6.0 and 6.9
// (binary64, 256), with one 7.6 and 12.8; more links than threads for four
// lanes each stay with the launches.  Four lanes gain nothing for
// Kennedy-Pendleton (4.6 in binary64 at 256 sites).
constexpr int SMALL_SITES = 1024;  // largest lattice of any kind
constexpr int SMALL_BLOCK = 512;   // threads at most
constexpr int SMALL_FOUR = SMALL_BLOCK / 2;  // sites whose links have four lanes each
constexpr bool small_four(bool creutz, bool over) { return creutz && !over; }
constexpr int small_sites(bool f32, bool creutz, bool over) {
    return over ? SMALL_SITES : creutz ? SMALL_FOUR : f32 ? SMALL_SITES : SMALL_SITES / 2;
}
struct SmallRun {
    unsigned long long seed;
    unsigned int sweep0;   // Philox sweep word of the first sweep
    int nsweeps, over;     // over: over-relaxation instead of heat bath
    int every, nm;         // measured sweeps: every `every`-th, nm of them
};
size_t small_lds_bytes(bool f32, int sites);
// false: the launch shape is not available; errp (nullable): where a single
// lattice's error word goes.
bool launch_small_run(const KArgs &a, bool f32, int nlat, int sites, const SmallRun &r, double *outp, double *outl,
                      unsigned *errp, hipStream_t s);

// Optional timing events stamped by the launch itself (both null: none).
struct Ev {
    hipEvent_t a = nullptr, b = nullptr;
};

void launch_heatbath(const KArgs &a, bool f32, int mu, int par, int nl, int block, int grid, hipStream_t s,
                     bool trace, bool plaq, const Ev &ev = Ev{});
// Workgroups of `block` threads the heat-bath substep kernels keep resident
// per compute unit (the smallest over the four directions), 0 if unknown.
int heatbath_blocks_per_cu(bool f32, int nl, int block);
void launch_overrelax(const KArgs &a, bool f32, int mu, int par, int block, int grid, hipStream_t s,
                      const Ev &ev = Ev{});
void launch_init(const KArgs &a, bool f32, int hot, int block, int grid, hipStream_t s);
void launch_from_canon(const KArgs &a, bool f32, const double *canon, int block, hipStream_t s);
void launch_to_canon(const KArgs &a, bool f32, const void *src, int ndir, double *canon, int block,
                     hipStream_t s);
void launch_unit_defect(const KArgs &a, bool f32, unsigned long long *out, int block, hipStream_t s);
void launch_plaquette(const KArgs &a, bool f32, double *part, int block, int grid, hipStream_t s);
// Polyakov partials: one (hi, lo) pair per spatial tile; with a.nslots > 0
// they go to series slot ((sweep - run_base) / every) % nslots (2 * ntiles
// doubles per slot).
void launch_polyakov(const KArgs &a, bool f32, double *part, int block, int grid, hipStream_t s);
// The same measurements of a single lattice of at most ONE_TILES tiles in one
// launch: results and error word straight to mapped host memory.
constexpr int ONE_TILES = 2;
// The Polyakov loop so, and up to which Nt: two tiles' products of Nt links follow
// one another there, and in binary64 wait longer for their loads.  us a call and in
// two launches: 4^4 18 and 23 (both precisions); binary32 8 x 8 x 6 x 64 25.5 and 26.4,
// 8^3 x 128 33 and 31, x 1024 230 and 98, one tile 4^3 x 4096 263 and 277; binary64 8^3
// x 16 22.5 and 24.5, 8 x 8 x 6 x 64 36 and 29, 8^3 x 1024 582 and 135, one tile 2^3 x 64
// 25 and 26, 4^3 x 4096 1376 and 462.
constexpr bool polyakov_in_one(bool f32, int tiles, int Nt) {
    return tiles == 1 ? f32 || Nt <= 64 : tiles <= ONE_TILES && Nt <= (f32 ? 64 : 24);
}
void launch_plaquette_one(const KArgs &a, bool f32, int block, double *out, unsigned *err, hipStream_t s);
void launch_polyakov_one(const KArgs &a, bool f32, int block, double *out, unsigned *err, hipStream_t s);
// Final reduction of the standalone measurements: `chunks` workgroups per
// lattice, cnt[nlat] arrival tickets (zero between launches), chunk scratch
// of 6 doubles per workgroup.  pp: k_plaquette partials (4 per tile) ->
// outp[l * ostride + 0..2] = (avg, spatial, temporal); pl: Polyakov
// partials -> outl[l * ostride]; the error word -> err.
void launch_finalize(const LatDesc *desc, int nlat, int chunks, const double *pp, const double *pl,
                     unsigned *cnt, double *chunk, double *outp, double *outl, long long ostride, const DevState *st,
                     unsigned *err, hipStream_t s);
// Series values of nsw consecutive measured sweeps, slots slot0 .. slot0 +
// nsw - 1 (mod nslots): plaquette from the heat-bath partials (12 doubles
// per heat-bath tile per slot: 3 planes x 4 wavefronts, unused entries zero;
// slot stride pp_stride doubles) and Polyakov loop from the Polyakov
// partials (slot stride pl_stride); either may be null.  Two launches: C
// chunk sums per (lattice, sweep) into `chunk` (6 doubles each, nlat * nsw *
// C of them), then one fixed-order sum per (lattice, sweep) written to
// outp / outl[l * ostride + out0 + j] for sweep j of the batch.
void launch_series(const LatDesc *desc, int nlat, const double *pp, long long pp_stride, const double *pl,
                   long long pl_stride, int slot0, int nslots, int nsw, int C, double *chunk, double *outp,
                   double *outl, long long ostride, int out0, hipStream_t s);
// Seed, sweep word (also the `next` word) and series base of the device
// state, set by a one-thread kernel so that no host synchronisation is
// needed before the work that reads them (the error word is left alone).
void launch_set_state(DevState *st, unsigned long long seed, unsigned sweep, unsigned run_base, hipStream_t s);
void launch_set_state_mapped(DevState *st, const unsigned *src, hipStream_t s);
// Zero the error word.
void launch_clear_err(DevState *st, hipStream_t s);
// Copy the error word to `out` (mapped host memory).
void launch_err_to_host(const DevState *st, unsigned *out, hipStream_t s);
void launch_ape(const KArgs &a, bool f32, const void *src, int src_raw, void *dst, double alpha, int block,
                int grid, hipStream_t s);
// All steps in one launch, a workgroup per time slice of up to this many sites,
constexpr int ape_slice(bool f32) { return f32 ? 1024 : 512; }
// and whether that is the shorter way.  us here and as one launch per step: 2^3 x 64,
// 25 steps, 52 and 122 (binary32), 53 and 138; but 2^3 x 16384 288 and 154, 466 and
// 208: in a slice of fewer than 48 sites lanes idle, which many slices pay for (4^2 x 2
// x 4096, 2, 5 and 25 steps 22 and 21, 31 and 36, 88 and 155; 4 x 2^2 x 16384, 25 steps,
// 270 and 214).  Binary32 slices above 256 sites take more
// steps to pay for being loaded by one workgroup: 1024 sites x 64 times, 2, 5 and 25
// steps 22 and 19, 30 and 30, 86 and 128; a little so do slices that leave a quarter
// of their lanes idle (96 sites x 16384, 2 and 5 steps 76 and 71, 149 and 185).
constexpr bool ape_in_slices(bool f32, int ns, int nt, int nsteps) {
    if (ns > ape_slice(f32) || nsteps < 2) return false;
    if (ns < 48 && nt > (ns >= 24 && nsteps >= 5 ? 4096 : 64 * ns)) return false;
    return !f32 || nsteps >= (ns > 256 ? 5 : 4 * ns <= 3 * ((ns + 63) / 64 * 64) ? 3 : 2);
}
void launch_ape_slices(const KArgs &a, bool f32, int ns, int nt, const void *src, int src_raw, void *dst, double alpha,
                       int nsteps, hipStream_t s);
// Wilson loops: prefix products of the temporal links (times 0 .. next - 1),
// the spatial links and weights in that gauge, line by line, the loop traces of
// one pass of times (several passes beyond T = 16) and their final sums, written
// to mapped host memory with the error word.
constexpr int wl_ke(bool f32) { return f32 ? 8 : 6; }  // line elements per lane at most
struct WDir {             // split of one direction, see k_wloops
    int N, lines, XC, XE, G, TC, NB, ngrp, nxc, ntc, unit0;
};
struct WPlan {
    WDir d[3];
    int nunits, nel;            // units; LDS elements of the largest unit
    int block, grid, nc, lds;   // threads, workgroups, rows per lane, LDS bytes
    int toff, Tp, Tall;         // times toff < T <= toff + Tp of Tall
};
// Split of the times after toff, at most `step` (16, 8 or 4) of them; false if
// none fits the LDS.  The sums of a pass take 8 Rmax step bytes per wavefront,
// which at 16 times leaves no room for the lines from some Rmax on (cubes with Rmax
// their side: 82 sites in binary64, 112 in binary32; at 8 times 138 in binary64).
bool wloops_plan(bool f32, const int *n, int Rmax, int Tmax, int toff, int step, WPlan &out);
void launch_wgauge(const KArgs &a, bool f32, int ns, int next, void *P, hipStream_t s);
void launch_wlinks(const KArgs &a, bool f32, const int *n, const void *sp, int sp_raw, int next, const void *P, void *L,
                   void *w, hipStream_t s);
void launch_wloops(const KArgs &a, bool f32, const WPlan &p, int Rmax, int next, const void *L, const void *w,
                   double *part, hipStream_t s);
// The same by transport: the lines of every R <= Rmax (3 Rmax V quaternions),
// then the traces, wtrace_groups() partials per (R, T).
void launch_wlines(const KArgs &a, bool f32, long long V, const void *sp, int sp_raw, int Rmax, void *sl, int block,
                   hipStream_t s);
void launch_wtrace(const KArgs &a, bool f32, int Rmax, int Tmax, long long V, int Nt, const void *sl, double *part,
                   int block, hipStream_t s);
int wtrace_groups(long long V, int block);
// Whether a call goes by transport.
bool wloops_transport(bool f32, const int *n, int Rmax, int Tmax);
void launch_wfinal(const LatDesc *desc, int nparts, int Rmax, int Tmax, const double *part, double *out,
                   const DevState *st, unsigned *err, hipStream_t s);

}  // namespace su2
