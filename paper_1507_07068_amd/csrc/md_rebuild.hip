// Task 1 of the MD step on gfx950: skin test and Verlet-list rebuild.  Included by
// md_kernels.hip.
//
//   k_decide        one block, a wavefront per replica: skin test (Section 2.6) -> rebuild flags
//   k_bin           wrap periodic coordinates, cell of every atom / carbon, cell counts (with a
//                   single replica each block takes the skin decision itself, no k_decide)
//   k_scan          exclusive scan of all cell counts (one pass, decoupled look-back)
//   k_scatter       atom slots / carbon indices into their cells at the ranks k_bin took
//                   (arbitrary order within a cell), with the (cell, id) sort keys; marks
//                   the 27-cell stencil of every occupied carbon cell; lists the list build's
//                   work items (list_items)
//   k_sort_gather   one lane per slot: rank within its cell by (cell, id), gather the atom
//                   state into sorted order (so the final order is canonical); atoms in a
//                   marked carbon cell join the near list
//   k_rebuild       those four as phases of one launch (small systems)
//   k_list_bricks   one block per work item, a brick of cells (md_bricks.hpp) or part of a crowded
//                   one: the brick's window is staged in LDS, each atom scans its nine cell rows
//                   of it; copies the sorted state back.  Its leading blocks build the Cr-C lists (xlist_pass: one
//                   wavefront per near atom).  k_list_rows (one lane per atom from global
//                   memory, for periodic axes with fewer than 3 cells) is followed by
//                   k_xlist, the same Cr-C pass as a launch of its own.
//   k_inner_pos, k_mid_check, k_mid_list, k_inner_list   two-tier lists: the inner lists refilled
//                   every step from the outer ones, by way of middle lists where those pay
//
// Every build kernel after the decision returns at once when no replica needs a rebuild, so
// a step without a rebuild costs a few empty launches.
#pragma once

#include <type_traits>

#include "md_bricks.hpp"
#include "md_device.hpp"

namespace md {

struct BuildArgs {
  const RepDesc* R;
  RepState* S;
  const int* tile_rep;   // [ntiles]
  int4* items;           // [ntot] the list build's work items: replica, brick of it, first and last + 1
                         // of the brick's centers (null: k_list_rows builds the lists)
  int* nitems;           // their number
  int* nbk;              // bricks of all replicas, each the work item of its number (0: more than
                         // there is room for, and empty ones have no item)
  const int* c_rep;      // [ctot] replica of each carbon
  int* any;              // 1 if some replica rebuilds in this step
  int* abort;            // sticky: a bounded wait of a build gave up; no build runs until
                         // md_clear_flags (which also zeroes the cell counts it left behind)
  double4* q;
  double* v;
  double* f;
  uint8_t* fixed;
  int* id;
  const double* xc;
  double* xref;
  int* cellid;           // [ntot] cell of each atom slot
  int* crank;            // [ntot] rank of the slot among the atoms binned into its cell
  int* perm;             // [ntot] slots by cell (cells in order, arbitrary order within one)
  long long* skey;       // [ntot] (cell, id) sort key of perm's entries
  double4* tq;
  float4* tqf;           // [ntot] sorted positions relative to the replica's grid origin, FP32
  int4* qs;              // [ntot] fixed-point cell-local shadow of q (x, y, z, F' bits)
  long long* bcell;      // [ntot] build cell of each atom slot (pack_cell)
  double* tv;
  double* tf;
  uint8_t* tfixed;
  int* tid;
  int* count;            // [ncell_all]
  int* start;            // [ncell_all + 1]
  int* hcell;            // [ctot]
  int* hrank;            // [ctot] rank of the carbon among those binned into its cell
  int* hlist;            // [ctot] carbons by cell (arbitrary order within a cell)
  double4* hsorted;      // [ctot] carbons by cell, ascending index within a cell: position at
                         // zero indenter displacement, the carbon's index (as bits) in .w
  long long* scan_state; // [scan_blocks] published chunk sums of k_scan
  int* scan_ticket;      // chunk ticket of k_scan
  int* sync;             // k_rebuild's counters, zero between builds
  int* hnear;            // [carbon cells]: the cell has a carbon in its 27-cell stencil
  int* idx;
  int* cnt;
  int* xidx;
  int* xcnt;
  int* near;             // [ntot]: replica r's near atoms at near[a0_r ...]
  double* fme;           // [ntot][4]: last Morse force and energy per atom (0 if none)
  int ncell_all, ncell_cr, ntiles, ctot;
  const int* bt_rep;     // [nbt] replica of each group of bricks (several replicas only)
  int nbt;               // groups of bricks (see list_items)
  int parts;             // blocks that share a work item in the list build
  int nbin;              // tile blocks' worth of work of k_bin, k_scatter, k_sort_gather: the Cr
                         // tiles, then 256-carbon groups (the grids stride over them)
  int nrb;               // k_rebuild's work items: nbin, and more for the bricks and the scan
  int near_blocks;       // grid of k_xlist
  int xblocks;           // leading blocks of k_list_bricks that build the Cr-C lists (0: none)
  int commit_ref;        // k_scan records the indenter position of this build (k_bin decided)
  int copy_f;            // the forces are permuted with the atoms (0 inside md_run: no kick reads
                         // them before the next force pass that stores them)
  int scan_chunk, scan_blocks;
  int spin_limit;        // polls of k_scan's look-back before it gives up (< 0: at once)
};

constexpr int MAXC = 512;           // candidates staged per window in k_xlist
#ifndef MD_SG_KEYS
#define MD_SG_KEYS 8
#endif
constexpr int SG_KEYS = MD_SG_KEYS;   // keys of a cell k_sort_gather loads at a time
constexpr int WAVES_PER_BLOCK = BLOCK / WAVE;
#ifndef MD_LIST_WAVES
#define MD_LIST_WAVES 6
#endif
#ifndef MD_LIST_GROUP
#define MD_LIST_GROUP 4
#endif
constexpr int LIST_GROUP = MD_LIST_GROUP;   // candidates screened together per atom in k_list_bricks
static_assert(LIST_STAGE % LIST_GROUP == 0, "whole groups");
static_assert(LIST_GROUP >= 1 && LIST_GROUP <= 32, "a group's passing bits fit the 32-bit mask k_list_bricks appends from");


__device__ __forceinline__ bool rebuild_off(const BuildArgs& A) { return *A.any == 0; }

// One block of DECIDE_THREADS decides every replica (skin test, then the cell grid of the
// build) and ORs the outcomes into the launch-wide flag: the whole block per replica when
// there are few, else a group of lanes per replica (up to a wavefront; see below).
constexpr int DECIDE_THREADS = 1024;
constexpr int DECIDE_BLOCKWIDE = 4;   // replicas up to which the whole block takes each one

// Per-replica part of k_decide.  Reduce(v, op) reduces over the threads that share the
// replica (a wavefront or the block); `lead` marks the thread that writes.
// Skin test (Section 2.6) and cell grid of replica r, the same in every thread that calls it
// (every thread of the block calls it together: maxr is a block or wavefront reduction).
struct BuildGrid {
  int need;
  double glo[3], ginv[3], gedge[3], qscale;
  int gd[3];
};
// The replica's parts are entries first .. first + count - 1 of dmax_tile / tile_box.
template <class MaxReduce>
__device__ __forceinline__ BuildGrid decide_grid(const Consts& K, const BuildArgs& A, int r,
                                                 const double* dmax_tile, const double* tile_box, int force,
                                                 int first, int count, int t0, int tstep, MaxReduce maxr) {
  const RepDesc& d = A.R[r];
  const RepState& s = A.S[r];
  BuildGrid g;
  double m = 0.0;
#pragma unroll 8
  for (int t = t0; t < count; t += tstep) m = fmax(m, dmax_tile[first + t]);   // loads together
  m = maxr(m);
  g.need = !*A.abort && (force || (m > K.half_skin_sq) || (fabs(s.ind_z - s.ind_z_ref) > K.half_skin));
  if (!g.need) return g;   // uniform over the threads of the replica
  // cell grid of this build: the box along periodic axes, the atoms' extent along open ones
  for (int a = 0; a < 3; ++a) {
    if (d.per[a]) {
      g.glo[a] = d.lo[a];
      g.ginv[a] = d.ginv[a];
      g.gedge[a] = d.len[a] / d.gcap[a];
      g.gd[a] = d.gcap[a];
      continue;
    }
    double mn = INFINITY, mx = -INFINITY;
#pragma unroll 4
    for (int t = t0; t < count; t += tstep) {
      mn = fmin(mn, tile_box[6 * (int64_t)(first + t) + a]);
      mx = fmax(mx, tile_box[6 * (int64_t)(first + t) + 3 + a]);
    }
    mn = -maxr(-mn);
    mx = maxr(mx);
    if (!(mn <= mx)) {   // no atoms (or non-finite positions): fall back to the box
      mn = d.lo[a];
      mx = d.lo[a] + d.len[a];
    }
    const double edge = K.rlist * (1.0 + 1e-9);
    const double ext = fmax(mx - mn, edge);
    const int gc = (int)fmin(fmax(floor(ext / edge), 1.0), (double)d.gcap[a]);
    g.glo[a] = mn;
    g.ginv[a] = gc / ext;
    g.gedge[a] = ext / gc;
    g.gd[a] = gc;
  }
  // shadow scale: the longest cell edge spans at most 2^29 units
  const double emax = fmax(g.gedge[0], fmax(g.gedge[1], g.gedge[2]));
  g.qscale = ldexp(1.0, 29 - (int)ceil(log2(emax)));
  return g;
}

// Records the outcome in the replica's state (one thread).
__device__ __forceinline__ void record_grid(const Consts& K, const RepDesc& d, RepState& s, const BuildGrid& g) {
  s.rebuild = g.need;
  if (!g.need) return;
  choose_bricks(d.n, d.bcap, g.gd, s.bn);
  for (int a = 0; a < 3; ++a) s.bq[a] = g.gd[a] / s.bn[a];
  s.mid_ok = 0;
  s.nnear_old = s.nnear;
  s.nnear = 0;
  for (int a = 0; a < 3; ++a) {
    s.glo[a] = g.glo[a];
    s.ginv[a] = g.ginv[a];
    s.gedge[a] = g.gedge[a];
    s.gd[a] = g.gd[a];
  }
  s.qscale = g.qscale;
  // FP32 screen of the list build: r2f, the squared separation from FP32 coordinates relative to
  // the grid origin (with the image shift), decides the pair when it lies outside
  // [rl2 - delta, rl2 + delta); pairs inside that band get the exact FP64 test.  With u = 2^-24,
  // coordinates within E of the origin and a periodic length L, each separation component
  // carries an error of at most eta = u (3E + 2L + 3R) for |component| <= R = r_list + 1, so
  // |r2f - r2| <= sum over axes of (2 R eta + eta^2) + 4 u (rl2 + R^2); delta is twice that.
  // Pairs farther than R apart are far outside the band.
  const double u = 0x1p-24, R = K.rlist + 1.0;
  double err = 4.0 * u * (K.rlist_sq + R * R);
  for (int a = 0; a < 3; ++a) {
    const double E = g.gd[a] / g.ginv[a] + 2.0 * R;
    const double eta = u * (3.0 * E + (d.per[a] ? 2.0 * d.len[a] : 0.0) + 3.0 * R);
    err += 2.0 * R * eta + eta * eta;
  }
  const double delta = 2.0 * err + 1e-6;
  s.scr_lo = (float)(K.rlist_sq - delta);
  s.scr_hi = (float)(K.rlist_sq + delta);
}

// The list build's work items before any brick is split (one thread).
__device__ __forceinline__ void number_items(const Consts& K, const BuildArgs& A, int bricks) {
  const int nbk = bricks + K.ntot / BRICK_NT <= K.ntot ? bricks : 0;
  *A.nbk = nbk;
  *A.nitems = nbk;
}

template <class MaxReduce>
__device__ __forceinline__ bool decide_replica(const Consts& K, BuildArgs& A, int r, const double* dmax_tile,
                                               const double* tile_box, int force, int ppt, int t0, int tstep,
                                               bool lead, MaxReduce maxr) {
  const BuildGrid g = decide_grid(K, A, r, dmax_tile, tile_box, force, A.R[r].t0 * ppt, A.R[r].nt * ppt, t0,
                                  tstep, maxr);
  if (lead) record_grid(K, A.R[r], A.S[r], g);
  return g.need;
}

__global__ __launch_bounds__(DECIDE_THREADS) void k_decide(Consts K, BuildArgs A,
                                                           const double* __restrict__ dmax_tile,
                                                           const double* __restrict__ tile_box, int force,
                                                           int ppt) {
  __shared__ int any_sh;
  if (threadIdx.x == 0) any_sh = 0;
  __syncthreads();
  if (K.nrep <= DECIDE_BLOCKWIDE) {
    for (int r = 0; r < K.nrep; ++r) {
      const bool need = decide_replica(K, A, r, dmax_tile, tile_box, force, ppt, threadIdx.x, DECIDE_THREADS,
                                       threadIdx.x == 0, [](double v) { return block_max<DECIDE_THREADS>(v); });
      if (need && threadIdx.x == 0) any_sh = 1;
    }
  } else {
    // groups of G lanes (a power of two, G <= 64), as many as there are replicas up to
    // 1024 / G: group g takes replicas g, g + 1024 / G, ... (so the replicas' loads go out
    // together rather than a wavefront's replicas one after another)
    int G = WAVE;
    while (G > 1 && (DECIDE_THREADS / G) < K.nrep) G >>= 1;
    const int sub = threadIdx.x % G, grp = threadIdx.x / G, ng = DECIDE_THREADS / G;
    for (int r0 = 0; r0 < K.nrep; r0 += ng) {   // (uniform: every group steps together)
      const int r = r0 + grp;
      const bool mine = r < K.nrep;
      // groups past the last replica repeat replica 0's decision without recording it
      const bool need = decide_replica(K, A, mine ? r : 0, dmax_tile, tile_box, force, ppt, sub, G,
                                       mine && sub == 0, [G](double v) {
                                         for (int o = G / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, WAVE));
                                         return v;
                                       });
      if (need && mine && sub == 0) atomicOr(&any_sh, 1);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) *A.any = any_sh;
  if (any_sh) {   // launch-wide numbering of the bricks
    int carry = 0;
    if (K.nrep <= WAVE) {
      if (threadIdx.x < WAVE) {
        const int r = threadIdx.x, c = r < K.nrep ? brick_count(A.S[r].bn) : 0, incl = wave_scan(c);
        if (r < K.nrep) A.S[r].bk0 = incl - c;
        carry = __shfl(incl, WAVE - 1, WAVE);
      }
    } else {
      for (int r0 = 0; r0 < K.nrep; r0 += DECIDE_THREADS) {
        const int r = r0 + threadIdx.x;
        int tot;
        const int ex = block_exclusive_scan<DECIDE_THREADS>(r < K.nrep ? brick_count(A.S[r].bn) : 0, &tot);
        if (r < K.nrep) A.S[r].bk0 = carry + ex;
        carry += tot;
      }
    }
    if (threadIdx.x == 0) number_items(K, A, carry);
  }
  for (int r = threadIdx.x; r < K.nrep; r += DECIDE_THREADS) {   // builds are counted here
    RepState& s = A.S[r];
    if (s.rebuild) {
      s.nbuilds += 1;
      s.ind_z_ref = s.ind_z;
    }
  }
}

__device__ __forceinline__ int cr_cell_of(const RepDesc& d, const RepState& s, double x, double y, double z) {
  int cx = cell_coord(x, s.glo[0], s.ginv[0], s.gd[0]);
  int cy = cell_coord(y, s.glo[1], s.ginv[1], s.gd[1]);
  int cz = cell_coord(z, s.glo[2], s.ginv[2], s.gd[2]);
  return d.g0 + (cz * s.gd[1] + cy) * s.gd[0] + cx;
}

// Coordinate folded into [lo, lo + len) on a periodic axis (binning of carbons only).
__device__ __forceinline__ double fold(double x, double lo, double len, int per) {
  if (!per) return x;
  return x - len * floor((x - lo) / len);
}

__device__ __forceinline__ void c_cell_coords(const RepDesc& d, double x, double y, double z, int& hx,
                                              int& hy, int& hz) {
  hx = cell_coord(fold(x, d.lo[0], d.len[0], d.per[0]), d.lo[0], d.hinv[0], d.hd[0]);
  hy = cell_coord(fold(y, d.lo[1], d.len[1], d.per[1]), d.lo[1], d.hinv[1], d.hd[1]);
  hz = cell_coord(fold(z, d.lo[2], d.len[2], d.per[2]), d.lo[2], d.hinv[2], d.hd[2]);
}

// Rank of this lane's atom among the atoms binned into cell `cid`: consecutive lanes with
// the same cell (the common case, atoms arrive in the previous build's cell order) form a
// run that takes its ranks with one atomic add.  Every lane of the wave calls it together.
__device__ __forceinline__ int bin_rank(int* count, int cid, bool live) {
  const int lane = threadIdx.x % WAVE;
  const int key = live ? cid : -1;
  const int prev = __shfl_up(key, 1, WAVE);
  const bool head = live && (lane == 0 || prev != key);
  const unsigned long long heads = __ballot(head);
  const unsigned long long stops = __ballot(head || !live);   // first lane of the next run
  const unsigned long long upto = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
  const unsigned long long below = heads & upto;                // heads at lanes <= lane
  const int start = below ? 63 - __builtin_clzll(below) : 0;
  int base = 0;
  if (head) {
    const unsigned long long after = stops & ~upto;
    const int end = after ? __builtin_ctzll(after) : WAVE;
    base = atomicAdd(&count[cid], end - lane);
  }
  base = __shfl(base, start, WAVE);
  return base + (lane - start);
}

// The nparts per-part displacement maxima and boxes of a single replica reduced to
// gridDim.x partial ones in the same layout (block b takes a contiguous chunk): the
// maximum, the minima and the maxima of each axis (the neutral values where a chunk is
// empty).  The skin decision then reads those few instead of every part.
__global__ __launch_bounds__(BLOCK) void k_parts_reduce(const double* __restrict__ dmax_tile,
                                                        const double* __restrict__ tile_box, int nparts,
                                                        double* __restrict__ dmax_out,
                                                        double* __restrict__ box_out) {
  const int chunk = (nparts + gridDim.x - 1) / gridDim.x;
  const int p0 = blockIdx.x * chunk, p1 = min(p0 + chunk, nparts);
  // the maximum, then per axis the negated minimum and the maximum
  double v[7] = {0.0, -INFINITY, -INFINITY, -INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int p = p0 + threadIdx.x; p < p1; p += BLOCK) {
    v[0] = fmax(v[0], dmax_tile[p]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[1 + a] = fmax(v[1 + a], -tile_box[6 * (int64_t)p + a]);
      v[4 + a] = fmax(v[4 + a], tile_box[6 * (int64_t)p + 3 + a]);
    }
  }
  block_max_to0<BLOCK, 7>(v);
  if (threadIdx.x == 0) {
    dmax_out[blockIdx.x] = v[0];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      box_out[6 * blockIdx.x + a] = -v[1 + a];
      box_out[6 * blockIdx.x + 3 + a] = v[4 + a];
    }
  }
}

// The skin decision and the cell grid of a single replica without a forced build, taken by every
// block of a launch alike from the nparts per-part maxima and boxes (or their partial reductions
// by k_parts_reduce; so no separate decision launch).
__device__ __forceinline__ BuildGrid decide_alike(const Consts& K, const BuildArgs& A,
                                                  const double* __restrict__ dmax_tile,
                                                  const double* __restrict__ tile_box, int nparts) {
  return decide_grid(K, A, 0, dmax_tile, tile_box, 0, 0, nparts, threadIdx.x, BLOCK,
                     [](double v) { return block_max<BLOCK>(v); });
}

// Records that decision (one thread of the launch).  The indenter reference position, which every
// block reads for the decision, is recorded once no block can read it any more (k_scan, or the
// end of k_rebuild).
__device__ __forceinline__ void record_alike(const Consts& K, const BuildArgs& A, const BuildGrid& g1) {
  RepState& s0 = A.S[0];
  record_grid(K, A.R[0], s0, g1);
  *A.any = g1.need;
  if (g1.need) {
    s0.nbuilds += 1;
    s0.bk0 = 0;
    number_items(K, A, brick_count(s0.bn));
  }
}

// Work item b of the binning: b < ntiles, a tile of Cr atoms; else 256 carbons.  DECIDE: with the
// grid just decided (its record may be under way).
template <bool DECIDE>
__device__ __forceinline__ void bin_item(const Consts& K, const BuildArgs& A, const BuildGrid& g1, int b) {
  if (b < A.ntiles) {
    const int r = A.tile_rep[b];
    if (!DECIDE && !A.S[r].rebuild) return;
    const RepDesc& d = A.R[r];
    const int64_t i = (int64_t)b * TILE + threadIdx.x;
    const bool live = i < (int64_t)d.a0 + d.n;
    int cid = -1;
    if (live) {
      double4 p = A.q[i];
      double xyz[3] = {p.x, p.y, p.z};
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (!d.per[a]) continue;
        const double hi = d.lo[a] + d.len[a];
        if (xyz[a] >= hi)
          xyz[a] -= d.len[a];
        else if (xyz[a] < d.lo[a])
          xyz[a] += d.len[a];
      }
      p.x = xyz[0];
      p.y = xyz[1];
      p.z = xyz[2];
      if (DECIDE) {   // the grid just decided (block 0 may be recording it meanwhile)
        const int cx = cell_coord(p.x, g1.glo[0], g1.ginv[0], g1.gd[0]);
        const int cy = cell_coord(p.y, g1.glo[1], g1.ginv[1], g1.gd[1]);
        const int cz = cell_coord(p.z, g1.glo[2], g1.ginv[2], g1.gd[2]);
        cid = d.g0 + (cz * g1.gd[1] + cy) * g1.gd[0] + cx;
      } else {
        cid = cr_cell_of(d, A.S[r], p.x, p.y, p.z);   // before the stores (which could alias S)
      }
      A.q[i] = p;
      A.cellid[i] = cid;
    }
    const int rank = bin_rank(A.count, cid, live);
    if (live) A.crank[i] = rank;
  } else {
    const int64_t k = (int64_t)(b - A.ntiles) * BLOCK + threadIdx.x;
    int r = -1;
    if (k < A.ctot) {
      r = A.c_rep[k];
      if (!DECIDE && !A.S[r].rebuild) r = -1;
    }
    if (r >= 0) {
      const RepDesc& d = A.R[r];
      const double z = A.xc[3 * k + 2] + A.S[r].ind_z;
      int hx, hy, hz;
      c_cell_coords(d, A.xc[3 * k + 0], A.xc[3 * k + 1], z, hx, hy, hz);
      const int hid = d.h0 + (hz * d.hd[1] + hy) * d.hd[0] + hx;
      A.hcell[k] = hid;
      A.hrank[k] = atomicAdd(&A.count[hid], 1);
    }
  }
}

// Blocks stride over the binning's work items.  DECIDE: every block takes the decision first;
// block 0 records it.
template <bool DECIDE>
__global__ __launch_bounds__(BLOCK) void k_bin(Consts K, BuildArgs A, const double* __restrict__ dmax_tile,
                                               const double* __restrict__ tile_box, int nparts) {
  BuildGrid g1;
  if (DECIDE) {
    g1 = decide_alike(K, A, dmax_tile, tile_box, nparts);
    if (blockIdx.x == 0 && threadIdx.x == 0) record_alike(K, A, g1);
    if (!g1.need) return;
  } else if (rebuild_off(A)) {
    return;
  }
  if (blockIdx.x == 0) {   // fresh state for this build's k_scan
    for (int t = threadIdx.x; t < A.scan_blocks; t += BLOCK) A.scan_state[t] = 0;
    if (threadIdx.x == 0) *A.scan_ticket = 0;
  }
  for (int b = blockIdx.x; b < A.nbin; b += gridDim.x) bin_item<DECIDE>(K, A, g1, b);   // (b uniform over the block)
}

// Exclusive scan of all cell counts in one launch: each block scans SCAN_CHUNK cells and
// finds the sum of the chunks before it by looking back over the published chunk states
// (single-pass scan with decoupled look-back, Merrill and Garland 2016).  Chunks are
// taken in ticket order, so a block only waits for blocks that are already running; the
// wait is bounded and a timeout is reported in the status words.
constexpr int SCAN_PER_THREAD = 8;
constexpr long long SCAN_AGG = 1ll << 32, SCAN_INCL = 2ll << 32;

// Chunk b (blocks take them in ascending order).
__device__ __forceinline__ void scan_chunk(const BuildArgs& A, int b) {
  __shared__ int excl_sh;
  const int c0 = b * A.scan_chunk + threadIdx.x * SCAN_PER_THREAD;
  int v[SCAN_PER_THREAD];
  int sum = 0;
#pragma unroll
  for (int u = 0; u < SCAN_PER_THREAD; ++u) {
    v[u] = (c0 + u < A.ncell_all) ? A.count[c0 + u] : 0;
    sum += v[u];
  }
  int tot;
  const int pre = block_exclusive_scan(sum, &tot);
  // wave 0 publishes this chunk and looks back 64 chunks at a time.  A published word holds
  // both the flag and the sum, and nothing else a chunk writes is read before the next
  // launch, so the atomics are relaxed (agent scope): a release or acquire here would write
  // back or invalidate the per-XCD L2 at every publication and poll.
  if (threadIdx.x < WAVE) {
    const int lane = threadIdx.x;
    long long* st = A.scan_state;
    int excl = 0;
    if (b == 0) {
      if (lane == 0)
        __hip_atomic_store(&st[0], SCAN_INCL | (unsigned)tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      if (lane == 0)
        __hip_atomic_store(&st[b], SCAN_AGG | (unsigned)tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int top = b - 1, spins = 0;
      while (true) {
        const int j = top - lane;   // lane 0 is the nearest predecessor; j < 0 reads as prefix 0
        const long long w =
            j >= 0 ? __hip_atomic_load(&st[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : SCAN_INCL;
        const long long flag = w & ~0xffffffffll;
        const unsigned long long incl = __ballot(flag == SCAN_INCL);
        const unsigned long long ready = __ballot(flag != 0);
        const int first = incl ? __builtin_ctzll(incl) : WAVE;   // nearest inclusive prefix
        const unsigned long long need = first < WAVE ? ((2ull << first) - 1ull) : ~0ull;
        if ((ready & need) != need || A.spin_limit < 0) {   // some chunk in between has not published yet
          if (++spins > A.spin_limit) {
            // give up: this build is invalid.  The later build kernels of this step see no
            // rebuild (so nothing is scattered with a wrong prefix), and no build runs until
            // md_clear_flags.
            if (lane == 0) {
              A.S[0].sync_timeout = 1;
              *A.abort = 1;
              *A.any = 0;
            }
            break;
          }
          __builtin_amdgcn_s_sleep(1);
          continue;
        }
        excl += wave_sum(lane <= first ? (int)(unsigned)(w & 0xffffffffll) : 0);
        if (first < WAVE) break;
        top -= WAVE;
      }
      if (lane == 0)
        __hip_atomic_store(&st[b], SCAN_INCL | (unsigned)(excl + tot), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) {
      excl_sh = excl;
      if (b == A.scan_blocks - 1) A.start[A.ncell_all] = excl + tot;
    }
  }
  __syncthreads();
  int run = excl_sh + pre;
#pragma unroll
  for (int u = 0; u < SCAN_PER_THREAD; ++u) {
    if (c0 + u < A.ncell_all) {
      A.start[c0 + u] = run;
      if (c0 + u >= A.ncell_cr) A.hnear[c0 + u - A.ncell_cr] = 0;
    }
    run += v[u];
  }
}

__global__ __launch_bounds__(BLOCK) void k_scan(BuildArgs A) {
  if (rebuild_off(A)) return;
  __shared__ int chunk_sh;
  if (threadIdx.x == 0) chunk_sh = atomicAdd(A.scan_ticket, 1);
  __syncthreads();
  const int b = chunk_sh;
  if (A.commit_ref && b == 0 && threadIdx.x == 0) {   // k_bin decided: this build's indenter position
    RepState& s0 = A.S[0];
    s0.ind_z_ref = s0.ind_z;
  }
  scan_chunk(A, b);
}

// The list build's work items of group j of the bricks: as many for a brick as let a block's threads
// take an item's centers at once.  Bricks are cut for the replica's mean density, and with vacuum in
// its grid (a film with a gap above it, a cluster, atoms far from a surface) most are empty and the
// others hold several blocks' worth of centers.  A brick's first item has the brick's number, so that
// neighbouring bricks run at the same time and find their windows in the caches (in the order of an
// atomic counter the build over 14 A cells takes 1.13 of the time), and the rest follow after all
// bricks.  Where there are more bricks than room for that, only the items with centers are placed, by
// the counter (no more of them than atoms).  LG lanes count a brick's centers, a cell row each.
// Forced builds with one item per brick and with these: a 216k-atom slab in a periodic box of four
// times its height 155 and 108 us, twenty atoms 200 A above it 157 and 112, a cluster of 75k atoms in
// a box of 500 A 180 and 113; films without vacuum the same (the list kernel's blocks read an item in
// place of a count).
constexpr int BRICK_GROUP = 32;   // bricks per group
__device__ __forceinline__ void list_items(const Consts& K, const BuildArgs& A, int j) {
  constexpr int LG = BLOCK / BRICK_GROUP, ROWS = (BRICK_MAX * BRICK_MAX + LG - 1) / LG;
  const int r = K.nrep == 1 ? 0 : A.bt_rep[j];
  const RepDesc& d = A.R[r];
  const RepState& S = A.S[r];
  const int nb = brick_count(S.bn), sub = threadIdx.x % LG, own = *A.nbk > 0 ? 1 : 0;
  const int gx = S.gd[0], gy = S.gd[1];
  for (int l0 = (j - d.bt0) * BRICK_GROUP; l0 < nb; l0 += d.nbt * BRICK_GROUP) {   // uniform over the block
    const int lb = l0 + threadIdx.x / LG;
    int m = 0;
    if (lb < nb && S.rebuild) {
      const int iyz = lb / S.bn[0], ix = lb - iyz * S.bn[0], iz = iyz / S.bn[1], iy = iyz - iz * S.bn[1];
      const int x0 = brick_first(ix, S.bq[0], gx, S.bn[0]), x1 = brick_first(ix + 1, S.bq[0], gx, S.bn[0]);
      const int y0 = brick_first(iy, S.bq[1], gy, S.bn[1]), ny = brick_first(iy + 1, S.bq[1], gy, S.bn[1]) - y0;
      const int z0 = brick_first(iz, S.bq[2], S.gd[2], S.bn[2]);
      const int rows = ny * (brick_first(iz + 1, S.bq[2], S.gd[2], S.bn[2]) - z0);
      const float inv = 1.0f / (float)ny;
      int from[ROWS], to[ROWS];
#pragma unroll
      for (int j = 0; j < ROWS; ++j) {   // all loads together (past the last row: that row's)
        const int t = min(sub + j * LG, rows - 1), rz = (int)(((float)t + 0.5f) * inv);
        const int* st = A.start + d.g0 + ((z0 + rz) * gy + y0 + (t - rz * ny)) * gx;
        from[j] = st[x0];
        to[j] = st[x1];
      }
#pragma unroll
      for (int j = 0; j < ROWS; ++j) m += sub + j * LG < rows ? to[j] - from[j] : 0;
    }
#pragma unroll
    for (int o = LG / 2; o > 0; o >>= 1) m += __shfl_xor(m, o, WAVE);
    if (sub != 0 || lb >= nb) m = 0;
    const int k = (m + BRICK_NT - 1) / BRICK_NT, more = max(k - own, 0);
    int at = 0;
    if (__any(more > 0)) {   // (no brick of most films)
      const int incl = wave_scan(more);
      if (threadIdx.x % WAVE == WAVE - 1) at = atomicAdd(A.nitems, incl);
      at = __shfl(at, WAVE - 1, WAVE) + incl - more;
    }
    if (sub == 0 && lb < nb) {
      if (own) A.items[S.bk0 + lb] = make_int4(r, lb, 0, k ? m / k : 0);
      for (int j = own; j < k; ++j)
        A.items[at++] = make_int4(r, lb, (int)((long long)m * j / k), (int)((long long)m * (j + 1) / k));
    }
  }
}

// Work item b of the scatter into cell order, as bin_item.
__device__ __forceinline__ void scatter_item(const Consts& K, const BuildArgs& A, int b) {
  if (b < A.ntiles) {
    const int r = A.tile_rep[b];
    if (!A.S[r].rebuild) return;
    const RepDesc& d = A.R[r];
    const int64_t i = (int64_t)b * TILE + threadIdx.x;
    if (i >= (int64_t)d.a0 + d.n) return;
    const int cid = A.cellid[i];
    const int pos = d.a0 + (A.start[cid] - A.start[d.g0]) + A.crank[i];
    A.perm[pos] = (int)i;
    A.skey[pos] = ((long long)cid << 32) | (unsigned)A.id[i];
    // the Cr-C records (force, energy) are nonzero only at near-list slots: zeroing those of
    // the previous build's near list (lane k takes entry k) leaves every record zero, and the
    // Cr-C pass rewrites the new near atoms' records
    const int64_t k = i - d.a0;
    if (k < A.S[r].nnear_old) {
      const int64_t pn = A.near[d.a0 + k];
      A.fme[4 * pn + 0] = 0.0;
      A.fme[4 * pn + 1] = 0.0;
      A.fme[4 * pn + 2] = 0.0;
      A.fme[4 * pn + 3] = 0.0;
    }
  } else {
    const int64_t k = (int64_t)(b - A.ntiles) * BLOCK + threadIdx.x;
    if (k >= A.ctot) return;
    const int r = A.c_rep[k];
    if (!A.S[r].rebuild) return;
    const RepDesc& d = A.R[r];
    const int hid = A.hcell[k];
    const int rank = A.hrank[k];
    A.hlist[d.c0 + (A.start[hid] - A.start[d.h0]) + rank] = (int)k;
    if (rank == 0) {
      // one carbon per occupied carbon cell: every cell of its stencil can hold Cr atoms
      // within reach of a carbon (k_scan cleared the marks).  The descriptor is read into
      // registers first: a store could alias it and would make every read after it wait.
      const int h0 = d.h0, hd0 = d.hd[0], hd1 = d.hd[1], hd2 = d.hd[2];
      const int p0 = d.per[0], p1 = d.per[1], p2 = d.per[2];
      int* __restrict__ hn = A.hnear + (h0 - A.ncell_cr);
      const int lc = hid - h0;
      const int hx = lc % hd0, hy = (lc / hd0) % hd1, hz = lc / (hd0 * hd1);
      const int msx = stencil_n(hd0, p0), msy = stencil_n(hd1, p1), msz = stencil_n(hd2, p2);
      for (int tz = 0; tz < msz; ++tz) {
        const int z = stencil_cell(hz, tz, hd2, p2);
        for (int ty = 0; ty < msy; ++ty) {
          const int y = stencil_cell(hy, ty, hd1, p1);
          for (int tx = 0; tx < msx; ++tx) {
            const int x = stencil_cell(hx, tx, hd0, p0);
            if (x >= 0 && y >= 0 && z >= 0) hn[(z * hd1 + y) * hd0 + x] = 1;
          }
        }
      }
    }
  }
}

__global__ __launch_bounds__(BLOCK) void k_scatter(Consts K, BuildArgs A) {
  if (rebuild_off(A)) return;
  for (int b = blockIdx.x; b < A.nbt + A.nbin; b += gridDim.x) {   // (b uniform over the block)
    if (b < A.nbt) list_items(K, A, b);
    else scatter_item(K, A, b - A.nbt);
  }
}

// One lane per slot in cell order.  Work item b < ntiles: a tile of Cr slots; else 256 carbon
// slots.  A slot's final position is the start of its cell
// plus the number of atoms of that cell with a smaller (cell, id) key (cells hold a few
// atoms), so the final order is canonical; the atom's state is gathered there.
__device__ __forceinline__ void sort_item(const Consts& K, const BuildArgs& A, int b) {
  if (b < A.ntiles) {
    const int r = A.tile_rep[b];
    RepState& S = A.S[r];
    if (!S.rebuild) return;
    const RepDesc& d = A.R[r];
    const int u = b * TILE + threadIdx.x;
    bool near = false;
    int p = 0;
    if (u < d.a0 + d.n) {
      const long long key = A.skey[u];
      const int c = (int)(key >> 32);
      const int sbase = d.a0 - A.start[d.g0];
      const int s0 = sbase + A.start[c], s1 = sbase + A.start[c + 1];
      const int e = A.perm[u];
      int rank = 0;
      // SG_KEYS independent key loads at a time: the index is clamped into the cell (which
      // holds this atom) rather than the load made conditional, so that no load waits on
      // the one before it
      for (int t = s0; t < s1; t += SG_KEYS) {
        long long kk[SG_KEYS];
#pragma unroll
        for (int u = 0; u < SG_KEYS; ++u) kk[u] = A.skey[min(t + u, s1 - 1)];
#pragma unroll
        for (int u = 0; u < SG_KEYS; ++u) rank += (t + u < s1 && kk[u] < key) ? 1 : 0;
      }
      if (u == s0) A.count[c] = 0;   // zero again for the next rebuild
      p = s0 + rank;
      // the atom's state, each value stored as it arrives (measured faster here than all
      // loads first)
      const double4 qe = A.q[e];
      A.tq[p] = qe;
      A.tqf[p] = make_float4((float)(qe.x - S.glo[0]), (float)(qe.y - S.glo[1]), (float)(qe.z - S.glo[2]), 0.0f);
      A.tv[3 * p + 0] = A.v[3 * e + 0];
      A.tv[3 * p + 1] = A.v[3 * e + 1];
      A.tv[3 * p + 2] = A.v[3 * e + 2];
      if (A.copy_f) {
        A.tf[3 * p + 0] = A.f[3 * e + 0];
        A.tf[3 * p + 1] = A.f[3 * e + 1];
        A.tf[3 * p + 2] = A.f[3 * e + 2];
      }
      A.tfixed[p] = A.fixed[e];
      A.tid[p] = A.id[e];
      // no Cr-C list until the Cr-C list build of this rebuild says otherwise (k_scatter
      // zeroed the Cr-C records)
      A.xcnt[p] = 0;
      if (d.nc > 0) {   // in the stencil of an occupied carbon cell: the atom gets a Cr-C list
        int hx, hy, hz;
        c_cell_coords(d, qe.x, qe.y, qe.z, hx, hy, hz);
        near = A.hnear[d.h0 - A.ncell_cr + (hz * d.hd[1] + hy) * d.hd[0] + hx] != 0;
      }
    }
    const int lane = threadIdx.x % WAVE;
    const unsigned long long nm = __ballot(near);
    if (nm) {   // append this wave's near atoms (order within the near list is irrelevant)
      const int lead = __builtin_ctzll(nm);
      int first = 0;
      if (lane == lead) first = atomicAdd(&S.nnear, __popcll(nm));
      first = __shfl(first, lead, WAVE);
      if (near) A.near[d.a0 + first + __popcll(nm & ((1ull << lane) - 1ull))] = p;
    }
  } else {
    const int64_t u = (int64_t)(b - A.ntiles) * BLOCK + threadIdx.x;
    if (u >= A.ctot) return;
    const int r = A.c_rep[u];   // carbon slots of a replica are its carbon index range
    if (!A.S[r].rebuild) return;
    const RepDesc& d = A.R[r];
    const int e = A.hlist[u];
    const int c = A.hcell[e];
    const int hb = d.c0 - A.start[d.h0];
    const int s0 = hb + A.start[c], s1 = hb + A.start[c + 1];
    int rank = 0;
    for (int t = s0; t < s1; t += SG_KEYS) {   // SG_KEYS independent loads at a time (as above)
      int hh[SG_KEYS];
#pragma unroll
      for (int u = 0; u < SG_KEYS; ++u) hh[u] = A.hlist[min(t + u, s1 - 1)];
#pragma unroll
      for (int u = 0; u < SG_KEYS; ++u) rank += (t + u < s1 && hh[u] < e) ? 1 : 0;
    }
    A.hsorted[s0 + rank] = make_double4(A.xc[3 * e + 0], A.xc[3 * e + 1], A.xc[3 * e + 2],
                                        __longlong_as_double((long long)e));
    if (u == s0) A.count[c] = 0;   // zero again for the next rebuild
  }
}

__global__ __launch_bounds__(BLOCK) void k_sort_gather(Consts K, BuildArgs A) {
  if (rebuild_off(A)) return;
  for (int b = blockIdx.x; b < A.nbin; b += gridDim.x) sort_item(K, A, b);   // (b uniform over the block)
}

// k_bin, k_scan, k_scatter and k_sort_gather in one launch, for systems of few work items
// (at most REBUILD_ITEMS; at most REBUILD_CHUNKS chunks of cells).  The holders of the items scan the
// chunks and list the bricks' work items too, so there are more items than the binning's: one per
// group of bricks, and as many as chunks (250 atoms strewn over 400 A, 419 chunks: 1.39 ms a forced build with one
// item, 116 us with 48; four launches 57 us, but 18 against 12 us a step without a rebuild).  A step without a rebuild, most of a run's, then pays for one launch
// that finds nothing to do in place of four (about 2 us each, beside passes of 8 to 20 us).
// Blocks take the binning's items from a counter and keep them for the later phases, each of
// which waits for the end of the one before: only blocks that hold items keep another back, and
// those run, so the waits end whichever of the launch's blocks have been placed (they are bounded
// all the same).  The fences around a wait carry the phase's stores to every XCD.
enum { SY_TAKEN = 0, SY_BIN, SY_SCAN, SY_SCATTER, SY_LEFT, SY_WORDS };
constexpr int SYNC_STRIDE = 16;                      // a counter to a 64-byte line
constexpr int SYNC_INTS = SY_WORDS * SYNC_STRIDE;
constexpr int PHASE_SPINS = 1 << 22;
// A build's phases in one launch take 21 us at 8 items, as the four launches do, but 36 at 41
// and 46 at 64, where the waits cost more than launches.  Films of 100 steps, this against the
// four launches: 1,024 atoms 0.89 of the time (cold) and 0.94 (melting, a rebuild every few
// steps), 8,192 atoms 0.90 and 0.97, 16,000 0.96 and 1.06.
constexpr int REBUILD_ITEMS = 48;
constexpr int REBUILD_CHUNKS = 512;

// Counts the block's `mine` items of a phase of `items` and waits for the others' (false: given
// up, as a scan that does; scan: or one of its chunks did).
__device__ __forceinline__ bool phase_end(const BuildArgs& A, int* done, int mine, int items, bool scan = false) {
  __shared__ int ok_sh;
  const bool alone = gridDim.x == 1;   // (a system of one item: no other block's stores to wait for)
  if (!alone) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");   // each thread's stores of this phase
  __syncthreads();
  if (threadIdx.x == 0) {
    if (mine && !alone) atomicAdd(done, mine);
    int spins = 0;
    bool ok = true;
    while (ok && !alone && __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < items) {
      if (++spins > PHASE_SPINS) {
        A.S[0].sync_timeout = 1;
        *A.any = 0;
        __hip_atomic_store(A.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = false;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    if (ok && scan) ok = __hip_atomic_load(A.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
    ok_sh = ok ? 1 : 0;
  }
  __syncthreads();
  if (!alone) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the other blocks' stores
  const bool ok = ok_sh != 0;
  __syncthreads();   // (ok_sh is free again)
  return ok;
}

template <bool DECIDE>
__global__ __launch_bounds__(BLOCK) void k_rebuild(Consts K, BuildArgs A, const double* __restrict__ dmax_tile,
                                                   const double* __restrict__ tile_box, int nparts) {
  BuildGrid g1;
  if (DECIDE) {
    g1 = decide_alike(K, A, dmax_tile, tile_box, nparts);
    if (!g1.need) {
      if (blockIdx.x == 0 && threadIdx.x == 0) record_alike(K, A, g1);
      return;
    }
  } else if (rebuild_off(A)) {
    return;
  }
  __shared__ int own[REBUILD_ITEMS + 1];   // this block's items, ascending
  int n = 0;
  while (true) {
    if (threadIdx.x == 0) own[n] = atomicAdd(A.sync + SY_TAKEN * SYNC_STRIDE, 1);
    __syncthreads();
    const int b = own[n];
    if (b >= A.nrb) break;
    ++n;
    if (b == 0) {   // (the record and the scan's fresh state are part of the phase)
      if (DECIDE && threadIdx.x == 0) record_alike(K, A, g1);
      for (int t = threadIdx.x; t < A.scan_blocks; t += BLOCK) A.scan_state[t] = 0;
    }
    bin_item<DECIDE>(K, A, g1, b);
  }
  if (!phase_end(A, A.sync + SY_BIN * SYNC_STRIDE, n, A.nrb)) return;
  // the scan's chunks go to the holders of the items of the same number (modulo their count); a
  // holder takes its chunks in ascending order, so the lowest unfinished one is always under way
  int chunks = 0;
  for (int c0 = 0; c0 < A.scan_blocks; c0 += A.nrb)
    for (int k = 0; k < n; ++k)
      if (c0 + own[k] < A.scan_blocks) {
        scan_chunk(A, c0 + own[k]);
        __syncthreads();   // (the chunk's shared words are free again)
        ++chunks;
      }
  // (a scan that gave up: nothing is scattered, and the counters stay until md_clear_flags)
  if (!phase_end(A, A.sync + SY_SCAN * SYNC_STRIDE, chunks, A.scan_blocks, true)) return;
  for (int k = 0; k < n; ++k) {
    // (the groups of bricks to the items past the binning's first, which have nothing to scatter)
    for (int j = own[k] >= A.nbin ? own[k] - A.nbin : own[k] - A.nbin + A.nrb; j < A.nbt; j += A.nrb) list_items(K, A, j);
    scatter_item(K, A, own[k]);
  }
  if (!phase_end(A, A.sync + SY_SCATTER * SYNC_STRIDE, n, A.nrb)) return;
  for (int k = 0; k < n; ++k) sort_item(K, A, own[k]);
  // the last block to leave, when every block has decided and looked for its last item, records
  // the indenter position and clears the counters for the next build
  if (threadIdx.x == 0 && atomicAdd(A.sync + SY_LEFT * SYNC_STRIDE, 1) == (int)gridDim.x - 1) {
    if (A.commit_ref) A.S[0].ind_z_ref = A.S[0].ind_z;
    for (int t = 0; t < SYNC_INTS; t += SYNC_STRIDE) A.sync[t] = 0;
  }
}

// Cr-Cr lists, one lane per sorted Cr atom.  The candidates of the atom are those of the
// cells around its own: nine cell rows (y, z), each holding x-cells cx-1 .. cx+1, which are
// one contiguous range of the sorted order (two where the row wraps around a periodic x
// axis).  Entries are written rows in order (z-major), along x, then by slot, at the
// interleaved positions the tpa lanes of the force passes read.  Along a periodic axis with
// >= 3 cells the periodic image of a candidate is fixed by the cell it comes from
// (separation + 0 or -+ length: the same rounding as the minimum image for every pair
// inside the list radius); along a periodic axis with fewer cells each cell is visited once
// and the minimum image is taken pair by pair.
__global__ __launch_bounds__(BLOCK) void k_list_rows(Consts K, BuildArgs A) {
  if (rebuild_off(A)) return;
  const int T = K.lt;
  const int tile = blockIdx.x;
  const int r = A.tile_rep[tile];
  RepState& S = A.S[r];
  if (!S.rebuild) return;
  const RepDesc& d = A.R[r];
  const int p = tile * TILE + threadIdx.x;
  const bool live = p < d.a0 + d.n;
  const int cap = K.cap;
  if (live) {
    const double4 pi = A.tq[p];
    const int gx = S.gd[0], gy = S.gd[1], gz = S.gd[2];
    const int cx = cell_coord(pi.x, S.glo[0], S.ginv[0], gx);
    const int cy = cell_coord(pi.y, S.glo[1], S.ginv[1], gy);
    const int cz = cell_coord(pi.z, S.glo[2], S.ginv[2], gz);
    const int sbase = d.a0 - A.start[d.g0];   // sorted slot = sbase + start[cell]
    const double rl2 = K.rlist_sq;
    const double4* __restrict__ tq = A.tq;
    // entry k at idx[(k / T) * row + k % T]: wp walks the slots in entry order
    const int64_t row = K.ntot * T;
    int* __restrict__ wp = A.idx + (int64_t)p * T;
    // pairwise minimum image on periodic axes with fewer than 3 cells
    const bool mx = d.per[0] && gx < 3, my = d.per[1] && gy < 3, mz = d.per[2] && gz < 3;
    // x segments (first cell, last cell, shift), the same for every row
    int xa0 = cx - 1, xb0 = cx + 1, xa1 = 0, xb1 = -1;
    double sh0 = 0.0, sh1 = 0.0;
    if (mx) {
      xa0 = 0;
      xb0 = gx - 1;
    } else if (d.per[0]) {
      if (cx == 0) {
        xa0 = gx - 1; xb0 = gx - 1; sh0 = -d.len[0];
        xa1 = 0; xb1 = 1;
      } else if (cx == gx - 1) {
        xa0 = gx - 2; xb0 = gx - 1;
        xa1 = 0; xb1 = 0; sh1 = d.len[0];
      }
    } else {
      xa0 = max(xa0, 0);
      xb0 = min(xb0, gx - 1);
    }
    const int nsy = stencil_n(gy, d.per[1]), nsz = stencil_n(gz, d.per[2]);
    int count = 0;
    auto append = [&](int j) {
      if (count < cap) *wp = j;
      ++count;
      wp += (count & (T - 1)) ? 1 : row - (T - 1);
    };
    for (int rr = 0; rr < 9; ++rr) {
      const int tz = rr / 3, ty = rr % 3;
      if (tz >= nsz || ty >= nsy) continue;
      const int z = stencil_cell(cz, tz, gz, d.per[2]);
      const int y = stencil_cell(cy, ty, gy, d.per[1]);
      if (z < 0 || y < 0) continue;
      const int uz = cz + tz - 1, uy = cy + ty - 1;   // unwrapped row (image shift)
      const double shz = (d.per[2] && !mz) ? (uz < 0 ? -d.len[2] : (uz >= gz ? d.len[2] : 0.0)) : 0.0;
      const double shy = (d.per[1] && !my) ? (uy < 0 ? -d.len[1] : (uy >= gy ? d.len[1] : 0.0)) : 0.0;
      const int crow = d.g0 + (z * gy + y) * gx;
      for (int sg = 0; sg < 2; ++sg) {
        const int xa = sg ? xa1 : xa0, xb = sg ? xb1 : xb0;
        if (xb < xa) continue;
        const double shx = sg ? sh1 : sh0;
        const int j0 = sbase + A.start[crow + xa], j1 = sbase + A.start[crow + xb + 1];
        auto exact = [&](int j) {
          const double4 pj = tq[j];
          double ex = pj.x - pi.x, ey = pj.y - pi.y, ez = pj.z - pi.z;
          ex = mx ? min_image(ex, d.len[0], d.half[0], 1) : ex + shx;
          ey = my ? min_image(ey, d.len[1], d.half[1], 1) : ey + shy;
          ez = mz ? min_image(ez, d.len[2], d.half[2], 1) : ez + shz;
          return dist_sq_exact(ex, ey, ez) < rl2;
        };
        for (int j = j0; j < j1; ++j)
          if (j != p && exact(j)) append(j);
      }
    }
    A.cnt[p] = min(count, cap);
    if (count > cap) atomicMax(&S.overflow, count);
    {
      // copy-back of the sorted state, all loads before the first store
      const double v0 = A.tv[3 * p + 0], v1 = A.tv[3 * p + 1], v2 = A.tv[3 * p + 2];
      const bool cf = A.copy_f;
      const double f0 = cf ? A.tf[3 * p + 0] : 0.0, f1 = cf ? A.tf[3 * p + 1] : 0.0, f2 = cf ? A.tf[3 * p + 2] : 0.0;
      const uint8_t fx = A.tfixed[p];
      const int ide = A.tid[p];
      A.q[p] = pi;
      if (K.shadow) {
        const long long bc = pack_cell(cx, cy, cz);
        A.bcell[p] = bc;
        A.qs[p] = cell_local(S, bc, pi.x, pi.y, pi.z, (float)pi.w);
      }
      A.xref[3 * p + 0] = pi.x;
      A.xref[3 * p + 1] = pi.y;
      A.xref[3 * p + 2] = pi.z;
      A.v[3 * p + 0] = v0;
      A.v[3 * p + 1] = v1;
      A.v[3 * p + 2] = v2;
      if (cf) {
        A.f[3 * p + 0] = f0;
        A.f[3 * p + 1] = f1;
        A.f[3 * p + 2] = f2;
      }
      A.fixed[p] = fx;
      A.id[p] = ide;
    }
  }
}

// Cr-C list {k : |xc_k + ind_z - q_p|^2 < (rc + skin)^2}, atom-major: xidx[p * xcap + n],
// for the atoms of the near list of each rebuilding replica.  One wavefront per near atom
// (stride over those of all rebuilding replicas), its lanes sharing the 27 carbon cells
// around the atom; the passing carbons are compacted in candidate order with a ballot.  Runs
// in blocks bid of nb blocks of NT threads; cand and pre are the block's LDS scratch
// (NT / WAVE x MAXC slots, XL_FLAT_MAXREP + 1 prefixes).  Reads the sorted positions
// (tq) and the near list written by k_sort_gather, so it may run beside the Cr-Cr list build.
constexpr int XL_FLAT_MAXREP = FLAT_MAXREP - 1;   // replicas of the flattened index space
template <int NT>
__device__ __forceinline__ void xlist_pass(const Consts& K, const BuildArgs& A, int (*cand_sh)[MAXC], int* pre,
                                           int bid, int nb) {
  const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
  const int gw = bid * (NT / WAVE) + w, nw = nb * (NT / WAVE);
  auto one = [&](int r, int item) {   // near atom `item` of replica r, on this wavefront
    RepState& S = A.S[r];
    const RepDesc& d = A.R[r];
    const double iz = S.ind_z;
    const int hbase = A.start[d.h0];
    const int msx = stencil_n(d.hd[0], d.per[0]), msy = stencil_n(d.hd[1], d.per[1]),
              msz = stencil_n(d.hd[2], d.per[2]);
    const int ms = msx * msy * msz;
    const int64_t pa = A.near[d.a0 + item];
    const double4 pi = A.tq[pa];
    int hx, hy, hz;
    c_cell_coords(d, pi.x, pi.y, pi.z, hx, hy, hz);
    int ks = 0, kn = 0;
    if (lane < ms) {
      const int tx = lane % msx, ty = (lane / msx) % msy, tz = lane / (msx * msy);
      const int x = stencil_cell(hx, tx, d.hd[0], d.per[0]);
      const int y = stencil_cell(hy, ty, d.hd[1], d.per[1]);
      const int z = stencil_cell(hz, tz, d.hd[2], d.per[2]);
      if (x >= 0 && y >= 0 && z >= 0) {
        const int hid = d.h0 + (z * d.hd[1] + y) * d.hd[0] + x;
        ks = d.c0 + (A.start[hid] - hbase);
        kn = A.start[hid + 1] - A.start[hid];
      }
    }
    int pref = kn;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int y = __shfl_up(pref, o, WAVE);
      if (lane >= o) pref += y;
    }
    const int total = __shfl(pref, WAVE - 1, WAVE);
    pref -= kn;
    int n = 0;
    for (int w0 = 0; w0 < total; w0 += MAXC) {
      const int lo = max(0, w0 - pref), hi = min(kn, w0 + MAXC - pref);
      for (int e = lo; e < hi; ++e) cand_sh[w][pref + e - w0] = ks + e;   // sorted carbon slots
      wave_sync();
      const int wn = min(MAXC, total - w0);
      for (int k0 = 0; k0 < wn; k0 += WAVE) {
        bool pred = false;
        int k = 0;
        if (k0 + lane < wn) {
          const double4 c4 = A.hsorted[cand_sh[w][k0 + lane]];
          k = (int)__double_as_longlong(c4.w);
          const double ex = min_image(c4.x - pi.x, d.len[0], d.half[0], d.per[0]);
          const double ey = min_image(c4.y - pi.y, d.len[1], d.half[1], d.per[1]);
          const double ez = min_image((c4.z + iz) - pi.z, d.len[2], d.half[2], d.per[2]);
          pred = dist_sq_exact(ex, ey, ez) < K.rxlist_sq;
        }
        const unsigned long long m2 = __ballot(pred);
        const int below = __popcll(m2 & ((1ull << lane) - 1ull));
        if (pred && n + below < K.xcap) A.xidx[pa * K.xcap + n + below] = k;
        n += __popcll(m2);
      }
      wave_sync();
    }
    if (lane == 0) {
      A.xcnt[pa] = min(n, K.xcap);
      if (n > K.xcap) atomicMax(&S.xoverflow, n);
    }
  };
  if (K.nrep <= XL_FLAT_MAXREP) {   // near atoms of all rebuilding replicas as one index space
    const int total = flat_prefix<NT>(K.nrep, pre, [&](int r) { return A.S[r].rebuild ? A.S[r].nnear : 0; });
    for (int g = gw; g < total; g += nw) {
      const int r = flat_replica(pre, K.nrep, g);
      one(r, g - pre[r]);
    }
  } else {
    for (int r = 0; r < K.nrep; ++r) {
      if (!A.S[r].rebuild) continue;
      for (int item = gw; item < A.S[r].nnear; item += nw) one(r, item);
    }
  }
}

// Cr-Cr lists over bricks (replicas whose periodic axes all have >= 3 list cells).  A block
// takes a work item (a brick, or up to BRICK_NT of a crowded one's centers; see list_items) or one
// of `parts` shares of its centers, stages the brick's window in LDS as
// FP32 coordinates relative to the grid origin plus the image shift of the row and of the piece
// across an x face, with the slot in the fourth word, and gives every center one lane.  A
// center's candidates in one of its nine neighbouring cell rows (z-major, then y), x-cells
// cx-1 .. cx+1, are a contiguous range of window positions, so the candidate order (rows, along
// x, by slot) is the same as in k_list_rows and the lists are identical.  An FP32 screen decides
// all but a band around the list radius, which gets the exact FP64 test (see record_grid).
//
// A window over LIST_STAGE atoms is staged in pieces of that size.  Where a block's centers leave
// threads over (large cells, a share of a brick), the lanes of a center take its candidates in
// runs and place their entries after a prefix over the lanes.
//
// Bound by VALU work (0.86 of the issue slots on the 8M-atom film, 0.82 on the 1M-atom one; the
// screen and the append loop), with the partly filled lines of the entry stores behind it.  Against
// one block per run of cells of a single cell row, which staged nine windows' worth of atoms per
// center instead of 3.4 and had one lane per center (this kernel in forced builds of films with
// 0.05 A of noise, us): 8M atoms 1303 against 1413, 1M 168 against 201, 216k 47 against 65, with
// the paper's form 402 against 623, its outer lists 1407 against 4165, the 10k-atom film of the
// paper's protocol 55 against 185, a 2k-atom bulk 18 against 34.  Held to 6 wavefronts per SIMD (three blocks per compute unit): at 5
// two blocks fit and the 8M film takes 1.55 ms, at 7 or 8 the registers spill (1.46).

// Image shift (FP64) along an axis of an unwrapped cell coordinate u of a grid of g cells.
__device__ __forceinline__ double cell_shift(int u, int g, int per, double len) {
  return per ? (u < 0 ? -len : (u >= g ? len : 0.0)) : 0.0;
}

__global__ __launch_bounds__(BRICK_NT, MD_LIST_WAVES) void k_list_bricks(Consts K, BuildArgs A) {
  if (rebuild_off(A)) return;
  // staged candidates: x, y, z, slot bits (a group may read past the last)
  __shared__ float4 sq[LIST_STAGE + LIST_GROUP];
  __shared__ BrickTab tab;
  __shared__ int toff[BRICK_ROWS][BRICK_CELLS];   // per row: window position of cells x0-1 .. x1+2
  __shared__ float2 rsh[BRICK_ROWS];              // per row: FP32 image shift along y and z
  __shared__ int csh[BRICK_NT], psh[BRICK_NT];    // the centers' counts and slots
  static_assert(sizeof(sq) >= sizeof(int) * (BRICK_NT / WAVE * MAXC + XL_FLAT_MAXREP + 1),
                "the Cr-C list blocks work in the staging buffer");
  if ((int)blockIdx.x < A.xblocks) {   // leading blocks: the Cr-C lists
    int* scratch = reinterpret_cast<int*>(sq);
    xlist_pass<BRICK_NT>(K, A, reinterpret_cast<int(*)[MAXC]>(scratch), scratch + BRICK_NT / WAVE * MAXC, blockIdx.x,
                         A.xblocks);
    return;
  }
  const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
  const int nitems = uniform(*A.nitems), nbk = uniform(*A.nbk), nb = (int)gridDim.x - A.xblocks;
  // (items in launch order: neighbouring bricks on different XCDs, so that a batch's rebuilding
  // replicas spread over the chip; the further items of crowded bricks before all, as the last
  // bricks may be a vacuum's)
  for (int u = (int)blockIdx.x - A.xblocks; u < nitems * A.parts; u += nb) {
    const int item = A.parts == 1 ? u : u / A.parts, share = u - item * A.parts;
    const int4 it = A.items[item < nitems - nbk ? item + nbk : item - (nitems - nbk)];
    const int r = uniform(it.x), i_lo = uniform(it.z), i_n = uniform(it.w) - i_lo;
    const int c_lo = i_lo + i_n * share / A.parts, c_hi = i_lo + i_n * (share + 1) / A.parts;
    if (c_lo >= c_hi) continue;   // uniform over the block
    RepState& S = A.S[r];
    const RepDesc& d = A.R[r];
    const int per[3] = {uniform(d.per[0]), uniform(d.per[1]), uniform(d.per[2])};
    const double len0 = uniform(d.len[0]), len1 = uniform(d.len[1]), len2 = uniform(d.len[2]);
    const int sbase = uniform(d.a0 - A.start[d.g0]);   // sorted slot = sbase + start[cell]
    __syncthreads();   // the previous item's tables, stage and counts are no longer read
    if (wave == 0) brick_tables(brick_geom(S.gd, S.bn, S.bq, per, d.g0, uniform(it.y)), per, A.start, sbase, tab);
    __syncthreads();
    BrickHdr b;
    b.nry = uniform(tab.hdr.nry);
    b.nrows = uniform(tab.hdr.nrows);
    b.x0 = uniform(tab.hdr.x0);
    b.x1 = uniform(tab.hdr.x1);
    b.y0 = uniform(tab.hdr.y0);
    b.z0 = uniform(tab.hdr.z0);
    b.gx = uniform(tab.hdr.gx);
    b.gy = uniform(tab.hdr.gy);
    b.gz = uniform(tab.hdr.gz);
    b.xa = uniform(tab.hdr.xa);
    b.xb = uniform(tab.hdr.xb);
    const int W = uniform(tab.roff[BRICK_ROWS]);   // atoms of the window
    constexpr int CW = 16;   // threads per row of the offsets (BRICK_CELLS of them work)
    static_assert(CW >= BRICK_CELLS, "a row's offsets");
    for (int e = threadIdx.x; e < b.nrows * CW; e += BRICK_NT) {
      const int row = e / CW, k = e % CW, u = b.x0 - 1 + k;   // unwrapped cell
      if (u > b.x1 + 2) continue;
      const int rw = tab.rw[row];
      int v = tab.roff[row];
      if (rw >= 0)
        v = u < b.xa ? v : (u <= b.xb + 1 ? v + tab.rp[row].w + (A.start[rw + u] - A.start[rw + b.xa]) : tab.roff[row + 1]);
      toff[row][k] = v;
      if (k == 0) {
        int uy, uz;
        brick_row(b, row, uy, uz);
        rsh[row] = make_float2((float)cell_shift(uy, b.gy, per[1], len1), (float)cell_shift(uz, b.gz, per[2], len2));
      }
    }
    const double rl2 = K.rlist_sq;
    const int cap = K.cap, T = K.lt;
    // entry k of atom p at idx[(k / T) * lrow + p * T + k % T] (fewer than 2^31 words)
    const unsigned lrow = (unsigned)K.ntot * T;
    const double4* __restrict__ tq = A.tq;
    const float4* __restrict__ tqf = A.tqf;
    const bool shadow = K.shadow;   // entries carry relative cells only for the FP32 shadow
    const float lo_f = uniform(S.scr_lo), hi_f = uniform(S.scr_hi);
    const unsigned band_bits = __float_as_uint(hi_f - lo_f);   // hi - lo, exact
    const float fxl = (float)(-len0), fxr = (float)len0;
    // lanes per center: as many (a power of two, up to 16) as let the threads take every center
    // of this share at once (an item has at most BRICK_NT)
    int gsh = 0;
    while (gsh < 4 && ((c_hi - c_lo) << (gsh + 1)) <= BRICK_NT) ++gsh;
    const int G = 1 << gsh, gl = lane & (G - 1);
    {
      const int c = c_lo + (threadIdx.x >> gsh);
      const bool live = c < c_hi;
      const int crow = brick_center_row(tab, live ? c : c_lo);
      const int p = tab.cs[crow] + (live ? c : c_lo);
      const float4 pf = tqf[p];
      const int cx = cell_coord(tq[p].x, uniform(S.glo[0]), uniform(S.ginv[0]), b.gx);
      int count = 0;
      unsigned off = (unsigned)p * T;   // the next entry's place (one lane per center)
      for (int G0 = 0; G0 < W; G0 += LIST_STAGE) {   // uniform over the block
        const int nch = min(LIST_STAGE, W - G0);
        __syncthreads();   // the offsets are written; the previous piece is no longer read
        {
          for (int row = wave; row < b.nrows; row += BRICK_NT / WAVE) {   // a row per wavefront
            const int ro = uniform(tab.roff[row]), nlm = uniform(tab.nlm[row]);
            const int g1 = min(uniform(tab.roff[row + 1]), G0 + nch) - ro;
            const int4 rp = tab.rp[row];
            const float2 yz = rsh[row];
            for (int gi = max(0, G0 - ro) + lane; gi < g1; gi += WAVE) {
              const int j = gi + (gi < rp.w ? rp.x : (gi < nlm ? rp.y : rp.z));
              const float4 cf = tqf[j];
              sq[ro + gi - G0] = make_float4(cf.x + (gi < rp.w ? fxl : (gi < nlm ? 0.0f : fxr)), cf.y + yz.x,
                                             cf.z + yz.y, __int_as_float(j));
            }
          }
          __syncthreads();
        }
        if (live) {
          const int s_self = brick_self(tab, crow, p) - G0;   // the center's own staged position
#pragma unroll 1
          for (int rr = 0; rr < 9; ++rr) {   // this center's range of each row
            const int row = crow + (rr / 3 - 1) * b.nry + (rr % 3 - 1);
            const int* to = toff[row] + (cx - b.x0);
            int e0 = to[0], e1 = to[3], b1 = 0, b2 = 0;
            if (shadow) {
              b1 = to[1] - G0;
              b2 = to[2] - G0;
            }
            if (W > LIST_STAGE) {   // the piece's part of the range
              e0 = max(e0, G0) - G0;
              e1 = min(e1, G0 + nch) - G0;
            }
            const int rcode = rr * 3;
            // exact FP64 test of staged candidate s (in the band, or NaN in the
            // single-candidate loop)
            auto exact = [&](int s) {
              int uy, uz;
              brick_row(b, row, uy, uz);
              const double shy = cell_shift(uy, b.gy, per[1], len1), shz = cell_shift(uz, b.gz, per[2], len2);
              const int gi = G0 + s - tab.roff[row];
              const double shx = gi < tab.rp[row].w ? -len0 : (gi < tab.nlm[row] ? 0.0 : len0);
              const double4 pi = tq[p], pj4 = tq[__float_as_int(sq[s].w)];
              return dist_sq_exact((pj4.x - pi.x) + shx, (pj4.y - pi.y) + shy, (pj4.z - pi.z) + shz) < rl2;
            };
            // The range is taken in runs of up to 32 candidates per lane, the center's lanes one
            // run after the other.  A lane gathers the passing candidates of its run as bits of
            // one mask and appends them in order together (the appending loop then runs as
            // often as the most passing candidates of a lane, not once per group screened),
            // after those of the center's lanes before it.  The center itself occurs once among
            // its candidates, in the middle row: its bit is cleared.
            for (int sb = e0; sb < e1;) {
              const int run = min(32, (e1 - sb + G - 1) >> gsh);
              const int s0 = sb + gl * run, s1 = min(s0 + run, e1);
              sb += run << gsh;
              // LIST_GROUP candidates at a time: the FP32 screen gives their in bits (the last
              // group's past the run are dropped), and the rare candidates in the band get the
              // exact test.  d = |r2| - lo: in when negative (its sign bit, shifted into acc); in
              // the band when 0 <= d < hi - lo, which compares as unsigned bit patterns (both
              // differences are exact there, by Sterbenz's lemma, and d >= lo beyond 2 lo).  The
              // absolute value clears the sign of a NaN, which then falls in neither: out, as
              // the exact test would decide.
              unsigned acc = 0;
              int s = s0;
              for (; s < s1; s += LIST_GROUP) {
                unsigned dmin = ~0u;
                float dd[LIST_GROUP];
#pragma unroll
                for (int u = 0; u < LIST_GROUP; ++u) {
                  const float4 cf = sq[s + u];
                  const float ex = cf.x - pf.x, ey = cf.y - pf.y, ez = cf.z - pf.z;
                  dd[u] = fabsf(ex * ex + ey * ey + ez * ez) - lo_f;
                  acc = __builtin_amdgcn_alignbit(acc, __float_as_uint(dd[u]), 31);
                  dmin = min(dmin, __float_as_uint(dd[u]));   // one test for the whole group
                }
                if (__builtin_expect(dmin < band_bits, 0)) {
#pragma unroll
                  for (int u = 0; u < LIST_GROUP; ++u)
                    if (__float_as_uint(dd[u]) < band_bits && s + u < s1 && exact(s + u)) acc |= 1u << (LIST_GROUP - 1 - u);
                }
              }
              // candidate s0 + c at bit 31 - c
              acc = s1 > s0 ? (acc >> (s - s1)) << (32 - (s1 - s0)) : 0u;
              if (rr == 4) {
                const unsigned self = (unsigned)(s_self - s0);
                if (self < 32u) acc &= ~(0x80000000u >> self);
              }
              int k = count, tot = __builtin_popcount(acc);
              if (G > 1) {   // entries of the center's lanes before this one
                int incl = tot;
                for (int o = 1; o < G; o <<= 1) {
                  const int up = __shfl(incl, lane - o, WAVE);
                  if (gl >= o) incl += up;
                }
                k += incl - tot;
                tot = __shfl(incl, lane | (G - 1), WAVE);
              }
              count += tot;
              if (G > 1) off = ((unsigned)k >> K.lt_shift) * lrow + (unsigned)p * T + (k & (T - 1));
              auto append = [&](auto full_c) {   // (full: some entries of these may not fit the capacity)
                for (; acc; ++k) {
                  const int at = __builtin_clz(acc), su = s0 + at;
                  acc &= ~(0x80000000u >> at);
                  const int code = shadow ? rcode + (su >= b1) + (su >= b2) : 0;
                  if (!decltype(full_c)::value || k < cap) A.idx[off] = __float_as_int(sq[su].w) | (code << LIST_IDX_BITS);
                  off += (k + 1) & (T - 1) ? 1u : lrow - (T - 1);
                }
              };
              if (k + __builtin_popcount(acc) <= cap) append(std::false_type{}); else append(std::true_type{});
            }
          }
        }
      }
      if (live && gl == 0) {
        csh[threadIdx.x >> gsh] = min(count, cap);
        psh[threadIdx.x >> gsh] = p;
        if (count > cap) atomicMax(&S.overflow, count);
      }
      __syncthreads();
      if ((int)threadIdx.x < c_hi - c_lo) {   // copy-back of the sorted state, one center per thread
        const int p = psh[threadIdx.x], kept = csh[threadIdx.x];
        // all loads before the first store (a store could alias a later load, which would
        // then wait for it)
        const double4 pi = tq[p];
        const double v0 = A.tv[3 * p + 0], v1 = A.tv[3 * p + 1], v2 = A.tv[3 * p + 2];
        const bool cf = A.copy_f;
        const double f0 = cf ? A.tf[3 * p + 0] : 0.0, f1 = cf ? A.tf[3 * p + 1] : 0.0, f2 = cf ? A.tf[3 * p + 2] : 0.0;
        const uint8_t fx = A.tfixed[p];
        const int ide = A.tid[p];
        A.cnt[p] = kept;
        A.q[p] = pi;
        if (K.shadow) {
          const int row = brick_center_row(tab, c_lo + threadIdx.x);
          int uy, uz;
          brick_row(b, row, uy, uz);
          const long long bc = pack_cell(cell_coord(pi.x, uniform(S.glo[0]), uniform(S.ginv[0]), b.gx), uy, uz);
          A.bcell[p] = bc;
          A.qs[p] = cell_local(S, bc, pi.x, pi.y, pi.z, (float)pi.w);
        }
        A.xref[3 * p + 0] = pi.x;
        A.xref[3 * p + 1] = pi.y;
        A.xref[3 * p + 2] = pi.z;
        A.v[3 * p + 0] = v0;
        A.v[3 * p + 1] = v1;
        A.v[3 * p + 2] = v2;
        if (cf) {
          A.f[3 * p + 0] = f0;
          A.f[3 * p + 1] = f1;
          A.f[3 * p + 2] = f2;
        }
        A.fixed[p] = fx;
        A.id[p] = ide;
      }
    }
  }
}

__global__ __launch_bounds__(BLOCK) void k_xlist(Consts K, BuildArgs A) {
  if (rebuild_off(A)) return;
  __shared__ int cand_sh[WAVES_PER_BLOCK][MAXC];
  __shared__ int pre[XL_FLAT_MAXREP + 1];
  xlist_pass<BLOCK>(K, A, cand_sh, pre, blockIdx.x, gridDim.x);
}

// Section 2.6's inner list, refilled every step: atom i's outer (Verlet) entries whose pair is
// closer than the largest Cr-Cr cutoff r* at the current positions (minimum image, the list
// build's exact FP64 predicate), in their outer-list order and in the outer list's layout and
// entry format.  INNER_G lanes share an atom and test INNER_G consecutive entries at a time (the
// next ones' indices loaded while the current positions are gathered); a ballot over the group
// gives each kept entry its place, so the order is the source list's.
//
// The source is a middle list: the outer entries closer than r* + mid_skin at the positions mref,
// taken again (k_mid_list) when an atom of the replica has moved more than mid_skin / 2 from
// there, the outer list is new, or a call finds other entries in it (k_mid_check).  Every pair within r* is then in it, as every pair within r*
// is in the outer list, so the inner list is the one that the outer list itself gives.  What
// bounds the refill is the gather of one position per source entry: the paper's form has about
// 940 outer entries an atom and 260 middle ones.  On the 216k-atom film the refill from the outer
// list took 787 us a step, from the middle one 222 (4 lanes an atom 231, 16 262), and the middle
// list itself takes 960, its check 180 a call.
constexpr int INNER_G = 8;
constexpr int MID_G = 16;

// The middle list (idx null: the workspace holds none, and the outer list is the source).
struct MidList {
  int* idx;       // [cap][ntot], laid out as the outer list
  int* cnt;       // [ntot]; < 0: more entries than cap, and the outer list is this atom's source
  float4* ref;    // [ntot] the positions (as k_inner_pos gives them) it was taken at
  ulonglong2* sum;   // [ntot] ListSum of the outer entries it was taken from
  int cap;
};

// Fingerprint of an atom's outer list: two sums of its entries x_k modulo 2^64, (x_k + a_k)(x_k + b_k)
// and x_k c_k, with keys that run with k, in any order.  Another word in the place of one entry changes
// one of them whatever the words (c_k is odd), and so do two entries that change places; other edits
// escape both with a chance of about 2^-128.  One multiply-add each: with a 64-bit mixing function per
// entry the check took 19 us on 10,000 atoms in place of 16 (216,000: 180 either way, 4.5 TB/s).
struct ListSum {
  unsigned long long q = 0, l = 0;
  __device__ __forceinline__ void add(int k, int e) {
    const unsigned x = (unsigned)e, n = (unsigned)k;
    const unsigned a = n * 0x9E3779B9u + 0x6A09E667u, b = n * 0xA54FF53Bu + 0x510E527Fu, c = n * 0x3C6EF372u + 0xBB67AE85u;
    q += (unsigned long long)(x + a) * (x + b);
    l += (unsigned long long)x * c;
  }
};

// Middle lists are kept from one call to the next, while the outer lists lie in the caller's arrays
// (and may be other arrays in the next call): a replica whose outer lists are not, entry for entry,
// those its middle lists were taken from has them marked.  The first refill of a call runs it; inside
// md_run only its own builds write the lists.  A lane per atom and CHECK_WAVES wavefronts over its
// entries, read once and coalesced.
constexpr int CHECK_WAVES = 16;
__global__ __launch_bounds__(CHECK_WAVES* WAVE) void k_mid_check(Consts K, const RepDesc* __restrict__ R,
                                                                RepState* __restrict__ S,
                                                                const int* __restrict__ tile_rep,
                                                                const int* __restrict__ idx, const int* __restrict__ cnt,
                                                                MidList M) {
  constexpr int PER_TILE = TILE / WAVE;   // blocks per tile
  constexpr int U = 8;                    // entries in flight per lane
  const int r = tile_rep[blockIdx.x / PER_TILE];
  const RepDesc& d = R[r];
  __shared__ int ok_sh;
  if (threadIdx.x == 0) ok_sh = S[r].mid_ok;   // (another block may clear it meanwhile)
  __syncthreads();
  if (!ok_sh) return;
  const int lane = threadIdx.x % WAVE, w = uniform((int)(threadIdx.x / WAVE));
  const int64_t i = (int64_t)blockIdx.x * WAVE + lane;
  const bool live = i < (int64_t)d.a0 + d.n;
  const int n = live ? cnt[i] : 0;
  const int T = K.lt;
  const unsigned stride = (unsigned)K.ntot * T, base = (unsigned)(live ? i : 0) * T;
  ListSum h;
  for (int k0 = w * U; k0 < n; k0 += CHECK_WAVES * U) {
    int e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(k0 + u, n - 1);
      e[u] = idx[((unsigned)k >> K.lt_shift) * stride + base + (unsigned)(k & (T - 1))];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k0 + u < n) h.add(k0 + u, e[u]);
  }
  __shared__ ulonglong2 part[CHECK_WAVES][WAVE];
  part[w][lane] = make_ulonglong2(h.q, h.l);
  __syncthreads();
  if (w == 0 && live) {
    unsigned long long q = 0, l = 0;
    for (int t = 0; t < CHECK_WAVES; ++t) {
      q += part[t][lane].x;
      l += part[t][lane].y;
    }
    const ulonglong2 was = M.sum[i];
    if (q != was.x || l != was.y) S[r].mid_ok = 0;
  }
}

// Bound on the error of an FP32 position relative to the grid origin, per axis, for atoms within
// R of the grid, images included (the list build's).
__device__ __forceinline__ double pos_err(const RepDesc& d, const RepState& s, int a, double R) {
  const double E = s.gd[a] / s.ginv[a] + 2.0 * R;
  return 0x1p-24 * (3.0 * E + (d.per[a] ? 2.0 * d.len[a] : 0.0) + 3.0 * R);
}

// FP32 positions relative to the replica's grid origin at the current positions, for the
// inner-list screen (one lane per atom slot; the list build's scratch copy, free between
// builds); an atom that has moved too far from the middle list's reference marks that list.
__global__ __launch_bounds__(BLOCK) void k_inner_pos(Consts K, const RepDesc* __restrict__ R, RepState* __restrict__ S,
                                                     const int* __restrict__ tile_rep, const double4* __restrict__ q,
                                                     float4* __restrict__ qf, MidList M) {
  static_assert(TILE == BLOCK, "one block per tile");
  const int r = tile_rep[blockIdx.x];
  const RepDesc& d = R[r];
  const int64_t i = (int64_t)blockIdx.x * TILE + threadIdx.x;
  if (i >= (int64_t)d.a0 + d.n) return;
  const double4 p = q[i];
  RepState& s = S[r];
  const float4 f = make_float4((float)(p.x - s.glo[0]), (float)(p.y - s.glo[1]), (float)(p.z - s.glo[2]), 0.0f);
  qf[i] = f;
  if (M.idx) {
    const float4 o = M.ref[i];
    const double R0 = K.rlist + 1.0;
    double err = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) err += 2.0 * pos_err(d, s, a, R0);
    const float th = (float)(0.5 * K.mid_skin * 0.999 - err);
    const float dx = f.x - o.x, dy = f.y - o.y, dz = f.z - o.z;
    const bool still = th > 0.0f && dx * dx + dy * dy + dz * dz <= th * th;   // (a NaN is not)
    if (!still) s.mid_ok = 0;
  }
}

__device__ __forceinline__ float min_image_f(float d, float len, float half, int per) {
  float s = (per && d > half) ? -len : 0.0f;
  s = (per && d < -half) ? len : s;
  return d + s;
}

// Entries of a list that are closer than sqrt(rc2), G lanes per atom, for the atoms of one
// 256 / G-atom block `lb`.  The FP32 squared separation decides outside a band around rc2
// that covers its error (the list build's bound, with R = sqrt(rc2) + 1 and positions within R
// of the grid); the band gets the exact FP64 test or, with MID, is kept.  On a replica with a
// periodic length under 2 R + 1 the FP32 minimum image could pick the other image of a pair
// inside the radius, and every entry lies in the band.  MID: the middle list from the outer one;
// else the inner list from the middle one (from the outer one where that has none).
template <int G, bool MID>
__device__ __forceinline__ void filter_list(const Consts& K, const RepDesc& d, RepState& s, int tile, int lb,
                                            const double4* __restrict__ q, const float4* __restrict__ qf,
                                            const int* __restrict__ idx, const int* __restrict__ cnt, const MidList& M,
                                            int* __restrict__ oidx, int* __restrict__ ocnt, int ocap, double rc2) {
  static_assert(WAVE % G == 0 && G < 32, "a lane group lies in one wavefront, its mask in 32 bits");
  constexpr int APB = BLOCK / G;   // atoms per block
  const int sub = threadIdx.x % G;
  const int64_t i = (int64_t)tile * TILE + (lb % G) * APB + threadIdx.x / G;
  const bool live = i < (int64_t)d.a0 + d.n;
  const double4 pi = live ? q[i] : make_double4(0.0, 0.0, 0.0, 0.0);
  const float4 pif = live ? qf[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  const bool img = wave_near_face(d, live, pi.x, pi.y, pi.z, K.rlist + 2.0 * K.half_skin);
  // every lane takes part in the ballots (atoms past the replica with an empty list)
  const int* src = idx;
  int n = 0;
  if (!MID && M.idx) {
    n = live ? M.cnt[i] : 0;
    if (n >= 0) src = M.idx;
    else n = cnt[i];
  } else {
    n = live ? cnt[i] : 0;
  }
  int nw = n;   // the wavefront's longest list
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) nw = max(nw, __shfl_xor(nw, o, WAVE));
  const int T = K.lt, sh = K.lt_shift;
  const unsigned stride = (unsigned)K.ntot * T, base = (unsigned)(live ? i : 0) * T;
  // word offset of entry k of atom i (32-bit: the lists hold fewer than 2^31 words)
  auto at_k = [&](int k) { return ((unsigned)k >> sh) * stride + base + (unsigned)(k & (T - 1)); };
  float lo_f = -1.0f, hi_f = INFINITY;   // (everything in the band)
  {
    const double u = 0x1p-24, Rr = sqrt(rc2) + 1.0;
    double err = 4.0 * u * (rc2 + Rr * Rr);
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double eta = pos_err(d, s, a, Rr);
      err += 2.0 * Rr * eta + eta * eta;
      ok = ok && !(d.per[a] && d.len[a] <= 2.0 * Rr + 1.0);
    }
    if (ok) {
      const double delta = 2.0 * err + 1e-6;
      lo_f = (float)(rc2 - delta);
      hi_f = (float)(rc2 + delta);
    }
  }
  const float len0 = (float)d.len[0], len1 = (float)d.len[1], len2 = (float)d.len[2];
  const float hf0 = (float)d.half[0], hf1 = (float)d.half[1], hf2 = (float)d.half[2];
  const int gshift = (int)(threadIdx.x % WAVE) - sub;   // the group's first lane
  const unsigned below = (1u << sub) - 1u;
  int c = 0;        // entries kept so far
  ListSum h;        // MID: of this lane's entries
  int e = sub < n ? src[at_k(sub)] : 0;   // (slot 0 stands in for an entry past the list)
  for (int m0 = 0; m0 < nw; m0 += G) {
    const int k = m0 + sub;
    const float4 pjf = qf[list_slot(e)];
    const int en = k + G < n ? src[at_k(k + G)] : 0;
    float fx = pjf.x - pif.x, fy = pjf.y - pif.y, fz = pjf.z - pif.z;
    if (img) {
      fx = min_image_f(fx, len0, hf0, d.per[0]);
      fy = min_image_f(fy, len1, hf1, d.per[1]);
      fz = min_image_f(fz, len2, hf2, d.per[2]);
    }
    const float r2f = fx * fx + fy * fy + fz * fz;
    bool keep;
    if (MID) {
      keep = !(r2f >= hi_f);   // (NaN: kept)
    } else {
      keep = r2f < lo_f;
      if (k < n && !keep && !(r2f >= hi_f)) {   // the band (or NaN): the exact test
        const double4 pj = q[list_slot(e)];
        double ex = pj.x - pi.x, ey = pj.y - pi.y, ez = pj.z - pi.z;
        if (img) {
          ex = min_image(ex, d.len[0], d.half[0], d.per[0]);
          ey = min_image(ey, d.len[1], d.half[1], d.per[1]);
          ez = min_image(ez, d.len[2], d.half[2], d.per[2]);
        }
        keep = dist_sq_exact(ex, ey, ez) < rc2;
      }
    }
    keep = keep && k < n;
    if (MID && k < n) h.add(k, e);
    const unsigned gm = (unsigned)(__ballot(keep) >> gshift) & ((1u << G) - 1u);
    if (keep) {
      const int j = c + __popc(gm & below);
      if (j < ocap) oidx[at_k(j)] = e;
    }
    c += __popc(gm);
    e = en;
  }
  if (MID) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
      h.q += __shfl_xor(h.q, o, WAVE);
      h.l += __shfl_xor(h.l, o, WAVE);
    }
  }
  if (live && sub == 0) {
    if (MID) {
      ocnt[i] = c > ocap ? -1 : c;
      M.ref[i] = pif;
      M.sum[i] = make_ulonglong2(h.q, h.l);
    } else {
      ocnt[i] = min(c, ocap);
      if (c > ocap) atomicMax(&s.ioverflow, c);
    }
  }
}

// The middle lists of the replicas whose own no longer holds (blocks stride over the tiles, as
// most launches have none).
__global__ __launch_bounds__(BLOCK) void k_mid_list(Consts K, const RepDesc* __restrict__ R, RepState* __restrict__ S,
                                                    const int* __restrict__ tile_rep, const double4* __restrict__ q,
                                                    const float4* __restrict__ qf, const int* __restrict__ idx,
                                                    const int* __restrict__ cnt, MidList M, int nb) {
  for (int b = blockIdx.x; b < nb; b += gridDim.x) {
    const int lb = xcd_block(b, nb), tile = lb / MID_G, r = tile_rep[tile];
    if (S[r].mid_ok) continue;   // (uniform over the block)
    filter_list<MID_G, true>(K, R[r], S[r], tile, lb, q, qf, idx, cnt, M, M.idx, M.cnt, M.cap, K.mid_rc_sq);
  }
}

// One block per 256 / INNER_G atoms.
__global__ __launch_bounds__(BLOCK) void k_inner_list(Consts K, const RepDesc* __restrict__ R,
                                                      RepState* __restrict__ S, const int* __restrict__ tile_rep,
                                                      const double4* __restrict__ q, const float4* __restrict__ qf,
                                                      const int* __restrict__ idx, const int* __restrict__ cnt,
                                                      MidList M, int* __restrict__ iidx, int* __restrict__ icnt) {
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int tile = lb / INNER_G, r = tile_rep[tile];
  if (M.idx && lb % INNER_G == 0 && tile == R[r].t0 && threadIdx.x == 0) S[r].mid_ok = 1;   // (nothing here reads it)
  filter_list<INNER_G, false>(K, R[r], S[r], tile, lb, q, qf, idx, cnt, M, iidx, icnt, K.icap, K.icut_sq);
}

}  // namespace md
