// Bricks of the cell grid and their windows (gfx950), from which the list build takes its work items.
//
// A brick is a block of neighbouring cells of the sorted order; its window is those cells and
// one layer around them, as cell rows (z, then y), each the atoms of x-cells x0-1 .. x1+1 in
// slot order.  A row is one contiguous slot range, with the cell seen across a periodic x face
// placed at the end it is seen from: up to three pieces.  The rows laid end to end give every
// atom of the window a position.
#pragma once

#include "md_device.hpp"

namespace md {

constexpr int BRICK_NT = 512;   // threads of the list build's blocks
#ifndef MD_LIST_STAGE
#define MD_LIST_STAGE 2048
#endif
constexpr int LIST_STAGE = MD_LIST_STAGE;   // candidates k_list_bricks stages in LDS at a time

// Brick cut of a replica's grid gd with n atoms.  Edges grow one axis at a time while the window
// is expected to fit LIST_STAGE atoms (with a margin for the uneven filling of cells) and the
// brick BRICK_ATOMS: along x first (up to BRICK_MAX cells), which keeps the runs of atoms that
// are stored together long, then along y, z and x in turn.  At 6.4 atoms per cell that is
// 6 x 4 x 3 cells, 460 centers and 1540 atoms in the window; cubic bricks of 4 cells (410 and
// 1380) took 1387 against 1300 us per rebuild on the 8M-atom film and 55 against 50 us on the
// 216k-atom one.  Bricks are kept to the replica's capacity bcap whatever the density (then
// larger edges, whose windows may not fit).
__host__ __device__ inline void choose_bricks(int64_t n, int64_t bcap, const int (&gd)[3], int (&bn)[3]) {
  const double a = (double)n / ((double)gd[0] * gd[1] * gd[2]);   // atoms per cell
  int b[3] = {1, 1, 1};
  auto grows = [&](int x) {
    int t[3] = {b[0], b[1], b[2]};
    t[x] += 1;
    const double w = (double)(t[0] + 2) * (t[1] + 2) * (t[2] + 2) * a;
    return t[x] <= BRICK_MAX && t[x] <= gd[x] && w * 1.06 <= LIST_STAGE && (double)t[0] * t[1] * t[2] * a <= BRICK_ATOMS;
  };
  while (grows(0)) ++b[0];
  for (bool grown = true; grown;) {
    grown = false;
    for (int x = 1; x < 3; ++x)
      if (grows(x)) {
        ++b[x];
        grown = true;
      }
  }
  for (;;) {
    for (int x = 0; x < 3; ++x) bn[x] = (gd[x] + b[x] - 1) / b[x];
    if ((long long)bn[0] * bn[1] * bn[2] <= bcap) break;
    int s = -1;
    for (int x = 0; x < 3; ++x)
      if (b[x] < BRICK_MAX && b[x] < gd[x] && (s < 0 || b[x] < b[s])) s = x;
    if (s < 0) break;   // (bcap holds the cut into bricks of the largest edges)
    ++b[s];
  }
}

// Host bound of the bricks of a replica (see choose_bricks).
inline int64_t brick_capacity(int64_t n, const int (&gcap)[3]) {
  int64_t c = 1;
  for (int a = 0; a < 3; ++a) c *= (gcap[a] + BRICK_MAX - 1) / BRICK_MAX;
  return c + n / 24 + 8;
}

// LDS tables of a brick's window and centers.
struct BrickTab {
  BrickHdr hdr;
  int roff[BRICK_ROWS + 1];   // window position of each row's first atom; the last: all
  int coff[BRICK_ROWS + 1];   // centers before each row's
  int4 rp[BRICK_ROWS];        // slot of row-local index g: g + .x (g < .w, the cell across the lower x
                              // face), g + .y (the main piece), g + .z (across the upper face)
  int nlm[BRICK_ROWS];        // row-local end of the main piece
  int cs[BRICK_ROWS];         // slot of a row's center c is cs + c
  int rw[BRICK_ROWS];         // cell 0 of the row (-1: outside an open axis, or past the rows)
};

// First cell of brick i of an axis of g cells cut into bn bricks of q = g / bn cells, the first g % bn
// of them one more (nothing here grows past g, so 32 bits hold axes of any length).
__host__ __device__ inline int brick_first(int i, int q, int g, int bn) {
  const int left = g - q * bn;
  return i * q + (i < left ? i : left);
}

// Brick lb of a replica with grid gd cut into bn bricks.
__host__ __device__ inline BrickHdr brick_geom(const int (&gd)[3], const int (&bn)[3], const int (&bq)[3], const int (&per)[3],
                                               int g0, int lb) {
  BrickHdr b;
  b.gx = gd[0];
  b.gy = gd[1];
  b.gz = gd[2];
  b.g0 = g0;
  const int ix = lb % bn[0], iy = lb / bn[0] % bn[1], iz = lb / (bn[0] * bn[1]);
  b.x0 = brick_first(ix, bq[0], b.gx, bn[0]);
  b.x1 = brick_first(ix + 1, bq[0], b.gx, bn[0]) - 1;
  b.y0 = brick_first(iy, bq[1], b.gy, bn[1]);
  b.z0 = brick_first(iz, bq[2], b.gz, bn[2]);
  b.nry = brick_first(iy + 1, bq[1], b.gy, bn[1]) - b.y0 + 2;
  b.nrows = b.nry * (brick_first(iz + 1, bq[2], b.gz, bn[2]) - b.z0 + 2);
  b.xa = b.x0 > 0 ? b.x0 - 1 : 0;
  b.xb = b.x1 + 1 < b.gx ? b.x1 + 1 : b.gx - 1;
  b.flags = (per[0] && b.x0 == 0 ? BRICK_WL : 0) | (per[0] && b.x1 == b.gx - 1 ? BRICK_WR : 0);
  return b;
}

// Window row t's unwrapped cell row (y, z).
__device__ __forceinline__ void brick_row(const BrickHdr& b, int t, int& uy, int& uz) {
  const int rz = t / b.nry;
  uy = b.y0 - 1 + (t - rz * b.nry);
  uz = b.z0 - 1 + rz;
}

// Inclusive sum over the lanes of a wavefront up to this one.
__device__ __forceinline__ int wave_scan(int v) {
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const int u = __shfl_up(v, o, WAVE);
    if ((int)(threadIdx.x % WAVE) >= o) v += u;
  }
  return v;
}

// Fills the tables of brick b: one wavefront, a row per lane, the loads of a row together.
// start: scanned cell counts, sbase: the sorted slot of a start value is sbase + it.
__device__ __forceinline__ void brick_tables(const BrickHdr& b, const int (&per)[3], const int* __restrict__ start, int sbase,
                                             BrickTab& tab) {
  static_assert(BRICK_ROWS == WAVE, "a row per lane");
  const int t = threadIdx.x % WAVE;
  int rw = -1, len = 0, nlm = 0, nc = 0, cs = 0;
  int4 rp = make_int4(0, 0, 0, 0);
  if (t < b.nrows) {
    int uy, uz;
    brick_row(b, t, uy, uz);
    const int y = per[1] ? (uy < 0 ? uy + b.gy : (uy >= b.gy ? uy - b.gy : uy)) : (uy >= b.gy ? -1 : uy);
    const int z = per[2] ? (uz < 0 ? uz + b.gz : (uz >= b.gz ? uz - b.gz : uz)) : (uz >= b.gz ? -1 : uz);
    if (y >= 0 && z >= 0) rw = b.g0 + (z * b.gy + y) * b.gx;
    const int ry = uy - (b.y0 - 1), rz = uz - (b.z0 - 1);
    if (rw >= 0) {
      const int* __restrict__ st = start + rw;
      const int s_a = st[b.xa], s_m = st[b.xb + 1], s_l = st[b.gx - 1], s_e = st[b.gx], s_0 = st[0], s_1 = st[1],
                s_c = st[b.x0], s_d = st[b.x1 + 1];
      const int nl = (b.flags & BRICK_WL) ? s_e - s_l : 0;
      nlm = nl + (s_m - s_a);
      len = nlm + ((b.flags & BRICK_WR) ? s_1 - s_0 : 0);
      rp = make_int4(sbase + s_l, sbase + s_a - nl, sbase + s_0 - nlm, nl);
      if (ry >= 1 && ry <= b.nry - 2 && rz >= 1 && t < b.nrows - b.nry) nc = s_d - s_c;   // a row of the brick itself
      cs = sbase + s_c;
    }
  }
  const int wi = wave_scan(len), ci = wave_scan(nc);
  tab.roff[t] = wi - len;
  tab.coff[t] = ci - nc;
  tab.rp[t] = rp;
  tab.nlm[t] = nlm;
  tab.cs[t] = cs - (ci - nc);
  tab.rw[t] = rw;
  if (t == WAVE - 1) {
    tab.roff[BRICK_ROWS] = wi;
    tab.coff[BRICK_ROWS] = ci;
  }
  if (t == 0) tab.hdr = b;
}

// Window row of center c (the last row with coff <= c that has centers).
__device__ __forceinline__ int brick_center_row(const BrickTab& tab, int c) {
  int lo = 0;
#pragma unroll
  for (int s = BRICK_ROWS / 2; s > 0; s >>= 1)
    if (tab.coff[lo + s] <= c) lo += s;
  return lo;
}

// Window position of the center in slot p of row t.
__device__ __forceinline__ int brick_self(const BrickTab& tab, int t, int p) {
  return tab.roff[t] + (p - tab.rp[t].y);
}

__device__ __forceinline__ int brick_count(const int (&bn)[3]) { return bn[0] * bn[1] * bn[2]; }

}  // namespace md
