// One lattice step with the immersed-boundary phases running beside the
// collide.
//
// Only the cells whose source node lies in an active tile (the band, a
// fraction of a percent of a large lattice) carry an immersed force. Every
// other cell collides without waiting for the markers, so the latency-bound
// marker phases run in launches whose other workgroups stream the rest of the
// lattice ("bulk"):
//   k_step_macro   band macros, the tiles' marker lists, skinning of the next
//                  step's markers, part of the bulk (not for few markers);
//   k_step_interp  interpolation and forcing, from the band macros, or for few
//                  markers straight from the populations with the lists and
//                  the skinning beside it; part of the bulk;
//   k_step_band    per z-plane of an active tile: spreading into LDS, then the
//                  collide of its cells with the force taken from there (it
//                  never reaches memory); binning of the next step's tiles,
//                  the wrench, the rest of the bulk.
// More forcing passes and the implicit correction need the force at the nodes
// between passes: their passes run between k_step_macro and k_step_band in
// launches of their own.
//
// Nothing waits inside a launch. This step's markers and tile map (body set
// b[0]) are complete before its first launch; the next step's go to b[1], and
// the two sets alternate between steps. A launch reads the source buffer and
// writes the other one, each cell by one workgroup. The arithmetic is the
// same inline code as the separate kernels', so results agree bit for bit.
#pragma once

#include "ib.hpp"

namespace lbmib {

// At most this many markers are interpolated straight from the populations (two
// launches a step); more get the band macros first (three). The direct form saves
// a launch and pulls 27 x 16 short rows for each marker, 55 KB of L2 lines. Us a
// step from the macros and direct, F32, fish of 0.3 nx: 500 markers on 64x32x32
// 23.0, 18.9, on 128x64x64 33.2, 32.6, on 192x96x96 80.1, 74.5; 2,000 34.0, 32.2,
// then 34.8, 34.8 and 81.1, 79.4; 3,500 45.4, 45.6, then 36.8, 40.2 and 81.9, 82.4.
constexpr int kDirectMarkers = 2000;
// Sixteenths of the bulk in each launch before the last, enough to cover the
// marker work there (2, 3 and 4 of them: fin 37.3, 37.2, 36.0 us, fish 539,
// 537, 535 us).
constexpr int kBulkShare = 4;
// Most marker workgroups over tile parts and planes (steps of the fish and of
// spheres of 9,000 to 40,000 markers with 2,048 of either: the same within 1.2%;
// with 4,096 for the planes up to 4% longer).
constexpr int kMacroWorkgroups = 1024, kBandWorkgroups = 1024;
// Marker workgroups over the marker lists: one for 64 markers, at least 256. A
// list takes as long as there are chunks of markers to look through and markers in
// the tile, so many markers want a workgroup for every tile (192x96x96 in steps of
// the sphere of radius 30, 256 of them against this: 50,000 markers 150, 137 us,
// 200,000 431, 326, 1,000,000 1,895, 1,376; twice as many the same within 1%).
inline int list_workgroups(const EnvView &e) {
  const int most = e.n / 64 > 256 ? e.n / 64 : 256;
  return e.cap < most ? e.cap : most;
}

// The next step's skinning and binning, beside this step (pose null: none).
struct NextStep {
  const float *pose;
};

// F32 lattices of so many blocks of BT cells and more reserve LDS beyond a
// launch's own so that three blocks of the collide share a compute unit (see
// collide_lds): fish 547 against 566 us, 192x96x96 115.6 against 117.1, the
// 128x64x64 fin 36.6 against 36.0 us without; 2-byte ones never (fish 338
// against 291 us).
constexpr int kCapBlocks = 4096;

// Cell blk * BT + tid of the bulk, in x-fastest order. The tile map is read
// beside the populations, not before them (the memory clobber keeps the pulls
// above the branch): a band cell, whose pull is wasted, is rare, and a pull
// that waits for the map costs the F16 collide a third of its speed.
template <class S, bool XPER, bool ROT, bool YZ, bool TRT>
__device__ inline void bulk_cell(const EnvView &e, const BodySet &bs, const FrameF &fr, int cur, int blk, int tid) {
  const uint32_t cell = (uint32_t)blk * (uint32_t)BT + (uint32_t)tid, row = cell / (uint32_t)e.g.nx;
  const int z = (int)(row / (uint32_t)e.g.ny);
  if (z >= e.g.nz) return;
  const CellAt c = cell_at<XPER, YZ>(e.g, (int)(cell - row * (uint32_t)e.g.nx),
                                     (int)(row - (uint32_t)z * (uint32_t)e.g.ny), z);
  const int slot = ((const gmem<int> *)bs.tile_slot)[(c.xs >> 3) + e.g.tnx * ((c.ys >> 3) + e.g.tny * (c.zs >> 3))];
  float f[Q];
  collide_pull<S, XPER, YZ>(e, cur, c, f);
  asm volatile("" ::: "memory");
  if (slot >= 0) return;  // a band cell (source node in an active tile): its tile's workgroup collides it
  collide_finish<S, XPER, ROT, YZ, TRT>(e, fr, cur, c, f, 0.f, 0.f, 0.f);
}
inline int bulk_blocks(const EnvView &e) { return (int)(((size_t)e.g.nx * e.g.ny * e.g.nz + BT - 1) / BT); }

// Plane item % 8 of active tile item / 8: its immersed force into LDS, then the
// band cells whose source node lies in it: the plane's own cells, and the face
// nodes beyond it (the source node of a face node is its inward neighbour):
// along z the neighbouring face plane, along x and y those of a last tile that
// is one node wide (a dimension of 8k + 1). The plane's populations are pulled
// first, so that their latency overlaps the spreading. force: kForceAdd, the
// force starts from gfix (earlier forcing passes); kForceKeep, it is also
// written there (a recorded step).
// Its stores are ordinary ones: a tile's rows are 8 cells, 32 bytes of a line at
// F32, that L2 merges with the tile's x-neighbour (the planes of one number run
// on one XCD) and writes back whole; written nontemporal they go to memory as
// they are (384x192x192, sphere of radius 60 and 40,000 markers: 465 against
// 377 us a step in FP16, 875 against 865 in F32; fish 286 against 279, 528
// against 527).
enum { kForceAdd = 1, kForceKeep = 2 };
template <class S, bool XPER, bool ROT, bool YZ, bool TRT>
__device__ inline void band_item(const EnvView &e, const BodySet &bs, const FrameF &fr, int cur, int item, int tid,
                                 int force, SpreadLds<3> &s) {
  const GridArgs &g = e.g;
  const int slot = item >> 3, plane = item & 7;
  const TileAt t = active_of(bs, slot);
  const int x0 = t.x << 3, y0 = t.y << 3, z = (t.z << 3) + plane;
  if (z >= g.nz) return;  // uniform over the workgroup
  const int x = x0 + (tid & 7), y = y0 + ((tid >> 3) & 7);
  auto source_here = [&](const CellAt &c) { return ((c.xs >> 3) == t.x) & ((c.ys >> 3) == t.y) & (c.zs == z); };
  float f[Q];
  CellAt c{};
  bool own = tid < 64 && x < g.nx && y < g.ny;
  if (own) {
    c = cell_at<XPER, YZ>(g, x, y, z);
    own = source_here(c);
    if (own) collide_pull<S, XPER, YZ>(e, cur, c, f);
  }
  gmem<unsigned long long> *gp = (gmem<unsigned long long> *)e.gfix + (size_t)slot * 1536 + plane * 64;
  if (tid < 192) (&s.acc[0][0])[tid] = (force & kForceAdd) ? gp[512 * (tid >> 6) + (tid & 63)] : 0ull;
  spread_plane<false>(e, bs, t, plane, tid, s);
  if ((force & kForceKeep) && tid < 192) gp[512 * (tid >> 6) + (tid & 63)] = (&s.acc[0][0])[tid];
  auto finish = [&](const CellAt &cc, float ff[Q]) {
    const int lc = (cc.xs & 7) | ((cc.ys & 7) << 3);
    collide_finish<S, XPER, ROT, YZ, TRT, false>(e, fr, cur, cc, ff, from_fix(s.acc[0][lc]), from_fix(s.acc[1][lc]),
                                                 from_fix(s.acc[2][lc]));
  };
  if (own) finish(c, f);
  if (!XPER || YZ) {
    const int x1 = min(x0 + 8, g.nx), y1 = min(y0 + 8, g.ny);
    const int mx = !XPER && x1 == g.nx - 1, my = YZ && !g.yper && y1 == g.ny - 1;
    const int zlo = YZ && !g.zper && z == 1 ? 0 : z, zhi = YZ && !g.zper && z == g.nz - 2 ? g.nz - 1 : z;
    if (mx | my | (zlo != zhi)) {
      const int ex = x1 + mx - x0, ey = y1 + my - y0, cnt = ex * ey * (zhi - zlo + 1);
      for (int lc = tid; lc < cnt; lc += BT) {
        const int lx = lc % ex, r = lc / ex, ly = r % ey, zc = zlo + r / ey;
        if (zc == z && lx < 8 && ly < 8) continue;  // the plane's own
        const CellAt cc = cell_at<XPER, YZ>(g, x0 + lx, y0 + ly, zc);
        if (!source_here(cc)) continue;
        float ff[Q];
        collide_pull<S, XPER, YZ>(e, cur, cc, ff);
        finish(cc, ff);
      }
    }
  }
  __syncthreads();  // s is reused by the next item
}

// Which work workgroup blk of a launch has: first nfront workgroups of marker
// work (up to a multiple of eight, one per XCD, of which those past nfront have
// none), then the bulk. Returns whether it is a marker workgroup, else blk is set
// to the bulk block. Marker workgroups come first because the launch may end on
// them: spread over it, those of a body with many active tiles started late (eight
// after every 56 bulk blocks, sphere of radius 60 and 40,000 markers in
// 384x192x192: 870 against 655 us a step, of radius 35 in 320x176x170 438 against
// 391, 192x96x96 119.9 against 115.6; fish 526 against 528).
__device__ inline bool marker_block(int &blk, int nfront) {
  const int front = (nfront + 7) & ~7;
  if (blk < front) return true;
  blk -= front;
  return false;
}

constexpr int kStepMk = BT / 64;  // markers per workgroup of k_step_interp, one wave each

// Marker workgroups: nm over the halves of the active tiles, nl for the marker
// lists (over the active tiles), skin_items for the next step (none without
// one). The bulk starts at block 0.
template <class S, bool XPER, bool ROT, bool YZ, bool TRT>
__global__ void __launch_bounds__(BT, 4) k_step_macro(EnvView e, FrameF fr, int cur, int nm, int nl, NextStep next) {
  const int tid = threadIdx.x;
  int blk = blockIdx.x;
  const int ns = next.pose != nullptr ? skin_items<BT>(e.n) : 0;
  if (!marker_block(blk, nm + nl + ns)) {
    bulk_cell<S, XPER, ROT, YZ, TRT>(e, e.b[0], fr, cur, blk, tid);
  } else if (blk < nm) {
    const XcdWalk w = xcd_walk(2 * n_active_of(e, e.b[0]), blk, nm);
    for (int h = w.first; h < w.end; h += w.step) macro_item<BT, S, ROT>(e, e.b[0], fr, cur, h, tid);
  } else if (blk < nm + nl) {
    const int na = n_active_of(e, e.b[0]);
    for (int slot = blk - nm; slot < na; slot += nl) list_item<BT, kListLdsLone, 8>(e, e.b[0], slot, tid);
  } else if (blk < nm + nl + ns) {
    skin_item<BT>(e, e.b[1], next.pose, blk - nm - nl, tid);
  }
}

// After k_step_macro (nl = 0): marker workgroups interp_items<BT>(n) from the
// band macros. Without it (nl > 0): kStepMk markers a workgroup straight from the
// populations, nl for the marker lists, skin_items for the next step. The bulk
// starts at block first_bulk.
template <class S, bool XPER, bool ROT, bool YZ, bool TRT>
__global__ void __launch_bounds__(BT, 4) k_step_interp(EnvView e, FrameF fr, int cur, int nl, float *partials,
                                                       NextStep next, int first_bulk) {
  const int tid = threadIdx.x;
  int blk = blockIdx.x;
  const int ni = nl > 0 ? (e.n + kStepMk - 1) / kStepMk : interp_items<BT>(e.n);
  const int ns = nl > 0 && next.pose != nullptr ? skin_items<BT>(e.n) : 0;
  if (!marker_block(blk, ni + nl + ns)) {
    bulk_cell<S, XPER, ROT, YZ, TRT>(e, e.b[0], fr, cur, first_bulk + blk, tid);
  } else if (blk < ni) {
    if (nl > 0) {
      const int k = __builtin_amdgcn_readfirstlane(xcd_item(blk, ni) * kStepMk + (tid >> 6));
      if (k < e.n) interp_wave<S, ROT>(e, e.b[0], fr, cur, k, tid & 63, partials);
    } else {
      interp_item<BT, ROT, false>(e, e.b[0], fr, xcd_item(blk, ni), tid, partials);
    }
  } else if (blk < ni + nl) {
    const int na = n_active_of(e, e.b[0]);
    for (int slot = blk - ni; slot < na; slot += nl) list_item<BT, kListLdsLone, 8>(e, e.b[0], slot, tid);
  } else if (blk < ni + nl + ns) {
    skin_item<BT>(e, e.b[1], next.pose, blk - ni - nl, tid);
  }
}

// Marker workgroups: nt over the planes of the active tiles, one for the wrench
// (null: none; by_marker: from shares that k_step_interp took straight from the
// populations), active_items for the next step's binning (next.pose null: none).
// The bulk starts at block first_bulk.
template <class S, bool XPER, bool ROT, bool YZ, bool TRT>
__global__ void __launch_bounds__(BT, 4) k_step_band(EnvView e, FrameF fr, int cur, int nt, int force, float *wrench,
                                                     int by_marker, NextStep next, int first_bulk) {
  const int tid = threadIdx.x;
  int blk = blockIdx.x;
  const int nw = wrench != nullptr ? 1 : 0, nb = next.pose != nullptr ? active_items<BT>(e) : 0;
  if (!marker_block(blk, nt + nw + nb)) {
    bulk_cell<S, XPER, ROT, YZ, TRT>(e, e.b[0], fr, cur, first_bulk + blk, tid);
  } else if (blk < nt) {
    __shared__ SpreadLds<3> s;
    const int items = 8 * n_active_of(e, e.b[0]);
    for (int item = blk; item < items; item += nt)
      band_item<S, XPER, ROT, YZ, TRT>(e, e.b[0], fr, cur, item, tid, force, s);
  } else if (blk < nt + nw) {
    wrench_sum<BT>(e.partials, e.n, by_marker != 0, wrench, tid);
  } else if (blk < nt + nw + nb) {
    active_item<BT>(e, e.b[1], blk - nt - nw, tid);
  }
}

}  // namespace lbmib
