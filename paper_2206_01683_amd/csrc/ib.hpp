// Immersed-boundary phases of one step: skinning, tile binning, interpolation
// with direct forcing, gather-form spreading and the body wrench.
//
// The immersed force lives only in "active" 8x8x8 tiles: tiles that some
// marker's 4x4x4 Peskin stencil touches. Each step rebuilds the active set.
// Every phase is a device function of (environment, work item) run by one
// workgroup of NT threads (256 in the single lattice's launches, mostly 512 in the
// batched ones), so the same code serves the single-lattice kernels, the batched
// per-phase kernels and the persistent batched kernel:
//   skin_item     NT markers: linear blend skinning, wrap/range guard, flag
//                 the tiles each stencil touches (plain stores), per-wave
//                 chunk boxes (tile range of 64 consecutive markers)
//   active_item   NT tiles: compact the flags into slots and an active list
//   list_item     one active tile: the list of the markers that touch it
//   macro_item    NT cells of an active tile: density and unforced velocity
//   interp_item,  U*_k, rho_k, direct forcing F_k, marker record, wrench
//   interp_wave   shares; from the band macros, or straight from the populations
//   spread_plane  one z-plane of an active tile per 256 threads: its markers add
//                 their stencil nodes into LDS in 64-bit fixed point
//                 (order-independent, so deterministic)
//   wrench_sum    adds the wrench partials in a fixed order
#pragma once

#include <type_traits>

#include "fluid.hpp"

namespace lbmib {

constexpr int WG = 512;              // threads per workgroup of the batched phases, k_active, k_macro and the adjoint
constexpr int REC = 20;              // floats per marker record: w[12], base[3], pad, fdv[3], pad
constexpr int kWavePer = WG / 64;    // markers per item of the one-wave-per-marker kernels (adjoint)
constexpr int kInterpMk = WG / 16;   // markers per CG apply item, 16 lanes each
constexpr int BT = 256;              // threads per workgroup of the single-lattice marker phases

__device__ inline int stencil_base(float X) { return (int)floorf(X) - 1; }

// Tiles of the nodes base..base+3 along one axis (wrapped when periodic),
// one per node; first[s] is false when node s's tile repeats an earlier
// node's. Fixed-size and fully unrolled, so everything stays in registers.
__device__ inline void axis_node_tiles(int base, int n, bool per, int t[4], bool first[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    int j = base + s;
    if (per) j = wrap_idx(j, n);
    t[s] = j >> 3;
    first[s] = true;
#pragma unroll
    for (int q = 0; q < s; ++q) first[s] = first[s] && t[q] != t[s];
  }
}

// Most tiles a stencil touches along an axis of n nodes: two, or three where
// it wraps across a last tile of one or two nodes.
__host__ __device__ inline int axis_tiles_most(int n) {
  const int tiles = (n + 7) >> 3, most = (n & 7) == 1 || (n & 7) == 2 ? 3 : 2;
  return tiles < most ? tiles : most;
}

// (base + 3 - lo) modulo n for base in -1 .. n-2. The stencil base..base+3
// (taken modulo n) has a node in the tile at lo exactly where this is below the
// tile's width plus three.
__device__ inline int axis_from(int base, int n, int lo) {
  const int d = base + 3 - lo;
  return d < 0 ? d + n : (d >= n ? d - n : d);
}

// Value of lane (this lane ^ o) of the wave (ds_bpermute). The lane id
// passes through an empty asm so that its arithmetic is redone where it is
// used: in the persistent kernel, hoisting it out of the step loop would hold
// one register per offset across every phase.
__device__ inline int xor_lane_addr(int o) {
  int lane = __lane_id();
  asm volatile("" : "+v"(lane));
  return (lane ^ o) << 2;
}
__device__ inline int shfl_xor_i(int v, int o) { return __builtin_amdgcn_ds_bpermute(xor_lane_addr(o), v); }
__device__ inline float shfl_xor_f(float v, int o) { return __int_as_float(shfl_xor_i(__float_as_int(v), o)); }

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += shfl_xor_f(v, o);
  return v;
}

__device__ inline bool box_hits(int packed, int t) { return t >= (packed & 0xFFFF) && t <= (packed >> 16); }

// --------------------------------------------------------------- skinning --
// Markers NT*item .. NT*item + NT - 1 with bone poses `pose` into the body set
// bs. Linear blend skinning X = sum_b w_b (R_b xrest + t_b), U = sum_b w_b
// (dR_b xrest + dt_b). Periodic axes: X wrapped into [0, n). Open x: markers
// must satisfy 2 <= X < nx - 3 so the stencil stays on nodes 1 .. nx-2; others
// raise the range guard and are clamped so that every access stays in bounds.
// Item 0 also clears the set's counters. (Always inlined: called as a
// function, its call would hold the persistent kernel's registers across it
// and push that kernel past its budget.)
template <int NT = WG>
__device__ __attribute__((always_inline)) inline void skin_item(const EnvView &e, const BodySet &bs,
                                                                const float *__restrict__ pose, int item, int tid) {
  const int k = item * NT + tid;
  const int n = e.n;
  if (k == 0) {
    bs.counters[0] = 0;  // active tiles of this step
    bs.counters[1] = 0;  // arrival count of the implicit correction's reductions
    bs.counters[2] = 0;  // entries of the marker lists
  }
  const int tns[3] = {e.g.tnx, e.g.tny, (e.g.nz + 7) >> 3};
  const int dims[3] = {e.g.nx, e.g.ny, e.g.nz};
  int lo[3] = {1 << 20, 1 << 20, 1 << 20}, hi[3] = {-1, -1, -1};
  // the environment's arrays through global pointers (see gmem)
  const gmem<float> *xrest = (const gmem<float> *)e.xrest, *nrest = (const gmem<float> *)e.nrest;
  const gmem<float> *weight = (const gmem<float> *)e.weight, *gpose = (const gmem<float> *)pose;
  const gmem<int> *bone = (const gmem<int> *)e.bone;
  gmem<float> *X = (gmem<float> *)bs.X, *U = (gmem<float> *)bs.U;
  gmem<int> *tile_flag = (gmem<int> *)e.tile_flag;
  if (k < n) {
    const float r0 = xrest[k], r1 = xrest[n + k], r2 = xrest[2 * n + k];
    float p[3] = {0.f, 0.f, 0.f}, v[3] = {0.f, 0.f, 0.f}, nv[3] = {0.f, 0.f, 0.f};
    float n0 = 0.f, n1 = 0.f, n2 = 0.f;
    if (e.slip) {
      n0 = nrest[k];
      n1 = nrest[n + k];
      n2 = nrest[2 * n + k];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int b = bone[j * n + k];
      float w = weight[j * n + k];
      if ((unsigned)b >= (unsigned)e.nbones) {
        atomicOr(e.guard, (int)GUARD_BONE);
        b = 0;
        w = 0.f;
      }
      const gmem<float> *P = gpose + 24 * b;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        p[r] += w * (P[3 * r] * r0 + P[3 * r + 1] * r1 + P[3 * r + 2] * r2 + P[9 + r]);
        v[r] += w * (P[12 + 3 * r] * r0 + P[12 + 3 * r + 1] * r1 + P[12 + 3 * r + 2] * r2 + P[21 + r]);
        nv[r] += w * (P[3 * r] * n0 + P[3 * r + 1] * n1 + P[3 * r + 2] * n2);
      }
      // one bone's 24 pose values live at a time: keeps the phase within the
      // register budget of the kernels it is inlined into
      __builtin_amdgcn_sched_barrier(0);
    }
    if (e.slip) {  // the rest normal turned by the blended rotations, unit length
      const float il = rsqrtf(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
#pragma unroll
      for (int r = 0; r < 3; ++r) ((gmem<float> *)bs.Nrm)[r * n + k] = nv[r] * il;
    }
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      const float nn = (float)dims[ax];
      const bool per = ax == 0 ? e.g.xper != 0 : (ax == 1 ? e.g.yper != 0 : e.g.zper != 0);
      if (per) {
        float q = p[ax] - nn * floorf(p[ax] / nn);
        if (!(q >= 0.f && q < nn)) q = 0.f;
        p[ax] = q;
      } else if (!(p[ax] >= 2.0f && p[ax] < nn - 3.0f)) {
        atomicOr(e.guard, (int)GUARD_MARKER_RANGE);
        p[ax] = (p[ax] >= 2.0f) ? nn - 3.5f : 2.0f;
      }
      X[ax * n + k] = p[ax];
      U[ax * n + k] = v[ax];
    }
    const int bs3[3] = {stencil_base(p[0]), stencil_base(p[1]), stencil_base(p[2])};
    gmem<short> *mb = (gmem<short> *)bs.mbase + 4 * (size_t)k;
    mb[0] = (short)bs3[0];
    mb[1] = (short)bs3[1];
    mb[2] = (short)bs3[2];
    mb[3] = 0;
    int tx[4], ty[4], tz[4];
    bool fx[4], fy[4], fz[4];
    axis_node_tiles(bs3[0], e.g.nx, e.g.xper, tx, fx);
    axis_node_tiles(bs3[1], e.g.ny, e.g.yper, ty, fy);
    axis_node_tiles(bs3[2], e.g.nz, e.g.zper, tz, fz);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int l = 0; l < 4; ++l)
          if (fz[i] && fy[j] && fx[l]) tile_flag[tx[l] + e.g.tnx * (ty[j] + e.g.tny * tz[i])] = 1;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      if (bs3[ax] < 0 || bs3[ax] + 3 >= dims[ax]) {  // wrapping stencil: whole axis
        lo[ax] = 0;
        hi[ax] = tns[ax] - 1;
      } else {
        lo[ax] = bs3[ax] >> 3;
        hi[ax] = (bs3[ax] + 3) >> 3;
      }
    }
  }
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo[ax] = min(lo[ax], shfl_xor_i(lo[ax], o));
      hi[ax] = max(hi[ax], shfl_xor_i(hi[ax], o));
    }
  }
  if ((tid & 63) == 0 && k < n) {
    gmem<int> *cb = (gmem<int> *)bs.chunk_box + 4 * (size_t)(k >> 6);
    cb[0] = lo[0] | (hi[0] << 16);
    cb[1] = lo[1] | (hi[1] << 16);
    cb[2] = lo[2] | (hi[2] << 16);
    cb[3] = 0;
  }
}

template <int NT = WG>
__device__ __host__ inline int skin_items(int n) {
  return (n + NT - 1) / NT;
}

// ---------------------------------------------------------- active tiles --
// Tiles NT*item .. NT*item + NT - 1 of the set bs: slots in workgroup order
// from one atomic per workgroup. Slot numbering only decides storage locations,
// never results. Clears the flags for the next step.
template <int NT = WG>
__device__ inline void active_item(const EnvView &e, const BodySet &bs, int item, int tid) {
  __shared__ int s_w[NT / 64];
  __shared__ int s_base;
  const int lane = tid & 63, wv = tid >> 6;
  const int t = item * NT + tid;
  int f = 0;
  if (t < e.ntiles) {
    f = e.tile_flag[t] != 0;
    e.tile_flag[t] = 0;
  }
  const unsigned long long bal = __ballot(f);
  if (lane == 0) s_w[wv] = __popcll(bal);
  __syncthreads();
  if (tid == 0) {
    int tot = 0;
    for (int q = 0; q < NT / 64; ++q) tot += s_w[q];
    s_base = tot ? atomicAdd(&bs.counters[0], tot) : 0;
  }
  __syncthreads();
  int pre = s_base;
  for (int q = 0; q < wv; ++q) pre += s_w[q];
  pre += __popcll(bal & ((1ull << lane) - 1ull));
  if (t < e.ntiles) {
    if (f && pre < e.cap) {
      bs.tile_slot[t] = pre;
      const int tx = t % e.g.tnx, rest = t / e.g.tnx;
      bs.active[pre] = make_int4(tx | ((rest % e.g.tny) << 16), rest / e.g.tny, 0, 0);
    } else {
      bs.tile_slot[t] = -1;
      if (f) atomicOr(e.guard, (int)GUARD_CAPACITY);
    }
  }
  __syncthreads();  // s_w / s_base are reused by the next item
}

template <int NT = WG>
__device__ __host__ inline int active_items(const EnvView &e) {
  return (e.ntiles + NT - 1) / NT;
}
__device__ inline int n_active_of(const EnvView &e, const BodySet &bs) {
  return min(((const gmem<int> *)bs.counters)[0], e.cap);
}
// Coordinates of a slot's tile (stored as such: a band workgroup needs them
// first, and two integer divisions are a third of its index arithmetic) and
// its marker list.
struct TileAt {
  int x, y, z, off, cnt;
};
__device__ inline TileAt active_of(const BodySet &bs, int slot) {
  const gmem<int> *p = (const gmem<int> *)bs.active + 4 * (size_t)slot;
  const int xy = p[0];
  return {xy & 0xFFFF, xy >> 16, p[1], p[2], p[3]};
}

// XCD-contiguous walk over work items 0 .. tot-1. The dispatcher hands
// workgroup b to XCD b % kXcds, and each XCD has its own L2; an active tile's
// x-rows are 8 cells (32 bytes at F32) of 128-byte lines that it shares with
// its x-neighbours, which hold the next slots. Giving each XCD one contiguous
// range of items makes those neighbours meet in one L2 instead of fetching
// each line once per XCD. Every item is visited exactly once for any grid;
// workgroups past the last multiple of kXcds take no items.
constexpr int kXcds = 8;
struct XcdWalk {
  int first, end, step;
};
__device__ inline XcdWalk xcd_walk(int tot, int blk, int grid) {
  const int per = grid / kXcds;
  if (per == 0) return {blk, tot, grid};  // small grid: plain stride
  const int x = blk % kXcds, r = blk / kXcds;
  if (r >= per) return {0, 0, 1};
  const int chunk = (tot + kXcds - 1) / kXcds;
  const int lo = x * chunk, hi = min(tot, lo + chunk);
  return {lo + r, hi, per};
}
__device__ inline XcdWalk xcd_walk(int tot) { return xcd_walk(tot, (int)blockIdx.x, (int)gridDim.x); }

// Item of workgroup blk in a grid of exactly `grid` workgroups, one item each,
// XCD-contiguous: with grid = 8q + m, XCD x (workgroups x, x + 8, ...) takes
// the q + (x < m) consecutive items from x q + min(x, m) on. A bijection of
// 0 .. grid-1, so every item runs once.
__device__ inline int xcd_item(int blk, int grid) {
  const int q = grid / kXcds, m = grid % kXcds, x = blk % kXcds;
  return x * q + min(x, m) + blk / kXcds;
}

// ----------------------------------------------------------- marker lists --
// Appends v to list[*count ...] for the lanes of this wave with `take`, below
// most entries; *count counts them all.
__device__ inline void wave_push(bool take, int v, int *list, int *count, int most, int lane) {
  const unsigned long long bal = __ballot(take);
  if (bal == 0ull) return;
  int at = 0;
  if (lane == 0) at = atomicAdd(count, (int)__popcll(bal));
  at = __builtin_amdgcn_readfirstlane(at) + __popcll(bal & ((1ull << lane) - 1ull));
  if (take && at < most) list[at] = v;
}

// Marker list of active tile `slot`: entries k | d << kListShift for every
// marker k whose stencil touches the tile, d = axis_from of its z (k < 2^24,
// d < 16). Built once
// per step, so that the spreading, whose planes spread over many workgroups,
// starts from it instead of scanning the markers in each. NT threads test the
// chunk boxes, then the markers of the chunks whose box meets the tile, and
// collect the hits in LDS (LDS of them; a longer list is found again and written
// out directly). Order is arbitrary. A wave has PER chunks in flight and takes
// its place in the list once for all of them (a step of a fish of 12,000 markers
// and 40 nodes in 100x52x52, k_step_macro: 22.9 to 14.9 us with 8 chunks instead
// of 4, a place each, and 4,096 hits instead of 1,024).
constexpr int kListLds = 1024;      // batches: the persistent kernel's LDS holds the spreading too
constexpr int kListLdsLone = 4096;  // a single lattice
// 28, not 24: of a marker index masked to 24 bits the compiler (ROCm 7.2) takes
// the record's address as a 24-bit multiply, drops the mask, and then folds it
// into a 32-bit multiply-add, which sees the bits above.
constexpr int kListShift = 28;
template <int NT, int LDS = kListLds, int PER = 4>
__device__ inline void list_item(const EnvView &e, const BodySet &bs, int slot, int tid) {
  __shared__ int s_hit[LDS], s_chunk[NT], s_n[3];  // [0] chunks, [1] hits, [2] first entry
  constexpr int WAVES = NT / 64;
  const GridArgs &g = e.g;
  const TileAt t = active_of(bs, slot);
  const int x0 = t.x * 8, y0 = t.y * 8, z0 = t.z * 8;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wx = min(8, g.nx - x0) + 3, wy = min(8, g.ny - y0) + 3, wz = min(8, g.nz - z0) + 3;
  const int n = e.n, nchunks = (n + 63) >> 6;
  int *out = s_hit;
  int most = LDS, cnt = 0;
  for (int pass = 0; pass < 2; ++pass) {
    if (tid < 2) s_n[tid] = 0;
    __syncthreads();
    for (int c0 = 0; c0 < nchunks; c0 += NT) {
      const int cl = c0 + tid;
      bool meets = false;
      if (cl < nchunks) {
        const gmem<int> *bp = (const gmem<int> *)bs.chunk_box + 4 * (size_t)cl;
        const int4 box = make_int4(bp[0], bp[1], bp[2], bp[3]);
        meets = box_hits(box.x, t.x) && box_hits(box.y, t.y) && box_hits(box.z, t.z);
      }
      wave_push(meets, cl, s_chunk, &s_n[0], NT, lane);
      __syncthreads();
      const int nc = __builtin_amdgcn_readfirstlane(s_n[0]);
      for (int q0 = wv; q0 < nc; q0 += WAVES * PER) {
        short4 base[PER];
        int mk[PER], found = 0;
        unsigned long long bal[PER];
#pragma unroll
        for (int r = 0; r < PER; ++r) {
          mk[r] = n;
          if (q0 + r * WAVES < nc) {
            mk[r] = s_chunk[q0 + r * WAVES] * 64 + lane;
            const gmem<short> *mb = (const gmem<short> *)bs.mbase + 4 * (size_t)min(mk[r], n - 1);
            base[r] = make_short4(mb[0], mb[1], mb[2], mb[3]);
          }
        }
#pragma unroll
        for (int r = 0; r < PER; ++r) {
          bal[r] = 0ull;
          if (q0 + r * WAVES >= nc) continue;
          const int d = axis_from(base[r].z, g.nz, z0);
          bal[r] = __ballot(mk[r] < n && axis_from(base[r].x, g.nx, x0) < wx && axis_from(base[r].y, g.ny, y0) < wy &&
                            d < wz);
          mk[r] = (int)((unsigned)mk[r] | ((unsigned)d << kListShift));
          found += (int)__popcll(bal[r]);
        }
        if (found == 0) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_n[1], found);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int r = 0; r < PER; ++r) {
          const int to = at + (int)__popcll(bal[r] & ((1ull << lane) - 1ull));
          if ((bal[r] >> lane & 1ull) && to < most) out[to] = mk[r];
          at += (int)__popcll(bal[r]);
        }
      }
      __syncthreads();
      if (tid == 0) s_n[0] = 0;
      __syncthreads();
    }
    if (pass == 1) break;
    cnt = s_n[1];
    __syncthreads();
    if (tid == 0) {
      s_n[2] = cnt ? atomicAdd(&bs.counters[2], cnt) : 0;
      gmem<int> *p = (gmem<int> *)bs.active + 4 * (size_t)slot;
      p[2] = s_n[2];
      p[3] = cnt;
    }
    __syncthreads();
    out = e.list + s_n[2];
    most = cnt;
    if (cnt <= LDS) {
      for (int q = tid; q < cnt; q += NT) out[q] = s_hit[q];
      break;
    }
  }
  __syncthreads();  // the LDS arrays are reused by the next item
}

// ----------------------------------------------------------- band macros --
// Density and unforced velocity u* (frame force, no immersed force) at node
// (x, y, z) from the moments of its pulled deviations. Multiply-adds fuse
// within one expression only, so that every kernel this is inlined into
// rounds it the same way. m / rho is rounded before half the frame's
// acceleration is added where that varies over the nodes (ROT), the product with
// it fused otherwise: 2-byte populations carry a last bit that differs here on
// into the forces of later steps (implicit correction, BF16, 12 steps: 2e-3).
template <bool ROT>
__device__ inline vfloat4 macro_of(const FrameF &fr, float drho, float mx, float my, float mz, int x, int y, int z) {
#pragma clang fp contract(on)
  const float rho = 1.0f + drho;
  float ax, ay, az;
  frame_a0<ROT>(fr, (float)x, (float)y, (float)z, ax, ay, az);
  float ux, uy, uz;
  const float ir = 1.0f / rho;
  const float h = 0.5f;
  if (ROT)
    solve_coriolis<ROT>(fr, __builtin_fmaf(h, ax, mx * ir), __builtin_fmaf(h, ay, my * ir),
                        __builtin_fmaf(h, az, mz * ir), ux, uy, uz);
  else
    solve_coriolis<ROT>(fr, __builtin_fmaf(mx, ir, h * ax), __builtin_fmaf(my, ir, h * ay),
                        __builtin_fmaf(mz, ir, h * az), ux, uy, uz);
  return vfloat4{rho, ux, uy, uz};
}

// macro_of cells of active tiles, NT a workgroup: item `item` is the
// (item % (512 / NT))-th part of tile item / (512 / NT).
template <int NT, class S, bool ROT>
__device__ inline void macro_item(const EnvView &e, const BodySet &bs, const FrameF &fr, int cur, int item, int tid0) {
  const int slot = item / (512 / NT), tid = item % (512 / NT) * NT + tid0;
  using T = typename S::T;
  const gmem<T> *__restrict__ src = (const gmem<T> *)e.f[cur];
  const GridArgs &g = e.g;
  const TileAt t = active_of(bs, slot);
  const int x = t.x * 8 + (tid & 7), y = t.y * 8 + ((tid >> 3) & 7), z = t.z * 8 + (tid >> 6);
  vfloat4 out = {1.f, 0.f, 0.f, 0.f};
  if (x < g.nx && y < g.ny && z < g.nz && (g.xper || (x > 0 && x < g.nx - 1))) {
    const int xm = g.xper ? wrap_idx(x - 1, g.nx) : x - 1;
    const int xp = g.xper ? wrap_idx(x + 1, g.nx) : x + 1;
    float f[Q];  // deviations h_i = f_i - w_i
    pull27<S, true>(src, g, xm, x, xp, wrap_idx(y - 1, g.ny), y, wrap_idx(y + 1, g.ny),
                    wrap_idx(z - 1, g.nz), z, wrap_idx(z + 1, g.nz), f);
    float drho, mx, my, mz;
    moments(f, drho, mx, my, mz);
    out = macro_of<ROT>(fr, drho, mx, my, mz, x, y, z);
  }
  ((gmem<vfloat4> *)e.macro)[(size_t)slot * 512 + tid] = out;
}

// --------------------------------------------------------- interpolation --
// pass 0: U*_k = sum u* delta, rho_k = sum rho delta, F_k = 2 alpha rho_k (U_k - U*_k).
// pass p > 0 (multi-direct forcing): the interpolated velocity includes the
// current immersed force, u = u* + (I + [omega]x)^-1 g / (2 rho), and
// F_k += 2 alpha rho_k (U_k - U_k^interp).
// The record carries this pass's F increment times dV (spreading adds each
// pass into the step's force). With partials != nullptr: the markers' shares of
// the fluid's force, torque about the frame origin and power, eight floats each:
// summed over kShareMk consecutive markers, a row of the partials each
// (interp_item), or a row per marker (interp_wave).
// Node weight delta = wx (wy wz), the product the spreading uses. The 64-node
// sums add each x-row of four nodes in order, then the 16 rows by a butterfly,
// in both forms below: the same bits.
//   interp_item  (from the band macros) 16 lanes a marker, one x-row a lane;
//   interp_wave  (from the populations) one wave a marker, one node a lane: no
//                macro pass before it, for few markers.
// Value of the lane N places on in its row of 16 (DPP rotation: a register
// operand, where a shuffle goes through LDS). Where the values repeat with
// period 2 N over the row (N = 8 always), that is the value of lane ^ N.
template <int N>
__device__ inline float row_turn(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xF, 0xF, true));
}
// Sum over each 16 lanes, the same bits in all of them: a butterfly of xors.
__device__ inline float group16_sum(float v) {
  v += row_turn<8>(v);
  v += row_turn<4>(v);
  v += row_turn<2>(v);
  v += row_turn<1>(v);
  return v;
}

// Value of lane `lane` of the wave.
__device__ inline float lane_f(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(lane << 2, __float_as_int(v)));
}

// Stencil weights of a marker at X: lane q < 12 of the marker's lanes gets
// the weight of node q & 3 on axis q >> 2 (one square root a lane instead of
// six), the others a value nobody reads.
__device__ inline float stencil_weight(const float X[3], const int base[3], int q) {
  const int ax = min(q >> 2, 2);
  const float x = ax == 0 ? X[0] : (ax == 1 ? X[1] : X[2]);
  const int b = ax == 0 ? base[0] : (ax == 1 ? base[1] : base[2]);
  return peskin4(x - (float)(b + (q & 3)));
}

constexpr int kShareMk = 16;  // markers per row of the wrench partials
__device__ __host__ inline int share_rows(int n) { return (n + kShareMk - 1) / kShareMk; }

// What one lane does with marker k's sums: force, record and wrench share
// (the record's weights are stored by the caller).
template <bool MDF>
__device__ inline void force_marker(const EnvView &e, const BodySet &bs, const FrameF &fr, int k, float sr,
                                    const float Ui[3], const float Xk[3], const float Uk[3], float dvk,
                                    const int base[3], float part[7]) {
  // multiply-adds fuse only within one expression, never across statements,
  // so every kernel that inlines this rounds its outputs identically
#pragma clang fp contract(on)
  const int n = e.n;
  gmem<float> *F = (gmem<float> *)e.F, *mstate = (gmem<float> *)e.mstate;
  gmem<float> *r = (gmem<float> *)e.rec + (size_t)k * REC;
  float rk, Fk[3], inc[3];
  // velocity to correct: U - U^interp, or on a slip wall its normal part
  float dU[3] = {Uk[0] - Ui[0], Uk[1] - Ui[1], Uk[2] - Ui[2]};
  if (e.slip) {
    const float nk[3] = {bs.Nrm[k], bs.Nrm[n + k], bs.Nrm[2 * n + k]};
    const float dn = dU[0] * nk[0] + dU[1] * nk[1] + dU[2] * nk[2];
#pragma unroll
    for (int c = 0; c < 3; ++c) dU[c] = dn * nk[c];
  }
  if (!MDF) {
    rk = sr;
    mstate[k] = rk;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      mstate[(c + 1) * (size_t)n + k] = Ui[c];
      inc[c] = e.alpha2 * rk * dU[c];
      Fk[c] = inc[c];
    }
  } else {
    rk = mstate[k];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      inc[c] = e.alpha2 * rk * dU[c];
      Fk[c] = F[c * n + k] + inc[c];
    }
  }
  float fd[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    F[c * n + k] = Fk[c];
    fd[c] = Fk[c] * dvk;
  }
  *(gmem<vfloat4> *)(r + 12) = vfloat4{__int_as_float(base[0]), __int_as_float(base[1]), __int_as_float(base[2]), 0.f};
  *(gmem<vfloat4> *)(r + 16) = vfloat4{inc[0] * dvk, inc[1] * dvk, inc[2] * dvk, 0.f};
  // fluid on body: -F dV; torque (X - x0) x (-F dV); power F.U dV
  const float rx = Xk[0] - fr.org[0], ry = Xk[1] - fr.org[1], rz = Xk[2] - fr.org[2];
  part[0] = -fd[0];
  part[1] = -fd[1];
  part[2] = -fd[2];
  part[3] = -(ry * fd[2] - rz * fd[1]);
  part[4] = -(rz * fd[0] - rx * fd[2]);
  part[5] = -(rx * fd[1] - ry * fd[0]);
  part[6] = fd[0] * Uk[0] + fd[1] * Uk[1] + fd[2] * Uk[2];
}

// Column `col` of row r of the wrench partials, added in marker order: share(q)
// is that of the row's q-th marker, zero past the last one.
template <class F>
__device__ inline float share_sum(F share) {
  float sum = 0.f;
#pragma unroll
  for (int q = 0; q < kShareMk; ++q) sum += share(q);
  return sum;
}

// Markers NT / 16 a workgroup, from the band macros.
template <int NT, bool ROT, bool MDF>
__device__ inline void interp_item(const EnvView &e, const BodySet &bs, const FrameF &fr, int item, int tid,
                                   float *partials) {
#pragma clang fp contract(on)  // as force_marker
  const int sub = tid & 15, lane = tid & 63;
  const int k = item * (NT / 16) + (tid >> 4);
  const int n = e.n;
  const GridArgs &g = e.g;
  const bool live = k < n;
  // the environment's arrays through global pointers (see gmem)
  const gmem<float> *X = (const gmem<float> *)bs.X, *U = (const gmem<float> *)bs.U;
  const gmem<int> *tile_slot = (const gmem<int> *)bs.tile_slot;
  float Xk[3] = {0.f, 0.f, 0.f}, Uk[3] = {0.f, 0.f, 0.f}, dvk = 0.f;
  int base[3] = {0, 0, 0};
  float sr = 0.f, sx = 0.f, sy = 0.f, sz = 0.f;
  if (live) {
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      Xk[ax] = X[ax * n + k];
      // loaded now, used after the stencil gather: off the dependent chain
      Uk[ax] = U[ax * n + k];
      base[ax] = stencil_base(Xk[ax]);
    }
    dvk = ((const gmem<float> *)e.dv)[k];
  }
  // every lane takes part in the shuffles (a group of 16 is all live or all not)
  const float w = stencil_weight(Xk, base, sub);
  const int grp = lane & 48;
  float wx[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) wx[i] = lane_f(w, grp + i);
  const float wy = lane_f(w, grp + 4 + (sub & 3)), wz = lane_f(w, grp + 8 + (sub >> 2));
  if (live) {
    const int yn = wrap_idx(base[1] + (sub & 3), g.ny), zn = wrap_idx(base[2] + (sub >> 2), g.nz);
    const int trow = g.tnx * ((yn >> 3) + g.tny * (zn >> 3));
    const int lrow = ((yn & 7) << 3) | ((zn & 7) << 6);
    int sl[4], lc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int xn = g.xper ? wrap_idx(base[0] + i, g.nx) : base[0] + i;
      sl[i] = tile_slot[(xn >> 3) + trow];
      lc[i] = (xn & 7) | lrow;
    }
    vfloat4 m[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m[i] = vfloat4{0.f, 0.f, 0.f, 0.f};
      if (sl[i] >= 0)
        m[i] = ((const gmem<vfloat4> *)e.macro)[(size_t)sl[i] * 512 + lc[i]];
      else  // a tile beyond the capacity
        atomicOr(e.guard, (int)GUARD_CAPACITY);
    }
    if (MDF) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (sl[i] < 0) continue;
        const gmem<unsigned long long> *gp = (const gmem<unsigned long long> *)e.gfix + (size_t)sl[i] * 1536;
        const float h = 0.5f / m[i].x;
        float dx, dy, dz;
        solve_coriolis<ROT>(fr, from_fix(gp[lc[i]]) * h, from_fix(gp[512 + lc[i]]) * h, from_fix(gp[1024 + lc[i]]) * h,
                            dx, dy, dz);
        m[i].y += dx;
        m[i].z += dy;
        m[i].w += dz;
      }
    }
    const float wyz = wy * wz;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float d = wx[i] * wyz;
      sr += m[i].x * d;
      sx += m[i].y * d;
      sy += m[i].z * d;
      sz += m[i].w * d;
    }
  }
  sr = group16_sum(sr);
  sx = group16_sum(sx);
  sy = group16_sum(sy);
  sz = group16_sum(sz);
  float part[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (live) {
    if (sub < 12) ((gmem<float> *)e.rec)[(size_t)k * REC + sub] = w;
    const float Ui[3] = {sx, sy, sz};
    if (sub == 0) force_marker<MDF>(e, bs, fr, k, sr, Ui, Xk, Uk, dvk, base, part);
  }
  if (partials == nullptr) return;  // uniform over the workgroup
  constexpr int ROWS = NT / 16 / kShareMk;
  __shared__ float s_part[NT / 16][8];
  if (sub == 0)
    for (int q = 0; q < 7; ++q) s_part[tid >> 4][q] = part[q];
  __syncthreads();
  const int row = item * ROWS + (tid >> 3), col = tid & 7;
  if (tid < 8 * ROWS && row < share_rows(n))
    ((gmem<float> *)partials)[(size_t)row * 8 + col] =
        col < 7 ? share_sum([&](int q) { return s_part[(tid >> 3) * kShareMk + q][col]; }) : 0.f;
  __syncthreads();  // s_part is reused by the next item
}

// Value of lane i of this lane's group of four (DPP quad permute).
template <int I>
__device__ inline float quad_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), I * 0x55, 0xF, 0xF, true));
}

// Marker k by one wave (k uniform over it), first pass, straight from the
// populations of buffer cur: lane = node (lane & 3, (lane >> 2) & 3, lane >> 4)
// pulls its 27 populations and takes their moments, as macro_item does for the
// cells of the band, so no macro pass goes before.
template <class S, bool ROT>
__device__ inline void interp_wave(const EnvView &e, const BodySet &bs, const FrameF &fr, int cur, int k, int lane,
                                   float *partials) {
#pragma clang fp contract(on)  // as force_marker
  using T = typename S::T;
  const gmem<T> *__restrict__ src = (const gmem<T> *)e.f[cur];
  const GridArgs &g = e.g;
  const int n = e.n;
  const gmem<float> *X = (const gmem<float> *)bs.X, *U = (const gmem<float> *)bs.U;
  float Xk[3], Uk[3];
  int base[3];
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    Xk[ax] = X[ax * n + k];
    Uk[ax] = U[ax * n + k];
    base[ax] = stencil_base(Xk[ax]);
  }
  const float dvk = ((const gmem<float> *)e.dv)[k];
  const int x = g.xper ? wrap_idx(base[0] + (lane & 3), g.nx) : base[0] + (lane & 3);
  const int y = wrap_idx(base[1] + ((lane >> 2) & 3), g.ny), z = wrap_idx(base[2] + (lane >> 4), g.nz);
  const int sl = ((const gmem<int> *)bs.tile_slot)[(x >> 3) + g.tnx * ((y >> 3) + g.tny * (z >> 3))];
  float f[Q];  // deviations h_i
  pull27<S, true>(src, g, wrap_idx(x - 1, g.nx), x, wrap_idx(x + 1, g.nx), wrap_idx(y - 1, g.ny), y,
                  wrap_idx(y + 1, g.ny), wrap_idx(z - 1, g.nz), z, wrap_idx(z + 1, g.nz), f);
  // the weights while the populations are in flight
  const float w = stencil_weight(Xk, base, lane);
  const float wyz = lane_f(w, 4 + ((lane >> 2) & 3)) * lane_f(w, 8 + (lane >> 4));
  const float d = lane_f(w, lane & 3) * wyz;
  if (lane < 12) ((gmem<float> *)e.rec)[(size_t)k * REC + lane] = w;
  float drho, mx, my, mz;
  moments(f, drho, mx, my, mz);
  vfloat4 m = macro_of<ROT>(fr, drho, mx, my, mz, x, y, z);
  if (sl < 0) {  // a tile beyond the capacity
    m = vfloat4{0.f, 0.f, 0.f, 0.f};
    atomicOr(e.guard, (int)GUARD_CAPACITY);
  }
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  const float q[4] = {m.x, m.y, m.z, m.w};
  const float d0 = quad_lane<0>(d), d1 = quad_lane<1>(d), d2 = quad_lane<2>(d), d3 = quad_lane<3>(d);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    s[c] += quad_lane<0>(q[c]) * d0;
    s[c] += quad_lane<1>(q[c]) * d1;
    s[c] += quad_lane<2>(q[c]) * d2;
    s[c] += quad_lane<3>(q[c]) * d3;
  }
  // the 16 rows: lanes 4 apart, the butterfly of group16_sum
#pragma unroll
  for (int o = 32; o >= 16; o >>= 1)
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] += shfl_xor_f(s[c], o);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    s[c] += row_turn<8>(s[c]);
    s[c] += row_turn<4>(s[c]);
  }
  const float Ui[3] = {s[1], s[2], s[3]};
  if (lane == 0) {
    float part[7];
    force_marker<false>(e, bs, fr, k, s[0], Ui, Xk, Uk, dvk, base, part);
    if (partials != nullptr) {
      gmem<vfloat4> *p = (gmem<vfloat4> *)(partials + 8 * (size_t)k);
      p[0] = vfloat4{part[0], part[1], part[2], part[3]};
      p[1] = vfloat4{part[4], part[5], part[6], 0.f};
    }
  }
}

template <int NT = WG>
__device__ __host__ inline int interp_items(int n) {
  return (n + NT / 16 - 1) / (NT / 16);
}
__device__ __host__ inline int wave_items(int n) { return (n + kWavePer - 1) / kWavePer; }

// Wrench of the step by NT threads, in a fixed order whatever NT and the kernel:
// the markers' shares by rows of kShareMk (partials holds the rows, or by_marker
// the shares), the rows as WG / 8 interleaved sums and those one after the other,
// from the rows on in double precision, so that the rounding doesn't grow with
// the number of markers. One workgroup does it, in the launch that the step ends
// with: added marker by marker it was that launch's tail (12,000 markers on
// 384x192x192 in launches of their own: 553 us a step, 540 by rows; 200,000 on
// 192x96x96: 515 and 283).
template <int NT>
__device__ inline void wrench_sum(const float *__restrict__ partials, int n, bool by_marker,
                                  float *__restrict__ wrench, int tid) {
  __shared__ double s_red[WG];
  const gmem<float> *p = (const gmem<float> *)partials;
  const int rows = share_rows(n);
  for (int q = tid; q < WG; q += NT) {
    const int col = q & 7;
    double acc = 0.0;
    if (col < 7 && by_marker) {
      for (int r = q >> 3; r < rows; r += WG / 8)
        acc += share_sum([&](int j) {
          const int k = r * kShareMk + j;
          return k < n ? p[(size_t)k * 8 + col] : 0.f;
        });
    } else if (col < 7) {
#pragma unroll 8
      for (int r = q >> 3; r < rows; r += WG / 8) acc += p[(size_t)r * 8 + col];
    }
    s_red[q] = acc;
  }
  __syncthreads();
  if (tid < 8) {
    double sum = 0.0;
    for (int r2 = 0; r2 < WG / 8; ++r2) sum += s_red[r2 * 8 + tid];
    wrench[tid] = tid < 7 ? (float)sum : 0.f;
  }
  __syncthreads();
}

// --------------------------------------------------------------- spreading --
// The immersed force of one z-plane (64 cells) of an active tile per 256
// threads: g(x) = sum_k F_k dV_k delta(x - X_k). The plane's markers, those
// entries of the tile's list whose stencil has a node at this z, are collected in
// LDS, up to kHits of the list at a time; four lanes each take one, one lane per
// x-row of the stencil in this plane, which adds the row's nodes inside the
// tile into the plane's LDS cells with 64-bit LDS atomics (2^-40 fixed point).
// Integer sums make the result independent of every order, and a plane belongs
// to one workgroup, so its force is stored, or used from LDS, without global
// atomics.
// Planes, not tiles: the markers of a thin body crowd into few tiles (the
// 128x64x64 fin has 32 active ones, with up to 579 of its 3,000 markers), and
// the conversion to fixed point and the LDS atomics of one crowded tile on one
// compute unit were the whole phase's time. Two markers in flight in each group of
// four lanes, read where they are used, and no branch on a node: the conversions
// of 24 nodes' values overlap. k_spread, 12,000 markers of a fish of 40 nodes in
// 100x52x52: 28.1 us, 36.3 with a branch a node (28.7 with the values pinned
// before it), 31.0 with four markers, 30.9 with one and the next one's loads
// ahead; 36 when the records were staged in LDS, 256 at a time. The search
// direction takes one marker, a component a lane (the 128x64x64 fin, k_spread_cg:
// 8.4 us, 9.0 with two markers, 10.9 with all three components in each lane).
constexpr int kHits = 1024;

// w[q] becomes w[(q + r) & 3].
__device__ inline void rotate4(float (&w)[4], int r) {
  const float a0 = r & 1 ? w[1] : w[0], a1 = r & 1 ? w[2] : w[1], a2 = r & 1 ? w[3] : w[2], a3 = r & 1 ? w[0] : w[3];
  w[0] = r & 2 ? a2 : a0;
  w[1] = r & 2 ? a3 : a1;
  w[2] = r & 2 ? a0 : a2;
  w[3] = r & 2 ? a1 : a3;
}

template <int NC>
struct alignas(16) SpreadLds {
  unsigned long long acc[2 * NC][64];  // the plane's cells; the second half takes the nodes outside, and is not read
  int hit[kHits];  // k | node << kListShift: the marker and its stencil node at this z
  int nhit;
};

__device__ inline float cg_direction(const EnvView &e, int k, int c, float beta, bool first);

// Plane `plane` of tile t by the 256 threads tid = 0 .. 255 (each 256 threads
// of a larger workgroup take a plane of the same tile). The record's values
// from FIRST on (NC of them) are spread; CG: instead the search direction of
// the implicit correction's conjugate-gradient step (cg_direction with beta,
// first). s.acc holds the start value (visible after the first barrier here);
// a barrier ends the call.
template <bool CG, int NC = 3, int FIRST = 16, int U = CG ? 1 : 2>
__device__ inline void spread_plane(const EnvView &e, const BodySet &bs, const TileAt &t, int plane, int tid,
                                    SpreadLds<NC> &s, const float *beta = nullptr, bool first = true) {
  const GridArgs &g = e.g;
  const int x0 = t.x * 8, y0 = t.y * 8, lane = tid & 63;
  const int n = e.n;
  const gmem<int> *list = (const gmem<int> *)e.list + t.off;
  constexpr int PER = kHits / 256, kMask = (1 << kListShift) - 1;
  const int cc = min(lane & 3, 2);
  const float bc = CG && !first ? beta[cc] : 0.f;
  for (int c0 = 0; c0 < t.cnt; c0 += kHits) {
    int entry[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) entry[r] = c0 + 256 * r + tid < t.cnt ? list[c0 + 256 * r + tid] : 0;
    if (tid == 0) s.nhit = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      if (c0 + 256 * r >= t.cnt) break;  // uniform
      int sz = plane + 3 - (int)((unsigned)entry[r] >> kListShift);  // the stencil node at this z, modulo nz
      sz = sz < 0 ? sz + g.nz : (sz >= g.nz ? sz - g.nz : sz);
      const bool hit = c0 + 256 * r + tid < t.cnt && sz < 4;
      wave_push(hit, (int)((unsigned)(entry[r] & kMask) | (unsigned)sz << kListShift), s.hit, &s.nhit, kHits, lane);
    }
    __syncthreads();
    const int m = s.nhit;
    for (int j0 = tid >> 2; j0 < m; j0 += 64 * U) {
      vfloat4 wx[U], ba[U], fd[U];  // the record: x weights, base and value 15, values 16 .. 18
      float wyz[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int h = s.hit[min(j0 + 64 * u, m - 1)], k = h & kMask;
        const gmem<float> *rp = (const gmem<float> *)e.rec + (size_t)k * REC;
        wx[u] = *(const gmem<vfloat4> *)rp;
        ba[u] = *(const gmem<vfloat4> *)(rp + 12);
        fd[u] = *(const gmem<vfloat4> *)(rp + 16);
        wyz[u] = rp[4 + (lane & 3)] * rp[8 + (int)((unsigned)h >> kListShift)];
        if (CG) {  // a component in each of the first three lanes of the four
          float p = cg_direction(e, k, cc, bc, first);
          if (e.slip) p = quad_lane<0>(p) * bs.Nrm[(size_t)cc * n + k];  // the search direction is a normal force p n
          fd[u] = vfloat4{quad_lane<0>(p), quad_lane<1>(p), quad_lane<2>(p), 0.f};
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int ly = wrap_idx(__float_as_int(ba[u].y) + (lane & 3), g.ny) - y0;
        const bool row = j0 + 64 * u < m && (unsigned)ly < 8u;
        // neighbouring markers start at different nodes of their rows: a wave's
        // markers crowd on the same cells, and LDS atomics on one cell come one
        // after the other (48 lattices of 4,045 markers: 149 to 116 us with a
        // wave a plane, 93 to 73 with 256 threads)
        float w[4] = {wx[u].x, wx[u].y, wx[u].z, wx[u].w};
        rotate4(w, lane >> 2);
        const float v[4] = {ba[u].w, fd[u].x, fd[u].y, fd[u].z};  // record values 15 .. 18
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int bx = __float_as_int(ba[u].x) + ((q + (lane >> 2)) & 3);
          const int lx = (g.xper ? wrap_idx(bx, g.nx) : bx) - x0;
          const int cell = row && (unsigned)lx < 8u ? lx | (ly << 3) : 64 * NC + lane;
          const float d = w[q] * wyz[u];
#pragma unroll
          for (int c = 0; c < NC; ++c) atomicAdd(&s.acc[0][0] + 64 * c + cell, to_fix(v[FIRST - 15 + c] * d));
        }
      }
    }
    __syncthreads();
  }
  if (t.cnt == 0) __syncthreads();
}

// Spreading items of NT threads per active tile: NT / 256 planes each.
template <int NT>
constexpr int kSpreadParts = 8 * 256 / NT;

// Item `item` of the spreading into target (NC planes of 512 cells per slot);
// add: on top of what it holds (the earlier passes of multi-direct forcing).
template <int NT, bool CG, int NC = 3, int FIRST = 16>
__device__ inline void spread_item(const EnvView &e, const BodySet &bs, int item, int tid, unsigned long long *target,
                                   bool add, const float *beta = nullptr, bool first = true) {
  __shared__ SpreadLds<NC> lds[NT / 256];
  SpreadLds<NC> &s = lds[tid / 256];
  const int slot = item / kSpreadParts<NT>, plane = item % kSpreadParts<NT> * (NT / 256) + tid / 256, lt = tid % 256;
  gmem<unsigned long long> *gp = (gmem<unsigned long long> *)target + (size_t)slot * NC * 512 + plane * 64;
  const TileAt t = active_of(bs, slot);
  for (int q = lt; q < NC * 64; q += 256) (&s.acc[0][0])[q] = add ? gp[512 * (q >> 6) + (q & 63)] : 0ull;
  spread_plane<CG, NC, FIRST>(e, bs, t, plane, lt, s, beta, first);
  for (int q = lt; q < NC * 64; q += 256) gp[512 * (q >> 6) + (q & 63)] = (&s.acc[0][0])[q];
  __syncthreads();
}

// ----------------------------------------------- single-lattice launches --
__global__ void __launch_bounds__(BT) k_skin_mark(EnvView e, const float *pose) {
  skin_item<BT>(e, e.b[0], pose, blockIdx.x, threadIdx.x);
}

__global__ void __launch_bounds__(WG) k_active(EnvView e) { active_item(e, e.b[0], blockIdx.x, threadIdx.x); }

template <class S, bool ROT>
__global__ void __launch_bounds__(WG) k_macro(EnvView e, FrameF fr, int cur) {
  const XcdWalk w = xcd_walk(n_active_of(e, e.b[0]));
  for (int slot = w.first; slot < w.end; slot += w.step) {
    list_item<WG, kListLdsLone, 8>(e, e.b[0], slot, threadIdx.x);
    macro_item<WG, S, ROT>(e, e.b[0], fr, cur, slot, threadIdx.x);
  }
}

// Grid: exactly interp_items<BT>(n) workgroups. The markers of one XCD are
// consecutive, so its L2 holds the band macros of their stretch of body.
template <bool ROT, bool MDF>
__global__ void __launch_bounds__(BT) k_interp(EnvView e, FrameF fr, float *partials) {
  interp_item<BT, ROT, MDF>(e, e.b[0], fr, xcd_item(blockIdx.x, gridDim.x), threadIdx.x, partials);
}

// wrench != nullptr: workgroup 0 first sums the interpolation partials.
__global__ void __launch_bounds__(BT) k_spread(EnvView e, float *wrench, int add) {
  if (blockIdx.x == 0 && wrench != nullptr) wrench_sum<BT>(e.partials, e.n, false, wrench, threadIdx.x);
  const int items = kSpreadParts<BT> * n_active_of(e, e.b[0]);
  for (int item = blockIdx.x; item < items; item += gridDim.x)
    spread_item<BT, false>(e, e.b[0], item, threadIdx.x, e.gfix, add != 0);
}

// ------------------------------------------- implicit velocity correction --
// The marker forces G_k = F_k dV_k solve S G = (I + [omega]x)(U - U*) with
// S = interp . 1/(2 rho) . spread (the implicit immersed boundary of Wu and
// Shu, cited in the paper's Introduction): interpolating u* + M spread(G) /
// (2 rho) then gives U at every marker, M = (I + [omega]x)^-1 the Coriolis
// solve of the fluid velocity. M is the same at every node, so S acts on each
// component alone and is symmetric positive semidefinite; conjugate
// gradients with the diagonal preconditioner 2 rho_k (S's diagonal is
// (3/8)^3 / (2 rho) for a uniform density) take mdf_iters steps from G = 0.
// The spread and the interpolation of S use the weights of the marker record,
// so the discrete S is exactly symmetric up to float rounding. On a slip wall
// the unknown is one normal force gamma_k n_k per marker: the vectors keep it
// in component 0 (the others stay zero, and their guarded alpha and beta
// vanish), the spread takes p n and the apply the normal part of S p n,
// (N^T S N) gamma = N^T (U - U*); the frame must not rotate.
//
// Per step, after the first interpolation pass (rho_k, U*_k, record):
//   cg_init_item     r = (I + [omega]x)(U - U*), G = 0; rz_0 = r.z, z = 2 rho_k r
//   step j = 0, 1, ...:
//     spread (CG)    p_j = z_j + beta_j p_{j-1} (p_0 = z_0) computed per
//                    marker hit, spread into gcg
//     cg_apply_item  q = S p_j from gcg; stores p_j and q; p.q rows
//     cg_update_item alpha_j = rz_j / p_j.q; G += alpha_j p_j; r -= alpha_j q;
//                    rz_{j+1};
//                    beta_{j+1} = rz_{j+1} / rz_j; on the last step F = G / dV,
//                    the record carries G, wrench partials
//   then the ordinary spread of the record into gfix.
// Each dot product is a sum of per-workgroup partial rows added in row order:
// p.q by every update workgroup; r.z by the init or update workgroup that
// arrives last (cg_last_arrival), which stores rz and beta for the kernels
// that follow. Every workgroup uses the same values, and the step is
// deterministic.
constexpr int kCgWG = 256;     // markers per init and update workgroup
constexpr int kCgMaxSteps = 16;
__device__ __host__ inline int cg_items(int n) { return (n + kCgWG - 1) / kCgWG; }
// Partial rows and scalars, 4 floats each: p.q rows (one per apply
// workgroup), r.z rows (one per init/update workgroup), then rz_j and beta_j
// for j = 0 .. kCgMaxSteps.
__device__ __host__ inline size_t cg_part_floats(int n) {
  return 4 * ((size_t)interp_items(n) + (size_t)cg_items(n) + 2 * (kCgMaxSteps + 1));
}
__device__ inline float *cg_pq(const EnvView &e) { return e.cgpart; }
__device__ inline float *cg_rzp(const EnvView &e) { return e.cgpart + 4 * (size_t)interp_items(e.n); }
__device__ inline float *cg_scal(const EnvView &e, int which, int j) {  // which: 0 rz, 1 beta
  return cg_rzp(e) + 4 * (size_t)cg_items(e.n) + 4 * (size_t)(which * (kCgMaxSteps + 1) + j);
}

// Sums of parts[j][0..2] over j < m in row order, by the whole workgroup (a
// multiple of 64 threads, at most 1024). Ends with a barrier.
__device__ inline void cg_sum3(const float *__restrict__ parts, int m, float out[3]) {
  __shared__ float s[3][16];
  const int tid = threadIdx.x, nt = blockDim.x;
  float a[3] = {0.f, 0.f, 0.f};
  for (int j = tid; j < m; j += nt)
#pragma unroll
    for (int c = 0; c < 3; ++c) a[c] += parts[4 * (size_t)j + c];
#pragma unroll
  for (int c = 0; c < 3; ++c) a[c] = wave_sum(a[c]);
  if ((tid & 63) == 0)
#pragma unroll
    for (int c = 0; c < 3; ++c) s[c][tid >> 6] = a[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    float t = 0.f;
    for (int w = 0; w < (nt >> 6); ++w) t += s[c][w];
    out[c] = t;
  }
  __syncthreads();
}

// Workgroup sums of v[0..2] written to part[0..2] by thread 0. Ends with a
// barrier.
__device__ inline void cg_part3(const float v[3], float *__restrict__ part) {
  __shared__ float s[3][16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  float w[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) w[c] = wave_sum(v[c]);
  if (lane == 0)
#pragma unroll
    for (int c = 0; c < 3; ++c) s[c][wv] = w[c];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float t = 0.f;
      for (int q = 0; q < (int)(blockDim.x >> 6); ++q) t += s[c][q];
      part[c] = t;
    }
  __syncthreads();
}

// Called by every thread of each of `count` workgroups after thread 0 has
// written the workgroup's partial row: true in the workgroup that arrives
// last, which then sees every row. That workgroup resets the counter for the
// next kernel.
__device__ inline bool cg_last_arrival(int *counter, int count) {
  __shared__ int s_last;
  if (threadIdx.x == 0) {
    __threadfence();  // the row, visible device-wide before the arrival
    const int prev = atomicAdd(counter, 1);
    s_last = prev == count - 1 ? 1 : 0;
    if (s_last) atomicExch(counter, 0);
  }
  __syncthreads();
  const bool last = s_last != 0;
  if (last) __threadfence();
  return last;
}

// Component c of the search direction of marker k: p = z + beta p_prev,
// z = 2 rho_k r (p = z on the first step).
__device__ inline float cg_direction(const EnvView &e, int k, int c, float beta, bool first) {
  const int n = e.n;
  const float *r = e.cg + 3 * (size_t)n, *pp = e.cg + 6 * (size_t)n;
  const float z = 2.0f * e.mstate[k] * r[c * n + k];
  return first ? z : z + beta * pp[c * n + k];
}

template <bool ROT>
__device__ inline void cg_init_item(const EnvView &e, const BodySet &bs, const FrameF &fr, int item) {
  const int n = e.n, k = item * kCgWG + (int)threadIdx.x;
  float rz[3] = {0.f, 0.f, 0.f};
  if (k < n) {
    float R[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) R[c] = bs.U[c * n + k] - e.mstate[(c + 1) * (size_t)n + k];
    float r[3] = {R[0], R[1], R[2]};
    if (ROT) {
      float wx, wy, wz;
      cross3(fr.omg, R[0], R[1], R[2], wx, wy, wz);
      r[0] += wx;
      r[1] += wy;
      r[2] += wz;
    }
    if (e.slip) {  // one unknown per marker, the normal force: r = n.(U - U*) in component 0
      r[0] = bs.Nrm[k] * R[0] + bs.Nrm[n + k] * R[1] + bs.Nrm[2 * (size_t)n + k] * R[2];
      r[1] = r[2] = 0.f;
    }
    const float p2 = 2.0f * e.mstate[k];
    float *G = e.cg, *rr = e.cg + 3 * (size_t)n;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      G[c * n + k] = 0.f;
      rr[c * n + k] = r[c];
      rz[c] = r[c] * (p2 * r[c]);
    }
  }
  cg_part3(rz, cg_rzp(e) + 4 * (size_t)item);
  if (cg_last_arrival(bs.counters + 1, cg_items(n))) {
    float t[3];
    cg_sum3(cg_rzp(e), cg_items(n), t);
    if (threadIdx.x < 3) cg_scal(e, 0, 0)[threadIdx.x] = t[threadIdx.x];
  }
}

// Markers 32*item .. 32*item+31, 16 lanes each, lane = x-row of stencil
// nodes (as interp_item): q_k = sum_x delta(x - X_k) gcg(x) / (2 rho(x)) with
// gcg the spread of step j's search direction, which is stored here. The
// weights are the record's, multiplied as the spreading multiplies them, so
// the discrete S is symmetric.
__device__ inline void cg_apply_item(const EnvView &e, const BodySet &bs, int item, int tid, int j) {
#pragma clang fp contract(on)  // as interp_item
  __shared__ float s_pq[kInterpMk][3];
  const int sub = tid & 15, mk = tid >> 4;
  const int k = item * kInterpMk + mk;
  const int n = e.n;
  const GridArgs &g = e.g;
  const bool live = k < n;
  float pq[3] = {0.f, 0.f, 0.f};
  float v[3] = {0.f, 0.f, 0.f};
  if (live) {
    const float *r = e.rec + (size_t)k * REC;
    const int jy = __float_as_int(r[13]) + (sub & 3), jz = __float_as_int(r[14]) + (sub >> 2);
    const int bx = __float_as_int(r[12]);
    const float wyz = r[4 + (sub & 3)] * r[8 + (sub >> 2)];
    const int yn = wrap_idx(jy, g.ny), zn = wrap_idx(jz, g.nz);
    const int trow = g.tnx * ((yn >> 3) + g.tny * (zn >> 3));
    const int lrow = ((yn & 7) << 3) | ((zn & 7) << 6);
    int sl[4], lc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int xn = g.xper ? wrap_idx(bx + i, g.nx) : bx + i;
      sl[i] = bs.tile_slot[(xn >> 3) + trow];
      lc[i] = (xn & 7) | lrow;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (sl[i] < 0) continue;  // never: the first interpolation pass checked every stencil node
      const unsigned long long *gq = e.gcg + (size_t)sl[i] * 1536;
      const float h = 0.5f / e.macro[(size_t)sl[i] * 512 + lc[i]].x;
      const float d = r[i] * wyz;
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c] += (from_fix(gq[512 * c + lc[i]]) * h) * d;
    }
  }
  const float qx = group16_sum(v[0]), qy = group16_sum(v[1]), qz = group16_sum(v[2]);
  if (live && sub == 0) {
    float q[3] = {qx, qy, qz};
    if (e.slip) {  // n . (S p n)
      q[0] = bs.Nrm[k] * qx + bs.Nrm[n + k] * qy + bs.Nrm[2 * (size_t)n + k] * qz;
      q[1] = q[2] = 0.f;
    }
    const float *beta = cg_scal(e, 1, j);
    float p[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = cg_direction(e, k, c, j == 0 ? 0.f : beta[c], j == 0);
    float *qv = e.cg + 9 * (size_t)n, *pv = e.cg + 6 * (size_t)n;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      qv[c * n + k] = q[c];
      pv[c * n + k] = p[c];
      pq[c] = p[c] * q[c];
    }
  }
  if (sub == 0)
#pragma unroll
    for (int c = 0; c < 3; ++c) s_pq[mk][c] = pq[c];
  __syncthreads();
  if (tid < 3) {
    float t = 0.f;
    for (int q = 0; q < kInterpMk; ++q) t += s_pq[q][tid];
    cg_pq(e)[4 * (size_t)item + tid] = t;
  }
}

// Step j of conjugate gradients for markers item*kCgWG ... On the last step
// also the outputs: F = G / dV, the record's spread value G, and the markers'
// wrench shares.
__device__ inline void cg_update_item(const EnvView &e, const BodySet &bs, const FrameF &fr, int item, int j,
                                      bool last) {
#pragma clang fp contract(on)  // as interp_item
  const int n = e.n, k = item * kCgWG + (int)threadIdx.x;
  float pq[3], alpha[3];
  cg_sum3(cg_pq(e), interp_items(n), pq);  // every workgroup, in row order
  const float *rz = cg_scal(e, 0, j);
#pragma unroll
  for (int c = 0; c < 3; ++c) alpha[c] = pq[c] > 0.f ? rz[c] / pq[c] : 0.f;
  float rzn[3] = {0.f, 0.f, 0.f}, part[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (k < n) {
    float *G = e.cg, *r = e.cg + 3 * (size_t)n;
    const float *p = e.cg + 6 * (size_t)n, *q = e.cg + 9 * (size_t)n;
    const float p2 = 2.0f * e.mstate[k];
    float Gk[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float a = alpha[c];
      Gk[c] = G[c * n + k] + a * p[c * n + k];
      const float rk = r[c * n + k] - a * q[c * n + k];
      G[c * n + k] = Gk[c];
      r[c * n + k] = rk;
      rzn[c] = rk * (p2 * rk);
    }
    if (last) {
      if (e.slip) {  // the normal force gamma n
        const float gam = Gk[0];
        Gk[0] = gam * bs.Nrm[k];
        Gk[1] = gam * bs.Nrm[n + k];
        Gk[2] = gam * bs.Nrm[2 * (size_t)n + k];
      }
      const float idv = 1.0f / e.dv[k];
      float *rec = e.rec + (size_t)k * REC;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        e.F[c * n + k] = Gk[c] * idv;
        rec[16 + c] = Gk[c];
      }
      const float Uk[3] = {bs.U[k], bs.U[n + k], bs.U[2 * n + k]};
      const float rx = bs.X[k] - fr.org[0], ry = bs.X[n + k] - fr.org[1], rzz = bs.X[2 * n + k] - fr.org[2];
      part[0] = -Gk[0];
      part[1] = -Gk[1];
      part[2] = -Gk[2];
      part[3] = -(ry * Gk[2] - rzz * Gk[1]);
      part[4] = -(rzz * Gk[0] - rx * Gk[2]);
      part[5] = -(rx * Gk[1] - ry * Gk[0]);
      part[6] = Gk[0] * Uk[0] + Gk[1] * Uk[1] + Gk[2] * Uk[2];
    }
  }
  if (!last) {
    cg_part3(rzn, cg_rzp(e) + 4 * (size_t)item);
    if (cg_last_arrival(bs.counters + 1, cg_items(n))) {
      float t[3];
      cg_sum3(cg_rzp(e), cg_items(n), t);
      if (threadIdx.x < 3) {
        const float rz0 = cg_scal(e, 0, j)[threadIdx.x];
        cg_scal(e, 0, j + 1)[threadIdx.x] = t[threadIdx.x];
        cg_scal(e, 1, j + 1)[threadIdx.x] = rz0 != 0.f ? t[threadIdx.x] / rz0 : 0.f;
      }
    }
    return;
  }
  __shared__ float s_part[7][kCgWG + 1];  // the wrench rows, as interp_item
#pragma unroll
  for (int q = 0; q < 7; ++q) s_part[q][threadIdx.x] = part[q];
  __syncthreads();
  const int row = item * (kCgWG / kShareMk) + (int)(threadIdx.x >> 3), col = threadIdx.x & 7;
  if (threadIdx.x < 8 * (kCgWG / kShareMk) && row < share_rows(n))
    e.partials[8 * (size_t)row + col] =
        col < 7 ? share_sum([&](int q) { return s_part[col][(threadIdx.x >> 3) * kShareMk + q]; }) : 0.f;
}

template <bool ROT>
__global__ void __launch_bounds__(kCgWG) k_cg_init(EnvView e, FrameF fr) {
  cg_init_item<ROT>(e, e.b[0], fr, blockIdx.x);
}

// Spreading of step j's search direction into gcg.
__global__ void __launch_bounds__(BT) k_spread_cg(EnvView e, int j) {
  const int items = kSpreadParts<BT> * n_active_of(e, e.b[0]);
  const float *beta = cg_scal(e, 1, j);
  for (int item = blockIdx.x; item < items; item += gridDim.x)
    spread_item<BT, true>(e, e.b[0], item, threadIdx.x, e.gcg, false, beta, j == 0);
}

// Grid: exactly interp_items(n) workgroups (the last-arrival count).
__global__ void __launch_bounds__(WG) k_cg_apply(EnvView e, int j) {
  cg_apply_item(e, e.b[0], xcd_item(blockIdx.x, gridDim.x), threadIdx.x, j);
}

// Grid: exactly cg_items(n) workgroups.
__global__ void __launch_bounds__(kCgWG) k_cg_update(EnvView e, FrameF fr, int j, int last) {
  cg_update_item(e, e.b[0], fr, blockIdx.x, j, last != 0);
}

// Block reduction of 8 floats over the workgroup.
__device__ inline void block_sum8(float v[8], float *smem /* [16][8] + 8 */) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = wave_sum(v[q]);
  if (lane == 0)
    for (int q = 0; q < 8; ++q) smem[wv * 8 + q] = v[q];
  __syncthreads();
  if (threadIdx.x < 8) {
    float s = 0.f;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) s += smem[w * 8 + threadIdx.x];
    smem[128 + threadIdx.x] = s;
  }
  __syncthreads();
  for (int q = 0; q < 8; ++q) v[q] = smem[128 + q];
}

// Fluid force, torque about `center`, and power sum F.U dV, for the whole body
// (blockIdx.x == 0) or one bone's blend-weighted share (blockIdx.x == 1 + b).
__global__ void __launch_bounds__(1024) k_wrench(const float *__restrict__ X, const float *__restrict__ U,
                                                 const float *__restrict__ F, const float *__restrict__ dv,
                                                 const int *__restrict__ bone, const float *__restrict__ weight,
                                                 int n, float c0, float c1, float c2, float *__restrict__ out) {
  __shared__ float smem[16 * 8 + 8];
  const int b = (int)blockIdx.x - 1;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    float wk = 1.0f;
    if (b >= 0) wk = (bone[k] == b ? weight[k] : 0.f) + (bone[n + k] == b ? weight[n + k] : 0.f);
    const float s = wk * dv[k];
    const float fx = F[k] * s, fy = F[n + k] * s, fz = F[2 * n + k] * s;
    const float rx = X[k] - c0, ry = X[n + k] - c1, rz = X[2 * n + k] - c2;
    v[0] -= fx;
    v[1] -= fy;
    v[2] -= fz;
    v[3] -= ry * fz - rz * fy;
    v[4] -= rz * fx - rx * fz;
    v[5] -= rx * fy - ry * fx;
    v[6] += fx * U[k] + fy * U[n + k] + fz * U[2 * n + k];
  }
  block_sum8(v, smem);
  if (threadIdx.x < 8) out[blockIdx.x * 8 + threadIdx.x] = threadIdx.x < 7 ? v[threadIdx.x] : 0.f;
}

}  // namespace lbmib
