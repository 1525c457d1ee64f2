// Several time steps per launch on tiles kept in LDS.
//
// A grid that fits the caches is bound by latency, not bandwidth, when each
// step is a launch of its own: the launch itself, the dependent loads of the
// tile, the descriptor and the populations, and the drained stores come to
// about 5 us a step, however few nodes there are.  Here one block takes a tile
// of the grid through an even number m of steps: it copies the tile's
// populations, with a halo of m nodes, from the planes into LDS (same slots,
// same storage type, all of a node in consecutive words: with a plane for each
// slot, as in HBM, every access formed its own address, 35 of a node's 360 vector
// instructions), runs the step's own node code on the LDS copy in place
// (the AA pattern needs one barrier per step), on a region that shrinks by one
// node per step towards the tile, and copies the tile's slots to a second set
// of planes.  Tiles overlap only where they read, so blocks never wait for
// each other; the planes of the two sets alternate from launch to launch.
// Every node sees the same operations in the same order as in single steps.
#pragma once

#include <vector>

#include "lbm_axi_dev.h"

namespace lbmaxi {

// The tile's nodes [j0, j1) x [k0, k1) of instance inst (inst < 0: none).
struct StepTile {
  int inst, j0, j1, k0, k1, pad0, pad1, pad2;
};

// Columns [jl, jh) and rows [kl, kh) of a tile widened by m nodes within the
// grid.  A tile that does not span a z-periodic grid takes its rows unwrapped,
// shifted up by nz so that none is negative.
struct TileRegion {
  int jl, jh, kl, kh;
};

__host__ __device__ inline bool tile_unwrapped(const InstDev& D, const StepTile& T) {
  return D.side_z == SIDE_PERIODIC && T.k1 - T.k0 < D.nz;
}

__host__ __device__ inline TileRegion tile_region(const InstDev& D, const StepTile& T, int m) {
  TileRegion g;
  g.jl = T.j0 - m > 0 ? T.j0 - m : 0;
  g.jh = T.j1 + m < D.nr ? T.j1 + m : D.nr;
  if (tile_unwrapped(D, T)) {
    g.kl = T.k0 + D.nz - m;
    g.kh = T.k1 + D.nz + m;
  } else {
    g.kl = T.k0 - m > 0 ? T.k0 - m : 0;
    g.kh = T.k1 + m < D.nz ? T.k1 + m : D.nz;
  }
  return g;
}

// The region held in LDS for m steps: an axial boundary row beside its
// outermost fluid row comes along, since the fluid row's nodes write it.
__host__ __device__ inline TileRegion tile_load_region(const InstDev& D, const StepTile& T, int m) {
  TileRegion g = tile_region(D, T, m);
  if (z_bounded(D)) {
    if (g.kl == 1) g.kl = 0;
    if (g.kh == D.nz - 1) g.kh = D.nz;
  }
  return g;
}

// The most steps per launch that an instance takes: an unwrapped region reaches m
// rows beyond its tile, and no row may be more than one period away (tile_row).
inline int tile_max_steps(const InstDev& D) { return D.side_z == SIDE_PERIODIC ? D.nz & ~1 : 1 << 20; }

// Whether a tile's regions for up to m steps lie in the rows and columns that stand for
// the instance's nodes (what k_tile reads then lies in the instance's planes), and none
// ends beside a radial wall column that it leaves out: the boundary nodes next to that
// column count it as a wall (whom they send to, and with which random bits), so a region
// holds the wall or stays clear of its owners.
inline bool tile_inside(const InstDev& D, const StepTile& T, int m) {
  if (D.side_rmin == SIDE_WALL && T.j0 > 0 && T.j0 <= m + 1) return false;
  if (D.side_rmax == SIDE_WALL && T.j1 < D.nr && T.j1 + m >= D.nr - 1) return false;
  const TileRegion g = tile_load_region(D, T, m);
  return g.jl >= 0 && g.jh <= D.nr && g.kl >= 0 && g.kh <= (tile_unwrapped(D, T) ? 3 * D.nz : D.nz) && T.j0 >= g.jl &&
         T.j1 <= g.jh;
}

// Cuts of an instance into tiles for m steps, so that a tile's region is at most vw
// columns wide: columns cj[i] .. cj[i + 1], rows ck[i] .. ck[i + 1] of about h.
// Tiles at either radial side need no halo there and are wider by m.
inline void tile_cuts(const InstDev& D, int vw, int m, int h, std::vector<int>& cj, std::vector<int>& ck) {
  int n = 1, cap = vw;
  while (cap < D.nr) {
    ++n;
    cap = 2 * (vw - m) + (n - 2) * (vw - 2 * m);
  }
  cj.assign(1, 0);
  for (int i = 1; i < n; ++i) cj.push_back((int)((int64_t)D.nr * (vw - m + (i - 1) * (vw - 2 * m)) / cap));
  cj.push_back(D.nr);
  const int nk = (D.nz + h - 1) / h;
  ck.clear();
  for (int i = 0; i <= nk; ++i) ck.push_back((int)((int64_t)D.nz * i / nk));
}

// LDS bytes of n nodes.
template <typename S>
__host__ __device__ inline size_t tile_bytes(size_t n) {
  return n * (4 * TileNode<S>::WORDS);
}

// Descriptor of region g held at lds in rows of vw nodes: the instance's, with
// its planes in LDS.
template <typename S>
__host__ __device__ inline InstDev tile_desc(const InstDev& D, const StepTile& T, const TileRegion& g, int vw,
                                             unsigned char* lds) {
  InstDev L = D;
  const int n = vw * (g.kh - g.kl);
  L.plane = n;
  L.stride = vw;
  L.t_base = g.kl * vw + g.jl;
  L.t_stride = D.stride;
  L.pop = lds;
  L.g0 = (float*)lds + TileNode<S>::G0;
  L.phi = (const float*)lds + TileNode<S>::PHI;
  if (tile_unwrapped(D, T)) {
    L.side_z = SIDE_UNWRAPPED;
    L.nz = 4 * D.nz;
  }
  return L;
}

// Row of the instance that row k of a region stands for.
__host__ __device__ inline int tile_row(const InstDev& D, const StepTile& T, int k) {
  if (!tile_unwrapped(D, T)) return k;
  return k >= 2 * D.nz ? k - 2 * D.nz : (k >= D.nz ? k - D.nz : k);
}

// Column a lane works on and its wall-lane flag, as in k_step: wall lanes take
// their owner's column (they share its wave: a row of the tile is at most one
// wave wide); without wall lanes, and where the owner keeps the wall, a
// radial wall column idles (false).
template <bool WL>
__host__ __device__ inline bool tile_lane(const InstDev& D, int j, int& wl) {
  wl = (D.side_rmin == SIDE_WALL && j == 0) ? 1 : (D.side_rmax == SIDE_WALL && j == D.nr - 1) ? -1 : 0;
  if (wl == 0) return true;
  return WL && (wl > 0 || wall_lane_rmax(D));
}

// The slots and porosity of the node at offset o of an instance's planes to
// its words in LDS (TileNode), and the slots back.
template <typename S>
__host__ __device__ inline void tile_in(const InstDev& D, int64_t o, uint32_t* n) {
  using N = TileNode<S>;
  if constexpr (sizeof(S) == 4) {
    float v[14];
#pragma unroll
    for (int q = 0; q < 14; ++q) v[q] = ((const float*)D.pop)[q * D.plane + o];
#pragma unroll
    for (int q = 0; q < 14; ++q) ((float*)n)[q] = v[q];
  } else {
    uint16_t v[5];
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 5; ++q) v[q] = ((const uint16_t*)D.pop)[q * D.plane + o];
#pragma unroll
    for (int a = 0; a < 4; ++a) w[a] = ((const uint32_t*)D.pop)[(5 + 2 * a) * (D.plane >> 1) + o];
    const float g = D.g0[o];
#pragma unroll
    for (int q = 0; q < 5; ++q) ((uint16_t*)n)[q] = v[q];
#pragma unroll
    for (int a = 0; a < 4; ++a) n[N::PAIR + a] = w[a];
    ((float*)n)[N::G0] = g;
  }
  if (D.phi_mode) ((float*)n)[N::PHI] = D.phi[o];
}
template <typename S>
__host__ __device__ inline void tile_out(const uint32_t* n, const InstDev& D, void* pop, float* g0, int64_t o) {
  using N = TileNode<S>;
  if constexpr (sizeof(S) == 4) {
#pragma unroll
    for (int q = 0; q < 14; ++q) ((float*)pop)[q * D.plane + o] = ((const float*)n)[q];
  } else {
#pragma unroll
    for (int q = 0; q < 5; ++q) ((uint16_t*)pop)[q * D.plane + o] = ((const uint16_t*)n)[q];
#pragma unroll
    for (int a = 0; a < 4; ++a) ((uint32_t*)pop)[(5 + 2 * a) * (D.plane >> 1) + o] = n[N::PAIR + a];
    g0[o] = ((const float*)n)[N::G0];
  }
}

// Boundary nodes of a region that no fluid lane takes: the axial boundary rows
// with their corners, and the radial walls that their owners keep (wall_node).
// They run on waves of their own beside the fluid waves: on the owner's lane they
// come after its update, three of them one by one at a corner, and the whole
// tile waits at the step's barrier.  Each kind (dr, dz) has its own code, so
// the kinds start at multiples of 32 threads: the axial rows first, then the
// corners, then the radial walls.
struct TileWalls {
  bool lo, hi, zlo, zhi;  // radial walls kept by their owners; axial rows
  int cols, rows, corner, radial, count;  // first threads of the corners and radial walls, threads
};
template <bool WL>
__host__ __device__ inline TileWalls tile_walls(const InstDev& D, const TileRegion& g) {
  TileWalls w;
  w.lo = D.side_rmin == SIDE_WALL && g.jl == 0 && !WL;
  w.hi = D.side_rmax == SIDE_WALL && g.jh == D.nr && !(WL && wall_lane_rmax(D));
  w.zlo = z_bounded(D) && g.kl == 0;
  w.zhi = z_bounded(D) && g.kh == D.nz;
  w.cols = (g.jh - g.jl + 31) / 32 * 32;
  w.rows = (g.kh - g.kl + 31) / 32 * 32;
  const bool rm = D.side_rmin == SIDE_WALL && g.jl == 0, rp = D.side_rmax == SIDE_WALL && g.jh == D.nr;
  w.corner = w.cols * (w.zlo + w.zhi);
  w.radial = w.corner + ((w.zlo || w.zhi) && (rm || rp) ? 32 : 0);
  w.count = w.radial + w.rows * (w.lo + w.hi);
  return w;
}
// Threads that a block sets aside for them: whole waves.
__host__ __device__ inline int tile_wall_threads(const TileWalls& w) { return (w.count + 63) / 64 * 64; }
// Boundary node of thread idx: its owner (j, k) and code 3 (dr + 1) + dz + 1; false: none.
__host__ __device__ inline bool tile_wall(const InstDev& D, const TileRegion& g, const TileWalls& w, int idx, int& j,
                                          int& k, int& code) {
  int dr = 0, dz = 0;
  if (idx < w.corner) {
    const int row = idx / w.cols, jb = g.jl + idx - row * w.cols;
    const bool radial = (D.side_rmin == SIDE_WALL && jb == 0) || (D.side_rmax == SIDE_WALL && jb == D.nr - 1);
    dz = jb >= g.jh || radial ? 0 : (w.zlo && row == 0 ? -1 : 1);
    j = jb;
    k = dz < 0 ? 1 : D.nz - 2;
  } else if (idx < w.radial) {
    const int q = idx - w.corner;  // corners: (r_min, r_max) x (z_min, z_max)
    dr = q & 1 ? 1 : -1;
    dz = q & 2 ? 1 : -1;
    const bool there = q < 4 && (dr < 0 ? D.side_rmin == SIDE_WALL && g.jl == 0 : D.side_rmax == SIDE_WALL && g.jh == D.nr) &&
                       (dz < 0 ? w.zlo : w.zhi);
    if (!there) dr = dz = 0;
    j = dr < 0 ? 1 : D.nr - 2;
    k = dz < 0 ? 1 : D.nz - 2;
  } else if (idx < w.count) {
    const int side = (idx - w.radial) / w.rows;
    k = g.kl + idx - w.radial - side * w.rows;
    dr = side == 0 && w.lo ? -1 : 1;
    j = dr < 0 ? 1 : D.nr - 2;
    if (k >= g.kh || (z_bounded(D) && (k == 0 || k == D.nz - 1))) dr = 0;
  }
  code = 3 * (dr + 1) + dz + 1;
  return dr != 0 || dz != 0;
}
// Whether that boundary node is in the region a of a step (with its owner's row).
__host__ __device__ inline bool tile_wall_in(const TileRegion& a, int j, int k, int code) {
  const int jb = j + code / 3 - 1;
  return jb >= a.jl && jb < a.jh && k >= a.kl && k < a.kh;
}

// n (even) steps from level t in launches of at most m, each an even number: launch(i,
// steps, level) is the i-th and returns 0 or an error, which ends the run.  The planes alternate,
// so the launches come in pairs and t moves with each pair: whatever fails, the
// handle's own planes hold the state of level t.
template <typename Launch>
int tile_pairs(long long& t, int n, int m, Launch&& launch) {
  const int pairs = (n + 2 * m - 1) / (2 * m);
  int done = 0;
  for (int i = 0; i < 2 * pairs; i += 2) {
    const int mid = 2 * (int)((int64_t)(n / 2) * (i + 1) / (2 * pairs));
    const int end = 2 * (int)((int64_t)(n / 2) * (i + 2) / (2 * pairs));
    if (const int rc = launch(i, mid - done, t)) return rc;
    if (const int rc = launch(i + 1, end - mid, t + (mid - done))) return rc;
    t += end - done;
    done = end;
  }
  return 0;
}

constexpr int TILE_NT = 512;  // threads of a tile block
constexpr int TILE_VWLOG = 5, TILE_VW = 1 << TILE_VWLOG;  // columns of a tile with its halo

// nsteps (even) steps from time level t of every tile's instance, planes of src to
// planes of dst.  The last waves of a block take one boundary node each (tile_wall),
// the nf threads before them the fluid nodes and, with WL (as the handle's single
// steps have it), the radial wall lanes.
template <typename S, bool WL>
__global__ __launch_bounds__(TILE_NT) __attribute__((amdgpu_waves_per_eu(4))) void k_tile(const InstDev* __restrict__ src, const InstDev* __restrict__ dst,
                                                  const StepTile* __restrict__ tiles,
                                                  const int* __restrict__ status, int vwlog, int nsteps,
                                                  long long t) {
  extern __shared__ __attribute__((aligned(16))) unsigned char tile_lds[];
  const StepTile T = tiles[blockIdx.x];
  if (T.inst < 0 || status[T.inst] != RUN) return;
  const InstDev D = src[T.inst];
  // vwlog = TILE_VWLOG as an argument: with the constant the compiler hoists ten
  // more registers out of the step loop (FP32, 64 of 128^2: 18.6 and 18.2 us)
  const int vw = 1 << vwlog, c = (int)threadIdx.x & (vw - 1), rg = (int)threadIdx.x >> vwlog;
  const TileRegion g = tile_load_region(D, T, nsteps);
  const int RB = (int)blockDim.x >> vwlog;
  const InstDev L = tile_desc<S>(D, T, g, vw, tile_lds);
  uint32_t* lds = (uint32_t*)tile_lds;
  int j = g.jl + c;
  if (j < g.jh)
    for (int k = g.kl + rg; k < g.kh; k += RB) {
      tile_in<S>(D, row_off(tile_row(D, T, k), D.stride) + j, lds + mul24(((k - g.kl) << vwlog) + c, TileNode<S>::WORDS));
    }
  const FieldOut fo{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  const TileWalls w = tile_walls<WL>(D, g);
  const int nf = (int)blockDim.x - tile_wall_threads(w), RG = nf >> vwlog;
  const bool walls = w.count > 0;  // the same for the whole block
  if ((int)threadIdx.x < nf) {
    int wl;
    const bool lane = tile_lane<WL>(D, j, wl) && j < g.jh;
    const RowC R = make_row(D, j + wl);
    for (int i = 0; i < nsteps; ++i) {
      __syncthreads();
      if (walls) __syncthreads();  // the boundary nodes' owners are loaded
      const TileRegion a = tile_region(D, T, nsteps - i);
      const uint32_t seed = step_seed(t + i);
      const int kb = z_bounded(D) && a.kl == 0 ? 1 : a.kl, ke = z_bounded(D) && a.kh == D.nz ? D.nz - 1 : a.kh;
      const bool in = lane && j >= a.jl && j < a.jh;
      if (i & 1) {
        for (int k = g.kl + rg; k < ke; k += RG)
          if (in && k >= kb) node_update<S, true, MODE_TILE, ADDR_TILE, WL>(L, R, j + wl, k, 0, fo, seed, wl);
      } else {
        for (int k = g.kl + rg; k < ke; k += RG)
          if (in && k >= kb) node_update<S, false, MODE_TILE, ADDR_TILE, WL>(L, R, j + wl, k, 0, fo, seed, wl);
      }
    }
  } else {
    int jo = 0, ko = 0, code = 0;
    const bool wall = tile_wall(D, g, w, (int)threadIdx.x - nf, jo, ko, code);
    const RowC R = make_row(D, jo);
    for (int i = 0; i < nsteps; ++i) {
      __syncthreads();
      const TileRegion a = tile_region(D, T, nsteps - i);
      const uint32_t seed = step_seed(t + i);
      const bool in = wall && tile_wall_in(a, jo, ko, code);
      float s[9], tt[5], ph = 0.0f;
      if (in) {
        if (i & 1) node_load<S, true, ADDR_TILE>(L, R, jo, ko, s, tt, ph);
        else node_load<S, false, ADDR_TILE>(L, R, jo, ko, s, tt, ph);
      }
      if (walls) __syncthreads();
      if (in) {
        if (i & 1) node_update_loaded<S, true, MODE_WALL, ADDR_TILE, WL>(L, R, jo, ko, code, fo, seed, s, tt, ph, 0);
        else node_update_loaded<S, false, MODE_WALL, ADDR_TILE, WL>(L, R, jo, ko, code, fo, seed, s, tt, ph, 0);
      }
    }
  }
  __syncthreads();
  const InstDev* O = dst + T.inst;
  if (j >= T.j0 && j < T.j1)
    for (int k = g.kl + rg; k < g.kh; k += RB) {
      const int kt = tile_unwrapped(D, T) ? k - D.nz : k;
      if (kt < T.k0 || kt >= T.k1) continue;
      tile_out<S>(lds + mul24(((k - g.kl) << vwlog) + c, TileNode<S>::WORDS), D, O->pop, O->g0,
                  row_off(tile_row(D, T, k), D.stride) + j);
    }
}

}  // namespace lbmaxi
