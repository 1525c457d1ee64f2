// Host build of the tile steps (csrc/lbm_axi_tile.h) for the CPU test
// tests/test_tile_steps_host.py: every tile runs as a block of k_tile does, one
// row of lanes at a time (the lanes of a row share a wave: all load before any
// stores), on a buffer between guard bytes; the same problem also runs in single
// steps on the planes in place.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <string>
#include <vector>

#include "../paper_1409_5929_amd/csrc/lbm_axi_desc.h"
#include "../paper_1409_5929_amd/csrc/lbm_axi_tile.h"

using namespace lbmaxi;

namespace {

const FieldOut NONE{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};

struct Lane {
  int j, wl;
  RowC R;
  float s[9], t[5], ph;
};
struct Wall {
  int j, k, code;
  RowC R;
  float s[9], t[5], ph;
};

// One row of lanes [jl, jh) of planes D (columns and wall lanes as of `real`).
template <typename S, bool ODD, int MODE, int ADDR, bool WL>
void step_row(const InstDev& real, const InstDev& D, int k, int jl, int jh, uint32_t seed) {
  std::vector<Lane> lanes;
  for (int j = jl; j < jh; ++j) {
    Lane L;
    if (!tile_lane<WL>(real, j, L.wl)) continue;
    L.j = j + L.wl;
    L.R = make_row(real, L.j);
    node_load<S, ODD, ADDR>(D, L.R, L.j, k, L.s, L.t, L.ph);
    lanes.push_back(L);
  }
  for (Lane& L : lanes)
    node_update_loaded<S, ODD, MODE, ADDR, WL>(D, L.R, L.j, k, 0, NONE, seed, L.s, L.t, L.ph, L.wl);
}

template <typename S, bool WL>
bool tile_block(const InstDev& D, const InstDev& O, const StepTile& T, int vw, int nsteps, long long t) {
  const size_t GUARD = 4096;
  const TileRegion g = tile_load_region(D, T, nsteps);
  if (!tile_inside(D, T, nsteps)) return false;
  if (g.jh - g.jl > vw) return false;
  const size_t bytes = tile_bytes<S>((size_t)vw * (g.kh - g.kl));
  std::vector<unsigned char> mem(bytes + 2 * GUARD, 0xFF);  // NaN wherever nothing was written
  unsigned char* lds = mem.data() + GUARD;
  const InstDev L = tile_desc<S>(D, T, g, vw, lds);
  for (int k = g.kl; k < g.kh; ++k)
    for (int j = g.jl; j < g.jh; ++j) {
      tile_in<S>(D, row_off(tile_row(D, T, k), D.stride) + j,
                 (uint32_t*)lds + ((k - g.kl) * vw + j - g.jl) * TileNode<S>::WORDS);
    }
  for (int i = 0; i < nsteps; ++i) {
    const TileRegion a = tile_region(D, T, nsteps - i);
    const int kb = z_bounded(D) && a.kl == 0 ? 1 : a.kl, ke = z_bounded(D) && a.kh == D.nz ? D.nz - 1 : a.kh;
    std::vector<Wall> walls;  // the boundary nodes load before the fluid nodes store
    const TileWalls w = tile_walls<WL>(D, g);
    for (int idx = 0; idx < w.count; ++idx) {
      Wall b;
      if (!tile_wall(D, g, w, idx, b.j, b.k, b.code) || !tile_wall_in(a, b.j, b.k, b.code)) continue;
      b.R = make_row(D, b.j);
      if (i & 1) node_load<S, true, ADDR_TILE>(L, b.R, b.j, b.k, b.s, b.t, b.ph);
      else node_load<S, false, ADDR_TILE>(L, b.R, b.j, b.k, b.s, b.t, b.ph);
      walls.push_back(b);
    }
    for (int k = kb; k < ke; ++k) {
      if (i & 1) step_row<S, true, MODE_TILE, ADDR_TILE, WL>(D, L, k, a.jl, a.jh, step_seed(t + i));
      else step_row<S, false, MODE_TILE, ADDR_TILE, WL>(D, L, k, a.jl, a.jh, step_seed(t + i));
    }
    for (Wall& b : walls) {
      const uint32_t seed = step_seed(t + i);
      if (i & 1)
        node_update_loaded<S, true, MODE_WALL, ADDR_TILE, WL>(L, b.R, b.j, b.k, b.code, NONE, seed, b.s, b.t, b.ph, 0);
      else
        node_update_loaded<S, false, MODE_WALL, ADDR_TILE, WL>(L, b.R, b.j, b.k, b.code, NONE, seed, b.s, b.t, b.ph, 0);
    }
  }
  for (int k = g.kl; k < g.kh; ++k) {
    const int kt = tile_unwrapped(D, T) ? k - D.nz : k;
    if (kt < T.k0 || kt >= T.k1) continue;
    for (int j = T.j0; j < T.j1; ++j)
      tile_out<S>((uint32_t*)lds + ((k - g.kl) * vw + j - g.jl) * TileNode<S>::WORDS, D, O.pop, O.g0,
                  row_off(tile_row(D, T, k), D.stride) + j);
  }
  for (size_t b = 0; b < GUARD; ++b)
    if (mem[b] != 0xFF || mem[GUARD + bytes + b] != 0xFF) return false;
  return true;
}

template <typename S, bool WL>
int run(const lbm_axi_params* p, const float* phi_field, const float* init, int nsteps, int m, int vw, int h,
        float* tiled, float* single) {
  InstDev D;
  std::string err;
  if (describe(*p, phi_field != nullptr, D, err)) return -1;
  std::vector<float> phi;
  if (phi_field) {
    phi.assign(D.plane, (float)p->phi);
    for (int k = 0; k < p->nz; ++k) memcpy(&phi[(size_t)k * D.stride], phi_field + (size_t)k * p->nr, 4 * p->nr);
    D.phi = phi.data();
  }
  const size_t bytes = (size_t)D.plane * 14 * sizeof(S);
  std::vector<unsigned char> pop[3];
  std::vector<float> g0[3];
  InstDev I[3];  // tiled: two sets of planes; single steps
  for (int q = 0; q < 3; ++q) {
    pop[q].assign(bytes, 0xFF);
    g0[q].assign(D.plane, NAN);
    I[q] = D;
    I[q].pop = pop[q].data();
    I[q].g0 = sizeof(S) == 4 ? (float*)pop[q].data() + 9 * D.plane : g0[q].data();
  }
  const size_t n = (size_t)D.nr * D.nz;
  for (int q : {0, 2})
    for (int k = 0; k < D.nz; ++k)
      for (int j = 0; j < D.nr; ++j) {
        const size_t o = (size_t)k * D.nr + j;
        init_node<S>(I[q], j, k, init[o], init[n + o], init[2 * n + o]);
      }
  std::vector<int> cj, ck;
  m = std::min(m, tile_max_steps(D));
  tile_cuts(D, vw, m, h, cj, ck);
  int cur = 0;
  for (int t = 0; t < nsteps;) {
    const int s = std::min(m, nsteps - t);
    for (size_t a = 0; a + 1 < ck.size(); ++a)
      for (size_t b = 0; b + 1 < cj.size(); ++b)
        if (!tile_block<S, WL>(I[cur], I[cur ^ 1], StepTile{0, cj[b], cj[b + 1], ck[a], ck[a + 1], 0, 0, 0}, vw, s, t))
          return -2;
    cur ^= 1;
    t += s;
  }
  for (int t = 0; t < nsteps; ++t)
    for (int k = z_bounded(D) ? 1 : 0; k < (z_bounded(D) ? D.nz - 1 : D.nz); ++k) {
      if (t & 1) step_row<S, true, MODE_STEP, ADDR_FLAT, WL>(D, I[2], k, 0, D.nr, step_seed(t));
      else step_row<S, false, MODE_STEP, ADDR_FLAT, WL>(D, I[2], k, 0, D.nr, step_seed(t));
    }
  for (int q : {cur, 2}) {
    float* f = q == 2 ? single : tiled;
    const FieldOut fo{f, f + n, nullptr, f + 2 * n, nullptr, f + 3 * n};
    for (int j = 0; j < D.nr; ++j) {
      if ((D.side_rmin == SIDE_WALL && j == 0) || (D.side_rmax == SIDE_WALL && j == D.nr - 1)) continue;
      const RowC R = make_row(D, j);
      for (int k = z_bounded(D) ? 1 : 0; k < (z_bounded(D) ? D.nz - 1 : D.nz); ++k)
        node_update<S, false, MODE_FIELDS>(I[q], R, j, k, 0, fo, 0u);
    }
  }
  return 0;
}

}  // namespace

// nsteps (even) steps from start fields init in launches of at most m (even) steps on
// tiles of vw columns and about h rows, and in single steps; u_z, u_r, T and rho - 1
// of both ([4][nz][nr]).  0, -1 for a bad problem, -2 when a tile is wider than vw or
// wrote outside its buffer.
extern "C" int host_tile_steps(const lbm_axi_params* p, const float* phi_field, const float* init, int nsteps, int m,
                               int vw, int h, int wall_lanes, float* tiled, float* single) {
  if (p->storage == LBM_STORE_FP32)
    return wall_lanes ? run<float, true>(p, phi_field, init, nsteps, m, vw, h, tiled, single)
                      : run<float, false>(p, phi_field, init, nsteps, m, vw, h, tiled, single);
  return wall_lanes ? run<__half, true>(p, phi_field, init, nsteps, m, vw, h, tiled, single)
                    : run<__half, false>(p, phi_field, init, nsteps, m, vw, h, tiled, single);
}

// Whether every tile of about h rows may take m steps (tile_inside), and the most steps.
extern "C" int host_tile_inside(const lbm_axi_params* p, int m, int vw, int h, int* most) {
  InstDev D;
  std::string err;
  if (describe(*p, false, D, err)) return -1;
  *most = tile_max_steps(D);
  std::vector<int> cj, ck;
  tile_cuts(D, vw, m, h, cj, ck);
  for (size_t a = 0; a + 1 < ck.size(); ++a)
    for (size_t b = 0; b + 1 < cj.size(); ++b)
      if (!tile_inside(D, StepTile{0, cj[b], cj[b + 1], ck[a], ck[a + 1], 0, 0, 0}, m)) return 0;
  return 1;
}
