// Two liquid steps per launch (step2_cell.hpp) of a single lattice, alone or coupled to bubbles.
//
// With bubbles, a pair of method steps is
//   bubble half n; k_slab: step n of the planes the bubbles reach, into the middle buffer;
//   bubble half n + 1; k_step2: both steps of every other plane, and step n + 1 of those planes.
// The planes the bubbles reach in the pair are the slab [a, b): every force window of step n with a
// plane to spare on either side, and the velocity windows the second half reads (which hold its
// force windows). The bubble update finds a and b on the device as it moves each bubble. Outside the
// slab no cell holds force in either step, nor is its velocity read.
#include <algorithm>
#include <utility>

#include "step2_cell.hpp"

namespace lbm {
namespace {

// Compute units of the chip: the workgroups of this pass that run at a time.
constexpr uint32_t kStep2Cus = 256;

// The slab [a, b) from its words; empty without bubbles.
__device__ __forceinline__ void slab_range(const uint32_t* words, int nz, int& a, int& b) {
  a = b = 0;
  if (words && words[1] != 0u) {
    a = max(0, (int)(kSlabBase - words[0]));
    b = min(nz, (int)words[1]);
  }
}

// One step of one cell by flat index, inside a loop over cells. The strides are made opaque in every
// iteration: hoisted out of the loop, the 38 offsets that follow from them fill the registers.
template <typename T, bool FS>
__device__ __forceinline__ void step_one(const gchar* src, gchar* dst, gchar* F, gchar* U,
                                         const gchar* tiles, const Geom& G0, T omega, int flags,
                                         uint32_t cell, uint32_t fs) {
  Geom G = G0;
  asm volatile("" : "+s"(G.qs), "+s"(G.zs), "+s"(G.nx));
  const uint32_t z = cell / G.plane, rem = cell - z * G.plane;
  const uint32_t y = rem / (uint32_t)G.nx, x = rem - y * (uint32_t)G.nx;
  const uint32_t tile = ((z >> 3) * G.tny + (y >> 3)) * G.tnx + (x >> 3);
  step_cell_bb<T, FS>(src, dst, F, U, tiles, tile, G, omega, flags, (int)x, (int)y, z, fs);
}

template <typename T>
struct Step2Args {
  const T* src;
  const T* mid;  // step n + 1 of the slab (and a plane beside it), or null
  T* dst;
  T* F;
  T* U;
  const uint8_t* tiles;  // mask of the second step
  uint8_t* tiles_next;   // cleared
  const uint32_t* slab;  // slab words of the pair, or null
  Geom G;
  T omega;
  Tiles2 L;
  uint32_t ntiles;
  int flags;
  int dirty;  // no slab: some tile of the mask may be set
};

// A workgroup per (tile, chunk of the planes outside the slab); each then takes its share of the
// slab's cells, so the launch stays balanced whatever the slab holds.
template <typename T, int FACES, bool FORCE>
__global__ __launch_bounds__(step2_threads<T>()) void k_step2(Step2Args<T> A) {
  constexpr int NT = step2_threads<T>();
  __shared__ Plane2<T, NT> s[2];
  const Geom& G = A.G;
  const uint32_t nblocks = gridDim.x;
  const uint32_t b = xcd_remap(blockIdx.x, nblocks);
  const uint32_t txi = b % A.L.ntx, r = b / A.L.ntx;
  const uint32_t tyi = r % A.L.nty, ch = r / A.L.nty;
  int sa, sb;
  slab_range(A.slab, G.nz, sa, sb);
  Lattice2 D;
  D.src = gbytes<T>(A.src);
  D.dst = gbytes<T>(A.dst);
  D.F = gbytes<T>(A.F);
  D.U = gbytes<T>(A.U);
  D.tiles = gbytes<uint8_t>(A.tiles);
  D.u_all = A.flags & LBM_FLAG_WRITE_U_ALL;
  if (A.slab) {
    slab_range(A.slab + 2, G.nz, D.fa, D.fb);  // planes of the second half's windows: whole tiles
    D.fa &= ~(int)(kTile - 1);
    D.fb = (D.fb + (int)kTile - 1) & ~(int)(kTile - 1);
  } else {
    D.fa = 0;
    D.fb = A.dirty ? G.nz : 0;
  }
  // chunk of the planes outside the slab, counted without it
  const uint32_t nzb = (uint32_t)(G.nz - (sb - sa));
  const int c0 = (int)(ch * nzb / A.L.nchunk), c1 = (int)((ch + 1) * nzb / A.L.nchunk);
  if (c0 < min(c1, sa)) march2<T, FACES, FORCE, NT>(s, G, D, A.omega, A.L, txi, tyi, c0, min(c1, sa));
  if (max(c0, sa) < c1)
    march2<T, FACES, FORCE, NT>(s, G, D, A.omega, A.L, txi, tyi, max(c0, sa) + (sb - sa), c1 + (sb - sa));
  if constexpr (FACES != FACES_GENERAL && !FORCE) {
    const uint32_t cells = (uint32_t)(sb - sa) * G.plane, first = (uint32_t)sa * G.plane;
    const uint32_t fs = FACES == FACES_WALLS ? free_slip_faces(G) : 0u;
#pragma unroll 1
    for (uint32_t k = blockIdx.x * NT + threadIdx.x; k < cells; k += nblocks * NT) {
      step_one<T, FACES == FACES_WALLS>(gbytes<T>(A.mid), D.dst, gbytes<T>(A.F), D.U, D.tiles, G, A.omega,
                                        A.flags, first + k, fs);
    }
  }
  for (uint32_t k = blockIdx.x * NT + threadIdx.x; k < A.ntiles; k += nblocks * NT) A.tiles_next[k] = 0;
}

// Step n of the slab's planes and one beside it on either side, from the current state into the
// middle buffer, with the force of the first bubble half. The planes are widened to whole tiles, so
// that the velocity is written in every tile that half flagged.
template <typename T, bool FS>
__global__ __launch_bounds__(256) void k_slab(const T* __restrict__ src, T* __restrict__ mid,
                                              T* __restrict__ F, T* __restrict__ U,
                                              const uint8_t* __restrict__ tiles,
                                              uint8_t* __restrict__ tiles_next,
                                              const uint32_t* __restrict__ slab, Geom G, T omega,
                                              int flags, uint32_t ntiles) {
  int a, b;
  slab_range(slab, G.nz, a, b);
  if (a < b) {
    a = max(0, min(a - 1, a & ~(int)(kTile - 1)));
    b = min(G.nz, max(b + 1, (b + (int)kTile - 1) & ~(int)(kTile - 1)));
  }
  const uint32_t cells = (uint32_t)(b - a) * G.plane, first = (uint32_t)a * G.plane;
  const uint32_t fs = FS ? free_slip_faces(G) : 0u;
#pragma unroll 1
  for (uint32_t k = blockIdx.x * 256 + threadIdx.x; k < cells; k += gridDim.x * 256) {
    step_one<T, FS>(gbytes<T>(src), gbytes<T>(mid), gbytes<T>(F), gbytes<T>(U), gbytes<uint8_t>(tiles), G,
                    omega, flags, first + k, fs);
  }
  for (uint32_t k = blockIdx.x * 256 + threadIdx.x; k < ntiles; k += gridDim.x * 256) tiles_next[k] = 0;
}

// Threads a tile of ox by oy output cells takes at most.
uint32_t tile_threads(const Geom& G, uint32_t ox, uint32_t oy) {
  const bool perx = G.bc[0] == BC_PER, pery = G.bc[2] == BC_PER;
  const uint32_t nx = (uint32_t)G.nx, ny = (uint32_t)G.ny;
  const uint32_t ntx = div_up(nx, ox), nty = div_up(ny, oy);
  const uint32_t hx = perx ? 2 : ntx == 1 ? 0 : ntx == 2 ? 1 : 2, hy = pery ? 2 : nty == 1 ? 0 : nty == 2 ? 1 : 2;
  return (ox + hx) * (oy + hy);
}

}  // namespace

// Tiles and chunks of a lattice for the two-step pass. A compute unit holds one workgroup, so a
// launch takes time in proportion to the planes a workgroup marches, two of them beside its chunk,
// times its rows, two of them beside its tile (most of a halo row's loads hit the L2, so this
// counts it too high; measured within 5 % of the best of a sweep on eleven lattices from 30 x 30 x
// 90 to 256 x 256 x 256). Pieces of rows cost a quarter more than whole ones, whose loads and stores
// are contiguous over the tile: 128 x 128 x 512 FP32 122 us per step in whole rows of 6, 132 us in
// tiles of 64 x 13; 256 x 256 x 256 253 us in whole rows of 2 (every intermediate row computed
// twice), 284 us in tiles of 64 x 13, 264 us in tiles of 128 x 5.
bool choose_tiles2(const Geom& G, size_t elem, Tiles2* best) {
  const uint32_t threads = elem == 4 ? step2_threads<float>() : step2_threads<double>();
  const uint32_t align = 128u / (uint32_t)elem;  // cells of a cache line
  const uint32_t nx = (uint32_t)G.nx, ny = (uint32_t)G.ny, nz = (uint32_t)G.nz;
  double cost = 1e30;
  for (uint32_t ox = nx; ox >= 1; ox = ox == nx ? (nx - 1) / align * align : ox - align) {
    for (uint32_t oy = 1; oy <= ny && oy <= threads && tile_threads(G, ox, oy) <= threads; ++oy) {
      const uint32_t ntx = div_up(nx, ox), nty = div_up(ny, oy), nt = ntx * nty;
      const uint32_t nc = std::max(1u, std::min(nz, kStep2Cus / nt));
      const double v = (double)div_up(nt * nc, kStep2Cus) * ((double)nz / nc + 2.0) * ox * (oy + 2.0) *
                       (ox == nx ? 1.0 : 1.25);
      if (v < cost) {
        cost = v;
        *best = {ox, oy, ntx, nty, nc};
      }
    }
    if (ox < align) break;
  }
  return cost < 1e30;
}

namespace {

template <typename T, int FACES, bool FORCE>
hipError_t launch_typed(lbm_ctx* c, const uint32_t* slab) {
  const Geom& G = c->geom;
  Step2Args<T> A;
  A.src = static_cast<const T*>(c->pops[c->hs.cur]);
  A.mid = static_cast<const T*>(c->mid);
  A.dst = static_cast<T*>(c->pops[c->hs.cur ^ 1]);
  A.F = static_cast<T*>(c->force);
  A.U = static_cast<T*>(c->vel);
  A.tiles = c->tiles[c->hs.flag_cur];
  A.tiles_next = c->tiles[c->hs.flag_cur ^ 1];
  A.slab = slab;
  A.G = G;
  A.omega = (T)c->desc.omega;
  A.flags = c->desc.flags;
  A.ntiles = c->ntiles;
  A.dirty = c->hs.flag_clean[c->hs.flag_cur] ? 0 : 1;
  A.L = c->tiles2;
  const uint32_t n = A.L.ntx * A.L.nty * A.L.nchunk;
  hipLaunchKernelGGL((k_step2<T, FACES, FORCE>), dim3(n), dim3(step2_threads<T>()), 0, c->stream, A);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_faces(lbm_ctx* c, const uint32_t* slab) {
  const bool force = c->desc.flags & LBM_FLAG_STATIC_FORCE;
  if (c->periodic)
    return force ? launch_typed<T, FACES_GENERAL, true>(c, slab) : launch_typed<T, FACES_GENERAL, false>(c, slab);
  if (c->general)
    return force ? launch_typed<T, FACES_WALLS, true>(c, slab) : launch_typed<T, FACES_WALLS, false>(c, slab);
  return force ? launch_typed<T, FACES_BB, true>(c, slab) : launch_typed<T, FACES_BB, false>(c, slab);
}

template <typename T, bool FS>
hipError_t launch_slab_typed(lbm_ctx* c, const uint32_t* slab) {
  const Geom& G = c->geom;
  hipLaunchKernelGGL((k_slab<T, FS>), dim3(std::min(div_up(G.N, 256), 2048u)), dim3(256), step_lds(c),
                     c->stream, static_cast<const T*>(c->pops[c->hs.cur]), static_cast<T*>(c->mid),
                     static_cast<T*>(c->force), static_cast<T*>(c->vel), c->tiles[c->hs.flag_cur],
                     c->tiles[c->hs.flag_cur ^ 1], slab, G, (T)c->desc.omega, c->desc.flags, c->ntiles);
  return hipGetLastError();
}

}  // namespace

bool can_step2(const lbm_ctx* c) {
  return c->tiles2.ox != 0 && c->step_vec == 1;
}

hipError_t launch_step2(lbm_ctx* c, const uint32_t* slab) {
  const hipError_t e = timed(c, c->stream, [&] {
    return c->elem == 4 ? launch_faces<float>(c, slab) : launch_faces<double>(c, slab);
  });
  if (e == hipSuccess) {
    c->hs.cur ^= 1;
    c->hs.flag_clean[c->hs.flag_cur ^ 1] = true;
    c->hs.last_overlapped = false;
    c->hs.forced = false;
    c->hs.steps += 2;
  }
  return e;
}

hipError_t launch_slab(lbm_ctx* c, const uint32_t* slab) {
  hipError_t e;
  if (c->elem == 4)
    e = c->general ? launch_slab_typed<float, true>(c, slab) : launch_slab_typed<float, false>(c, slab);
  else
    e = c->general ? launch_slab_typed<double, true>(c, slab) : launch_slab_typed<double, false>(c, slab);
  if (e == hipSuccess) c->hs.flag_clean[c->hs.flag_cur ^ 1] = true;
  return e;
}

}  // namespace lbm
