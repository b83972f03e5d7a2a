// Two liquid steps per launch (step2_cell.hpp) of a single lattice, alone or coupled to bubbles.
//
// With bubbles, a pair of method steps is
//   bubble half n; k_slab: step n of the cells the bubbles reach, into the middle buffer;
//   bubble half n + 1; k_step2: both steps of every other cell, and step n + 1 of those.
// The cells the bubbles reach in the pair are a box, the slab, of rows and planes across all x: every
// force window of step n with a cell to spare on either side, and the velocity windows the second half
// reads (which hold its force windows). The bubble update finds it on the device as it moves each bubble.
// Outside it no cell holds force in either step, nor is its velocity read.
//
// An overlapped pair knows its slab beforehand (windows widened by the cells a bubble may move, reported
// if one moves further) and runs the bubble halves and k_slab beside the launch of everything else.
#include <algorithm>
#include <utility>

#include "step2_cell.hpp"

namespace lbm {
namespace {

template <typename T, int FACES, bool FORCE>
__global__ __launch_bounds__(step2_threads<T>()) void k_step2(Step2Args<T> A) {
  __shared__ Plane2<T, step2_threads<T>()> s[2];
  step2_block<T, FACES, FORCE>(s, A, xcd_remap(blockIdx.x, gridDim.x));
}

template <typename T, bool FS>
__global__ __launch_bounds__(256) void k_slab(SlabArgs<T> A) {
  slab_block<T, FS>(A, blockIdx.x, gridDim.x);
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
// counts it too high; within 6 % of the best of a sweep on eleven lattices from 30 x 30 x 90 to
// 256 x 256 x 256). Pieces of rows cost more than whole ones, whose loads and stores are contiguous
// over the tile, a piece of 512 bytes a quarter, of 128 bytes twice as much: 128 x 128 x 512 FP32
// 122 us per step in whole rows of 6, 132 us in tiles of 64 x 13, 144 us of 32 x 16; 256 x 256 x 256
// 253 us in whole rows of 2 (every intermediate row computed twice), 264 us in tiles of 128 x 5, 284 us
// of 64 x 13, 304 us of 32 x 16; 128 x 128 x 512 FP64 249 us in whole rows of 2, 264 us in tiles of
// 64 x 5, 299 us of 16 x 16.
bool choose_tiles2(const Geom& G, size_t elem, uint32_t cus, Tiles2* best) {
  const uint32_t threads = elem == 4 ? step2_threads<float>() : step2_threads<double>();
  const uint32_t align = 128u / (uint32_t)elem;  // cells of a cache line
  const uint32_t nx = (uint32_t)G.nx, ny = (uint32_t)G.ny, nz = (uint32_t)G.nz;
  double cost = 1e30;
  for (uint32_t ox = nx; ox >= 1; ox = ox == nx ? (nx - 1) / align * align : ox - align) {
    for (uint32_t oy = 1; oy <= ny && oy <= threads && tile_threads(G, ox, oy) <= threads; ++oy) {
      const uint32_t ntx = div_up(nx, ox), nty = div_up(ny, oy), nt = ntx * nty;
      const uint32_t nc = std::max(1u, std::min(nz, cus / nt));
      const double v = (double)div_up(nt * nc, cus) * ((double)nz / nc + 2.0) * ox * (oy + 2.0) *
                       (ox == nx ? 1.0 : 1.0 + 128.0 / ((double)ox * elem));
      if (v < cost) {
        cost = v;
        *best = {ox, oy, ntx, nty, nc};
      }
    }
    if (ox < align) break;
  }
  return cost < 1e30;
}

// Microseconds of a launch of two steps and of two launches of one, fitted to 360 lattices of 0.13 to 3 million
// cells (FP32 and FP64, walls, free-slip tops and periodic axes, 4 to 3000 cells wide; all but 3 % of the
// choices between the two are the faster one or within 10 % of it). A workgroup takes as long for a plane however
// few threads it has, so narrow lattices lose: 8 x 8 x 20000 FP32 with a free-slip top 233 us against 59 us,
// 16 x 16 x 4000 59 and 50, 32 x 32 x 800 58 and 42; 64 x 64 x 192 30 and 35 with walls, 38 and 38 with that top,
// 37 and 44 periodic; 128 x 100 x 100 41 and 56; 48 x 48 x 144 FP64 29 and 35, 64 x 64 x 192 49 and 68.
Pairs choose_pairs(const Geom& G, size_t elem) {
  Pairs p = {};
  if (G.N < step2_min_cells(elem) || !bb_fast_ok(G, elem) || !choose_tiles2(G, elem, kCus, &p.alone) ||
      !choose_tiles2(G, elem, kCusBeside, &p.beside)) {
    p.alone = p.beside = Tiles2{};
    return p;
  }
  bool walls = true, periodic = false;
  for (int f = 0; f < 6; ++f) {
    walls = walls && G.bc[f] == BC_BB;
    periodic = periodic || G.bc[f] == BC_PER;
  }
  const double mb = 38e-6 * elem;  // a step's bytes per cell, in millions
  const double chunk = p.alone.nchunk == 1 ? G.nz + 1.0 : div_up(G.nz, p.alone.nchunk) + 2.0;
  const double planes = div_up(p.alone.ntx * p.alone.nty * p.alone.nchunk, kCus) * chunk;
  const double two = (walls ? 8.0 : 7.0) + (walls ? 1.7 : 2.55) * planes + (G.stream1 ? 0.125 : 0.07) * mb * G.N;
  const double rate = G.stream1 ? (periodic ? 0.24 : 0.16) : periodic ? 0.14 : walls ? 0.112 : 0.127;
  const double singles = 2.0 * ((periodic ? 7.0 : 5.0) + rate * mb * G.N);
  p.liquid = two < singles;
  if (periodic || G.N < pair_min_cells(elem)) return p;
  // with bubbles: the slab's two steps on top, of rows across all x (2000 x 8 x 60 FP32, one bubble: 95 us in a
  // pair, 79 in two steps; 64 x 64 x 200 74 and 75, with a free-slip top 81 and 78; 72 x 72 x 216 81 and 90, 86 and
  // 92). Overlapped single steps take some 30 us a pair longer than serial ones (the region launch and the
  // waits), overlapped pairs do not: 64 x 64 x 200 71 and 102.
  const double slab = 3.0 + 0.3 * mb * G.nx * std::min(G.ny, 16) * std::min(G.nz, 16);
  p.serial = two + slab < singles;
  p.overlapped = two + slab < singles + 30.0;
  return p;
}

namespace {

template <typename T, int FACES, bool FORCE>
hipError_t launch_typed(lbm_ctx* c, const uint32_t* slab, bool bulk) {
  const Geom& G = c->geom;
  Step2Args<T> A;
  A.src = static_cast<const T*>(c->pops[c->hs.cur]);
  A.mid = static_cast<const T*>(c->pops[third_buffer(c->hs)]);
  A.dst = static_cast<T*>(c->pops[c->hs.nxt]);
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
  A.bulk = bulk ? 1 : 0;
  A.L = bulk ? c->pairs.beside : c->pairs.alone;
  const uint32_t n = A.L.ntx * A.L.nty * A.L.nchunk;
  hipLaunchKernelGGL((k_step2<T, FACES, FORCE>), dim3(n), dim3(step2_threads<T>()), 0, c->stream, A);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_faces(lbm_ctx* c, const uint32_t* slab, bool bulk) {
  const bool force = c->desc.flags & LBM_FLAG_STATIC_FORCE;
  if (c->periodic)
    return force ? launch_typed<T, FACES_GENERAL, true>(c, slab, bulk)
                 : launch_typed<T, FACES_GENERAL, false>(c, slab, bulk);
  if (c->general)
    return force ? launch_typed<T, FACES_WALLS, true>(c, slab, bulk)
                 : launch_typed<T, FACES_WALLS, false>(c, slab, bulk);
  return force ? launch_typed<T, FACES_BB, true>(c, slab, bulk) : launch_typed<T, FACES_BB, false>(c, slab, bulk);
}

template <typename T, bool FS>
hipError_t launch_slab_typed(lbm_ctx* c, const uint32_t* slab, int part, hipStream_t s) {
  const Geom& G = c->geom;
  const bool second = part == SLAB_SECOND;
  void* const mid = c->pops[third_buffer(c->hs)];
  const void* src = second ? mid : c->pops[c->hs.cur];
  void* dst = second ? c->pops[c->hs.nxt] : mid;
  const SlabArgs<T> A = {static_cast<const T*>(src), static_cast<T*>(dst), static_cast<T*>(c->force),
                         static_cast<T*>(c->vel), c->tiles[c->hs.flag_cur], c->tiles[c->hs.flag_cur ^ 1], slab, G,
                         (T)c->desc.omega, c->desc.flags, c->ntiles,
                         part == SLAB_FIRST ? c->pairs.alone.oy : c->pairs.beside.oy, part};
  hipLaunchKernelGGL((k_slab<T, FS>), dim3(std::min(div_up(G.N, 256), 2048u)), dim3(256),
                     part == SLAB_FIRST_WHOLE ? 0 : step_lds(c), s, A);
  return hipGetLastError();
}

hipError_t launch_slab_part(lbm_ctx* c, const uint32_t* slab, int part, hipStream_t s) {
  hipError_t e;
  if (c->elem == 4)
    e = c->general ? launch_slab_typed<float, true>(c, slab, part, s) : launch_slab_typed<float, false>(c, slab, part, s);
  else
    e = c->general ? launch_slab_typed<double, true>(c, slab, part, s)
                   : launch_slab_typed<double, false>(c, slab, part, s);
  if (e == hipSuccess) c->hs.flag_clean[c->hs.flag_cur ^ 1] = true;
  return e;
}

}  // namespace

bool can_step2(const lbm_ctx* c) {
  return c->pairs.alone.ox != 0 && c->step_vec == 1;
}

hipError_t launch_step2(lbm_ctx* c, const uint32_t* slab) {
  const hipError_t e = timed(c, c->stream, [&] {
    return c->elem == 4 ? launch_faces<float>(c, slab, false) : launch_faces<double>(c, slab, false);
  });
  if (e == hipSuccess) {
    swap_buffers(c->hs);
    c->hs.flag_clean[c->hs.flag_cur ^ 1] = true;
    c->hs.last_overlapped = false;
    c->hs.forced = false;
    c->hs.steps += 2;
  }
  return e;
}

hipError_t launch_slab(lbm_ctx* c, const uint32_t* slab) {
  return launch_slab_part(c, slab, SLAB_FIRST, c->stream);
}

hipError_t launch_pair_bulk(lbm_ctx* c, const uint32_t* slab) {
  return timed(c, c->stream, [&] {
    return c->elem == 4 ? launch_faces<float>(c, slab, true) : launch_faces<double>(c, slab, true);
  });
}

hipError_t launch_pair_first(lbm_ctx* c, const uint32_t* slab, hipStream_t s) {
  return launch_slab_part(c, slab, SLAB_FIRST_WHOLE, s);
}

hipError_t launch_pair_second(lbm_ctx* c, const uint32_t* slab) {
  const hipError_t e = launch_slab_part(c, slab, SLAB_SECOND, c->stream);
  if (e == hipSuccess) {
    swap_buffers(c->hs);
    c->hs.last_overlapped = c->hs.last_pair = true;
    c->hs.forced = false;
    c->hs.steps += 2;
  }
  return e;
}

}  // namespace lbm
