// Two liquid steps in one pass over a range of z-planes (eq. (13)-(16) applied twice with the face
// conditions of Sec. 3.3), shared by the single-lattice and the batched launches.
//
// What bounds it: one step of the fused kernel moves 152 B per FP32 site (19 loads, 19 stores) at
// the rate a plain copy reaches, so a lattice can only go faster by moving fewer bytes. Here a
// workgroup marches along z over a tile of x and y: the intermediate state of a plane is computed
// from the source buffer (19 loads per site), crosses the workgroup through LDS, and the second
// step is stored (19 stores per site): 152 B per site for two steps, plus the re-read of a tile's
// halo (one site around it along x and y where the tile ends inside the lattice, one plane above
// and below its range), most of which hits the L2 since the neighbouring tiles run beside it.
//
// Registers and LDS: populations that stay in their column (rest, +z, -z) never leave registers; the
// other 16 of a plane go through LDS, double-buffered (one barrier per plane). Each thread pulls what
// the plane just finished gives to its own output cells right after the barrier: the c_z = -1
// populations complete the output plane below, the c_z = 0 and +1 ones wait in registers (9 for one
// plane, 5 for two). The loads of the next plane are issued before the second collision and its
// stores, so they are in flight meanwhile and their wait does not include the stores.
//
// The tile takes whole rows of x where they fit (an output row is then one contiguous store and
// needs no halo along x), else aligned pieces of rows with the halo columns in threads of their own.
#pragma once

#include <utility>

#include "step_cell.hpp"

namespace lbm {

// Faces of a lattice or batch (template parameter of the liquid kernels): every face bounce-back,
// walls only (bounce-back or free slip), or some face periodic.
enum : int { FACES_BB = 0, FACES_WALLS = 1, FACES_GENERAL = 2 };

// Populations by c_z; kUp[m] and kDown[m] share c_x and c_y, and so do their lateral walls.
constexpr int kUp[5] = {4, 10, 11, 14, 15};
constexpr int kDown[5] = {5, 12, 13, 16, 17};
constexpr int kFlat[9] = {18, 0, 1, 2, 3, 6, 7, 8, 9};

// LDS slot of a population that leaves its column (c_x or c_y nonzero).
__host__ __device__ constexpr int lds_slot(int q) {
  for (int i = 1; i < 9; ++i)
    if (kFlat[i] == q) return i - 1;
  for (int i = 1; i < 5; ++i) {
    if (kUp[i] == q) return 7 + i;
    if (kDown[i] == q) return 11 + i;
  }
  return 0;
}
__host__ __device__ constexpr bool in_lds(int q) { return CX[q] != 0 || CY[q] != 0; }

// Lateral walls (bits of the walls mask) beyond which the source of population q lies.
__host__ __device__ constexpr uint32_t lat_mask(int q) {
  return (CX[q] > 0 ? 1u : 0u) | (CX[q] < 0 ? 2u : 0u) | (CY[q] > 0 ? 4u : 0u) | (CY[q] < 0 ? 8u : 0u);
}

// Compile-time loops: over all populations, and over the members of kUp, kDown and kFlat that cross
// the workgroup (f receives the member's index and population as constants).
template <class Fn, int... Qs>
__device__ __forceinline__ void for_q(Fn&& f, std::integer_sequence<int, Qs...>) {
  (f(std::integral_constant<int, Qs>{}), ...);
}
template <class Fn>
__device__ __forceinline__ void for_each_q(Fn&& f) {
  for_q(f, std::make_integer_sequence<int, 19>{});
}
template <const int* LIST, int... Ms>
struct CrossList {
  template <class Fn>
  __device__ __forceinline__ void operator()(Fn&& f) const {
    (f(std::integral_constant<int, Ms>{}, std::integral_constant<int, LIST[Ms]>{}), ...);
  }
};
using ForUp = CrossList<kUp, 1, 2, 3, 4>;
using ForDown = CrossList<kDown, 1, 2, 3, 4>;
using ForFlat = CrossList<kFlat, 1, 2, 3, 4, 5, 6, 7, 8>;

template <typename T, int NT>
struct Plane2 {
  T v[16 * NT];
};

// Threads of a workgroup: FP32 holds 121-128 VGPRs, FP64 about 200.
template <typename T>
constexpr int step2_threads() {
  return sizeof(T) == 4 ? 1024 : 512;
}

// What the pass reads and writes of one lattice.
struct Lattice2 {
  const gchar* src;
  gchar* dst;
  const gchar* F;   // FORCE: the static force field
  gchar* U;
  const gchar* tiles;  // tiles whose velocity the second step writes
  int fa, fb;          // planes [fa, fb) that may hold such tiles
  bool u_all;          // write the velocity everywhere
};

// Two steps of the output cells of tile (txi, tyi), planes [z0, z1), by the whole workgroup.
// FORCE: a static force field, read in every cell and never cleared (its velocity is written
// everywhere); else no cell the pass computes holds force in either step.
template <typename T, int FACES, bool FORCE, int NT>
__device__ void march2(Plane2<T, NT>* s, const Geom& G, const Lattice2& A, T omega, const Tiles2& L,
                       uint32_t txi, uint32_t tyi, int z0, int z1) {
  constexpr bool FS = FACES != FACES_BB;
  constexpr bool PER = FACES == FACES_GENERAL;
  constexpr uint32_t esz = sizeof(T);
  const bool perx = PER && G.bc[0] == BC_PER, pery = PER && G.bc[2] == BC_PER,
             perz = PER && G.bc[4] == BC_PER;
  const int ox0 = (int)(txi * L.ox), ox1 = min(ox0 + (int)L.ox, G.nx);
  const int oy0 = (int)(tyi * L.oy), oy1 = min(oy0 + (int)L.oy, G.ny);
  // halo rows and columns: beyond a tile edge inside the lattice or on a periodic axis
  const bool hl = perx || ox0 > 0, hr = perx || ox1 < G.nx;
  const int iy0 = pery || oy0 > 0 ? oy0 - 1 : oy0, iy1 = pery || oy1 < G.ny ? oy1 + 1 : oy1;
  const int w = ox1 - ox0, h = iy1 - iy0, body = w * h;
  const int t = threadIdx.x;
  // this thread's intermediate cell: row j of the tile; column i of the body, or a halo column
  int i, j;
  bool main = t < body;
  if (main) {
    j = t / w;
    i = t - j * w;
  } else {
    j = t - body;
    i = hl ? -1 : w;
    if (hl && j >= h) {
      j -= h;
      i = w;
    }
  }
  const bool act = main || (j < h && (i < 0 ? hl : hr));
  int x = ox0 + i, y = iy0 + j;
  const bool out = main && y >= oy0 && y < oy1;
  if constexpr (PER) {
    if (x < 0) x += G.nx;
    if (x >= G.nx) x -= G.nx;
    if (y < 0) y += G.ny;
    if (y >= G.ny) y -= G.ny;
  }
  const bool xlo = act && x == 0, xhi = act && x == G.nx - 1;
  const bool ylo = act && y == 0, yhi = act && y == G.ny - 1;
  // lateral walls beside the cell
  const uint32_t lat = (xlo && !perx ? 1u : 0u) | (xhi && !perx ? 2u : 0u) |
                       (ylo && !pery ? 4u : 0u) | (yhi && !pery ? 8u : 0u);
  const uint32_t fs = FS ? free_slip_faces(G) : 0u;
  // per wavefront: 0 no lane beside a lateral face, 1 only beside bounce-back faces normal to x
  // (every wavefront of whole rows), 2 anything else
  const bool xface = __any(xlo || xhi), yface = __any(ylo || yhi);
  const int path = !xface && !yface ? 0 : (!yface && !perx && !(fs & 3u) ? 1 : 2);
  // What the addresses of the pulls follow from: the lateral walls beside the cell, its LDS index,
  // those of its neighbours along x and the index stride of y there (halo columns follow the body),
  // and on periodic axes the byte offsets of its neighbours. They are made opaque in every
  // iteration: the compiler otherwise keeps some 50 addresses and conditions of the pulls in registers
  // across the loop and spills (FP32: 142 registers).
  struct Lane {
    uint32_t lat;
    int t, xm, sm, xp, sp;
    int dxm, dxp, dym, dyp;
  } ln;
  ln.lat = lat;
  ln.t = t;
  ln.xm = i > 0 ? t - 1 : (hl ? body + j : t);
  ln.sm = i > 0 ? w : 1;
  ln.xp = i < w - 1 ? t + 1 : (hr ? body + (hl ? h : 0) + j : t);
  ln.sp = i < w - 1 ? w : 1;
  ln.dxm = ln.dxp = ln.dym = ln.dyp = 0;
  if constexpr (PER) {
    ln.dxm = (xlo && perx ? G.nx - 1 : -1) * (int)esz;
    ln.dxp = (xhi && perx ? 1 - G.nx : 1) * (int)esz;
    ln.dym = (ylo && pery ? G.ny - 1 : -1) * G.nx * (int)esz;
    ln.dyp = (yhi && pery ? 1 - G.ny : 1) * G.nx * (int)esz;
  }
  auto opaque = [&] {
    asm volatile("" : "+v"(ln.lat), "+v"(ln.t), "+v"(ln.xm), "+v"(ln.sm), "+v"(ln.xp), "+v"(ln.sp));
    if constexpr (PER) asm volatile("" : "+v"(ln.dxm), "+v"(ln.dxp), "+v"(ln.dym), "+v"(ln.dyp));
  };
  const uint32_t xy4 = ((uint32_t)y * G.nx + (uint32_t)x) * esz;
  const uint32_t zs4 = G.zs * esz, n4 = G.N * esz, plane4 = G.plane * esz;
  const bool stream = G.stream2;

  // the 19 populations arriving at the cell in plane k of the source buffer (and its force)
  auto load = [&](int k, T* g, T* f) {
    if (!act) return;
    int kz = k;
    if constexpr (PER) {
      if (perz && kz < 0) kz += G.nz;
      if (perz && kz >= G.nz) kz -= G.nz;
    }
    const uint32_t lc4 = xy4 + (uint32_t)kz * zs4;
    if constexpr (FORCE) {
      const uint32_t c4 = xy4 + (uint32_t)kz * plane4;
      f[0] = load_at<T>(A.F, c4);
      f[1] = load_at<T>(A.F, c4 + n4);
      f[2] = load_at<T>(A.F, c4 + 2 * n4);
    }
    const bool inner = kz > 0 && kz < G.nz - 1;
    if (path == 0 && inner) {
      auto one = [&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const int64_t at = ((int64_t)q * G.qs - (CX[q] + CY[q] * G.nx) - (int64_t)CZ[q] * G.zs) * (int)esz;
        g[q] = load_at<T>(A.src + at, lc4);
      };
      for_each_q(one);
    } else if (path == 1 && inner) {
      auto one = [&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if constexpr (CX[q] == 0) {
          const int64_t at = ((int64_t)q * G.qs - CY[q] * G.nx - (int64_t)CZ[q] * G.zs) * (int)esz;
          g[q] = load_at<T>(A.src + at, lc4);
        } else {
          // the population or, beyond the wall, the cell's own opposite, from the lower one's base
          constexpr int o = opposite(q), q0 = q < o ? q : o;
          const uint32_t k0 = (uint32_t)(q - q0) * G.qs * esz -
                              (uint32_t)(CX[q] + CY[q] * G.nx + CZ[q] * (int)G.zs) * esz;
          const uint32_t kb = (uint32_t)(o - q0) * G.qs * esz;
          const bool beyond = ln.lat & lat_mask(q);
          g[q] = load_at<T>(A.src + (int64_t)q0 * G.qs * (int)esz, lc4 + (beyond ? kb : k0));
        }
      };
      for_each_q(one);
    } else if constexpr (!PER) {
      const uint32_t walls = ln.lat | (kz == 0 ? 16u : 0u) | (kz == G.nz - 1 ? 32u : 0u);
      pull_bb_all<T, FS>(g, A.src, G, lc4, walls, fs, std::make_integer_sequence<int, 19>{});
    } else {
      // the rules of pull_index with 32-bit byte offsets: wrapped neighbours on periodic axes
      const uint32_t walls = ln.lat | (kz == 0 && !perz ? 16u : 0u) | (kz == G.nz - 1 && !perz ? 32u : 0u);
      // modulo 2^32: a state of 2 to 4 GiB spans more than an int
      const uint32_t round_z = (uint32_t)(G.nz - 1) * zs4;
      const uint32_t dzm = kz == 0 && perz ? round_z : 0u - zs4;
      const uint32_t dzp = kz == G.nz - 1 && perz ? 0u - round_z : zs4;
      const uint32_t qs4 = G.qs * esz;
      auto one = [&](auto qc) {
        constexpr int q = decltype(qc)::value;
        constexpr uint32_t m = lat_mask(q) | (CZ[q] > 0 ? 16u : 0u) | (CZ[q] < 0 ? 32u : 0u);
        const uint32_t dx = (uint32_t)(CX[q] > 0 ? ln.dxm : CX[q] < 0 ? ln.dxp : 0);
        const uint32_t dy = (uint32_t)(CY[q] > 0 ? ln.dym : CY[q] < 0 ? ln.dyp : 0);
        const uint32_t dz = CZ[q] > 0 ? dzm : CZ[q] < 0 ? dzp : 0u;
        const uint32_t hit = walls & m;
        uint32_t at = (uint32_t)q * qs4 + dx + dy + dz;
        if (hit) {
          at = (uint32_t)opposite(q) * qs4;
          if ((hit & (hit - 1u)) == 0u && (hit & fs)) {
            const uint32_t ax = (uint32_t)mirrored(q, 0) * qs4 + dy + dz;
            const uint32_t ay = (uint32_t)mirrored(q, 1) * qs4 + dx + dz;
            const uint32_t az = (uint32_t)mirrored(q, 2) * qs4 + dx + dy;
            at = (hit & 3u) ? ax : (hit & 12u) ? ay : az;
          }
        }
        g[q] = load_at<T>(A.src, lc4 + at);
      };
      for_each_q(one);
    }
  };

  // Population q arriving laterally at the cell from the plane in sp_. Beyond one free-slip wall:
  // the mirrored population with that axis' shift dropped; beyond bounce-back walls an in-plane
  // population is the cell's own opposite (for c_z != 0 that opposite belongs to the output plane:
  // the caller's).
  auto pull_lat = [&](const Plane2<T, NT>& sp_, auto qc, auto pc) -> T {
    constexpr int q = decltype(qc)::value, P = decltype(pc)::value;
    constexpr int cx = CX[q], cy = CY[q], o = CZ[q] == 0 ? opposite(q) : q;
    const int nb = cx == 0 ? ln.t : cx > 0 ? ln.xm : ln.xp;
    const int stride = cx == 0 ? w : cx > 0 ? ln.sm : ln.sp;
    int at = nb - cy * stride + lds_slot(q) * NT;
    if constexpr (P == 1 && cx != 0 && CZ[q] == 0) {
      if (ln.lat & lat_mask(q)) at = lds_slot(o) * NT + ln.t;
    }
    if constexpr (P == 2) {
      const uint32_t hit = ln.lat & lat_mask(q);
      if (hit) {
        at = lds_slot(o) * NT + ln.t;
        if (FS && (hit & (hit - 1u)) == 0u && (hit & fs)) {
          const int mx = lds_slot(mirrored(q, 0)) * NT + ln.t - cy * w;
          const int my = lds_slot(mirrored(q, 1)) * NT + nb;
          at = (hit & 3u) ? mx : my;
        }
      }
    }
    return sp_.v[at];
  };
  auto pulls = [&](const Plane2<T, NT>& sp_, auto list, T* v) {
    auto go = [&](auto pc) {
      list([&](auto mc, auto qc) { v[decltype(mc)::value] = pull_lat(sp_, qc, pc); });
    };
    if (path == 0)
      go(std::integral_constant<int, 0>{});
    else if (path == 1)
      go(std::integral_constant<int, 1>{});
    else
      go(std::integral_constant<int, 2>{});
  };

  T up1[5], up2[5], in1[9], gn[19];
  T fn[3] = {T(0), T(0), T(0)}, f1[3] = {T(0), T(0), T(0)};
#pragma unroll
  for (int m = 0; m < 5; ++m) up1[m] = up2[m] = T(0);
#pragma unroll
  for (int m = 0; m < 9; ++m) in1[m] = T(0);

  const int ka = perz ? z0 - 1 : max(z0 - 1, 0);
  __syncthreads();  // the LDS planes of a previous range
  load(ka, gn, fn);
  int p = 0;
  // the last iteration completes plane z1 - 1; at the top of the lattice it has no plane of its own
#pragma unroll 1
  for (int k = ka; k <= z1; ++k, p ^= 1) {
    opaque();
    const bool plane = perz || k < G.nz;
    const Plane2<T, NT>& sp_ = s[p];
    const Plane2<T, NT>& sq = s[p ^ 1];
    T rest = T(0), gz = T(0), gmz = T(0);
    T f0[3] = {fn[0], fn[1], fn[2]};
    if (plane && act) {
      T ux, uy, uz;
      collide<T, FORCE>(gn, f0[0], f0[1], f0[2], omega, ux, uy, uz);
#pragma unroll
      for (int q = 0; q < 18; ++q)
        if (in_lds(q)) s[p].v[lds_slot(q) * NT + ln.t] = gn[q];
      rest = gn[18];
      gz = gn[4];
      gmz = gn[5];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (k < z1 && (perz || k + 1 < G.nz)) load(k + 1, gn, fn);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    if (out) {
      T dn[5];
      dn[0] = gmz;
      if (plane) pulls(sp_, ForDown{}, dn);
      if (k - 1 >= z0) {
        // complete output plane k - 1
        T f[19], ux, uy, uz;
#pragma unroll
        for (int m = 0; m < 5; ++m) {
          f[kUp[m]] = up2[m];
          f[kDown[m]] = dn[m];
        }
#pragma unroll
        for (int m = 0; m < 9; ++m) f[kFlat[m]] = in1[m];
        if (!plane) {  // top wall: mirrored at a free-slip face, else the own opposite
          const bool zfs = FS && (fs & 32u);
          f[kDown[0]] = up1[0];
#pragma unroll
          for (int m = 1; m < 5; ++m) {
            const T o = sq.v[lds_slot(opposite(kDown[m])) * NT + ln.t];
            f[kDown[m]] = zfs && !(ln.lat & lat_mask(kDown[m])) ? up1[m] : o;
          }
        } else if (path != 0) {
          // beyond a lateral bounce-back wall: the own opposite of plane k - 1
#pragma unroll
          for (int m = 1; m < 5; ++m)
            if ((ln.lat & ~fs) & lat_mask(kDown[m])) f[kDown[m]] = sq.v[lds_slot(opposite(kDown[m])) * NT + ln.t];
        }
        collide<T, FORCE>(f, f1[0], f1[1], f1[2], omega, ux, uy, uz);
        const int zo = k - 1;
        const uint32_t lc4 = xy4 + (uint32_t)zo * zs4;
        if (stream) {
          keep_branch();
#pragma unroll
          for (int q = 0; q < 19; ++q)
            __builtin_nontemporal_store(
                f[q], reinterpret_cast<gmem<T>*>(A.dst + (int64_t)q * G.qs * (int)esz + lc4));
          keep_branch();
        } else {
#pragma unroll
          for (int q = 0; q < 19; ++q) store_at<T>(A.dst + (int64_t)q * G.qs * (int)esz, lc4, f[q]);
        }
        const bool flagged_planes = zo >= A.fa && zo < A.fb;
        if (FORCE || A.u_all || flagged_planes) {
          bool write = FORCE || A.u_all;
          if (!write)
            write = load_at<uint8_t>(A.tiles, (((uint32_t)zo >> 3) * G.tny + ((uint32_t)y >> 3)) * G.tnx +
                                                  ((uint32_t)x >> 3)) != 0;
          if (write) {
            const uint32_t c4 = xy4 + (uint32_t)zo * plane4;
            store_at<T>(A.U, c4, ux);
            store_at<T>(A.U, c4 + n4, uy);
            store_at<T>(A.U, c4 + 2 * n4, uz);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (plane) {
        in1[0] = rest;
        pulls(sp_, ForFlat{}, in1);
        // c_z = +1 of output plane k: pulled from plane k - 1, or beyond a wall
        if (!perz && k == 0) {
          const bool zfs = FS && (fs & 16u);
          up1[0] = gmz;
#pragma unroll
          for (int m = 1; m < 5; ++m) {
            const T o = sp_.v[lds_slot(opposite(kUp[m])) * NT + ln.t];
            up1[m] = zfs && !(ln.lat & lat_mask(kUp[m])) ? dn[m] : o;
          }
        } else if (path != 0) {
#pragma unroll
          for (int m = 1; m < 5; ++m)
            if ((ln.lat & ~fs) & lat_mask(kUp[m])) up1[m] = sp_.v[lds_slot(opposite(kUp[m])) * NT + ln.t];
        }
#pragma unroll
        for (int m = 0; m < 5; ++m) up2[m] = up1[m];
        up1[0] = gz;
        pulls(sp_, ForUp{}, up1);
        f1[0] = f0[0];
        f1[1] = f0[1];
        f1[2] = f0[2];
      }
    }
  }
}

// One step of one cell, inside a loop over cells. The strides are made opaque in every
// iteration: hoisted out of the loop, the 38 offsets that follow from them fill the registers.
template <typename T, bool FS>
__device__ __forceinline__ void step_one(const gchar* src, gchar* dst, gchar* F, gchar* U,
                                         const gchar* tiles, const Geom& G0, T omega, int flags,
                                         uint32_t x, uint32_t y, uint32_t z, uint32_t fs) {
  Geom G = G0;
  asm volatile("" : "+s"(G.qs), "+s"(G.zs), "+s"(G.nx));
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
  int bulk;   // an overlapped pair's planes outside the slab (whole tiles) and nothing else
};

// One workgroup's share of a two-step launch: block b of the lattice's tiles and chunks of planes. Of a
// tile whose rows the slab holds, the planes outside the slab in two steps and as many parts of those
// inside in one, so that the launch stays balanced whatever the slab holds.
template <typename T, int FACES, bool FORCE>
__device__ __forceinline__ void step2_block(Plane2<T, step2_threads<T>()>* s, const Step2Args<T>& A, uint32_t b) {
  constexpr int NT = step2_threads<T>();
  const Geom& G = A.G;
  const uint32_t nblocks = A.L.ntx * A.L.nty * A.L.nchunk;
  const uint32_t txi = b % A.L.ntx, r = b / A.L.ntx;
  const uint32_t tyi = r % A.L.nty, ch = r / A.L.nty;
  const Box box = slab_box(A.slab, G, A.bulk, A.L.oy);
  const int y0 = (int)(tyi * A.L.oy), y1 = min(y0 + (int)A.L.oy, G.ny);
  const bool in_slab = y0 < box.yb && y1 > box.ya;  // the box holds whole tiles of rows
  const int sa = in_slab ? box.za : 0, sb = in_slab ? box.zb : 0;
  Lattice2 D;
  D.src = gbytes<T>(A.src);
  D.dst = gbytes<T>(A.dst);
  D.F = gbytes<T>(A.F);
  D.U = gbytes<T>(A.U);
  D.tiles = gbytes<uint8_t>(A.tiles);
  D.u_all = A.flags & LBM_FLAG_WRITE_U_ALL;
  if (A.bulk) {
    D.fa = D.fb = 0;  // every flagged tile lies in the slab
  } else if (A.slab) {
    const Box f = slab_box(A.slab + 4, G, true, 1);  // planes of the second half's windows
    D.fa = f.za;
    D.fb = f.zb;
  } else {
    D.fa = 0;
    D.fb = A.dirty ? G.nz : 0;
  }
  // chunk of the planes outside the slab, counted without it; the march is one call site for the parts
  // below and above the slab (twice its code does not fit the instruction cache)
  const uint32_t nzb = (uint32_t)(G.nz - (sb - sa));
  const int c0 = (int)(ch * nzb / A.L.nchunk), c1 = (int)((ch + 1) * nzb / A.L.nchunk);
#pragma unroll 1
  for (int part = 0; part < 2; ++part) {
    const int z0 = part == 0 ? c0 : max(c0, sa) + (sb - sa), z1 = part == 0 ? min(c1, sa) : c1 + (sb - sa);
    if (z0 < z1) march2<T, FACES, FORCE, NT>(s, G, D, A.omega, A.L, txi, tyi, z0, z1);
  }
  if (A.bulk) return;
  if constexpr (FACES != FACES_GENERAL && !FORCE) {
    const uint32_t nzs = (uint32_t)(sb - sa);
    const int p0 = sa + (int)(ch * nzs / A.L.nchunk), p1 = sa + (int)((ch + 1) * nzs / A.L.nchunk);
    const int x0 = (int)(txi * A.L.ox), x1 = min(x0 + (int)A.L.ox, G.nx);
    const uint32_t fs = FACES == FACES_WALLS ? free_slip_faces(G) : 0u;
    const uint32_t w = (uint32_t)(x1 - x0), wh = w * (uint32_t)(y1 - y0), cells = wh * (uint32_t)(p1 - p0);
#pragma unroll 1
    for (uint32_t k = threadIdx.x; k < cells; k += NT) {
      const uint32_t z = k / wh, rem = k - z * wh, y = rem / w, x = rem - y * w;
      step_one<T, FACES == FACES_WALLS>(gbytes<T>(A.mid), D.dst, gbytes<T>(A.F), D.U, D.tiles, G, A.omega,
                                        A.flags, (uint32_t)x0 + x, (uint32_t)y0 + y, (uint32_t)p0 + z, fs);
    }
  }
  for (uint32_t k = b * NT + threadIdx.x; k < A.ntiles; k += nblocks * NT) A.tiles_next[k] = 0;
}

// One step of a slab's cells from src into dst. SLAB_FIRST: step n of a pair, from the current state into
// the middle buffer, with one row and plane beside the slab on every side; widened to whole force
// tiles, so that the velocity is written in every tile the first bubble half flagged. SLAB_FIRST_WHOLE:
// the same of an overlapped pair, whose slab is whole tiles. SLAB_SECOND: its step n + 1.
enum : int { SLAB_FIRST = 0, SLAB_FIRST_WHOLE = 1, SLAB_SECOND = 2 };

template <typename T>
struct SlabArgs {
  const T* src;
  T* dst;
  T* F;
  T* U;
  const uint8_t* tiles;
  uint8_t* tiles_next;
  const uint32_t* slab;
  Geom G;
  T omega;
  int flags;
  uint32_t ntiles, oy;
  int part;
};

// The cells in turn over the 256-thread workgroups [0, nblocks).
template <typename T, bool FS>
__device__ __forceinline__ void slab_block(const SlabArgs<T>& A, uint32_t block, uint32_t nblocks) {
  const Geom& G = A.G;
  Box b = slab_box(A.slab, G, A.part != SLAB_FIRST, A.oy);
  if (b.zb > b.za && A.part != SLAB_SECOND) {
    constexpr int m = (int)kTile - 1;
    b.za = max(0, min(b.za - 1, b.za & ~m));
    b.ya = max(0, min(b.ya - 1, b.ya & ~m));
    b.zb = min(G.nz, max(b.zb + 1, (b.zb + m) & ~m));
    b.yb = min(G.ny, max(b.yb + 1, (b.yb + m) & ~m));
  }
  const uint32_t rows = (uint32_t)(b.yb - b.ya) * (uint32_t)G.nx, cells = rows * (uint32_t)(b.zb - b.za);
  const uint32_t fs = FS ? free_slip_faces(G) : 0u;
#pragma unroll 1
  for (uint32_t k = block * 256 + threadIdx.x; k < cells; k += nblocks * 256) {
    const uint32_t z = k / rows, rem = k - z * rows, y = rem / (uint32_t)G.nx, x = rem - y * (uint32_t)G.nx;
    step_one<T, FS>(gbytes<T>(A.src), gbytes<T>(A.dst), gbytes<T>(A.F), gbytes<T>(A.U), gbytes<uint8_t>(A.tiles),
                    G, A.omega, A.flags, x, (uint32_t)b.ya + y, (uint32_t)b.za + z, fs);
  }
  for (uint32_t k = block * 256 + threadIdx.x; k < A.ntiles; k += nblocks * 256) A.tiles_next[k] = 0;
}

}  // namespace lbm
