// Macroscopic fields and global sums of the current state (eq. (10)), the pre-collision
// population view, and a plain fill kernel. The stored buffer holds post-collision populations,
// so both gathers apply the streaming step (with the face conditions) on the fly.
#include <utility>

#include "collide.hpp"
#include "step2_cell.hpp"
#include "wave.hpp"

namespace lbm {
namespace {

constexpr int kThreads = 256;

// The 19 populations arriving at a cell. With walls only (and 32-bit byte offsets) as the
// liquid step pulls them: with the general pull k_moments was held by its address arithmetic.
template <typename T, int FACES>
__device__ __forceinline__ void pull_cell(T* g, const T* __restrict__ src, const Geom& G, uint32_t cell,
                                          uint32_t x, uint32_t y, uint32_t z) {
  const uint32_t lc = layout_cell(G, cell, z);
  if constexpr (FACES == FACES_GENERAL) {
    const CellNbr nb = cell_neighbours(G, (int)x, (int)y, (int)z);
    pull_all<true>(g, src, G, lc, nb, std::make_integer_sequence<int, 19>{});
  } else {
    pull_bb_all<T, FACES == FACES_WALLS>(g, gbytes<T>(src), G, lc * (uint32_t)sizeof(T),
                                         wall_bits(G, (int)x, (int)y, z),
                                         FACES == FACES_WALLS ? free_slip_faces(G) : 0u,
                                         std::make_integer_sequence<int, 19>{});
  }
}

// What bounds it: the 92 bytes of a cell in FP32 (76 read, 16 written). 128 x 128 x 512 with a free-slip
// top: 147 us (5.2 TB/s); with the general pull and each cell loaded when its turn came 229 us.
// Grid-stride over cells; per-block partial sums of (sum drho, sum rho u) in double precision. The next
// cell's populations are on their way while a cell's are summed; its coordinates follow by addition.
template <typename T, int FACES>
__global__ __launch_bounds__(kThreads) void k_moments(const T* __restrict__ src, T* __restrict__ rho,
                                                      T* __restrict__ u, double* __restrict__ partials,
                                                      Geom G) {
  __shared__ double s[4][kThreads / 64];
  double acc[4] = {0, 0, 0, 0};
  const uint32_t stride = gridDim.x * kThreads;
  const uint32_t sz = stride / G.plane, sr = stride - sz * G.plane, sy = sr / (uint32_t)G.nx,
                 sx = sr - sy * (uint32_t)G.nx;
  uint32_t next = blockIdx.x * kThreads + threadIdx.x;
  uint32_t z = next / G.plane, y = (next - z * G.plane) / (uint32_t)G.nx,
           x = next - z * G.plane - y * (uint32_t)G.nx;
  T gn[19];
  if (next < G.N) pull_cell<T, FACES>(gn, src, G, next, x, y, z);
  while (next < G.N) {
    const uint32_t cell = next;
    T g[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) g[q] = gn[q];
    next += stride;
    x += sx;
    y += sy;
    z += sz;
    if (x >= (uint32_t)G.nx) {
      x -= (uint32_t)G.nx;
      ++y;
    }
    if (y >= (uint32_t)G.ny) {
      y -= (uint32_t)G.ny;
      ++z;
    }
    if (next < G.N) pull_cell<T, FACES>(gn, src, G, next, x, y, z);
    double drho = 0, m[3] = {0, 0, 0};
#pragma unroll
    for (int q = 0; q < 19; ++q) {
      drho += (double)g[q];
      if (CX[q]) m[0] += CX[q] * (double)g[q];
      if (CY[q]) m[1] += CY[q] * (double)g[q];
      if (CZ[q]) m[2] += CZ[q] * (double)g[q];
    }
    if (rho) rho[cell] = (T)(1.0 + drho);
    if (u) {
      const double r = 1.0 + drho;
      u[cell] = (T)(m[0] / r);
      u[G.N + cell] = (T)(m[1] / r);
      u[2 * (size_t)G.N + cell] = (T)(m[2] / r);
    }
    acc[0] += drho;
    acc[1] += m[0];
    acc[2] += m[1];
    acc[3] += m[2];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double v = wave_sum(acc[k]);
    if ((threadIdx.x & 63) == 0) s[k][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    double v = 0;
    for (int w = 0; w < kThreads / 64; ++w) v += s[threadIdx.x][w];
    partials[blockIdx.x * 4 + threadIdx.x] = v;
  }
}

// One block: fixed-order sum of the partials (deterministic), result[0] = N + sum drho. The kernel status
// goes behind the sums, so that the host reads both in one copy.
__global__ __launch_bounds__(kThreads) void k_reduce(const double* __restrict__ partials, int nblocks,
                                                     double ncells, const int32_t* __restrict__ status,
                                                     double* __restrict__ result) {
  __shared__ double s[4][kThreads / 64];
  double acc[4] = {0, 0, 0, 0};
  for (int b = threadIdx.x; b < nblocks; b += kThreads)
    for (int k = 0; k < 4; ++k) acc[k] += partials[b * 4 + k];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double v = wave_sum(acc[k]);
    if ((threadIdx.x & 63) == 0) s[k][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    double v = 0;
    for (int w = 0; w < kThreads / 64; ++w) v += s[threadIdx.x][w];
    result[threadIdx.x] = threadIdx.x == 0 ? ncells + v : v;
    if (threadIdx.x == 0) *reinterpret_cast<int32_t*>(result + 4) = *status;
  }
}

template <typename T, int FACES>
__global__ __launch_bounds__(kThreads) void k_populations(const T* __restrict__ src, T* __restrict__ out,
                                                          Geom G) {
  const uint32_t cell = blockIdx.x * kThreads + threadIdx.x;
  if (cell >= G.N) return;
  const uint32_t x = cell % G.nx, y = (cell / G.nx) % G.ny, z = cell / G.plane;
  T g[19];
  pull_cell<T, FACES>(g, src, G, cell, x, y, z);
  // exported in the plain (19, nz, ny, nx) order whatever the buffer layout, stored as a step stores
  if (G.stream1) {
    keep_branch();
#pragma unroll
    for (int q = 0; q < 19; ++q) __builtin_nontemporal_store(g[q], &out[(size_t)q * G.N + cell]);
    keep_branch();
  } else {
#pragma unroll
    for (int q = 0; q < 19; ++q) out[(size_t)q * G.N + cell] = g[q];
  }
}

__global__ __launch_bounds__(kThreads) void k_fill(uint32_t* __restrict__ p, size_t words) {
  const size_t stride = (size_t)gridDim.x * kThreads;
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < words; i += stride) p[i] = 0u;
}

__global__ void k_fill_bytes(uint8_t* __restrict__ p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

template <typename T, int FACES>
hipError_t moments_typed(lbm_ctx* c, void* rho, void* u) {
  const uint32_t blocks = c->nred;
  c->bins_clean = false;
  hipLaunchKernelGGL((k_moments<T, FACES>), dim3(blocks), dim3(kThreads), 0, c->stream,
                     static_cast<const T*>(c->pops[c->hs.cur]), static_cast<T*>(rho),
                     static_cast<T*>(u), c->partials, c->geom);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(kThreads), 0, c->stream, c->partials, (int)blocks,
                     (double)c->geom.N, c->status, c->result);
  return hipGetLastError();
}

template <typename T, int FACES>
hipError_t populations_typed(lbm_ctx* c, void* out) {
  // A copy of the state. Beyond the caches in the 5 workgroups per compute unit the FP32 liquid step runs with
  // (128 x 128 x 512 FP32 209 us, 6.1 TB/s, 224 us uncapped, 206 us in 3, but 330 us with periodic axes along y and
  // z; FP64 441, 447 and 429 us, 447, 474 and 466 us); uncapped where it fits in them (64 x 64 x 192 with such
  // axes 17.5 us, 19.5 in 5).
  hipLaunchKernelGGL((k_populations<T, FACES>), dim3(div_up(c->geom.N, kThreads)), dim3(kThreads),
                     c->geom.stream1 ? occupancy_lds(c->lds_per_cu, 5) : 0, c->stream,
                     static_cast<const T*>(c->pops[c->hs.cur]), static_cast<T*>(out), c->geom);
  return hipGetLastError();
}

// Periodic axes and states of 4 GiB and more take the general pull.
int pull_faces(const lbm_ctx* c) {
  if (c->periodic || !bb_fast_ok(c->geom, c->elem)) return FACES_GENERAL;
  return c->general ? FACES_WALLS : FACES_BB;
}

}  // namespace

hipError_t launch_moments(lbm_ctx* c, void* rho, void* u, bool) {
  switch (pull_faces(c)) {
    case FACES_BB:
      return c->elem == 4 ? moments_typed<float, FACES_BB>(c, rho, u) : moments_typed<double, FACES_BB>(c, rho, u);
    case FACES_WALLS:
      return c->elem == 4 ? moments_typed<float, FACES_WALLS>(c, rho, u)
                          : moments_typed<double, FACES_WALLS>(c, rho, u);
    default:
      return c->elem == 4 ? moments_typed<float, FACES_GENERAL>(c, rho, u)
                          : moments_typed<double, FACES_GENERAL>(c, rho, u);
  }
}

hipError_t launch_populations(lbm_ctx* c, void* out) {
  switch (pull_faces(c)) {
    case FACES_BB:
      return c->elem == 4 ? populations_typed<float, FACES_BB>(c, out) : populations_typed<double, FACES_BB>(c, out);
    case FACES_WALLS:
      return c->elem == 4 ? populations_typed<float, FACES_WALLS>(c, out)
                          : populations_typed<double, FACES_WALLS>(c, out);
    default:
      return c->elem == 4 ? populations_typed<float, FACES_GENERAL>(c, out)
                          : populations_typed<double, FACES_GENERAL>(c, out);
  }
}

hipError_t launch_fill(void* ptr, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  const size_t words = bytes / 4;
  if (words) {
    size_t blocks = (words + kThreads - 1) / kThreads;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill, dim3((uint32_t)blocks), dim3(kThreads), 0, s,
                       static_cast<uint32_t*>(ptr), words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const size_t tail = bytes - words * 4;
  if (tail) {
    hipLaunchKernelGGL(k_fill_bytes, dim3(1), dim3(64), 0, s, static_cast<uint8_t*>(ptr) + words * 4,
                       tail);
    return hipGetLastError();
  }
  return hipSuccess;
}

}  // namespace lbm
