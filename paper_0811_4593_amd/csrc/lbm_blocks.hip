// lbm_blocks.hip -- several time steps per launch for small lattices.
//
// A lattice of a few ten thousand nodes is swept in less time than it takes
// to start and drain a kernel (4-6 us a step), so what counts is the steps a
// launch makes.  Here a workgroup owns a block of bx x by x bz nodes and makes
// STEPS steps of it without any exchange with the others: step t is computed
// on the block and STEPS - t nodes around it, the first from HBM (through L2),
// the later ones from LDS, and only the last is written back.  The nodes
// around the blocks are computed by several workgroups, 1.8 (bars) to 4.1
// (cubes) times the updates in all, on compute units that would stand idle.  The arithmetic of
// every node is the single sweep's, so the state is the same bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "d3q19.hpp"
#include "lbm_internal.hpp"
#include "node_update.hpp"

namespace lbm {

namespace {

template <class T>
struct BlockArgs {
  int nx, ny, nz;
  size_t pop_stride, row_stride;  // PopLayout
  int blocks_x, blocks_y;
  unsigned step;
  NodeParams<T> p;
};

// A block of BX x BY x BZ nodes; step t of STEPS is computed on the block and
// STEPS - t nodes around it.
template <int STEPS, int BX, int BY, int BZ>
struct Block {
  static constexpr int kSteps = STEPS, kBX = BX, kBY = BY, kBZ = BZ;
  static constexpr int cells(int t) {
    return (BX + 2 * (STEPS - t)) * (BY + 2 * (STEPS - t)) * (BZ + 2 * (STEPS - t));
  }
  static constexpr int kThreads = cells(1) <= 1024 ? (cells(1) + 63) / 64 * 64 : 1024;
  // LDS elements: the populations of step 1's cells and, for three steps, of
  // step 2's.
  static_assert(STEPS == 2 || STEPS == 3, "the steps block_steps_kernel makes");
  static constexpr int kElements = 19 * (cells(1) + (STEPS > 2 ? cells(2) : 0));
};

// i wrapped into [0, n) for -n <= i < 2 n.
__device__ __forceinline__ int wrapped(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// Step t of the block at (ox, oy, oz): from HBM (t = 1) or the previous step's
// cells in LDS (prev), to LDS (next) or HBM (t = STEPS).
template <class F, class B, int t>
__device__ __forceinline__ void block_step(const typename F::S *__restrict__ src, typename F::S *__restrict__ dst,
                                           const BlockArgs<typename Codec<typename F::S>::T> &a,
                                           int ox, int oy, int oz, const typename F::S *prev, typename F::S *next) {
  using S = typename F::S;
  using T = typename Codec<S>::T;
  constexpr int h = B::kSteps - t;
  constexpr int ex = B::kBX + 2 * h, ey = B::kBY + 2 * h, cells = B::cells(t);
  constexpr int px = ex + 2, py = ey + 2, pcells = t > 1 ? B::cells(t > 1 ? t - 1 : 1) : 0;
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  for (unsigned i = threadIdx.x; i < unsigned(cells); i += unsigned(B::kThreads)) {
    const unsigned r = i / unsigned(ex), lx = i - r * unsigned(ex), lz = r / unsigned(ey), ly = r - lz * unsigned(ey);
    const int gx = ox - h + int(lx), gy = oy - h + int(ly), gz = oz - h + int(lz);
    // Nothing is read beyond a bounded face, nor beyond the last block's part
    // of a periodic axis by more than h nodes.
    const bool out = ((a.p.bc_mask & 1u) && (gx < 0 || gx >= nx)) || ((a.p.bc_mask & 4u) && (gy < 0 || gy >= ny)) ||
                     ((a.p.bc_mask & 16u) && (gz < 0 || gz >= nz)) || gx >= nx + h || gy >= ny + h || gz >= nz + h;
    if (out) continue;
    const int x = wrapped(gx, nx), y = wrapped(gy, ny), z = wrapped(gz, nz);
    T f[19];
    if constexpr (t == 1) {
      const unsigned xs[3] = {x == nx - 1 ? 0u : unsigned(x) + 1u, unsigned(x), x == 0 ? unsigned(nx) - 1u : unsigned(x) - 1u};
      const unsigned ys[3] = {y == ny - 1 ? 0u : unsigned(y) + 1u, unsigned(y), y == 0 ? unsigned(ny) - 1u : unsigned(y) - 1u};
      const unsigned zs[3] = {z == nz - 1 ? 0u : unsigned(z) + 1u, unsigned(z), z == 0 ? unsigned(nz) - 1u : unsigned(z) - 1u};
      S raw[19];
#pragma unroll
      for (int k = 0; k < 19; ++k)
        raw[k] = src[size_t(k) * a.pop_stride + size_t(ys[cy(k) + 1] + unsigned(ny) * zs[cz(k) + 1]) * a.row_stride +
                     xs[cx(k) + 1]];
#pragma unroll
      for (int k = 0; k < 19; ++k) f[k] = Codec<S>::load(raw[k]);
    } else {
      // the previous step's cells reach one node further on every side
      const S *from = prev + (lz * unsigned(py) + ly) * unsigned(px) + lx;
#pragma unroll
      for (int k = 0; k < 19; ++k)
        f[k] = Codec<S>::load(from[k * pcells + ((1 - cz(k)) * py + 1 - cy(k)) * px + 1 - cx(k)]);
    }
    unsigned m = 0;
    if (x == 0) m |= a.p.bc_mask & 1u;
    if (x == nx - 1) m |= a.p.bc_mask & 2u;
    if (y == 0) m |= a.p.bc_mask & 4u;
    if (y == ny - 1) m |= a.p.bc_mask & 8u;
    if (z == 0) m |= a.p.bc_mask & 16u;
    if (z == nz - 1) m |= a.p.bc_mask & 32u;
    if (__builtin_amdgcn_ballot_w64(m != 0u))
      box_boundary_rule<T>(f, m, a.p);
    bgk_collide<T>(f, a.p.omega, a.p.tau_f);
    const unsigned row = unsigned(z) * unsigned(ny) + unsigned(y);
    const unsigned r0 = F::kStochastic ? fmix32((row * unsigned(nx) + unsigned(x)) * 0x9e3779b1u + step_key(a.step + unsigned(t - 1))) : 0u;
    S e[19];
#pragma unroll
    for (int k = 0; k < 19; ++k) e[k] = store_form<F>(f[k], r0 + unsigned(k + 1) * 0x9e3779b9u);
    complete(e);
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      if constexpr (t < B::kSteps)
        next[k * cells + int(i)] = e[k];
      else
        dst[size_t(k) * a.pop_stride + size_t(row) * a.row_stride + unsigned(x)] = e[k];
    }
  }
}

template <class F, class B>
__global__ __launch_bounds__(B::kThreads) void block_steps_kernel(const typename F::S *__restrict__ src,
                                                                  typename F::S *__restrict__ dst,
                                                                  BlockArgs<typename Codec<typename F::S>::T> a) {
  using S = typename F::S;
  __shared__ S cells[B::kElements];
  const unsigned b = blockIdx.x, bx = b % unsigned(a.blocks_x), r = b / unsigned(a.blocks_x);
  const int ox = int(bx) * B::kBX, oy = int(r % unsigned(a.blocks_y)) * B::kBY, oz = int(r / unsigned(a.blocks_y)) * B::kBZ;
  S *const one = cells, *const two = cells + 19 * B::cells(1);
  block_step<F, B, 1>(src, dst, a, ox, oy, oz, nullptr, one);
  __syncthreads();
  block_step<F, B, 2>(src, dst, a, ox, oy, oz, one, two);
  if constexpr (B::kSteps == 3) {
    __syncthreads();
    block_step<F, B, 3>(src, dst, a, ox, oy, oz, two, nullptr);
  }
}

template <class F, class B>
hipError_t launch_t(const SweepConfig &c, const void *src, void *dst, hipStream_t s) {
  using S = typename F::S;
  using T = typename Codec<S>::T;
  static_assert(B::kElements * sizeof(S) <= 159 * 1024, "LDS of a workgroup");
  BlockArgs<T> a;
  a.nx = c.nx;
  a.ny = c.ny;
  a.nz = c.nz;
  a.pop_stride = c.layout.pop_stride;
  a.row_stride = c.layout.row_stride;
  a.blocks_x = (c.nx + B::kBX - 1) / B::kBX;
  a.blocks_y = (c.ny + B::kBY - 1) / B::kBY;
  const unsigned blocks = unsigned(a.blocks_x) * unsigned(a.blocks_y) * unsigned((c.nz + B::kBZ - 1) / B::kBZ);
  a.step = c.step;
  a.p.bc_mask = c.bc_mask;
  a.p.p_mask = c.p_mask;
  a.p.rule_flags = c.rule_flags;
  a.p.omega = T(1.0 / c.tau);
  for (int d = 0; d < 3; ++d) a.p.tau_f[d] = unit<T>() * T(c.tau * c.force[d]);
  for (int f = 0; f < 6; ++f) a.p.rho_p[f] = unit<T>() * T(c.rho_p[f]);
  for (int f = 0; f < 6; ++f)
    for (int d = 0; d < 3; ++d) a.p.fv.v[f][d] = T(c.v[f][d]);
  set_face_divisors<T>(a.p);
  block_steps_kernel<F, B><<<dim3(blocks), dim3(B::kThreads), 0, s>>>(static_cast<const S *>(src), static_cast<S *>(dst), a);
  return hipGetLastError();
}

using Cube = Block<3, 4, 4, 4>;
using Bar = Block<2, 16, 4, 4>;

template <class B>
size_t blocks_of(const SweepConfig &c) {
  return size_t((c.nx + B::kBX - 1) / B::kBX) * size_t((c.ny + B::kBY - 1) / B::kBY) *
         size_t((c.nz + B::kBZ - 1) / B::kBZ);
}

}  // namespace

// Cubes of three steps while there is a compute unit for each (up to about
// 16000 nodes with 256 units), then bars of two steps (up to about 65000):
// measured per step, single sweeps and so: 16 x 16 x 32 FP64 4.9 / 3.1 us, FP32 5.3 / 2.7;
// 16^3 FP32 duct 5.7 / 3.4; 32^3 FP32 5.9 / 4.7; 64 x 32 x 32 FP32 5.9 / 5.6.
// A second round of workgroups costs more than it saves (cubes on 32^3: 5.5
// us, on 64 x 32 x 32: 8.5).
int block_steps(const SweepConfig &c, int compute_units) {
  if (c.nx < 3 || c.ny < 3 || c.nz < 3) return 0;  // wrapped() goes once around
  if (blocks_of<Cube>(c) <= size_t(compute_units)) return Cube::kSteps;
  if (blocks_of<Bar>(c) <= size_t(compute_units)) return Bar::kSteps;
  return 0;
}

hipError_t launch_block_steps(const SweepConfig &c, int steps, const void *src, void *dst, hipStream_t s) {
  if (c.nx < 3 || c.ny < 3 || c.nz < 3) return hipErrorInvalidValue;
#define LBM_CASE(ST, F)                                                \
  case ST:                                                             \
    if (steps == Cube::kSteps) return launch_t<F, Cube>(c, src, dst, s); \
    if (steps == Bar::kSteps) return launch_t<F, Bar>(c, src, dst, s);   \
    break;
  switch (c.storage) {
    LBM_CASE(kStoreF64, FormF64)
    LBM_CASE(kStoreF32, FormF32)
    LBM_CASE(kStoreF16, FormF16)
    LBM_CASE(kStoreF16SR, FormF16SR)
  }
#undef LBM_CASE
  return hipErrorInvalidValue;
}

}  // namespace lbm
