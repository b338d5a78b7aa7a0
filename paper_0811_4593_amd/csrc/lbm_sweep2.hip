// lbm_sweep2.hip -- two time steps per pass over HBM (temporal blocking) for
// lattices in the row-major layout.
//
// The single sweep reads and writes every population once per step, so at
// the HBM bandwidth it can do no better than a copy.  Here a workgroup owns a
// tile of 64 x BYI nodes in x and y and a range of z-planes, and streams
// along z: at each plane it first computes step 1 on the tile plus a
// one-node halo in x and y (pulling from HBM, halo nodes wrapped as the
// single sweep wraps its sources), keeps the results in LDS, and then
// computes step 2 on the tile's interior from LDS and writes it to HBM.  Per
// node and two steps it reads the 19 populations once (plus the halo, shared
// with the neighbouring tiles through L2) and writes them once: about half
// the bytes of two single sweeps.  The arithmetic of every node is the single
// sweep's (the same boundary rules, collision, rounding and random words), so
// the state after the pass equals the state after two single sweeps bit for
// bit.  The update of one workgroup's box is sweep2_box (sweep2_box.hpp),
// which the batch runtime's multi-lattice pass calls as well.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "d3q19.hpp"
#include "lbm_internal.hpp"
#include "node_update.hpp"
#include "sweep2_box.hpp"

namespace lbm {

template <class F, int BYI>
__global__ __launch_bounds__((Sweep2Tile<F, BYI>::kThreads), (Sweep2Tile<F, BYI>::kWaves)) void sweep2_kernel(
    const typename F::S *__restrict__ src, typename F::S *__restrict__ dst,
    Sweep2Args<typename Codec<typename F::S>::T> a) {
  using S = typename F::S;
  __shared__ S ring[kRingPlanes * Sweep2Tile<F, BYI>::kPlane];
  const unsigned b = logical_block(blockIdx.x, gridDim.x, a.xcd_remap, 1u);
  const unsigned tx = b % unsigned(a.tiles_x), rest = b / unsigned(a.tiles_x);
  const unsigned ty = rest % unsigned(a.tiles_y), tz = rest / unsigned(a.tiles_y);
  sweep2_box<F, BYI>((global_ptr<const S>)src, (global_ptr<S>)dst, a, tx, ty, tz, ring);
}

template <class F, int BYI>
static hipError_t launch_sweep2_t(const SweepConfig &c, int zc, const void *src, void *dst, hipStream_t s) {
  using S = typename F::S;
  using T = typename Codec<S>::T;
  Sweep2Args<T> a;
  a.nx = c.nx;
  a.ny = c.ny;
  a.nz = c.nz;
  a.pop_stride = c.layout.pop_stride;
  a.row_stride = c.layout.row_stride;
  a.tiles_x = (c.nx + 63) / 64;
  a.tiles_y = (c.ny + BYI - 1) / BYI;
  a.zc = zc;
  a.xcd_remap = c.xcd_remap == 1 ? 1 : 0;
  a.key0 = step_key(c.step);
  a.key1 = step_key(c.step + 1u);
  a.p.bc_mask = c.bc_mask;
  a.p.p_mask = c.p_mask;
  a.p.rule_flags = c.rule_flags;
  a.p.omega = T(1.0 / c.tau);
  for (int d = 0; d < 3; ++d) a.p.tau_f[d] = unit<T>() * T(c.tau * c.force[d]);
  for (int f = 0; f < 6; ++f) a.p.rho_p[f] = unit<T>() * T(c.rho_p[f]);
  for (int f = 0; f < 6; ++f)
    for (int d = 0; d < 3; ++d) a.p.fv.v[f][d] = T(c.v[f][d]);
  set_face_divisors<T>(a.p);
  const size_t tiles_z = (size_t(c.nz) + size_t(zc) - 1) / size_t(zc);
  const size_t nblocks = size_t(a.tiles_x) * size_t(a.tiles_y) * tiles_z;
  if (nblocks == 0 || nblocks > 0x7fffffffu) return hipErrorInvalidValue;
  sweep2_kernel<F, BYI><<<dim3(unsigned(nblocks)), dim3(Sweep2Tile<F, BYI>::kThreads), 0, s>>>(
      static_cast<const S *>(src), static_cast<S *>(dst), a);
  return hipGetLastError();
}

// Row-major, with planes below 4 GiB: the pass addresses a plane by 32-bit
// offsets within one buffer descriptor.  Larger planes (28 million FP64 or 56
// million FP32 nodes each) take the single sweep.
bool sweep2_takes(const PopLayout &lay, int ny, int storage) {
  const size_t esize = storage == kStoreF64 ? 8 : (storage == kStoreF32 ? 4 : 2);
  return lay.row_stride == 19 * lay.pop_stride && lay.row_stride * esize * size_t(ny) < (size_t(1) << 32);
}

int sweep2_rows(int storage, int tile_rows) {
  switch (storage) {
    case kStoreF64: return Sweep2Rows<FormF64>::kBYI;
    case kStoreF32: return tile_rows ? tile_rows : Sweep2Rows<FormF32>::kBYI;
    case kStoreF16: return tile_rows ? tile_rows : Sweep2Rows<FormF16>::kBYI;
    default: return tile_rows ? tile_rows : Sweep2Rows<FormF16SR>::kBYI;
  }
}

// Time of a pass, from what a round takes (one z plane of a workgroup, every
// compute unit with its own or two small tiles): workgroups run in waves of
// `slots`, each zc + 2 rounds.  Measured rounds: FP32 6.3 us (1024 x 512 x
// 512) to 7.5 us (112^3, where every workgroup has boundary nodes), FP64 6.6,
// FP16 4.9, and 6 us for the launch.
PassPlan sweep2_plan(const SweepConfig &c, int rows, int compute_units) {
  const double round_us = c.storage == kStoreF64 ? 6.6 : (c.storage == kStoreF32 ? 7.0 : 4.9);
  const long slots = long(compute_units) * (rows == 5 ? 2 : 1);
  const int by = sweep2_rows(c.storage, rows);
  const long layer = long((c.nx + 63) / 64) * ((c.ny + by - 1) / by);
  PassPlan best{0, 0.0};
  const long first = c.nz > 4096 ? (c.nz + 31) / 32 : 1;  // a long axis: 32 planes
  for (long ranges = first; ranges <= c.nz; ++ranges) {
    const int zc = int((c.nz + ranges - 1) / ranges);
    // Longer ranges let neighbouring workgroups drift apart and fetch their
    // common lines twice (1024 x 512 x 512 FP32: 32 planes 8.4 ms, 64 8.8,
    // 128 9.0); shorter ones redo too many planes.
    if (zc > 96) continue;
    if (zc < 4) break;
    const long waves = (layer * ((c.nz + zc - 1) / zc) + slots - 1) / slots;
    const double us = double(waves) * (zc + 2) * round_us * (zc > 48 ? 1.05 : 1.0) + 6.0;
    if (best.zc == 0 || us < best.us) best = {zc, us};
    if (first > 1) break;
  }
  return best;
}

// The single sweep moves 2 * 19 elements per node at 5.5 to 6.0 TB/s.
int sweep2_pays(const SweepConfig &c, int compute_units) {
  if (!sweep2_takes(c.layout, c.ny, c.storage)) return 0;
  const double bytes = 38.0 * (c.storage == kStoreF64 ? 8 : (c.storage == kStoreF32 ? 4 : 2)) * c.nx * c.ny * c.nz;
  const double single_us = bytes / (c.storage == kStoreF64 ? 5.5e6 : (c.storage == kStoreF32 ? 5.6e6 : 6.0e6));
  const PassPlan p = sweep2_plan(c, 0, compute_units);
  return p.zc > 0 && p.us < 0.97 * 2.0 * single_us ? p.zc : 0;
}

hipError_t launch_sweep2(const SweepConfig &c, int zc, int rows, const void *src, void *dst, hipStream_t s) {
  if (!sweep2_takes(c.layout, c.ny, c.storage) || zc < 1) return hipErrorInvalidValue;
  switch (c.storage) {
    case kStoreF64: return launch_sweep2_t<FormF64, Sweep2Rows<FormF64>::kBYI>(c, zc, src, dst, s);
    case kStoreF32:
      if (rows == 5) return launch_sweep2_t<FormF32, 5>(c, zc, src, dst, s);
      if (rows == 12) return launch_sweep2_t<FormF32, 12>(c, zc, src, dst, s);
      return launch_sweep2_t<FormF32, Sweep2Rows<FormF32>::kBYI>(c, zc, src, dst, s);
    case kStoreF16:
      if (rows == 5) return launch_sweep2_t<FormF16, 5>(c, zc, src, dst, s);
      if (rows == 12) return launch_sweep2_t<FormF16, 12>(c, zc, src, dst, s);
      return launch_sweep2_t<FormF16, Sweep2Rows<FormF16>::kBYI>(c, zc, src, dst, s);
    case kStoreF16SR:
      if (rows == 5) return launch_sweep2_t<FormF16SR, 5>(c, zc, src, dst, s);
      if (rows == 12) return launch_sweep2_t<FormF16SR, 12>(c, zc, src, dst, s);
      return launch_sweep2_t<FormF16SR, Sweep2Rows<FormF16SR>::kBYI>(c, zc, src, dst, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm
