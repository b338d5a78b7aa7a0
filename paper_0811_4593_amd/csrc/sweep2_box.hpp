// sweep2_box.hpp -- the two-steps-per-pass update of one workgroup's box
// (tile and z range) for lattices in the row-major layout, shared by the
// single-lattice kernel and the multi-lattice (batch) kernel, so that a
// lattice gets the same bits whichever kernel advances it.
//
// A workgroup owns a tile of 64 x BYI nodes in x and y and a range of
// z-planes, and streams along z: at each plane it first computes step 1 on
// the tile plus a one-node halo in x and y (pulling from HBM, halo nodes
// wrapped as the single sweep wraps its sources), keeps the results in LDS,
// and then computes step 2 on the tile's interior from LDS and writes it to
// HBM.  The arithmetic of every node is the single sweep's (the same
// boundary rules, collision, rounding and random words), so the state after
// the pass equals the state after two single sweeps bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

#include "d3q19.hpp"
#include "node_update.hpp"

namespace lbm {

// The thread that computes step 1 of the node (x, y) also computes its step
// 2, so the three populations that move along z or not at all (cx = cy = 0)
// stay in its registers.  The 16 others pass through LDS: step 2 at plane z
// pulls population k from plane z - cz(k) of step 1, so a step-1 plane's
// populations with cz = -1 are read by step 2 in the same round, those with
// cz = 0 one round later and those with cz = +1 two rounds later: rings of
// 1, 2 and 3 slots, 4 + 2 * 8 + 3 * 4 = 32 population planes in all.
__host__ __device__ constexpr bool own_column(int k) { return cx(k) == 0 && cy(k) == 0; }
__host__ __device__ constexpr int ring_depth(int k) { return cz(k) < 0 ? 1 : (cz(k) == 0 ? 2 : 3); }
// Rank of population k among those of its cz that pass through LDS.
__host__ __device__ constexpr int ring_rank(int k) {
  int r = 0;
  for (int j = 0; j < k; ++j) r += (!own_column(j) && cz(j) == cz(k)) ? 1 : 0;
  return r;
}
// First plane of each ring, and planes of one of its slots.
__host__ __device__ constexpr int ring_first(int c) { return c < 0 ? 0 : (c == 0 ? 4 : 20); }
__host__ __device__ constexpr int ring_slot_planes(int c) { return c == 0 ? 8 : 4; }
constexpr int kRingPlanes = 32;
static_assert(ring_rank(17) == 3 && ring_rank(11) == 7 && ring_rank(16) == 3, "4, 8 and 4 populations per slot");

template <class T>
struct Sweep2Args {
  int nx, ny, nz;
  size_t pop_stride, row_stride;  // row-major: R and 19 R
  int tiles_x, tiles_y, zc;       // tile grid (64 x BYI tiles) and planes per z range
  int xcd_remap;                  // LBM_XCD_SLABS or dispatch order
  unsigned key0, key1;            // step keys of the two steps (stochastic rounding)
  NodeParams<T> p;
};

// Faces of the bounded box the node (x, y, z) lies on (bit f: face f).
__device__ __forceinline__ unsigned box_faces(unsigned bc_mask, int x, int y, int z, int nx, int ny, int nz) {
  unsigned m = 0;
  if (x == 0) m |= bc_mask & 1u;
  if (x == nx - 1) m |= bc_mask & 2u;
  if (y == 0) m |= bc_mask & 4u;
  if (y == ny - 1) m |= bc_mask & 8u;
  if (z == 0) m |= bc_mask & 16u;
  if (z == nz - 1) m |= bc_mask & 32u;
  return m;
}

template <class F, int BYI>
struct Sweep2Tile {
  static constexpr int kHX = 66;                 // 64 interior columns + halo
  static constexpr int kHY = BYI + 2;            // BYI interior rows + halo
  static constexpr int kPlane = kHX * kHY;       // elements of one population plane
  static constexpr int kThreads = 64 * (BYI + 3);  // a wave per halo row and one for the halo columns
  // Waves per SIMD the register allocation has to leave room for: one
  // workgroup per compute unit, two of the small tiles (8 waves).
  static constexpr int kWaves = BYI <= 5 ? 4 : (BYI + 3 + 3) / 4;
};

// Every load issued so far has returned (vmcnt 0; gfx9 encoding with the
// other counters at their maxima).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }

// The two steps of one workgroup's box: tile (tx, ty) of 64 x BYI nodes and
// z range tz of a.zc planes, with the population ring `ring` in LDS
// (kRingPlanes * Sweep2Tile<F, BYI>::kPlane elements).  Every thread of the
// workgroup calls it (it holds barriers).
//
// Waves 0..BYI+1 each own a row of the tile and its halo, 64 columns; the
// last wave owns the halo columns left and right of every row.  A round
// (one z plane) of a wave: take the 19 loaded sources of its node, issue the
// loads of the next plane's, compute step 1 and write it to the ring;
// barrier; step 2 of its node one plane behind from the ring and its own
// registers; wait for the loads; store; barrier.  The loads so have the
// whole round to arrive, beneath both steps' arithmetic, and the wait, placed
// before the stores, never waits for a store (loads and stores share one
// counter that drains in order).  With one workgroup per compute unit a pass
// that loads, waits, computes and stores in turn leaves memory idle through
// the arithmetic and the other way round: without any arithmetic it still
// took 8.9 ms on the 1024 x 512 x 512 FP32 duct, with it 11.1 ms, this way
// 8.5-9.0 ms by the allocation (9.1-9.6 TB/s at the algorithmic 152 B per
// update; without arithmetic 8.1 ms).  512 x 256 x 256 FP64: 2.87 ms, 2.19 ms
// with the loads ahead and 7 rows (5 rows 2.38 ms, 6 rows 2.17-2.23 ms),
// 2.0-2.1 ms with one descriptor per plane and the shorter boundary rules.
//
// Every wave keeps to one row, so that its loads and stores are whole cache
// lines of it.  Lanes dealt to tiles of any width instead (rows of 200 nodes
// leave 22% of these idle) took 252 us per step against 188 on 300 x 150 x
// 200 FP32, 59 against 55 on 200 x 100 x 100: lines written in parts.
template <class F, int BYI>
__device__ __forceinline__ void sweep2_box(global_ptr<const typename F::S> src, global_ptr<typename F::S> dst,
                                           const Sweep2Args<typename Codec<typename F::S>::T> &a, unsigned tx,
                                           unsigned ty, unsigned tz, typename F::S *ring) {
  using S = typename F::S;
  using T = typename Codec<S>::T;
  using Tile = Sweep2Tile<F, BYI>;
  constexpr int HX = Tile::kHX, HY = Tile::kHY, PLANE = Tile::kPlane;
  __shared__ FaceVals<T> faces[6];
#pragma unroll
  for (unsigned f = 0; f < 6u; ++f)
    if (threadIdx.x == f)
      faces[f] = FaceVals<T>{{a.p.fv.v[f][0], a.p.fv.v[f][1], a.p.fv.v[f][2]}, a.p.rho_p[f], a.p.den[f], a.p.inv[f]};
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int x0 = int(tx) * 64, y0 = int(ty) * BYI, zb = int(tz) * a.zc;
  const int ze = min(zb + a.zc, nz);
  const int w = min(64, nx - x0), hyc = min(BYI, ny - y0);  // interior columns and rows of this tile
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int lane = int(threadIdx.x) & 63;
  const bool columns = wave == HY;
  // This lane's node: cell (hx, hy) of the tile with halo, lattice column x
  // and row y (halo nodes wrapped, as the single sweep's pull reads them;
  // idle lanes take a node of the tile).
  const bool live1 = columns ? lane < 2 * (hyc + 2) : lane < w;
  const int hy = columns ? min(lane >> 1, hyc + 1) : min(wave, hyc + 1);
  const int hx = columns ? ((lane & 1) ? w + 1 : 0) : min(lane + 1, w);
  int x = x0 + hx - 1, y = y0 + hy - 1;
  x += x < 0 ? nx : (x >= nx ? -nx : 0);
  y += y < 0 ? ny : (y >= ny ? -ny : 0);
  const bool rows1 = columns || wave <= hyc + 1;              // the wave has step-1 nodes
  const bool rows2 = !columns && wave >= 1 && wave <= hyc;  // and step-2 nodes
  const unsigned mxy = box_faces(a.p.bc_mask & 15u, x, y, -1, nx, ny, nz);
  const unsigned nxy = unsigned(y) * unsigned(nx) + unsigned(x);
  const unsigned nplane = unsigned(nx) * unsigned(ny);
  // Sources and destination of the lane's node.  A z plane's bytes fit 32
  // bits: one descriptor per plane (base at the plane's start, advanced from
  // round to round), the lane's offset within the plane for each of the nine
  // (cx, cy), and the population's start as scalar offset -- nothing per load
  // is recomputed in the loop, and the halo-column wave, whose rows differ by
  // lane, runs the same code.
  const unsigned rb = unsigned(a.row_stride) * unsigned(sizeof(S)), pb = unsigned(a.pop_stride) * unsigned(sizeof(S));
  const size_t zbytes = size_t(rb) * size_t(ny);
  unsigned off[3][3];  // [cy + 1][cx + 1]
  {
    const unsigned xs[3] = {x == nx - 1 ? 0u : unsigned(x) + 1u, unsigned(x), x == 0 ? unsigned(nx) - 1u : unsigned(x) - 1u};
    const unsigned ys[3] = {y == ny - 1 ? 0u : unsigned(y) + 1u, unsigned(y), y == 0 ? unsigned(ny) - 1u : unsigned(y) - 1u};
#pragma unroll
    for (int cyi = 0; cyi < 3; ++cyi)
#pragma unroll
      for (int cxi = 0; cxi < 3; ++cxi) off[cyi][cxi] = ys[cyi] * rb + xs[cxi] * unsigned(sizeof(S));
  }
  const char *const in = (const char *)(const S *)src, *const out = (const char *)(S *)dst;
  const char *plane[3];  // sources of the plane being loaded, index cz + 1: planes z + 1, z, z - 1
  S raw[19];
  // bytes: the plane's, or 0 to read nothing
  auto load = [&](unsigned bytes) {
#pragma unroll
    for (int k = 0; k < 19; ++k)
      raw[k] = buf_load<S>(raw_buffer(plane[cz(k) + 1], bytes), off[cy(k) + 1][cx(k) + 1], unsigned(k) * pb);
  };

  // LDS cells: `out` the lane's own cell, `in` the lowest cell step 2 reads.
  S *const own = ring + hy * HX + hx;
  const S *const low = own - HX - 1;
  S e18 = S(0), e4 = S(0), e4_before = S(0), e5 = S(0);  // own column: rest, +z (one and two rounds back), -z
  __syncthreads();  // the face table
  int zp = zb;  // the plane of plane[0], one above the one being loaded
  const int zm = zb == 0 ? nz - 1 : zb - 1;
  plane[2] = in + size_t(zm == 0 ? nz - 1 : zm - 1) * zbytes;
  plane[1] = in + size_t(zm) * zbytes;
  plane[0] = in + size_t(zp) * zbytes;
  const char *out_plane = out + size_t(zb) * zbytes;
  load(unsigned(zbytes));
  wait_loads();
  int s2 = 0, s3 = 0;  // ring slots of this round: p mod 2, p mod 3
  for (int zz = zb - 1; zz <= ze; ++zz) {
    const int z1 = zz < 0 ? zz + nz : (zz >= nz ? zz - nz : zz);
    const int s3_2 = s3 == 2 ? 0 : s3 + 1;  // slot of two rounds back (p - 2 = p + 1 mod 3)
    T f[19];
#pragma unroll
    for (int k = 0; k < 19; ++k) f[k] = Codec<S>::load(raw[k]);
    complete(f);
    zp = zp == nz - 1 ? 0 : zp + 1;
    plane[2] = plane[1];
    plane[1] = plane[0];
    plane[0] = zp == 0 ? in : plane[0] + zbytes;
    load(zz < ze ? unsigned(zbytes) : 0u);
    S e18_now = S(0), e4_now = S(0);
    if (rows1) {
      const unsigned m = mxy | (z1 == 0 ? a.p.bc_mask & 16u : 0u) | (z1 == nz - 1 ? a.p.bc_mask & 32u : 0u);
      if (__builtin_amdgcn_ballot_w64(m != 0u))
        box_boundary_rule_table<T>(f, m, a.p.p_mask, a.p.rule_flags, faces);
      bgk_collide<T>(f, a.p.omega, a.p.tau_f);
      const unsigned r0 = F::kStochastic ? fmix32((nxy + unsigned(z1) * nplane) * 0x9e3779b1u + a.key0) : 0u;
      S e[19];
#pragma unroll
      for (int k = 0; k < 19; ++k) e[k] = store_form<F>(f[k], r0 + unsigned(k + 1) * 0x9e3779b9u);
      complete(e);
      if (live1) {
#pragma unroll
        for (int k = 0; k < 19; ++k) {
          if (own_column(k)) continue;
          const int slot = cz(k) < 0 ? 0 : (cz(k) == 0 ? s2 : s3);
          (own + slot * ring_slot_planes(cz(k)) * PLANE)[(ring_first(cz(k)) + ring_rank(k)) * PLANE] = e[k];
        }
      }
      e18_now = e[18];
      e4_now = e[4];
      e5 = e[5];
    }
    __syncthreads();
    // Step 2 on the interior of plane zz - 1.
    if (rows2 && zz > zb) {
      const int z2 = zz - 1;
      T f[19];
#pragma unroll
      for (int k = 0; k < 19; ++k) {
        if (own_column(k)) {
          f[k] = Codec<S>::load(k == 18 ? e18 : (k == 4 ? e4_before : e5));
          continue;
        }
        const int slot = cz(k) < 0 ? 0 : (cz(k) == 0 ? 1 - s2 : s3_2);
        f[k] = Codec<S>::load((low + slot * ring_slot_planes(cz(k)) * PLANE)[
            (ring_first(cz(k)) + ring_rank(k)) * PLANE + (1 - cy(k)) * HX + (1 - cx(k))]);
      }
      const unsigned m = mxy | (z2 == 0 ? a.p.bc_mask & 16u : 0u) | (z2 == nz - 1 ? a.p.bc_mask & 32u : 0u);
      if (__builtin_amdgcn_ballot_w64(m != 0u))
        box_boundary_rule_table<T>(f, m, a.p.p_mask, a.p.rule_flags, faces);
      bgk_collide<T>(f, a.p.omega, a.p.tau_f);
      const unsigned r0 = F::kStochastic ? fmix32((nxy + unsigned(z2) * nplane) * 0x9e3779b1u + a.key1) : 0u;
      S e[19];
#pragma unroll
      for (int k = 0; k < 19; ++k) e[k] = store_form<F>(f[k], r0 + unsigned(k + 1) * 0x9e3779b9u);
      complete(e);
      wait_loads();
      if (live1) {
        const auto to = raw_buffer(out_plane, unsigned(zbytes));
#pragma unroll
        for (int k = 0; k < 19; ++k) buf_store_nt<S>(e[k], to, off[1][1], unsigned(k) * pb);
      }
      out_plane += zbytes;
    } else {
      wait_loads();
    }
    e18 = e18_now;
    e4_before = e4;
    e4 = e4_now;
    s2 = 1 - s2;
    s3 = s3 == 2 ? 0 : s3 + 1;
    __syncthreads();
  }
}

// Interior rows per tile of each storage form.  LDS holds 32 population
// planes of 66 x (BYI + 2) elements: 127 KB for FP32 with BYI = 13 (one
// workgroup of 16 waves per compute unit, the most a workgroup can have;
// step 1 then costs 1.2 times the updates it feeds), 152 KB for FP64 with
// BYI = 7 (the most that fits), 63 KB for FP16 with BYI = 13.
template <class F>
struct Sweep2Rows;
template <>
struct Sweep2Rows<FormF64> {
  static constexpr int kBYI = 7;
};
template <>
struct Sweep2Rows<FormF32> {
  static constexpr int kBYI = 13;
};
template <>
struct Sweep2Rows<FormF16> {
  static constexpr int kBYI = 13;
};
template <>
struct Sweep2Rows<FormF16SR> {
  static constexpr int kBYI = 13;
};

}  // namespace lbm
