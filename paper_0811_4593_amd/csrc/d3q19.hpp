// d3q19.hpp -- D3Q19 lattice constants and the per-node rules of the sweep,
// as device functions for gfx950.
//
// Population k = i - 1 where i numbers the lattice vectors as the columns of
// the matrix M (Sec. II, eq_deffs); weights from eq_weights.  Every rule is a
// template over the boundary normals, so after unrolling all population
// indices and lattice-vector components are compile-time constants: the 19
// populations of a node live in registers and are never indexed at run time.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace lbm {

__host__ __device__ constexpr int cx(int k) {
  constexpr int t[19] = {1, -1, 0, 0, 0, 0, 1, 1, 1, 1, -1, -1, -1, -1, 0, 0, 0, 0, 0};
  return t[k];
}
__host__ __device__ constexpr int cy(int k) {
  constexpr int t[19] = {0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, 1, -1, -1, 0};
  return t[k];
}
__host__ __device__ constexpr int cz(int k) {
  constexpr int t[19] = {0, 0, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, -1, 1, -1, 1, -1, 0};
  return t[k];
}
// Weight numerators over 36 (eq_weights).
__host__ __device__ constexpr int w36(int k) { return k < 6 ? 2 : (k < 18 ? 1 : 12); }

__host__ __device__ constexpr int index_of(int x, int y, int z) {
  for (int k = 0; k < 19; ++k)
    if (cx(k) == x && cy(k) == y && cz(k) == z) return k;
  return -1;
}
__host__ __device__ constexpr int opp(int k) { return index_of(-cx(k), -cy(k), -cz(k)); }

template <class T>
__device__ __forceinline__ T weight(int k) {
  return T(w36(k)) / T(36);
}

// c_k . n for an integer vector n = (nx, ny, nz).
__host__ __device__ constexpr int dotn(int k, int nx, int ny, int nz) {
  return cx(k) * nx + cy(k) * ny + cz(k) * nz;
}

// Bit mask (bit k) of the populations whose streaming source lies outside the
// domain at a node on boundary face f: c_k . n_f > 0, n_f the inward normal
// of face f (x=0, x=nx-1, y=0, y=ny-1, z=0, z=nz-1).
__host__ __device__ constexpr int face_normal(int f, int axis) {
  return (f / 2 == axis) ? ((f % 2 == 0) ? 1 : -1) : 0;
}
__host__ __device__ constexpr unsigned unknown_mask(int f) {
  unsigned m = 0;
  for (int k = 0; k < 19; ++k)
    if (dotn(k, face_normal(f, 0), face_normal(f, 1), face_normal(f, 2)) > 0) m |= 1u << k;
  return m;
}

// Face velocities in the compute type, indexed by face id (x0,x1,y0,y1,z0,z1).
template <class T>
struct FaceVel {
  T v[6][3];
};

// a * b + c, rounded once.  The rules and the collision write their
// multiply-adds out and switch the compiler's own contraction off: which
// products it fuses depends on the code around a call, and every kernel that
// advances a lattice has to give the same bits.
__device__ __forceinline__ double fused_add(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fused_add(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// a / den with inv = 1 / den rounded to nearest: the quotient a * inv
// corrected once by its exact remainder is the rounded quotient (Markstein,
// IBM J. Res. Dev. 34(1), 1990), in three operations where the division takes
// about twelve, one after the other.  For finite a: of an infinite one it makes
// NaN where the division gives infinity.  No state shows that: a is infinite
// only where a population of the node is, then its density is too, and the
// collision makes NaN of every population of the node (1.5 rho u^2 = infinity
// times 0, or NaN) either way.
template <class T>
__device__ __forceinline__ T quotient(T a, T den, T inv) {
  const T q = a * inv;
  return fused_add(fused_add(-den, q, a), inv, q);
}

// Unit of the update's arithmetic: it works on unit<T>() times the
// deviations (and densities): 2^8 in float, the arithmetic of the FP16 forms,
// which store that number.
template <class T>
__host__ __device__ constexpr T unit() {
  return sizeof(T) == 4 ? T(256) : T(1);
}

// Per-lattice parameters of the node update.
template <class T>
struct NodeParams {
  unsigned bc_mask;  // bit f: face f is bounded (velocity or pressure BC)
  unsigned p_mask;   // bit f: face f is a pressure face (subset of bc_mask)
  T omega;           // 1 / tau
  T tau_f[3];        // tau * F: velocity shift times rho inside f^eq (body force F), in unit<T>()
  FaceVel<T> fv;     // velocity faces: the velocity; pressure faces: the
                     // tangential velocity (normal component zero)
  T rho_p[6];        // prescribed density of each pressure face, in unit<T>()
  T den[6], inv[6];  // divisor of the face's bracket, 1 - v.n (velocity face)
                     // or rho_p (pressure face), and its reciprocal
  unsigned rule_flags;  // kRuleNoTransverse: face rule without the corrections N
};

// Comparison variant of the face rule: non-equilibrium bounce-back of every
// unknown without the transverse corrections N (Sec. IV, eq_f9NoNs-eq_f17NoNs).
constexpr unsigned kRuleNoTransverse = 1u;

// Velocity (velocity face) or tangential velocity and density (pressure face)
// of the face a node with the single-face mask m lies on.
template <class T>
__device__ __forceinline__ void face_values(unsigned m, const NodeParams<T> &p, T &vx, T &vy, T &vz, T &r0) {
  vx = T(0);
  vy = T(0);
  vz = T(0);
  r0 = unit<T>();
#pragma unroll
  for (int b = 0; b < 6; ++b)
    if (m == (1u << b)) {
      vx = p.fv.v[b][0];
      vy = p.fv.v[b][1];
      vz = p.fv.v[b][2];
      r0 = p.rho_p[b];
    }
}

// ---------------------------------------------------------------------------
// All rules below act on deviations d_k = f_k - w_k from the rest state.
// Opposite populations have equal weights and the weights of any set of
// links closed under c -> -c or lying in a lattice plane have zero first
// moment, so every rule of the paper keeps its form in d (bounce-back,
// the corrections N, the buried-link averages); only the density picks up
// the weight sum, rho = 1 + sum_k d_k.  Working in d keeps the FP32 and FP16
// forms accurate: the stored numbers are the small deviations, not f ~ w.
// ---------------------------------------------------------------------------

// ---------------------------------------------------------------------------
// Boundary rules of one node.  m has bit f set when the node lies on boundary
// face f (at most one bit per axis).  The face rule is instantiated per face
// (its unknowns and normal are constants); the edge and corner rule is
// written once for all of them, with the set of unknown populations U, the
// normals and the edge direction as per-lane values and each update a
// select.  Every population index is a compile-time constant, so the 19
// populations stay in registers and are never indexed at run time.  A wave
// whose lanes lie on one or two faces (the ends of x-rows) runs only those
// faces' rules.
//
// Face (one bit; Sec. IV, Appendix; general form of eq_bbshort):
//   rho (1 - v.n) = sum_{c.n=0} f + 2 sum_{c.n<0} f                       (eq_uin)
//                 = 1 + sum_{c.n<=0} d + sum_{c.n<0} d
//   for every unknown j (c_j.n > 0), i = -j:
//   f_j = f_i - 6 w_i rho (c_i.v) - (rho/3) (t_i.v) + 1/2 t_i.M           (eq_bbshort)
//   with t_i = c_i - (c_i.n) n = c_i + n and M = sum_{c.n=0} f c (the
//   in-plane momentum; t_i.M = c_i.M as M is normal to n).  The factor 6 w_i
//   is rho/3 on the normal link (eq_f5) and rho/6 on the diagonals
//   (eq_f9-eq_f17); the last two terms are the corrections N (eq_Nx, eq_Ny).
// Pressure face (Sec. IV eq_rhoin; Appendix): rho = rho0 is prescribed with
// the tangential velocity, and the normal component follows from the same
// bracket, v.n = 1 - (1 + sum_{c.n<=0} d + sum_{c.n<0} d) / rho0; the
// unknowns then take the same formula as above.
// Edge (two bits; Sec. V, eq_Nxzy, eq_edge, eq_buried) and corner (three
// bits; eq_corner), both no-slip:
//   buried links: unknown populations whose opposite is unknown as well
//   (the pair +-(n1 - n2) on an edge, the six c.(n1+n2+n3) = 0 on a corner);
//   every other unknown is bounced back, f_k = f_{-k}; on an edge the four
//   bounced links with c.e != 0 (e the edge direction) also get
//   -(c.e)(f_{+e} - f_{-e})/4, which removes the momentum along the edge;
//   buried links = (sum of the other moving populations) / D with D = 22
//   (edge) or 18 (corner) -- in deviations, the weights' share 22/36 or
//   18/36 cancels against the buried links' own weight 1/36; rest
//   population = 12 times that.  On an edge or corner of a pressure face the
//   buried links and the rest population instead take what the prescribed
//   density leaves, in the ratio of their weights (eq_buried_rho; Sec. V
//   corner form): in deviations (rho0 - 1 - s) / 14 (edge) or / 18 (corner),
//   s the sum of the other moving populations.
// ---------------------------------------------------------------------------
// Every rule is computed by all lanes of a wave in which some lane needs it
// and selected where it applies (mine): no divergent branches around it, and
// no register copies where they would join.  The few waves with boundary
// nodes are the ones the others of a workgroup wait for, so what counts is
// the length of the rules' dependent chains: in the two-step pass a plane of
// a workgroup at the faces took 7.4 us, 4.5 us with no rules at all.  This
// form against divergent branches and divisions, two steps per pass: 256 x 128
// x 128 FP32 0.110 -> 0.100 ms per step, 512 x 256 x 256 FP16 0.494 -> 0.458
// ms.  In the single sweep of rows of up to 64 nodes, where every wave holds
// both x faces and runs both rules, it is from 15% faster (64 x 64 x 65 FP16
// 7.7 -> 6.7 us per step) to 3% slower (48 x 100 x 100 FP32 19.6 -> 20.2);
// divergent branches around these rules there are slower still (21.3).

// Values of one face.
template <class T>
struct FaceVals {
  T v[3], r0;   // velocity or tangential velocity, prescribed density (in unit<T>())
  T den, inv;   // as NodeParams
};

// Divisor of the bracket of face b with velocity v or density r0.
template <class T, int b>
__host__ __device__ __forceinline__ T face_divisor(bool pressure, const T (&v)[3], T r0) {
  return pressure ? r0 : T(1) - T(face_normal(b, b / 2)) * v[b / 2];
}

// Face rule of face b (one bit of m; b a compile-time constant, so the set of
// unknowns U, the normal n and every population index are constants and only
// the unknowns' updates are computed).  pressure: b is a pressure face.  The
// sums run in population order.
template <class T, int b>
__device__ __forceinline__ void face_rule(T (&d)[19], bool mine, bool pressure, T keep_n, const FaceVals<T> &f) {
#pragma clang fp contract(off)
  constexpr unsigned U = unknown_mask(b);
  constexpr int s = face_normal(b, b / 2), ax = b / 2;
  T s_known = T(0), s_out = T(0), M[3] = {T(0), T(0), T(0)};
#pragma unroll
  for (int k = 0; k < 19; ++k) {
    const bool unk = (U >> k) & 1u;
    const bool out = (U >> opp(k)) & 1u;  // c_k.n < 0
    const int c[3] = {cx(k), cy(k), cz(k)};
    if (!unk) s_known += d[k];
    if (out) s_out += d[k];
    if (!unk && !out)
#pragma unroll
      for (int a = 0; a < 3; ++a)
        if (c[a]) M[a] += T(c[a]) * d[k];
  }
  const T B = unit<T>() + s_known + s_out;
  const T q = quotient(B, f.den, f.inv);
  T v[3] = {f.v[0], f.v[1], f.v[2]}, rho = q;
  if (pressure) {
    v[ax] += T(s) * (T(1) - q);  // normal velocity from the density
    rho = f.r0;
  }
  const T vn = T(s) * v[ax];
  const T rho3 = quotient(rho, T(3), T(1) / T(3));
#pragma unroll
  for (int j = 0; j < 18; ++j) {
    if (!((U >> j) & 1u)) continue;
    const int i = opp(j);
    const int c[3] = {cx(i), cy(i), cz(i)};
    T civ = T(c[ax]) * v[ax], ciM = T(0);
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (c[a] && a != ax) {
        civ += T(c[a]) * v[a];
        ciM = T(c[a]) * M[a];
      }
    const T e = fused_add(-(T(6 * w36(i)) / T(36) * rho), civ, d[i]);
    const T n = fused_add(T(0.5), ciM, -(rho3 * (civ + vn)));
    const T dj = fused_add(keep_n, n, e);
    d[j] = mine ? dj : d[j];
  }
}

// Edge (two bits of m) or corner (three bits), no-slip; r0: the density of a
// bordering pressure face when there is one (pressure; at most one, as
// pressure faces lie on one axis).  mine: m has two or three bits.
template <class T>
__device__ __forceinline__ void edge_corner_rule(T (&d)[19], bool mine, unsigned m, bool pressure, T r0) {
#pragma clang fp contract(off)
  // Populations that enter (U) and leave (O) through the node's plane on each
  // axis; buried: entering through one plane and leaving through another.
  unsigned U[3], O[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const bool lo = (m >> (2 * a)) & 1u, hi = (m >> (2 * a + 1)) & 1u;
    U[a] = lo ? unknown_mask(2 * a) : (hi ? unknown_mask(2 * a + 1) : 0u);
    O[a] = lo ? unknown_mask(2 * a + 1) : (hi ? unknown_mask(2 * a) : 0u);
  }
  unsigned bur = (U[0] & (O[1] | O[2])) | (U[1] & (O[0] | O[2])) | (U[2] & (O[0] | O[1]));
  unsigned bounced = (U[0] | U[1] | U[2]) & ~bur;
  bur = mine ? bur : 0u;
  bounced = mine ? bounced : 0u;
  const bool edge = __popc(m) == 2;
  // A quarter of the momentum along the edge, on the axis of an edge node
  // that has no plane.
  T P[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) P[a] = edge && U[a] == 0u ? T(0.25) * (d[2 * a] - d[2 * a + 1]) : T(0);
  // Of two opposite links at most one is bounced back.
#pragma unroll
  for (int k = 0; k < 18; ++k) {
    const int o = opp(k);
    if (o < k) continue;
    T to_k = d[o], to_o = d[k];
    const int c[3] = {cx(k), cy(k), cz(k)};
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (c[a]) {
        to_k -= T(c[a]) * P[a];
        to_o += T(c[a]) * P[a];
      }
    const T dk = d[k];
    d[k] = ((bounced >> k) & 1u) ? to_k : dk;
    d[o] = ((bounced >> o) & 1u) ? to_o : d[o];
  }
  T s = T(0);
#pragma unroll
  for (int k = 0; k < 18; ++k) s += ((bur >> k) & 1u) ? T(0) : d[k];
  T db = quotient(s, edge ? T(22) : T(18), edge ? T(1) / T(22) : T(1) / T(18));
  if (__builtin_amdgcn_ballot_w64(pressure)) {
    const T db_p = quotient(r0 - unit<T>() - s, edge ? T(14) : T(18), edge ? T(1) / T(14) : T(1) / T(18));
    db = pressure ? db_p : db;
  }
#pragma unroll
  for (int k = 6; k < 18; ++k) d[k] = ((bur >> k) & 1u) ? db : d[k];  // axis links are never buried
  d[18] = mine ? T(12) * db : d[18];
}

// Boundary rule of a node with face mask m: the face rules a wave's lanes
// need, then the edge and corner rule.  vals(b): the FaceVals of face b (b a
// std::integral_constant); pmask: the pressure faces among m's faces (p_mask
// for box faces, 0 for the walls of a complex geometry); density(pm): that
// of the pressure face in pm.
template <class T, class Vals, class Density>
__device__ __forceinline__ void apply_boundary_rule(T (&d)[19], unsigned m, unsigned pmask, unsigned rule_flags,
                                                    const Vals &vals, const Density &density) {
  const T keep_n = (rule_flags & kRuleNoTransverse) ? T(0) : T(1);
#define LBM_FACE(b)                                         \
  if (__builtin_amdgcn_ballot_w64(m == (1u << (b))))        \
    face_rule<T, b>(d, m == (1u << (b)), ((pmask >> (b)) & 1u) != 0u, keep_n, vals(std::integral_constant<int, b>()));
  LBM_FACE(0)
  LBM_FACE(1)
  LBM_FACE(2)
  LBM_FACE(3)
  LBM_FACE(4)
  LBM_FACE(5)
#undef LBM_FACE
  const bool corner = (m & (m - 1u)) != 0u;
  if (__builtin_amdgcn_ballot_w64(corner)) {
    const unsigned pm = m & pmask;
    edge_corner_rule<T>(d, corner, m, pm != 0u, density(pm));
  }
}

// Density of the pressure face among the faces pm (at most one bit).
template <class T, class Rho>
__device__ __forceinline__ T edge_density(unsigned pm, const Rho &rho) {
  T r0 = unit<T>();
#pragma unroll
  for (int b = 0; b < 6; ++b)
    if (pm & (1u << b)) r0 = rho(b);
  return r0;
}

// With face values per lane (a per-node velocity field, or the walls of a
// complex geometry).  (vx, vy, vz, r0): not used on edges and corners.
template <class T>
__device__ __forceinline__ void boundary_rule(T (&d)[19], unsigned m, const NodeParams<T> &p, unsigned pmask, T vx,
                                              T vy, T vz, T r0) {
  apply_boundary_rule<T>(
      d, m, pmask, p.rule_flags,
      [&](auto b) {
        FaceVals<T> f{{vx, vy, vz}, r0, T(1), T(1)};
        f.den = face_divisor<T, b()>(((pmask >> b()) & 1u) != 0u, f.v, r0);
        f.inv = T(1) / f.den;
        return f;
      },
      [&](unsigned pm) { return edge_density<T>(pm, [&](int b) { return p.rho_p[b]; }); });
}

// Of a box whose faces take the lattice's face parameters.
template <class T>
__device__ __forceinline__ void box_boundary_rule(T (&d)[19], unsigned m, const NodeParams<T> &p) {
  apply_boundary_rule<T>(
      d, m, p.p_mask, p.rule_flags,
      [&](auto b) {
        return FaceVals<T>{{p.fv.v[b()][0], p.fv.v[b()][1], p.fv.v[b()][2]}, p.rho_p[b()], p.den[b()], p.inv[b()]};
      },
      [&](unsigned pm) { return edge_density<T>(pm, [&](int b) { return p.rho_p[b]; }); });
}

// The same with the face values in a table in LDS: a kernel that runs the
// rule inside a loop keeps no scalar registers for them (the compiler
// otherwise holds them across the loop and spills).
template <class T>
__device__ __forceinline__ void box_boundary_rule_table(T (&d)[19], unsigned m, unsigned p_mask, unsigned rule_flags,
                                                        const FaceVals<T> *tab) {
  apply_boundary_rule<T>(
      d, m, p_mask, rule_flags, [&](auto b) { return tab[b()]; },
      [&](unsigned pm) { return edge_density<T>(pm, [&](int b) { return tab[b].r0; }); });
}

// Fill the divisors of every face from its velocity or density.
template <class T>
__host__ __device__ inline void set_face_divisors(NodeParams<T> &p) {
  const T d[6] = {face_divisor<T, 0>(p.p_mask & 1u, p.fv.v[0], p.rho_p[0]),
                  face_divisor<T, 1>(p.p_mask & 2u, p.fv.v[1], p.rho_p[1]),
                  face_divisor<T, 2>(p.p_mask & 4u, p.fv.v[2], p.rho_p[2]),
                  face_divisor<T, 3>(p.p_mask & 8u, p.fv.v[3], p.rho_p[3]),
                  face_divisor<T, 4>(p.p_mask & 16u, p.fv.v[4], p.rho_p[4]),
                  face_divisor<T, 5>(p.p_mask & 32u, p.fv.v[5], p.rho_p[5])};
  for (int f = 0; f < 6; ++f) {
    p.den[f] = d[f];
    p.inv[f] = T(1) / d[f];
  }
}

// ---------------------------------------------------------------------------
// Wall nodes of a complex geometry (Sec. V) that are not plane, concave-edge
// or corner nodes.  U: bit set of the unknown populations.
//
// Convex edge (eq_edge2): U is the single diagonal n1 + n2 (n1, n2 the
// normals of the two solid faces, pointing into the fluid).  It is bounced
// back; then the momentum along the edge e = n1 x n2, P = sum_j d_j c_j.e,
// is removed from the four populations travelling into the bulk with
// c.e != 0 (c = +-e + n1, +-e + n2): d_c -= (c.e) P / 4.
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ void convex_edge_rule(T (&d)[19], unsigned U) {
  int sx = 0, sy = 0, sz = 0;  // n1 + n2
#pragma unroll
  for (int k = 6; k < 18; ++k)
    if ((U >> k) & 1u) {
      sx = cx(k);
      sy = cy(k);
      sz = cz(k);
    }
  // e is the axis with no component in n1 + n2 (its sign does not matter).
  const int ex = sx == 0 ? 1 : 0, ey = sy == 0 ? 1 : 0, ez = sz == 0 ? 1 : 0;
  // (+ 0: a select between two plain array elements would be turned into a
  // load through a selected address, which forces the array into scratch.)
#pragma unroll
  for (int k = 6; k < 18; ++k) d[k] = ((U >> k) & 1u) ? d[opp(k)] + T(0) : d[k];
  T P = T(0);
#pragma unroll
  for (int k = 0; k < 18; ++k) {
    const int ce = cx(k) * ex + cy(k) * ey + cz(k) * ez;
    if (ce != 0) P += T(ce) * d[k];
  }
  const T Pq = T(0.25) * P;
#pragma unroll
  for (int k = 0; k < 18; ++k) {
    const int ce = cx(k) * ex + cy(k) * ey + cz(k) * ez;
    const int cs = cx(k) * sx + cy(k) * sy + cz(k) * sz;
    d[k] = (ce != 0 && cs == 1) ? d[k] - T(ce) * Pq : d[k];
  }
}

// Any other wall node (an edge meeting a plane, thin features): bounce back
// every unknown whose opposite is known; the buried links (opposite unknown
// as well) and the rest population take the others' mass in the ratio of the
// lattice weights -- in deviations d_b = w36_b * s / W36, s the sum of the
// non-buried moving deviations, W36 their weight sum in units of 1/36 (22 on
// a concave edge, 18 on a corner, 24 when nothing is buried).
template <class T>
__device__ __forceinline__ void general_wall_rule(T (&d)[19], unsigned U) {
  unsigned bur = 0;
#pragma unroll
  for (int k = 0; k < 18; ++k) bur |= ((U >> k) & (U >> opp(k)) & 1u) << k;
#pragma unroll
  for (int k = 0; k < 18; ++k) d[k] = (((U & ~bur) >> k) & 1u) ? d[opp(k)] + T(0) : d[k];  // + 0: see above
  T s = T(0);
  int W = 0;
#pragma unroll
  for (int k = 0; k < 18; ++k) {
    const bool b = (bur >> k) & 1u;
    s += b ? T(0) : d[k];
    W += b ? 0 : w36(k);
  }
  const T per = s / T(W);
#pragma unroll
  for (int k = 0; k < 18; ++k) d[k] = ((bur >> k) & 1u) ? T(w36(k)) * per : d[k];
  d[18] = T(12) * per;
}

// BGK collision towards the second-order equilibrium (eq_bgk, eq_feq), in
// deviations: rho = 1 + sum d, rho u = sum d c,
//   d_k^eq = f_k^eq - w_k = w_k (rho - 1) + w_k rho (3 c.u + 4.5 (c.u)^2 - 1.5 u^2),
//   d_k <- d_k + omega (d_k^eq - d_k), omega = 1/tau, c_s^2 = 1/3.
// A body force F enters as the velocity shift tau F / rho inside f^eq
// (eq_gravity): u = (sum d c + tau F) / rho.

// c_k . u of a diagonal link is one component's momentum times 1 / rho fused
// with the other component's velocity; whether the first component is the
// fused one.  x_first: that of every link with an x component is.  The
// extended sweep of FP16 with round-to-nearest has always summed them so; the
// other way 12 in 10^5 values of the six links that differ move by half a unit
// of the stored half, so a run that is continued or repeated needs it kept.
__host__ __device__ constexpr bool fuses_first(int k, bool x_first) {
  return cx(k) ? (x_first || (cx(k) < 0 && cy(k) + cz(k) < 0)) : !(cy(k) < 0 && cz(k) > 0);
}

template <class T, bool XFirst = false>
__device__ __forceinline__ void bgk_collide(T (&d)[19], T omega, const T (&tau_f)[3]) {
#pragma clang fp contract(off)
  // Moments: partial sums over the populations with c_a = +1, -1 (and, for
  // x, 0); each starts from its first term (0 + x is not foldable under
  // signed zeros, so a zero start would cost an instruction).
  static_assert(cx(0) == 1 && cx(1) == -1 && cy(2) == 1 && cy(3) == -1 && cz(4) == 1 && cz(5) == -1 &&
                    cx(2) == 0 && cx(3) == 0 && cx(4) == 0 && cx(5) == 0,
                "axis populations first (paper order, Sec. II)");
  T xp = d[0], xm = d[1], yp = d[2], ym = d[3], zp = d[4], zm = d[5];
  T x0 = (d[2] + d[3]) + (d[4] + d[5]);
#pragma unroll
  for (int k = 6; k < 19; ++k) {
    if (cx(k) > 0) xp += d[k];
    if (cx(k) < 0) xm += d[k];
    if (cx(k) == 0) x0 += d[k];
    if (cy(k) > 0) yp += d[k];
    if (cy(k) < 0) ym += d[k];
    if (cz(k) > 0) zp += d[k];
    if (cz(k) < 0) zm += d[k];
  }
  const T drho = (xp + xm) + x0;
  const T rho = unit<T>() + drho;
  // 1 / rho: correctly rounded in double; in float (the FP16 forms, whose
  // storage keeps 11 bits) the hardware reciprocal, within about 1 ulp, in
  // one instruction instead of the ten of a rounded division
  T ir;
  if constexpr (sizeof(T) == 4)
    ir = __builtin_amdgcn_rcpf(rho);
  else
    ir = T(1) / rho;
  const T j[3] = {xp - xm + tau_f[0], yp - ym + tau_f[1], zp - zm + tau_f[2]};
  const T u[3] = {j[0] * ir, j[1] * ir, j[2] * ir};
  // d_eq = w (drho + rho (3 cu + 4.5 cu^2 - 1.5 u^2)) = w (C + cu (B + A cu)), and
  // d + omega (d_eq - d) = (1 - omega) d + (omega w) (C + cu (B + A cu)).
  const T A = T(4.5) * rho, B = T(3) * rho;
  const T C = fused_add(-(T(1.5) * rho), fused_add(u[2], u[2], fused_add(u[0], u[0], u[1] * u[1])), drho);
  const T keep = T(1) - omega;
#pragma unroll
  for (int k = 0; k < 19; ++k) {
    const T ow = omega * weight<T>(k);
    T t = C;
    if (k != 18) {
      const int c[3] = {cx(k), cy(k), cz(k)};
      const int a = c[0] ? 0 : (c[1] ? 1 : 2);  // first moving component, and the second if there is one
      const int b = a == 0 ? (c[1] ? 1 : 2) : 2;
      T cu = T(c[a]) * u[a];
      if (b != a && c[b]) cu = fuses_first(k, XFirst) ? fused_add(T(c[a]) * j[a], ir, T(c[b]) * u[b]) : fused_add(T(c[b]) * j[b], ir, cu);
      t = fused_add(fused_add(A, cu, B), cu, C);
    }
    d[k] = fused_add(keep, d[k], ow * t);
  }
}

}  // namespace lbm
