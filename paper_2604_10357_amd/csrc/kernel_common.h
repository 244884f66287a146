// kernel_common.h -- device helpers shared by the element kernels: tile
// remapping, coefficient lookup, reference geometry and field gradients.
#pragma once

#include "rules.h"
#include "tlfea_internal.h"

namespace tlfea {
namespace {

// Workgroup b is dispatched to XCD b % 8; hand each XCD a contiguous tile range
// so the CSR rows a tile touches are shared with its neighbours in one L2.
__device__ __forceinline__ int remap_tile(int bid, int nblocks) {
  const int xcd = bid & 7, idx = bid >> 3;
  const int per = nblocks >> 3, extra = nblocks & 7;
  return xcd * per + (xcd < extra ? xcd : extra) + idx;
}

template <class Rule>
__device__ __forceinline__ int64_t coef_of(const int32_t* conn_e, int a) {
  if constexpr (Rule::MC == 1) return conn_e[a];
  else return 4 * (int64_t)conn_e[a >> 2] + (a & 3);
}

// element scale of each coefficient kind (ANCF: 1, lx/2, ly/2, H/2; T10: 1)
template <class Rule>
__device__ __forceinline__ void element_scales(const AsmArgs& a, int64_t ge, double* sc) {
  if constexpr (Rule::MC == 1) {
    sc[0] = sc[1] = sc[2] = sc[3] = 1.0;
  } else {
    sc[0] = 1.0;
    sc[1] = a.escale[2 * ge];
    sc[2] = a.escale[2 * ge + 1];
    sc[3] = a.half_h;
  }
}

template <class Rule>
__device__ __forceinline__ void load_geometry(const AsmArgs& a, int64_t ge, int q, double* Jinv, double& det) {
  const double* rec = a.geo + 10 * (a.affine ? ge : ge * Rule::NQ + q);
#pragma unroll
  for (int t = 0; t < 9; ++t) Jinv[t] = rec[t];
  det = rec[9];
}

// Gradient  sum_a (u_a - X_a) (x) g_a  (X may be null) of a nodal field u at point q.
// Formed as (sum_a u_a (x) dN_a) J0^-1: parent gradient first, then one 3x3 product.
// The gradients of the position functions sum to zero, so the value at the
// element's first coefficient is taken out of every position coefficient: the
// terms stay of the size of the element's own variation of the field.
template <class Rule>
__device__ __forceinline__ void field_gradient(const AsmArgs& a, int64_t ge, int q, const double* sc,
                                               const double* u, const double* X, const double* Jinv,
                                               double* out) {
  const int32_t* conn_e = a.conn + ge * Rule::NPN;
  double D[9], r0[3];
#pragma unroll
  for (int t = 0; t < 9; ++t) D[t] = 0.0;
  {
    const int64_t c0 = coef_of<Rule>(conn_e, 0);
#pragma unroll
    for (int i = 0; i < 3; ++i) r0[i] = X ? u[3 * c0 + i] - X[3 * c0 + i] : u[3 * c0 + i];
  }
#pragma unroll
  for (int al = 0; al < Rule::NEN; ++al) {
    const int64_t c = coef_of<Rule>(conn_e, al);
    const double s = sc[al % 4];
    const double w0 = Rule::dN_rt(q, al, 0) * s, w1 = Rule::dN_rt(q, al, 1) * s,
                 w2 = Rule::dN_rt(q, al, 2) * s;
    const bool position = Rule::MC == 1 || (al & 3) == 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const double d = (X ? u[3 * c + i] - X[3 * c + i] : u[3 * c + i]) - (position ? r0[i] : 0.0);
      D[3 * i] += d * w0;
      D[3 * i + 1] += d * w1;
      D[3 * i + 2] += d * w2;
    }
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int J = 0; J < 3; ++J)
      out[3 * i + J] = D[3 * i] * Jinv[J] + D[3 * i + 1] * Jinv[3 + J] + D[3 * i + 2] * Jinv[6 + J];
}

// Nodal values of a workgroup's elements in LDS: 6 doubles per (element,
// coefficient), u = q - X then qdot (zero without qdot), for elements
// e_lo .. e_lo + ne - 1.
template <class Rule>
__device__ __forceinline__ void gather_nodal(const AsmArgs& a, int64_t e_lo, int ne, double* nod) {
  constexpr int NEN = Rule::NEN, NPN = Rule::NPN;
  for (int idx = threadIdx.x; idx < ne * NEN; idx += blockDim.x) {
    const int le = idx / NEN, al = idx - le * NEN;
    const int64_t e = e_lo + le;
    double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (e < a.n_elem) {
      const int64_t c = coef_of<Rule>(a.conn + e * NPN, al);
#pragma unroll
      for (int i = 0; i < 3; ++i) v[i] = a.q[3 * c + i] - a.X[3 * c + i];
      if (a.qdot) {
#pragma unroll
        for (int i = 0; i < 3; ++i) v[3 + i] = a.qdot[3 * c + i];
      }
    }
#pragma unroll
    for (int t = 0; t < 6; ++t) nod[6 * idx + t] = v[t];
  }
}

// Parent gradients D = sum_a u_a (x) dN_a of T10 fields at the points of the
// five-point rule.  With u_cb the value of the node on edge (c, b) and u_cc that
// of corner c, the gradient at barycentric coordinates L is
//   D_k = g_k - g_0,  g_b = 4 sum_c L_c u_cb - u_b,
// and at the rule's points (the centroid, or L_c = 1/2 and the others 1/6)
//   centroid:          D_k = S_k,
//   point of corner c: D_k = 4/3 (u_ck - u_c0) + V_k,  V_k = 2/3 S_k - 1/3 (u_k - u_0),
//   S_k = sum over j other than 0, k of (u_jk - u_j0).
// V and S belong to the element and are formed once for it (18 values a field,
// V at 3 i + k, S at 9 + 3 i + k), so a point takes 18 operations a field
// instead of the 120 of the sum over ten nodes, and no gradient table; every
// term is a difference of two of the element's values, so no digits go to its
// rigid displacement.
constexpr int kT10Terms = 18;

// LDS doubles per element of the gathered fields u and qdot (and their terms)
template <class Rule>
constexpr int nodal_doubles() { return 6 * Rule::NEN + (Rule::MC == 1 ? 2 * kT10Terms : 0); }

// V and S of NF fields of `ne` elements: field f of element e at u + STRIDE * 10 e + 3 f
// (STRIDE doubles per node), the terms at terms + kT10Terms * (NF e + f).
// Called by every lane of the workgroup, between two barriers.
template <int NF, int STRIDE>
__device__ __forceinline__ void t10_element_terms(const double* u, int ne, double* terms) {
  for (int t = threadIdx.x; t < ne * 3 * NF; t += blockDim.x) {
    const int e = t / (3 * NF), r = t - 3 * NF * e;  // r = 3 f + i
    const double* n = u + STRIDE * 10 * e + r;
    const double u0 = n[0], e01 = n[4 * STRIDE], e12 = n[5 * STRIDE], e02 = n[6 * STRIDE], e03 = n[7 * STRIDE],
                 e13 = n[8 * STRIDE], e23 = n[9 * STRIDE];
    const double S[3] = {(e12 - e02) + (e13 - e03), (e12 - e01) + (e23 - e03), (e13 - e01) + (e23 - e02)};
    double* out = terms + kT10Terms * (t / 3) + 3 * (t % 3);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      out[k] = 2.0 / 3.0 * S[k] - 1.0 / 3.0 * (n[(k + 1) * STRIDE] - u0);
      out[9 + k] = S[k];
    }
  }
}

// D of one field at point q, u the field's values of the element (STRIDE doubles per node)
template <int STRIDE>
__device__ __forceinline__ void t10_parent_gradient(const double* u, const double* terms, int q, double (&D)[9]) {
  // nodes (c, 0), (c, 1), (c, 2), (c, 3) of the point's corner c = q - 1, four bits each
  const int row = q <= 1 ? 0x7640 : q == 2 ? 0x8514 : q == 3 ? 0x9256 : 0x3987;
  const double w = q == 0 ? 0.0 : 4.0 / 3.0;
  const double* T = terms + (q == 0 ? 9 : 0);
  const double* c0 = u + STRIDE * (row & 15);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double* ck = u + STRIDE * ((row >> (4 * (k + 1))) & 15);
#pragma unroll
    for (int i = 0; i < 3; ++i) D[3 * i + k] = w * (ck[i] - c0[i]) + T[3 * i + k];
  }
}

// Displacement and velocity gradients at point q of element e from its nodal
// values in LDS (ne: 6 doubles per coefficient): Hd = sum_a u_a (x) g_a,
// Fd = sum_a qdot_a (x) g_a, with g_a = J0^-T dN_a (Sec. 4.3, Eq. F_assembly).
// The position functions sum to one, so their gradients sum to zero and the
// first coefficient's values may be taken out of every position coefficient:
// the terms then stay of the size of the element's own deformation instead of
// its rigid displacement (a body turned far from the origin keeps the digits
// of its strain).  T10 takes the closed form above (terms: the element's V and
// S of both fields; other elements ignore it).  The four-coefficient
// elements run over the coefficients in steps of four (a full unroll keeps
// every table load in flight, which costs the shell half its waves) and skip
// the parent gradients that vanish at every point (Rule::grad_nz).
template <class Rule>
__device__ __forceinline__ void tile_kinematics(const AsmArgs& a, const double* ne, const double* terms, int64_t e, int q,
                                                double (&Jinv)[9], double& det, double (&Hd)[9], double (&Fd)[9]) {
  constexpr int NEN = Rule::NEN;
  load_geometry<Rule>(a, e, q, Jinv, det);
  double Du[9], Dv[9];
  if constexpr (Rule::MC == 1) {
    t10_parent_gradient<6>(ne, terms, q, Du);
    t10_parent_gradient<6>(ne + 3, terms + kT10Terms, q, Dv);
  } else {
    double sc[4], r0[6];
    element_scales<Rule>(a, e, sc);
#pragma unroll
    for (int t = 0; t < 9; ++t) Du[t] = Dv[t] = 0.0;
#pragma unroll
    for (int t = 0; t < 6; ++t) r0[t] = ne[t];
#pragma unroll 4
    for (int al = 0; al < NEN; ++al) {
      const double s = sc[al % 4];
      const bool position = (al & 3) == 0;
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        if (!Rule::grad_nz(al, m)) continue;
        const double w = Rule::dN_rt(q, al, m) * s;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          Du[3 * i + m] += (ne[6 * al + i] - (position ? r0[i] : 0.0)) * w;
          Dv[3 * i + m] += (ne[6 * al + 3 + i] - (position ? r0[3 + i] : 0.0)) * w;
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int J = 0; J < 3; ++J) {
      Hd[3 * i + J] = Du[3 * i] * Jinv[J] + Du[3 * i + 1] * Jinv[3 + J] + Du[3 * i + 2] * Jinv[6 + J];
      Fd[3 * i + J] = Dv[3 * i] * Jinv[J] + Dv[3 * i + 1] * Jinv[3 + J] + Dv[3 * i + 2] * Jinv[6 + J];
    }
}

// material constants of a launch: the host copy, or the device vector when given
__device__ __forceinline__ MatParams launch_material(const AsmArgs& a) {
  MatParams mp = a.mp;
  if (a.mp_dev) {
    mp.c0 = a.mp_dev[0];
    mp.c1 = a.mp_dev[1];
    mp.c2 = a.mp_dev[2];
    mp.eta = a.mp_dev[3];
    mp.lam_v = a.mp_dev[4];
  }
  return mp;
}

// Hd = F - I and Fdot at point q of element ge (float64).
template <class Rule>
__device__ __forceinline__ void load_kinematics(const AsmArgs& a, int64_t ge, int q, double* Hd, double* Fd,
                                                double* Jinv, double& det) {
  load_geometry<Rule>(a, ge, q, Jinv, det);
  double sc[4];
  element_scales<Rule>(a, ge, sc);
  field_gradient<Rule>(a, ge, q, sc, a.q, a.X, Jinv, Hd);
  if (a.qdot) {
    field_gradient<Rule>(a, ge, q, sc, a.qdot, nullptr, Jinv, Fd);
  } else {
#pragma unroll
    for (int t = 0; t < 9; ++t) Fd[t] = 0.0;
  }
}

// the assembly arguments of body `bi` of a batch
__device__ __forceinline__ AsmArgs body_args(const BatchArgs& b, const BatchBody& B, int bi) {
  AsmArgs a;
  a.conn = B.conn;
  a.X = B.X;
  a.geo = B.geo;
  a.escale = B.escale;
  a.half_h = B.half_h;
  a.affine = B.affine;
  a.n_elem = B.n_elem;
  a.n_tiles = 0;
  a.q = b.q + B.dof_off;
  a.qdot = b.qdot ? b.qdot + B.dof_off : nullptr;
  a.f = nullptr;
  a.vals = nullptr;
  a.row_off = B.row_off;
  a.rank = B.rank;
  a.mp = B.mp;
  a.alpha = b.h[bi];
  a.beta = 1.0;
  a.flags = b.flags;
  a.mp_dev = nullptr;
  return a;
}

}  // namespace
}  // namespace tlfea
