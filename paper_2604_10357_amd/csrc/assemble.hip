// assemble.hip -- internal force and tangent stiffness for gfx950, in two passes
// that write every output value exactly once and use no global atomics.
//
// What is computed (arXiv 2604.10357, Part II):
//   F  = I + sum_a (x_a - X_a) (x) g_a,  Fdot = sum_a xdot_a (x) g_a   (Sec. 4.3, Eq. F_assembly)
//   P  = P_el(F) + P_vis(F, Fdot)                                     (Sec. 4.3, Stage 1)
//   f_a = sum_q P g_a J0 w_q, summed over the elements of each DOF    (Eqs. fint_local, fint_global)
//   K_ab = sum_q A g_a g_b J0 w_q, summed into the fixed CSR pattern  (Sec. 4.4.2, Eq. tangent_block)
//
// The paper scatters per entry with atomicAdd and names two-pass
// scatter/reduction as the way around atomic contention.  On MI355X scattered
// float64 atomics retire at roughly the rate of random read-modify-writes, so
// this library never issues them:
//
//   pass 1 (one lane per element x quadrature point): gather the element,
//     form F and Fdot in float64, run the constitutive update and store the
//     point's tangent and stress in parent coordinates with the quadrature
//     volume folded in,
//        Ahat_imkn = dV sum_JL J0inv_mJ A_iJkL J0inv_nL,  Phat_im = dV sum_J P_iJ J0inv_mJ,
//     as one record of nine 10-value slots: slot (i, k) holds Ahat_imkn at
//     3 m + n and Phat_ik at 9 (90 values, padded to 96).
//   pass 2 (one workgroup per contiguous range of nodes): the CSR rows of
//     consecutive nodes form one contiguous segment, mirrored in LDS.  Each
//     lane owns one (node, incident element, coefficient row i, component k)
//     task, reads slot (i, k) of the element's records at every point and forms
//        t_n = sum_m dN_a,m Ahat_imkn,   K[a i, b k] += sum_n t_n dN_b,n,
//     where the parent gradients dN_b at each point are compile-time constants
//     (zeros skipped).  Results are added into the LDS segment in float64, and
//     the segment and the node forces are then written with plain coalesced
//     stores.  f_int comes out of the same pass from Phat.
//   Workgroups are remapped so each XCD walks a contiguous range of elements /
//   nodes, keeping the records a range reads in its own L2.
//
// Most tangents contract the element's points in pass 1 instead, into one block
// per (element, node) that pass 2 reads once (the element rows below).
#include <cstdlib>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "kernel_common.h"
#include "work_buffer.h"

// work area of the allocation-free force call, one copy per device
static __device__ __align__(256) unsigned char scratch[TLFEA_NOALLOC_SCRATCH_BYTES];

namespace tlfea {
namespace {

constexpr int kRecK = 96;  // tangent record: nine slots of kSlot values, padded
constexpr int kSlot = 10;  // slot (i, k): Ahat_imkn at 3 m + n, Phat_ik at 9
constexpr int kRecF = 12;  // force-only record: Phat_ik at 4 i + k

// 16-byte vectors as native clang vector types (HIP's struct vector types are
// not always promoted to registers)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <typename T>
struct Vec4 { using type = f32x4; };
template <>
struct Vec4<double> { using type = f64x2; };

// ordering of LDS accesses between the lanes of one wave
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// pass 1
// ---------------------------------------------------------------------------
template <class Rule, typename R, bool WANT_K>
__device__ __forceinline__ void stage_point(const AsmArgs& a, int64_t e, int q, R* rec) {
  double Hd[9], Fd[9], Jinv[9], det;
  load_kinematics<Rule>(a, e, q, Hd, Fd, Jinv, det);
  PointOut<R> o;
  const unsigned fl = point_update<R, WANT_K>(a.mp, Hd, Fd, det * Rule::w_rt(q), a.alpha, a.beta, o);
  if (fl) atomicOr(a.flags, fl);
  HatOut<R> h;
  to_parent<R, WANT_K>(o, Jinv, h);
  if constexpr (WANT_K) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        R* slot = rec + kSlot * (3 * i + k);
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
          for (int n = 0; n < 3; ++n) slot[3 * m + n] = hat_entry(h, i, m, k, n);
        slot[9] = h.P[3 * i + k];
      }
#pragma unroll
    for (int t = 9 * kSlot; t < kRecK; ++t) rec[t] = R(0);
  } else {
#pragma unroll
    for (int t = 0; t < 9; ++t) rec[4 * (t / 3) + t % 3] = h.P[t];
  }
}

template <class Rule, typename R, bool WANT_K>
__global__ __launch_bounds__(256) void k_stage(AsmArgs a, R* stage) {
  constexpr int NQ = Rule::NQ;
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= a.n_elem * NQ) return;
  stage_point<Rule, R, WANT_K>(a, p / NQ, (int)(p % NQ), stage + p * (WANT_K ? kRecK : kRecF));
}

// Value W of a tangent record (W is a compile-time index into the layout above).
template <int W, class FO, typename R>
__device__ __forceinline__ R record_value(const HatOut<R>& h) {
  if constexpr (W < 9 * kSlot) {
    constexpr int slot = W / kSlot, x = W % kSlot, i = slot / 3, k = slot % 3;
    if constexpr (x < 9) return hat_entry<FO>(h, i, x / 3, k, x % 3);
    else return h.P[3 * i + k];
  } else {
    return R(0);
  }
}

// Undamped materials: the tangent has major symmetry, Ahat_imkn = Ahat_knim
// (every term of the factored form is symmetric under (i, m) <-> (k, n) once
// the viscous parts are zero), so slot (k, i) is slot (i, k) transposed.  An
// element-row record then holds the six slots with i <= k, in the order (0,0),
// (0,1), (0,2), (1,1), (1,2), (2,2), each as above (Ahat at 3 m + n, Phat_ik at
// 9), then Phat_10, Phat_20, Phat_21 and one pad: 64 values instead of 92.
constexpr int kRecS = 64;

template <int W, typename R>
__device__ __forceinline__ R record_value_sym(const HatOut<R>& h) {
  if constexpr (W < 6 * kSlot) {
    constexpr int sl = W / kSlot, x = W % kSlot;
    constexpr int i = sl < 3 ? 0 : sl < 5 ? 1 : 2, k = sl < 3 ? sl : sl < 5 ? sl - 2 : 2;
    if constexpr (x < 9) return hat_entry(h, i, x / 3, k, x % 3);
    else return h.P[3 * i + k];
  } else if constexpr (W < 6 * kSlot + 3) {
    constexpr int j = W - 6 * kSlot, i = j == 0 ? 1 : 2, k = j == 2 ? 1 : 0;
    return h.P[3 * i + k];
  } else {
    return R(0);
  }
}

// Where the slot (i, k) of a task lies in a point record (full or symmetric
// layout), and whether its Ahat block is read transposed.
struct SlotRef {
  int off;  // first Ahat value
  int p;    // Phat_ik
  bool tr;
};
template <bool SYM>
__device__ __forceinline__ SlotRef slot_ref(int i, int k) {
  if constexpr (!SYM) {
    return {kSlot * (3 * i + k), kSlot * (3 * i + k) + 9, false};
  } else {
    const int lo = i < k ? i : k, hi = i < k ? k : i;
    const int sl = lo == 0 ? hi : lo == 1 ? hi + 2 : 5;
    const bool tr = i > k;
    return {kSlot * sl, tr ? 6 * kSlot + i + k - 1 : kSlot * sl + 9, tr};
  }
}

// Pass 1 with the tangent, one workgroup per 256 consecutive (element, point)
// indices.  The nodal values of the workgroup's elements (u = q - X and qdot
// per coefficient) are gathered into LDS once instead of once per point, and
// the records leave through a per-wave LDS transpose: each 128-byte piece of
// the wave's 64 records is one cache line, stored by 8 lanes with 16-byte
// writes, so every store instruction writes 8 whole lines.
template <class Rule>
constexpr int stage_elems() { return (kStageThreads - 1) / Rule::NQ + 2; }

template <class Rule, typename R>
constexpr size_t stage_lds_bytes() {
  const size_t nodal = (size_t)stage_elems<Rule>() * nodal_doubles<Rule>() * sizeof(double);
  const size_t trans = (size_t)kStageThreads * (128 + 16);
  return nodal > trans ? nodal : trans;
}

template <class Rule, typename R, bool SYM = false>
__device__ __forceinline__ void stage_tile(const AsmArgs& a, R* stage, int64_t blk) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, NPN = Rule::NPN;
  constexpr int REC = SYM ? kRecS : kRecK;  // record length (symmetric layout for undamped materials)
  constexpr int EB = stage_elems<Rule>();
  using V = typename Vec4<R>::type;
  constexpr int PER = (int)(sizeof(V) / sizeof(R));
  __shared__ __align__(16) unsigned char smem[stage_lds_bytes<Rule, R>()];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t npts = a.n_elem * NQ;
  const int64_t p0 = blk * kStageThreads;
  const int64_t e_lo = p0 / NQ;
  const int64_t p = p0 + tid;
  const bool act = p < npts;
  // 1. nodal values of the elements the block's points belong to
  double* nod = reinterpret_cast<double*>(smem);
  double* terms = nod + EB * NEN * 6;
  gather_nodal<Rule>(a, e_lo, EB, nod);
  __syncthreads();
  if constexpr (Rule::MC == 1) {
    t10_element_terms<2, 6>(nod, EB, terms);
    __syncthreads();
  }
  // 2. kinematics at the lane's point (lanes past the end evaluate the last
  //    point and store nothing)
  const int64_t pc = act ? p : npts - 1;
  const int64_t e = pc / NQ;
  const int q = (int)(pc - e * NQ);
  double Jinv[9], det, Hd[9], Fd[9];
  const int el = (int)(e - e_lo);
  tile_kinematics<Rule>(a, nod + 6 * NEN * el, terms + 2 * kT10Terms * el, e, q, Jinv, det, Hd, Fd);
  __syncthreads();  // the nodal values are consumed: the LDS becomes the transpose buffers
  PointOut<R> o;
  const unsigned fl = point_update<R, true>(a.mp, Hd, Fd, det * Rule::w_rt(q), a.alpha, a.beta, o);
  if (act && fl) atomicOr(a.flags, fl);
  HatOut<R> h;
  to_parent<R, true>(o, Jinv, h);
  // 3. records through the per-wave transpose, one 128-byte piece at a time
  constexpr int CW = 128 / (int)sizeof(R);       // values per piece
  constexpr int LS = CW + 16 / (int)sizeof(R);   // lane stride in the buffer (padded)
  R* tb = reinterpret_cast<R*>(smem) + wave * 64 * LS;
  const int64_t pw = p0 + 64 * wave;
  static_assert(REC % CW == 0, "records of whole 128-byte pieces");
  sfor<0, REC / CW>([&](auto cc) __attribute__((always_inline)) {
    constexpr int ch = decltype(cc)::value;
    wave_sync();
    sfor<0, CW / PER>([&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value;
      V v;
      sfor<0, PER>([&](auto xc) __attribute__((always_inline)) {
        constexpr int x = decltype(xc)::value;
        if constexpr (SYM) v[x] = record_value_sym<ch * CW + j * PER + x>(h);
        else v[x] = record_value<ch * CW + j * PER + x, FuseOther>(h);
      });
      *reinterpret_cast<V*>(tb + lane * LS + j * PER) = v;
    });
    wave_sync();
#pragma unroll
    for (int s8 = 0; s8 < 8; ++s8) {
      const int r = 8 * s8 + (lane >> 3), j = lane & 7;
      if (pw + r < npts)
        *reinterpret_cast<V*>(stage + (pw + r) * REC + ch * CW + j * PER) =
            *reinterpret_cast<const V*>(tb + r * LS + j * PER);
    }
  });
}

template <class Rule, typename R, bool SYM>
__global__ __launch_bounds__(kStageThreads) void k_stage_tile(AsmArgs a, R* stage) {
  stage_tile<Rule, R, SYM>(a, stage, blockIdx.x);
}

// many bodies: every body starts on a block of its own, found by bisection
template <class Rule, typename R>
__global__ __launch_bounds__(kStageThreads) void k_stage_batch(BatchArgs b) {
  const int64_t blk = blockIdx.x;
  int lo = 0, hi = b.n_bodies - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (b.bodies[mid].block_off <= blk) lo = mid; else hi = mid - 1;
  }
  const BatchBody& B = b.bodies[lo];
  const AsmArgs a = body_args(b, B, lo);
  stage_tile<Rule, R>(a, (R*)b.stage + B.point_off * kRecK, blk - B.block_off);
}

// ---------------------------------------------------------------------------
// pass 2
// ---------------------------------------------------------------------------
// Values one lane reads per point: its slot of a tangent record, or its Phat
// entry of a force record.
template <typename R, bool WANT_K>
struct Slot {
  static constexpr int N = WANT_K ? kSlot : 1;
  R v[N];
};

// read a slot from the wave's LDS copy of the records (8-byte aligned for
// float, 16-byte aligned for double)
template <typename R, bool WANT_K>
__device__ __forceinline__ void load_slot(const R* p, Slot<R, WANT_K>& s) {
  if constexpr (!WANT_K) {
    s.v[0] = *p;
  } else if constexpr (sizeof(R) == 8) {
#pragma unroll
    for (int t = 0; t < kSlot / 2; ++t) {
      const f64x2 x = reinterpret_cast<const f64x2*>(p)[t];
      s.v[2 * t] = x[0];
      s.v[2 * t + 1] = x[1];
    }
  } else {
#pragma unroll
    for (int t = 0; t < kSlot / 2; ++t) {
      const f32x2 x = reinterpret_cast<const f32x2*>(p)[t];
      s.v[2 * t] = x[0];
      s.v[2 * t + 1] = x[1];
    }
  }
}

// One point's contribution of a task (row i, component k of node a's
// coefficient al): with the slot of the task's element at point Q and the
// task's scaled parent gradient d = dN_al(Q) (times the coefficient scale),
//   t_n = sum_m d_m Ahat_imkn,  acc[b] += sum_n t_n dN_b,n(Q),  facc += Phat_ik d_k.
template <class Rule, typename R, bool WANT_F, bool WANT_K, int Q, int NB, bool KREC = WANT_K>
__device__ __forceinline__ void contract_point(const Slot<R, KREC>& s, R d0, R d1, R d2, int k, R (&acc)[NB],
                                               R& facc) {
  if constexpr (WANT_F) facc += (KREC ? s.v[9] : s.v[0]) * (k == 0 ? d0 : k == 1 ? d1 : d2);
  if constexpr (WANT_K) {
    R tn[3];
#pragma unroll
    for (int n = 0; n < 3; ++n) tn[n] = sum3<false>(s.v[n], d0, s.v[3 + n], d1, s.v[6 + n], d2);
    sfor<0, Rule::NEN>([&](auto bc) __attribute__((always_inline)) {
      constexpr int b = decltype(bc)::value;
      constexpr double c0 = Rule::dN(Q, b, 0), c1 = Rule::dN(Q, b, 1), c2 = Rule::dN(Q, b, 2);
      R v = acc[b];
      if constexpr (c0 != 0.0) v += tn[0] * R(c0);
      if constexpr (c1 != 0.0) v += tn[1] * R(c1);
      if constexpr (c2 != 0.0) v += tn[2] * R(c2);
      acc[b] = v;
    });
  }
}

// Pass-2 records travel through LDS: the 64 tasks of a wave touch at most
// chunk_incidences() consecutive incidences, whose records are copied, one
// point at a time, into a wave-private LDS buffer with 16-byte loads of
// consecutive lanes (whole cache lines per instruction); each lane then reads
// its own slot from there.  The copies of the next points are in flight in
// registers while a point is contracted.
constexpr int chunk_incidences(int tpi) { return (tpi + 62) / tpi + 1; }

// Float32 tangent records of short rules can be read two ways: through the
// LDS copy, or by the lane itself (its 10-value slot always lies in three
// aligned 16-byte pieces of the record), for all points at once.  The first
// kStagedPoints points take the LDS copy; splitting the points between the two
// paths did not beat reading them all directly (the default, 0).
#ifndef TLFEA_STAGED_POINTS
#define TLFEA_STAGED_POINTS 0
#endif
constexpr int kStagedPoints = TLFEA_STAGED_POINTS;

template <class Rule, typename R, bool WANT_K>
constexpr bool direct_slots() {
  return WANT_K && sizeof(R) == 4 && Rule::NQ <= 6;
}
// points of a rule that go through the LDS copy
template <class Rule, typename R, bool WANT_K>
constexpr int staged_points() {
  return direct_slots<Rule, R, WANT_K>() ? (kStagedPoints < Rule::NQ ? kStagedPoints : Rule::NQ) : Rule::NQ;
}

template <class Rule, typename R, bool WANT_K, bool SYM = false>
constexpr size_t wave_buf_bytes() {
  return staged_points<Rule, R, WANT_K>() == 0
             ? 0
             : (size_t)chunk_incidences(9 * Rule::MC) * (WANT_K ? (SYM ? kRecS : kRecK) : kRecF) * sizeof(R);
}

// The same with a run-time point index q (long rules); q is uniform across the
// wave, so the gradients dN_b(q) come through the scalar cache.
template <class Rule, typename R, bool WANT_F, bool WANT_K, int NB, bool KREC = WANT_K>
__device__ __forceinline__ void contract_point_rt(const Slot<R, KREC>& s, int q, int al, int k, R sc_al,
                                                  R (&acc)[NB], R& facc) {
  const R d0 = (R)Rule::dN_rt(q, al, 0) * sc_al, d1 = (R)Rule::dN_rt(q, al, 1) * sc_al,
          d2 = (R)Rule::dN_rt(q, al, 2) * sc_al;
  if constexpr (WANT_F) facc += (KREC ? s.v[9] : s.v[0]) * (k == 0 ? d0 : k == 1 ? d1 : d2);
  if constexpr (WANT_K) {
    R tn[3];
#pragma unroll
    for (int n = 0; n < 3; ++n) tn[n] = s.v[n] * d0 + s.v[3 + n] * d1 + s.v[6 + n] * d2;
#pragma unroll
    for (int b = 0; b < Rule::NEN; ++b)
      acc[b] += tn[0] * (R)Rule::dN_rt(q, b, 0) + tn[1] * (R)Rule::dN_rt(q, b, 1) + tn[2] * (R)Rule::dN_rt(q, b, 2);
  }
}

// The range's CSR values leave the LDS segment with plain coalesced stores:
// the whole segment, or (upper-triangle output) the suffix of every row from
// its diagonal on.  For the latter the range's upper row offsets are copied
// into LDS (after the force rows; the launch reserves the room), and groups of
// 16 lanes write a row each (one 128-byte line per store).  Called by every
// lane of the workgroup.
template <bool ACCUM>
__device__ __forceinline__ void write_segment(const GatherArgs& g, int64_t row0, int nrow, int nseg, int64_t seg0,
                                              double* lds, const int32_t* rowo) {
  if (!g.row_off_u) {
    double* out = g.vals + seg0;
    for (int t = threadIdx.x; t < nseg; t += blockDim.x) out[t] = ACCUM ? out[t] + lds[t] : lds[t];
    return;
  }
  int32_t* rowu = reinterpret_cast<int32_t*>(lds + nseg + nrow);
  const int32_t u_base = g.row_off_u[row0];
  for (int rr = threadIdx.x; rr <= nrow; rr += blockDim.x) rowu[rr] = g.row_off_u[row0 + rr] - u_base;
  __syncthreads();
  double* out = g.vals + u_base;
  constexpr int GL = 16;  // lanes per row
  const int sub = threadIdx.x % GL, groups = blockDim.x / GL;
  for (int rr = threadIdx.x / GL; rr < nrow; rr += groups) {
    const int u0 = rowu[rr], n = rowu[rr + 1] - u0;
    const int beg = (rr + 1 < nrow ? rowo[rr + 1] : nseg) - n;
    for (int j = sub; j < n; j += GL) out[u0 + j] = ACCUM ? out[u0 + j] + lds[beg + j] : lds[beg + j];
  }
}

// Newton matrix (Sec. 4.4.2, Eq. hessian): the LDS segment of a range starts
// from M_(I,k)(J,l) / h on the diagonal entries (d, d) of every 3x3 block
// ((I,k), (J,l)) of its rows (MC coefficients k per node; the segment is zero
// elsewhere).  Runs after the segment is cleared and before any contribution
// is added.  The range's mass entries (one MC x MC block per adjacent node
// pair) are contiguous in adjacency order, and a node's first entry within the
// range is rowo[3 MC n] / (9 MC^2) (each entry is one 3 x 3 MC piece of each
// of the node's 3 MC rows): a lane per entry finds its node by bisection.
template <int MC>
__device__ __forceinline__ void add_mass_term(const GatherArgs& g, int32_t I0, int nn, double* lds,
                                              const int32_t* rowo) {
  if (!g.mass) return;
  constexpr int RPN = 3 * MC, PER = 9 * MC * MC;
  const int32_t k0 = g.adj_off[I0];
  const int n_ent = g.adj_off[I0 + nn] - k0;
  for (int x = threadIdx.x; x < n_ent; x += blockDim.x) {
    int lo = 0, hi = nn - 1;  // last node whose first entry is <= x
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (rowo[RPN * mid] / PER <= x) lo = mid; else hi = mid - 1;
    }
    const int r = x - rowo[RPN * lo] / PER;
    const double* mx = g.mass + (int64_t)MC * MC * (k0 + x);
#pragma unroll
    for (int k = 0; k < MC; ++k)
#pragma unroll
      for (int l = 0; l < MC; ++l) {
        const double v = mx[MC * k + l] * g.inv_h;
#pragma unroll
        for (int d = 0; d < 3; ++d) lds[rowo[RPN * lo + 3 * k + d] + 3 * MC * r + 3 * l + d] = v;
      }
  }
}

// A slot read from a symmetric record: the lower slots (i > k) are the upper
// ones transposed, and Phat_ik of a lower slot lies after the six slots.
template <bool SYM, typename R, bool KREC>
__device__ __forceinline__ void sym_slot_fix(Slot<R, KREC>& sl, const R* recb, const SlotRef& sr) {
  if constexpr (SYM) {
    const R a1 = sl.v[1], a2 = sl.v[2], a5 = sl.v[5];
    sl.v[1] = sr.tr ? sl.v[3] : a1;
    sl.v[3] = sr.tr ? a1 : sl.v[3];
    sl.v[2] = sr.tr ? sl.v[6] : a2;
    sl.v[6] = sr.tr ? a2 : sl.v[6];
    sl.v[5] = sr.tr ? sl.v[7] : a5;
    sl.v[7] = sr.tr ? a5 : sl.v[7];
    sl.v[9] = recb[sr.p];
  }
}

// KREC: the records carry the tangent layout (a pass 1 with the tangent); the
// force alone can also be taken from them (WANT_K false).
// SYM: symmetric tangent records (float64 only; the lane's slot may be read
// transposed).
template <class Rule, typename R, bool WANT_F, bool WANT_K, bool ACCUM, bool KREC = WANT_K, bool SYM = false>
__device__ __forceinline__ void gather_range(const GatherArgs& g, int32_t I0, int32_t I1, unsigned char* smem,
                                             int32_t* pre, int32_t* rowo) {
  static_assert(KREC || !WANT_K, "the tangent needs tangent records");
  static_assert(!SYM || (KREC && sizeof(R) == 8), "symmetric records: float64 tangent records");
  constexpr int NQ = Rule::NQ, NPN = Rule::NPN, MC = Rule::MC, NEN = Rule::NEN;
  constexpr int RPN = 3 * MC;  // CSR rows per node
  constexpr int TPI = 3 * RPN; // tasks per incidence: (coefficient kind, row, component)
  constexpr int REC = KREC ? (SYM ? kRecS : kRecK) : kRecF;
  constexpr int NI = chunk_incidences(TPI);
  using V = typename Vec4<R>::type;
  constexpr int PER = (int)(sizeof(V) / sizeof(R));
  constexpr int NV = REC / PER;            // 16-byte pieces per record
  constexpr int KC = (NI * NV + 63) / 64;  // pieces each lane copies per point
  // short rules are unrolled over all points (gradients dN_b as compile-time
  // constants); long rules run over blocks of PB points
  constexpr bool UNROLL = NQ <= 6;
  constexpr int PB = UNROLL ? NQ : 3;
  static_assert(NQ % PB == 0, "point blocks must tile the rule");
  constexpr int PD = UNROLL ? (sizeof(R) == 4 ? NQ : 3) : PB;  // points whose pieces are in flight
  constexpr int NB = WANT_K ? NEN : 1;
  constexpr bool DIRECT = direct_slots<Rule, R, KREC>();
  constexpr int NS = staged_points<Rule, R, KREC>();  // points through the LDS copy (DIRECT: the first NS)
  constexpr int PDS = DIRECT ? (NS > 0 ? NS : 1) : PD;     // staged points in flight
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwave = blockDim.x >> 6;
  // LDS: incidence -> node table, wave record buffers, CSR segment + forces
  uint8_t* incn = smem;
  R* wbuf = reinterpret_cast<R*>(smem + g.inc_cap) + wave * NI * REC;
  double* lds = reinterpret_cast<double*>(smem + g.inc_cap + nwave * wave_buf_bytes<Rule, R, KREC, SYM>());
  const int nn = I1 - I0;
  const int64_t row0 = (int64_t)RPN * I0, row1 = (int64_t)RPN * I1;
  const int64_t seg0 = WANT_K ? g.row_off[row0] : 0, seg1 = WANT_K ? g.row_off[row1] : 0;
  const int nseg = (int)(seg1 - seg0);
  const int nrow = (int)(row1 - row0);
  double* lf = lds + nseg;
  for (int t = tid; t < nseg + nrow; t += blockDim.x) lds[t] = 0.0;
  // the incidence offsets are already a prefix sum: task offsets of the
  // range's nodes follow from one parallel load
  const int32_t inc0 = g.inc_off[I0];
  for (int n = tid; n <= nn; n += blockDim.x) pre[n] = TPI * (g.inc_off[I0 + n] - inc0);
  // segment-relative offsets of the range's CSR rows
  if constexpr (WANT_K)
    for (int rr = tid; rr < nrow; rr += blockDim.x) rowo[rr] = (int32_t)(g.row_off[row0 + rr] - seg0);
  __syncthreads();
  // range-local node of every incidence (nodes < kMaxRangeNodes fit a byte)
  for (int n = tid; n < nn; n += blockDim.x)
    for (int j = pre[n] / TPI; j < pre[n + 1] / TPI; ++j) incn[j] = (uint8_t)n;
  if constexpr (WANT_K) add_mass_term<MC>(g, I0, nn, lds, rowo);
  __syncthreads();
  const int ntask = pre[nn];
  // Tasks are ordered (node, incidence, kind, row, component): task t belongs
  // to incidence inc0 + t / TPI of the range.  The wave's chunk of an
  // iteration starting at task t0 covers incidences j0 .. j0 + ni - 1; lanes
  // past the last task repeat it and store nothing, and copy pieces past the
  // chunk's end repeat its last piece (in bounds, same value written twice).
  auto chunk = [&](int t0_, int& j0_, int& ni_) __attribute__((always_inline)) {
    const int cw = min(t0_ + 64 * wave, ntask - 1);
    j0_ = cw / TPI;
    ni_ = min(cw + 63, ntask - 1) / TPI - j0_ + 1;
  };
  // the lane's copy pieces in a full chunk (record rr0, piece pp0); in a
  // short chunk, pieces past its end become its last piece (ni - 1, NV - 1)
  int rr0[KC], pp0[KC];
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    rr0[k] = (lane + 64 * k) / NV;
    pp0[k] = lane + 64 * k - rr0[k] * NV;
  }
  // record addresses in 16-byte units (32 bits: checked on the host)
  const V* stagev = reinterpret_cast<const V*>(g.stage);
  constexpr uint32_t VPP = REC / PER;  // 16-byte pieces per point record
  // incidence entries an iteration needs (its copy pieces' and the lane's
  // own), fetched one iteration ahead
  auto fetch_inc = [&](int t0_, int32_t (&icp)[KC], int32_t& ime) __attribute__((always_inline)) {
    int j0_, ni_;
    chunk(t0_, j0_, ni_);
    if constexpr (NS > 0) {
#pragma unroll
      for (int k = 0; k < KC; ++k) icp[k] = g.inc[inc0 + j0_ + min(rr0[k], ni_ - 1)];
    }
    ime = g.inc[inc0 + min(t0_ + tid, ntask - 1) / TPI];
  };
  int32_t icp[KC], ime;
  fetch_inc(0, icp, ime);
  for (int t0 = 0; t0 < ntask; t0 += blockDim.x) {  // uniform across the workgroup
    const bool act = t0 + tid < ntask;
    const int t = min(t0 + tid, ntask - 1);
    int j0, ni;
    chunk(t0, j0, ni);
    uint32_t src[KC];
    int dst[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const bool in = rr0[k] < ni;
      src[k] = (uint32_t)(icp[k] >> 4) * (NQ * VPP) + (uint32_t)(in ? pp0[k] : NV - 1);
      dst[k] = in ? rr0[k] * REC + pp0[k] * PER : ni * REC - PER;
    }
    V buf[PDS][KC];
    if constexpr (NS > 0) {
      sfor<0, PDS>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
#pragma unroll
        for (int k = 0; k < KC; ++k) buf[q][k] = stagev[src[k] + q * VPP];
      });
    }
    const int32_t packed = ime;
    if (t0 + (int)blockDim.x < ntask) fetch_inc(t0 + blockDim.x, icp, ime);
    const int n = incn[t / TPI];
    const int r = t % TPI, ca = r / 9, i = (r / 3) % 3, k = r % 3;  // pre[] holds multiples of TPI
    const int64_t e = packed >> 4;
    const int a = packed & 15;
    const int al = MC * a + ca;
    const SlotRef sr = slot_ref<SYM>(i, k);
    const R* recb = wbuf + (t / TPI - j0) * REC;  // the lane's record in the wave buffer
    const R* mine = recb + (KREC ? sr.off : 4 * i + k);
    // slot-map row of (e, a): one aligned vector load
    constexpr int RST = rank_stride(NPN);
    uint32_t rkw[RST / 4];
    if constexpr (WANT_K) {
      const uint32_t* rp = reinterpret_cast<const uint32_t*>(g.rank + (e * NPN + a) * RST);
      if constexpr (RST == 16) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 w = *reinterpret_cast<const u32x4*>(rp);
        rkw[0] = w[0];
        rkw[1] = w[1];
        rkw[2] = w[2];
        rkw[3] = w[3];
      } else {
        rkw[0] = rp[0];
      }
    }
    double scd[4] = {1.0, 1.0, 1.0, 1.0};
    if constexpr (MC == 4) {
      scd[1] = g.escale[2 * e];
      scd[2] = g.escale[2 * e + 1];
      scd[3] = g.half_h;
    }
    const R sc_al = (R)(ca == 0 ? scd[0] : ca == 1 ? scd[1] : ca == 2 ? scd[2] : scd[3]);
    R acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = R(0);
    R facc = R(0);
    // DIRECT: the lane's slot s = 3 i + k sits at value 10 s of each point
    // record, inside pieces floor(10 s / 4) .. + 2, shifted by 0 (s even) or 2
    V own[DIRECT && NQ > NS ? NQ - NS : 1][3];
    const bool odd_slot = (3 * i + k) & 1;
    if constexpr (DIRECT && NQ > NS) {
      const uint32_t p0 = (uint32_t)(packed >> 4) * (NQ * VPP) + (uint32_t)((kSlot * (3 * i + k)) >> 2);
#pragma unroll
      for (int q = NS; q < NQ; ++q)
#pragma unroll
        for (int j = 0; j < 3; ++j) own[q - NS][j] = stagev[p0 + q * VPP + j];
    }
    if constexpr (UNROLL) {
      // the task's parent gradients at all points: one row of the table
      R dna[16];
      {
        using V4 = typename Vec4<R>::type;
        constexpr int P4 = (int)(sizeof(V4) / sizeof(R));
        const V4* rowv = reinterpret_cast<const V4*>(Rule::template rows<R>(al));
#pragma unroll
        for (int t = 0; t < 16 / P4; ++t) {
          const V4 x = rowv[t];
#pragma unroll
          for (int u = 0; u < P4; ++u) dna[P4 * t + u] = x[u] * sc_al;
        }
      }
      sfor<0, NQ>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        Slot<R, KREC> sl;
        if constexpr (DIRECT && q >= NS) {
#pragma unroll
          for (int x = 0; x < kSlot; ++x) {
            const R lo = own[q - NS][x >> 2][x & 3], hi = own[q - NS][(x + 2) >> 2][(x + 2) & 3];
            sl.v[x] = odd_slot ? hi : lo;
          }
        } else {
          wave_sync();  // every lane is done with the previous point's records
#pragma unroll
          for (int kk = 0; kk < KC; ++kk) *reinterpret_cast<V*>(wbuf + dst[kk]) = buf[q % PDS][kk];
          wave_sync();
          if constexpr (q + PDS < NS) {
#pragma unroll
            for (int kk = 0; kk < KC; ++kk)
              buf[q % PDS][kk] = stagev[src[kk] + (q + PDS) * VPP];
          }
          load_slot<R, KREC>(mine, sl);
          sym_slot_fix<SYM>(sl, recb, sr);
        }
        contract_point<Rule, R, WANT_F, WANT_K, q, NB, KREC>(sl, dna[3 * q], dna[3 * q + 1], dna[3 * q + 2], k, acc,
                                                             facc);
      });
    } else {
#pragma unroll 1
      for (int qb = 0; qb < NQ; qb += PB) {
        sfor<0, PB>([&](auto xc) __attribute__((always_inline)) {
          constexpr int x = decltype(xc)::value;
          const int q = qb + x;
          wave_sync();
#pragma unroll
          for (int kk = 0; kk < KC; ++kk) *reinterpret_cast<V*>(wbuf + dst[kk]) = buf[x][kk];
          wave_sync();
          if (q + PB < NQ) {
#pragma unroll
            for (int kk = 0; kk < KC; ++kk)
              buf[x][kk] = stagev[src[kk] + (uint32_t)(q + PB) * VPP];
          }
          Slot<R, KREC> sl;
          load_slot<R, KREC>(mine, sl);
          sym_slot_fix<SYM>(sl, recb, sr);
          contract_point_rt<Rule, R, WANT_F, WANT_K, NB, KREC>(sl, q, al, k, sc_al, acc, facc);
        });
      }
    }
    if (act) {
      const int rl = RPN * n + 3 * ca + i;  // row within the range
      if constexpr (WANT_F) atomicAdd(lf + rl, (double)facc);
      if constexpr (WANT_K) {
        double* dstp = lds + rowo[rl] + k;
#pragma unroll
        for (int b = 0; b < NEN; ++b) {
          const int pb = (MC == 1) ? b : (b >> 2), cb = (MC == 1) ? 0 : (b & 3);
          const int rank_b = (int)((rkw[pb >> 2] >> (8 * (pb & 3))) & 255u);
          atomicAdd(dstp + 3 * (MC * rank_b + cb), (double)acc[b] * scd[b % 4]);
        }
      }
    }
  }
  __syncthreads();
  if constexpr (WANT_K) write_segment<ACCUM>(g, row0, nrow, nseg, seg0, lds, rowo);
  if constexpr (WANT_F) {
    double* out = g.f + row0;
    for (int t = tid; t < nrow; t += blockDim.x) out[t] = ACCUM ? out[t] + lf[t] : lf[t];
  }
}

template <class Rule, typename R, bool WANT_F, bool WANT_K, bool ACCUM, bool KREC, bool SYM>
__global__ __launch_bounds__(512) void k_gather(GatherArgs g) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t pre[kMaxRangeNodes + 1];
  __shared__ int32_t rowo[kMaxRangeNodes * 3 * Rule::MC];
  const int r = remap_tile(blockIdx.x, gridDim.x);
  gather_range<Rule, R, WANT_F, WANT_K, ACCUM, KREC, SYM>(g, g.ranges[r], g.ranges[r + 1], smem, pre, rowo);
}

template <class Rule, typename R>
__global__ __launch_bounds__(512) void k_gather_batch(BatchArgs b) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t pre[kMaxRangeNodes + 1];
  __shared__ int32_t rowo[kMaxRangeNodes * 3 * Rule::MC];
  const int r = remap_tile(blockIdx.x, gridDim.x);
  const BatchRange br = b.ranges[r];
  const BatchBody& B = b.bodies[br.body];
  GatherArgs g{};
  g.ranges = nullptr;
  g.inc_off = B.inc_off;
  g.inc = B.inc;
  g.row_off = B.row_off;
  g.rank = B.rank;
  g.escale = B.escale;
  g.half_h = B.half_h;
  g.stage = (const R*)b.stage + B.point_off * kRecK;
  g.f = b.f + B.dof_off;
  g.vals = b.vals + B.nnz_off;
  g.inc_cap = b.inc_cap;
  gather_range<Rule, R, true, true, false>(g, br.I0, br.I1, smem, pre, rowo);
}

// ---------------------------------------------------------------------------
// element rows (T10, with the tangent)
// ---------------------------------------------------------------------------
// Pass 1 reduces over the points itself: a lane per point forms the point's
// tangent and stress, then a lane per task (element, node a, row i, component
// k) contracts the element's five points exactly as the gather does, giving
// the ten entries K_e[3a+i][3b+k], b = 0..9, summed over the points (Sec.
// 4.4.2, Eq. tangent_block), and its part P_ik dN_a,k of f_a,i (Eq.
// fint_local).  Each (element, node) row block goes to the node's place in the
// node-sorted incidence list, so that pass 2 reads the blocks of a node range
// as one contiguous run, each block once, instead of re-reading per-point
// records for every range that shares an element.
constexpr int kRowChunk = 32;           // row i of a block: K entry (k, b) at 10 k + b, f_i at 30, one pad
constexpr int kRowBlk = 3 * kRowChunk;  // block: rows i = 0, 1, 2 (float32: one cache line each)
constexpr int kRowElems = 12;           // most elements of a pass-1 workgroup: one wave, 60 point lanes
// Waves per SIMD.  float64: the point's factors and the accumulators need 340
// registers, and one wave with the overflow in accumulation registers beats
// two that spill 81 to scratch (pass 1 of 480,000 elements 1.03 against 1.11 ms).
template <typename R>
constexpr int row_min_waves() { return sizeof(R) == 4 ? 2 : 1; }
// Row blocks up to this size in all go through the caches, where pass 2 finds them
// (the memory-side cache holds 256 MB); larger ones are stored past them, which
// pass 1 gains from.  Whole call, through / past, of damped elements: 18,000 59 / 60
// us, 21,600 65 / 67, 24,000 71 / 70, 30,000 100 / 97, 36,000 116 / 106 where other
// meshes' calls lie between two of one (back to back on one mesh 30,000 80 / 86,
// 33,000 85 / 90, 36,000 99 / 93): the line is at 24,576 elements.  Undamped ones
// gain less from it, 21,600 70 / 72, 24,000 75 / 75, 30,000 104 / 101 (back to back
// 82 / 87, 33,000 103 / 93): 32,768 elements, below which neither use loses against
// the 105 (81) us of 30,000 elements before either store.
constexpr size_t kCachedRowBytes = (size_t)90 << 20, kCachedSymRowBytes = (size_t)120 << 20;
// Damped float32 tiles up to this many take a workgroup for each row component: two
// waves a SIMD.  Whole call, in one / in three workgroups a tile: 6 elements 15.4 /
// 11.4 us, 270 17.5 / 13.2, 600 17.2 / 15.4, 1,020 18.1 / 20.1 (a tile each).
constexpr int64_t kSplitRowTiles = 682;
constexpr int kLptTile = 25;            // elements per item of the persistent batch schedule (or 16)
// undamped materials, float32
constexpr int kSymElems = 25;           // elements per pass-1 workgroup
constexpr int kSymThreads = 128;        // 125 point lanes
constexpr int kRecL = 92;               // LDS record stride in values (a 16-byte multiple; ANCF rows)
constexpr int kRecSL = 68;              // of the shell's symmetric records: lanes store theirs to different banks (64: to the
                                        // same ones, 65,536 shells 352 us, so 345; the beam and T10 keep 64, with which one
                                        // workgroup more fits a CU: 500,000 beams 766 / 782, 480,000 T10 447 / 488)
constexpr int kDnL = 20;                // LDS stride of a node's gradient row (16 used; 20 keeps the rows
                                        // of the ten nodes on different banks)
constexpr int kStgL = 100;              // LDS stride of a staged row block (96 used; spreads the banks)

// One piece of a row block on its way to pass 2, past the caches (NT) or through
// them (a template argument: a branch on a value is merged into one plain store).
template <bool NT, typename V>
__device__ __forceinline__ void store_piece(V v, V* p) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// Phase B of the element rows for a symmetric tangent (undamped materials):
// K_e^(ki)[b, a] = K_e^(ik)[a, b], so only the slots i <= k are contracted.
// A wave takes one element at a time, a lane per task (node a, slot i <= k):
// 60 lanes, each forming the ten entries K_e[3a+i][3b+k] over the points.  The
// lanes put them into the element's ten row blocks in the wave's LDS buffer,
// at (a, i, k, b) and, for i < k, transposed at (b, k, i, a); f_a,i is the sum
// of the parts Phat_ik dN_a,k of the node's lanes, in a fixed order.  Then the
// wave stores the ten blocks with 16-byte stores of consecutive lanes.  Two
// thirds of the multiply-adds of the full contraction.
template <class Rule, bool NT>
__device__ __forceinline__ void elem_rows_sym_contract(const int32_t* __restrict__ incpos, float* __restrict__ rows,
                                                       int64_t e0, int ne, const float* rec, const float* dn,
                                                       float* stage_buf) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN;
  static_assert(6 * NEN <= 64, "a lane per (node, upper slot)");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* stg = stage_buf + wave * NEN * kStgL;
  const int tl = lane < 6 * NEN ? lane : 0;  // lanes past the tasks repeat task 0 and store nothing
  const int an = tl / 6, us = tl - 6 * an;
  const int i = us < 3 ? 0 : us < 5 ? 1 : 2, k = us < 3 ? us : us < 5 ? us - 2 : 2;
  const int so = kSlot * us, pt = 6 * kSlot + i + k - 1;  // the slot, Phat_ki (i < k)
  float dna[16];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const f32x4 x = reinterpret_cast<const f32x4*>(dn + kDnL * an)[u];
    dna[4 * u] = x[0];
    dna[4 * u + 1] = x[1];
    dna[4 * u + 2] = x[2];
    dna[4 * u + 3] = x[3];
  }
  for (int le = wave; le < ne; le += kSymThreads / 64) {  // uniform per wave
    const int32_t my_pos = lane < NEN ? incpos[(e0 + le) * NEN + lane] : 0;
    float acc[NEN], fd = 0.0f, ft = 0.0f;
#pragma unroll
    for (int b = 0; b < NEN; ++b) acc[b] = 0.0f;
    const float* base = rec + le * NQ * kRecS;
    sfor<0, NQ>([&](auto qc) __attribute__((always_inline)) {
      constexpr int qq = decltype(qc)::value;
      const float* r = base + qq * kRecS;
      Slot<float, true> sv;
#pragma unroll
      for (int x = 0; x < 5; ++x) {
        const f32x2 w = *reinterpret_cast<const f32x2*>(r + so + 2 * x);
        sv.v[2 * x] = w[0];
        sv.v[2 * x + 1] = w[1];
      }
      const float d0 = dna[3 * qq], d1 = dna[3 * qq + 1], d2 = dna[3 * qq + 2];
      contract_point<Rule, float, true, true, qq, NEN>(sv, d0, d1, d2, k, acc, fd);
      if (i < k) ft += r[pt] * (i == 0 ? d0 : d1);  // Phat_ki dN_a,i
    });
    wave_sync();  // the previous element's blocks have left the buffer
    if (lane < 6 * NEN) {
      float* own = stg + an * kStgL + kRowChunk * i + kSlot * k;
#pragma unroll
      for (int u = 0; u < NEN / 2; ++u) {
        f32x2 v;
        v[0] = acc[2 * u];
        v[1] = acc[2 * u + 1];
        *reinterpret_cast<f32x2*>(own + 2 * u) = v;
      }
      if (i < k) {
#pragma unroll
        for (int b = 0; b < NEN; ++b) stg[b * kStgL + kRowChunk * k + kSlot * i + an] = acc[b];
      }
    }
    // f_a,0 = (0,0) + (0,1) + (0,2);  f_a,1 = (1,0) + (1,1) + (1,2);  f_a,2 = (2,0) + (2,1) + (2,2),
    // the (k, i) parts with k > i from the lanes of slot (i, k)
    const int l0 = 6 * an;
    const float d01 = __shfl(fd, l0 + 1, 64), d02 = __shfl(fd, l0 + 2, 64), d12 = __shfl(fd, l0 + 4, 64);
    const float t01 = __shfl(ft, l0 + 1, 64), t02 = __shfl(ft, l0 + 2, 64), t12 = __shfl(ft, l0 + 4, 64);
    const float d00 = __shfl(fd, l0, 64), d11 = __shfl(fd, l0 + 3, 64), d22 = __shfl(fd, l0 + 5, 64);
    if (lane < 6 * NEN && us < 3) {
      const float fv = us == 0 ? (d00 + d01) + d02 : us == 1 ? (t01 + d11) + d12 : (t02 + t12) + d22;
      stg[an * kStgL + kRowChunk * us + 3 * kSlot] = fv;
      stg[an * kStgL + kRowChunk * us + 3 * kSlot + 1] = 0.0f;
    }
    wave_sync();
#pragma unroll
    for (int u = 0; u < (NEN * kRowBlk / 4 + 63) / 64; ++u) {
      const int pc = lane + 64 * u, bl = pc / (kRowBlk / 4), pi = pc - bl * (kRowBlk / 4);
      const int32_t pb = __shfl(my_pos, bl < NEN ? bl : 0, 64);
      if (bl < NEN)
        store_piece<NT>(*reinterpret_cast<const f32x4*>(stg + bl * kStgL + 4 * pi),
                        reinterpret_cast<f32x4*>(rows + (int64_t)pb * kRowBlk + 4 * pi));
    }
  }
}

// Symmetric tangent (undamped materials, float32): 25 elements in two waves,
// the 64-value records of all their points in LDS.  480,000 elements: 0.580 ms
// with plain stores, 0.466 with non-temporal ones.
template <class Rule, bool NT>
__global__ __launch_bounds__(kSymThreads) void k_elem_rows_sym(AsmArgs a, int tile,
                                                              const int32_t* __restrict__ incpos,
                                                              float* __restrict__ rows) {
  static_assert(Rule::MC == 1 && Rule::NEN == 10, "element rows are built for T10");
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, EB = kSymElems;
  static_assert(EB * NQ <= kSymThreads, "a lane per point");
  __shared__ __align__(16) float rec[EB * NQ * kRecS];
  __shared__ __align__(16) float dn[NEN * kDnL];  // parent gradients of every node at every point
  __shared__ __align__(16) float stage_buf[(kSymThreads / 64) * NEN * kStgL];  // per-wave blocks
  static_assert(EB * nodal_doubles<Rule>() * sizeof(double) <= sizeof(rec), "nodal values fit the record area");
  const int tid = threadIdx.x;
  const int64_t e0 = (int64_t)blockIdx.x * tile;
  const int ne = (int)(a.n_elem - e0 < tile ? a.n_elem - e0 : tile);
  // 1. nodal values, the gradient table, then each point's kinematics
  double* nod = reinterpret_cast<double*>(rec);
  gather_nodal<Rule>(a, e0, ne, nod);
  for (int idx = tid; idx < NEN * 16; idx += kSymThreads)
    dn[kDnL * (idx / 16) + idx % 16] = Rule::template rows<float>(idx / 16)[idx % 16];
  __syncthreads();
  double* terms = nod + EB * NEN * 6;
  t10_element_terms<2, 6>(nod, ne, terms);
  __syncthreads();
  const bool act = tid < ne * NQ;
  const int pl = act ? tid : 0;  // idle lanes evaluate point 0 and store nothing
  const int el = pl / NQ, q = pl - el * NQ;
  double Jinv[9], det, Hd[9], Fd[9];
  tile_kinematics<Rule>(a, nod + 6 * NEN * el, terms + 2 * kT10Terms * el, e0 + el, q, Jinv, det, Hd, Fd);
  __syncthreads();  // the nodal values are consumed: the LDS holds the records from here on
  // 2. the point's record into LDS, then the contraction
  PointOut<float> o;
  const unsigned fl = point_update<float, true>(a.mp, Hd, Fd, det * Rule::w_rt(q), a.alpha, a.beta, o);
  if (act && fl) atomicOr(a.flags, fl);
  HatOut<float> h;
  to_parent<float, true>(o, Jinv, h);
  if (act) {
    float* r = rec + pl * kRecS;
    sfor<0, kRecS / 4>([&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value;
      f32x4 v;
      sfor<0, 4>([&](auto xc) __attribute__((always_inline)) {
        constexpr int x = decltype(xc)::value;
        v[x] = record_value_sym<4 * j + x>(h);
      });
      *reinterpret_cast<f32x4*>(r + 4 * j) = v;
    });
  }
  __syncthreads();
  elem_rows_sym_contract<Rule, NT>(incpos, rows, e0, ne, rec, dn, stage_buf);
}

// The row blocks of elements e0 .. e0 + ne - 1 (ne <= kRowElems), one wave.
// A point's factors (HatOut) stay in its lane's registers; the rows i = 0, 1,
// 2 of the element matrices are formed one after the other, so that LDS holds
// only the three slots (i, k) of every point at a time (30 values instead of
// 90).  For each row the wave takes four elements at a time, a lane per
// (element, component k, nodes a and a + 5): the lane reads a slot once for
// both nodes, contracts the five points, and the 40 rows leave through LDS
// with 16-byte stores of consecutive lanes (whole cache lines).  A single wave
// needs no barrier, and waves in different phases share a SIMD.
// Large meshes' stores are non-temporal (NT; kCachedRowBytes): no line is written
// twice or read by this pass, and through the L2 (4 MB against the 13 MB that one
// XCD's waves have in flight) they left in an order that HBM took at 3.3 TB/s.
// Bound by instruction issue (5,000 a wave, 66 % of it) and by the 1.84 GB of
// stores.  480,000 elements, float32: 0.672 ms with two-wave workgroups of 25
// elements and whole records in LDS (53 KB, 1.5 waves per SIMD), 0.565 row by
// row in single waves, 0.465 with non-temporal stores; without any store it
// takes 0.375.  One node per lane, held to three waves per SIMD, is as fast.
// ONE: only row component `row` is formed (k_elem_rows).
template <class Rule, typename R, bool NT, bool ONE = false>
__device__ __forceinline__ void elem_rows_tile(const AsmArgs& a, const int32_t* __restrict__ incpos,
                                               R* __restrict__ rows, int64_t e0, int ne, int row = 0) {
  static_assert(Rule::MC == 1 && Rule::NEN == 10 && 3 * kSlot <= kRowChunk, "element rows are built for T10");
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, EB = kRowElems;
  constexpr int Z = sizeof(R) == 4 ? 2 : 1, HN = NEN / Z;  // nodes per lane, lanes per (element, component)
  constexpr int GRP = 64 / (3 * HN);                       // elements the wave contracts at a time
  static_assert(EB * NQ <= 64, "a lane per point");
  using V = typename Vec4<R>::type;
  typedef R R2 __attribute__((ext_vector_type(2)));
  constexpr int PER = (int)(sizeof(V) / sizeof(R));         // values per 16-byte piece
  constexpr int RS = 3 * kSlot + (sizeof(R) == 4 ? 6 : 0);  // stride of a point's slots: on different banks
  constexpr int SS = kRowChunk + 2;                         // stride of a staged row: the slots on different banks
  constexpr int DL = 16 + PER;                              // stride of a node's gradient row
  constexpr size_t NOD = (size_t)EB * nodal_doubles<Rule>() * sizeof(double), REC = (size_t)EB * NQ * RS * sizeof(R);
  __shared__ __align__(16) unsigned char smem[NOD > REC ? NOD : REC];
  __shared__ __align__(16) R stg[GRP * NEN * SS];
  __shared__ __align__(16) R dn[NEN * DL];  // parent gradients of every node at every point
  __shared__ int32_t pos[EB * NEN];         // incidence position of every (element, node)
  const int lane = threadIdx.x;
  // 1. nodal values, the tables of the tasks, then each point's kinematics
  double* nod = reinterpret_cast<double*>(smem);
  gather_nodal<Rule>(a, e0, ne, nod);
  for (int idx = lane; idx < ne * NEN; idx += 64) pos[idx] = incpos[e0 * NEN + idx];
  for (int idx = lane; idx < NEN * 16; idx += 64) dn[DL * (idx / 16) + idx % 16] = Rule::template rows<R>(idx / 16)[idx % 16];
  wave_sync();
  double* terms = nod + EB * NEN * 6;
  t10_element_terms<2, 6>(nod, ne, terms);
  wave_sync();
  const bool act = lane < ne * NQ;
  const int pl = act ? lane : 0;  // idle lanes evaluate point 0 and store nothing
  const int el = pl / NQ, q = pl - el * NQ;
  double Jinv[9], det, Hd[9], Fd[9];
  tile_kinematics<Rule>(a, nod + 6 * NEN * el, terms + 2 * kT10Terms * el, e0 + el, q, Jinv, det, Hd, Fd);
  PointOut<R> o;
  const unsigned fl = point_update<R, true>(a.mp, Hd, Fd, det * Rule::w_rt(q), a.alpha, a.beta, o);
  if (act && fl) atomicOr(a.flags, fl);
  HatOut<R> h;
  to_parent<R, true, FuseT10Full>(o, Jinv, h);
  // 2. row by row
  R* rec = reinterpret_cast<R*>(smem);  // the nodal values are consumed
  const int eg = lane / (3 * HN), an = (lane - 3 * HN * eg) / 3, k = lane % 3;  // lanes 60 .. 63: eg = GRP, idle
  sfor<0, 3>([&](auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value;
    if (ONE && i != row) return;  // uniform
    wave_sync();  // the previous row's slots are consumed
    if (act) {
      R* r = rec + pl * RS;
      sfor<0, (3 * kSlot + PER - 1) / PER>([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        V v;
        sfor<0, PER>([&](auto xc) __attribute__((always_inline)) {
          constexpr int w = PER * j + decltype(xc)::value;
          if constexpr (w < 3 * kSlot) v[decltype(xc)::value] = record_value<3 * kSlot * i + w, FuseT10Full>(h);
          else v[decltype(xc)::value] = R(0);
        });
        *reinterpret_cast<V*>(r + PER * j) = v;
      });
    }
    wave_sync();
#pragma unroll 1
    for (int g0 = 0; g0 < ne; g0 += GRP) {
      const int ng = ne - g0 < GRP ? ne - g0 : GRP;  // elements of this group
      const int le = g0 + (eg < ng ? eg : 0);                    // idle lanes repeat a live element
      R acc[Z][NEN], facc[Z];
#pragma unroll
      for (int z = 0; z < Z; ++z) {
#pragma unroll
        for (int b = 0; b < NEN; ++b) acc[z][b] = R(0);
        facc[z] = R(0);
      }
      const R* base = rec + le * NQ * RS + kSlot * k;
      const R* da = dn + DL * an;
      sfor<0, NQ>([&](auto qc) __attribute__((always_inline)) {
        constexpr int qq = decltype(qc)::value;
        Slot<R, true> sv;
        load_slot<R, true>(base + qq * RS, sv);
#pragma unroll
        for (int z = 0; z < Z; ++z) {
          const R* d = da + DL * HN * z + 3 * qq;
          contract_point<Rule, R, true, true, qq, NEN>(sv, d[0], d[1], d[2], k, acc[z], facc[z]);
        }
      });
      R f1[Z], f2[Z];
#pragma unroll
      for (int z = 0; z < Z; ++z) {
        f1[z] = __shfl_down(facc[z], 1, 64);
        f2[z] = __shfl_down(facc[z], 2, 64);
      }
      wave_sync();  // the previous rows have left the buffer
      if (eg < ng) {
#pragma unroll
        for (int z = 0; z < Z; ++z) {
          R* row = stg + (NEN * eg + an + HN * z) * SS;
#pragma unroll
          for (int u = 0; u < NEN / 2; ++u) {
            R2 v;
            v[0] = acc[z][2 * u];
            v[1] = acc[z][2 * u + 1];
            *reinterpret_cast<R2*>(row + kSlot * k + 2 * u) = v;
          }
          if (k == 0) {
            R2 v;
            v[0] = (facc[z] + f1[z]) + f2[z];
            v[1] = R(0);
            *reinterpret_cast<R2*>(row + 3 * kSlot) = v;
          }
        }
      }
      wave_sync();
      constexpr int NP = kRowChunk / PER;  // pieces per row
#pragma unroll
      for (int u = 0; u < (GRP * NEN * NP + 63) / 64; ++u) {
        const int pc = lane + 64 * u, bl = pc / NP, pi = pc - bl * NP;
        if (bl < ng * NEN) {
          const R2* src = reinterpret_cast<const R2*>(stg + bl * SS + PER * pi);
          V v;
#pragma unroll
          for (int t = 0; t < PER; ++t) v[t] = src[t / 2][t % 2];
          store_piece<NT>(v, reinterpret_cast<V*>(rows + (int64_t)pos[g0 * NEN + bl] * kRowBlk + kRowChunk * i + PER * pi));
        }
      }
    }
  });
}

// ONE: a workgroup for each row component of a tile (grid y), which form the points'
// factors three times over: for a mesh that leaves most of the GPU idle the chain of
// one wave is what it waits for.
template <class Rule, typename R, bool NT, bool ONE = false>
__global__ __launch_bounds__(64, (row_min_waves<R>())) void k_elem_rows(AsmArgs a, int tile,
                                                                           const int32_t* __restrict__ incpos,
                                                                           R* __restrict__ rows) {
  const int64_t e0 = (int64_t)blockIdx.x * tile;
  elem_rows_tile<Rule, R, NT, ONE>(a, incpos, rows, e0, (int)(a.n_elem - e0 < tile ? a.n_elem - e0 : tile), blockIdx.y);
}

// many bodies: every body starts on a workgroup of its own, found by bisection
template <class Rule, typename R, bool NT>
__global__ __launch_bounds__(64, (row_min_waves<R>())) void k_elem_rows_batch(BatchArgs b) {
  const int64_t blk = blockIdx.x;
  int lo = 0, hi = b.n_bodies - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (b.bodies[mid].rblock_off <= blk) lo = mid; else hi = mid - 1;
  }
  const BatchBody& B = b.bodies[lo];
  const AsmArgs a = body_args(b, B, lo);
  const int64_t e0 = (blk - B.rblock_off) * b.row_tile;
  elem_rows_tile<Rule, R, NT>(a, B.incpos, (R*)b.stage + B.blk_inc_off * kRowBlk, e0,
                          (int)(a.n_elem - e0 < b.row_tile ? a.n_elem - e0 : b.row_tile));
}

// Persistent form of the batch (the LPT schedule): a grid sized to what the
// GPU holds at once, whose workgroups take (body, tile) items from a counter
// in a list ordered longest first (full tiles of the largest bodies first,
// partial tiles last), EB elements per tile, which the wave takes in equal parts.
template <class Rule, int EB, bool NT>
__global__ __launch_bounds__(64, 2) void k_elem_rows_batch_lpt(BatchArgs b, const int2* __restrict__ items,
                                                                    int n_items, unsigned* __restrict__ counter) {
  __shared__ int item;
  for (;;) {
    __syncthreads();  // the previous item's LDS and its item index are consumed
    if (threadIdx.x == 0) item = (int)atomicAdd(counter, 1u);
    __syncthreads();
    const int it = item;
    if (it >= n_items) return;  // every wave of the workgroup leaves here together
    const int2 t = items[it];
    const BatchBody& B = b.bodies[t.x];
    const AsmArgs a = body_args(b, B, t.x);
    constexpr int parts = (EB + kRowElems - 1) / kRowElems, step = (EB + parts - 1) / parts;
    const int64_t end = (int64_t)(t.y + 1) * EB < a.n_elem ? (int64_t)(t.y + 1) * EB : a.n_elem;
#pragma unroll 1
    for (int64_t e0 = (int64_t)t.y * EB; e0 < end; e0 += step) {
      wave_sync();  // the previous part's LDS is consumed
      elem_rows_tile<Rule, float, NT>(a, B.incpos, (float*)b.stage + B.blk_inc_off * kRowBlk, e0,
                                  (int)(end - e0 < step ? end - e0 : step));
    }
  }
}

__global__ void k_reset_counters(unsigned* counters) {
  if (threadIdx.x < 2) counters[threadIdx.x] = 0u;
}

// Pass 2 over the row blocks: a lane per (incidence, row i, component k) task
// of the range loads its ten K entries (aligned 16-byte pieces of the row:
// five in float64, three in float32, shifted by 2 values for k = 1) and adds
// them into the range's LDS segment at row + 3 rank_b + k; the force entry
// follows those of k = 2 (in float32 in the same piece).
template <typename R, bool WANT_F, bool WANT_K, bool ACCUM>
__device__ __forceinline__ void gather_rows(const GatherArgs& g, int32_t I0, int32_t I1, unsigned char* smem,
                                            int32_t* pre, int32_t* rowo) {
  constexpr int TPI = 9;
  const int tid = threadIdx.x;
  uint8_t* incn = smem;
  double* lds = reinterpret_cast<double*>(smem + g.inc_cap);
  const int nn = I1 - I0;
  const int64_t row0 = 3LL * I0, row1 = 3LL * I1;
  const int64_t seg0 = WANT_K ? g.row_off[row0] : 0, seg1 = WANT_K ? g.row_off[row1] : 0;
  const int nseg = (int)(seg1 - seg0);
  const int nrow = (int)(row1 - row0);
  double* lf = lds + nseg;
  for (int t = tid; t < nseg + nrow; t += blockDim.x) lds[t] = 0.0;
  const int32_t inc0 = g.inc_off[I0];
  for (int n = tid; n <= nn; n += blockDim.x) pre[n] = TPI * (g.inc_off[I0 + n] - inc0);
  if constexpr (WANT_K)
    for (int rr = tid; rr < nrow; rr += blockDim.x) rowo[rr] = (int32_t)(g.row_off[row0 + rr] - seg0);
  __syncthreads();
  for (int n = tid; n < nn; n += blockDim.x)
    for (int j = pre[n] / TPI; j < pre[n + 1] / TPI; ++j) incn[j] = (uint8_t)n;
  if constexpr (WANT_K) add_mass_term<1>(g, I0, nn, lds, rowo);
  __syncthreads();
  const int ntask = pre[nn];
  using V = typename Vec4<R>::type;
  constexpr int PER = (int)(sizeof(V) / sizeof(R)), NP = sizeof(R) == 4 ? 3 : kSlot / 2;
  const R* blk = reinterpret_cast<const R*>(g.stage);
  const V* blkv = reinterpret_cast<const V*>(g.stage);
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  for (int t = tid; t < ntask; t += blockDim.x) {
    const int jl = t / TPI, sl = t - TPI * jl, i = sl / 3, k = sl - 3 * i;
    const uint32_t j = (uint32_t)(inc0 + jl);
    const int rl = 3 * incn[jl] + i;
    if constexpr (WANT_K) {
      // 16-byte units with 32-bit offsets (checked on the host)
      const uint32_t p0 = j * (uint32_t)(kRowBlk / PER) + (uint32_t)((kRowChunk * i + kSlot * k) / PER);
      V w[NP];
#pragma unroll
      for (int u = 0; u < NP; ++u) w[u] = blkv[p0 + u];
      R fv = R(0);
      if constexpr (WANT_F) {
        if constexpr (sizeof(R) == 4) fv = w[2][2];
        else if (k == 2) fv = blkv[p0 + NP][0];
      }
      const u32x4 rw = *reinterpret_cast<const u32x4*>(g.rank + (size_t)j * 16);
      const bool odd = sizeof(R) == 4 && k == 1;
      double* dstp = lds + rowo[rl] + k;
#pragma unroll
      for (int b = 0; b < 10; ++b) {
        R v = w[b / PER][b % PER];
        if constexpr (sizeof(R) == 4) v = odd ? w[(b + 2) / PER][(b + 2) % PER] : v;
        const int rank_b = (int)((rw[b >> 2] >> (8 * (b & 3))) & 255u);
        atomicAdd(dstp + 3 * rank_b, (double)v);
      }
      if constexpr (WANT_F)
        if (k == 2) atomicAdd(lf + rl, (double)fv);
    } else {
      if (k == 0) atomicAdd(lf + rl, (double)blk[(size_t)j * kRowBlk + kRowChunk * i + 3 * kSlot]);
    }
  }
  __syncthreads();
  if constexpr (WANT_K) write_segment<ACCUM>(g, row0, nrow, nseg, seg0, lds, rowo);
  if constexpr (WANT_F) {
    double* out = g.f + row0;
    for (int t = tid; t < nrow; t += blockDim.x) out[t] = ACCUM ? out[t] + lf[t] : lf[t];
  }
}

template <typename R, bool WANT_F, bool WANT_K, bool ACCUM>
__global__ __launch_bounds__(512) void k_gather_rows(GatherArgs g) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t pre[kMaxRangeNodes + 1];
  __shared__ int32_t rowo[kMaxRangeNodes * 3];
  const int r = remap_tile(blockIdx.x, gridDim.x);
  gather_rows<R, WANT_F, WANT_K, ACCUM>(g, g.ranges[r], g.ranges[r + 1], smem, pre, rowo);
}

template <typename R>
__global__ __launch_bounds__(512) void k_gather_rows_batch(BatchArgs b) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t pre[kMaxRangeNodes + 1];
  __shared__ int32_t rowo[kMaxRangeNodes * 3];
  const int r = remap_tile(blockIdx.x, gridDim.x);
  const BatchRange br = b.ranges[r];
  const BatchBody& B = b.bodies[br.body];
  GatherArgs g{};
  g.inc_off = B.inc_off;
  g.row_off = B.row_off;
  g.rank = B.rank_inc;
  g.stage = (const R*)b.stage + B.blk_inc_off * kRowBlk;
  g.f = b.f + B.dof_off;
  g.vals = b.vals + B.nnz_off;
  g.inc_cap = b.inc_cap;
  gather_rows<R, true, true, false>(g, br.I0, br.I1, smem, pre, rowo);
}

// persistent form: ranges taken from a counter, largest first
__global__ __launch_bounds__(512) void k_gather_rows_batch_lpt(BatchArgs b, const int32_t* __restrict__ order,
                                                               int n_items, unsigned* __restrict__ counter) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t pre[kMaxRangeNodes + 1];
  __shared__ int32_t rowo[kMaxRangeNodes * 3];
  __shared__ int item;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) item = (int)atomicAdd(counter, 1u);
    __syncthreads();
    const int it = item;
    if (it >= n_items) return;
    const BatchRange br = b.ranges[order[it]];
    const BatchBody& B = b.bodies[br.body];
    GatherArgs g{};
    g.inc_off = B.inc_off;
    g.row_off = B.row_off;
    g.rank = B.rank_inc;
    g.stage = (const float*)b.stage + B.blk_inc_off * kRowBlk;
    g.f = b.f + B.dof_off;
    g.vals = b.vals + B.nnz_off;
    g.inc_cap = b.inc_cap;
    gather_rows<float, true, true, false>(g, br.I0, br.I1, smem, pre, rowo);
  }
}

// ---------------------------------------------------------------------------
// element rows for ANCF (four coefficient vectors per node)
// ---------------------------------------------------------------------------
// The same split as for T10, for the shell and the beam: pass 1 contracts an
// element's points itself and leaves one block per (element, node) incidence
// at the node's place in the node-sorted incidence list; pass 2 reads every
// block once.  Block of an incidence: for row r = 3 c + i (coefficient kind c
// of the node, component i) and column component k, the NEN entries
// K_e[(a, i), (b, k)] over the element's coefficients b at (3 r + k) NEN + b,
// then the parts P^_ik dN_a,k s_a of f_a,i at 36 NEN + 3 r + k (the three
// parts of a row are added in pass 2).
constexpr int kRowsMcThreads = 128;
// Three points a step instead of two: undamped, 500,000 beams 1,337 -> 1,327 us and
// 50,000 152.9 -> 151.1; the full form (damped) 1,772 -> 1,769 and 198.2 -> 200.3.
#ifndef TLFEA_ROWS_MC_UNROLL
#define TLFEA_ROWS_MC_UNROLL 3
#endif
constexpr int kRowsMcUnroll = TLFEA_ROWS_MC_UNROLL;  // points contracted per step (divides 12, 18 and 48)
template <class Rule>
constexpr int rows_mc_elems() { return kRowsMcThreads / Rule::NQ; }
template <int NEN>
constexpr int rows_mc_block() { return 36 * NEN + 36; }

// What phase B of the float64 form needs of its elements from global memory, read
// before the first store: loads and stores retire in one order, so a load between
// the stores of two tasks waits for the earlier ones to reach memory (pass 1 of
// 65,536 shells 718 us, so 611; the float32 forms, with more waves to change to,
// do not gain).
template <class Rule, int EB>
struct RowsOut {
  double sc[4 * EB];             // coefficient scales by kind
  int32_t ip[Rule::NPN * EB];    // places of the element's incidences
  __device__ __forceinline__ void fill(const AsmArgs& a, const int32_t* __restrict__ incpos, int64_t e0, int ne) {
    for (int t = threadIdx.x; t < Rule::NPN * ne; t += blockDim.x) ip[t] = incpos[e0 * Rule::NPN + t];
    for (int le = threadIdx.x; le < ne; le += blockDim.x) element_scales<Rule>(a, e0 + le, sc + 4 * le);
  }
};

// floats between the records of two elements of the symmetric vector form, whose
// lanes read the slots of up to three elements at once: 256-byte records alone would
// put the same slot of all of them into the same banks
constexpr int kElemPad = 12;

// Phase B of the ANCF element rows for a symmetric tangent (undamped
// materials): only the slots i <= k are contracted, a lane per task (element,
// slot, coefficient a), coefficients fastest.  A task writes its NEN entries
// K_e[(a, i), (b, k)] as in the full form and, for i < k, the same values as
// the entries K_e[(b, k), (a, i)] of the blocks of the column coefficients'
// nodes (the lanes of consecutive a write consecutive values), plus the force
// parts of rows i and, for i < k, k.  Two thirds of the full form's tasks.  A lane
// takes two consecutive coefficients, which share the slot's values.  Bound by
// vector issue (two thirds of the time: 3,190 instructions a wave, half of them
// the points') and LDS.  Pass 1 of 500,000 beams 800 -> 749 us, 30,000 65 -> 54,
// against one coefficient a lane with all gradients multiplied; blocks gathered in
// LDS and stored whole took longer (970; non-temporal 773, but then pass 2 waits).
// acc += sum over n of T_n dN_b,n(q) without the gradients that vanish at every
// point; the order and the separate last addition are those of the full sum
// ((t1 d1 + t0 d0) + t2 d2 with fused multiply-adds, then the accumulator), so the
// results are the same bits.
template <class Rule>
__device__ __forceinline__ void add_column(float& acc, float t0, float t1, float t2, int q, int b) {
#pragma clang fp contract(off)
  float s = Rule::grad_nz(b, 1) ? fmaf(t0, Rule::dNf_rt(q, b, 0), t1 * Rule::dNf_rt(q, b, 1)) : t0 * Rule::dNf_rt(q, b, 0);
  if (Rule::grad_nz(b, 2)) s = fmaf(t2, Rule::dNf_rt(q, b, 2), s);
  acc = acc + s;
}

template <class Rule, int EB>
__device__ __forceinline__ void rows_mc_sym_contract(const AsmArgs& a, const int32_t* __restrict__ incpos,
                                                     float* __restrict__ rows, int64_t e0, int ne, const float* rec,
                                                     const float* dn) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, NPN = Rule::NPN, Z = 2, NT = NEN / Z * 6;
  constexpr int BLK = rows_mc_block<NEN>();
  static_assert(Rule::grad_nz(0, 0) && Rule::grad_nz(1, 0) && Rule::grad_nz(2, 0) && Rule::grad_nz(3, 0), "first term");
  const int tid = threadIdx.x;
  const int ntask = ne * NT;
  for (int t0 = 0; t0 < EB * NT; t0 += kRowsMcThreads) {
    const int t = t0 + tid;
    const bool on = t < ntask;
    const int tt = on ? t : ntask - 1;
    const int le = tt / NT, r6 = tt - le * NT, us = r6 / (NEN / Z), al = Z * (r6 - us * (NEN / Z));
    const int i = us < 3 ? 0 : us < 5 ? 1 : 2, k = us < 3 ? us : us < 5 ? us - 2 : 2;
    const int so = kSlot * us, pt = 6 * kSlot + i + k - 1;  // the slot, Phat_ki (i < k)
    float acc[Z][NEN], facc[Z], ft[Z];
#pragma unroll
    for (int z = 0; z < Z; ++z) {
#pragma unroll
      for (int b = 0; b < NEN; ++b) acc[z][b] = 0.0f;
      facc[z] = ft[z] = 0.0f;
    }
    const float* recp = rec + le * (NQ * kRecS + kElemPad);
#pragma unroll 1
    for (int q0 = 0; q0 < NQ; q0 += kRowsMcUnroll) {
      sfor<0, kRowsMcUnroll>([&](auto uc) __attribute__((always_inline)) {
        const int qq = q0 + decltype(uc)::value;
        const float* r = recp + qq * kRecS;
        float v[10];
#pragma unroll
        for (int x = 0; x < 5; ++x) {
          const f32x2 w = *reinterpret_cast<const f32x2*>(r + so + 2 * x);
          v[2 * x] = w[0];
          v[2 * x + 1] = w[1];
        }
        const float pk = i < k ? r[pt] : 0.0f;
        const float* d = dn + 3 * (NEN * qq + al);
#pragma unroll
        for (int z = 0; z < Z; ++z) {
          const float d0 = d[3 * z], d1 = d[3 * z + 1], d2 = d[3 * z + 2];
          const float t0n = sum3<false>(v[0], d0, v[3], d1, v[6], d2);
          const float t1n = sum3<false>(v[1], d0, v[4], d1, v[7], d2);
          const float t2n = sum3<false>(v[2], d0, v[5], d1, v[8], d2);
          facc[z] += v[9] * (k == 0 ? d0 : k == 1 ? d1 : d2);
          ft[z] += pk * (i == 0 ? d0 : d1);
#pragma unroll
          for (int b = 0; b < NEN; ++b) add_column<Rule>(acc[z][b], t0n, t1n, t2n, qq, b);
        }
      });
    }
    if (on) {
      double sc[4];
      element_scales<Rule>(a, e0 + le, sc);
      const int32_t* ip = incpos + (e0 + le) * NPN;
      float sa[Z];
#pragma unroll
      for (int z = 0; z < Z; ++z) {
        const int c = (al + z) & 3, r = 3 * c + i;  // block row (kind, i)
        sa[z] = (float)(z == 0 ? ((al & 3) == 0 ? sc[0] : sc[2]) : ((al & 3) == 0 ? sc[1] : sc[3]));
        float* blk = rows + (int64_t)ip[al >> 2] * BLK;
        f32x4* outv = reinterpret_cast<f32x4*>(blk + (3 * r + k) * NEN);
#pragma unroll
        for (int u = 0; u < NEN / 4; ++u) {
          f32x4 w;
#pragma unroll
          for (int x = 0; x < 4; ++x) w[x] = acc[z][4 * u + x] * sa[z] * (float)sc[x];  // b = 4 u + x: kind x
          outv[u] = w;
        }
        blk[36 * NEN + 3 * r + k] = facc[z] * sa[z];
        if (i < k) blk[36 * NEN + 3 * (3 * c + k) + i] = ft[z] * sa[z];
      }
      if (i < k) {
#pragma unroll
        for (int nb = 0; nb < NPN; ++nb) {
          float* ob = rows + (int64_t)ip[nb] * BLK;
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            f32x2 w;
#pragma unroll
            for (int z = 0; z < Z; ++z) w[z] = acc[z][4 * nb + x] * sa[z] * (float)sc[x];
            *reinterpret_cast<f32x2*>(ob + (3 * (3 * x + k) + i) * NEN + al) = w;
          }
        }
      }
    }
  }
}

// Phase B of the shell's element rows on the matrix cores.  With
// D[(q,m), a] = dN_a,m(q) (the parent gradients, the same for every element)
// and T[(q,m), b] = sum_n Ahat_q,imkn dN_b,n(q), the slot (i, k) of K_e is the
// 16 x 16 product K^(ik) = D^T T over the 3 NQ values of (q, m): one MFMA tile,
// no padding in a or b (sixteen coefficients), the (q, m) axis padded to a
// multiple of four.  A wave takes one element at a time and runs the 16x16x4
// FP32 MFMA over the (q, m) axis in steps of four, for all the element's slots
// at once (independent accumulators, so the matrix-core chain of one slot
// overlaps the others); in each step lane l feeds D[(q,m), l % 16] and forms
// T[(q,m), l % 16] of every slot (three multiply-adds each from the LDS
// record), (q, m) = 4 step + l / 16.  Lane l then holds K^(ik)[4 (l / 16) +
// r][l % 16], r < 4, and stores them with the scales into the block of node
// l / 16 (rows of kind r); for a symmetric tangent (SYM: the six slots i <= k)
// a lane of a slot with i < k also stores its four values, consecutive in a,
// as K_e[(b, k), (a, i)] into the block of the column's node.  The force parts
// are spread over the four lane groups (a quarter of the points each) and
// summed in a fixed order.
template <bool SYM, int S>
struct McSlot {
  static constexpr int i = SYM ? (S < 3 ? 0 : S < 5 ? 1 : 2) : S / 3;
  static constexpr int k = SYM ? (S < 3 ? S : S < 5 ? S - 2 : 2) : S % 3;
  static constexpr int off = SYM ? kSlot * S : kSlot * (3 * i + k);
};

template <class Rule, int EB, bool SYM>
__device__ __forceinline__ void rows_mc_mfma_contract(const AsmArgs& a, const int32_t* __restrict__ incpos,
                                                      float* __restrict__ rows, int64_t e0, int ne, const float* rec,
                                                      const float* dn) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, NPN = Rule::NPN, BLK = rows_mc_block<NEN>();
  static_assert(NEN == 16, "one 16 x 16 tile per slot");
  constexpr int RS = SYM ? kRecSL : kRecL;
  constexpr int KK = 3 * NQ, NSTEP = (KK + 3) / 4, NSL = SYM ? 6 : 9, NW = kRowsMcThreads / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c16 = lane & 15;
  for (int le = wave; le < ne; le += NW) {  // uniform per wave
    const float* re = rec + le * NQ * RS;
    f32x4 acc[NSL];
#pragma unroll
    for (int t = 0; t < NSL; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 2
    for (int st = 0; st < NSTEP; ++st) {
      const int kk = 4 * st + g;
      const bool live = kk < KK;
      const int q = live ? kk / 3 : 0, m = kk - 3 * q;
      const float* d = dn + 3 * (NEN * q + c16);  // dN_c16(q)
      const float d0 = d[0], d1 = d[1], d2 = d[2];
      const float av = live ? (m == 0 ? d0 : m == 1 ? d1 : d2) : 0.0f;
      const float* r = re + q * RS + 3 * (live ? m : 0);
      sfor<0, NSL>([&](auto sc_) __attribute__((always_inline)) {
        constexpr int S = decltype(sc_)::value;
        constexpr int off = McSlot<SYM, S>::off;
        const float bv = r[off] * d0 + r[off + 1] * d1 + r[off + 2] * d2;
        acc[S] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[S], 0, 0, 0);
      });
    }
    // force parts of node c16: Phat_ik dN_c16,k (and Phat_ki dN_c16,i for i < k), a quarter of the points per group
    float fd[NSL], ft[3];
#pragma unroll
    for (int t = 0; t < NSL; ++t) fd[t] = 0.0f;
#pragma unroll
    for (int t = 0; t < 3; ++t) ft[t] = 0.0f;
    for (int q = g; q < NQ; q += 4) {
      const float* d = dn + 3 * (NEN * q + c16);
      const float* r = re + q * RS;
      sfor<0, NSL>([&](auto sc_) __attribute__((always_inline)) {
        constexpr int S = decltype(sc_)::value, i = McSlot<SYM, S>::i, k = McSlot<SYM, S>::k;
        fd[S] += r[McSlot<SYM, S>::off + 9] * d[k];
        if constexpr (SYM && i < k) ft[i + k - 1] += r[6 * kSlot + i + k - 1] * d[i];
      });
    }
#pragma unroll
    for (int t = 0; t < NSL; ++t)
      fd[t] = ((fd[t] + __shfl_down(fd[t], 16, 64)) + __shfl_down(fd[t], 32, 64)) + __shfl_down(fd[t], 48, 64);
#pragma unroll
    for (int t = 0; t < 3; ++t)
      ft[t] = ((ft[t] + __shfl_down(ft[t], 16, 64)) + __shfl_down(ft[t], 32, 64)) + __shfl_down(ft[t], 48, 64);
    double sc[4];
    element_scales<Rule>(a, e0 + le, sc);
    const int32_t* ip = incpos + (e0 + le) * NPN;
    const float sb = (float)sc[c16 & 3], sa = sb;  // column scale of b = c16; row scale of a = c16 (forces)
    float* blk = rows + (int64_t)ip[g] * BLK;      // node of the rows a = 4 g + r
    float* cb = rows + (int64_t)ip[c16 >> 2] * BLK;  // node of coefficient c16
    sfor<0, NSL>([&](auto sc_) __attribute__((always_inline)) {
      constexpr int S = decltype(sc_)::value, i = McSlot<SYM, S>::i, k = McSlot<SYM, S>::k;
#pragma unroll
      for (int r = 0; r < 4; ++r) blk[(3 * (3 * r + i) + k) * NEN + c16] = acc[S][r] * (float)sc[r] * sb;
      if (g == 0) {
        cb[36 * NEN + 3 * (3 * (c16 & 3) + i) + k] = fd[S] * sa;
        if constexpr (SYM && i < k) cb[36 * NEN + 3 * (3 * (c16 & 3) + k) + i] = ft[i + k - 1] * sa;
      }
      if constexpr (SYM && i < k) {
        f32x4 w;
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = acc[S][r] * (float)sc[r] * sb;
        *reinterpret_cast<f32x4*>(cb + (3 * (3 * (c16 & 3) + k) + i) * NEN + 4 * g) = w;
      }
    });
  }
}

template <class Rule, bool SYM, bool MF>
__device__ __forceinline__ void elem_rows_mc_tile(const AsmArgs& a, const int32_t* __restrict__ incpos,
                                                  float* __restrict__ rows, int64_t blk) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, NPN = Rule::NPN, EB = rows_mc_elems<Rule>();
  constexpr int BLK = rows_mc_block<NEN>();
  constexpr int RS = SYM ? (MF ? kRecSL : kRecS) : kRecL;  // LDS record stride (symmetric layout for undamped materials)
  static_assert(Rule::MC == 4 && NEN % 4 == 0 && EB >= 1, "element rows of four-coefficient nodes");
  constexpr int PAD = SYM && !MF ? kElemPad : 0;
  constexpr size_t NOD = (size_t)EB * NEN * 6 * sizeof(double), REC = (size_t)EB * (NQ * RS + PAD) * sizeof(float);
  __shared__ __align__(16) unsigned char smem[NOD > REC ? NOD : REC];
  __shared__ float dn[NQ * NEN * 3];  // unit-scaled parent gradients, dN_a(q)_m at 3 (NEN q + a) + m
  const int tid = threadIdx.x;
  const int64_t e0 = blk * EB;
  const int ne = (int)(a.n_elem - e0 < EB ? a.n_elem - e0 : EB);
  double* nod = reinterpret_cast<double*>(smem);
  gather_nodal<Rule>(a, e0, ne, nod);
  for (int idx = tid; idx < NQ * NEN * 3; idx += kRowsMcThreads) {
    const int q = idx / (3 * NEN), r = idx - 3 * NEN * q;
    dn[idx] = Rule::dNf_rt(q, r / 3, r % 3);
  }
  __syncthreads();
  // 1. a lane per point: kinematics, constitutive update, the point's record
  //    (the tangent-record layout of the point-record path) into LDS
  const bool act = tid < ne * NQ;
  const int pl = act ? tid : 0;  // idle lanes evaluate point 0 and store nothing
  const int el = pl / NQ, q = pl - el * NQ;
  double Jinv[9], det, Hd[9], Fd[9];
  tile_kinematics<Rule>(a, nod + 6 * NEN * el, nullptr, e0 + el, q, Jinv, det, Hd, Fd);
  __syncthreads();  // the nodal values are consumed: the LDS holds the records from here on
  PointOut<float> o;
  const unsigned fl = point_update<float, true>(a.mp, Hd, Fd, det * Rule::w_rt(q), a.alpha, a.beta, o);
  if (act && fl) atomicOr(a.flags, fl);
  using FO = std::conditional_t<!SYM && NEN == 8, FuseBeamFull, FuseOther>;
  HatOut<float> h;
  to_parent<float, true, FO>(o, Jinv, h);
  float* rec = reinterpret_cast<float*>(smem);
  if (act) {
    float* r = rec + pl * RS + el * PAD;
    sfor<0, (SYM ? kRecS : kRecL) / 4>([&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value;
      f32x4 v;
      sfor<0, 4>([&](auto xc) __attribute__((always_inline)) {
        constexpr int x = decltype(xc)::value;
        if constexpr (SYM) v[x] = record_value_sym<4 * j + x>(h);
        else v[x] = record_value<4 * j + x, FO>(h);
      });
      *reinterpret_cast<f32x4*>(r + 4 * j) = v;
    });
  }
  __syncthreads();
  if constexpr (MF) {
    rows_mc_mfma_contract<Rule, EB, SYM>(a, incpos, rows, e0, ne, rec, dn);
  } else if constexpr (SYM) {
    rows_mc_sym_contract<Rule, EB>(a, incpos, rows, e0, ne, rec, dn);
  } else {
    // 2. a lane per task (element, coefficient a, row i, component k), tasks in
    //    block order; the point loop is uniform across the workgroup, so the
    //    gradients dN_b(q) of the columns come through the scalar cache
    const int ntask = ne * NEN * 9;
    for (int t0 = 0; t0 < EB * NEN * 9; t0 += kRowsMcThreads) {
      const int t = t0 + tid;
      const bool on = t < ntask;
      const int tt = on ? t : ntask - 1;
      const int le = tt / (NEN * 9), r9 = tt - le * NEN * 9, al = r9 / 9, s = r9 - 9 * al;  // s = 3 i + k
      const int k = s % 3;
      float acc[NEN];
#pragma unroll
      for (int b = 0; b < NEN; ++b) acc[b] = 0.0f;
      float facc = 0.0f;
      const float* recp = rec + le * NQ * RS + kSlot * s;
      static_assert(NQ % kRowsMcUnroll == 0, "point steps tile the rule");
#pragma unroll 1
      for (int q0 = 0; q0 < NQ; q0 += kRowsMcUnroll) {
        sfor<0, kRowsMcUnroll>([&](auto uc) __attribute__((always_inline)) {
          const int qq = q0 + decltype(uc)::value;
          Slot<float, true> sv;
          load_slot<float, true>(recp + qq * RS, sv);
          const float(&v)[10] = sv.v;
          const float* d = dn + 3 * (NEN * qq + al);
          const float d0 = d[0], d1 = d[1], d2 = d[2];
          const float t0n = v[0] * d0 + v[3] * d1 + v[6] * d2;
          const float t1n = v[1] * d0 + v[4] * d1 + v[7] * d2;
          const float t2n = v[2] * d0 + v[5] * d1 + v[8] * d2;
          facc += v[9] * (k == 0 ? d0 : k == 1 ? d1 : d2);
#pragma unroll
          for (int b = 0; b < NEN; ++b)
            acc[b] += t0n * Rule::dNf_rt(qq, b, 0) + t1n * Rule::dNf_rt(qq, b, 1) + t2n * Rule::dNf_rt(qq, b, 2);
        });
      }
      if (on) {
        double sc[4];
        element_scales<Rule>(a, e0 + le, sc);
        const float s_a = (float)sc[al & 3];
        const int64_t pos = incpos[(e0 + le) * NPN + (al >> 2)];
        const int r = 3 * (al & 3) + s / 3;  // block row (kind, i)
        float* blk = rows + pos * BLK;
        f32x4* outv = reinterpret_cast<f32x4*>(blk + (3 * r + k) * NEN);
#pragma unroll
        for (int u = 0; u < NEN / 4; ++u) {
          f32x4 w;
#pragma unroll
          for (int x = 0; x < 4; ++x) w[x] = acc[4 * u + x] * s_a * (float)sc[x];  // b = 4 u + x: kind x
          outv[u] = w;
        }
        blk[36 * NEN + 3 * r + k] = facc * s_a;
      }
    }
  }
}

template <class Rule, bool SYM, bool MF>
__global__ __launch_bounds__(kRowsMcThreads) void k_elem_rows_mc(AsmArgs a, const int32_t* __restrict__ incpos,
                                                                 float* __restrict__ rows) {
  elem_rows_mc_tile<Rule, SYM, MF>(a, incpos, rows, blockIdx.x);
}

// many bodies: every body starts on a workgroup of its own, found by bisection;
// the full tangent layout (the bodies' materials may differ)
template <class Rule, bool MF>
__global__ __launch_bounds__(kRowsMcThreads) void k_elem_rows_mc_batch(BatchArgs b) {
  const int64_t blk = blockIdx.x;
  int lo = 0, hi = b.n_bodies - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (b.bodies[mid].rblock_off <= blk) lo = mid; else hi = mid - 1;
  }
  const BatchBody& B = b.bodies[lo];
  const AsmArgs a = body_args(b, B, lo);
  elem_rows_mc_tile<Rule, false, MF>(a, B.incpos, (float*)b.stage + B.blk_inc_off * rows_mc_block<Rule::NEN>(),
                                     blk - B.rblock_off);
}

// The float64 form.  A point's tangent takes 250 registers, so two waves run per
// SIMD, and as for T10 the factors stay in registers and LDS holds the slots of
// one row component i at a time (240 bytes per point).  Elements per workgroup:
// whole elements in one wave (beam, 60 lanes), two (3x3x2 shell, 126) or four
// (4x4x3, 240).  Against point records, which pass 2 read once per node of the
// element, the whole call: 500,000 beams 2,825 -> 2,140 us, 65,536 3x3x2 shells
// 1,166 -> 1,003 (damped 1,510 -> 1,068), 10,000 4x4x3 shells 434 -> 257 (605 ->
// 291).  Bound by the phases in turn, which two waves overlap little: of the
// beams' 1,343 us in pass 1 the points take 380, the contraction 380 and the
// 2.6 GB of stores the rest; of the 65,536 shells' 611 the points take 290.
template <class Rule>
constexpr int rows64_threads() { return Rule::NQ == 48 ? 256 : Rule::NQ == 18 ? 128 : 64; }
template <class Rule>
constexpr int rows64_elems() { return rows64_threads<Rule>() / Rule::NQ; }

// Value of lane C of the lane's row of 16.
template <int C>
__device__ __forceinline__ double row_lane(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + C, 0xf, 0xf, true);
}

// One row component i of the beam's elements: a lane per (element, component k,
// kind of coefficient) takes the coefficients of both nodes, which reads a slot
// once for two rows, over all points.  The column gradients are wave-uniform and
// come through the scalar cache; those that vanish at every point are skipped.
// The rows go through LDS, so that a store writes 192 consecutive bytes (straight
// from the lanes, 16 bytes every 64: pass 1 1,381 us, with non-temporal stores
// 3,700; through LDS 1,343).
template <class Rule, int I, int EB>
__device__ __forceinline__ void rows64_vector(const RowsOut<Rule, EB>& ro, double* __restrict__ rows, int ne,
                                              double* rec, const double* dn, double* fst) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, NPN = Rule::NPN, TH = rows64_threads<Rule>();
  constexpr int BLK = rows_mc_block<NEN>(), RS = 3 * kSlot, Z = 2, NA = NEN / Z;
  const int tid = threadIdx.x, ntask = ne * NA * 3;
  static_assert(EB * NA * 3 <= TH, "a lane per task");
  {
    const bool on = tid < ntask;
    const int t = on ? tid : ntask - 1;
    const int le = t / (3 * NA), r = t - 3 * NA * le, al = r / 3, k = r - 3 * al;
    double acc[Z][NEN], facc[Z];
#pragma unroll
    for (int z = 0; z < Z; ++z) {
#pragma unroll
      for (int b = 0; b < NEN; ++b) acc[z][b] = 0.0;
      facc[z] = 0.0;
    }
    const double* recp = rec + le * NQ * RS + kSlot * k;
#pragma unroll 2
    for (int qq = 0; qq < NQ; ++qq) {
      Slot<double, true> sv;
      load_slot<double, true>(recp + qq * RS, sv);
#pragma unroll
      for (int z = 0; z < Z; ++z) {
        const double* d = dn + NEN * qq + al + NA * z;
        const double d0 = d[0], d1 = d[NEN * NQ], d2 = d[2 * NEN * NQ];
        double tn[3];
#pragma unroll
        for (int n = 0; n < 3; ++n) tn[n] = sv.v[n] * d0 + sv.v[3 + n] * d1 + sv.v[6 + n] * d2;
        facc[z] += sv.v[9] * (k == 0 ? d0 : k == 1 ? d1 : d2);
#pragma unroll
        for (int b = 0; b < NEN; ++b)
#pragma unroll
          for (int n = 0; n < 3; ++n)
            if (Rule::grad_nz(b, n)) acc[z][b] += tn[n] * Rule::dN_rt(qq, b, n);
      }
    }
    const double* sc = ro.sc + 4 * le;
    __syncthreads();  // the slots are consumed: the LDS takes the block rows [element][coefficient][k][b]
    if (on) {
#pragma unroll
      for (int z = 0; z < Z; ++z) {
        const int az = al + NA * z;
        const double s_a = sc[az & 3];
#pragma unroll
        for (int u = 0; u < NEN / 2; ++u) {
          f64x2 w;
          w[0] = acc[z][2 * u] * s_a * sc[(2 * u) % 4];
          w[1] = acc[z][2 * u + 1] * s_a * sc[(2 * u + 1) % 4];
          *reinterpret_cast<f64x2*>(rec + ((le * NEN + az) * 3 + k) * NEN + 2 * u) = w;
        }
        fst[(le * NEN + az) * 9 + 3 * I + k] = facc[z] * s_a;
      }
    }
    __syncthreads();
    constexpr int PR = 3 * NEN / 2;  // pairs per row
    for (int p = tid; p < ne * NEN * PR; p += TH) {
      const int ra = p / PR, x = p - ra * PR, az = ra & (NEN - 1);
      double* o = rows + (int64_t)ro.ip[ra >> 2] * BLK + (3 * (az & 3) + I) * 3 * NEN + 2 * x;
      const f64x2 w = *reinterpret_cast<const f64x2*>(rec + ra * 3 * NEN + 2 * x);
      *reinterpret_cast<f64x2*>(o) = w;
    }
    if (I == 2)
      for (int p = tid; p < ne * NPN * 18; p += TH) {
        const int in = p / 18, x = p - in * 18;
        const f64x2 w = *reinterpret_cast<const f64x2*>(fst + in * 36 + 2 * x);
        f64x2* o = reinterpret_cast<f64x2*>(rows + (int64_t)ro.ip[in] * BLK + 36 * NEN + 2 * x);
        *o = w;
      }
  }
}

// One row component i of the shell's elements on the matrix cores: a wave takes
// the 16 x 16 tile K^(ik)_ab = sum over (q, n) of T_n(q)[a] dN_b,n(q), T_n(q)[a] =
// sum_m Ahat_q,imkn dN_a,m(q), as 16x16x4 products over four points per n (the
// point axis is padded to a multiple of four with zeros).  Lane l takes position
// p = l % 16 of both sides at point l / 16 of the four: the three gradients it reads
// serve as A's factor and as B, and a slot value is read once per row of 16 lanes
// and passed along the row, so a step reads four doubles per lane for three
// products (the vector form: thirteen for 57 multiply-adds, bound by LDS; pass 1 of 65,536
// 3x3x2 shells 835 us, so 611).  For an undamped material the slots i <= k alone
// are multiplied and stored a second time, transposed.
// Position p stands for coefficient 4 (p % 4) + p / 4.  The product leaves lane l the
// rows at positions l / 16 + 4 r, r < 4, of column position l % 16: coefficients
// 4 (l / 16) + r, so a lane holds the four kinds of node l / 16, whose transposed
// entries are consecutive in a block.
template <class Rule, bool SYM, int I, int EB>
__device__ __forceinline__ void rows64_matrix(const RowsOut<Rule, EB>& ro, double* __restrict__ rows, int ne,
                                              const double* rec, const double* dn) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, NPN = Rule::NPN, NW = rows64_threads<Rule>() / 64;
  constexpr int BLK = rows_mc_block<NEN>(), RS = 3 * kSlot, NG = (NQ + 3) / 4;
  static_assert(NEN == 16 && NPN == 4, "one 16 x 16 tile per slot");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = 4 * (lane & 3) + ((lane >> 2) & 3);
  const int sl = (lane & 15) < kSlot ? lane & 15 : kSlot - 1;
#pragma unroll 1
  for (int t = wave; t < 3 * ne; t += NW) {  // uniform per wave
    const int kk = t / ne, le = t - kk * ne;
    const int k = I + kk < 3 ? I + kk : I + kk - 3;  // the slots k >= i first
    const bool tile = !SYM || k >= I;
    const double* re = rec + le * NQ * RS + kSlot * k + sl;
    f64x4 acc{0.0, 0.0, 0.0, 0.0};
    double facc = 0.0;
    double d[3], v;
    auto load = [&](int gq) __attribute__((always_inline)) {
      const int q = 4 * gq + g;
      const bool live = NQ % 4 == 0 || q < NQ;
      const int qc = live ? q : NQ - 1;
      const double* p = dn + NEN * qc + c;
#pragma unroll
      for (int m = 0; m < 3; ++m) d[m] = p[m * NEN * NQ];
      v = re[qc * RS];
      if (!live) {
        v = 0.0;
#pragma unroll
        for (int m = 0; m < 3; ++m) d[m] = 0.0;
      }
    };
    load(0);
#pragma unroll 4
    for (int gq = 0; gq < NG; ++gq) {
      const double d0 = d[0], d1 = d[1], d2 = d[2], vv = v;
      if (gq + 1 < NG) load(gq + 1);
      facc += row_lane<9>(vv) * (k == 0 ? d0 : k == 1 ? d1 : d2);
      if (tile) {
        const double t0 = row_lane<0>(vv) * d0 + row_lane<3>(vv) * d1 + row_lane<6>(vv) * d2;
        const double t1 = row_lane<1>(vv) * d0 + row_lane<4>(vv) * d1 + row_lane<7>(vv) * d2;
        const double t2 = row_lane<2>(vv) * d0 + row_lane<5>(vv) * d1 + row_lane<8>(vv) * d2;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(t0, d0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(t1, d1, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(t2, d2, acc, 0, 0, 0);
      }
    }
    facc += __shfl_xor(facc, 16);
    facc += __shfl_xor(facc, 32);
    const double* sc = ro.sc + 4 * le;
    const int kc = c & 3;
    const double s_c = sc[kc];
    const int32_t* ip = ro.ip + NPN * le;
    if (tile) {
      double* ob = rows + (int64_t)ip[g] * BLK + (3 * I + k) * NEN + c;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[r] *= sc[r] * s_c;
        ob[9 * NEN * r] = acc[r];
      }
      if (SYM && k > I) {
        f64x2* tb = reinterpret_cast<f64x2*>(rows + (int64_t)ip[c >> 2] * BLK + (3 * (3 * kc + k) + I) * NEN + 4 * g);
        tb[0] = f64x2{acc[0], acc[1]};
        tb[1] = f64x2{acc[2], acc[3]};
      }
    }
    if (g == 0) rows[(int64_t)ip[c >> 2] * BLK + 36 * NEN + 3 * (3 * kc + I) + k] = facc * s_c;
  }
}

template <class Rule, bool SYM>
__device__ __forceinline__ void elem_rows_mc64_tile(const AsmArgs& a, const int32_t* __restrict__ incpos,
                                                    double* __restrict__ rows, int64_t blk) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, TH = rows64_threads<Rule>(), EB = rows64_elems<Rule>();
  constexpr int RS = 3 * kSlot;
  static_assert(Rule::MC == 4 && EB >= 1 && NQ % 2 == 0, "element rows of four-coefficient nodes");
  constexpr size_t NOD = (size_t)EB * NEN * 6, REC = (size_t)EB * NQ * RS;
  __shared__ __align__(16) double smem[NOD > REC ? NOD : REC];
  __shared__ __align__(16) double fst[NEN == 16 ? 2 : EB * NEN * 9];  // force parts
  __shared__ double dn[3 * NQ * NEN];  // unit-scaled parent gradients, dN_a(q)_m at NEN (NQ m + q) + a
  const int tid = threadIdx.x;
  const int64_t e0 = blk * EB;
  const int ne = (int)(a.n_elem - e0 < EB ? a.n_elem - e0 : EB);
  __shared__ RowsOut<Rule, EB> ro;
  ro.fill(a, incpos, e0, ne);
  gather_nodal<Rule>(a, e0, ne, smem);
  for (int idx = tid; idx < NQ * NEN * 3; idx += TH) {
    const int m = idx / (NQ * NEN), r = idx - m * NQ * NEN;
    dn[idx] = Rule::dN_rt(r / NEN, r % NEN, m);
  }
  __syncthreads();
  const bool act = tid < ne * NQ;
  const int pl = act ? tid : 0;  // idle lanes evaluate point 0 and store nothing
  const int el = pl / NQ, q = pl - el * NQ;
  double Jinv[9], det, Hd[9], Fd[9];
  tile_kinematics<Rule>(a, smem + 6 * NEN * el, nullptr, e0 + el, q, Jinv, det, Hd, Fd);
  PointOut<double> o;
  const unsigned fl = point_update<double, true>(a.mp, Hd, Fd, det * Rule::w_rt(q), a.alpha, a.beta, o);
  if (act && fl) atomicOr(a.flags, fl);
  HatOut<double> h;
  to_parent<double, true>(o, Jinv, h);
  sfor<0, 3>([&](auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value;
    __syncthreads();  // the nodal values, or the previous component's slots, are consumed
    if (act) {
      double* r = smem + pl * RS;
      if constexpr (SYM && i > 0) {  // of the slots k < i the force part alone
#pragma unroll
        for (int k = 0; k < i; ++k) r[kSlot * k + 9] = h.P[3 * i + k];
      }
      sfor<(SYM ? i * kSlot / 2 : 0), RS / 2>([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        f64x2 v;
        v[0] = record_value<3 * kSlot * i + 2 * j, FuseOther>(h);
        v[1] = record_value<3 * kSlot * i + 2 * j + 1, FuseOther>(h);
        *reinterpret_cast<f64x2*>(r + 2 * j) = v;
      });
    }
    __syncthreads();
    if constexpr (NEN == 16) rows64_matrix<Rule, SYM, i>(ro, rows, ne, smem, dn);
    else rows64_vector<Rule, i>(ro, rows, ne, smem, dn, fst);
  });
}

template <class Rule, bool SYM>
__global__ __launch_bounds__(rows64_threads<Rule>(), 2) void k_elem_rows_mc64(AsmArgs a,
                                                                              const int32_t* __restrict__ incpos,
                                                                              double* __restrict__ rows) {
  elem_rows_mc64_tile<Rule, SYM>(a, incpos, rows, blockIdx.x);
}

template <class Rule>
__global__ __launch_bounds__(rows64_threads<Rule>(), 2) void k_elem_rows_mc64_batch(BatchArgs b) {
  const int64_t blk = blockIdx.x;
  int lo = 0, hi = b.n_bodies - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (b.bodies[mid].rblock_off <= blk) lo = mid; else hi = mid - 1;
  }
  const BatchBody& B = b.bodies[lo];
  const AsmArgs a = body_args(b, B, lo);
  elem_rows_mc64_tile<Rule, false>(a, B.incpos, (double*)b.stage + B.blk_inc_off * rows_mc_block<Rule::NEN>(),
                            blk - B.rblock_off);
}

// Pass 2 over the ANCF row blocks: a lane per (incidence, row r, component k)
// loads its NEN entries (16-byte pieces) and its element's rank row (4 bytes,
// element order), and adds them into the range's LDS segment at
// row + 3 (4 rank_b + c_b) + k; every lane adds its force part to the row.
template <class Rule, typename R, bool WANT_F, bool WANT_K, bool ACCUM>
__device__ __forceinline__ void gather_rows_mc(const GatherArgs& g, int32_t I0, int32_t I1, unsigned char* smem,
                                               int32_t* pre, int32_t* rowo) {
  constexpr int NEN = Rule::NEN, NPN = Rule::NPN, MC = 4, RPN = 3 * MC, TPI = 9 * MC;
  constexpr int BLK = rows_mc_block<NEN>();
  const int tid = threadIdx.x;
  uint8_t* incn = smem;
  double* lds = reinterpret_cast<double*>(smem + g.inc_cap);
  const int nn = I1 - I0;
  const int64_t row0 = (int64_t)RPN * I0, row1 = (int64_t)RPN * I1;
  const int64_t seg0 = WANT_K ? g.row_off[row0] : 0, seg1 = WANT_K ? g.row_off[row1] : 0;
  const int nseg = (int)(seg1 - seg0);
  const int nrow = (int)(row1 - row0);
  double* lf = lds + nseg;
  for (int t = tid; t < nseg + nrow; t += blockDim.x) lds[t] = 0.0;
  const int32_t inc0 = g.inc_off[I0];
  for (int n = tid; n <= nn; n += blockDim.x) pre[n] = TPI * (g.inc_off[I0 + n] - inc0);
  if constexpr (WANT_K)
    for (int rr = tid; rr < nrow; rr += blockDim.x) rowo[rr] = (int32_t)(g.row_off[row0 + rr] - seg0);
  __syncthreads();
  for (int n = tid; n < nn; n += blockDim.x)
    for (int j = pre[n] / TPI; j < pre[n + 1] / TPI; ++j) incn[j] = (uint8_t)n;
  if constexpr (WANT_K) add_mass_term<MC>(g, I0, nn, lds, rowo);
  __syncthreads();
  const int ntask = pre[nn];
  using V = typename Vec4<R>::type;
  constexpr int PER = (int)(sizeof(V) / sizeof(R));
  const R* blk = reinterpret_cast<const R*>(g.stage);
  for (int t = tid; t < ntask; t += blockDim.x) {
    const int jl = t / TPI, sl = t - TPI * jl, r = sl / 3, k = sl - 3 * r;
    const int64_t j = inc0 + jl;
    const int rl = RPN * incn[jl] + r;
    const R* bj = blk + j * BLK;
    if constexpr (WANT_K) {
      R val[NEN];
      const V* p = reinterpret_cast<const V*>(bj + (3 * r + k) * NEN);
#pragma unroll
      for (int u = 0; u < NEN / PER; ++u) {
        const V w = p[u];
#pragma unroll
        for (int x = 0; x < PER; ++x) val[PER * u + x] = w[x];
      }
      const int32_t v = g.inc[j];
      const int64_t ea = (int64_t)(v >> 4) * NPN + (v & 15);
      const uint32_t rw = *reinterpret_cast<const uint32_t*>(g.rank + ea * rank_stride(NPN));
      double* dstp = lds + rowo[rl] + k;
#pragma unroll
      for (int b = 0; b < NEN; ++b) {
        const int rank_b = (int)((rw >> (8 * (b >> 2))) & 255u);
        atomicAdd(dstp + 3 * (MC * rank_b + (b & 3)), (double)val[b]);
      }
    }
    if constexpr (WANT_F) atomicAdd(lf + rl, (double)bj[36 * NEN + 3 * r + k]);
  }
  __syncthreads();
  if constexpr (WANT_K) write_segment<ACCUM>(g, row0, nrow, nseg, seg0, lds, rowo);
  if constexpr (WANT_F) {
    double* out = g.f + row0;
    for (int t = tid; t < nrow; t += blockDim.x) out[t] = ACCUM ? out[t] + lf[t] : lf[t];
  }
}

template <class Rule, typename R, bool WANT_F, bool WANT_K, bool ACCUM>
__global__ __launch_bounds__(512) void k_gather_rows_mc(GatherArgs g) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t pre[kMaxRangeNodes + 1];
  __shared__ int32_t rowo[kMaxRangeNodes * 12];
  const int r = remap_tile(blockIdx.x, gridDim.x);
  gather_rows_mc<Rule, R, WANT_F, WANT_K, ACCUM>(g, g.ranges[r], g.ranges[r + 1], smem, pre, rowo);
}

template <class Rule, typename R>
__global__ __launch_bounds__(512) void k_gather_rows_mc_batch(BatchArgs b) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t pre[kMaxRangeNodes + 1];
  __shared__ int32_t rowo[kMaxRangeNodes * 12];
  const int r = remap_tile(blockIdx.x, gridDim.x);
  const BatchRange br = b.ranges[r];
  const BatchBody& B = b.bodies[br.body];
  GatherArgs g{};
  g.inc_off = B.inc_off;
  g.inc = B.inc;
  g.row_off = B.row_off;
  g.rank = B.rank;
  g.stage = (const R*)b.stage + B.blk_inc_off * rows_mc_block<Rule::NEN>();
  g.f = b.f + B.dof_off;
  g.vals = b.vals + B.nnz_off;
  g.inc_cap = b.inc_cap;
  gather_rows_mc<Rule, R, true, true, false>(g, br.I0, br.I1, smem, pre, rowo);
}

// ---------------------------------------------------------------------------
// internal force alone (every element type)
// ---------------------------------------------------------------------------
// Pass 1 keeps each element's points in one workgroup: a lane per point forms
// Phat = dV P J0^-T (Sec. 4.3, Stage 1) into LDS, then a lane per (element,
// coefficient a) sums f_a = sum_q Phat_q dN_a(q) s_a over the element's points
// (Eq. fint_local, in the record precision) and writes the three values to the
// node-sorted incidence position of (element, node of a), 3 MC values per
// incidence.  Pass 2 adds each pattern node's incidence blocks in a fixed order,
// a lane per row of f, in float64: no atomics, the same sums on every call.
// Bound by instruction issue (about 900 per point, a third of them float64).
// 480,000 T10, mixed: 0.156 ms a call with the kinematics as a sum over ten
// nodes (132 VGPRs), 0.115 ms with the element terms of kernel_common.h (108
// VGPRs, four waves per SIMD).
constexpr int kForceThreads = 256;
template <class Rule>
constexpr int force_elems() { return kForceThreads / Rule::NQ; }
// waves per SIMD the registers allow without spilling
template <class Rule, typename R>
constexpr int force_min_waves() { return sizeof(R) == 4 && Rule::NEN <= 10 ? 4 : 3; }

template <class Rule, typename R>
__global__ __launch_bounds__(kForceThreads, (force_min_waves<Rule, R>())) void k_elem_force(AsmArgs a, const int32_t* __restrict__ incpos,
                                                             R* __restrict__ blocks) {
  constexpr int NQ = Rule::NQ, NEN = Rule::NEN, NPN = Rule::NPN, MC = Rule::MC, EB = force_elems<Rule>();
  constexpr size_t NOD = (size_t)EB * nodal_doubles<Rule>() * sizeof(double), PH = (size_t)EB * NQ * 9 * sizeof(R);
  __shared__ __align__(16) unsigned char smem[NOD > PH ? NOD : PH];
  __shared__ R dn[NQ * NEN * 3];  // unit-scaled parent gradients, dN_a(q)_m at 3 (NEN q + a) + m
  const int tid = threadIdx.x;
  const int64_t e0 = (int64_t)blockIdx.x * EB;
  const int ne = (int)(a.n_elem - e0 < EB ? a.n_elem - e0 : EB);
  double* nod = reinterpret_cast<double*>(smem);
  gather_nodal<Rule>(a, e0, ne, nod);
  for (int idx = tid; idx < NQ * NEN * 3; idx += kForceThreads) {
    const int q = idx / (3 * NEN), r = idx - 3 * NEN * q;
    dn[idx] = (R)Rule::dN_rt(q, r / 3, r % 3);
  }
  __syncthreads();
  double* terms = nod + EB * NEN * 6;
  if constexpr (MC == 1) {
    t10_element_terms<2, 6>(nod, ne, terms);
    __syncthreads();
  }
  const bool act = tid < ne * NQ;
  const int pl = act ? tid : 0;  // idle lanes evaluate point 0 and store nothing
  const int el = pl / NQ, q = pl - el * NQ;
  double Jinv[9], det, Hd[9], Fd[9];
  tile_kinematics<Rule>(a, nod + 6 * NEN * el, terms + 2 * kT10Terms * el, e0 + el, q, Jinv, det, Hd, Fd);
  __syncthreads();  // the nodal values are consumed: the LDS holds Phat from here on
  PointOut<R> o;
  const MatParams mp = launch_material(a);
  const unsigned fl = point_update<R, false>(mp, Hd, Fd, det * Rule::w_rt(q), a.alpha, a.beta, o);
  if (act && fl) atomicOr(a.flags, fl);
  HatOut<R> h;
  to_parent<R, false>(o, Jinv, h);
  R* ph = reinterpret_cast<R*>(smem);
  if (act) {
#pragma unroll
    for (int t = 0; t < 9; ++t) ph[9 * pl + t] = h.P[t];
  }
  __syncthreads();
  for (int t = tid; t < ne * NEN; t += kForceThreads) {
    const int le = t / NEN, al = t - le * NEN;
    R f0 = R(0), f1 = R(0), f2 = R(0);
    for (int qq = 0; qq < NQ; ++qq) {
      const R* p = ph + 9 * (le * NQ + qq);
      const R* d = dn + 3 * (NEN * qq + al);
      const R d0 = d[0], d1 = d[1], d2 = d[2];
      f0 += p[0] * d0 + p[1] * d1 + p[2] * d2;
      f1 += p[3] * d0 + p[4] * d1 + p[5] * d2;
      f2 += p[6] * d0 + p[7] * d1 + p[8] * d2;
    }
    double sc[4];
    element_scales<Rule>(a, e0 + le, sc);
    const R s = (R)sc[al % 4];
    const int64_t pos = incpos[(e0 + le) * NPN + al / MC];
    R* out = blocks + pos * (3 * MC) + 3 * (al % MC);
    out[0] = f0 * s;
    out[1] = f1 * s;
    out[2] = f2 * s;
  }
}

template <typename R>
__global__ __launch_bounds__(256) void k_force_sum(const int32_t* __restrict__ inc_off, const R* __restrict__ blocks,
                                                   int64_t n_rows, int rpn, bool accum, double* __restrict__ f) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rows) return;
  const int64_t I = r / rpn;
  const int j = (int)(r - I * rpn);
  // four loads in flight, summed in incidence order
  double s = 0.0;
  int32_t x = inc_off[I];
  const int32_t x1 = inc_off[I + 1];
  for (; x + 4 <= x1; x += 4) {
    const R* b = blocks + (int64_t)x * rpn + j;
    const double v0 = (double)b[0], v1 = (double)b[rpn], v2 = (double)b[2 * rpn], v3 = (double)b[3 * rpn];
    s += v0;
    s += v1;
    s += v2;
    s += v3;
  }
  for (; x < x1; ++x) s += (double)blocks[(int64_t)x * rpn + j];
  f[r] = accum ? f[r] + s : s;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int grid_of(int64_t n, int b) { return (int)((n + b - 1) / b); }

template <class Rule, typename R>
int launch_force_rule(const Mesh& m, const AsmArgs& a, void* blk, hipStream_t s) {
  constexpr int EB = force_elems<Rule>();
  const int64_t blocks = (m.n_elem + EB - 1) / EB;
  if (blocks > INT32_MAX) return TLFEA_ERR_TOO_LARGE;
  if (blocks > 0)
    hipLaunchKernelGGL((k_elem_force<Rule, R>), dim3((unsigned)blocks), dim3(kForceThreads), 0, s, a, m.d_incpos,
                       (R*)blk);
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

template <typename R>
int launch_force_prec(const Mesh& m, const AsmArgs& a, void* blk, hipStream_t s) {
  if (m.elem_type == TLFEA_T10) return launch_force_rule<RuleT10, R>(m, a, blk, s);
  if (m.elem_type == TLFEA_ANCF3243) return launch_force_rule<RuleBeam, R>(m, a, blk, s);
  if (m.gl[0] == 3) return launch_force_rule<RuleAncf<3, 3, 2>, R>(m, a, blk, s);
  return launch_force_rule<RuleAncf<4, 4, 3>, R>(m, a, blk, s);
}

int launch_force_sum(const Mesh& m, const void* blk, double* f, bool accum, hipStream_t s) {
  const int rpn = 3 * m.mc;
  if (m.n_dof > 0) {
    if (m.precision == TLFEA_MIXED)
      hipLaunchKernelGGL(k_force_sum<float>, dim3(grid_of(m.n_dof, 256)), dim3(256), 0, s, m.d_inc_off,
                         (const float*)blk, m.n_dof, rpn, accum, f);
    else
      hipLaunchKernelGGL(k_force_sum<double>, dim3(grid_of(m.n_dof, 256)), dim3(256), 0, s, m.d_inc_off,
                         (const double*)blk, m.n_dof, rpn, accum, f);
  }
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

// Dynamic LDS beyond 64 KiB has to be allowed per kernel; the largest size
// granted so far is remembered per kernel (by address: kernels of one
// signature share a template instantiation here) and device.
template <typename Kernel>
int allow_lds(Kernel* kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return TLFEA_OK;
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, size_t> granted;
  int dev = 0, max_bytes = 0;
  TLFEA_HIP_CHECK(hipGetDevice(&dev));
  const auto key = std::make_pair(reinterpret_cast<const void*>(kernel), dev);
  std::lock_guard<std::mutex> lock(mu);
  auto it = granted.find(key);
  if (it != granted.end() && bytes <= it->second) return TLFEA_OK;
  TLFEA_HIP_CHECK(hipDeviceGetAttribute(&max_bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  if (bytes > (size_t)max_bytes) return TLFEA_ERR_UNSUPPORTED;
  TLFEA_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  granted[key] = bytes;
  return TLFEA_OK;
}

template <class Rule, typename R>
int launch_points_rule(const Mesh& m, const AsmArgs& a, bool want_k, hipStream_t s) {
  const int64_t npts = m.n_elem * Rule::NQ;
  if (npts > (int64_t)INT32_MAX * 256) return TLFEA_ERR_TOO_LARGE;
  if (npts == 0) return TLFEA_OK;
  R* stage = (R*)m.d_stage;
  if (want_k && point_records_sym(m, true))
    hipLaunchKernelGGL((k_stage_tile<Rule, R, sizeof(R) == 8>), dim3(grid_of(npts, kStageThreads)),
                       dim3(kStageThreads), 0, s, a, stage);
  else if (want_k)
    hipLaunchKernelGGL((k_stage_tile<Rule, R, false>), dim3(grid_of(npts, kStageThreads)), dim3(kStageThreads), 0,
                       s, a, stage);
  else
    hipLaunchKernelGGL((k_stage<Rule, R, false>), dim3(grid_of(npts, 256)), dim3(256), 0, s, a, stage);
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

// LDS for a range's upper row offsets (upper-triangle output), 8-byte multiple
size_t upper_table_bytes(const Mesh& m) { return 8 * (size_t)((m.max_range_rows + 2) / 2); }

// pass 2 addresses records in 16-byte units with 32-bit offsets
template <class Rule, typename R>
bool records_addressable(int64_t n_elem, bool want_k) {
  const int64_t pieces = (int64_t)Rule::NQ * (want_k ? kRecK : kRecF) * (int64_t)sizeof(R) / 16;
  return n_elem * pieces < ((int64_t)1 << 32);
}

template <class Rule, typename R>
int launch_nodes_rule(const Mesh& m, const void* stage, double* f, double* vals, bool accum, hipStream_t s,
                      const GatherOptions& mt, bool tangent_records) {
  const bool want_f = f != nullptr, want_k = vals != nullptr;
  if (want_k && !tangent_records) return TLFEA_ERR_INVALID;
  const bool krec = tangent_records;
  const bool sym = krec && m.staged_sym;  // symmetric float64 records from pass 1
  if (!records_addressable<Rule, R>(m.n_elem, want_k)) return TLFEA_ERR_TOO_LARGE;
  GatherArgs g{};
  g.ranges = m.d_ranges;
  g.inc_off = m.d_inc_off;
  g.inc = m.d_inc;
  g.row_off = m.d_row_off;
  g.rank = m.d_rank;
  g.escale = m.d_escale;
  g.half_h = 0.5 * m.thickness;
  g.stage = stage;
  g.f = f;
  g.vals = vals;
  g.mass = mt.mass;
  g.adj_off = m.d_adj_off;
  g.inv_h = mt.inv_h;
  g.row_off_u = mt.row_off_u;
  g.inc_cap = (int)((m.max_range_inc + 15) / 16 * 16);
  const int waves = record_waves(m.tune, m.n_ranges);
  const size_t lds = sizeof(double) * (want_k ? m.max_range_values : m.max_range_rows) + g.inc_cap +
                     (size_t)waves * (krec ? (sym ? wave_buf_bytes<Rule, R, true, sizeof(R) == 8>()
                                                  : wave_buf_bytes<Rule, R, true>())
                                           : wave_buf_bytes<Rule, R, false>()) +
                     (mt.row_off_u ? upper_table_bytes(m) : 0);
  const dim3 grid((unsigned)m.n_ranges), blk(64 * waves);
#define TLFEA_GATHER_S(F, K, A, KR, SY)                                              \
  do {                                                                               \
    if (int rc = allow_lds(k_gather<Rule, R, F, K, A, KR, SY>, lds)) return rc;      \
    hipLaunchKernelGGL((k_gather<Rule, R, F, K, A, KR, SY>), grid, blk, lds, s, g); \
  } while (0)
#define TLFEA_GATHER(F, K, A, KR)                                                            \
  do {                                                                                       \
    if (KR && sym) TLFEA_GATHER_S(F, K, A, KR, (KR && sizeof(R) == 8)); else TLFEA_GATHER_S(F, K, A, KR, false); \
  } while (0)
  if (want_k && want_f) {
    if (accum) TLFEA_GATHER(true, true, true, true); else TLFEA_GATHER(true, true, false, true);
  } else if (want_k) {
    if (accum) TLFEA_GATHER(false, true, true, true); else TLFEA_GATHER(false, true, false, true);
  } else if (krec) {  // the force alone from tangent records
    if (accum) TLFEA_GATHER(true, false, true, true); else TLFEA_GATHER(true, false, false, true);
  } else {
    if (accum) TLFEA_GATHER(true, false, true, false); else TLFEA_GATHER(true, false, false, false);
  }
#undef TLFEA_GATHER
#undef TLFEA_GATHER_S
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

// Elements per workgroup of `waves` waves: as few as give every SIMD of the GPU
// (256 CUs x 4) a wave, then up to `most`.  A small mesh is bound by the chain
// of one wave, which is as long as its tile; from 1,024 waves on the point work,
// which a short tile leaves lanes idle for, counts more.
int tile_for(int64_t n_elem, int most, int waves) {
  const int64_t groups = 1024 / waves;
  return (int)std::min<int64_t>(most, std::max<int64_t>(1, (n_elem + groups - 1) / groups));
}

// pass 2 addresses T10 row blocks in 16-byte units with 32-bit offsets
bool rows_addressable(const Mesh& m, size_t value_bytes) {
  return m.n_elem * m.n_pn * (int64_t)(kRowBlk * value_bytes / 16) < ((int64_t)1 << 32);
}

// pass 2 over the element row blocks
template <typename R>
int launch_rows_nodes(const Mesh& m, double* f, double* vals, bool accum, hipStream_t s, const GatherOptions& mt) {
  const bool want_f = f != nullptr, want_k = vals != nullptr;
  if (!rows_addressable(m, sizeof(R))) return TLFEA_ERR_TOO_LARGE;
  GatherArgs g{};
  g.ranges = m.d_ranges;
  g.inc_off = m.d_inc_off;
  g.row_off = m.d_row_off;
  g.rank = m.d_rank_inc;
  g.stage = m.d_stage;
  g.f = f;
  g.vals = vals;
  g.mass = mt.mass;
  g.adj_off = m.d_adj_off;
  g.inv_h = mt.inv_h;
  g.row_off_u = mt.row_off_u;
  g.inc_cap = (int)((m.max_range_inc + 15) / 16 * 16);
  const size_t lds = sizeof(double) * (want_k ? m.max_range_values : m.max_range_rows) + g.inc_cap +
                     (mt.row_off_u ? upper_table_bytes(m) : 0);
  const dim3 grid((unsigned)m.n_ranges), blk(64 * m.tune.waves);
#define TLFEA_GATHER(F, K, A)                                              \
  do {                                                                     \
    if (int rc = allow_lds(k_gather_rows<R, F, K, A>, lds)) return rc;        \
    hipLaunchKernelGGL((k_gather_rows<R, F, K, A>), grid, blk, lds, s, g);   \
  } while (0)
  if (want_k && want_f) {
    if (accum) TLFEA_GATHER(true, true, true); else TLFEA_GATHER(true, true, false);
  } else if (want_k) {
    if (accum) TLFEA_GATHER(false, true, true); else TLFEA_GATHER(false, true, false);
  } else {
    if (accum) TLFEA_GATHER(true, false, true); else TLFEA_GATHER(true, false, false);
  }
#undef TLFEA_GATHER
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

// Undamped materials take the symmetric record layout in the element-row
// pass 1 (TLFEA_SYM_RECORDS=0 keeps the full layout, for comparisons).
bool sym_records(const Mesh& m) {
  static const bool on = [] {
    const char* v = std::getenv("TLFEA_SYM_RECORDS");
    return !(v && v[0] == '0');
  }();
  return on && m.mp.eta == 0.0 && m.mp.lam_v == 0.0;
}

// The shell's element-row contraction on the matrix cores (TLFEA_MC_MFMA=0
// keeps the vector form, for comparisons).
bool mc_mfma() {
  static const bool on = [] {
    const char* v = std::getenv("TLFEA_MC_MFMA");
    return !(v && v[0] == '0');
  }();
  return on;
}

template <class Rule>
int launch_rows_mc_points(const Mesh& m, const AsmArgs& a, hipStream_t s) {
  const int eb = m.precision == TLFEA_MIXED ? rows_mc_elems<Rule>() : rows64_elems<Rule>();
  const int64_t blocks = (m.n_elem + eb - 1) / eb;
  if (blocks > INT32_MAX) return TLFEA_ERR_TOO_LARGE;
  if (m.precision == TLFEA_FP64) {
    const dim3 grid((unsigned)blocks), th(rows64_threads<Rule>());
    if (blocks > 0 && sym_records(m) && Rule::NEN == 16)
      hipLaunchKernelGGL((k_elem_rows_mc64<Rule, Rule::NEN == 16>), grid, th, 0, s, a, m.d_incpos, (double*)m.d_stage);
    else if (blocks > 0)
      hipLaunchKernelGGL((k_elem_rows_mc64<Rule, false>), grid, th, 0, s, a, m.d_incpos, (double*)m.d_stage);
    TLFEA_HIP_CHECK(hipGetLastError());
    return TLFEA_OK;
  }
  // the shell's 16 x 16 slot tiles on the matrix cores (the beam's 8 x 8 slots
  // would fill half a tile: slower than its vector form, measured)
  constexpr bool MF = Rule::NEN == 16;
  if (blocks > 0) {
    if (sym_records(m) && mc_mfma())
      hipLaunchKernelGGL((k_elem_rows_mc<Rule, true, MF>), dim3((unsigned)blocks), dim3(kRowsMcThreads), 0, s,
                         a, m.d_incpos, (float*)m.d_stage);
    else if (sym_records(m))
      hipLaunchKernelGGL((k_elem_rows_mc<Rule, true, false>), dim3((unsigned)blocks), dim3(kRowsMcThreads), 0, s,
                         a, m.d_incpos, (float*)m.d_stage);
    else if (mc_mfma())
      hipLaunchKernelGGL((k_elem_rows_mc<Rule, false, MF>), dim3((unsigned)blocks), dim3(kRowsMcThreads), 0, s,
                         a, m.d_incpos, (float*)m.d_stage);
    else
      hipLaunchKernelGGL((k_elem_rows_mc<Rule, false, false>), dim3((unsigned)blocks), dim3(kRowsMcThreads), 0, s,
                         a, m.d_incpos, (float*)m.d_stage);
  }
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

template <class Rule, typename R>
int launch_rows_mc_nodes(const Mesh& m, double* f, double* vals, bool accum, hipStream_t s, const GatherOptions& mt) {
  const bool want_f = f != nullptr, want_k = vals != nullptr;
  GatherArgs g{};
  g.ranges = m.d_ranges;
  g.inc_off = m.d_inc_off;
  g.inc = m.d_inc;
  g.row_off = m.d_row_off;
  g.rank = m.d_rank;
  g.stage = m.d_stage;
  g.f = f;
  g.vals = vals;
  g.mass = mt.mass;
  g.adj_off = m.d_adj_off;
  g.inv_h = mt.inv_h;
  g.row_off_u = mt.row_off_u;
  g.inc_cap = (int)((m.max_range_inc + 15) / 16 * 16);
  const size_t lds = sizeof(double) * (want_k ? m.max_range_values : m.max_range_rows) + g.inc_cap +
                     (mt.row_off_u ? upper_table_bytes(m) : 0);
  const dim3 grid((unsigned)m.n_ranges), blk(64 * (want_k ? m.tune.waves : record_waves(m.tune, m.n_ranges)));
#define TLFEA_GATHER(F, K, A)                                                   \
  do {                                                                          \
    if (int rc = allow_lds(k_gather_rows_mc<Rule, R, F, K, A>, lds)) return rc;    \
    hipLaunchKernelGGL((k_gather_rows_mc<Rule, R, F, K, A>), grid, blk, lds, s, g); \
  } while (0)
  if (want_k && want_f) {
    if (accum) TLFEA_GATHER(true, true, true); else TLFEA_GATHER(true, true, false);
  } else if (want_k) {
    if (accum) TLFEA_GATHER(false, true, true); else TLFEA_GATHER(false, true, false);
  } else {
    if (accum) TLFEA_GATHER(true, false, true); else TLFEA_GATHER(true, false, false);
  }
#undef TLFEA_GATHER
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

// pass 2 over the row blocks (the two shell rules differ in pass 1 only)
template <typename R>
int launch_rows_nodes_prec(const Mesh& m, double* f, double* vals, bool accum, hipStream_t s, const GatherOptions& mt) {
  if (m.elem_type == TLFEA_T10) return launch_rows_nodes<R>(m, f, vals, accum, s, mt);
  if (m.elem_type == TLFEA_ANCF3243) return launch_rows_mc_nodes<RuleBeam, R>(m, f, vals, accum, s, mt);
  return launch_rows_mc_nodes<RuleAncf<3, 3, 2>, R>(m, f, vals, accum, s, mt);
}

template <typename R>
int launch_points_prec(const Mesh& m, const AsmArgs& a, bool want_k, hipStream_t s) {
  if (m.elem_type == TLFEA_T10) return launch_points_rule<RuleT10, R>(m, a, want_k, s);
  if (m.elem_type == TLFEA_ANCF3243) return launch_points_rule<RuleBeam, R>(m, a, want_k, s);
  if (m.gl[0] == 3) return launch_points_rule<RuleAncf<3, 3, 2>, R>(m, a, want_k, s);
  return launch_points_rule<RuleAncf<4, 4, 3>, R>(m, a, want_k, s);
}

template <typename R>
int launch_nodes_prec(const Mesh& m, double* f, double* vals, bool accum, hipStream_t s, const GatherOptions& mt) {
  const bool kr = m.staged == 2;  // tangent records (else force records)
  if (m.elem_type == TLFEA_T10) return launch_nodes_rule<RuleT10, R>(m, m.d_stage, f, vals, accum, s, mt, kr);
  if (m.elem_type == TLFEA_ANCF3243)
    return launch_nodes_rule<RuleBeam, R>(m, m.d_stage, f, vals, accum, s, mt, kr);
  if (m.gl[0] == 3) return launch_nodes_rule<RuleAncf<3, 3, 2>, R>(m, m.d_stage, f, vals, accum, s, mt, kr);
  return launch_nodes_rule<RuleAncf<4, 4, 3>, R>(m, m.d_stage, f, vals, accum, s, mt, kr);
}

template <class Rule, typename R>
int launch_batch_rule(const GatherTuning& tu, const BatchArgs& b, int n_ranges, size_t lds, hipStream_t s) {
  if (b.n_blocks > 0)
    hipLaunchKernelGGL((k_stage_batch<Rule, R>), dim3((unsigned)b.n_blocks), dim3(kStageThreads), 0, s, b);
  TLFEA_HIP_CHECK(hipGetLastError());
  const int waves = record_waves(tu, n_ranges);
  const size_t lds_all = lds + b.inc_cap + (size_t)waves * wave_buf_bytes<Rule, R, true>();
  if (int rc = allow_lds(k_gather_batch<Rule, R>, lds_all)) return rc;
  hipLaunchKernelGGL((k_gather_batch<Rule, R>), dim3(n_ranges), dim3(64 * waves), lds_all, s, b);
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

__global__ void k_zero(double* __restrict__ p, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0.0;
}

}  // namespace

static bool rows_on() {
  static const bool on = [] {
    const char* v = std::getenv("TLFEA_ELEMENT_ROWS");
    return !(v && v[0] == '0');
  }();
  return on;
}

// float64 element rows (T10): pass 1 has one wave per SIMD and writes 3.7 GB of
// blocks for 480,000 elements, pass 2 reads each once; point records are half
// that size, but pass 2 reads them 6.5 times.  Whole call, rows against records:
// 30,000 elements 148 / 144 us, 49,200 247 / 245, 49,800 249 / 249, 60,000 271 / 311,
// 480,000 2,070 / 2,382: the line is where the fifth round of 1,024 waves starts.  Undamped meshes keep the symmetric records
// (480,000: 2,014 / 1,795).
constexpr int64_t kRows64MinElems = 4 * 1024 * kRowElems;

// float64 element rows of the 3x3x2 shell: a workgroup's 21 slot tiles are a chain
// that a small mesh waits for.  f and K, rows / records with their four waves:
// undamped 1,024 elements 54 / 42 us, 3,025 79 / 75, 4,096 84 / 87, 6,400 96 / 121,
// 10,000 172 / 176, 40,000 643 / 763; damped 2,704 89 / 76, 3,025 92 / 91, 4,096 96 /
// 111, 10,000 185 / 223.  K alone gains less (the rows hold the force anyway): damped
// 4,096 95 / 96, undamped 83 / 79, 10,000 170 / 160, 25,600 429 / 444; the line is
// f and K's.  Batches have full records and few elements a workgroup: 3,200 bodies of
// one element 107 / 181, 40 of 100 104 / 113.
constexpr int64_t kRows64MinShellBatch = 3000;

// The 4x4x3 shell, whose records are the larger (36.9 KB an element against 19.6),
// takes rows at every size (1 element 18 / 40 us, 64 39 / 71, 10,000 257 / 434).
//
// float64 element rows of the beam: one wave's chain takes 14 us, which the records
// of a few elements undercut, the symmetric ones of an undamped mesh those of a few
// more (rows / records: damped 3 elements 18.3 / 16.8 us, 4 19.0 / 20.4, 8 21.0 /
// 25.2; undamped 1 16.3 / 12.8, 6 19.1 / 18.4, 8 20.0 / 22.1, 100 22 / 25, 500,000
// 2,140 / 2,825).  Batches have full records, so the first line holds for them.
constexpr int64_t kRows64MinBeam = 4, kRows64MinBeamSym = 8;

bool use_rows_batch(const Mesh& m, int64_t n_elem) {
  if (!rows_on() || !m.d_incpos || (m.elem_type == TLFEA_T10 && !m.d_rank_inc)) return false;
  if (m.precision == TLFEA_MIXED) return true;
  if (m.elem_type == TLFEA_T10) return n_elem >= kRows64MinElems && rows_addressable(m, sizeof(double));
  if (m.elem_type == TLFEA_ANCF3243) return n_elem >= kRows64MinBeam;
  return m.gl[0] != 3 || n_elem >= kRows64MinShellBatch;
}

static size_t rows_bytes(const Mesh& m) {
  const size_t r = m.precision == TLFEA_MIXED ? sizeof(float) : sizeof(double);
  return (size_t)m.n_elem * m.n_pn * (m.elem_type == TLFEA_T10 ? kRowBlk : 36 * m.n_en + 36) * r;
}

bool rows_past_caches(size_t bytes, bool sym) { return bytes > (sym ? kCachedSymRowBytes : kCachedRowBytes); }

static size_t record_bytes(const Mesh& m) { return (size_t)m.n_elem * m.n_qp * stage_record_bytes(m.precision); }

bool use_rows(const Mesh& m, bool want_k) {
  if (!want_k || !use_rows_batch(m, m.n_elem)) return false;
  if (m.precision == TLFEA_MIXED) return true;
  if (m.elem_type == TLFEA_ANCF3443 && m.gl[0] == 3 && m.n_elem < kRows64MinShell) return false;
  if (sym_records(m) && (m.elem_type == TLFEA_T10 || (m.elem_type == TLFEA_ANCF3243 && m.n_elem < kRows64MinBeamSym)))
    return false;
  return buffer_takes_rows(rows_bytes(m), record_bytes(m), m.stage_cap);
}

// The float64 point records of a tangent pass take the symmetric layout for
// undamped materials (64 values instead of 96).
bool point_records_sym(const Mesh& m, bool want_k) {
  return want_k && m.precision == TLFEA_FP64 && sym_records(m);
}

bool use_force_blocks(const Mesh& m, bool want_k) {
  static const bool on = [] {
    const char* v = std::getenv("TLFEA_FORCE_BLOCKS");
    return !(v && v[0] == '0');
  }();
  return on && !want_k && m.d_incpos;
}

size_t stage_bytes_min(const Mesh& m, bool want_k) {
  return want_k && m.precision == TLFEA_FP64 ? record_bytes(m) : stage_bytes(m, want_k);
}

size_t stage_bytes(const Mesh& m, bool want_k) {
  // between the beam's lines the form follows the material: the buffer fits both
  if (use_rows(m, want_k)) return m.n_elem < kRows64MinBeamSym ? std::max(rows_bytes(m), record_bytes(m)) : rows_bytes(m);
  const size_t r = m.precision == TLFEA_MIXED ? sizeof(float) : sizeof(double);
  if (use_force_blocks(m, want_k)) return (size_t)m.n_elem * m.n_pn * 3 * m.mc * r;
  return want_k ? record_bytes(m) : (size_t)m.n_elem * m.n_qp * kRecF * r;
}

int lpt_tile_elems() { return kLptTile; }

size_t row_block_bytes_for(int elem_type, int precision) {
  const size_t r = precision == TLFEA_MIXED ? sizeof(float) : sizeof(double);
  if (elem_type == TLFEA_T10) return kRowBlk * r;
  return (elem_type == TLFEA_ANCF3243 ? rows_mc_block<RuleBeam::NEN>() : rows_mc_block<16>()) * r;
}
template <class Rule>
static int mc_elems(int precision) {
  return precision == TLFEA_MIXED ? rows_mc_elems<Rule>() : rows64_elems<Rule>();
}
int row_elems_for(int elem_type, int gl0, int precision, int64_t n_elem) {
  if (elem_type == TLFEA_T10) return tile_for(n_elem, kRowElems, 1);
  if (elem_type == TLFEA_ANCF3243) return mc_elems<RuleBeam>(precision);
  return gl0 == 3 ? mc_elems<RuleAncf<3, 3, 2>>(precision) : mc_elems<RuleAncf<4, 4, 3>>(precision);
}

int schedule_tile(int elem_type, int gl0) {
  return elem_type == TLFEA_T10 ? kLptTile : row_elems_for(elem_type, gl0, TLFEA_MIXED, 0);
}

size_t stage_record_bytes(int precision) {
  return (size_t)kRecK * (precision == TLFEA_MIXED ? sizeof(float) : sizeof(double));
}

// Workgroups of the persistent batch kernels one CU holds at once (tile kernel
// for EB elements per tile; range kernel for the given shape and LDS bytes).
using LptKernel = void (*)(BatchArgs, const int2*, int, unsigned*);
static LptKernel lpt_kernel(int tile_elems, bool nt) {
  if (tile_elems == 16) return nt ? k_elem_rows_batch_lpt<RuleT10, 16, true> : k_elem_rows_batch_lpt<RuleT10, 16, false>;
  return nt ? k_elem_rows_batch_lpt<RuleT10, kLptTile, true> : k_elem_rows_batch_lpt<RuleT10, kLptTile, false>;
}

int batch_lpt_occupancy(int tile_elems, bool rows_nt, int waves, size_t lds_all, int* tiles_per_cu, int* ranges_per_cu) {
  int nt = 0, nr = 0;
  TLFEA_HIP_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &nt, reinterpret_cast<const void*>(lpt_kernel(tile_elems, rows_nt)), 64, 0));
  if (int rc = allow_lds(k_gather_rows_batch_lpt, lds_all)) return rc;
  TLFEA_HIP_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &nr, reinterpret_cast<const void*>(k_gather_rows_batch_lpt), 64 * waves, lds_all));
  *tiles_per_cu = std::max(nt, 1);
  *ranges_per_cu = std::max(nr, 1);
  return TLFEA_OK;
}

int launch_zero(double* p, int64_t n, hipStream_t s) {
  if (n <= 0) return TLFEA_OK;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

int launch_points(const Mesh& m, const AsmArgs& a, bool want_k, hipStream_t s) {
  if (use_force_blocks(m, want_k))
    return m.precision == TLFEA_MIXED ? launch_force_prec<float>(m, a, m.d_stage, s)
                                     : launch_force_prec<double>(m, a, m.d_stage, s);
  if (use_rows(m, want_k) && m.elem_type != TLFEA_T10) {
    if (m.elem_type == TLFEA_ANCF3243) return launch_rows_mc_points<RuleBeam>(m, a, s);
    if (m.gl[0] == 3) return launch_rows_mc_points<RuleAncf<3, 3, 2>>(m, a, s);
    return launch_rows_mc_points<RuleAncf<4, 4, 3>>(m, a, s);
  }
  if (use_rows(m, want_k)) {
    const bool sym = m.precision == TLFEA_MIXED && sym_records(m);
    const int tile = tile_for(m.n_elem, sym ? kSymElems : kRowElems, sym ? kSymThreads / 64 : 1);
    const int64_t blocks = (m.n_elem + tile - 1) / tile;
    if (blocks > INT32_MAX) return TLFEA_ERR_TOO_LARGE;
    if (blocks > 0) {
      const dim3 grid((unsigned)blocks);
      const bool nt = rows_past_caches(rows_bytes(m), sym);
      if (sym)
        hipLaunchKernelGGL((nt ? k_elem_rows_sym<RuleT10, true> : k_elem_rows_sym<RuleT10, false>), grid,
                           dim3(kSymThreads), 0, s, a, tile, m.d_incpos, (float*)m.d_stage);
      else if (m.precision == TLFEA_MIXED && blocks <= kSplitRowTiles)
        hipLaunchKernelGGL((k_elem_rows<RuleT10, float, false, true>), dim3(grid.x, 3), dim3(64), 0, s, a, tile,
                           m.d_incpos, (float*)m.d_stage);
      else if (m.precision == TLFEA_MIXED)
        hipLaunchKernelGGL((nt ? k_elem_rows<RuleT10, float, true> : k_elem_rows<RuleT10, float, false>), grid, dim3(64), 0,
                           s, a, tile, m.d_incpos, (float*)m.d_stage);
      else  // float64 rows start far above the cached size
        hipLaunchKernelGGL((k_elem_rows<RuleT10, double, true>), grid, dim3(64), 0, s, a, tile, m.d_incpos,
                           (double*)m.d_stage);
    }
    TLFEA_HIP_CHECK(hipGetLastError());
    return TLFEA_OK;
  }
  if (m.precision == TLFEA_MIXED) return launch_points_prec<float>(m, a, want_k, s);
  return launch_points_prec<double>(m, a, want_k, s);
}

int launch_nodes(const Mesh& m, double* f, double* vals, bool accum, hipStream_t s, const GatherOptions& mt) {
  if (mt.mass && !vals) return TLFEA_ERR_INVALID;
  if (m.n_ranges == 0) {  // no nodes: only the (empty) outputs to clear
    if (accum) return TLFEA_OK;
    int rc = f ? launch_zero(f, m.n_dof, s) : TLFEA_OK;
    return (rc || !vals) ? rc : launch_zero(vals, mt.row_off_u ? m.nnz_u : m.nnz, s);
  }
  if (m.staged == 3)
    return m.precision == TLFEA_MIXED ? launch_rows_nodes_prec<float>(m, f, vals, accum, s, mt)
                                      : launch_rows_nodes_prec<double>(m, f, vals, accum, s, mt);
  if (m.staged == 4) return vals ? TLFEA_ERR_INVALID : launch_force_sum(m, m.d_stage, f, accum, s);
  if (m.precision == TLFEA_MIXED) return launch_nodes_prec<float>(m, f, vals, accum, s, mt);
  return launch_nodes_prec<double>(m, f, vals, accum, s, mt);
}

// Fixed work area of the allocation-free force call: the force blocks of one
// call (3 mc values per incidence).  The kernels take its device address,
// looked up once per device with that device current; the array's name in
// host code is only a host-side stand-in for the symbol.
int noalloc_scratch(void** out) {
  static std::mutex mu;
  static std::map<int, void*> addr;
  int dev = 0;
  TLFEA_HIP_CHECK(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(mu);
  auto it = addr.find(dev);
  if (it == addr.end()) {
    void* p = nullptr;
    TLFEA_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return TLFEA_ERR_HIP;
    it = addr.emplace(dev, p).first;
  }
  *out = it->second;
  return TLFEA_OK;
}

size_t noalloc_force_bytes(const Mesh& m) {
  return (size_t)m.n_elem * m.n_pn * 3 * m.mc * (m.precision == TLFEA_MIXED ? sizeof(float) : sizeof(double));
}

int launch_force_noalloc(const Mesh& m, const AsmArgs& a, double* f, hipStream_t s) {
  if (!m.d_incpos) return TLFEA_ERR_NO_PATTERN;
  if (noalloc_force_bytes(m) > kNoallocScratchBytes) return TLFEA_ERR_TOO_LARGE;
  void* blk = nullptr;
  if (int rc = noalloc_scratch(&blk)) return rc;
  // every incidence block is written by pass 1 before pass 2 reads it: nothing to clear
  int rc = m.precision == TLFEA_MIXED ? launch_force_prec<float>(m, a, blk, s) : launch_force_prec<double>(m, a, blk, s);
  if (rc) return rc;
  return launch_force_sum(m, blk, f, false, s);
}

int launch_force_points(Mesh& m, const AsmArgs& a, hipStream_t s) {
  if (m.n_elem == 0) return TLFEA_OK;  // no blocks
  if (!m.d_incpos) return TLFEA_ERR_NO_PATTERN;
  const size_t rsz = m.precision == TLFEA_MIXED ? sizeof(float) : sizeof(double);
  if (int rc = ensure_stage(m, (size_t)m.n_elem * m.n_pn * 3 * m.mc * rsz)) return rc;
  const int rc = m.precision == TLFEA_MIXED ? launch_force_prec<float>(m, a, m.d_stage, s)
                                            : launch_force_prec<double>(m, a, m.d_stage, s);
  m.staged = rc ? 0 : 4;
  m.staged_precision = m.precision;
  return rc;
}

int launch_force_blocks(Mesh& m, const AsmArgs& a, double* f, hipStream_t s) {
  if (!m.d_incpos) return TLFEA_ERR_NO_PATTERN;
  if (int rc = launch_force_points(m, a, s)) return rc;
  return launch_force_sum(m, m.d_stage, f, false, s);
}

__global__ void k_params(int kind, const double* __restrict__ p, double* __restrict__ mp) {
  if (threadIdx.x != 0) return;
  if (kind == TLFEA_SVK) {
    const double E = p[0], nu = p[1];
    mp[0] = E * nu / ((1.0 + nu) * (1.0 - 2.0 * nu));
    mp[1] = E / (2.0 * (1.0 + nu));
    mp[2] = 0.0;
  } else {
    mp[0] = p[0];
    mp[1] = p[1];
    mp[2] = p[2];
  }
  mp[3] = p[3];
  mp[4] = p[4];
}

int launch_params(const Mesh& m, const double* d_params, hipStream_t s) {
  hipLaunchKernelGGL(k_params, dim3(1), dim3(64), 0, s, m.material, d_params, m.d_mp);
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

template <typename R>
int launch_rows_batch(const GatherTuning& tu, const BatchArgs& b, int n_ranges, size_t lds, hipStream_t s) {
  // float64 rows start far above the cached size
  if (b.n_rblocks > 0) {
    const dim3 grid((unsigned)b.n_rblocks);
    if (sizeof(R) == 8 || b.nt)
      hipLaunchKernelGGL((k_elem_rows_batch<RuleT10, R, true>), grid, dim3(64), 0, s, b);
    else
      hipLaunchKernelGGL((k_elem_rows_batch<RuleT10, float, false>), grid, dim3(64), 0, s, b);
  }
  TLFEA_HIP_CHECK(hipGetLastError());
  const size_t lds_all = lds + b.inc_cap;
  if (int rc = allow_lds(k_gather_rows_batch<R>, lds_all)) return rc;
  hipLaunchKernelGGL(k_gather_rows_batch<R>, dim3(n_ranges), dim3(64 * tu.waves), lds_all, s, b);
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

template <class Rule, typename R>
int launch_rows_mc_batch(const GatherTuning& tu, const BatchArgs& b, int n_ranges, size_t lds, hipStream_t s) {
  constexpr bool MF = Rule::NEN == 16;  // the shell's slot tiles on the matrix cores
  if (b.n_rblocks > 0) {
    const dim3 grid((unsigned)b.n_rblocks);
    if (sizeof(R) == 8)
      hipLaunchKernelGGL(k_elem_rows_mc64_batch<Rule>, grid, dim3(rows64_threads<Rule>()), 0, s, b);
    else if (mc_mfma())
      hipLaunchKernelGGL((k_elem_rows_mc_batch<Rule, MF>), grid, dim3(kRowsMcThreads), 0, s, b);
    else
      hipLaunchKernelGGL((k_elem_rows_mc_batch<Rule, false>), grid, dim3(kRowsMcThreads), 0, s, b);
  }
  TLFEA_HIP_CHECK(hipGetLastError());
  const size_t lds_all = lds + b.inc_cap;
  if (int rc = allow_lds(k_gather_rows_mc_batch<Rule, R>, lds_all)) return rc;
  hipLaunchKernelGGL((k_gather_rows_mc_batch<Rule, R>), dim3(n_ranges), dim3(64 * tu.waves), lds_all, s, b);
  TLFEA_HIP_CHECK(hipGetLastError());
  return TLFEA_OK;
}

template <typename R>
int launch_rows_batch_prec(int elem_type, int gl0, const GatherTuning& tu, const BatchArgs& b, int n_ranges, size_t lds,
                           hipStream_t s) {
  if (elem_type == TLFEA_T10) return launch_rows_batch<R>(tu, b, n_ranges, lds, s);
  if (elem_type == TLFEA_ANCF3243) return launch_rows_mc_batch<RuleBeam, R>(tu, b, n_ranges, lds, s);
  if (gl0 == 3) return launch_rows_mc_batch<RuleAncf<3, 3, 2>, R>(tu, b, n_ranges, lds, s);
  return launch_rows_mc_batch<RuleAncf<4, 4, 3>, R>(tu, b, n_ranges, lds, s);
}

int launch_batch(int elem_type, int gl0, int precision, const GatherTuning& tu, const BatchArgs& b,
                 int n_ranges, size_t lds, hipStream_t s, const BatchSchedule& sc) {
  if (n_ranges == 0) return TLFEA_OK;
  if (b.rows && sc.persistent) {
    hipLaunchKernelGGL(k_reset_counters, dim3(1), dim3(64), 0, s, sc.counters);
    if (sc.n_tiles > 0)
      hipLaunchKernelGGL(lpt_kernel(sc.tile_elems, b.nt != 0), dim3(sc.grid_tiles), dim3(64), 0, s, b, sc.tiles,
                         sc.n_tiles, sc.counters);
    TLFEA_HIP_CHECK(hipGetLastError());
    const size_t lds_all = lds + b.inc_cap;
    if (int rc = allow_lds(k_gather_rows_batch_lpt, lds_all)) return rc;
    hipLaunchKernelGGL(k_gather_rows_batch_lpt, dim3(sc.grid_ranges), dim3(64 * tu.waves), lds_all, s, b,
                       sc.range_order, n_ranges, sc.counters + 1);
    TLFEA_HIP_CHECK(hipGetLastError());
    return TLFEA_OK;
  }
  const bool mixed = precision == TLFEA_MIXED;
  if (b.rows)
    return mixed ? launch_rows_batch_prec<float>(elem_type, gl0, tu, b, n_ranges, lds, s)
                 : launch_rows_batch_prec<double>(elem_type, gl0, tu, b, n_ranges, lds, s);
  if (elem_type == TLFEA_T10)
    return mixed ? launch_batch_rule<RuleT10, float>(tu, b, n_ranges, lds, s)
                 : launch_batch_rule<RuleT10, double>(tu, b, n_ranges, lds, s);
  if (elem_type == TLFEA_ANCF3243)
    return mixed ? launch_batch_rule<RuleBeam, float>(tu, b, n_ranges, lds, s)
                 : launch_batch_rule<RuleBeam, double>(tu, b, n_ranges, lds, s);
  if (gl0 == 3)
    return mixed ? launch_batch_rule<RuleAncf<3, 3, 2>, float>(tu, b, n_ranges, lds, s)
                 : launch_batch_rule<RuleAncf<3, 3, 2>, double>(tu, b, n_ranges, lds, s);
  return mixed ? launch_batch_rule<RuleAncf<4, 4, 3>, float>(tu, b, n_ranges, lds, s)
               : launch_batch_rule<RuleAncf<4, 4, 3>, double>(tu, b, n_ranges, lds, s);
}

}  // namespace tlfea
