// adamw.hip -- the first-order inner solver of a time step (Sec. 4.5, without
// constraint terms): the velocity v minimises the incremental potential whose
// gradient is g(v) = M (v - v_n)/h + f_int(q_n + h v, v) - f_ext, by AdamW, the
// Adam method with decoupled weight decay (Loshchilov and Hutter, ICLR 2019):
//   m <- b1 m + (1 - b1) g,   s <- b2 s + (1 - b2) g^2            (moments)
//   v <- v - lr (m / (1 - b1^l) / (sqrt(s / (1 - b2^l)) + eps) + wd v)
// at iteration l, then q = q_n + h v for the next force evaluation.
//
// Arranged for the GPU: each inner iteration is three launches on the caller's
// stream.  One per-DOF kernel applies the moment and velocity updates fused with
// q = q_n + h v and v - v_n; then pass 1 of the force-only assembly, and the
// gradient over the mass rows, which takes f_int from the element force blocks
// itself.  The bias-correction divisors of the iterations between two
// convergence checks are tabulated in device memory by one kernel (no per-DOF
// power).  In a long solve those iterations are captured once into a HIP graph
// and replayed (kMinReplays below).
// Every launch of a mid-sized mesh is bound by its latency: 18,000 T10 elements
// took 51 us an iteration with six launches (counter, update, both force passes,
// v - v_n, gradient).  Convergence (||g|| <= eps_in (1 + ||v||) or ||g|| <= eps_rel
// ||g_0||, g_0 the first gradient) is checked on the host from norms reduced on
// the device in a fixed order.
#include <cmath>

#include "tlfea_internal.h"

using tlfea::Mesh;

namespace tlfea {
namespace {

constexpr int kNormBlocks = 256;

// Capturing and instantiating the iterations between two checks costs about 9 us
// each, a replayed iteration of a small mesh saves about 1.3 us over launching it
// (96 elements, checks every 50: 15.8 against 17.1 us; every 25, 26 iterations:
// 29.4 against 19.9; 18,000 elements, 26 iterations: 38.1 against 29.5).
constexpr int kMinReplays = 8;

// Iterations whose divisors are tabulated at a time: the table stays 64 KiB however
// rarely the caller checks.
constexpr int kCorrTable = 4096;

struct AdamwArgs {
  double lr, beta1, beta2, eps, wd, h;
};

__global__ void k_fill(double* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

// the bias-correction divisors 1 - b1^l, 1 - b2^l of the next n iterations, and
// the iteration counter advanced past them (one workgroup)
__global__ __launch_bounds__(256) void k_corr(AdamwArgs p, int64_t* l, int n, double* corr) {
  const int64_t l0 = *l;
  __syncthreads();
  for (int t = threadIdx.x; t < n; t += blockDim.x) {
    const double it = (double)(l0 + 1 + t);
    corr[2 * t] = 1.0 - std::pow(p.beta1, it);
    corr[2 * t + 1] = 1.0 - std::pow(p.beta2, it);
  }
  if (threadIdx.x == 0) *l = l0 + n;
}

// per DOF: the two moments, the decoupled-decay velocity update, the step map,
// and (dv not null) v - v_n for the gradient
__global__ void k_adamw(AdamwArgs p, const double* __restrict__ corr, int64_t n, const double* __restrict__ g,
                        const double* __restrict__ q_n, double* __restrict__ m, double* __restrict__ s,
                        double* __restrict__ v, double* __restrict__ q, const double* __restrict__ v_n,
                        double* __restrict__ dv) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double gi = g[i];
  const double mi = p.beta1 * m[i] + (1.0 - p.beta1) * gi;
  const double si = p.beta2 * s[i] + (1.0 - p.beta2) * gi * gi;
  m[i] = mi;
  s[i] = si;
  const double vi = v[i];
  const double vn = vi - p.lr * ((mi / corr[0]) / (std::sqrt(si / corr[1]) + p.eps) + p.wd * vi);
  v[i] = vn;
  q[i] = q_n[i] + p.h * vn;
  if (dv) dv[i] = vn - v_n[i];
}

// partial sums of g.g and v.v per block (fixed order), then one block adds them
__global__ __launch_bounds__(256) void k_norms(const double* g, const double* v, int64_t n, double* part) {
  __shared__ double red[2][256];
  double a = 0.0, b = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    a += g[i] * g[i];
    b += v[i] * v[i];
  }
  red[0][threadIdx.x] = a;
  red[1][threadIdx.x] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      red[0][threadIdx.x] += red[0][threadIdx.x + o];
      red[1][threadIdx.x] += red[1][threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = red[0][0];
    part[2 * blockIdx.x + 1] = red[1][0];
  }
}

// (a lane per partial and a tree: 20 us as one lane's chain of 256 loads)
__global__ __launch_bounds__(kNormBlocks) void k_norms_final(const double* part, double* out) {
  __shared__ double red[2][kNormBlocks];
  const int t = threadIdx.x;
  red[0][t] = part[2 * t];
  red[1][t] = part[2 * t + 1];
  __syncthreads();
  for (int o = kNormBlocks / 2; o > 0; o >>= 1) {
    if (t < o) {
      red[0][t] += red[0][t + o];
      red[1][t] += red[1][t + o];
    }
    __syncthreads();
  }
  if (t < 2) out[t] = std::sqrt(red[t][0]);
}

int blocks_for(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, 1 << 20); }

}  // namespace
}  // namespace tlfea

namespace {

// one inner iteration on stream s, corr its two divisors (no allocation after
// the first, no synchronisation)
int adamw_iteration(tlfea_mesh_t mesh, const tlfea::AdamwArgs& a, const double* q_n, const double* v_n,
                    const double* f_ext, double* v, double* q, double* m, double* sm, double* g, double* f,
                    const double* corr, hipStream_t s) {
  Mesh& me = mesh->m;
  const int64_t n = me.n_dof;
  if (n == 0) return TLFEA_OK;
  if (int rc = tlfea::ensure_dv(me)) return rc;
  double* dv = me.mc == 1 ? me.d_dv : nullptr;
  hipLaunchKernelGGL(tlfea::k_adamw, dim3(tlfea::blocks_for(n)), dim3(256), 0, s, a, corr, n, g, q_n, m, sm, v, q, v_n,
                     dv);
  TLFEA_HIP_CHECK(hipGetLastError());
  me.last_stream = s;
  const tlfea::AsmArgs fa = tlfea::make_args(me, q, v, nullptr, nullptr, 1.0, 0.0);
  if (int rc = tlfea::launch_force_points(me, fa, s)) return rc;
  return tlfea::launch_gradient_blocks(me, v, v_n, f_ext, a.h, f, g, s);
}

}  // namespace

TLFEA_API int tlfea_adamw_solve(tlfea_mesh_t mesh, const tlfea_adamw_params* p, double h, const double* d_q_n,
                                const double* d_v_n, const double* d_f_ext, double* d_v, double* d_q,
                                double* d_work, int32_t max_iters, int32_t check_every, double eps_in,
                                double eps_rel, int32_t* iters_out, double* gnorm_out, void* stream) {
  if (!mesh || !p || !d_q_n || !d_v_n || !d_v || !d_q || !d_work || max_iters < 1 || check_every < 1 ||
      !(h > 0.0) || !std::isfinite(h) || !(p->lr > 0.0) || !(p->beta1 >= 0.0 && p->beta1 < 1.0) ||
      !(p->beta2 >= 0.0 && p->beta2 < 1.0) || !(p->eps > 0.0) || !(p->weight_decay >= 0.0) ||
      !(eps_in >= 0.0) || !(eps_rel >= 0.0))
    return TLFEA_ERR_INVALID;
  Mesh& m = mesh->m;
  if (!m.has_pattern) return TLFEA_ERR_NO_PATTERN;
  if (!m.d_mass) return TLFEA_ERR_INVALID;
  if (hipSetDevice(m.device) != hipSuccess) return TLFEA_ERR_HIP;
  auto s = (hipStream_t)stream;
  if (!s) return TLFEA_ERR_INVALID;  // the legacy stream cannot be captured
  const int64_t n = m.n_dof;
  double* mom = d_work;
  double* sec = d_work + n;
  double* g = d_work + 2 * n;
  double* f = d_work + 3 * n;
  // device scalars: iteration counter, norm partials and norms, then the
  // bias-correction divisors of the next iterations
  const size_t scalars = 2 * tlfea::kNormBlocks + 6;
  if (!m.d_solver) {
    if (hipMalloc(&m.d_solver, sizeof(double) * (scalars + 2 * tlfea::kCorrTable)) != hipSuccess) {
      (void)hipGetLastError();
      m.d_solver = nullptr;
      return TLFEA_ERR_NOMEM;
    }
  }
  auto* d_l = reinterpret_cast<int64_t*>(m.d_solver);
  double* part = m.d_solver + 3;
  double* norms = m.d_solver + 3 + 2 * tlfea::kNormBlocks;
  double* corr = m.d_solver + scalars;
  const tlfea::AdamwArgs a{p->lr, p->beta1, p->beta2, p->eps, p->weight_decay, h};
  // g = m = s = 0 and l = 0 (fill kernels: nothing here is a memset)
  hipLaunchKernelGGL(tlfea::k_fill, dim3(tlfea::blocks_for(3 * n)), dim3(256), 0, s, d_work, 3 * n);
  hipLaunchKernelGGL(tlfea::k_fill, dim3(1), dim3(64), 0, s, m.d_solver, (int64_t)1);
  TLFEA_HIP_CHECK(hipGetLastError());
  auto iterations = [&](int32_t count) -> int {
    int rc = TLFEA_OK;
    for (int32_t done = 0; done < count && !rc;) {
      const int32_t n_corr = std::min<int32_t>(count - done, tlfea::kCorrTable);
      hipLaunchKernelGGL(tlfea::k_corr, dim3(1), dim3(256), 0, s, a, d_l, n_corr, corr);
      TLFEA_HIP_CHECK(hipGetLastError());
      for (int32_t i = 0; i < n_corr && !rc; ++i)
        rc = adamw_iteration(mesh, a, d_q_n, d_v_n, d_f_ext, d_v, d_q, mom, sec, g, f, corr + 2 * i, s);
      done += n_corr;
    }
    return rc;
  };
  auto norms_to_host = [&](double* out) -> int {
    hipLaunchKernelGGL(tlfea::k_norms, dim3(tlfea::kNormBlocks), dim3(256), 0, s, g, d_v, n, part);
    hipLaunchKernelGGL(tlfea::k_norms_final, dim3(1), dim3(tlfea::kNormBlocks), 0, s, part, norms);
    TLFEA_HIP_CHECK(hipGetLastError());
    TLFEA_HIP_CHECK(hipMemcpyAsync(out, norms, 2 * sizeof(double), hipMemcpyDeviceToHost, s));
    TLFEA_HIP_CHECK(hipStreamSynchronize(s));
    return TLFEA_OK;
  };
  // the first iteration runs eagerly: it allocates what the assembly needs and gives g_0
  int rc = iterations(1);
  if (rc) return rc;
  double nrm[2];
  if ((rc = norms_to_host(nrm))) return rc;
  const double g0 = nrm[0];
  int32_t done = 1;
  bool conv = nrm[0] <= eps_in * (1.0 + nrm[1]) || nrm[0] <= eps_rel * g0;
  hipGraphExec_t exec = nullptr;
  int32_t exec_len = 0;
  while (!conv && done < max_iters) {
    const int32_t chunk = std::min<int32_t>(check_every, max_iters - done);
    const bool replay = chunk == exec_len || (max_iters - done) / chunk >= tlfea::kMinReplays;
    if (!replay) {
      if ((rc = iterations(chunk))) {
        if (exec) (void)hipGraphExecDestroy(exec);
        return rc;
      }
    } else if (chunk != exec_len) {
      if (exec) (void)hipGraphExecDestroy(exec);
      exec = nullptr;
      TLFEA_HIP_CHECK(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
      rc = iterations(chunk);
      hipGraph_t graph = nullptr;
      const hipError_t e1 = hipStreamEndCapture(s, &graph);
      hipError_t e2 = hipSuccess;
      if (!rc && e1 == hipSuccess) e2 = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
      if (graph) (void)hipGraphDestroy(graph);
      if (rc || e1 != hipSuccess || e2 != hipSuccess) {
        if (exec) (void)hipGraphExecDestroy(exec);
        (void)hipGetLastError();
        return rc ? rc : TLFEA_ERR_HIP;
      }
      exec_len = chunk;
    }
    if (replay && hipGraphLaunch(exec, s) != hipSuccess) {
      (void)hipGraphExecDestroy(exec);
      return TLFEA_ERR_HIP;
    }
    done += chunk;
    if ((rc = norms_to_host(nrm))) {
      (void)hipGraphExecDestroy(exec);
      return rc;
    }
    conv = nrm[0] <= eps_in * (1.0 + nrm[1]) || nrm[0] <= eps_rel * g0;
  }
  if (exec) (void)hipGraphExecDestroy(exec);
  if (iters_out) *iters_out = done;
  if (gnorm_out) *gnorm_out = nrm[0];
  return TLFEA_OK;
}
