// Forward quantities of the acceptance-oriented training surrogate (Sec. "Acceptance-Oriented
// Training") along target trajectories x*: prefix log-likelihoods of the dependent proposal
// log q(x*_{1:l}) = log sum_z pi_z prod_{j<=l} q_j(x*_j | z) (Eq. cp-drafter) and of the target,
// the importance ratios log r_l (Eq. acceptance-length-objective), the acceptance probabilities
// A_j = min(1, p_j(x*_j) / q(x*_j | x*_<j)) with the conditional as a ratio of consecutive
// prefix likelihoods, S_l = sum_{i<=l} prod_{j<=i} A_j, the truncation l_tau and the per-block
// surrogate J = sum_{l<=l_tau} (log r_l + log S_l) (Eq. subblock-objective), and the marginalised
// block NLL -log q(x*_{1:K}) (Eq. dependent-nll).
//
// One wavefront per block (long blocks; shorter ones take the parallel form below), lane =
// category: each lane accumulates its branch's log-likelihood of
// the trajectory prefix in binary64 and the wavefront takes the log-sum-exp over categories at
// every prefix length. Only K * R gathered branch log-probabilities and K target log-probabilities
// are read per block.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "contract.hpp"
#include "kernels.hpp"
#include "wave.hpp"

namespace dbl {
namespace {

__device__ __forceinline__ double wave_logsumexp(double v) {
  const double m = wave_max_f64(v);
  if (!(m > -INFINITY)) return -INFINITY;
  return m + log(wave_sum_f64(exp(v - m)));
}

__global__ __launch_bounds__(64) void objective_kernel(ObjectiveArgs a) {
  const BlockArgs& k_ = a.blk;
  const int64_t b = blockIdx.x;
  const int lane = lane_id();
  const int R = static_cast<int>(k_.R);
  const int64_t V = k_.V;
  // log pi_z: the prior's log-weights normalised over the categories.
  const double L0 = prior_log_weight(k_.prior + b * k_.R, R, k_.z_temp);
  const double lse0 = wave_logsumexp(lane < R ? L0 : -INFINITY);  // whole wavefront active
  const double log_pi = lane < R ? L0 - lse0 : -INFINITY;
  const double log_tau = log(static_cast<double>(a.tau));
  double cum = log_pi, prev_logq = 0.0, logp_cum = 0.0, prodA = 1.0, S = 0.0, J = 0.0;
  double logq = 0.0;
  int ell_tau = static_cast<int>(k_.K);
  bool done = false;
  for (int64_t j = 0; j < k_.K; ++j) {
    const int32_t x = a.x[b * k_.K + j];
    const bool ok = x >= 0 && x < V;
    const int64_t row = (b * k_.K + j) * k_.R + lane;
    const float lq = ok && lane < R
                         ? flat_lq(k_.tls[row * V + x], k_.lmass[row * k_.nT + x / kTile], k_.lse[row])
                         : -INFINITY;
    cum += static_cast<double>(lq);
    logq = wave_logsumexp(lane < R ? cum : -INFINITY);
    const double lp = ok ? static_cast<double>(a.logp[(b * k_.K + j) * V + x]) : -INFINITY;
    logp_cum += lp;
    const double A = fmin(1.0, exp(lp - (logq - prev_logq)));
    prodA *= A;
    S += prodA;
    const double log_r = logq - logp_cum;
    if (!done) {
      J += log_r + log(S);
      if (log_r < log_tau) {
        done = true;
        ell_tau = static_cast<int>(j) + 1;
      }
    }
    if (lane == 0) {
      if (a.log_r) a.log_r[b * k_.K + j] = static_cast<float>(log_r);
      if (a.S) a.S[b * k_.K + j] = static_cast<float>(S);
    }
    prev_logq = logq;
  }
  if (lane == 0) {
    a.ell_tau[b] = ell_tau;
    a.J[b] = static_cast<float>(J);
    a.nll[b] = static_cast<float>(-logq);
  }
}

// Parallel form of objective_kernel for K * R <= kObjMaxKR and K <= kObjMaxK, one 256-thread
// workgroup per block. The prefix likelihoods depend only on the trajectory, so every position is
// taken at once: the K R + K gathers are issued together, thread (k, z) folds its own prefix
// log pi_z + lq_{0,z} + ... + lq_{k,z} in position order, a segment of lanes per position takes
// the log-sum-exp over categories, and wavefront 0 forms A_j, S_l and J with one position per
// lane, the products and sums over positions in order. The same operations in the same order as
// objective_kernel, whose walk waits for every position's gathers and reductions in turn:
// 39 -> 10 us at 32 blocks with K = R = 16 (expected length and objective together 811 -> 786 us).
constexpr int kObjMaxKR = 2048;
constexpr int kObjMaxK = 256;

__global__ __launch_bounds__(256) void objective_parallel_kernel(ObjectiveArgs a) {
  const BlockArgs& k_ = a.blk;
  const int64_t b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = tid >> 6;
  const int R = static_cast<int>(k_.R);
  const int K = static_cast<int>(k_.K);
  const int KR = K * R;
  const int64_t V = k_.V;
  __shared__ float s_lq[kObjMaxKR];
  __shared__ double s_pi[kMaxR];
  __shared__ double s_logq[kObjMaxK];
  __shared__ double s_lp[kObjMaxK];
  for (int i = tid; i < KR; i += 256) {
    const int k = i / R, z = i % R;
    const int32_t x = a.x[b * k_.K + k];
    const bool ok = x >= 0 && x < V;
    const int64_t v = ok ? x : 0;  // in-bounds loads, unused when the id is out of range
    const int64_t row = (b * k_.K + k) * k_.R + z;
    const float lq = flat_lq(k_.tls[row * V + v], k_.lmass[row * k_.nT + v / kTile], k_.lse[row]);
    s_lq[i] = ok ? lq : -INFINITY;
  }
  for (int k = tid; k < K; k += 256) {
    const int32_t x = a.x[b * k_.K + k];
    const bool ok = x >= 0 && x < V;
    const float lp = a.logp[(b * k_.K + k) * V + (ok ? x : 0)];
    s_lp[k] = ok ? static_cast<double>(lp) : -INFINITY;
  }
  if (wave == 0) {  // log pi_z: the prior's log-weights normalised over the categories
    const double L0 = prior_log_weight(k_.prior + b * k_.R, R, k_.z_temp);
    const double lse0 = wave_logsumexp(lane < R ? L0 : -INFINITY);
    if (lane < R) s_pi[lane] = L0 - lse0;
  }
  __syncthreads();
  // 64 / G positions per wavefront at a time, one segment of G lanes each (lane z = category).
  // The segment's butterfly is the wavefront's, whose other lanes would only add zeros.
  auto prefixes = [&](auto g_c) {
    constexpr int G = decltype(g_c)::value, P = 64 / G;
    const int seg = lane / G, z = lane % G;
    for (int k0 = wave * P; k0 < K; k0 += 4 * P) {
      const int k = k0 + seg;
      const bool own = k < K && z < R;
      double cum = -INFINITY;
      if (own) {
        cum = s_pi[z];
        for (int j = 0; j <= k; ++j) cum += static_cast<double>(s_lq[j * R + z]);
      }
      double m = cum;
#pragma unroll
      for (int o = G / 2; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
      double e = m > -INFINITY ? exp(cum - m) : 0.0;
#pragma unroll
      for (int o = G / 2; o > 0; o >>= 1) e += __shfl_xor(e, o);
      if (k < K && z == 0) s_logq[k] = m > -INFINITY ? m + log(e) : -INFINITY;
    }
  };
  if (R <= 8)
    prefixes(std::integral_constant<int, 8>{});
  else if (R <= 16)
    prefixes(std::integral_constant<int, 16>{});
  else if (R <= 32)
    prefixes(std::integral_constant<int, 32>{});
  else
    prefixes(std::integral_constant<int, 64>{});
  __syncthreads();
  if (wave != 0) return;
  const double log_tau = log(static_cast<double>(a.tau));
  double logp_cum = 0.0, prodA = 1.0, S = 0.0, J = 0.0;
  int ell_tau = K;
  bool done = false;
  for (int k0 = 0; k0 < K; k0 += 64) {
    const int k = k0 + lane;
    const int kn = min(64, K - k0);
    const double logq = k < K ? s_logq[k] : 0.0;
    const double lp = k < K ? s_lp[k] : 0.0;
    const double prev = k > 0 && k < K ? s_logq[k - 1] : 0.0;
    const double A = fmin(1.0, exp(lp - (logq - prev)));
    double my_cum = 0.0, my_S = 1.0;
    for (int j = 0; j < kn; ++j) {  // uniform: every lane takes the same steps
      logp_cum += lane_f64(lp, j);
      prodA *= lane_f64(A, j);
      S += prodA;
      my_cum = j == lane ? logp_cum : my_cum;
      my_S = j == lane ? S : my_S;
    }
    const double log_r = logq - my_cum;
    const double term = log_r + log(my_S);
    const uint64_t low = __ballot(k < K && log_r < log_tau);
    if (!done) {
      const int upto = low ? __ffsll(static_cast<unsigned long long>(low)) : kn;
      for (int j = 0; j < upto; ++j) J += lane_f64(term, j);
      if (low) {
        done = true;
        ell_tau = k0 + upto;
      }
    }
    if (k < K) {
      if (a.log_r) a.log_r[b * k_.K + k] = static_cast<float>(log_r);
      if (a.S) a.S[b * k_.K + k] = static_cast<float>(my_S);
    }
  }
  if (lane == 0) {
    a.ell_tau[b] = ell_tau;
    a.J[b] = static_cast<float>(J);
    a.nll[b] = static_cast<float>(-s_logq[K - 1]);
  }
}

}  // namespace

hipError_t launch_objective(const ObjectiveArgs& a, hipStream_t stream) {
  if (a.blk.B > 0x7fffffff) return hipErrorInvalidConfiguration;
  // Blocks whose gathers fit the parallel form's LDS; the walk only for longer ones.
  if (a.blk.K * a.blk.R <= kObjMaxKR && a.blk.K <= kObjMaxK)
    hipLaunchKernelGGL(objective_parallel_kernel, dim3(static_cast<unsigned>(a.blk.B)), dim3(256),
                       0, stream, a);
  else
    hipLaunchKernelGGL(objective_kernel, dim3(static_cast<unsigned>(a.blk.B)), dim3(64), 0,
                       stream, a);
  return hipGetLastError();
}

}  // namespace dbl
