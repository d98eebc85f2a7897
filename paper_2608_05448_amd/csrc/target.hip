// Target-side sampling transform and early-determinism estimate.
//
// filter   one workgroup per row, or several (split rows, with a workspace): the logits divided by
//          the temperature, restricted by top-k and then top-p, renormalised; -inf outside the kept
//          set. Both cuts are exact selections over order-preserving 32-bit keys of
//          s = fl32(logit / T), in general by radix (four 8-bit digit passes with LDS histograms):
//          by count for top-k (every value equal to the k-th largest is kept), by the determinism
//          contract's integer masses floor(detexp32(fl32(s - max)) 2^40) for top-p, where tokens are
//          taken by decreasing s and, among equal s, increasing id, while the mass before them is
//          below ceil(p * total). Integer histograms make the kept set independent of summation
//          order. Temperature 0 keeps the lowest-index maximum only.
// early_determinism   per sampled block, (1/b) sum_j prod_{i<=j} p(x_i); the estimate is their
//          mean (appendix "Target-Block Early Determinism").
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "contract.hpp"
#include "kernels.hpp"
#include "wave.hpp"

namespace dbl {
namespace {

constexpr int kFT = 1024;  // threads per row
constexpr int kFW = kFT / 64;

__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Workgroup reductions over kFT threads (every thread calls them).
__device__ __forceinline__ uint64_t block_sum_u64(uint64_t v, uint64_t* red) {
  v = wave_sum_u64(v);
  if (lane_id() == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint64_t s = 0;
#pragma unroll
  for (int w = 0; w < kFW; ++w) s += red[w];
  __syncthreads();
  return s;
}

__device__ __forceinline__ double block_sum_f64(double v, double* red) {
  v = wave_sum_f64(v);
  if (lane_id() == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < kFW; ++w) s += red[w];
  __syncthreads();
  return s;
}

__device__ __forceinline__ uint64_t block_max_u64(uint64_t v, uint64_t* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t t = __shfl_xor(v, o);
    v = t > v ? t : v;
  }
  if (lane_id() == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint64_t m = 0;
#pragma unroll
  for (int w = 0; w < kFW; ++w) m = red[w] > m ? red[w] : m;
  __syncthreads();
  return m;
}

// Picks, from a 256-bin histogram of the current digit (largest digit first), the digit whose
// bin holds the `need`-th unit counted from the top; returns it and what lies in larger digits.
__device__ __forceinline__ void pick_digit(const uint64_t* hist, uint64_t need, uint32_t* digit,
                                           uint64_t* above, uint32_t* sh_digit,
                                           uint64_t* sh_above) {
  if (threadIdx.x == 0) {
    uint64_t acc = 0;
    int d = 255;
    for (; d > 0; --d) {
      if (acc + hist[d] >= need) break;
      acc += hist[d];
    }
    *sh_digit = static_cast<uint32_t>(d);
    *sh_above = acc;
  }
  __syncthreads();
  *digit = *sh_digit;
  *above = *sh_above;
  __syncthreads();
}

// Calls fn(v, logit(v)) for every id of the row. When the row is 16-byte aligned and V is a
// multiple of 4 the loads are float4, issued kB at a time per thread so that one workgroup keeps
// enough bytes in flight to stream its row.
constexpr int kBatch = 8;

template <int kB = kBatch, class F>
__device__ __forceinline__ void row_scan_raw(const float* in, int64_t V, bool vec, F fn) {
  if (vec) {
    const float4* in4 = reinterpret_cast<const float4*>(in);
    const int64_t n4 = V >> 2;
    auto one = [&](int64_t j, const float4& x) {
      fn(4 * j, x.x);
      fn(4 * j + 1, x.y);
      fn(4 * j + 2, x.z);
      fn(4 * j + 3, x.w);
    };
    int64_t j = threadIdx.x;
    for (; j + (kB - 1) * kFT < n4; j += kB * kFT) {
      float4 x[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) x[u] = in4[j + u * kFT];
#pragma unroll
      for (int u = 0; u < kB; ++u) one(j + u * kFT, x[u]);
    }
    for (; j < n4; j += kFT) one(j, in4[j]);
  } else {
    for (int64_t v = threadIdx.x; v < V; v += kFT) fn(v, in[v]);
  }
}

// As row_scan_raw, with fn(v, s(v)), s(v) = fl32(logit(v) / T).
template <int kB = kBatch, class F>
__device__ __forceinline__ void row_scan(const float* in, int64_t V, float T, bool vec, F fn) {
  row_scan_raw<kB>(in, V, vec, [&](int64_t v, float x) { fn(v, __fdiv_rn(x, T)); });
}

__device__ __forceinline__ float key_value(uint32_t x) {
  return __uint_as_float((x & 0x80000000u) ? (x & 0x7FFFFFFFu) : ~x);
}

constexpr uint32_t kKeyNegInf = 0x007FFFFFu;  // order_key(-inf)
constexpr uint32_t kKeyPosInf = 0xFF800000u;  // order_key(+inf)

// Rounded division by T > 0 is monotone (non-decreasing) in the dividend, so the logits x with
// fl32(x / T) >= s form an upper set in key order. Returns its least key: a bisection over the
// keys of the non-NaN floats, every thread computing the same value.
__device__ __forceinline__ uint32_t least_logit_key(uint32_t s_key, float T) {
  auto ok = [&](uint32_t k) { return order_key(__fdiv_rn(key_value(k), T)) >= s_key; };
  if (ok(kKeyNegInf)) return kKeyNegInf;
  uint32_t lo = kKeyNegInf, hi = kKeyPosInf;  // ok(lo) false, ok(hi) true
  while (hi - lo > 1) {
    const uint32_t mid = lo + (hi - lo) / 2;
    if (ok(mid)) hi = mid; else lo = mid;
  }
  return hi;
}

// Sort key of a token: key(s) in the high word, ~id in the low word, so that a descending order
// visits tokens by decreasing s and, among equal s, increasing id.
__device__ __forceinline__ uint64_t visit_key(uint32_t key, int64_t v) {
  return (static_cast<uint64_t>(key) << 32) | (0xFFFFFFFFu - static_cast<uint32_t>(v));
}

// k-th largest of the 64 x 4 keys held by a wavefront (k <= 256): the largest t with at least k
// of them >= t, by bisection with ballots; no LDS, no barrier.
__device__ __forceinline__ uint32_t wave_kth_largest(uint32_t t0, uint32_t t1, uint32_t t2,
                                                     uint32_t t3, int k) {
  uint64_t lo = 0, hi = 0xFFFFFFFFu;  // count(>= lo) >= k always (every key is >= 0)
  while (lo < hi) {
    const uint64_t mid = lo + (hi - lo + 1) / 2;
    const uint32_t m32 = static_cast<uint32_t>(mid);
    const int c = __popcll(__ballot(t0 >= m32)) + __popcll(__ballot(t1 >= m32)) +
                  __popcll(__ballot(t2 >= m32)) + __popcll(__ballot(t3 >= m32));
    if (c >= k) lo = mid; else hi = mid - 1;
  }
  return static_cast<uint32_t>(lo);
}

// Fast path for top-k (0 < k <= kFastK < V): one streaming read and one streaming write of the
// row (fl32(x / T) is monotone in x, so selections on s are made on the logits' keys and only
// candidates are divided):
//   1. every thread writes -inf over its part of the output row and keeps the four largest logit
//      keys it sees;
//   2. a lower bound t of the row's k-th largest key: the largest over wavefronts of each
//      wavefront's k-th largest held key (k <= 256), else the k-th largest of all 4096 held keys
//      (workgroup bisection); each is the k-th largest of part of the row;
//   3. only threads holding a key >= x_low = least_logit_key(fl32(t / T)) can own a token with
//      s >= fl32(t / T) (their other logits are below their fourth largest); they re-read their
//      own ids and append every such token, with its s, to an LDS list;
//   4. the list is sorted in visiting order (s descending, id ascending); both cuts and the
//      normaliser follow from it, and the kept tokens' log-probabilities overwrite the -inf.
// Returns false (the caller then runs the radix path, which rewrites the whole row) if the list
// would overflow LDS.
constexpr int kFastK = 1024;
constexpr int kCandCap = 4096;

// Sorts cand[0, n) (n <= kCandCap, all keys different and nonzero) in descending order; all kFT
// threads call it, and it ends with a barrier. Up to kRankMax keys, each thread counts the keys
// larger than its own (LDS reads that all lanes share) and stores its key at that place: two
// barriers, about 14 cycles per key, where the network below takes 300 per stage (28 stages for
// 128 keys, 45 for 512). Above, a bitonic network over the list padded with zeros to a power of two
// (every visiting key has a nonzero low word, ids being below 2^32 - 1).
constexpr int kRankMax = 512;

__device__ void block_sort_desc(uint64_t* cand, int n) {
  const int tid = threadIdx.x;
  if (n <= kRankMax) {
    const uint64_t mine = tid < n ? cand[tid] : 0;
    int rank = 0;
    if (tid < n) {
#pragma unroll 8
      for (int j = 0; j < n; ++j) rank += cand[j] > mine ? 1 : 0;
    }
    __syncthreads();
    if (tid < n) cand[rank] = mine;
    __syncthreads();
    return;
  }
  int np = 64;
  while (np < n) np <<= 1;
  for (int i = n + tid; i < np; i += kFT) cand[i] = 0;
  __syncthreads();
  for (int size = 2; size <= np; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = tid; i < (np >> 1); i += kFT) {
        const int i0 = 2 * i - (i & (stride - 1));  // the pair (i0, i0 + stride)
        const int i1 = i0 + stride;
        const bool desc = (i0 & size) == 0;
        const uint64_t x = cand[i0], y = cand[i1];
        if ((x < y) == desc) {
          cand[i0] = y;
          cand[i1] = x;
        }
      }
      __syncthreads();
    }
  }
}

// Wavefront 0 alone, when the tokens tied with or above the k-th largest s number at most 64
// (the usual case for small k): e is lane l's token, the l-th in visiting order (0 from lane nk on);
// both cuts and the normaliser are wavefront reductions, with no workgroup barrier.
__device__ void finish_small(const FilterArgs& a, float* out, uint64_t e, int nk) {
  const int lane = lane_id();
  const float sv = key_value(static_cast<uint32_t>(e >> 32));
  const float m = __shfl(sv, 0);
  int nkeep = nk;
  if (a.top_p < 1.0f) {
    const uint64_t P = lane < nk ? quant_detexp32(__fsub_rn(sv, m)) : 0;
    const uint64_t incl = wave_incl_scan_u64(P);
    const uint64_t z = __shfl(incl, 63);
    uint64_t tp = static_cast<uint64_t>(ceil(__dmul_rn(static_cast<double>(a.top_p),
                                                       static_cast<double>(z))));
    if (tp == 0) tp = 1;
    nkeep = __popcll(__ballot(lane < nk && incl - P < tp));
  }
  const double x = lane < nkeep ? exp(static_cast<double>(sv) - static_cast<double>(m)) : 0.0;
  const double lse = log(wave_sum_f64(x));
  if (lane < nkeep) {
    const int64_t v = 0xFFFFFFFFu - static_cast<uint32_t>(e);
    out[v] = static_cast<float>(static_cast<double>(sv) - static_cast<double>(m) - lse);
  }
}

// Both cuts, the normaliser and the kept tokens of a list sorted in visiting order that holds every
// token at or above the row's k-th largest s (n >= k). All kFT threads call it.
__device__ void finish_sorted(const FilterArgs& a, float* out, const uint64_t* cand, int n,
                              uint64_t* red, double* redd) {
  const int tid = threadIdx.x;
  const int k = static_cast<int>(a.top_k);
  auto key_at = [&](int i) { return static_cast<uint32_t>(cand[i] >> 32); };
  const float m = key_value(key_at(0));
  // top-k: the first k entries and every later one tied with the k-th (n >= k: the list holds
  // every token at or above the row's k-th largest key)
  const uint32_t tk = key_at(k - 1);
  int nk = k;
  while (nk < n && key_at(nk) >= tk) ++nk;
  int nkeep = nk;
  if (a.top_p < 1.0f) {
    // integer masses of the first nk entries, four per thread in list order; a token is kept
    // while the mass before it is below T_p = ceil(p Z)
    uint64_t P[4], loc = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = 4 * tid + j;
      P[j] = i < nk ? quant_detexp32(__fsub_rn(key_value(key_at(i)), m)) : 0;
      loc += P[j];
    }
    const uint64_t incl = wave_incl_scan_u64(loc);
    if (lane_id() == 63) red[tid >> 6] = incl;
    __syncthreads();
    uint64_t base = 0, z = 0;
#pragma unroll
    for (int w = 0; w < kFW; ++w) {
      const uint64_t r = red[w];
      base += w < (tid >> 6) ? r : 0;
      z += r;
    }
    __syncthreads();
    uint64_t tp = static_cast<uint64_t>(ceil(__dmul_rn(static_cast<double>(a.top_p),
                                                       static_cast<double>(z))));
    if (tp == 0) tp = 1;
    uint64_t before = base + incl - loc;
    uint64_t c = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (4 * tid + j < nk) {
        c += before < tp ? 1 : 0;
        before += P[j];
      }
    }
    nkeep = static_cast<int>(block_sum_u64(c, red));
  }
  double se = 0.0;
  for (int i = tid; i < nkeep; i += kFT)
    se += exp(static_cast<double>(key_value(key_at(i))) - static_cast<double>(m));
  const double lse = log(block_sum_f64(se, redd));
  // kept tokens (the first nkeep entries of the list)
  for (int i = tid; i < nkeep; i += kFT) {
    const uint64_t e = cand[i];
    const int64_t v = 0xFFFFFFFFu - static_cast<uint32_t>(e);
    out[v] = static_cast<float>(static_cast<double>(key_value(static_cast<uint32_t>(e >> 32))) -
                                static_cast<double>(m) - lse);
  }
}

// Wavefront 0: moves the nk (<= 64) entries of cand[0, n) with key >= tk to the front, in list
// order (an entry moves only towards the front, past entries this wavefront has already read).
__device__ void front_small(uint64_t* cand, int n, uint32_t tk) {
  const int lane = lane_id();
  int base = 0;
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int i = i0 + lane;
    const uint64_t c = i < n ? cand[i] : 0;
    const bool in = i < n && static_cast<uint32_t>(c >> 32) >= tk;
    const uint64_t msk = __ballot(in);
    if (in) cand[base + __popcll(msk & ((1ull << lane) - 1))] = c;
    base += __popcll(msk);
    asm volatile("" ::: "memory");
  }
}

// Sorts a candidate list - visiting keys (key of s, ~id) of every token whose s is at least a
// lower bound of the row's k-th largest s - in visiting order (s descending, id ascending),
// applies both cuts and writes the kept tokens' log-probabilities; the rest of the output row
// already holds -inf. Needs n >= k and n <= kCandCap; all kFT threads call it.
__device__ void finish_candidates(const FilterArgs& a, float* out, uint64_t* cand, int n,
                                  uint64_t* red, double* redd) {
  const int tid = threadIdx.x;
  const int k = static_cast<int>(a.top_k);
  // Wavefront 0: the k-th largest key of the list (bisection with ballots over the list) and
  // how many entries are at or above it.
  if (tid < 64) {
    uint64_t lo = 0, hi = 0xFFFFFFFFu;
    int c = 0;
    if (n <= 8 * 64) {  // up to 8 keys per lane, in registers; counts by ballot
      uint32_t kk[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = tid + 64 * j;
        kk[j] = i < n ? static_cast<uint32_t>(cand[i] >> 32) : 0;
      }
      auto count = [&](uint32_t t) {
        int r = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) r += __popcll(__ballot(kk[j] >= t && tid + 64 * j < n));
        return r;
      };
      uint32_t top = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) top = max(top, kk[j]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) top = max(top, static_cast<uint32_t>(__shfl_xor(top, o)));
      hi = top;
      while (lo < hi) {
        const uint64_t mid = lo + (hi - lo + 1) / 2;
        if (count(static_cast<uint32_t>(mid)) >= k) lo = mid; else hi = mid - 1;
      }
      c = count(static_cast<uint32_t>(lo));
    } else {
      auto count = [&](uint64_t t) {
        int r = 0;
        for (int i = tid; i < n; i += 64) r += static_cast<uint32_t>(cand[i] >> 32) >= t ? 1 : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o);
        return r;
      };
      while (lo < hi) {
        const uint64_t mid = lo + (hi - lo + 1) / 2;
        if (count(mid) >= k) lo = mid; else hi = mid - 1;
      }
      c = count(lo);
    }
    if (tid == 0) {
      red[0] = lo;
      red[1] = static_cast<uint64_t>(c);
    }
  }
  __syncthreads();
  const uint32_t tk0 = static_cast<uint32_t>(red[0]);
  const int nk0 = static_cast<int>(red[1]);
  __syncthreads();
  if (nk0 <= 64) {
    if (tid < 64) {
      front_small(cand, n, tk0);
      // each lane counts the larger keys (all differ) for its place in visiting order
      const uint64_t mine = tid < nk0 ? cand[tid] : 0;
      int rank = 0;
#pragma unroll 4
      for (int j = 0; j < nk0; ++j) rank += lane_u64(mine, j) > mine ? 1 : 0;
      asm volatile("" ::: "memory");
      if (tid < nk0) cand[rank] = mine;
      asm volatile("" ::: "memory");
      finish_small(a, out, tid < nk0 ? cand[tid] : 0, nk0);
    }
    return;
  }
  block_sort_desc(cand, n);
  finish_sorted(a, out, cand, n, red, redd);
}

__device__ bool filter_fast(const FilterArgs& a, const float* in, float* out, bool vec,
                            uint64_t* cand, int* resc, uint64_t* red, double* redd, int* sh_n,
                            int* sh_r) {
  const int tid = threadIdx.x;
  const int64_t V = a.V;
  const float T = a.temperature;
  const int k = static_cast<int>(a.top_k);
  // 1. -inf over the row; per-thread top-4 logit keys
  uint32_t t0 = 0, t1 = 0, t2 = 0, t3 = 0;
  auto insert = [&](float lv) {
    uint32_t x = order_key(lv);  // insertion into t0 >= t1 >= t2 >= t3, branch-free
    uint32_t y = max(t0, x);
    x = min(t0, x);
    t0 = y;
    y = max(t1, x);
    x = min(t1, x);
    t1 = y;
    y = max(t2, x);
    x = min(t2, x);
    t2 = y;
    t3 = max(t3, x);
  };
  if (vec) {
    const float4* in4 = reinterpret_cast<const float4*>(in);
    float4* out4 = reinterpret_cast<float4*>(out);
    const int64_t n4 = V >> 2;
    const float4 ninf = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    int64_t j = tid;
    for (; j + (kBatch - 1) * kFT < n4; j += kBatch * kFT) {
      float4 x[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) x[u] = in4[j + u * kFT];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        out4[j + u * kFT] = ninf;
        insert(x[u].x);
        insert(x[u].y);
        insert(x[u].z);
        insert(x[u].w);
      }
    }
    for (; j < n4; j += kFT) {
      const float4 x = in4[j];
      out4[j] = ninf;
      insert(x.x);
      insert(x.y);
      insert(x.z);
      insert(x.w);
    }
  } else {
    for (int64_t v = tid; v < V; v += kFT) {
      insert(in[v]);
      out[v] = -INFINITY;
    }
  }
  // The kept tokens' values are stored later, possibly by other threads, over these -inf: wait
  // for this thread's stores before the barriers that follow.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // 2. lower bound of the row's k-th largest logit key
  uint32_t tlow;
  if (k <= 256) {
    tlow = static_cast<uint32_t>(block_max_u64(wave_kth_largest(t0, t1, t2, t3, k), red));
  } else {
    uint64_t lo = 0, hi = block_max_u64(t0, red);
    while (lo < hi) {
      const uint64_t mid = lo + (hi - lo + 1) / 2;
      const uint32_t m32 = static_cast<uint32_t>(mid);
      const uint32_t c = __popcll(__ballot(t0 >= m32)) + __popcll(__ballot(t1 >= m32)) +
                         __popcll(__ballot(t2 >= m32)) + __popcll(__ballot(t3 >= m32));
      if (lane_id() == 0) red[tid >> 6] = c;
      __syncthreads();
      uint64_t tot = 0;
#pragma unroll
      for (int w = 0; w < kFW; ++w) tot += red[w];
      __syncthreads();
      if (tot >= static_cast<uint64_t>(k)) lo = mid; else hi = mid - 1;
    }
    tlow = static_cast<uint32_t>(lo);
  }
  const uint32_t s_low = order_key(__fdiv_rn(key_value(tlow), T));
  const uint32_t x_low = least_logit_key(s_low, T);
  // 3. candidates from the threads that hold a key >= x_low: their ids are re-read by the whole
  //    workgroup (item w = (listed thread w / G, its w % G-th load), G loads per thread)
  if (tid == 0) {
    *sh_n = 0;
    *sh_r = 0;
  }
  __syncthreads();
  if (t0 >= x_low) resc[atomicAdd(sh_r, 1)] = tid;
  __syncthreads();
  const int nr = *sh_r;
  const int64_t units = vec ? (V >> 2) : V;              // float4 groups or single ids
  const int G = static_cast<int>((units + kFT - 1) / kFT);  // loads per thread, at most
  const int64_t items = static_cast<int64_t>(nr) * G;
  auto take = [&](int64_t v, float lv) {
    if (order_key(lv) >= x_low) {
      const int slot = atomicAdd(sh_n, 1);
      if (slot < kCandCap) cand[slot] = visit_key(order_key(__fdiv_rn(lv, T)), v);
    }
  };
  for (int64_t w0 = tid; w0 < items; w0 += kBatch * kFT) {
    int64_t jj[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int64_t w = w0 + static_cast<int64_t>(b) * kFT;
      const int64_t j = w < items ? resc[w / G] + (w % G) * static_cast<int64_t>(kFT) : units;
      jj[b] = j < units ? j : -1;
    }
    if (vec) {
      const float4* in4 = reinterpret_cast<const float4*>(in);
      float4 x[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) x[b] = jj[b] >= 0 ? in4[jj[b]] : make_float4(0, 0, 0, 0);
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        if (jj[b] < 0) continue;
        take(4 * jj[b], x[b].x);
        take(4 * jj[b] + 1, x[b].y);
        take(4 * jj[b] + 2, x[b].z);
        take(4 * jj[b] + 3, x[b].w);
      }
    } else {
      float x[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) x[b] = jj[b] >= 0 ? in[jj[b]] : 0.0f;
#pragma unroll
      for (int b = 0; b < kBatch; ++b)
        if (jj[b] >= 0) take(jj[b], x[b]);
    }
  }
  __syncthreads();
  const int n = *sh_n;
  __syncthreads();
  if (n > kCandCap) return false;
  finish_candidates(a, out, cand, n, red, redd);
  return true;
}

// General path: exact radix selections over the keys of s (every k, and the nucleus alone),
// reading the row several times and writing all of it. MAX: m_known is the row's largest s.
template <bool MAX = false>
__device__ void filter_general(const FilterArgs& a, const float* in, float* out, bool vec,
                               uint64_t* hist, uint64_t* red, double* redd, uint32_t* sh_digit,
                               uint64_t* sh_above, float m_known = 0.0f) {
  const int tid = threadIdx.x;
  const int64_t V = a.V;
  const float T = a.temperature;
  auto s_of = [&](int64_t v) { return __fdiv_rn(in[v], T); };
  float m = m_known;
  if constexpr (!MAX) {  // row maximum (key of the largest s)
    uint32_t mk = 0;
    row_scan<4>(in, V, T, vec, [&](int64_t, float sv) {
      const uint32_t k = order_key(sv);
      mk = k > mk ? k : mk;
    });
    m = key_value(static_cast<uint32_t>(block_max_u64(mk, red)));
  }

  // Top-k: the k-th largest key, by count.
  uint32_t tk = 0;  // keep keys >= tk
  if (a.top_k > 0 && a.top_k < V) {
    uint32_t prefix = 0, pmask = 0;
    uint64_t need = static_cast<uint64_t>(a.top_k);
    for (int shift = 24; shift >= 0; shift -= 8) {
      for (int i = tid; i < 256; i += kFT) hist[i] = 0;
      __syncthreads();
      row_scan<4>(in, V, T, vec, [&](int64_t, float sv) {
        const uint32_t k = order_key(sv);
        if ((k & pmask) == prefix)
          atomicAdd(reinterpret_cast<unsigned long long*>(&hist[(k >> shift) & 255]), 1ull);
      });
      __syncthreads();
      uint32_t d;
      uint64_t above;
      pick_digit(hist, need, &d, &above, sh_digit, sh_above);
      need -= above;
      prefix |= d << shift;
      pmask |= 255u << shift;
    }
    tk = prefix;
  }

  // Top-p: the crossing key by integer mass, then how many of the tokens at it are kept.
  uint32_t tp = 0;          // keep keys > tp, and the first n_tie tokens with key == tp
  uint64_t n_tie = ~0ull;
  if (a.top_p < 1.0f) {
    auto mass = [&](float sv, uint32_t k) -> uint64_t {
      return k >= tk ? quant_detexp32(__fsub_rn(sv, m)) : 0;
    };
    uint32_t prefix = 0, pmask = 0;
    uint64_t need = 0, tie_mass = 0;
    for (int shift = 24; shift >= 0; shift -= 8) {
      for (int i = tid; i < 256; i += kFT) hist[i] = 0;
      __syncthreads();
      row_scan<4>(in, V, T, vec, [&](int64_t, float sv) {
        const uint32_t k = order_key(sv);
        if ((k & pmask) == prefix) {
          const uint64_t P = mass(sv, k);
          if (P) atomicAdd(reinterpret_cast<unsigned long long*>(&hist[(k >> shift) & 255]),
                           static_cast<unsigned long long>(P));
        }
      });
      __syncthreads();
      if (shift == 24) {  // total mass of the kept set: T_p = ceil(p Z)
        uint64_t z = 0;
        for (int i = 0; i < 256; ++i) z += hist[i];
        need = static_cast<uint64_t>(ceil(__dmul_rn(static_cast<double>(a.top_p),
                                                    static_cast<double>(z))));
        if (need == 0) need = 1;
      }
      uint32_t d;
      uint64_t above;
      pick_digit(hist, need, &d, &above, sh_digit, sh_above);
      need -= above;
      if (shift == 0) tie_mass = hist[d];
      prefix |= d << shift;
      pmask |= 255u << shift;
    }
    tp = prefix;
    // Every token at key tp has the same mass; count how many of them there are.
    uint64_t cnt = 0;
    row_scan<4>(in, V, T, vec, [&](int64_t, float sv) { cnt += order_key(sv) == tp ? 1 : 0; });
    cnt = block_sum_u64(cnt, red);
    const uint64_t each = tie_mass / cnt;
    n_tie = (need + each - 1) / each;  // tokens at tp needed to reach T_p
    if (n_tie >= cnt) n_tie = ~0ull;
  }

  // Rank among the tokens at key tp (increasing id) when only some of them are kept: each
  // thread owns a contiguous run of ids.
  const int64_t per = (V + kFT - 1) / kFT;
  const int64_t r0 = min(V, tid * per), r1 = min(V, r0 + per);
  uint64_t tie_before = 0;
  if (n_tie != ~0ull) {
    uint64_t c = 0;
    for (int64_t v = r0; v < r1; ++v) c += order_key(s_of(v)) == tp ? 1 : 0;
    // exclusive scan of c over threads
    uint64_t incl = wave_incl_scan_u64(c);
    if (lane_id() == 63) red[tid >> 6] = incl;
    __syncthreads();
    uint64_t base = 0;
    for (int w = 0; w < (tid >> 6); ++w) base += red[w];
    __syncthreads();
    tie_before = base + incl - c;
  }
  auto kept = [&](int64_t v, uint32_t k, uint64_t rank) {
    if (k < tk) return false;
    if (a.top_p < 1.0f) {
      if (k < tp) return false;
      if (k == tp && n_tie != ~0ull && rank >= n_tie) return false;
    }
    return true;
  };

  // Normaliser over the kept set, then the output row: strided (coalesced) passes unless only
  // some of the tokens at the top-p cut are kept, which needs the id-ordered runs.
  auto pass = [&](auto fn) {
    if (n_tie == ~0ull) {
      row_scan<4>(in, V, T, vec, [&](int64_t v, float sv) { fn(v, sv, 0ull); });
    } else {
      uint64_t rank = tie_before;
      for (int64_t v = r0; v < r1; ++v) {
        const float sv = s_of(v);
        fn(v, sv, rank);
        if (order_key(sv) == tp) ++rank;
      }
    }
  };
  double se = 0.0;
  pass([&](int64_t v, float s, uint64_t rank) {
    if (kept(v, order_key(s), rank)) se += exp(static_cast<double>(s) - static_cast<double>(m));
  });
  const double lse = log(block_sum_f64(se, redd));
  pass([&](int64_t v, float s, uint64_t rank) {
    out[v] = kept(v, order_key(s), rank)
                 ? static_cast<float>(static_cast<double>(s) - static_cast<double>(m) - lse)
                 : -INFINITY;
  });
}

// Nucleus alone (top_k off, p < 1): with m the row maximum, every token's integer mass
// P(v) = floor(detexp32(fl32(s - m)) 2^40) goes to one of kNucBins bins by
// floor((m - s) kNucScale), which is non-increasing in s, so bins are ordered like s and tokens
// of one bin are contiguous in visiting order. The bin where the running mass reaches
// T_p = ceil(p Z) is the only one whose tokens need ordering: they are gathered and sorted, and
// the cut is found in it. Tokens with P = 0 follow all positive masses, whose total Z >= T_p, so
// they are never kept. The normaliser is the kept integer mass times 2^-40, within 2^-40 per
// token plus detexp32's rounding of the binary64 sum of exp(s - m). Four reads and one write of
// the row. Returns false (nothing written) if the cut's bin holds more than kCandCap tokens.
constexpr int kNucBins = 2048;
constexpr float kNucScale = kNucBins / 27.8f;  // P(v) = 0 below s - m = -40 ln 2 = -27.73
// Every token of a bin <= kNucSureBin has s - m > -27.16, so detexp32 > 1.5e-12 > 2^-40 and
// P(v) >= 1: when the cut's bin is one of them, the later passes need only the bins.
constexpr int kNucSureBin = 2000;

// The bin where the running mass of a row's bins (b0, b1: this thread's bins 2 tid and 2 tid + 1)
// reaches T_p = ceil(p Z), the mass before it and T_p. False if the row has no mass (no finite
// logit). All kFT threads call it; it starts and ends with a barrier.
__device__ __forceinline__ bool nucleus_crossing(uint64_t b0, uint64_t b1, float top_p,
                                                 uint64_t* red, int* bstar, uint64_t* before,
                                                 uint64_t* tp_out) {
  const int tid = threadIdx.x;
  const uint64_t loc = b0 + b1;
  const uint64_t incl = wave_incl_scan_u64(loc);
  __syncthreads();
  if (lane_id() == 63) red[tid >> 6] = incl;
  __syncthreads();
  uint64_t base = 0, z = 0;
#pragma unroll
  for (int w = 0; w < kFW; ++w) {
    const uint64_t r = red[w];
    base += w < (tid >> 6) ? r : 0;
    z += r;
  }
  __syncthreads();
  uint64_t tp = static_cast<uint64_t>(ceil(__dmul_rn(static_cast<double>(top_p),
                                                     static_cast<double>(z))));
  if (tp == 0) tp = 1;
  const uint64_t ex0 = base + incl - loc, ex1 = ex0 + b0;  // mass before bins 2 tid, 2 tid + 1
  if (ex0 < tp && tp <= ex1) {
    red[0] = 2 * tid;
    red[1] = ex0;
  } else if (ex1 < tp && tp <= ex1 + b1) {
    red[0] = 2 * tid + 1;
    red[1] = ex1;
  }
  __syncthreads();
  *bstar = static_cast<int>(red[0]);
  *before = red[1];
  *tp_out = tp;
  __syncthreads();
  return z > 0;
}

// Orders the crossing bin's n tokens (0 < n <= kCandCap, `before` the mass of the earlier bins)
// and takes those whose preceding mass is below T_p: returns the log-normaliser of the kept set,
// relative to the row's maximum m, and in `cut` the last kept token's visiting key.
__device__ __forceinline__ double nucleus_kept(uint64_t* cand, int n, float m, uint64_t before,
                                               uint64_t tp, uint64_t* red, uint64_t* cut) {
  const int tid = threadIdx.x;
  block_sort_desc(cand, n);
  // kept prefix of the bin: four entries per thread in visiting order
  uint64_t P4[4], l4 = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = 4 * tid + j;
    P4[j] = i < n ? quant_detexp32(__fsub_rn(key_value(static_cast<uint32_t>(cand[i] >> 32)), m)) : 0;
    l4 += P4[j];
  }
  const uint64_t inc4 = wave_incl_scan_u64(l4);
  if (lane_id() == 63) red[tid >> 6] = inc4;
  __syncthreads();
  uint64_t base4 = 0;
#pragma unroll
  for (int w = 0; w < kFW; ++w) base4 += w < (tid >> 6) ? red[w] : 0;
  __syncthreads();
  uint64_t run = before + base4 + inc4 - l4;
  uint64_t cnt = 0, kept_mass = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (4 * tid + j < n && run < tp) {
      ++cnt;
      kept_mass += P4[j];
    }
    run += P4[j];
  }
  const uint64_t nkeep = block_sum_u64(cnt, red);
  const uint64_t kmass = before + block_sum_u64(kept_mass, red);
  *cut = cand[nkeep - 1];
  return log(static_cast<double>(kmass)) - 40.0 * 0.6931471805599453;
}

__device__ bool filter_nucleus(const FilterArgs& a, const float* in, float* out, bool vec,
                               uint64_t* bins, uint64_t* cand, uint64_t* red, int* sh_n) {
  const int tid = threadIdx.x;
  const int64_t V = a.V;
  const float T = a.temperature;
  // 1. maximum (division by T is monotone: the largest s is that of the largest logit)
  uint32_t mk = 0;
  row_scan_raw<4>(in, V, vec, [&](int64_t, float lv) {
    const uint32_t x = order_key(lv);
    mk = x > mk ? x : mk;
  });
  const float m = __fdiv_rn(key_value(static_cast<uint32_t>(block_max_u64(mk, red))), T);
  // s = fl32(x / T); x / 1 is x exactly, so T = 1 needs no division
  auto scan = [&](auto fn) {
    if (T == 1.0f)
      row_scan_raw<2>(in, V, vec, fn);
    else
      row_scan<2>(in, V, T, vec, fn);
  };
  auto mass_bin = [&](float sv, uint64_t* P) {
    const float d = __fsub_rn(sv, m);
    *P = quant_detexp32(d);
    return min(kNucBins - 1, static_cast<int>(__fmul_rn(-d, kNucScale)));
  };
  // 2. integer mass per bin
  for (int i = tid; i < kNucBins; i += kFT) bins[i] = 0;
  __syncthreads();
  scan([&](int64_t, float sv) {
    uint64_t P;
    const int b = mass_bin(sv, &P);
    if (P) atomicAdd(reinterpret_cast<unsigned long long*>(&bins[b]), static_cast<unsigned long long>(P));
  });
  __syncthreads();
  if (tid == 0) *sh_n = 0;
  const uint64_t b0 = bins[2 * tid], b1 = bins[2 * tid + 1];
  __syncthreads();
  int bstar;
  uint64_t before, tp;
  if (!nucleus_crossing(b0, b1, a.top_p, red, &bstar, &before, &tp)) return false;
  auto bin_of = [&](float sv) {
    return min(kNucBins - 1, static_cast<int>(__fmul_rn(-__fsub_rn(sv, m), kNucScale)));
  };
  const bool sure = bstar <= kNucSureBin;
  // 3. the crossing bin's tokens, then their order
  if (sure) {
    scan([&](int64_t v, float sv) {
      if (bin_of(sv) == bstar) {
        const int slot = atomicAdd(sh_n, 1);
        if (slot < kCandCap) cand[slot] = visit_key(order_key(sv), v);
      }
    });
  } else {
    scan([&](int64_t v, float sv) {
      uint64_t P;
      if (mass_bin(sv, &P) == bstar && P) {
        const int slot = atomicAdd(sh_n, 1);
        if (slot < kCandCap) cand[slot] = visit_key(order_key(sv), v);
      }
    });
  }
  __syncthreads();
  const int n = *sh_n;
  __syncthreads();
  if (n > kCandCap) return false;
  uint64_t cut;
  const double lse = nucleus_kept(cand, n, m, before, tp, red, &cut);
  // 4. output row
  if (sure) {
    scan([&](int64_t v, float sv) {
      const int b = bin_of(sv);
      const bool kept = b < bstar || (b == bstar && visit_key(order_key(sv), v) >= cut);
      out[v] = kept ? static_cast<float>(static_cast<double>(sv) - static_cast<double>(m) - lse)
                    : -INFINITY;
    });
  } else {
    scan([&](int64_t v, float sv) {
      uint64_t P;
      const int b = mass_bin(sv, &P);
      const bool kept = P && (b < bstar || (b == bstar && visit_key(order_key(sv), v) >= cut));
      out[v] = kept ? static_cast<float>(static_cast<double>(sv) - static_cast<double>(m) - lse)
                    : -INFINITY;
    });
  }
  return true;
}

// Rows with the nucleus alone (T > 0, top_k off, p < 1): the binned path, or the general one
// when the cut's bin is too crowded.
__global__ __launch_bounds__(kFT) void filter_nucleus_kernel(FilterArgs a) {
  __shared__ uint64_t hist[256];
  __shared__ uint64_t nbins[kNucBins];
  __shared__ uint64_t cand[kCandCap];
  __shared__ int sh_n;
  __shared__ uint64_t red[kFW];
  __shared__ double redd[kFW];
  __shared__ uint32_t sh_digit;
  __shared__ uint64_t sh_above;
  const int64_t n = blockIdx.x;
  const int64_t V = a.V;
  const float* in = a.logits + n * V;
  float* out = a.logp + n * V;
  const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(in) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  if (filter_nucleus(a, in, out, vec, nbins, cand, red, &sh_n)) return;
  filter_general(a, in, out, vec, hist, red, redd, &sh_digit, &sh_above);
}

// ---------------------------------------------------------------------------------------
// Rows split over several workgroups (T > 0, V >= kSplitMinV, with a workspace): one workgroup
// per row leaves most of the chip idle for the rows of a few sequences and, with four passes over
// the row each bound by one CU, ran 272 nucleus rows of 151,936 logits in 286 us; with every pass
// split they are bound by the passes' traffic. A row is read in 16-byte groups at any alignment
// of its start (global vector loads need 4-byte alignment only); the groups past V are masked.
// ---------------------------------------------------------------------------------------
constexpr int64_t kSplitMinV = 16384;  // two segments; below, one workgroup covers the row at once
// The nucleus alone takes six launches when split, and from 32,768 ids (one mass part) they pay:
// 300 rows 76 -> 69 us, 16 rows 36 -> 34 us, where 300 rows of 20,000 ids took 62 us split against 53.
constexpr int64_t kSplitMinNucleus = 32768;

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// The TH * U groups of four logits that a workgroup of TH threads holds from element e0 of the
// row on: thread t has groups t, t + TH, ...; elements past V read as -inf.
template <int TH, int U>
__device__ __forceinline__ void load_groups(const float* in, int64_t V, int64_t e0, int tid,
                                            float (&x)[U][4]) {
  if (e0 + 4 * TH * U <= V) {
    f32x4u g[U];
#pragma unroll
    for (int i = 0; i < U; ++i)
      g[i] = *reinterpret_cast<const f32x4u*>(in + e0 + 4 * (tid + i * TH));
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) x[i][q] = g[i][q];
  } else {
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t v = e0 + 4 * (tid + i * TH) + q;
        x[i][q] = v < V ? in[v] : -INFINITY;
      }
  }
}

template <int TH, int U>
__device__ __forceinline__ void store_groups(float* out, int64_t V, int64_t e0, int tid,
                                             const float (&x)[U][4]) {
  if (e0 + 4 * TH * U <= V) {
#pragma unroll
    for (int i = 0; i < U; ++i)
      *reinterpret_cast<f32x4u*>(out + e0 + 4 * (tid + i * TH)) =
          f32x4u{x[i][0], x[i][1], x[i][2], x[i][3]};
  } else {
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t v = e0 + 4 * (tid + i * TH) + q;
        if (v < V) out[v] = x[i][q];
      }
  }
}

// A segment: the 8192 elements that 256 threads hold in registers.
constexpr int kSegT = 256;
constexpr int kSegU = 8;
constexpr int kSegElems = 4 * kSegT * kSegU;
static_assert((int64_t{1} << 24) / kSegElems * 16 <= kFilterRowBytes, "segment results of a row");

__host__ __device__ constexpr int64_t n_segs(int64_t V) { return (V + kSegElems - 1) / kSegElems; }

// Largest key of a 256-thread group (threads 256 g .. 256 g + 255); `red` holds 4 words per group.
// Every thread of the workgroup calls it.
__device__ __forceinline__ uint32_t group_max_u32(uint32_t v, uint32_t* red, int grp) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, static_cast<uint32_t>(__shfl_xor(v, o)));
  if (lane_id() == 0) red[4 * grp + ((threadIdx.x >> 6) & 3)] = v;
  __syncthreads();
  const uint32_t m = max(max(red[4 * grp], red[4 * grp + 1]), max(red[4 * grp + 2], red[4 * grp + 3]));
  __syncthreads();
  return m;
}

// Maximum m of s and sum of exp(s - m) of one segment, by a group of 256 threads (group grp of
// the workgroup; every thread calls it): the same order of operations whichever kernel runs it.
struct SegStat {
  float m;
  float pad;
  double sum;
};

__device__ __forceinline__ SegStat seg_stat(const float* in, int64_t V, int64_t seg, bool live,
                                            float T, int grp, uint32_t* red, double* redd) {
  const int t = threadIdx.x & (kSegT - 1);
  float x[kSegU][4];
  // a group without a segment takes part with an empty one
  load_groups<kSegT, kSegU>(in, live ? V : 0, live ? seg * kSegElems : 0, t, x);
  uint32_t mk = 0;
#pragma unroll
  for (int i = 0; i < kSegU; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) mk = max(mk, order_key(x[i][q]));
  const float m = __fdiv_rn(key_value(group_max_u32(mk, red, grp)), T);
  // A segment of -inf alone has the sum 0; a NaN anywhere makes it NaN.
  const double md = m == -INFINITY ? 0.0 : static_cast<double>(m);
  const int64_t left = live ? V - seg * kSegElems : 0;  // groups of four past V add nothing
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < kSegU; ++i)
    if (4 * kSegT * i < left)
#pragma unroll
      for (int q = 0; q < 4; ++q) s += exp(static_cast<double>(__fdiv_rn(x[i][q], T)) - md);
  s = wave_sum_f64(s);
  if (lane_id() == 0) redd[4 * grp + ((threadIdx.x >> 6) & 3)] = s;
  __syncthreads();
  const double sum = (redd[4 * grp] + redd[4 * grp + 1]) + (redd[4 * grp + 2] + redd[4 * grp + 3]);
  __syncthreads();
  return SegStat{m, 0.0f, sum};
}

// The row's maximum and log-normaliser from its segments' statistics; every wavefront computes
// the same.
__device__ __forceinline__ void merge_stats(const SegStat* st, int n, float* m, double* lse) {
  const int lane = lane_id();
  float mx = -INFINITY;
  bool nan = false;
  for (int i = lane; i < n; i += 64) {
    nan = nan || st[i].m != st[i].m;
    mx = fmaxf(mx, st[i].m);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if (__ballot(nan)) mx = NAN;  // a NaN logit is the row's maximum in key order
  double s = 0.0;
  for (int i = lane; i < n; i += 64)
    s += st[i].sum * exp(static_cast<double>(st[i].m) - static_cast<double>(mx));
  *m = mx;
  *lse = log(wave_sum_f64(s));
}

__device__ __forceinline__ float log_prob(float sv, float m, double lse) {
  return static_cast<float>(static_cast<double>(sv) - static_cast<double>(m) - lse);
}

// Temperature alone, split: statistics per segment, then the output. Two reads and one write of
// the row, bound by that traffic and the binary64 exponentials: 272 rows of 151,936 logits 110 us, 16
// rows 16 us, where one workgroup per row with three reads took 251 and 115 (a polynomial good to 2^-32
// in place of the exponential: 97 and 14 us).
__global__ __launch_bounds__(kSegT) void filter_stats_kernel(FilterArgs a, int segs) {
  __shared__ uint32_t red[4];
  __shared__ double redd[4];
  const int64_t row = blockIdx.x / segs, seg = blockIdx.x % segs;
  const SegStat st = seg_stat(a.logits + row * a.V, a.V, seg, true, a.temperature, 0, red, redd);
  if (threadIdx.x == 0)
    reinterpret_cast<SegStat*>(a.row_ws + row * kFilterRowBytes)[seg] = st;
}

__global__ __launch_bounds__(kSegT) void filter_scale_kernel(FilterArgs a, int segs) {
  const int64_t row = blockIdx.x / segs, seg = blockIdx.x % segs;
  float x[kSegU][4];
  load_groups<kSegT, kSegU>(a.logits + row * a.V, a.V, seg * kSegElems, threadIdx.x, x);
  float m;
  double lse;
  merge_stats(reinterpret_cast<const SegStat*>(a.row_ws + row * kFilterRowBytes), segs, &m, &lse);
#pragma unroll
  for (int i = 0; i < kSegU; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) x[i][q] = log_prob(__fdiv_rn(x[i][q], a.temperature), m, lse);
  store_groups<kSegT, kSegU>(a.logp + row * a.V, a.V, seg * kSegElems, threadIdx.x, x);
}

// Temperature alone, rows of up to two segments: one 256-thread workgroup per row with the same
// arithmetic, five to a CU (1000 rows of 3000 ids: 14 us, against 34 with the 1024-thread form
// below, of which a CU holds one; at 16,384 ids 300 rows take 22 us, split, at one id more, 21).
constexpr int kRowSegs = 2;
__global__ __launch_bounds__(kSegT) void filter_scale_rows_kernel(FilterArgs a, int segs) {
  __shared__ uint32_t red[4];
  __shared__ double redd[4];
  __shared__ SegStat st[kRowSegs];
  const float* in = a.logits + blockIdx.x * a.V;
  float* out = a.logp + blockIdx.x * a.V;
  for (int seg = 0; seg < segs; ++seg) {
    const SegStat s = seg_stat(in, a.V, seg, true, a.temperature, 0, red, redd);
    if (threadIdx.x == 0) st[seg] = s;
  }
  __syncthreads();
  float m;
  double lse;
  merge_stats(st, segs, &m, &lse);
  for (int64_t e0 = 0; e0 < a.V; e0 += 8 * kSegT) {
    float x[2][4];
    load_groups<kSegT, 2>(in, a.V, e0, threadIdx.x, x);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) x[i][q] = log_prob(__fdiv_rn(x[i][q], a.temperature), m, lse);
    store_groups<kSegT, 2>(out, a.V, e0, threadIdx.x, x);
  }
}

// Temperature alone, one workgroup per row: its four groups take the segments in turn, with the
// split form's arithmetic, so both give the same bits. `st` holds n_segs(V) statistics.
__device__ void filter_scale_row(const FilterArgs& a, const float* in, float* out, SegStat* st,
                                 uint32_t* red, double* redd) {
  const int grp = threadIdx.x / kSegT;
  const int n = static_cast<int>(n_segs(a.V));
  for (int s0 = 0; s0 < n; s0 += kFT / kSegT) {
    const int seg = s0 + grp;
    const SegStat s = seg_stat(in, a.V, seg, seg < n, a.temperature, grp, red, redd);
    if (seg < n && threadIdx.x % kSegT == 0) st[seg] = s;
  }
  __syncthreads();
  float m;
  double lse;
  merge_stats(st, n, &m, &lse);
  for (int64_t e0 = 0; e0 < a.V; e0 += 16 * kFT) {
    float x[4][4];
    load_groups<kFT, 4>(in, a.V, e0, threadIdx.x, x);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) x[i][q] = log_prob(__fdiv_rn(x[i][q], a.temperature), m, lse);
    store_groups<kFT, 4>(out, a.V, e0, threadIdx.x, x);
  }
}

// Least key k with ok(k), for a predicate that holds from some key on (and at +inf): 64 probes
// per step, one per lane; every wavefront computes it.
template <class F>
__device__ __forceinline__ uint32_t least_key(F ok) {
  if (ok(kKeyNegInf)) return kKeyNegInf;
  uint32_t lo = kKeyNegInf, hi = kKeyPosInf;  // ok(lo) false, ok(hi) true
  while (hi - lo > 1) {
    const uint32_t step = (hi - lo + 63) / 64;
    const uint64_t at = static_cast<uint64_t>(lo) + static_cast<uint64_t>(lane_id() + 1) * step;
    const uint32_t probe = at < hi ? static_cast<uint32_t>(at) : hi;
    const uint64_t hit = __ballot(probe == hi || ok(probe));
    const int f = __ffsll(static_cast<unsigned long long>(hit)) - 1;  // the last lane's probe is hi
    const uint32_t nhi = static_cast<uint32_t>(__shfl(static_cast<int>(probe), f));
    if (f > 0) lo = static_cast<uint32_t>(__shfl(static_cast<int>(probe), f - 1));
    hi = nhi;
  }
  return hi;
}

// Top-k, split (0 < k <= 256): every segment workgroup streams its share of the row once, writing
// -inf and keeping each thread's largest logit key, and takes the k-th largest of its 512 thread
// maxima as a lower bound of its share's k-th largest: about k (1 + k / 1024) tokens of the share
// reach it, where bounds from parts of the share let through several times as many. The threads
// that hold such tokens read their groups again (from L2) and append them to the share's list in
// the workspace, headed by the bound, the count and the share's j-th largest thread maximum,
// j = ceil(k / shares). A merge workgroup per row keeps the tokens that reach the largest of the
// shares' bounds and the least of their j-th largest (j tokens of every share reach that one, so
// the row's k-th largest does): two or three times k of them, selects among them and finishes.
// 16 rows of 151,936 at k = 50: 10.7 + 7.5 us, against 23 + 54 us with 4 shares per row, bounds per
// wavefront and a merge that bisected 1,600 candidates; 272 rows at k = 20 82 us (112).
// 16 shares per row up to k = 128, 8 above: k tokens per share and the overshoot stay within a
// share's list, and the smallest row (kSplitMinV) still has more non-empty threads than k. Where the
// logits fall with the id a thread holds several of the largest and its neighbours the next, so up to 4 k
// tokens reach the bound, or, in a flat tail, as many as share its 18 bits: a list that overflows is left
// out if its share's largest key is below the row's bound, and otherwise its share is read again by the
// merge workgroup, against the row's bound (16 rows, k = 128, falling by 1.1 log(id) with noise 0.7: 27 us,
// where the general path took 467; without noise 30 us). Rows with fewer than k ids above -inf, or with
// more than kCandCap tokens at the row's bound, take the general path.
constexpr int kTopThreads = 512;
constexpr int kTopEntries = kFilterRowBytes / 8;  // over all shares of a row, two heads each included
__host__ __device__ constexpr int top_shares(int64_t k) { return k <= 128 ? 16 : 8; }
static_assert(kSplitMinV / 4 / top_shares(128) >= 128 && kSplitMinV / 4 / top_shares(256) >= 256,
              "at least k non-empty threads per share");

struct ShareGroups {  // groups of four ids g0 <= g < g1, those below gfull within V
  int64_t g0, g1, gfull;
};
__device__ __forceinline__ ShareGroups share_groups(int64_t V, int shares, int share) {
  const int64_t groups = (V + 3) / 4;
  const int64_t per = (groups + shares - 1) / shares;
  const int64_t g0 = min(groups, share * per), g1 = min(groups, g0 + per);
  return {g0, g1, min(g1, V / 4)};
}

__global__ __launch_bounds__(kTopThreads) void filter_topk_share_kernel(FilterArgs a, int shares) {
  __shared__ int s_bin[3][kTopThreads];
  __shared__ int s_wave[2][kTopThreads / 64];
  __shared__ int s_pick[2][2];
  static_assert(kTopThreads == 512, "one histogram bin per thread");
  __shared__ int sh_n;
  const int64_t row = blockIdx.x / shares;
  const int share = static_cast<int>(blockIdx.x % shares);
  const int tid = threadIdx.x;
  const int64_t V = a.V;
  const float T = a.temperature;
  const int k = static_cast<int>(a.top_k);
  const int cap = kTopEntries / shares - 2;
  const float* in = a.logits + row * V;
  float* out = a.logp + row * V;
  // This share's groups of four; thread t has g0 + t, g0 + t + 512, ...
  const auto [g0, g1, gfull] = share_groups(V, shares, share);
  uint32_t top = 0;
  auto see = [&](float x) { top = max(top, order_key(x)); };
  const f32x4u ninf = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  int64_t j = g0 + tid;
  for (; j + (kBatch - 1) * kTopThreads < gfull; j += kBatch * kTopThreads) {
    f32x4u x[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      x[u] = *reinterpret_cast<const f32x4u*>(in + 4 * (j + u * kTopThreads));
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      *reinterpret_cast<f32x4u*>(out + 4 * (j + u * kTopThreads)) = ninf;
#pragma unroll
      for (int q = 0; q < 4; ++q) see(x[u][q]);
    }
  }
#pragma unroll 4
  for (; j < gfull; j += kTopThreads) {
    const f32x4u x = *reinterpret_cast<const f32x4u*>(in + 4 * j);
    *reinterpret_cast<f32x4u*>(out + 4 * j) = ninf;
#pragma unroll
    for (int q = 0; q < 4; ++q) see(x[q]);
  }
  if (j < g1)  // the row's last, partial group
    for (int64_t v = 4 * j; v < V; ++v) {
      see(in[v]);
      out[v] = -INFINITY;
    }
  // Lower bounds of the share's k-th and j-th largest logit keys: those of its thread maxima, to 18
  // bits of the key, by two levels of 512-bin histograms (thread t counts from the top: bin 511 - t).
  const int need[2] = {k, (k + shares - 1) / shares};
  s_bin[0][tid] = 0;
  s_bin[1][tid] = 0;
  s_bin[2][tid] = 0;
  if (tid == 0) sh_n = 0;
  __syncthreads();
  atomicAdd(&s_bin[2][top >> 23], 1);
  __syncthreads();
  auto pick = [&](const int* bins, int n, int q) {  // the bin the n-th from the top is in
    const int c = bins[kTopThreads - 1 - tid];
    int upto = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(upto, o);
      if (lane_id() >= o) upto += t;
    }
    if (lane_id() == 63) s_wave[q][tid >> 6] = upto;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kTopThreads / 64; ++w) upto += w < (tid >> 6) ? s_wave[q][w] : 0;
    if (upto >= n && upto - c < n) {
      s_pick[q][0] = kTopThreads - 1 - tid;
      s_pick[q][1] = n - (upto - c);  // its place in the bin
    }
  };
  pick(s_bin[2], need[0], 0);
  pick(s_bin[2], need[1], 1);
  __syncthreads();
  const uint32_t b0 = s_pick[0][0], b1 = s_pick[1][0];
  const int n0 = s_pick[0][1], n1 = s_pick[1][1];
  if ((top >> 23) == b0) atomicAdd(&s_bin[0][(top >> 14) & 511], 1);
  if ((top >> 23) == b1) atomicAdd(&s_bin[1][(top >> 14) & 511], 1);
  __syncthreads();
  pick(s_bin[0], n0, 0);
  pick(s_bin[1], n1, 1);
  __syncthreads();
  const uint32_t lo = (b0 << 23) | (static_cast<uint32_t>(s_pick[0][0]) << 14);
  const uint32_t jth = (b1 << 23) | (static_cast<uint32_t>(s_pick[1][0]) << 14);
  // A share with fewer than k threads holding a logit above -inf (a masked part of the vocabulary)
  // lists all of those and gives no bound.
  const bool bound = lo > kKeyNegInf;
  const uint32_t s_low = bound ? order_key(__fdiv_rn(key_value(lo), T)) : 0;
  uint32_t x_low = kKeyNegInf + 1;
  if (bound) {  // the least logit key with that s: almost always within 64 of the bound's
    auto reaches = [&](uint32_t q) { return order_key(__fdiv_rn(key_value(q), T)) >= s_low; };
    const uint64_t hit = lo > kKeyNegInf + 64 ? __ballot(reaches(lo - 63 + lane_id())) : 1;
    x_low = (hit & 1) ? least_key(reaches)
                      : lo - 64 + static_cast<uint32_t>(__ffsll(static_cast<unsigned long long>(hit)));
  }
  uint64_t* list = reinterpret_cast<uint64_t*>(a.row_ws + row * kFilterRowBytes) +
                   static_cast<int64_t>(share) * (cap + 2);
  auto take = [&](int64_t v, float x) {
    if (order_key(x) >= x_low) {
      const int slot = atomicAdd(&sh_n, 1);
      if (slot < cap) list[2 + slot] = visit_key(order_key(__fdiv_rn(x, T)), v);
    }
  };
  if (top >= x_low) {
    int64_t i = g0 + tid;
#pragma unroll 4
    for (; i < gfull; i += kTopThreads) {
      const f32x4u x = *reinterpret_cast<const f32x4u*>(in + 4 * i);
#pragma unroll
      for (int q = 0; q < 4; ++q) take(4 * i + q, x[q]);
    }
    if (i < g1)
      for (int64_t v = 4 * i; v < V; ++v) take(v, in[v]);
  }
  __syncthreads();
  // The share's largest key, by which the merge tells whether it needs a list that overflowed.
  uint32_t most = 0;
  if (__builtin_expect(sh_n > cap, 0)) {  // workgroup-uniform
    most = top;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = max(most, static_cast<uint32_t>(__shfl_xor(most, o)));
    if (lane_id() == 0) s_wave[0][tid >> 6] = static_cast<int>(most);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kTopThreads / 64; ++w)
      most = max(most, static_cast<uint32_t>(s_wave[0][w]));
    most = order_key(__fdiv_rn(key_value(most), T));
  }
  if (tid == 0) {
    list[0] = (static_cast<uint64_t>(s_low) << 32) | static_cast<uint32_t>(sh_n);
    list[1] = (static_cast<uint64_t>(most) << 32) |
              (jth > kKeyNegInf ? order_key(__fdiv_rn(key_value(jth), T)) : 0);
  }
}

// Eight waves per SIMD, so that two rows share a CU: the fallback's registers spill, the usual path's
// do not.
__global__ __launch_bounds__(kFT, 8) void filter_topk_merge_kernel(FilterArgs a, int shares) {
  __shared__ uint64_t hist[256];
  __shared__ uint64_t cand[kCandCap];
  __shared__ int sh_n;
  __shared__ uint64_t red[kFW];
  __shared__ double redd[kFW];
  __shared__ uint32_t sh_digit;
  __shared__ uint64_t sh_above;
  static_assert(kCandCap >= kTopEntries, "every list entry of a row fits");
  const int64_t row = blockIdx.x;
  const int64_t V = a.V;
  const int tid = threadIdx.x;
  const float* in = a.logits + row * V;
  float* out = a.logp + row * V;
  const uint64_t* lists = reinterpret_cast<const uint64_t*>(a.row_ws + row * kFilterRowBytes);
  const int per = kTopEntries / shares;
  // entries tid, tid + kFT, ... of the lists, loaded with the heads (unwritten ones are not used)
  uint64_t e[kTopEntries / kFT];
#pragma unroll
  for (int i = 0; i < kTopEntries / kFT; ++i) e[i] = lists[tid + i * kFT];
  const uint64_t head = lists[(lane_id() % shares) * per];
  const uint64_t ends = lists[(lane_id() % shares) * per + 1];
  uint32_t kth = 0, jth = 0xFFFFFFFFu;  // over the 16 lanes that hold every share's heads, by scalar reads
#pragma unroll
  for (int l = 0; l < 16; ++l) {
    kth = max(kth, static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(head >> 32), l)));
    jth = min(jth, static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(ends), l)));
  }
  const uint32_t least = max(kth, jth);
  // Shares whose list overflowed (logits that fall with the id, or coarse ones) and that hold a token
  // that counts: their ids are read again, against the row's bound. The usual path, without any, comes
  // first and shares no address with this one (its spills cost 0.5 us there).
  const uint64_t over = __ballot(lane_id() < shares &&
                                 static_cast<int>(static_cast<uint32_t>(head)) > per - 2 &&
                                 static_cast<uint32_t>(ends >> 32) >= least);
  if (tid == 0) sh_n = 0;
  __syncthreads();
  if (__builtin_expect(over == 0, 1)) {
#pragma unroll
    for (int i = 0; i < kTopEntries / kFT; ++i) {
      const int at = tid + i * kFT, share = at / per, slot = at % per;
      const int cnt = static_cast<int>(static_cast<uint32_t>(__shfl(head, share)));
      if (slot > 1 && slot < 2 + cnt && static_cast<uint32_t>(e[i] >> 32) >= least)
        cand[atomicAdd(&sh_n, 1)] = e[i];
    }
  } else if (least) {
    const float T = a.temperature;
    const uint32_t x_low =
        least_key([&](uint32_t q) { return order_key(__fdiv_rn(key_value(q), T)) >= least; });
    auto keep = [&](uint64_t c) {
      const int slot = atomicAdd(&sh_n, 1);
      if (slot < kCandCap) cand[slot] = c;
    };
    auto take = [&](int64_t v, float x) {
      if (order_key(x) >= x_low) keep(visit_key(order_key(__fdiv_rn(x, T)), v));
    };
    for (int share = 0; share < shares; ++share) {
      if (over >> share & 1) {
        const auto [g0, g1, gfull] = share_groups(V, shares, share);
        int64_t i = g0 + tid;
#pragma unroll 4
        for (; i < gfull; i += kFT) {
          const f32x4u x = *reinterpret_cast<const f32x4u*>(in + 4 * i);
#pragma unroll
          for (int q = 0; q < 4; ++q) take(4 * i + q, x[q]);
        }
        if (i < g1)
          for (int64_t v = 4 * i; v < V; ++v) take(v, in[v]);
      } else {
        const uint64_t* list = lists + share * per;
        const int cnt = min(static_cast<int>(static_cast<uint32_t>(list[0])), per - 2);
        for (int i = tid; i < cnt; i += kFT)
          if (static_cast<uint32_t>(list[2 + i] >> 32) >= least) keep(list[2 + i]);
      }
    }
  }
  __syncthreads();
  const int n = sh_n;
  // Without a bound (too few threads of every share hold a logit above -inf) the lists hold all of
  // those logits, if none overflowed.
  if (__builtin_expect(n > kCandCap || n < a.top_k || (over && !least), 0)) {
    const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(in) & 15) == 0 &&
                     (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    filter_general(a, in, out, vec, hist, red, redd, &sh_digit, &sh_above);
    return;
  }
  block_sort_desc(cand, n);
  // the tokens at or above the k-th largest s: at most 64 of them finish in wavefront 0
  const uint32_t tk = static_cast<uint32_t>(cand[a.top_k - 1] >> 32);
  if (n <= 64 || static_cast<uint32_t>(cand[64] >> 32) < tk) {
    if (tid < 64) {
      const uint64_t c = tid < n ? cand[tid] : 0;
      const bool in = tid < n && static_cast<uint32_t>(c >> 32) >= tk;
      finish_small(a, out, in ? c : 0, __popcll(__ballot(in)));
    }
    return;
  }
  finish_sorted(a, out, cand, n, red, redd);
}

// Nucleus alone, split: the same integer decisions as filter_nucleus in six launches.
//   1. max      largest logit key per segment (and the row's bins cleared);
//   2. mass     integer mass per bin: 32,768 ids per workgroup in LDS bins, whose non-empty ones
//               are added to the row's bins (integer sums: any order gives the same);
//   3. edge     one workgroup per row: the crossing bin, and its ends as logits (bins are
//               non-increasing in the logit, so a bin is an interval of logits);
//   4. gather   the crossing bin's tokens appended to the row's list: the row is read again with two
//               compares per id;
//   5. cut      one workgroup per row: the list's order, the cut and the normaliser, or, where the
//               bin's tokens cannot be listed, the general path from the maximum on;
//   6. write    kept ids by comparing logit keys, so only kept ids are divided.
// The mass pass is bound by its arithmetic (about 50 lane instructions per id for the contract's
// division and quantised exponential), the others by the row's traffic. 272 rows of 151,936
// logits at T = 0.7: 27 + 54 + 8 + 25 + 10 + 53 us (169 us per call, 276 with one workgroup per
// row); 16 rows 40 us (123).
struct NucleusRow {  // a row's workspace: this, then the bins and seg_max[segs], later the list
  uint64_t before, tp;
  double lse;
  float m;
  float edge[2];  // the crossing bin's logits: [edge[0], edge[1])
  int bin;        // the crossing bin; up to kNucSureBin every token of it has positive mass
  int count;      // tokens listed
  int listed;     // the row has mass, and its crossing bin may fit the list
};
constexpr int64_t kNucMaxSegs = (int64_t{1} << 24) / kSegElems;
static_assert(sizeof(NucleusRow) % 8 == 0 &&
                  sizeof(NucleusRow) + 8 * kNucBins + 4 * kNucMaxSegs <= kFilterRowBytes,
              "a row's workspace");
// Entries of the list, which takes the place of the bins and maxima once the edge is known: 4,090,
// where the one-workgroup form's holds kCandCap.
constexpr int kNucList = static_cast<int>((kFilterRowBytes - sizeof(NucleusRow)) / 8);
static_assert(kNucList <= kCandCap && kNucList >= kCandCap - 8, "the list's entries");
constexpr int kMassU = 8;
constexpr int kMassElems = 4 * kFT * kMassU;

__device__ __forceinline__ NucleusRow* nucleus_row(const FilterArgs& a, int64_t row) {
  return reinterpret_cast<NucleusRow*>(a.row_ws + row * kFilterRowBytes);
}
__device__ __forceinline__ uint64_t* nucleus_bins(NucleusRow* w) {
  return reinterpret_cast<uint64_t*>(w + 1);
}
__device__ __forceinline__ uint32_t* nucleus_seg_max(NucleusRow* w) {
  return reinterpret_cast<uint32_t*>(nucleus_bins(w) + kNucBins);
}
__device__ __forceinline__ uint64_t* nucleus_list(NucleusRow* w) {
  return reinterpret_cast<uint64_t*>(w + 1);
}

// s of the row's largest logit, from the segments' keys; every wavefront computes it.
__device__ __forceinline__ float nucleus_max(NucleusRow* w, int segs, float T) {
  uint32_t k = 0;
  for (int i = lane_id(); i < segs; i += 64) k = max(k, nucleus_seg_max(w)[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) k = max(k, static_cast<uint32_t>(__shfl_xor(k, o)));
  return __fdiv_rn(key_value(k), T);
}

__global__ __launch_bounds__(kSegT) void nucleus_max_kernel(FilterArgs a, int segs) {
  __shared__ uint32_t red[4];
  const int64_t row = blockIdx.x / segs, seg = blockIdx.x % segs;
  NucleusRow* w = nucleus_row(a, row);
  float x[kSegU][4];
  load_groups<kSegT, kSegU>(a.logits + row * a.V, a.V, seg * kSegElems, threadIdx.x, x);
  if (seg == 0)
    for (int i = threadIdx.x; i < kNucBins; i += kSegT) nucleus_bins(w)[i] = 0;
  uint32_t k = 0;
#pragma unroll
  for (int i = 0; i < kSegU; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) k = max(k, order_key(x[i][q]));
  k = group_max_u32(k, red, 0);
  if (threadIdx.x == 0) nucleus_seg_max(w)[seg] = k;
}

__global__ __launch_bounds__(kFT) void nucleus_mass_kernel(FilterArgs a, int parts, int segs) {
  __shared__ uint64_t bins[kNucBins];
  const int64_t row = blockIdx.x / parts, part = blockIdx.x % parts;
  NucleusRow* w = nucleus_row(a, row);
  const float T = a.temperature;
  float x[kMassU][4];
  load_groups<kFT, kMassU>(a.logits + row * a.V, a.V, part * kMassElems, threadIdx.x, x);
  const float m = nucleus_max(w, segs, T);
  for (int i = threadIdx.x; i < kNucBins; i += kFT) bins[i] = 0;
  __syncthreads();
  auto add = [&](float sv) {
    const float d = __fsub_rn(sv, m);
    const uint64_t P = quant_detexp32(d);
    const int b = min(kNucBins - 1, static_cast<int>(__fmul_rn(-d, kNucScale)));
    if (P) atomicAdd(reinterpret_cast<unsigned long long*>(&bins[b]),
                     static_cast<unsigned long long>(P));
  };
  auto all = [&](auto scale) {
#pragma unroll
    for (int i = 0; i < kMassU; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) add(scale(x[i][q]));
  };
  // Quotient's short form needs |x| >= 2^-100 (or 0, or an infinity, whose NaN has mass 0 as
  // -inf must); a smaller logit's s is below 2^-79, where its last bit cannot change s - m once
  // |m| >= 2^-50.
  const Quotient div(T);
  if (T == 1.0f)
    all([](float v) { return v; });
  else if (div.short_form && fabsf(m) >= 0x1p-50f)
    all([&](float v) { return div.quick(v); });
  else
    all([&](float v) { return __fdiv_rn(v, T); });
  __syncthreads();
  for (int i = threadIdx.x; i < kNucBins; i += kFT)
    if (bins[i]) atomicAdd(reinterpret_cast<unsigned long long*>(&nucleus_bins(w)[i]),
                           static_cast<unsigned long long>(bins[i]));
}

__global__ __launch_bounds__(kFT) void nucleus_edge_kernel(FilterArgs a, int segs) {
  __shared__ uint64_t red[kFW];
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x;
  const float T = a.temperature;
  NucleusRow* w = nucleus_row(a, row);
  const uint64_t m0 = nucleus_bins(w)[2 * tid], m1 = nucleus_bins(w)[2 * tid + 1];
  const float m = nucleus_max(w, segs, T);
  int bstar;
  uint64_t before, tp;
  const bool live = nucleus_crossing(m0, m1, a.top_p, red, &bstar, &before, &tp);
  if (tid < 128) {  // the ends of the crossing bin, one per wavefront
    const int below = bstar - (tid >> 6);
    const uint32_t k = least_key([&](uint32_t q) {
      const float d = __fsub_rn(__fdiv_rn(key_value(q), T), m);
      return min(kNucBins - 1, static_cast<int>(__fmul_rn(-d, kNucScale))) <= below;
    });
    if (lane_id() == 0) w->edge[tid >> 6] = key_value(k);
  }
  if (tid == 0) {
    w->before = before;
    w->tp = tp;
    w->m = m;
    w->bin = bstar;
    w->count = 0;
    // No token of bin b has more mass than 2^40 e^(-b / kNucScale): a crossing bin that must hold more
    // tokens than the one-workgroup form lists is not gathered either.
    const double most = 0x1p40 * exp(-static_cast<double>(bstar) / static_cast<double>(kNucScale));
    w->listed = live && static_cast<double>(nucleus_bins(w)[live ? bstar : 0]) <=
                            1.001 * (kCandCap + 1) * most;
  }
}

__global__ __launch_bounds__(kSegT) void nucleus_gather_kernel(FilterArgs a, int segs) {
  const int64_t row = blockIdx.x / segs, seg = blockIdx.x % segs;
  const float* in = a.logits + row * a.V;
  NucleusRow* w = nucleus_row(a, row);
  float x[kSegU][4];
  load_groups<kSegT, kSegU>(in, a.V, seg * kSegElems, threadIdx.x, x);
  if (!w->listed) return;
  __shared__ int s_n, s_base;
  const float lo = w->edge[0], hi = w->edge[1], m = w->m;
  const bool sure = w->bin <= kNucSureBin;
  uint32_t hit = 0;
#pragma unroll
  for (int i = 0; i < kSegU; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) hit |= x[i][q] >= lo && x[i][q] < hi ? 1u << (4 * i + q) : 0;
  // Few, as a rule: read again rather than picked out of the registers.
  auto id_of = [&](int at) {
    return seg * kSegElems + 4 * (static_cast<int>(threadIdx.x) + (at >> 2) * kSegT) + (at & 3);
  };
  auto s_of = [&](int64_t v) { return __fdiv_rn(in[v], a.temperature); };
  for (uint32_t left = hit; left; left &= left - 1) {
    const int at = __ffs(static_cast<int>(left)) - 1;
    const int64_t v = id_of(at);  // past V: a masked place of the last segment
    if (v >= a.V || !(sure || quant_detexp32(__fsub_rn(s_of(v), m)))) hit &= ~(1u << at);
  }
  // One addition to the row's counter per workgroup: with one per token, rows whose bin holds
  // thousands wait for each other's.
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  int slot = hit ? atomicAdd(&s_n, __popc(hit)) : 0;
  __syncthreads();
  if (s_n == 0) return;  // workgroup-uniform
  if (threadIdx.x == 0) s_base = atomicAdd(&w->count, s_n);
  __syncthreads();
  slot += s_base;
  uint64_t* list = nucleus_list(w);
  for (; hit; hit &= hit - 1, ++slot) {
    const int64_t v = id_of(__ffs(static_cast<int>(hit)) - 1);
    if (slot < kNucList) list[slot] = visit_key(order_key(s_of(v)), v);
  }
}

// Eight waves per SIMD, so that two rows share a CU (272 rows: 13.1 -> 10.3 us); only the fallback spills.
__global__ __launch_bounds__(kFT, 8) void nucleus_cut_kernel(FilterArgs a) {
  __shared__ uint64_t hist[256];
  __shared__ uint64_t nbins[kNucBins];
  __shared__ uint64_t cand[kCandCap];
  __shared__ int sh_n;
  __shared__ uint64_t red[kFW];
  __shared__ double redd[kFW];
  __shared__ uint32_t sh_digit;
  __shared__ uint64_t sh_above;
  __shared__ uint32_t s_key[2];
  const int64_t row = blockIdx.x;
  const int64_t V = a.V;
  const float T = a.temperature;
  const int tid = threadIdx.x;
  NucleusRow* w = nucleus_row(a, row);
  const uint64_t* list = nucleus_list(w);
  const int n = w->count;
  const float m = w->m;
  if (!w->listed || n > kNucList) {  // a row without mass, or a bin that does not fit
    const float* in = a.logits + row * V;
    float* out = a.logp + row * V;
    const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(in) & 15) == 0 &&
                     (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    if (!w->listed || n > kCandCap || !filter_nucleus(a, in, out, vec, nbins, cand, red, &sh_n))
      filter_general<true>(a, in, out, vec, hist, red, redd, &sh_digit, &sh_above, m);
    if (tid == 0) a.cuts[row] = FilterCut{0, 0, 0, 1};
    return;
  }
  for (int i = tid; i < n; i += kFT) cand[i] = list[i];
  __syncthreads();
  uint64_t cut;
  const double lse = nucleus_kept(cand, n, m, w->before, w->tp, red, &cut);
  const uint32_t ck = static_cast<uint32_t>(cut >> 32);
  // logit keys whose s reaches the last kept token's, and whose s is above it
  if (tid < 128) {
    const uint32_t least = ck + (tid >> 6);
    const uint32_t k = least_key([&](uint32_t q) { return order_key(__fdiv_rn(key_value(q), T)) >= least; });
    if (lane_id() == 0) s_key[tid >> 6] = k;
  }
  __syncthreads();
  if (tid == 0) {
    w->lse = lse;
    a.cuts[row] = FilterCut{s_key[1], s_key[0], 0xFFFFFFFFu - static_cast<uint32_t>(cut), 0};
  }
}

__global__ __launch_bounds__(kSegT) void nucleus_write_kernel(FilterArgs a, int segs) {
  const int64_t row = blockIdx.x / segs, seg = blockIdx.x % segs;
  const NucleusRow* w = nucleus_row(a, row);
  float x[kSegU][4];
  load_groups<kSegT, kSegU>(a.logits + row * a.V, a.V, seg * kSegElems, threadIdx.x, x);
  const FilterCut c = a.cuts[row];
  if (c.done) return;
  const float m = w->m;
  const double lse = w->lse;
  // A NaN with the sign bit set, the least key, stays NaN where filter_nucleus, which takes it for a
  // token of bin 0, keeps it.
  const bool keep_nan = w->bin > 0 && w->bin <= kNucSureBin;
#pragma unroll
  for (int i = 0; i < kSegU; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t k = order_key(x[i][q]);
      const uint32_t v = static_cast<uint32_t>(seg * kSegElems + 4 * (threadIdx.x + i * kSegT) + q);
      const bool kept = k >= c.key_above || (k >= c.key_at && v <= c.last_id) ||
                        (keep_nan && x[i][q] != x[i][q]);
      float o = -INFINITY;
      if (kept) o = log_prob(__fdiv_rn(x[i][q], a.temperature), m, lse);
      x[i][q] = o;
    }
  store_groups<kSegT, kSegU>(a.logp + row * a.V, a.V, seg * kSegElems, threadIdx.x, x);
}

// One workgroup per row: every filter, for short rows and for calls without a workspace.
__global__ __launch_bounds__(kFT) void filter_kernel(FilterArgs a) {
  __shared__ uint64_t hist[256];
  __shared__ uint64_t cand[kCandCap];
  __shared__ int resc[kFT];
  __shared__ int sh_n, sh_r;
  __shared__ uint64_t red[kFW];
  __shared__ uint32_t redk[kFW];
  __shared__ double redd[kFW];
  __shared__ uint32_t sh_digit;
  __shared__ uint64_t sh_above;
  const int64_t n = blockIdx.x;
  const int64_t V = a.V;
  const float* in = a.logits + n * V;
  float* out = a.logp + n * V;
  const int tid = threadIdx.x;

  if (a.temperature == 0.0f) {  // lowest-index maximum
    uint64_t best = 0;
    for (int64_t v = tid; v < V; v += kFT) {
      const uint64_t k = (static_cast<uint64_t>(order_key(in[v])) << 32) |
                         (0xFFFFFFFFu - static_cast<uint32_t>(v));
      best = k > best ? k : best;
    }
    best = block_max_u64(best, red);
    const int64_t arg = 0xFFFFFFFFu - static_cast<uint32_t>(best);
    for (int64_t v = tid; v < V; v += kFT) out[v] = v == arg ? 0.0f : -INFINITY;
    return;
  }
  const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(in) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  if (a.top_k > 0 && a.top_k <= kFastK && a.top_k < V &&
      filter_fast(a, in, out, vec, cand, resc, red, redd, &sh_n, &sh_r))
    return;

  if ((a.top_k == 0 || a.top_k >= V) && a.top_p == 1.0f) {
    static_assert(sizeof(cand) >= (int64_t{1} << 24) / kSegElems * sizeof(SegStat),
                  "statistics of every segment");
    filter_scale_row(a, in, out, reinterpret_cast<SegStat*>(cand), redk, redd);
    return;
  }
  filter_general(a, in, out, vec, hist, red, redd, &sh_digit, &sh_above);
}

// Per sampled block: (1/b) sum_j prod_{i<=j} p(x_i); one thread per block.
__global__ __launch_bounds__(256) void determinism_terms_kernel(DeterminismArgs a) {
  const int64_t mblk = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (mblk >= a.M) return;
  double prod = 1.0, sum = 0.0;
  for (int64_t i = 0; i < a.b; ++i) {
    const int32_t x = a.x[mblk * a.b + i];
    const double lp = x >= 0 && x < a.V
                          ? static_cast<double>(a.logp[(mblk * a.b + i) * a.V + x])
                          : -INFINITY;
    prod *= exp(lp);
    sum += prod;
  }
  a.terms[mblk] = static_cast<float>(sum / static_cast<double>(a.b));
}

// Mean of the per-block terms in a fixed order (one workgroup).
__global__ __launch_bounds__(kFT) void determinism_mean_kernel(DeterminismArgs a) {
  __shared__ double redd[kFW];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < a.M; i += kFT) s += static_cast<double>(a.terms[i]);
  s = block_sum_f64(s, redd);
  if (threadIdx.x == 0) *a.mean = static_cast<float>(s / static_cast<double>(a.M));
}

}  // namespace

hipError_t launch_filter(const FilterArgs& a, hipStream_t stream) {
  if (a.N > 0x7fffffff / 4) return hipErrorInvalidConfiguration;
  const dim3 rows(static_cast<unsigned>(a.N));
  const bool k_off = a.top_k == 0 || a.top_k >= a.V;
  const bool nucleus = a.temperature > 0.0f && k_off && a.top_p < 1.0f;
  const int segs = static_cast<int>(n_segs(a.V));
  // Split rows: with a workspace, from two segments on (the whole grids below stay in range).
  const bool split = a.row_ws && a.cuts && a.temperature > 0.0f && a.V >= kSplitMinV &&
                     a.N <= 0x7fffffff / (segs > 16 ? segs : 16);
  auto grid = [&](int per_row) { return dim3(static_cast<unsigned>(a.N * per_row)); };
  hipError_t e;
  if (a.temperature > 0.0f && k_off && !nucleus && segs <= kRowSegs) {
    hipLaunchKernelGGL(filter_scale_rows_kernel, rows, dim3(kSegT), 0, stream, a, segs);
  } else if (split && nucleus && a.V >= kSplitMinNucleus) {
    const int parts = static_cast<int>((a.V + kMassElems - 1) / kMassElems);
    hipLaunchKernelGGL(nucleus_max_kernel, grid(segs), dim3(kSegT), 0, stream, a, segs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(nucleus_mass_kernel, grid(parts), dim3(kFT), 0, stream, a, parts, segs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(nucleus_edge_kernel, rows, dim3(kFT), 0, stream, a, segs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(nucleus_gather_kernel, grid(segs), dim3(kSegT), 0, stream, a, segs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(nucleus_cut_kernel, rows, dim3(kFT), 0, stream, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(nucleus_write_kernel, grid(segs), dim3(kSegT), 0, stream, a, segs);
  } else if (split && k_off && !nucleus) {
    hipLaunchKernelGGL(filter_stats_kernel, grid(segs), dim3(kSegT), 0, stream, a, segs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(filter_scale_kernel, grid(segs), dim3(kSegT), 0, stream, a, segs);
  } else if (split && !k_off && a.top_k <= 256) {
    const int shares = top_shares(a.top_k);
    hipLaunchKernelGGL(filter_topk_share_kernel, grid(shares), dim3(kTopThreads), 0, stream, a,
                       shares);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(filter_topk_merge_kernel, rows, dim3(kFT), 0, stream, a, shares);
  } else if (nucleus) {
    hipLaunchKernelGGL(filter_nucleus_kernel, rows, dim3(kFT), 0, stream, a);
  } else {
    hipLaunchKernelGGL(filter_kernel, rows, dim3(kFT), 0, stream, a);
  }
  return hipGetLastError();
}

hipError_t launch_determinism(const DeterminismArgs& a, hipStream_t stream) {
  const int64_t blocks = (a.M + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(determinism_terms_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
                     stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !a.mean) return e;
  hipLaunchKernelGGL(determinism_mean_kernel, dim3(1), dim3(kFT), 0, stream, a);
  return hipGetLastError();
}

}  // namespace dbl
