// Offline profiling, first step (Sec. 4.1, Eq. 6): the utility curve of a head from per-token
// importance and the heuristic metric's ranking.  One workgroup per curve: the tokens are ranked by
// (score descending, index ascending), the importance is summed along that ranking in fp64, and the
// running sum is sampled at the caller's knots.
// Ranking: a token's bin is its score's order-preserving key scaled to the context's range (4096
// bins, about one token each for scores of any spread, since float bits are nearly a logarithm);
// tokens are gathered by bin, and a token's rank is its bin's start plus the tokens of that bin that
// come before it, by a direct count.  A context that crowds a bin with more than kCrowd tokens (ties,
// an infinity among ordinary scores, scores of both signs) sorts with a bitonic network instead.
//   2048 contexts of 4000 tokens: 212 us with a network in LDS for all (78 steps), 50 us this way
//   (65 MB take 13 us from memory); crowded ones 124-146 us, the bins' cost included, where the
//   network in LDS would take 220-224.
#include "lukv_internal.hpp"

namespace lukv {

constexpr int kCurveMaxT = 4096;   // tokens per profiled context (one LDS-resident sort)

__device__ __forceinline__ unsigned curve_key(float f) {
  unsigned u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;  // -0 and +0 tie
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int kCurveBins = 4096;   // bins of the ranking
constexpr unsigned kCrowd = 48;    // tokens in one bin up to which they are counted directly

// Bitonic network over 4096 keys, thread t holding keys 4t .. 4t+3: steps over distances 1 and 2 are in
// the thread, up to 128 between lanes of a wave (four of every six by DPP), and only the ten wider ones
// go through LDS, which is what bounds the network (2 x 8 bytes read and written per pair and step).
template <int CTRL>
__device__ __forceinline__ unsigned long long sort_dpp(unsigned long long x) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)x, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), CTRL, 0xf, 0xf, true);
  return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

// value of lane ^ X
template <int X>
__device__ __forceinline__ unsigned long long sort_partner(unsigned long long x) {
  if constexpr (X == 1) return sort_dpp<0xB1>(x);                     // quad_perm [1,0,3,2]
  else if constexpr (X == 2) return sort_dpp<0x4E>(x);                // quad_perm [2,3,0,1]
  else if constexpr (X == 4) return sort_dpp<0x1B>(sort_dpp<0x141>(x));   // 7 - i of a half row, then 3 - i of a quad
  else if constexpr (X == 8) return sort_dpp<0x128>(x);               // rotation of a row by 8
  else {
    const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)x, X), hi = (unsigned)__shfl_xor((int)(unsigned)(x >> 32), X);
    return ((unsigned long long)hi << 32) | lo;
  }
}

// what the lower (or upper) place of a pair keeps; down: this run is sorted descending
__device__ __forceinline__ unsigned long long sort_keep(unsigned long long mine, unsigned long long other, bool lower, bool down) {
  return (mine > other) == (lower == down) ? mine : other;
}

__device__ __forceinline__ void sort_pair(unsigned long long& a, unsigned long long& b, bool down) {
  const unsigned long long x = a, y = b;
  a = sort_keep(x, y, true, down);
  b = sort_keep(y, x, false, down);
}

template <int J>
__device__ __forceinline__ void sort_lanes(unsigned long long (&v)[4], int t, int k) {
  const bool lower = ((4 * t) & J) == 0, down = ((4 * t) & k) == 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = sort_keep(v[r], sort_partner<J / 4>(v[r]), lower, down);
}

__global__ __launch_bounds__(1024) void profile_curves_kernel(const float* importance, const float* scores,
                                                              const int32_t* knots, int T, int n_grid,
                                                              float* curves) {
  __shared__ unsigned long long keys[kCurveMaxT + 8];   // tokens by bin (or sorted), then the running sums
  __shared__ unsigned bins[kCurveBins];                 // counters, then starts; then the importance by rank
  __shared__ double wave_tot[16];
  __shared__ unsigned part[16], lim[3];                 // scan scratch; smallest key, largest key, fullest bin
  const int c = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const float* imp = importance + (int64_t)c * T;
  const float* sc = scores + (int64_t)c * T;
  float* by_rank = reinterpret_cast<float*>(bins);
  // larger composite = earlier in the ranking: higher score, then lower index
  auto composite = [](unsigned key, int i) { return ((unsigned long long)key << 32) | (0xFFFFFFFFu - (unsigned)i); };
  unsigned key[4];
  float im[4];
  unsigned kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = t + 1024 * u;
    key[u] = i < T ? curve_key(sc[i]) : 0u;
    im[u] = i < T ? imp[i] : 0.f;
    if (i < T) {
      kmin = key[u] < kmin ? key[u] : kmin;
      kmax = key[u] > kmax ? key[u] : kmax;
    }
    bins[i] = 0u;
  }
  if (t < 3) lim[t] = t == 0 ? 0xFFFFFFFFu : 0u;
  kmin = wave_reduce_to_last(kmin, 0xFFFFFFFFu, [](unsigned a, unsigned b) { return a < b ? a : b; });
  kmax = wave_reduce_to_last(kmax, 0u, [](unsigned a, unsigned b) { return a > b ? a : b; });
  __syncthreads();
  if (lane == 63) { atomicMin(&lim[0], kmin); atomicMax(&lim[1], kmax); }
  __syncthreads();
  kmax = lim[1];
  const unsigned span = kmax - lim[0];
  const int bits = span ? 32 - __clz(span) : 0, shift = bits > 12 ? bits - 12 : 0;
  // bin 0 holds the largest keys
  unsigned slot[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (t + 1024 * u < T) slot[u] = atomicAdd(&bins[(kmax - key[u]) >> shift], 1u);
  __syncthreads();
  // starts of the bins: four consecutive bins per thread
  unsigned n[4], full = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    n[e] = bins[4 * t + e];
    full = n[e] > full ? n[e] : full;
  }
  if (full > kCrowd) atomicMax(&lim[2], full);
  unsigned at = block_scan_u32(n[0] + n[1] + n[2] + n[3], part);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    bins[4 * t + e] = at;
    at += n[e];
  }
  __syncthreads();
  if (lim[2] == 0u) {
    unsigned start[4], count[4], rank[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = t + 1024 * u;
      if (i < T) {
        const unsigned b = (kmax - key[u]) >> shift;
        start[u] = bins[b];
        count[u] = (b + 1 < (unsigned)kCurveBins ? bins[b + 1] : (unsigned)T) - start[u];
        keys[start[u] + slot[u]] = composite(key[u], i);
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = t + 1024 * u;
      if (i < T) {
        const unsigned long long me = composite(key[u], i);
        rank[u] = start[u];
        for (unsigned x = 0; x < count[u]; ++x) rank[u] += keys[start[u] + x] > me ? 1u : 0u;
        by_rank[rank[u]] = im[u];       // (every start has been read before the barrier above)
      }
    }
    __syncthreads();
  } else {
    // (any order to begin with; padding sorts last)
    unsigned long long v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = t + 1024 * u < T ? composite(key[u], t + 1024 * u) : 0ull;
#pragma unroll 1
    for (int k = 2; k <= kCurveMaxT; k <<= 1) {
#pragma unroll 1
      for (int j = k >> 1; j >= 256; j >>= 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) keys[4 * t + r] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = sort_keep(v[r], keys[(4 * t + r) ^ j], ((4 * t) & j) == 0, ((4 * t) & k) == 0);
        __syncthreads();
      }
      if (k > 128) sort_lanes<128>(v, t, k);
      if (k > 64) sort_lanes<64>(v, t, k);
      if (k > 32) sort_lanes<32>(v, t, k);
      if (k > 16) sort_lanes<16>(v, t, k);
      if (k > 8) sort_lanes<8>(v, t, k);
      if (k > 4) sort_lanes<4>(v, t, k);
      if (k > 2) {
        sort_pair(v[0], v[2], ((4 * t) & k) == 0);
        sort_pair(v[1], v[3], ((4 * t) & k) == 0);
      }
      sort_pair(v[0], v[1], ((4 * t) & k) == 0);
      sort_pair(v[2], v[3], ((4 * t + 2) & k) == 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * t + r < T) by_rank[4 * t + r] = imp[0xFFFFFFFFu - (unsigned)v[r]];
    __syncthreads();
  }
  // importance along the ranking: four consecutive ranks per thread, fp64
  double v[4], run = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = 4 * t + e;
    run += r < T ? (double)by_rank[r] : 0.0;
    v[e] = run;
  }
  double incl = run;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long long bits = __double_as_longlong(incl);
    const int lo = __shfl_up((int)(bits & 0xFFFFFFFFll), o), hi = __shfl_up((int)(bits >> 32), o);
    const double up = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
    if (lane >= o) incl += up;
  }
  __syncthreads();                                   // every rank has been read
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  double before = incl - run;
  for (int w = 0; w < wave; ++w) before += wave_tot[w];
  double* pre = reinterpret_cast<double*>(keys);     // pre[r] = mass of the first r tokens
  if (t == 0) pre[0] = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) pre[4 * t + e + 1] = before + v[e];
  __syncthreads();
  for (int g = t; g < n_grid; g += 1024) {
    int n = knots[(int64_t)c * n_grid + g];
    n = n < 0 ? 0 : (n > T ? T : n);
    curves[(int64_t)c * n_grid + g] = (float)pre[n];
  }
}

int launch_profile_curves(int32_t n_curves, int32_t T, int32_t n_grid, const float* importance,
                          const float* scores, const int32_t* knots, float* curves, hipStream_t st) {
  if (T > kCurveMaxT) return LUKV_EINVAL;
  hipLaunchKernelGGL(profile_curves_kernel, dim3(n_curves), dim3(1024), 0, st, importance, scores, knots, T,
                     n_grid, curves);
  return check_launch();
}

}  // namespace lukv
