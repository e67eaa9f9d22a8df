// Consumer of the compacted cache: one decode step's attention over the retained entries of
// every head (Sec. 3.2, Eq. 3 restricted to the index set I_{l,h}).  The packed K and V rows of
// head hi sit at [offsets[hi], offsets[hi+1]); the G query heads of a group share them.
//   decode_partial - bound by the read of K and V, so there is no staging: a wave loads K rows in
//                    the layout of a matrix-core operand and V rows coalesced.  The logits of 16
//                    rows and up to 16 queries are one small product (exact products, 32-bit sums),
//                    which leaves a query's logits in one lane per row of 16 lanes: one exponential
//                    per logit, where a dot product spread over a row's lanes has all of them take
//                    it.  The weighted V sums stay on the vector ALU (32-bit probabilities), a
//                    probability reaching its row of lanes by a broadcast.  A row of lanes keeps a
//                    running (maximum, sum, weighted values) of its own rows; rows of lanes and
//                    waves meet once per head, in LDS.
//   decode_combine - one workgroup per (query head, head): merges the partial results.
// Row counts live on the device (they are budgets), so the host cannot size a grid by them.  The
// packed rows are cut into blocks of R rows, head hi owning the block numbers
// [offsets[hi] / R + hi, offsets[hi+1] / R + hi + 1) (one more than it needs at most, and no sum
// over the heads before it), and a fixed number of workgroups takes equal contiguous shares of
// them, so uneven heads cost nothing and no workgroup is launched for rows that do not exist.  A
// workgroup that meets a head leaves one partial result, in slot (workgroup + head): both only
// grow along the blocks, so no two share a slot.
//   Call times, 52 428 rows of 8 heads / 2.8 M rows of 512 heads (1.43 GB, bf16, d 128, G 4):
//     15.9 / 398 us  one workgroup per 128 rows of the longest possible head (4 of 5 to 12 of 13 of
//                    them empty), a partial result per block, dot products and a butterfly per row
//     17.6 / 265 us  equal shares
//     13.6 / 257 us  and the logits on the matrix cores
//     13.6 / 234 us  and the larger streamed
//     12.9 / 225 us  and 512 workgroups, shares at most a block apart (6.4 TB/s on the larger)
#include <type_traits>

#include "lukv_internal.hpp"

namespace lukv {

constexpr int kDecMaxGroup = 16;   // query heads per KV head the decode kernels take
constexpr int kDecWaves = 4;       // waves of a workgroup of decode_partial (their 16 rows of lanes meet at its end)

constexpr int64_t kDecStreamBytes = 256ll << 20;   // bytes of K and V from which they are streamed

struct DecGeom {
  int32_t n_layers, n_q_heads, n_kv_heads, group, n_seqs, n_heads_total;
  int32_t wgs_shift, singles;   // 1 << wgs_shift shares, or a share per block up to `singles` blocks
  float scale_log2e;
};

// Workgroups: two per CU, which every form has resident at once (16-bit rows and four query heads: four).
// More of them leave more partial results and, where the rest does not fit, a second round: 105 000 rows
// of 8 heads 20.5 us with 2048, 17.2 with 512 (bf16, d 128, G 4), in float32 35.4 and 27.7 (one workgroup
// per 128 rows: 23.2 and 30.9).  More heads than that are short ones, most often, and a workgroup meets
// several, one after the other: 4096 heads of 90 rows 42.9 us with 512, 37.0 with 2048.
// Up to 768 blocks are taken by as many workgroups where those are resident too (582 blocks of 16 heads
// 11.6 us, in 512 shares 12.5).
static int dec_wgs_shift(const HostCfg& hc) { return hc.n_hi <= 512 ? 9 : hc.g.group <= 4 ? 11 : 10; }
static int dec_singles(const HostCfg& hc, int shift) {
  const bool four = hc.g.head_dim == 64 || (!hc.g.f32 && hc.g.group <= 4);     // four workgroups a CU
  return four && shift == 9 ? 768 : 1 << shift;
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}

// value of lane N of this lane's row of 16 lanes
template <int N>
__device__ __forceinline__ float row_lane(float x) { return dpp_f<0x150 + N>(x); }

// maximum over a row of 16 lanes, left in every one of them
__device__ __forceinline__ float row_allmax(float x) {
  x = fmaxf(x, dpp_f<0xB1>(x));           // quad_perm [1,0,3,2]
  x = fmaxf(x, dpp_f<0x4E>(x));           // quad_perm [2,3,0,1]
  x = fmaxf(x, dpp_f<0x141>(x));          // row_half_mirror: lane i <-> 7 - i
  return fmaxf(x, dpp_f<0x140>(x));       // row_mirror: lane i <-> 15 - i
}

// acc += K piece * Q piece: 16 rows x 16 queries.  Lane l supplies 16 bytes of row (or query) l % 16;
// both operands take the same bytes of a row, so the order of the products inside does not matter.
// Result: acc[i] is row 4 * (l / 16) + i, query l % 16.
template <bool F32>
__device__ __forceinline__ f32x4 dec_mma(u32x4 k, u32x4 q, f32x4 acc) {
  if constexpr (!F32) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k), __builtin_bit_cast(bf16x8, q), acc, 0, 0, 0);
  } else {
    const f32x4 fk = __builtin_bit_cast(f32x4, k), fq = __builtin_bit_cast(f32x4, q);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fk[e], fq[e], acc, 0, 0, 0);
    return acc;
  }
}

// Geometry of a wave's step: kTiles tiles of 16 rows.  Of K a lane loads 16-byte pieces of one row of
// the tile, four lanes 64 neighbouring bytes; of V its piece (1/16 of a row) of four rows.
template <bool F32, int D>
struct DecTile {
  static constexpr int kEsize = F32 ? 4 : 2;
  static constexpr int kTiles = !F32 && D == 64 ? 2 : 1;
  static constexpr int kKLoads = D * kEsize / 64;       // K pieces per lane and tile: 2, 4 or 8
  static constexpr int kEpl = D / 16;                   // V elements per lane and row
  static constexpr int kVWords = D * kEsize / 64;       // 32-bit words they take: 2, 4 or 8
  static constexpr int kWaveRows = 16 * kTiles;
  static constexpr int kRows = kDecWaves * kWaveRows;   // rows per block: 64 or 128
  static constexpr int kShift = kRows == 64 ? 6 : 7;
  static_assert((1 << kShift) == kRows, "rows per block is a power of two");
};

// Block numbers of all heads, from `first`, the first head's, on.  Workgroup w takes the blocks from
// w * total >> shift on (all shares equal or one apart), or block w up to `singles` blocks.
struct DecShare { int64_t first; unsigned total; };

template <int SHIFT>
__device__ __forceinline__ DecShare dec_share(const DecGeom& g, int64_t off_first, int64_t off_last) {
  DecShare s;
  s.first = off_first >> SHIFT;
  s.total = (unsigned)((off_last >> SHIFT) - s.first + g.n_heads_total);
  return s;
}

__device__ __forceinline__ unsigned share_begin(const DecGeom& g, unsigned w, unsigned total) {
  if (total <= (unsigned)g.singles) return min(w, total);
  return w >> g.wgs_shift ? total : (unsigned)((uint64_t)w * total >> g.wgs_shift);
}

// the workgroup whose share holds block b: the largest w with w * total < (b + 1) << wgs_shift
__device__ __forceinline__ unsigned share_of(const DecGeom& g, unsigned b, unsigned total) {
  if (total <= (unsigned)g.singles) return b;
  if (total < (1u << 20)) return (((b + 1u) << g.wgs_shift) - 1u) / total;
  return (unsigned)(((((uint64_t)b + 1u) << g.wgs_shift) - 1u) / total);
}

__device__ __forceinline__ int64_t lane_i64(int64_t v, int src) {
  const int lo = __builtin_amdgcn_readlane((int)(v & 0xFFFFFFFFll), src);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), src);
  return ((int64_t)hi << 32) | (unsigned)lo;
}

template <bool STREAM>
__device__ __forceinline__ u32x4 dec_load(const char* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  else return *reinterpret_cast<const u32x4*>(p);
}

// W = 2, 4 or 8 words, aligned to 8 or 16 bytes
template <int W, bool STREAM>
__device__ __forceinline__ void dec_load_words(unsigned (&dst)[W], const char* p) {
  if constexpr (W >= 4) {
#pragma unroll
    for (int w = 0; w < W / 4; ++w) {
      const u32x4 x = dec_load<STREAM>(p + 16 * w);
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[4 * w + e] = x[e];
    }
  } else {
    typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
    const u32x2* p2 = reinterpret_cast<const u32x2*>(p);
    const u32x2 x = STREAM ? __builtin_nontemporal_load(p2) : *p2;
    dst[0] = x[0];
    dst[1] = x[1];
  }
}

__device__ __forceinline__ float dec_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// acc of query gq *= factor of lane gq of the row of lanes, for every gq
template <int NG, int EPL, int GQ = 0>
__device__ __forceinline__ void rescale(float (&acc)[NG][EPL], float factor) {
  if constexpr (GQ < NG) {
    const float f = row_lane<GQ>(factor);
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[GQ][e] *= f;
    rescale<NG, EPL, GQ + 1>(acc, factor);
  }
}

// acc of query gq += (p of lane gq of the row of lanes) * v
template <int NG, int EPL, int GQ = 0>
__device__ __forceinline__ void weigh(float (&acc)[NG][EPL], float p, const float (&v)[EPL]) {
  if constexpr (GQ < NG) {
    const float f = row_lane<GQ>(p);
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[GQ][e] = fmaf(f, v[e], acc[GQ][e]);
    weigh<NG, EPL, GQ + 1>(acc, p, v);
  }
}

// a += sum over the entries of (weight of lane `entry` of the row of lanes) * src[entry * stride]
template <int NE, int E = 0>
__device__ __forceinline__ void sum_entries(float& a, float w, const float* src, int stride) {
  if constexpr (E < NE) {
    a = fmaf(row_lane<E>(w), src[E * stride], a);
    sum_entries<NE, E + 1>(a, w, src, stride);
  }
}

// NG query heads' values at a time (blockIdx.y picks the NG-group when the GQA group is larger).
template <bool F32, int D, int NG>
__global__ __launch_bounds__(64 * kDecWaves, NG <= 4 ? (!F32 ? 4 : D == 64 ? 3 : 2) : 2) void decode_partial_kernel(
    DecGeom g, const char* q, const char* kp, const char* vp, const int64_t* offsets, float* part) {
  using T = DecTile<F32, D>;
  constexpr int EPL = T::kEpl, KL = T::kKLoads, VW = T::kVWords, NT = T::kTiles, R = T::kRows, WR = T::kWaveRows;
  constexpr int kRowBytes = D * T::kEsize;
  constexpr int NE = 4 * kDecWaves;                     // (wave, row of lanes) pairs that meet in LDS
  __shared__ float wm[NG][NE], wl[NG][NE];
  __shared__ __align__(16) float wacc[NE][NG][D];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int c = lane & 15, j = lane >> 4;
  const int G = g.group, g0 = blockIdx.y * NG;
  // The head that owns this workgroup's first block, by 64 probes a round.  The first round's loads
  // also bring the ends of the rows, and with up to 63 heads every offset there is: one dependent
  // load ahead of the rows.
  const int NH = g.n_heads_total;
  int step = NH <= 63 ? 1 : (NH + 63) >> 6;
  int64_t probe = offsets[min(lane * step, NH)];
  const int64_t off_last = offsets[NH];
  const int64_t off_first = lane_i64(probe, 0);
  const DecShare sh = dec_share<T::kShift>(g, off_first, off_last);
  unsigned f = share_begin(g, blockIdx.x, sh.total);
  const unsigned f_end = share_begin(g, blockIdx.x + 1, sh.total);
  if (f >= f_end) return;
  int hi = 0;
  for (int n = NH;;) {
    const int i = lane * step;
    const bool below = i < n && (probe >> T::kShift) - sh.first + hi + i <= (int64_t)f;
    const int at = max((int)__popcll(__ballot(below)) - 1, 0) * step;
    hi += at;
    n = min(step, n - at);
    if (n <= 1) break;
    step = (n + 63) >> 6;
    probe = offsets[min(hi + lane * step, NH)];
  }
  hi = __builtin_amdgcn_readfirstlane(hi);
  // More rows than the last-level cache holds are read with non-temporal loads, which the memory
  // serves at a higher rate (a plain read of 2 GiB: 6.2 against 7.0 TB/s): 1.43 GB 257 -> 234 us with 2048
  // workgroups.  Fewer may still be in the cache from the step before, and lose: 27 MB 13.3 -> 14.1 us.
  // Groups of more than eight take two passes and read the rows again.
  auto share = [&](auto stream_tag) __attribute__((always_inline)) {
  constexpr bool kStream = decltype(stream_tag)::value;
  for (; f < f_end && hi < NH; ++hi) {
    const int64_t o0 = NH <= 63 ? lane_i64(probe, hi) : offsets[hi];
    const int64_t o1 = NH <= 63 ? lane_i64(probe, hi + 1) : offsets[hi + 1];
    const int64_t b0 = (o0 >> T::kShift) - sh.first + hi, b1 = (o1 >> T::kShift) - sh.first + hi + 1;
    // (offsets that fall somewhere have no such numbering: nothing is read or written out of range then)
    if ((int64_t)f < b0 || (int64_t)f >= b1) continue;
    const unsigned fe = (unsigned)min((int64_t)f_end, b1);
    // rows of this head that this workgroup takes; this wave's steps start at r0, R apart (a head's
    // bytes fit 32 bits: at most 2^20 rows of 512 bytes)
    const int end = (int)min(o1 - o0, ((int64_t)fe - b0) * R);
    int r0 = (int)((int64_t)f - b0) * R + WR * wave;
    const char* kh = kp + o0 * kRowBytes;
    const char* vh = vp + o0 * kRowBytes;
    // rows beyond the end are clamped to the last one (and weighted 0)
    u32x4 kr[NT][KL];
    unsigned vr[NT][4][VW];
    auto fetch_k = [&](int row) {
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const char* src = kh + (unsigned)min(row + 16 * n + c, end - 1) * (unsigned)kRowBytes + 16u * (unsigned)j;
#pragma unroll
        for (int s = 0; s < KL; ++s) kr[n][s] = dec_load<kStream>(src + 64 * s);
      }
    };
    auto fetch_v = [&](int row) {
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const char* src = vh + (unsigned)min(row + 16 * n + 4 * j + i, end - 1) * (unsigned)kRowBytes + 4u * VW * (unsigned)c;
          dec_load_words<VW, kStream>(vr[n][i], src);
        }
    };
    // loads go out in the order their data is used: queries (beyond the NG-group: its last, unused), K, V
    const int kvh = hi % g.n_kv_heads, layer = (hi / g.n_kv_heads) % g.n_layers;
    const int seq = hi / (g.n_kv_heads * g.n_layers);
    u32x4 qr[KL];
    {
      const int64_t row = ((int64_t)layer * g.n_q_heads + kvh * G + min(g0 + c, G - 1)) * g.n_seqs + seq;
#pragma unroll
      for (int s = 0; s < KL; ++s) qr[s] = *reinterpret_cast<const u32x4*>(q + row * kRowBytes + 16 * j + 64 * s);
    }
    if (r0 < end) {
      fetch_k(r0);
      fetch_v(r0);
    }
    __builtin_amdgcn_sched_barrier(0);

    // Lane (c, j): running maximum (of the logits in units of log2, so that a probability is one
    // fused multiply-add and one exp2) and sum of query c over the rows 4j .. 4j+3 of every tile; and
    // of those rows' V, weighted, its own piece for every query: a row of 16 lanes shares one
    // reference, and the probabilities of a query reach its lanes by a row broadcast.
    float m = -INFINITY, l = 0.f, acc[NG][EPL];
#pragma unroll
    for (int gq = 0; gq < NG; ++gq)
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[gq][e] = 0.f;
#pragma unroll 1
    for (; r0 < end; r0 += R) {
      f32x4 p[NT];
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        // (independent products, added pairwise: half the rounding error of one chain)
        constexpr int NC = KL < 4 ? KL : 4;
        f32x4 x[NC];
#pragma unroll
        for (int s = 0; s < KL; ++s) x[s % NC] = dec_mma<F32>(kr[n][s], qr[s], s < NC ? f32x4{0.f, 0.f, 0.f, 0.f} : x[s % NC]);
#pragma unroll
        for (int w = NC / 2; w > 0; w /= 2)
#pragma unroll
          for (int s = 0; s < w; ++s) x[s] += x[s + w];
        p[n] = x[0];
      }
      // the next step's K rows replace the ones just used, and its V rows likewise below (after the
      // last step that is one row again and again: a branch here costs registers)
      fetch_k(r0 + R);
      float mn = -INFINITY;
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (r0 + 16 * n + 4 * j + i >= end) p[n][i] = -INFINITY;
          mn = fmaxf(mn, p[n][i]);
        }
      mn = fmaxf(m, mn * g.scale_log2e);
      const float ms = mn == -INFINITY ? 0.f : mn;         // (no live row met yet)
      const float keep = dec_exp2(m - ms);
      m = mn;
      l *= keep;
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          p[n][i] = dec_exp2(fmaf(p[n][i], g.scale_log2e, -ms));     // a row beyond the end: exp2(-inf) = 0
          l += p[n][i];
        }
      rescale<NG, EPL>(acc, keep);
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float vf[EPL];
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            if constexpr (F32) vf[e] = __uint_as_float(vr[n][i][e]);
            else vf[e] = __uint_as_float((e & 1) ? (vr[n][i][e >> 1] & 0xFFFF0000u) : (vr[n][i][e >> 1] << 16));
          }
          weigh<NG, EPL>(acc, p[n][i], vf);
        }
      fetch_v(r0 + R);
    }
    __syncthreads();                  // the previous head's results have been read
    {
      const int en = 4 * wave + j;
#pragma unroll
      for (int gq = 0; gq < NG; ++gq)
#pragma unroll
        for (int e = 0; e < EPL; e += 4)
          *reinterpret_cast<f32x4*>(&wacc[en][gq][c * EPL + e]) = f32x4{acc[gq][e], acc[gq][e + 1], acc[gq][e + 2], acc[gq][e + 3]};
      if (c < NG) {
        wm[c][en] = m;
        wl[c][en] = l;
      }
    }
    __syncthreads();
    // the NE results under their common maximum; a row of lanes holds the weights of one query
    float* my_part = part + ((int64_t)blockIdx.x + hi) * G * (D + 2);
#pragma unroll
    for (int o0 = 0; o0 < NG * D; o0 += 64 * kDecWaves) {
      const int o = o0 + t, gq = o / D, x = o - gq * D;    // (gq is the same over a wave: D >= 64)
      const float mine = wm[gq][c], M = row_allmax(mine);
      const float w = dec_exp2(mine - (M == -INFINITY ? 0.f : M));     // (the head's spare block: no row at all)
      float a = 0.f;
      sum_entries<NE>(a, w, &wacc[0][gq][x], NG * D);
      float s = w * wl[gq][c];
      s += dpp_f<0xB1>(s);
      s += dpp_f<0x4E>(s);
      s += dpp_f<0x141>(s);
      s += dpp_f<0x140>(s);
      if (g0 + gq < G) {
        float* dst = my_part + (g0 + gq) * (D + 2);
        dst[x] = a;
        if (x == 0) {
          dst[D] = M;
          dst[D + 1] = s;
        }
      }
    }
    f = fe;
  }
  };
  if (gridDim.y == 1 && (off_last - off_first) * (2 * kRowBytes) >= kDecStreamBytes) share(std::true_type{});
  else share(std::false_type{});
}

// One workgroup per (query head of the group, head, CW columns): the partial results of the
// workgroups that met the head are merged in one pass.  CW threads own the columns and NT / CW
// groups of them share the partial results; a group keeps a running maximum and rescales its sums
// when it grows (U values in flight at a time), and the groups meet once in LDS.
template <int D, int SHIFT, int NT, int CW, int U>
__global__ __launch_bounds__(NT) void decode_combine_kernel(DecGeom g, const int64_t* offsets, const float* part,
                                                            float* out) {
  constexpr int NP = NT / CW;           // groups of CW threads that share the partial results
  __shared__ float pm[NP], pl[NP];
  __shared__ float accs[NP][CW];
  const int gq = blockIdx.x, hi = blockIdx.y, t = threadIdx.x;
  const int G = g.group;
  const int kvh = hi % g.n_kv_heads, layer = (hi / g.n_kv_heads) % g.n_layers;
  const int seq = hi / (g.n_kv_heads * g.n_layers);
  const DecShare sh = dec_share<SHIFT>(g, offsets[0], offsets[g.n_heads_total]);
  const int64_t o0 = offsets[hi], o1 = offsets[hi + 1];
  const int x = t % CW, pt = t / CW, x0 = blockIdx.z * CW;
  float* dst = out + (((int64_t)layer * g.n_q_heads + kvh * G + gq) * g.n_seqs + seq) * D + x0;
  if (o1 <= o0) {
    if (t < CW) dst[t] = 0.f;
    return;
  }
  const unsigned b0 = (unsigned)((o0 >> SHIFT) - sh.first + hi), b1 = (unsigned)((o1 >> SHIFT) - sh.first + hi);
  const unsigned last = (unsigned)g.singles - 1u;        // (no limit but where offsets fall)
  const int w0 = (int)min(share_of(g, b0, sh.total), last);
  const int n_part = (int)min(share_of(g, b1, sh.total), last) - w0 + 1;
  const float* hp = part + (((int64_t)w0 + hi) * G + gq) * (D + 2);
  const int64_t bstride = (int64_t)G * (D + 2);
  float m_run = -INFINITY, a = 0.f, l = 0.f;
  for (int i0 = pt; i0 < n_part; i0 += NP * U) {
    float mb[U], lb[U], vb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * NP;
      const bool in = i < n_part;
      const float* bp = hp + (int64_t)(in ? i : i0) * bstride;
      const float mv = bp[D];
      mb[u] = in ? mv : -INFINITY;
      lb[u] = bp[D + 1];
      vb[u] = bp[x0 + x];
    }
    float m_new = m_run;
#pragma unroll
    for (int u = 0; u < U; ++u) m_new = fmaxf(m_new, mb[u]);
    const float ms = m_new == -INFINITY ? 0.f : m_new;           // (a partial result without rows)
    const float keep = dec_exp2(m_run - ms);                       // exp(-inf) = 0 the first time
    a *= keep;
    l *= keep;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float e = dec_exp2(mb[u] - ms);
      a = fmaf(vb[u], e, a);
      l = fmaf(lb[u], e, l);
    }
    m_run = m_new;
  }
  accs[pt][x] = a;
  if (x == 0) {
    pm[pt] = m_run;
    pl[pt] = l;
  }
  __syncthreads();
  if (t < CW) {
    float M = pm[0];
#pragma unroll
    for (int q2 = 1; q2 < NP; ++q2) M = fmaxf(M, pm[q2]);        // finite: the head has a row
    float tot = 0.f, den = 0.f;
#pragma unroll
    for (int q2 = 0; q2 < NP; ++q2) {
      const float e = dec_exp2(pm[q2] - M);                        // a group without rows: exp(-inf) = 0
      tot = fmaf(accs[q2][t], e, tot);
      den = fmaf(pl[q2], e, den);
    }
    dst[t] = tot / den;
  }
}

// One slot per workgroup and head.  (Never less than what one slot per 128 rows of the longest
// possible head takes, the size this query has always answered.)
int64_t decode_workspace_bytes(const HostCfg& hc) {
  const int64_t slots = (int64_t)hc.n_hi + dec_singles(hc, dec_wgs_shift(hc));
  const int64_t by_rows = (int64_t)hc.n_hi * ((hc.max_len + 127) / 128);
  return (slots > by_rows ? slots : by_rows) * hc.g.group * (hc.g.head_dim + 2) * 4;
}

template <bool F32, int D, int NG>
static int launch_decode_t(const HostCfg& hc, const void* q, const void* kp, const void* vp,
                           const int64_t* offsets, float* out, char* ws, hipStream_t st) {
  constexpr int S = DecTile<F32, D>::kShift;
  const Geom& g = hc.g;
  DecGeom dg{g.n_layers, g.n_q_heads, g.n_kv_heads, g.group, hc.seq.n_seqs, hc.n_hi, dec_wgs_shift(hc),
             dec_singles(hc, dec_wgs_shift(hc)),
             g.scale_log2e};
  float* part = reinterpret_cast<float*>(ws);
  hipLaunchKernelGGL((decode_partial_kernel<F32, D, NG>), dim3(dg.singles, (g.group + NG - 1) / NG),
                     dim3(64 * kDecWaves), 0, st, dg, (const char*)q, (const char*)kp, (const char*)vp, offsets, part);
  // Few heads, so many partial results of each: 32 groups share them and a workgroup takes 32 columns
  // (8 heads, 52 428 rows: 13.2 us a call against 17.5 with one workgroup for all columns).  Otherwise a
  // handful of partial results each, little to share, and the groups' workgroups would queue (64 heads
  // of 60 rows, G 4: 7.7 us against 11.0).
  if (hc.n_hi <= 8 || (hc.n_hi <= 32 && hc.n_hi * g.group <= 128))
    hipLaunchKernelGGL((decode_combine_kernel<D, S, 1024, 32, 4>), dim3(g.group, hc.n_hi, D / 32), dim3(1024), 0, st, dg,
                       offsets, (const float*)part, out);
  else
    hipLaunchKernelGGL((decode_combine_kernel<D, S, 256, D, 4>), dim3(g.group, hc.n_hi), dim3(256), 0, st, dg, offsets,
                       (const float*)part, out);
  return check_launch();
}

template <bool F32, int D>
static int launch_decode_g(const HostCfg& hc, const void* q, const void* kp, const void* vp,
                           const int64_t* offsets, float* out, char* ws, hipStream_t st) {
  // four queries at a time for small groups, eight otherwise (larger groups take several passes)
  if (hc.g.group <= 4) return launch_decode_t<F32, D, 4>(hc, q, kp, vp, offsets, out, ws, st);
  return launch_decode_t<F32, D, 8>(hc, q, kp, vp, offsets, out, ws, st);
}

int launch_decode(const HostCfg& hc, const void* q, const void* kp, const void* vp, const int64_t* offsets,
                  float* out, char* ws, hipStream_t st) {
  const Geom& g = hc.g;
  if (g.group > kDecMaxGroup) return LUKV_EINVAL;
  if (!g.f32 && g.head_dim == 128) return launch_decode_g<false, 128>(hc, q, kp, vp, offsets, out, ws, st);
  if (!g.f32 && g.head_dim == 64) return launch_decode_g<false, 64>(hc, q, kp, vp, offsets, out, ws, st);
  if (g.f32 && g.head_dim == 128) return launch_decode_g<true, 128>(hc, q, kp, vp, offsets, out, ws, st);
  if (g.f32 && g.head_dim == 64) return launch_decode_g<true, 64>(hc, q, kp, vp, offsets, out, ws, st);
  return LUKV_EDTYPE;
}

}  // namespace lukv
