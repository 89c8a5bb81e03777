// Pairwise registration on gfx950 after L-ORB: multi-probe LSH matching of the descriptors
// (Sec. 4.2.1; Alg. 3, step 1) and PROSAC screening with the transformation it yields
// (Sec. 4.2.2; Alg. 3, step 2; Alg. 4, step 5).
//
//   distance   L1 of the ternary descriptors = popcount(gt ^ gt') + popcount(lt ^ lt')
//   LSH        bit sampling of the "greater" string: table l's key has bit b = gt bit P[l][b]
//   probes     a query's own key and the k keys one bit away, in every table; a reference
//              point is a candidate when its key is one of them in some table
//   match      the nearest candidate by (distance, reference index), kept when <= D
//   PROSAC     m = 4, quality order (distance, query index), the growth function of Chum
//              and Matas (T_N given), draws from input uniforms, 4-point DLT (h33 = 1) in
//              FP64, degenerate samples (three collinear points) skipped, inliers by squared
//              reprojection error <= eps^2 with w > 0, a fixed budget of hypotheses, the best
//              by inlier count (ties to the earlier), then the least-squares DLT over its
//              inliers on Hartley-normalised coordinates (>= 5 inliers).
//
// Matching evaluates the probe predicate over every (query, reference) pair instead of
// building hash tables: the candidates, and hence the matches, are the same, and at the
// point counts of a detection area (hundreds to a few thousand) a wave per query scanning
// the reference keys and descriptors from L2 is faster than bucket lists.
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include <algorithm>
#include <climits>
#include <cmath>

#include "kernarg.h"
#include "stitch_internal.h"

using namespace stitch;

namespace {

constexpr int kMaxTables = 16, kMaxKeyBits = 24;
constexpr int kMaxPoints = 1 << 16;
constexpr int kMaxHyp = 1 << 16;
constexpr int kSample = 4;
constexpr int kMaxPairs = 256;

struct LshParams {
  int32_t tables, kbits, words, pad;          // words: 32-bit words per bit string (nd / 32)
  int16_t pos[kMaxTables][kMaxKeyBits];
};

__device__ __forceinline__ uint32_t key_of(const uint32_t* gt, const LshParams& P, int l) {
  uint32_t key = 0;
  for (int b = 0; b < P.kbits; ++b) {
    const int p = P.pos[l][b];
    key |= ((gt[p >> 5] >> (p & 31)) & 1u) << b;
  }
  return key;
}

// keys[l][i] of the first count rows of desc (rows of 2 * words uint32); each thread copies
// its row's "greater" words to LDS first, so the bit reads are LDS reads
__device__ __forceinline__ void lsh_keys_body(const uint32_t* __restrict__ desc, const int32_t* __restrict__ count,
                                              int cap, const LshParams& P, uint32_t* __restrict__ keys, int bx) {
  __shared__ uint32_t sRow[256][17];
  const int i = bx * 256 + threadIdx.x;
  const int n = min(*count, cap);
  if (i >= n) return;                               // no block barrier below
  const uint32_t* gt = desc + (int64_t)i * 2 * P.words;
  uint32_t* row = sRow[threadIdx.x];
  for (int w = 0; w < P.words; ++w) row[w] = gt[w];
  for (int l = 0; l < P.tables; ++l) keys[(int64_t)l * cap + i] = key_of(row, P, l);
}

__global__ void __launch_bounds__(256) k_lsh_keys(const uint32_t* __restrict__ desc, const int32_t* __restrict__ count,
                                                  int cap, const LshParams P, uint32_t* __restrict__ keys) {
  lsh_keys_body(desc, count, cap, P, keys, blockIdx.x);
}

// One wave per query: lanes stride over the reference points, then a (distance, index) min.
// Bound by the trips to memory: a lane reads the keys of eight tables for two reference points
// at once, and a candidate's descriptor 32 bytes at a time.  (Key by key with an exit at the
// first hit, every read waited for the one before: three pairs of 500 points, six tables,
// 21 us; now 10 us.)
__device__ __forceinline__ void lsh_match_body(const uint32_t* __restrict__ desc_a,
                                               const int32_t* __restrict__ count_a, int cap_a,
                                               const uint32_t* __restrict__ desc_b,
                                               const int32_t* __restrict__ count_b, int cap_b, const LshParams& P,
                                               const uint32_t* __restrict__ keys_a,
                                               const uint32_t* __restrict__ keys_b, int max_dist,
                                               int32_t* __restrict__ match, int32_t* __restrict__ dist, int bx) {
  const int lane = threadIdx.x & 63;
  const int i = bx * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (i >= cap_a) return;                           // whole waves leave; no block barrier below
  const int na = min(*count_a, cap_a), nb = min(*count_b, cap_b);
  if (i >= na) {
    if (lane == 0) {
      match[i] = -1;
      dist[i] = -1;
    }
    return;
  }
  const int words = P.words, tables = P.tables;
  const uint2* da = reinterpret_cast<const uint2*>(desc_a + (int64_t)i * 2 * words);
  unsigned long long best = ~0ull;                  // (distance << 32) | index
  for (int j0 = lane; j0 < nb; j0 += 128) {
    const int jj[2] = {j0, min(j0 + 64, nb - 1)};   // (a repeated last point changes nothing)
    bool cand[2] = {false, false};
    for (int l0 = 0; l0 < tables; l0 += 8) {
      uint32_t ka[8], kb[8][2];
#pragma unroll
      for (int l = 0; l < 8; ++l) {                 // (so does a repeated last table)
        const int t = min(l0 + l, tables - 1);
        ka[l] = keys_a[(int64_t)t * cap_a + i];
        kb[l][0] = keys_b[(int64_t)t * cap_b + jj[0]];
        kb[l][1] = keys_b[(int64_t)t * cap_b + jj[1]];
      }
#pragma unroll
      for (int l = 0; l < 8; ++l) {
        cand[0] |= __popc(ka[l] ^ kb[l][0]) <= 1;
        cand[1] |= __popc(ka[l] ^ kb[l][1]) <= 1;
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!cand[h]) continue;
      const uint2* db = reinterpret_cast<const uint2*>(desc_b + (int64_t)jj[h] * 2 * words);
      int d = 0;
      for (int w0 = 0; w0 < words; w0 += 4) {
        uint2 y[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) y[w] = db[min(w0 + w, words - 1)];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint2 x = da[min(w0 + w, words - 1)];
          const int pc = __popc(x.x ^ y[w].x) + __popc(x.y ^ y[w].y);
          d += w0 + w < words ? pc : 0;
        }
      }
      const unsigned long long kd = ((unsigned long long)d << 32) | (uint32_t)jj[h];
      best = kd < best ? kd : best;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o);
    best = other < best ? other : best;
  }
  if (lane == 0) {
    const int d = (int)(best >> 32);
    const bool ok = best != ~0ull && d <= max_dist;
    match[i] = ok ? (int)(uint32_t)best : -1;
    dist[i] = ok ? d : -1;
  }
}

__global__ void __launch_bounds__(256) k_lsh_match(const uint32_t* __restrict__ desc_a,
                                                   const int32_t* __restrict__ count_a, int cap_a,
                                                   const uint32_t* __restrict__ desc_b,
                                                   const int32_t* __restrict__ count_b, int cap_b, const LshParams P,
                                                   const uint32_t* __restrict__ keys_a,
                                                   const uint32_t* __restrict__ keys_b, int max_dist,
                                                   int32_t* __restrict__ match, int32_t* __restrict__ dist) {
  lsh_match_body(desc_a, count_a, cap_a, desc_b, count_b, cap_b, P, keys_a, keys_b, max_dist, match, dist, blockIdx.x);
}

// Several pairs per launch: blockIdx.y selects the pair (keys: pair y / 2, side y % 2), its
// descriptor read from a device table; blocks past a pair's own extent leave at once.
struct LshPairDev {
  const uint32_t* desc_a;
  const int32_t* count_a;
  const uint32_t* desc_b;
  const int32_t* count_b;
  uint32_t* keys_a;
  uint32_t* keys_b;
  int32_t* match;
  int32_t* dist;
  int32_t cap_a, cap_b;
};

// Up to kArgPairs pairs travel as a kernel argument (taken at launch: no upload and no host
// wait, and the launch can be captured into a graph); more come from a device table.
constexpr int kArgPairs = 16;
template <typename D>
struct PairArgs {
  D p[kArgPairs];
};
// A block's descriptor, by scalar reads, from the table or from the kernel's first argument
// (PairArgs<D>): neither is written meanwhile.  (Through a pointer to either, every field was a read
// per lane.)
template <typename D>
__device__ __forceinline__ D pair_of(const D* __restrict__ table, int i) {
  static_assert(sizeof(D) % 4 == 0, "whole dwords");
  typedef const __attribute__((address_space(4))) uint32_t* ConstWords;
  const ConstWords w = (ConstWords)(table ? (const __attribute__((address_space(4))) D*)table + i : first_arg<D>() + i);
  D q;
  uint32_t* d = reinterpret_cast<uint32_t*>(&q);
#pragma unroll
  for (int k = 0; k < (int)(sizeof(D) / 4); ++k) d[k] = w[k];
  return q;
}

__global__ void __launch_bounds__(256) k_lsh_keys_multi(const PairArgs<LshPairDev>,
                                                        const LshPairDev* __restrict__ pairs, const LshParams P) {
  const LshPairDev q = pair_of(pairs, blockIdx.y >> 1);
  const bool b = blockIdx.y & 1;
  const int cap = b ? q.cap_b : q.cap_a;
  if ((int)blockIdx.x * 256 >= cap) return;
  lsh_keys_body(b ? q.desc_b : q.desc_a, b ? q.count_b : q.count_a, cap, P, b ? q.keys_b : q.keys_a, blockIdx.x);
}

__global__ void __launch_bounds__(256) k_lsh_match_multi(const PairArgs<LshPairDev>,
                                                         const LshPairDev* __restrict__ pairs, const LshParams P,
                                                         int max_dist) {
  const LshPairDev q = pair_of(pairs, blockIdx.y);
  if ((int)blockIdx.x * 4 >= q.cap_a) return;
  lsh_match_body(q.desc_a, q.count_a, q.cap_a, q.desc_b, q.count_b, q.cap_b, P, q.keys_a, q.keys_b, max_dist, q.match,
                 q.dist, blockIdx.x);
}

// ---------------------------------------------------------------------------- PROSAC
struct ProsacWs {            // offsets into the workspace
  size_t misc, qa, qb, qi, tp, hyp_h, hyp_ok;
};

// ---- moves within a wave (no LDS memory, no address registers) ----
// Lane l's value, l the same in every lane.
__device__ __forceinline__ double lane_of(double v, int l) {
  const long long b = __builtin_bit_cast(long long, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), l);
  return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
// Value of lane ^ X for X = 1, 2, 8 (within a row of 16 lanes), 4, 16 (within 32) and 32.
template <int X>
__device__ __forceinline__ int swap32(int v) {
  if (X == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);        // quad_perm 1 0 3 2
  if (X == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);        // quad_perm 2 3 0 1
  if (X == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true);       // row_ror 8
  if (X == 4) return __builtin_amdgcn_ds_swizzle(v, (4 << 10) | 0x1F);
  if (X == 16) return __builtin_amdgcn_ds_swizzle(v, (16 << 10) | 0x1F);
  return __shfl_xor(v, 32);
}
template <int X>
__device__ __forceinline__ double swap64(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const uint32_t lo = (uint32_t)swap32<X>((int)b), hi = (uint32_t)swap32<X>((int)(b >> 32));
  return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}

// The growth function T'_n, n = 4 .. M, by one wave: T_{n+1} = T_n (n + 1) / (n - 3) in FP64, each
// rounded, T' the sum of ceil(T_{n+1} - T_n) from 1.  The chain of T is serial; a step is one
// product p and, in place of a division (some fifteen dependent operations), the quotient from the
// divisor's reciprocal r and one correction: q0 = T c with c = (n + 1) r, beside p, then
// q = q0 + (p - b q0) r.  That is the rounded quotient: q0 is within four of its last places, b
// is a whole number below 2^16, so p - b q0 is exact (a multiple of q0's last place, at most
// 2^19 of them), q's error before its rounding is below 2^-50 of a last place, and p / b lies
// no closer than 1 / 2b of one to a midpoint between two doubles (it is none itself: b
// times an odd 54-bit number has more than 53 bits).  Sixty-four steps' r and c come from the
// wave's lanes, and their sums go out together: 500 matches took 37 us division by division,
// the whole kernel now takes 19.
__device__ __forceinline__ void prosac_growth(double T_N, int M, int64_t* __restrict__ tp) {
  const int lane = threadIdx.x & 63;
  double T = T_N;
  for (int i = 0; i < kSample; ++i) T = T * (double)(kSample - i) / (double)(M - i);
  if (lane == 0) tp[kSample] = 1;
  if (!(T > 0x1p-900)) {                            // quotients too small for the correction
    if (lane != 0) return;
    for (int n = kSample; n < M; ++n) {
      const double Tn = T * (double)(n + 1) / (double)(n + 1 - kSample);
      tp[n + 1] = tp[n] + (int64_t)ceil(Tn - T);
      T = Tn;
    }
    return;
  }
  __shared__ double sStep[64][4];                   // r, c, n + 1 and -b of 64 steps
  __shared__ double sT[64];
  auto settle = [] {                                // the wave's LDS writes before its reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  int64_t total = 1;
  for (int n0 = kSample; n0 < M; n0 += 64) {
    const double b = (double)(n0 + lane + 1 - kSample), up = (double)(n0 + lane + 1), r = 1.0 / b;
    sStep[lane][0] = r;
    sStep[lane][1] = up * r;
    sStep[lane][2] = up;
    sStep[lane][3] = -b;
    settle();
    const double first = T;
#pragma unroll 16
    for (int i = 0; i < 64; ++i) {                  // (steps past M end nowhere)
      const double p = T * sStep[i][2], q0 = T * sStep[i][1];
      T = __builtin_fma(__builtin_fma(sStep[i][3], q0, p), sStep[i][0], q0);
      sT[i] = T;
    }
    settle();
    const int steps = min(64, M - n0);
    const double Tl = lane ? sT[(lane + 63) & 63] : first;
    int64_t d = lane < steps ? (int64_t)ceil(sT[lane] - Tl) : 0;
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t e = __shfl_up(d, o);
      if (lane >= o) d += e;
    }
    if (lane < steps) tp[n0 + lane + 1] = total + d;
    total += __shfl(d, 63);
    settle();
  }
}

// misc: [0] M = number of matches
// one block of 1024 threads: matches in quality order, and T'_n for n = 4 .. M
__device__ __forceinline__ void prosac_prepare_body(const int32_t* __restrict__ pts_a,
                                                    const int32_t* __restrict__ pts_b, int cap_b,
                                                    const int32_t* __restrict__ match,
                                                    const int32_t* __restrict__ dist,
                                                    const int32_t* __restrict__ count_a, int cap_a, double T_N,
                                                    int32_t* __restrict__ misc, int2* __restrict__ qa,
                                                    int2* __restrict__ qb, int32_t* __restrict__ qi,
                                                    int64_t* __restrict__ tp) {
  constexpr int kStage = 16384;                      // ranking keys staged in LDS up to here
  __shared__ int sM;
  __shared__ __attribute__((aligned(16))) int32_t sKey[kStage];
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int na = min(*count_a, cap_a);
  // ranking key of query j: its distance when it has a match (below INT32_MAX), else
  // INT32_MAX, which precedes nothing and equals no valid key
  auto key = [&](int j) -> int {
    const int mj = match[j], dj = dist[j];
    return (mj >= 0 && mj < cap_b) ? min(dj, INT32_MAX - 1) : INT32_MAX;
  };
  const bool staged = na <= kStage;
  const int npad = (na + 3) & ~3;
  if (tid == 0) sM = 0;
  __syncthreads();
  // the keys, and the number of valid matches
  int local = 0;
  for (int j = tid; j < npad; j += 1024) {
    const int k = j < na ? key(j) : INT32_MAX;
    if (staged) sKey[j] = k;
    local += k != INT32_MAX;
  }
  for (int o = 32; o > 0; o >>= 1) local += __shfl_xor(local, o);
  if ((tid & 63) == 0) atomicAdd(&sM, local);
  __syncthreads();
  const int M = sM;
  // the growth function, on the last wave, ahead of its share of the ranking (the others go on)
  if (wv == 15 && M >= kSample) {
    __builtin_amdgcn_s_setprio(2);
    prosac_growth(T_N, M, tp);
    __builtin_amdgcn_s_setprio(0);
  }
  if (tid == 0) misc[0] = M;
  // rank of match i: the valid matches ordered before it by (distance, query index): keys up
  // to its own before it, keys below its own after it
  if (staged) {
    for (int i = tid; i < na; i += 1024) {
      const int ki = sKey[i];
      if (ki == INT32_MAX) continue;
      int r = 0;
      const int mi = match[i];                       // on its way meanwhile
      const int2 a = make_int2(pts_a[2 * i], pts_a[2 * i + 1]);
      const int2 b = make_int2(pts_b[2 * mi], pts_b[2 * mi + 1]);
      const int first = i & ~63, last = min(first + 64, npad);   // the wave's own matches
      int j = 0;
#pragma unroll 4
      for (; j < first; j += 4) {
        const int4 v = *reinterpret_cast<const int4*>(&sKey[j]);
        r += (v.x <= ki) + (v.y <= ki) + (v.z <= ki) + (v.w <= ki);
      }
#pragma unroll 4
      for (; j < last; j += 4) {
        const int4 v = *reinterpret_cast<const int4*>(&sKey[j]);
        r += (v.x < ki + (j < i)) + (v.y < ki + (j + 1 < i)) + (v.z < ki + (j + 2 < i)) + (v.w < ki + (j + 3 < i));
      }
#pragma unroll 4
      for (; j < npad; j += 4) {
        const int4 v = *reinterpret_cast<const int4*>(&sKey[j]);
        r += (v.x < ki) + (v.y < ki) + (v.z < ki) + (v.w < ki);
      }
      qa[r] = a;
      qb[r] = b;
      qi[r] = i;
    }
    return;
  }
  // more keys than are staged at once: 1024 matches against a stage of keys after another (read from
  // memory by every wave, 65000 matches took 763 ms, 818 with both reads of a key unconditional; now 142)
  for (int i0 = 0; i0 < na; i0 += 1024) {
    const int i = i0 + tid;
    const int ki = i < na ? key(i) : INT32_MAX;
    const int k0 = min(ki, INT32_MAX - 1);
    int r = 0;
    for (int t0 = 0; t0 < na; t0 += kStage) {
      const int n = min(na - t0, kStage);
      __syncthreads();
      for (int j = tid; j < ((n + 3) & ~3); j += 1024) sKey[j] = j < n ? key(t0 + j) : INT32_MAX;
      __syncthreads();
#pragma unroll 4
      for (int j = 0; j < n; j += 4) {
        const int4 v = *reinterpret_cast<const int4*>(&sKey[j]);
        const int at = t0 + j;
        r += (v.x < k0 + (at < i)) + (v.y < k0 + (at + 1 < i)) + (v.z < k0 + (at + 2 < i)) + (v.w < k0 + (at + 3 < i));
      }
    }
    if (ki == INT32_MAX) continue;
    const int mi = match[i];
    qa[r] = make_int2(pts_a[2 * i], pts_a[2 * i + 1]);
    qb[r] = make_int2(pts_b[2 * mi], pts_b[2 * mi + 1]);
    qi[r] = i;
  }
}

__global__ void __launch_bounds__(1024) k_prosac_prepare(const int32_t* __restrict__ pts_a,
                                                         const int32_t* __restrict__ pts_b, int cap_b,
                                                         const int32_t* __restrict__ match,
                                                         const int32_t* __restrict__ dist,
                                                         const int32_t* __restrict__ count_a, int cap_a, double T_N,
                                                         int32_t* __restrict__ misc, int2* __restrict__ qa,
                                                         int2* __restrict__ qb, int32_t* __restrict__ qi,
                                                         int64_t* __restrict__ tp) {
  prosac_prepare_body(pts_a, pts_b, cap_b, match, dist, count_a, cap_a, T_N, misc, qa, qb, qi, tp);
}

__device__ __forceinline__ bool collinear(int2 p, int2 q, int2 r) {
  return (int64_t)(q.x - p.x) * (r.y - p.y) - (int64_t)(q.y - p.y) * (r.x - p.x) == 0;
}

__device__ __forceinline__ bool degenerate4(const int2 (&p)[4]) {
  return collinear(p[0], p[1], p[2]) | collinear(p[0], p[1], p[3]) | collinear(p[0], p[2], p[3]) |
         collinear(p[1], p[2], p[3]);
}

// Solve the 8 x 8 system A x = b with one wave: lane l holds a = A[l / 8][l % 8] and bv =
// b[l / 8].  Gaussian elimination with partial pivoting (largest |pivot|, the first row on
// ties), then back substitution; returns x[l % 8] in every lane, and false (in every lane) when
// a pivot is zero.  Rows stay in their lanes and carry their place instead of being swapped;
// every column finds its own largest entry, of which column k's is read.  Bound by its serial
// chain of moves and divisions, of which the moves are now few and need no address (DPP,
// swizzle, readlane): k_prosac_hyp, 1024 hypotheses for each of three pairs, 25 -> 14.7 us.
__device__ __forceinline__ bool wave_solve8(double a, double bv, double& x_mine) {
  const int lane = threadIdx.x & 63, r = lane >> 3, c = lane & 7;
  int place = r;                                     // of this lane's row
  int at[8];                                         // row lanes 8 at[k] .. hold pivot row k
  auto better = [](double v2, int p2, double& v, int& p) {
    const bool t = v2 > v || (v2 == v && p2 < p);
    v = t ? v2 : v;
    p = t ? p2 : p;
  };
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const double col = __shfl(a, (lane & 56) + k);
    double v = place >= k ? fabs(a) : -1.0;
    int p = place * 8 + r;
    better(swap64<8>(v), swap32<8>(p), v, p);
    better(swap64<16>(v), swap32<16>(p), v, p);
    better(swap64<32>(v), swap32<32>(p), v, p);
    if (!(lane_of(v, k) > 0.0)) return false;
    p = __builtin_amdgcn_readlane(p, k);
    const int g = p & 7;
    at[k] = g;
    place = r == g ? k : place == k ? p >> 3 : place;
    const double prow = __shfl(a, g * 8 + c), piv = lane_of(a, g * 8 + k), bk = lane_of(bv, g * 8);
    const double f = col / piv;
    if (place > k) {
      if (c >= k) a = __builtin_fma(-f, prow, a);
      bv = __builtin_fma(-f, bk, bv);
    }
  }
  x_mine = 0.0;
#pragma unroll
  for (int k = 7; k >= 0; --k) {
    double t = c > k ? a * x_mine : 0.0;             // of every row; row k's sum is read
    t += 0.0;
    t += swap64<4>(t);
    t += swap64<2>(t);
    t += swap64<1>(t);
    const double xk = (lane_of(bv, at[k] * 8) - lane_of(t, at[k] * 8)) / lane_of(a, at[k] * 8 + k);
    if (c == k) x_mine = xk;
  }
  return true;
}

// squared reprojection test in the order of its definition (no contraction)
__device__ __forceinline__ bool is_inlier(const double* H, int2 p, int2 q, double eps2) {
#pragma clang fp contract(off)
  const double x = p.x, y = p.y;
  const double X = H[0] * x + H[1] * y + H[2];
  const double Y = H[3] * x + H[4] * y + H[5];
  const double W = H[6] * x + H[7] * y + H[8];
  if (!(W > 0.0)) return false;
  const double ex = X / W - (double)q.x, ey = Y / W - (double)q.y;
  return ex * ex + ey * ey <= eps2;
}

// r-th index of [0, R) not among the kN first of `chosen`, in increasing order
template <int kN>
__device__ __forceinline__ int nth_free(int r, const int (&chosen)[4]) {
  int s[3] = {INT32_MAX, INT32_MAX, INT32_MAX};        // sorted, the unused ones last
#pragma unroll
  for (int k = 0; k < kN; ++k) s[k] = chosen[k];
  auto order = [&](int a, int b) {
    const int lo = min(s[a], s[b]), hi = max(s[a], s[b]);
    s[a] = lo;
    s[b] = hi;
  };
  order(0, 1);
  order(1, 2);
  order(0, 1);
#pragma unroll
  for (int k = 0; k < 3; ++k) r += s[k] <= r ? 1 : 0;
  return r;
}

// rows of the DLT system (h33 = 1) for a correspondence (x, y) -> (u, v):
//   r0 = [x, y, 1, 0, 0, 0, -u x, -u y] (right side u), r1 = [0, 0, 0, x, y, 1, -v x, -v y] (v)
__device__ __forceinline__ double row0(int i, double x, double y, double u) {
  return i == 0 ? x : i == 1 ? y : i == 2 ? 1.0 : i == 6 ? -u * x : i == 7 ? -u * y : 0.0;
}
__device__ __forceinline__ double row1(int i, double x, double y, double v) {
  return i == 3 ? x : i == 4 ? y : i == 5 ? 1.0 : i == 6 ? -v * x : i == 7 ? -v * y : 0.0;
}

// one wave per hypothesis t: its sample (by every lane alike), its model and its inlier count
__device__ __forceinline__ void prosac_hyp_body(const int32_t* __restrict__ misc, const int2* __restrict__ qa,
                                                const int2* __restrict__ qb, const int64_t* __restrict__ tp,
                                                int nhyp, const double* __restrict__ uniforms, double eps2,
                                                double* __restrict__ hyp_h, int32_t* __restrict__ hyp_ok,
                                                int32_t* __restrict__ hyp_counts, int bx) {
  const int lane = threadIdx.x & 63;
  const int t = bx * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);   // hypothesis t + 1 of the schedule
  if (t >= nhyp) return;                              // whole waves; no block barrier below
  double u[4];
  for (int k = 0; k < 4; ++k) u[k] = uniforms[(int64_t)t * 4 + k];
  const int M = misc[0];
  if (M < kSample) {
    if (lane == 0) {
      hyp_ok[t] = 0;
      hyp_counts[t] = 0;
    }
    return;
  }
  // n_t = 4 + #{n in [4, M-1] : T'_n <= t+1}: the increasing T' searched 64 ways at a time for
  // the first n in [4, M) with T'_n > tt (or M)
  const int64_t tt = t + 1;
  int n = kSample, left = M - kSample;
  while (left > 0) {
    const int step = (left + 63) >> 6, q = (lane + 1) * step - 1;    // ends of up to 64 parts
    const bool below = q < left && tp[n + q] <= tt;
    const int parts = __popcll(__ballot(below));
    n += parts * step;
    left = min(left - parts * step, step - 1);
  }
  const bool nth = !(tp[n] < tt);
  int idx[4] = {0, 0, 0, 0};
  const int R = nth ? n - 1 : n;
  // clamped into the range (uniforms outside [0, 1), even NaN, cannot index outside it)
  auto pick = [&](int k) {
    const double f = floor(u[k] * (double)(R - k));
    return f >= 0.0 ? (int)fmin(f, (double)(R - k - 1)) : 0;
  };
  idx[0] = nth_free<0>(pick(0), idx);
  idx[1] = nth_free<1>(pick(1), idx);
  idx[2] = nth_free<2>(pick(2), idx);
  idx[3] = nth ? n - 1 : nth_free<3>(pick(3), idx);
  int2 pa[4], pb[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    pa[k] = qa[idx[k]];
    pb[k] = qb[idx[k]];
  }
  double h = 0.0;
  bool ok = !degenerate4(pa) && !degenerate4(pb);
  if (ok) {
    // lane (row, col) of the 8 x 8 DLT system: rows 2k, 2k+1 from correspondence k
    const int r = lane >> 3, c = lane & 7, k = r >> 1;
    auto of = [k](int a0, int a1, int a2, int a3) { return (double)(k == 0 ? a0 : k == 1 ? a1 : k == 2 ? a2 : a3); };
    const double x = of(pa[0].x, pa[1].x, pa[2].x, pa[3].x), y = of(pa[0].y, pa[1].y, pa[2].y, pa[3].y);
    const double u2 = of(pb[0].x, pb[1].x, pb[2].x, pb[3].x), v2 = of(pb[0].y, pb[1].y, pb[2].y, pb[3].y);
    const double a = (r & 1) ? row1(c, x, y, v2) : row0(c, x, y, u2);
    ok = wave_solve8(a, (r & 1) ? v2 : u2, h);
    h = ok ? h : 0.0;
  }
  double H[9];
#pragma unroll
  for (int i = 0; i < 8; ++i) H[i] = lane_of(h, i);
  H[8] = 1.0;
  int cnt = 0;
  if (ok) {
    // two points a lane at once
    for (int k = lane; k < M; k += 128) {
      const int k2 = min(k + 64, M - 1);
      const int2 a1 = qa[k], b1 = qb[k], a2 = qa[k2], b2 = qb[k2];
      cnt += is_inlier(H, a1, b1, eps2);
      cnt += (k + 64 < M) & is_inlier(H, a2, b2, eps2);
    }
  }
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
  if (lane == 0) {
    hyp_ok[t] = ok;
    hyp_counts[t] = ok ? cnt : 0;
  }
  if (lane < 9) hyp_h[(int64_t)t * 9 + lane] = lane < 8 ? h : 1.0;
}

__global__ void __launch_bounds__(256) k_prosac_hyp(const int32_t* __restrict__ misc, const int2* __restrict__ qa,
                                                    const int2* __restrict__ qb, const int64_t* __restrict__ tp,
                                                    int nhyp, const double* __restrict__ uniforms, double eps2,
                                                    double* __restrict__ hyp_h, int32_t* __restrict__ hyp_ok,
                                                    int32_t* __restrict__ hyp_counts) {
  prosac_hyp_body(misc, qa, qb, tp, nhyp, uniforms, eps2, hyp_h, hyp_ok, hyp_counts, blockIdx.x);
}

// sum over a wave, in every lane
__device__ __forceinline__ double wave_sum(double v) {
  v += swap64<1>(v);
  v += swap64<2>(v);
  v += swap64<4>(v);
  v += swap64<8>(v);
  v += swap64<16>(v);
  v += swap64<32>(v);
  return v;
}

// block-wide sums (kWaves waves) of N values into every thread; sRed holds kWaves x N partials,
// added in a fixed order
template <int kWaves, int N>
__device__ __forceinline__ void block_sums(double* sRed, double (&v)[N]) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double s = wave_sum(v[i]);
    if (lane == 0) sRed[w * N + i] = s;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double s = 0.0;
    for (int k = 0; k < kWaves; ++k) s += sRed[k * N + i];
    v[i] = s;
  }
}

constexpr int kFinalThreads = 512, kFinalWaves = kFinalThreads / 64;
constexpr int kMoments = 22;

// One block of kFinalThreads: the best hypothesis, its inliers, the least-squares refit.  A chain of
// short steps, each bound by one trip to memory or one reduction.  The normal equations' 72
// entries are 22 different sums over the inliers -- the moments of (1, u, v, u^2 + v^2) with (1,
// x, y, xx, xy, yy) -- so a thread adds its points' moments and one reduction ends them
// (entry by entry, seven threads each over a seventh of the points, every point read
// again behind its flag: 75 us for 500 points and 1024 hypotheses; now 16 us).
__device__ __forceinline__ void prosac_final_body(const int32_t* __restrict__ misc,
                                                  const int2* __restrict__ qa, const int2* __restrict__ qb,
                                                  const int32_t* __restrict__ qi, int cap_a, int nhyp,
                                                  const double* __restrict__ hyp_h,
                                                  const int32_t* __restrict__ hyp_ok,
                                                  const int32_t* __restrict__ hyp_counts, double eps2,
                                                  double* __restrict__ H_out, int32_t* __restrict__ inliers,
                                                  uint8_t* __restrict__ mask) {
  __shared__ unsigned long long sBest[kFinalWaves];
  __shared__ double sRed[kFinalWaves * kMoments];
  __shared__ uint32_t sFlag[kMaxPoints / 32];
  const int tid = threadIdx.x, lane = tid & 63;
  const int M = misc[0];
  for (int i = tid; i < cap_a; i += kFinalThreads) mask[i] = 0;
  // best: most inliers, then the earliest hypothesis; key (count + 1) << 32 | (2^32-1 - t)
  unsigned long long best = 0ull;
  for (int t = tid; t < nhyp; t += kFinalThreads) {
    const int ok = hyp_ok[t], count = hyp_counts[t];
    const unsigned long long k = ((unsigned long long)(count + 1) << 32) | (0xFFFFFFFFull - (unsigned)t);
    best = ok && k > best ? k : best;
  }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o);
    best = other > best ? other : best;
  }
  if (lane == 0) sBest[tid >> 6] = best;
  __syncthreads();
  for (int w = 0; w < kFinalWaves; ++w) best = sBest[w] > best ? sBest[w] : best;
  if (best == 0ull) {                                 // no valid hypothesis
    if (tid < 9) H_out[tid] = 0.0;
    if (tid == 0) *inliers = 0;
    return;
  }
  const int tb = (int)(0xFFFFFFFFull - (best & 0xFFFFFFFFull));
  double Hb[9];
  for (int c = 0; c < 9; ++c) Hb[c] = hyp_h[(int64_t)tb * 9 + c];
  // inliers of the best model (flags, mask over queries) and the sums for the normalisation
  double m[5] = {0, 0, 0, 0, 0};
  for (int k0 = 0; k0 < M; k0 += kFinalThreads) {     // every lane in every turn: a ballot a wave
    const int k = k0 + tid, kc = min(k, M - 1);
    const int2 a = qa[kc], b = qb[kc];
    const int i = qi[kc];
    const bool in = (k < M) & is_inlier(Hb, a, b, eps2);
    const uint64_t bits = __ballot(in);
    if (lane < 2 && k - lane < M) sFlag[((k - lane) >> 5) + lane] = (uint32_t)(bits >> (32 * lane));
    if (in) {
      mask[i] = 1;
      m[0] += 1.0;
      m[1] += a.x;
      m[2] += a.y;
      m[3] += b.x;
      m[4] += b.y;
    }
  }
  block_sums<kFinalWaves>(sRed, m);                   // (its barriers also publish sFlag)
  const double n_in = m[0];
  if (tid == 0) *inliers = (int)n_in;
  if (n_in < 5.0) {
    if (tid < 9) H_out[tid] = Hb[tid] / Hb[8];
    return;
  }
  const double cx = m[1] / n_in, cy = m[2] / n_in, cu = m[3] / n_in, cv = m[4] / n_in;
  auto flag = [&](int k) { return ((sFlag[k >> 5] >> (k & 31)) & 1u) != 0; };
  double d[2] = {0, 0};
  for (int k = tid; k < M; k += kFinalThreads) {
    const int2 a = qa[k], b = qb[k];
    if (flag(k)) {
      d[0] += sqrt((a.x - cx) * (a.x - cx) + (a.y - cy) * (a.y - cy));
      d[1] += sqrt((b.x - cu) * (b.x - cu) + (b.y - cv) * (b.y - cv));
    }
  }
  block_sums<kFinalWaves>(sRed, d);
  const double s_a = sqrt(2.0) / (d[0] / n_in);
  const double s_b = sqrt(2.0) / (d[1] / n_in);
  // moments: [0..4] x y xx xy yy (the count is n_in), [5..10] u times 1 x y xx xy yy, [11..16] v
  // times the same, [17..21] w = u^2 + v^2 times x y xx xy yy
  double S[kMoments] = {};
  for (int k = tid; k < M; k += kFinalThreads) {
    const int2 a = qa[k], b = qb[k];
    if (flag(k)) {
      const double x = s_a * (a.x - cx), y = s_a * (a.y - cy), u = s_b * (b.x - cu), v = s_b * (b.y - cv);
      const double xx = x * x, xy = x * y, yy = y * y, w = u * u + v * v;
      S[0] += x; S[1] += y; S[2] += xx; S[3] += xy; S[4] += yy;
      S[5] += u; S[6] += u * x; S[7] += u * y; S[8] += u * xx; S[9] += u * xy; S[10] += u * yy;
      S[11] += v; S[12] += v * x; S[13] += v * y; S[14] += v * xx; S[15] += v * xy; S[16] += v * yy;
      S[17] += w * x; S[18] += w * y; S[19] += w * xx; S[20] += w * xy; S[21] += w * yy;
    }
  }
  block_sums<kFinalWaves>(sRed, S);
  if (tid < 64) {                                     // wave 0 solves the normal equations
    // A^T A = [P 0 -U; 0 P -V; -U' -V' W] and A^T b, with P of (x y 1), U and V its products
    // with u (x, y), v (x, y), and W of (x y) by w
    const int r = tid >> 3, c = tid & 7;
    const double P[3][3] = {{S[2], S[3], S[0]}, {S[3], S[4], S[1]}, {S[0], S[1], n_in}};
    const double U[3][2] = {{S[8], S[9]}, {S[9], S[10]}, {S[6], S[7]}};
    const double V[3][2] = {{S[14], S[15]}, {S[15], S[16]}, {S[12], S[13]}};
    const double W[2][2] = {{S[19], S[20]}, {S[20], S[21]}};
    const double rhs[8] = {S[6], S[7], S[5], S[12], S[13], S[11], -S[17], -S[18]};
    double a = 0.0, bv = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      bv = r == i ? rhs[i] : bv;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const double e = i < 3 && j < 3 ? P[i % 3][j % 3]
                         : i >= 3 && i < 6 && j >= 3 && j < 6 ? P[i % 3][j % 3]
                         : i < 3 && j >= 6 ? -U[i % 3][j & 1] : j < 3 && i >= 6 ? -U[j % 3][i & 1]
                         : i < 6 && j >= 6 ? -V[i % 3][j & 1] : j < 6 && i >= 6 ? -V[j % 3][i & 1]
                         : i >= 6 && j >= 6 ? W[i & 1][j & 1] : 0.0;
        a = r == i && c == j ? e : a;
      }
    }
    double h = 0.0;
    if (wave_solve8(a, bv, h)) {
      // H = Tb^-1 Hn Ta with Ta = [s_a 0 -s_a cx; 0 s_a -s_a cy; 0 0 1], Tb likewise: lane 3 r + c
      // its entry (r, c), in every lane also entry (2, 2)
      double Hn[9];
#pragma unroll
      for (int i = 0; i < 8; ++i) Hn[i] = lane_of(h, i);
      Hn[8] = 1.0;
      const double ib = 1.0 / s_b;
      double HT[9];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        HT[3 * i] = Hn[3 * i] * s_a;
        HT[3 * i + 1] = Hn[3 * i + 1] * s_a;
        HT[3 * i + 2] = Hn[3 * i] * (-s_a * cx) + Hn[3 * i + 1] * (-s_a * cy) + Hn[3 * i + 2];
      }
      double e = 0.0;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        e = tid == i ? ib * HT[i] + cu * HT[6 + i] : e;
        e = tid == 3 + i ? ib * HT[3 + i] + cv * HT[6 + i] : e;
        e = tid == 6 + i ? HT[6 + i] : e;
      }
      if (tid < 9) H_out[tid] = e / HT[8];
    } else if (tid < 9) {
      H_out[tid] = Hb[tid] / Hb[8];
    }
  }
}

__global__ void __launch_bounds__(kFinalThreads) k_prosac_final(const int32_t* __restrict__ misc,
                                                       const int2* __restrict__ qa, const int2* __restrict__ qb,
                                                       const int32_t* __restrict__ qi, int cap_a, int nhyp,
                                                       const double* __restrict__ hyp_h,
                                                       const int32_t* __restrict__ hyp_ok,
                                                       const int32_t* __restrict__ hyp_counts, double eps2,
                                                       double* __restrict__ H_out, int32_t* __restrict__ inliers,
                                                       uint8_t* __restrict__ mask) {
  prosac_final_body(misc, qa, qb, qi, cap_a, nhyp, hyp_h, hyp_ok, hyp_counts, eps2, H_out, inliers, mask);
}

// Several pairs per launch of each PROSAC stage: blockIdx.y selects the pair and its
// descriptor (inputs, outputs and workspace region) from a device table.
struct ProsacPairDev {
  const int32_t* pts_a;
  const int32_t* pts_b;
  const int32_t* match;
  const int32_t* dist;
  const int32_t* count_a;
  const double* uniforms;
  int32_t* misc;
  int2* qa;
  int2* qb;
  int32_t* qi;
  int64_t* tp;
  double* hyp_h;
  int32_t* hyp_ok;
  int32_t* hyp_counts;
  double* H;
  int32_t* inliers;
  uint8_t* mask;
  int32_t cap_a, cap_b;
};

__global__ void __launch_bounds__(1024) k_prosac_prepare_multi(const PairArgs<ProsacPairDev>,
                                                                const ProsacPairDev* __restrict__ pairs, double T_N) {
  const ProsacPairDev q = pair_of(pairs, blockIdx.y);
  prosac_prepare_body(q.pts_a, q.pts_b, q.cap_b, q.match, q.dist, q.count_a, q.cap_a, T_N, q.misc, q.qa, q.qb, q.qi,
                      q.tp);
}

__global__ void __launch_bounds__(256) k_prosac_hyp_multi(const PairArgs<ProsacPairDev>,
                                                          const ProsacPairDev* __restrict__ pairs, int nhyp, double eps2) {
  const ProsacPairDev q = pair_of(pairs, blockIdx.y);
  prosac_hyp_body(q.misc, q.qa, q.qb, q.tp, nhyp, q.uniforms, eps2, q.hyp_h, q.hyp_ok, q.hyp_counts, blockIdx.x);
}

__global__ void __launch_bounds__(kFinalThreads) k_prosac_final_multi(const PairArgs<ProsacPairDev>,
                                                                      const ProsacPairDev* __restrict__ pairs, int nhyp,
                                                                      double eps2) {
  const ProsacPairDev q = pair_of(pairs, blockIdx.y);
  prosac_final_body(q.misc, q.qa, q.qb, q.qi, q.cap_a, nhyp, q.hyp_h, q.hyp_ok, q.hyp_counts, eps2, q.H, q.inliers,
                    q.mask);
}

size_t up(size_t v) { return (v + 255) & ~(size_t)255; }

ProsacWs prosac_layout(int cap_a, int nhyp, size_t* total) {
  ProsacWs L;
  size_t o = 0;
  L.misc = o; o += 256;
  L.qa = o; o += up((size_t)cap_a * 8);
  L.qb = o; o += up((size_t)cap_a * 8);
  L.qi = o; o += up((size_t)cap_a * 4);
  L.tp = o; o += up((size_t)(cap_a + 1) * 8);
  L.hyp_h = o; o += up((size_t)nhyp * 9 * 8);
  L.hyp_ok = o; o += up((size_t)nhyp * 4);
  *total = o;
  return L;
}

}  // namespace

extern "C" {

size_t stitch_lsh_match_workspace_bytes(int32_t cap_a, int32_t cap_b, int32_t tables) {
  if (cap_a < 1 || cap_b < 1 || cap_a > kMaxPoints || cap_b > kMaxPoints || tables < 1 || tables > kMaxTables)
    return 0;
  return up((size_t)tables * cap_a * 4) + up((size_t)tables * cap_b * 4);
}

stitch_status stitch_lsh_match(int32_t nd, const uint32_t* desc_a, const int32_t* count_a, int32_t cap_a,
                               const uint32_t* desc_b, const int32_t* count_b, int32_t cap_b, int32_t tables,
                               int32_t kbits, const int32_t* positions, int32_t max_dist, int32_t* match,
                               int32_t* dist, void* workspace, size_t workspace_bytes, void* stream) {
  if (!desc_a || !count_a || !desc_b || !count_b || !match || !dist || (kbits > 0 && !positions))
    return fail(STITCH_E_NULL, "a descriptor, count, output or the positions is NULL");
  if (nd < 32 || nd > 512 || nd % 32) return fail(STITCH_E_SHAPE, "nd = %d is not a multiple of 32 in 32..512", nd);
  if (cap_a < 1 || cap_b < 1 || cap_a > kMaxPoints || cap_b > kMaxPoints)
    return fail(STITCH_E_SHAPE, "capacities must lie in 1..%d", kMaxPoints);
  if (tables < 1 || tables > kMaxTables || kbits < 0 || kbits > kMaxKeyBits)
    return fail(STITCH_E_SHAPE, "tables in 1..%d and key bits in 0..%d", kMaxTables, kMaxKeyBits);
  if ((uintptr_t)desc_a & 7 || (uintptr_t)desc_b & 7)
    return fail(STITCH_E_SHAPE, "descriptors must be 8-byte aligned");
  LshParams P{};
  P.tables = tables;
  P.kbits = kbits;
  P.words = nd / 32;
  for (int l = 0; l < tables; ++l)
    for (int b = 0; b < kbits; ++b) {
      const int p = positions[l * kbits + b];
      if (p < 0 || p >= nd) return fail(STITCH_E_SHAPE, "bit position %d outside 0..%d", p, nd - 1);
      P.pos[l][b] = (int16_t)p;
    }
  const size_t need = stitch_lsh_match_workspace_bytes(cap_a, cap_b, tables);
  if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255))
    return fail(STITCH_E_WORKSPACE, "workspace missing, misaligned or smaller than %zu bytes", need);
  uint32_t* keys_a = (uint32_t*)workspace;
  uint32_t* keys_b = (uint32_t*)((uint8_t*)workspace + up((size_t)tables * cap_a * 4));
  const hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_lsh_keys, dim3((cap_a + 255) / 256), dim3(256), 0, s, desc_a, count_a, cap_a, P, keys_a);
  hipLaunchKernelGGL(k_lsh_keys, dim3((cap_b + 255) / 256), dim3(256), 0, s, desc_b, count_b, cap_b, P, keys_b);
  hipLaunchKernelGGL(k_lsh_match, dim3((cap_a + 3) / 4), dim3(256), 0, s, desc_a, count_a, cap_a, desc_b, count_b,
                     cap_b, P, keys_a, keys_b, max_dist, match, dist);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "matching launch");
  return STITCH_OK;
}

size_t stitch_lsh_match_multi_workspace_bytes(int32_t npairs, const stitch_match_pair* pairs, int32_t tables) {
  if (npairs < 1 || npairs > kMaxPairs || !pairs) return 0;
  size_t total = up((size_t)npairs * sizeof(LshPairDev));
  for (int p = 0; p < npairs; ++p) {
    const size_t one = stitch_lsh_match_workspace_bytes(pairs[p].cap_a, pairs[p].cap_b, tables);
    if (!one) return 0;
    total += one;
  }
  return total;
}

stitch_status stitch_lsh_match_multi(int32_t npairs, const stitch_match_pair* pairs, int32_t nd, int32_t tables,
                                     int32_t kbits, const int32_t* positions, int32_t max_dist, void* workspace,
                                     size_t workspace_bytes, void* stream) {
  if (!pairs || (kbits > 0 && !positions)) return fail(STITCH_E_NULL, "pairs or the positions is NULL");
  if (npairs < 1 || npairs > kMaxPairs) return fail(STITCH_E_SHAPE, "npairs = %d outside 1..%d", npairs, kMaxPairs);
  if (nd < 32 || nd > 512 || nd % 32) return fail(STITCH_E_SHAPE, "nd = %d is not a multiple of 32 in 32..512", nd);
  if (tables < 1 || tables > kMaxTables || kbits < 0 || kbits > kMaxKeyBits)
    return fail(STITCH_E_SHAPE, "tables in 1..%d and key bits in 0..%d", kMaxTables, kMaxKeyBits);
  LshParams P{};
  P.tables = tables;
  P.kbits = kbits;
  P.words = nd / 32;
  for (int l = 0; l < tables; ++l)
    for (int b = 0; b < kbits; ++b) {
      const int q = positions[l * kbits + b];
      if (q < 0 || q >= nd) return fail(STITCH_E_SHAPE, "bit position %d outside 0..%d", q, nd - 1);
      P.pos[l][b] = (int16_t)q;
    }
  for (int p = 0; p < npairs; ++p) {
    const stitch_match_pair& m = pairs[p];
    if (!m.desc_a || !m.count_a || !m.desc_b || !m.count_b || !m.match || !m.dist)
      return fail(STITCH_E_NULL, "pair %d: a descriptor, count or output is NULL", p);
    if (m.cap_a < 1 || m.cap_b < 1 || m.cap_a > kMaxPoints || m.cap_b > kMaxPoints)
      return fail(STITCH_E_SHAPE, "pair %d: capacities must lie in 1..%d", p, kMaxPoints);
    if ((uintptr_t)m.desc_a & 7 || (uintptr_t)m.desc_b & 7)
      return fail(STITCH_E_SHAPE, "pair %d: descriptors must be 8-byte aligned", p);
  }
  const size_t need = stitch_lsh_match_multi_workspace_bytes(npairs, pairs, tables);
  if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255))
    return fail(STITCH_E_WORKSPACE, "workspace missing, misaligned or smaller than %zu bytes", need);
  int cap_max = 1, capa_max = 1;
  std::vector<LshPairDev> tab((size_t)npairs);
  uint8_t* ws = (uint8_t*)workspace;
  size_t o = up((size_t)npairs * sizeof(LshPairDev));
  for (int p = 0; p < npairs; ++p) {
    const stitch_match_pair& m = pairs[p];
    LshPairDev& d = tab[p];
    d.desc_a = m.desc_a; d.count_a = m.count_a; d.cap_a = m.cap_a;
    d.desc_b = m.desc_b; d.count_b = m.count_b; d.cap_b = m.cap_b;
    d.match = m.match; d.dist = m.dist;
    d.keys_a = (uint32_t*)(ws + o); o += up((size_t)tables * m.cap_a * 4);
    d.keys_b = (uint32_t*)(ws + o); o += up((size_t)tables * m.cap_b * 4);
    cap_max = std::max(cap_max, std::max(m.cap_a, m.cap_b));
    capa_max = std::max(capa_max, m.cap_a);
  }
  const hipStream_t s = (hipStream_t)stream;
  PairArgs<LshPairDev> args{};
  const LshPairDev* dev = nullptr;
  hipError_t e = hipSuccess;
  if (npairs <= kArgPairs) {
    for (int p = 0; p < npairs; ++p) args.p[p] = tab[p];
  } else {
    e = hipMemcpyAsync(workspace, tab.data(), tab.size() * sizeof(LshPairDev), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "matching table upload");
    dev = (const LshPairDev*)workspace;
  }
  hipLaunchKernelGGL(k_lsh_keys_multi, dim3((cap_max + 255) / 256, 2 * npairs), dim3(256), 0, s, args, dev, P);
  hipLaunchKernelGGL(k_lsh_match_multi, dim3((capa_max + 3) / 4, npairs), dim3(256), 0, s, args, dev, P, max_dist);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "matching launch");
  return STITCH_OK;
}

size_t stitch_prosac_workspace_bytes(int32_t cap_a, int32_t nhyp) {
  if (cap_a < 1 || cap_a > kMaxPoints || nhyp < 1 || nhyp > kMaxHyp) return 0;
  size_t total = 0;
  prosac_layout(cap_a, nhyp, &total);
  return total;
}

}  // extern "C"

namespace {

// Scratch of the allocation-free PROSAC entry point: one array per device that runs it,
// held until the process ends.  Host code never passes `scratch` itself to a kernel (on the
// host it only names the symbol); it passes the device address from hipGetSymbolAddress.
constexpr size_t kProsacScratchBytes = (size_t)1 << 20;
constexpr int kMaxDevices = 64;
__device__ __align__(256) uint8_t scratch[kProsacScratchBytes];
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's copy of the scratch array (its address is looked up once per device,
// with that device current).
stitch_status prosac_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "current device");
  if (dev < 0 || dev >= kMaxDevices) return fail(STITCH_E_DEVICE, "device %d outside 0..%d", dev, kMaxDevices - 1);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol, "scratch address");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return STITCH_OK;
}

stitch_status prosac_run(const int32_t* pts_a, const int32_t* pts_b, int32_t cap_b, const int32_t* match,
                         const int32_t* dist, const int32_t* count_a, int32_t cap_a, int32_t nhyp,
                         const double* uniforms, double T_N, double eps, double* H, int32_t* inliers,
                         uint8_t* inlier_mask, int32_t* hyp_counts, void* workspace, size_t workspace_bytes,
                         void* stream, bool own_scratch);

}  // namespace

extern "C" {

stitch_status stitch_prosac(const int32_t* pts_a, const int32_t* pts_b, int32_t cap_b, const int32_t* match,
                            const int32_t* dist, const int32_t* count_a, int32_t cap_a, int32_t nhyp,
                            const double* uniforms, double T_N, double eps, double* H, int32_t* inliers,
                            uint8_t* inlier_mask, int32_t* hyp_counts, void* workspace, size_t workspace_bytes,
                            void* stream) {
  return prosac_run(pts_a, pts_b, cap_b, match, dist, count_a, cap_a, nhyp, uniforms, T_N, eps, H, inliers,
                    inlier_mask, hyp_counts, workspace, workspace_bytes, stream, false);
}

stitch_status stitch_prosac_noalloc(const int32_t* pts_a, const int32_t* pts_b, int32_t cap_b, const int32_t* match,
                                    const int32_t* dist, const int32_t* count_a, int32_t cap_a, int32_t nhyp,
                                    const double* uniforms, double T_N, double eps, double* H, int32_t* inliers,
                                    uint8_t* inlier_mask, int32_t* hyp_counts, void* stream) {
  return prosac_run(pts_a, pts_b, cap_b, match, dist, count_a, cap_a, nhyp, uniforms, T_N, eps, H, inliers,
                    inlier_mask, hyp_counts, nullptr, 0, stream, true);
}

}  // extern "C"

namespace {

stitch_status prosac_run(const int32_t* pts_a, const int32_t* pts_b, int32_t cap_b, const int32_t* match,
                         const int32_t* dist, const int32_t* count_a, int32_t cap_a, int32_t nhyp,
                         const double* uniforms, double T_N, double eps, double* H, int32_t* inliers,
                         uint8_t* inlier_mask, int32_t* hyp_counts, void* workspace, size_t workspace_bytes,
                         void* stream, bool own_scratch) {
  if (!pts_a || !pts_b || !match || !dist || !count_a || !uniforms || !H || !inliers || !inlier_mask || !hyp_counts)
    return fail(STITCH_E_NULL, "an input or output is NULL");
  if (cap_a < 1 || cap_a > kMaxPoints || cap_b < 1 || cap_b > kMaxPoints)
    return fail(STITCH_E_SHAPE, "capacities must lie in 1..%d", kMaxPoints);
  if (nhyp < 1 || nhyp > kMaxHyp) return fail(STITCH_E_SHAPE, "nhyp = %d outside 1..%d", nhyp, kMaxHyp);
  if (!(T_N > 0.0) || !std::isfinite(T_N) || !(eps > 0.0) || !std::isfinite(eps))
    return fail(STITCH_E_SHAPE, "T_N and eps must be positive and finite");
  // the schedule T'_n grows to about T_N + M and is kept in int64: T_N up to 2^53 (where
  // every integer is still a double) leaves it far inside the range
  if (T_N > 0x1p53)
    return fail(STITCH_E_SHAPE, "T_N = %g exceeds 2^53", T_N);
  size_t need = 0;
  const ProsacWs L = prosac_layout(cap_a, nhyp, &need);
  if (own_scratch) {
    if (need > kProsacScratchBytes)
      return fail(STITCH_E_SHAPE, "cap_a = %d and nhyp = %d need %zu bytes of scratch; the allocation-free call "
                  "holds %zu", cap_a, nhyp, need, kProsacScratchBytes);
    const stitch_status st = prosac_scratch(&workspace);
    if (st) return st;
    workspace_bytes = kProsacScratchBytes;
  }
  if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255))
    return fail(STITCH_E_WORKSPACE, "workspace missing, misaligned or smaller than %zu bytes", need);
  uint8_t* ws = (uint8_t*)workspace;
  int32_t* misc = (int32_t*)(ws + L.misc);
  int2* qa = (int2*)(ws + L.qa);
  int2* qb = (int2*)(ws + L.qb);
  int32_t* qi = (int32_t*)(ws + L.qi);
  int64_t* tp = (int64_t*)(ws + L.tp);
  double* hyp_h = (double*)(ws + L.hyp_h);
  int32_t* hyp_ok = (int32_t*)(ws + L.hyp_ok);
  const double eps2 = eps * eps;
  const hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_prosac_prepare, dim3(1), dim3(1024), 0, s, pts_a, pts_b, cap_b, match, dist, count_a, cap_a,
                     T_N, misc, qa, qb, qi, tp);
  hipLaunchKernelGGL(k_prosac_hyp, dim3((nhyp + 3) / 4), dim3(256), 0, s, misc, qa, qb, tp, nhyp, uniforms, eps2,
                     hyp_h, hyp_ok, hyp_counts);
  hipLaunchKernelGGL(k_prosac_final, dim3(1), dim3(kFinalThreads), 0, s, misc, qa, qb, qi, cap_a, nhyp, hyp_h, hyp_ok,
                     hyp_counts, eps2, H, inliers, inlier_mask);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "PROSAC launch");
  return STITCH_OK;
}

}  // namespace

namespace {

size_t prosac_multi_bytes(int32_t npairs, const stitch_prosac_pair* pairs, int32_t nhyp) {
  if (npairs < 1 || npairs > kMaxPairs || !pairs || nhyp < 1 || nhyp > kMaxHyp) return 0;
  size_t total = up((size_t)npairs * sizeof(ProsacPairDev));
  for (int p = 0; p < npairs; ++p) {
    if (pairs[p].cap_a < 1 || pairs[p].cap_a > kMaxPoints) return 0;
    size_t one = 0;
    prosac_layout(pairs[p].cap_a, nhyp, &one);
    total += one;
  }
  return total;
}

}  // namespace

extern "C" {

size_t stitch_prosac_multi_workspace_bytes(int32_t npairs, const stitch_prosac_pair* pairs, int32_t nhyp) {
  return prosac_multi_bytes(npairs, pairs, nhyp);
}

stitch_status stitch_prosac_multi(int32_t npairs, const stitch_prosac_pair* pairs, int32_t nhyp, double T_N,
                                  double eps, void* workspace, size_t workspace_bytes, void* stream) {
  if (!pairs) return fail(STITCH_E_NULL, "pairs is NULL");
  if (npairs < 1 || npairs > kMaxPairs) return fail(STITCH_E_SHAPE, "npairs = %d outside 1..%d", npairs, kMaxPairs);
  if (nhyp < 1 || nhyp > kMaxHyp) return fail(STITCH_E_SHAPE, "nhyp = %d outside 1..%d", nhyp, kMaxHyp);
  if (!(T_N > 0.0) || !std::isfinite(T_N) || !(eps > 0.0) || !std::isfinite(eps))
    return fail(STITCH_E_SHAPE, "T_N and eps must be positive and finite");
  if (T_N > 0x1p53) return fail(STITCH_E_SHAPE, "T_N = %g exceeds 2^53", T_N);
  for (int p = 0; p < npairs; ++p) {
    const stitch_prosac_pair& m = pairs[p];
    if (!m.pts_a || !m.pts_b || !m.match || !m.dist || !m.count_a || !m.uniforms || !m.H || !m.inliers ||
        !m.inlier_mask || !m.hyp_counts)
      return fail(STITCH_E_NULL, "pair %d: an input or output is NULL", p);
    if (m.cap_a < 1 || m.cap_a > kMaxPoints || m.cap_b < 1 || m.cap_b > kMaxPoints)
      return fail(STITCH_E_SHAPE, "pair %d: capacities must lie in 1..%d", p, kMaxPoints);
  }
  const size_t need = prosac_multi_bytes(npairs, pairs, nhyp);
  if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255))
    return fail(STITCH_E_WORKSPACE, "workspace missing, misaligned or smaller than %zu bytes", need);
  std::vector<ProsacPairDev> tab((size_t)npairs);
  uint8_t* ws = (uint8_t*)workspace;
  size_t o = up((size_t)npairs * sizeof(ProsacPairDev));
  for (int p = 0; p < npairs; ++p) {
    const stitch_prosac_pair& m = pairs[p];
    size_t one = 0;
    const ProsacWs L = prosac_layout(m.cap_a, nhyp, &one);
    ProsacPairDev& d = tab[p];
    d.pts_a = m.pts_a; d.pts_b = m.pts_b; d.match = m.match; d.dist = m.dist; d.count_a = m.count_a;
    d.uniforms = m.uniforms; d.cap_a = m.cap_a; d.cap_b = m.cap_b;
    d.misc = (int32_t*)(ws + o + L.misc);
    d.qa = (int2*)(ws + o + L.qa);
    d.qb = (int2*)(ws + o + L.qb);
    d.qi = (int32_t*)(ws + o + L.qi);
    d.tp = (int64_t*)(ws + o + L.tp);
    d.hyp_h = (double*)(ws + o + L.hyp_h);
    d.hyp_ok = (int32_t*)(ws + o + L.hyp_ok);
    d.hyp_counts = m.hyp_counts; d.H = m.H; d.inliers = m.inliers; d.mask = m.inlier_mask;
    o += one;
  }
  const double eps2 = eps * eps;
  const hipStream_t s = (hipStream_t)stream;
  PairArgs<ProsacPairDev> args{};
  const ProsacPairDev* dev = nullptr;
  hipError_t e = hipSuccess;
  if (npairs <= kArgPairs) {
    for (int p = 0; p < npairs; ++p) args.p[p] = tab[p];
  } else {
    e = hipMemcpyAsync(workspace, tab.data(), tab.size() * sizeof(ProsacPairDev), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "PROSAC table upload");
    dev = (const ProsacPairDev*)workspace;
  }
  hipLaunchKernelGGL(k_prosac_prepare_multi, dim3(1, npairs), dim3(1024), 0, s, args, dev, T_N);
  hipLaunchKernelGGL(k_prosac_hyp_multi, dim3((nhyp + 3) / 4, npairs), dim3(256), 0, s, args, dev, nhyp, eps2);
  hipLaunchKernelGGL(k_prosac_final_multi, dim3(1, npairs), dim3(kFinalThreads), 0, s, args, dev, nhyp, eps2);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "PROSAC launch");
  return STITCH_OK;
}

}  // extern "C"
