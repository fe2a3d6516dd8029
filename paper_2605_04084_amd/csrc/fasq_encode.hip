// Calibration-free PQ encoding (FASQ Sec. 3.1.1, Alg. 1): Lloyd's k-means over
// the sub-vectors of a weight matrix, with one codebook shared by every
// subspace (the format the matmul kernels consume).
//
// Definition (the paper leaves these details open):
//   * point p = n * (K / d) + s is w[n, s*d : (s+1)*d]; W is [N x K] row-major,
//     so the points are P = N * K / d consecutive runs of d fp16 values;
//   * assignment: squared Euclidean distance evaluated in fp32 as
//     acc = 0; acc = acc + (w_i - c_i) * (w_i - c_i), i = 0 .. d-1, every
//     operation rounded separately (no fused multiply-add); the lowest index
//     wins a tie;
//   * update: the cluster sum is exact (an fp16 value times 2^24 is an
//     integer; |w| < 128 keeps the sums inside 64 bits), then
//     mean = (fp64(sum) * 2^-24) / fp64(count), rounded to fp16 (nearest,
//     ties to even); an empty cluster keeps its codeword;
//   * iters updates, then a last assignment against the final codebook gives
//     the ids, packed in the library's id format.
// Exact integer sums make the result independent of the order in which the
// atomics land: the encoder is deterministic.
#include <type_traits>

#include "fasq_device.h"
#include "fasq_internal.h"

namespace fasq {

namespace {

constexpr int kEncThreads = 512;                     // 8 waves
constexpr int kEncWaves = kEncThreads / kWave;
constexpr int kEncSuper = 64;                        // codewords per superblock (two MFMA tiles)
constexpr int kEncTileBytes = 64 * 1024;             // codewords and norms in LDS (two workgroups per CU)
constexpr int kEncDirectThreads = 256;
constexpr int kEncDirectPoints = 4;
constexpr int kEncDirectMax = 64;                    // codewords up to which every distance is evaluated
constexpr int kEncFineMax = 512;                     // codewords up to which the MFMA kernel keeps blocks of 8
constexpr int kEncWholeGroups = 3;                   // groups of points after one with many open points that skip the minima
constexpr int kEncBlock = 8;                         // codewords per block where every distance is evaluated
constexpr int kEncUpdateThreads = 256;               // at least the largest d
constexpr int kEncSumThreads = 1024;
constexpr int kEncSumBytes = 150 * 1024;             // LDS for the cluster sums of a workgroup
constexpr int kEncSumMaxRanges = 8;                  // passes over the points the tables are worth
constexpr float kQScale = 16777216.0f;               // 2^24
constexpr double kQInv = 1.0 / 16777216.0;

// fp64 -> fp16, round to nearest, ties to even, by integer operations on the
// fp64 encoding (one rounding step; inputs are finite).
__device__ __forceinline__ uint16_t f64_to_f16_rne(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint16_t sign = (uint16_t)((b >> 48) & 0x8000u);
  const int ex = (int)((b >> 52) & 0x7FF);
  if (ex == 0) return sign;  // zero or an fp64 subnormal: far below half the smallest fp16
  const uint64_t m = (b & ((uint64_t(1) << 52) - 1)) | (uint64_t(1) << 52);  // 53-bit significand
  const int e = ex - 1023;  // v = m * 2^(e - 52)
  if (e > 15) return sign | 0x7C00u;
  int shift;  // bits of m below the fp16 result's last place
  if (e >= -14) shift = 42;            // normal: 11 significant bits kept
  else if (e >= -25) shift = 28 - e;   // subnormal: result in units of 2^-24
  else return sign;                    // below 2^-25: rounds to zero
  const uint64_t q = m >> shift;
  const uint64_t rem = m & ((uint64_t(1) << shift) - 1);
  const uint64_t half = uint64_t(1) << (shift - 1);
  uint32_t r = (uint32_t)q + ((rem > half || (rem == half && (q & 1))) ? 1u : 0u);
  if (e >= -14) {
    // r in [2^10, 2^11]; a carry to 2^11 moves up one binade
    int ee = e + 15;
    if (r == 0x800u) { r = 0x400u; ++ee; }
    if (ee >= 31) return sign | 0x7C00u;
    return sign | (uint16_t)(ee << 10) | (uint16_t)(r & 0x3FFu);
  }
  // subnormal result r * 2^-24, r <= 2^10 (2^10 is the smallest normal, exponent field 1)
  return sign | (uint16_t)r;
}

__global__ void k_enc_copy(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

__global__ void k_enc_zero(int64_t* __restrict__ p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// Squared distance in fp32, operations in the defined order, no contraction.
// The padding of both vectors is zero: it adds +0 to a sum that is never -0,
// so the bits are those of the d real components.
template <int DP>
__device__ __forceinline__ float sq_dist(const float* p, const float* c) {
#pragma clang fp contract(off)
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < DP; ++i) {
    const float diff = p[i] - c[i];
    acc = acc + diff * diff;
  }
  return acc;
}

// The same with the codeword in fp16.  From four components on p_i - c_i is an
// fma by minus one (the same bits), which takes a half operand as it is
// (v_fma_mix): 2048 x 2048, d = 4, C = 4096, every distance 2.86 -> 2.75 ms;
// d = 2, C = 256 0.24 -> 0.27 ms.
template <int D>
__device__ __forceinline__ float sq_dist_half(const float* p, const half_t* c, float minus_one) {
#pragma clang fp contract(off)
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const float ci = static_cast<float>(c[i]);
    const float diff = D >= 4 ? __builtin_fmaf(ci, minus_one, p[i]) : p[i] - ci;
    acc = i == 0 ? diff * diff : acc + diff * diff;
  }
  return acc;
}

// Codewords in LDS: DP halves each (d padded with zeros), 64 to a superblock,
// and one unused read's worth after each superblock, so that lanes that read
// the same place of different superblocks spread over the banks.
template <int DP>
struct EncTile {
  static constexpr int CW = DP * 2;                                   // bytes per codeword
  static constexpr int SB = kEncSuper * CW + (CW < 16 ? CW : 16);     // bytes per superblock
  static constexpr int PER = SB + kEncSuper * 4;                      // with its norms
  static constexpr int MAX = kEncTileBytes / PER * kEncSuper;         // codewords per tile
  __device__ static uint32_t at(int k) { return (uint32_t)(k / kEncSuper) * SB + (uint32_t)(k % kEncSuper) * CW; }
};

template <int DP>
__device__ __forceinline__ void lds_codeword(const uint8_t* tile, int k, float* c) {
  const uint8_t* q = tile + EncTile<DP>::at(k);
  half_t v[DP];
  if constexpr (DP == 2) *reinterpret_cast<uint32_t*>(v) = *reinterpret_cast<const uint32_t*>(q);
  else if constexpr (DP == 4) *reinterpret_cast<u32x2*>(v) = *reinterpret_cast<const u32x2*>(q);
  else {
#pragma unroll
    for (int j = 0; j < DP / 8; ++j) reinterpret_cast<u32x4*>(v)[j] = reinterpret_cast<const u32x4*>(q)[j];
  }
#pragma unroll
  for (int i = 0; i < DP; ++i) c[i] = static_cast<float>(v[i]);
}

template <int DP>
__device__ __forceinline__ void global_vector(const half_t* __restrict__ src, int64_t k, int d, float* c) {
  if (d == DP) {  // one wide load
#pragma unroll
    for (int i = 0; i < DP; ++i) c[i] = static_cast<float>(src[k * DP + i]);
  } else {
#pragma unroll
    for (int i = 0; i < DP; ++i) c[i] = i < d ? static_cast<float>(src[k * d + i]) : 0.f;
  }
}

// Vector k of d halves, padded with zeros.
template <int DP>
__device__ __forceinline__ void half_vector(const half_t* __restrict__ src, int64_t k, int d, half_t* v) {
  if (d == DP) {  // one wide load, at any alignment
    __builtin_memcpy(v, src + k * DP, DP * 2);
  } else {
#pragma unroll
    for (int i = 0; i < DP; ++i) v[i] = i < d ? src[k * d + i] : static_cast<half_t>(0.f);
  }
}

// Assignment of every point to its nearest codeword, every distance
// evaluated: for codebooks up to kEncDirectMax, where the fixed work of the
// MFMA kernel per tile of points exceeds it.  One thread takes
// kEncDirectPoints points; the codebook is fp32 in LDS, read by broadcast.
// With ACCUM the cluster sums and counts gather in an LDS table on the way.
template <int DP, bool ACCUM>
__global__ __launch_bounds__(kEncDirectThreads) void k_enc_direct(const half_t* __restrict__ w, int64_t P, int d,
                                                                  const half_t* __restrict__ cb, int C,
                                                                  uint32_t* __restrict__ assign,
                                                                  unsigned long long* __restrict__ sums,
                                                                  unsigned long long* __restrict__ counts) {
  constexpr int PPT = kEncDirectPoints;
  __shared__ float tile[kEncDirectMax * DP];
  __shared__ unsigned long long agg[ACCUM ? kEncDirectMax * (DP + 1) : 1];  // [C][d + 1] sums, count
  if constexpr (ACCUM) {
    for (int i = threadIdx.x; i < C * (d + 1); i += blockDim.x) agg[i] = 0;
  }
  for (int i = threadIdx.x; i < C * DP; i += blockDim.x)
    tile[i] = i % DP < d ? static_cast<float>(cb[(int64_t)(i / DP) * d + i % DP]) : 0.f;
  __syncthreads();
  const int64_t group = (int64_t)kEncDirectThreads * PPT;
  for (int64_t g0 = blockIdx.x * group; g0 < P; g0 += (int64_t)gridDim.x * group) {
    float pv[PPT][DP];
    float best[PPT];
    uint32_t bk[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      const int64_t p = g0 + (int64_t)j * kEncDirectThreads + threadIdx.x;
      global_vector<DP>(w, p < P ? p : P - 1, d, pv[j]);
      best[j] = __builtin_inff();
      bk[j] = 0;
    }
#pragma unroll 4
    for (int k = 0; k < C; ++k) {
#pragma unroll
      for (int j = 0; j < PPT; ++j) {
        const float dist = sq_dist<DP>(pv[j], tile + k * DP);
        if (dist < best[j]) {  // strict: the lowest index keeps a tie
          best[j] = dist;
          bk[j] = (uint32_t)k;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      const int64_t p = g0 + (int64_t)j * kEncDirectThreads + threadIdx.x;
      if (p >= P) continue;
      assign[p] = bk[j];
      if constexpr (ACCUM) {
        unsigned long long* t = agg + bk[j] * (d + 1);
#pragma unroll
        for (int i = 0; i < DP; ++i)
          if (i < d) atomicAdd(t + i, (unsigned long long)(int64_t)(pv[j][i] * kQScale));  // exact
        atomicAdd(t + d, 1ull);
      }
    }
  }
  if constexpr (ACCUM) {
    __syncthreads();
    for (int i = threadIdx.x; i < C * (d + 1); i += blockDim.x) {
      const int k = i / (d + 1), c = i - k * (d + 1);
      if (agg[i] != 0) atomicAdd(c < d ? &sums[k * d + c] : &counts[k], agg[i]);
    }
  }
}

// FN tiles of enc_every_distance, with the codebook in LDS at address 0 (LDS)
// or in global memory.  DE: components that count.
template <int DP, int FN, bool LDS, int DE>
__device__ __forceinline__ void enc_every_pass(const half_t* __restrict__ w, int64_t P, int d,
                                               const half_t* __restrict__ cb, int C, uint32_t* __restrict__ assign,
                                               int64_t p0) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x % kWave, h = lane >> 5, col = lane & 31;
  const float inf = __builtin_inff();
  float minus_one = -1.f;
  asm volatile("" : "+v"(minus_one));
  auto codeword = [&](int k, half_t* c) {
    if constexpr (LDS) __builtin_memcpy(c, smem + EncTile<DP>::at(k), DP * 2);
    else half_vector<DP>(cb, k, d, c);
  };
  float pv[FN][DP], best[FN];
  int blk[FN];
#pragma unroll
  for (int f = 0; f < FN; ++f) {
    const int64_t p = p0 + f * 32 + col;
    global_vector<DP>(w, p < P ? p : P - 1, d, pv[f]);
    best[f] = inf;
    blk[f] = 0;
  }
  auto block = [&](int k, bool tail) {
    float v[FN];
#pragma unroll
    for (int j = 0; j < kEncBlock; j += 2) {
      half_t c0[DP], c1[DP];
      codeword(!tail || k + j < C ? k + j : C - 1, c0);
      codeword(!tail || k + j + 1 < C ? k + j + 1 : C - 1, c1);
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        const float s0 = sq_dist_half<DE>(pv[f], c0, minus_one), s1 = sq_dist_half<DE>(pv[f], c1, minus_one);
        v[f] = j == 0 ? __builtin_fminf(s0, s1) : __builtin_fminf(__builtin_fminf(v[f], s0), s1);
      }
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      // strict: the lowest block keeps a tie; selects, since the minimum of
      // a block of NaN distances is a NaN and must leave the best as it is
      const bool less = v[f] < best[f];
      blk[f] = less ? k : blk[f];
      best[f] = less ? v[f] : best[f];
    }
  };
  int k = kEncBlock * h;
  for (; k + kEncBlock <= C; k += 2 * kEncBlock) block(k, false);
  if (k < C) block(k, true);
#pragma unroll
  for (int f = 0; f < FN; ++f) {
    uint32_t bk = 0;
    for (int j = kEncBlock - 1; j >= 0; --j) {
      const int kk = blk[f] + j < C ? blk[f] + j : C - 1;
      half_t c[DP];
      codeword(kk, c);
      if (best[f] < inf && sq_dist_half<DE>(pv[f], c, minus_one) == best[f]) bk = (uint32_t)kk;
    }
    const float ob = __shfl_xor(best[f], 32, kWave);
    const uint32_t ok = (uint32_t)__shfl_xor((int)bk, 32, kWave);
    if (ob < best[f] || (ob == best[f] && ok < bk)) bk = ok;
    const int64_t p = p0 + f * 32 + col;
    if (p < P && h == 0) assign[p] = bk;
  }
}

// Every distance of the wave's FN tiles of 32 points from p0 on, where the
// minima of k_enc_assign leave many of them open (repeated codewords, weights
// with a large common offset, many codewords for d = 1).  A lane takes its
// point of each tile and the blocks of kEncBlock codewords of its half: one
// codeword read serves FN points, a block's minimum takes one v_min3 for two
// distances, and the codeword is looked for in the smallest block at the end.
// Bound by vector issue (12 to 13 instructions a pair at d = 4, 7 at d = 2).
// One assignment and update of such points, with each point's codebook walked
// by its own two lanes / this: 2048 x 2048, d = 2, C = 256, offset 0.5 758 / 251
// us, half of the sub-vectors pruned 756 / 257; 1024 x 1024, d = 1, C = 1024
// 605 / 252, half pruned 800 / 226; d = 4, C = 65536, 512 x 2048, offset 31.4 /
// 16.8 ms; 2048 x 2048, d = 4, C = 4096, offset 3.74 / 2.74 ms.  (A function of
// its own: its registers are not the matrix-core loop's.)
template <int DP, int FN, bool ONE>
__device__ __attribute__((noinline)) void enc_every_distance(const half_t* __restrict__ w, int64_t P, int d,
                                                             const half_t* __restrict__ cb, int C,
                                                             uint32_t* __restrict__ assign, int64_t p0, bool bad) {
  constexpr int NF = DP >= 8 && FN > 2 ? 2 : FN;  // tiles at a time (registers)
  for (int f = 0; f < FN; f += NF) {
    const int64_t pf = p0 + f * 32;
    if (ONE && !bad) {
      if (DP == 2 && d == 1) enc_every_pass<DP, NF, ONE, 1>(w, P, d, cb, C, assign, pf);
      else enc_every_pass<DP, NF, ONE, DP>(w, P, d, cb, C, assign, pf);
    } else {
      if (DP == 2 && d == 1) enc_every_pass<DP, NF, false, 1>(w, P, d, cb, C, assign, pf);
      else enc_every_pass<DP, NF, false, DP>(w, P, d, cb, C, assign, pf);
    }
  }
}

// NP of a wave's open points (bits of lo and hi, which lose them; where fewer
// are left the last one is repeated), the codewords dealt to the lanes.
template <int DP, bool ONE, int NP>
__device__ __forceinline__ void enc_open_batch(const half_t* __restrict__ w, int d, const half_t* __restrict__ cb,
                                               int C, uint32_t* __restrict__ assign, int64_t p0, bool bad,
                                               uint64_t& lo, uint64_t& hi) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x % kWave;
  int q[NP];
  float pv[NP][DP], best[NP];
  uint32_t bk[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    if (lo) {
      q[j] = __ffsll((unsigned long long)lo) - 1;
      lo &= lo - 1;
    } else if (hi) {
      q[j] = __ffsll((unsigned long long)hi) + 63;
      hi &= hi - 1;
    } else {
      q[j] = q[j > 0 ? j - 1 : 0];
    }
    global_vector<DP>(w, p0 + q[j], d, pv[j]);
#pragma unroll
    for (int i = 0; i < DP; ++i)  // alike in all lanes: scalar registers
      pv[j][i] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, pv[j][i])));
    best[j] = __builtin_inff();
    bk[j] = 0;
  }
  auto scan = [&](auto lds) {
    for (int k = lane; k < C; k += kWave) {
      float c[DP];
      if constexpr (decltype(lds)::value) lds_codeword<DP>(smem, k, c);
      else global_vector<DP>(cb, k, d, c);
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const float dist = sq_dist<DP>(pv[j], c);
        bk[j] = dist < best[j] ? (uint32_t)k : bk[j];  // strict: the lowest index keeps a tie
        best[j] = dist < best[j] ? dist : best[j];
      }
    }
  };
  if (ONE && !bad) scan(std::integral_constant<bool, ONE>{});
  else scan(std::false_type{});
  auto merge = [&](float& b, uint32_t& k, float give_b, uint32_t give_k, int m) {
    const float ob = __shfl_xor(give_b, m, kWave);
    const uint32_t ok = (uint32_t)__shfl_xor((int)give_k, m, kWave);
    const bool take = ob < b || (ob == b && ok < k);
    b = take ? ob : b;
    k = take ? ok : k;
  };
  // each step halves the points a lane keeps, then the lanes of its one
#pragma unroll
  for (int m = kWave / 2, n = NP / 2; m > 0; m /= 2, n /= 2) {
    if (n == 0) {
      merge(best[0], bk[0], best[0], bk[0], m);
    } else {
      const bool up = lane & m;
#pragma unroll
      for (int j = 0; j < n; ++j) {
        const float gb = up ? best[j] : best[j + n];
        const uint32_t gk = up ? bk[j] : bk[j + n];
        best[j] = up ? best[j + n] : best[j];
        bk[j] = up ? bk[j + n] : bk[j];
        merge(best[j], bk[j], gb, gk, m);
      }
    }
  }
  int mine = q[0];  // (a repeated point is written alike)
#pragma unroll
  for (int j = 1; j < NP; ++j) mine = lane / (kWave / NP) == j ? q[j] : mine;
  if (lane % (kWave / NP) == 0) assign[p0 + mine] = bk[0];
}

// The few open points of a wave's tiles (one bit each): four share a codeword
// read, the last one or two take it alone.
template <int DP, bool ONE>
__device__ __attribute__((noinline)) void enc_open_points(const half_t* __restrict__ w, int d,
                                                          const half_t* __restrict__ cb, int C,
                                                          uint32_t* __restrict__ assign, int64_t p0, bool bad,
                                                          uint64_t lo, uint64_t hi) {
  while (lo | hi) {
    if (__popcll(lo) + __popcll(hi) > 2) enc_open_batch<DP, ONE, 4>(w, d, cb, C, assign, p0, bad, lo, hi);
    else enc_open_batch<DP, ONE, 1>(w, d, cb, C, assign, p0, bad, lo, hi);
  }
}

// Assignment of every point to its nearest codeword on the matrix cores.
//
// The defined distance costs 3 d + 2 vector operations per (point, codeword)
// pair.  Instead the matrix cores give s = |c|^2 / 2 - p.c, which orders the
// codewords like the distance up to a bounded error, and the defined distance
// is evaluated only where that error leaves a choice:
//   * v_mfma_f32_32x32x16_f16 with 32 codewords as rows, 32 points as columns
//     and the norms |c|^2 / 2 as the C operand.  Lane l holds column l % 32
//     and 16 of the rows, in SUB blocks of 16 / SUB codewords; a block's
//     minimum takes one v_min3 for two codewords.  Each lane keeps the
//     smallest block minimum b1, its block, and the second smallest b2.
//   * Every codeword that can win has s <= min s + tau.  A lane whose b1 lies
//     in that range evaluates the defined distance of that block's codewords;
//     the two lanes of a point are merged by (distance, id).
//   * If b2 lies in the range too (or the minimum is not finite), the point is
//     open: its whole codebook is evaluated, four points at a time with the
//     codewords dealt to the lanes.  Where a tile has more of them than that
//     is worth (open_max), every distance of the wave's points is, and of its
//     next kEncWholeGroups groups without the minima.
// tau: fp32 sums of d + 1 terms differ from the exact s by at most
// (d + 2) 2^-22 (|p| + |c|)^2 / 2 whatever the order and rounding of the
// additions (one ulp each), and the defined distance from the exact one by
// (d + 3) 2^-24 of itself.  For the codewords that matter |c| <= |p| + dist
// and dist^2 = |p|^2 + 2 s, so R = 2.01 |p| + 1.01 dist bounds |p| + |c| (the
// margins cover the error of dist itself) and tau = R^2 (d + 3) 2^-21.
// Non-finite codewords can never win (their distance is inf or NaN): they
// are staged as zeros with an infinite norm.
// Bound by vector issue: per MFMA (32 cycles) 8 v_min3 (4 cycles each) and 3
// more instructions, which overlap the matrix core by about half only.
// Measured, 4096 x 4096, d = 4, C = 4096 (17.2 G pairs): 0.66-0.75 ms per
// assignment, every distance evaluated 4.7 ms; d = 2, C = 256: 0.20 against
// 0.44 ms; d = 8, C = 256: 0.08 against 0.26 ms; d = 16, C = 256: 0.07 against
// 4.9 ms (a run-time d); d = 4, C = 65536 (256 rows): 1.7 against 9.7 ms.
// At C = 64 the two are even (d = 2: 0.15 against 0.11 ms every distance,
// d = 8: 0.083 both, d = 1: 0.28 against 0.22), hence kEncDirectMax.  Blocks
// of 8 (SUB = 2) halve the final evaluation, which outweighs the minima up to
// 512 codewords.
// FN: tiles of 32 points per wave (each codeword fragment and its norms serve
// all of them).  ONE: the codebook is one LDS tile; else it is staged tile by
// tile for every group of points, and the final evaluation reads L2.
template <int DP, int FN, int SUB, bool ONE>
__global__ __launch_bounds__(kEncThreads, 4) void k_enc_assign(const half_t* __restrict__ w, int64_t P, int d,
                                                               const half_t* __restrict__ cb, int C,
                                                               uint32_t* __restrict__ assign) {
  using Tile = EncTile<DP>;
  constexpr int BL = 16 / SUB;  // codewords per block and lane
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int tile_cap = ONE ? (C + kEncSuper - 1) / kEncSuper * kEncSuper : Tile::MAX;  // codewords per tile
  const int ntiles = ONE ? 1 : (C + tile_cap - 1) / tile_cap;
  uint8_t* cw = smem;
  float* norms = reinterpret_cast<float*>(smem + (tile_cap / kEncSuper * Tile::SB + 15) / 16 * 16);
  int* odd = reinterpret_cast<int*>(norms + tile_cap);  // ONE: the tile holds non-finite codewords

  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int h = lane >> 5, col = lane & 31;
  const float inf = __builtin_inff();

  // codewords [k0, k0 + nk), padded to whole superblocks by the last one (with
  // an infinite norm; where its distance ties, the lower index has it)
  auto stage = [&](int k0, int nk) {
    const int n = (nk + kEncSuper - 1) / kEncSuper * kEncSuper;
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
      float c[DP];
      float norm = 0.f;
      bool ok = true;
      global_vector<DP>(cb, k0 + (k < nk ? k : nk - 1), d, c);
#pragma unroll
      for (int i = 0; i < DP; ++i) {
        norm = __builtin_fmaf(c[i], c[i], norm);
        ok = ok && __builtin_fabsf(c[i]) < inf;
      }
      uint8_t* q = cw + Tile::at(k);
#pragma unroll
      for (int i = 0; i < DP; i += 2) {
        half2_t v;
        v[0] = ok ? static_cast<half_t>(c[i]) : static_cast<half_t>(0.f);
        v[1] = ok ? static_cast<half_t>(c[i + 1]) : static_cast<half_t>(0.f);
        *reinterpret_cast<uint32_t*>(q + i * 2) = as_u32(v);
      }
      norms[k] = ok && k < nk ? 0.5f * norm : inf;
      if (ONE && !ok) *odd = 1;
    }
  };
  // the codeword fragment of rows [k, k + 32) of the tile: K values 8 h .. 8 h + 7
  auto read_rows = [&](int k) {
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    const uint8_t* q = cw + Tile::at(k) + col * Tile::CW;
    if constexpr (DP == 16) {
      v = *reinterpret_cast<const u32x4*>(q + 16 * h);
    } else if (h == 0) {
      if constexpr (DP == 2) v[0] = *reinterpret_cast<const uint32_t*>(q);
      else if constexpr (DP == 4) {
        const u32x2 t = *reinterpret_cast<const u32x2*>(q);
        v[0] = t[0]; v[1] = t[1];
      } else v = *reinterpret_cast<const u32x4*>(q);
    }
    return __builtin_bit_cast(half8_t, v);
  };
  auto read_norms = [&](int k) {  // rows (i / 4) * 8 + 4 h + i % 4 of the tile at k
    float16_t n;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float4_t t = *reinterpret_cast<const float4_t*>(norms + k + 8 * j + 4 * h);
#pragma unroll
      for (int i = 0; i < 4; ++i) n[4 * j + i] = t[i];
    }
    return n;
  };
  auto row_of = [&](int i) { return (i / 4) * 8 + 4 * h + i % 4; };  // i in [0, 16)

  if constexpr (ONE) {
    if (threadIdx.x == 0) *odd = 0;
    __syncthreads();
    stage(0, C);
    __syncthreads();
  }
  const bool bad = ONE && *odd != 0;
  // opaque infinities: minima that start from one take three operands from
  // the first step on (v_min3 throughout), and the median with the other is
  // the minimum of two values without the instruction that quiets a NaN
  float top = inf, bottom = -inf;
  asm volatile("" : "+v"(top), "+v"(bottom));

  // Vector instructions: an open point costs C / 64 rounds of 3 d + 5 and about
  // 150 for its merge, every distance of a tile C / 2 times 3 d + 1.
  const int open_max = (int)((int64_t)(C / 2) * (3 * d + 1) / ((C / 64) * (3 * d + 5) + 150));
  int skip = 0;  // groups to come whose every distance is evaluated straight away

  const int64_t group = (int64_t)kEncWaves * FN * 32;
  for (int64_t g0 = blockIdx.x * group; g0 < P; g0 += (int64_t)gridDim.x * group) {
    const int64_t p0 = g0 + (int64_t)wave * FN * 32;  // first point of the wave
    // B operands: the negated points (K values past d are zero)
    half8_t b[FN];
    float b1[FN], b2[FN];
    int i1[FN];
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      const int64_t p = p0 + f * 32 + col;
      const int64_t pc = p < P ? p : P - 1;
#pragma unroll
      for (int i = 0; i < 8; ++i) b[f][i] = static_cast<half_t>(0.f);
      if (DP == 16 || h == 0) {
#pragma unroll
        for (int i = 0; i < (DP < 8 ? DP : 8); ++i) {
          const int c = DP == 16 ? 8 * h + i : i;
          if (c < d) b[f][i] = -w[pc * d + c];
        }
      }
      b1[f] = b2[f] = inf;
      i1[f] = 0;
    }
    const bool skipped = skip > 0;
    skip -= skipped;
    for (int t = 0; t < ntiles; ++t) {
      const int k0 = t * tile_cap;
      const int nk = C - k0 < tile_cap ? C - k0 : tile_cap;
      if constexpr (!ONE) {
        __syncthreads();  // everyone is done with the previous tile
        stage(k0, nk);
        __syncthreads();
      }
      if (skipped) continue;
      for (int k = 0; k < nk; k += 32) {
        const half8_t a = read_rows(k);
        const float16_t n = read_norms(k);
        const int blk = (k0 + k) / 32 * SUB;
#pragma unroll
        for (int f = 0; f < FN; ++f) {
          const float16_t s = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b[f], n, 0, 0, 0);
#pragma unroll
          for (int j = 0; j < SUB; ++j) {
            float v = top;
#pragma unroll
            for (int i = 0; i < BL; i += 2) v = __builtin_fminf(__builtin_fminf(v, s[j * BL + i]), s[j * BL + i + 1]);
            i1[f] = v < b1[f] ? blk + j : i1[f];
            b2[f] = __builtin_amdgcn_fmed3f(v, b1[f], b2[f]);
            b1[f] = __builtin_amdgcn_fmed3f(v, b1[f], bottom);
          }
        }
      }
    }
    // the wave's points, and those that the minima leave open, per tile
    half_t ph[FN][DP];
    float thr[FN];
    uint32_t open[FN];
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      const int64_t p = p0 + f * 32 + col;
      half_vector<DP>(w, p < P ? p : P - 1, d, ph[f]);
    }
    bool whole = skipped, some = false;
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      float pn = 0.f;
#pragma unroll
      for (int i = 0; i < DP; ++i) pn = __builtin_fmaf(static_cast<float>(ph[f][i]), static_cast<float>(ph[f][i]), pn);
      const float gb = __builtin_fminf(b1[f], __shfl_xor(b1[f], 32, kWave));
      const float r = 2.01f * __builtin_amdgcn_sqrtf(pn) + 1.01f * __builtin_amdgcn_sqrtf(__builtin_fmaxf(pn + 2.f * gb, 0.f));
      thr[f] = gb + r * r * ((float)(d + 3) * 4.76837158203125e-7f);  // 2^-21
      // not (x < y): true for NaN as well
      const bool slow = !(__builtin_fabsf(gb) < inf) || !(b2[f] > thr[f]);
      const uint64_t both = __ballot(slow && p0 + f * 32 + col < P);
      open[f] = (uint32_t)(both | (both >> 32));
      some = some || open[f] != 0;
      whole = whole || __popc(open[f]) > open_max;
    }
    if (whole) {
      if (!skipped) skip = kEncWholeGroups;
      enc_every_distance<DP, FN, ONE>(w, P, d, cb, C, assign, p0, bad);
      continue;
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      const int64_t p = p0 + f * 32 + col;
      float pv[DP];
#pragma unroll
      for (int i = 0; i < DP; ++i) pv[i] = static_cast<float>(ph[f][i]);
      float best = inf;
      uint32_t bk = 0;
      auto consider = [&](int k) {  // strict: the lowest index keeps a tie
        float c[DP];
        if constexpr (ONE) lds_codeword<DP>(cw, k, c);
        else global_vector<DP>(cb, k, d, c);
        const float dist = sq_dist<DP>(pv, c);
        // (an infinite norm in LDS: a codeword staged as zeros, or padding)
        if (dist < best && (!bad || norms[k] < inf)) {
          best = dist;
          bk = (uint32_t)k;
        }
      };
      if (b1[f] <= thr[f]) {
        const int k = i1[f] / SUB * 32, i0 = i1[f] % SUB * BL;
        if (!ONE || bad) {
          for (int i = 0; i < BL; ++i) {
            const int kk = k + (i0 / 4) * 8 + row_of(i);  // i0 is a multiple of 4
            consider(ONE || kk < C ? kk : C - 1);
          }
        } else {
          // reads in batches, then selects: no branch and one wait per batch
          constexpr int RB = DP == 16 ? 4 : BL < 8 ? BL : 8;
#pragma unroll
          for (int j = 0; j < BL; j += RB) {
            float c[RB][DP];
#pragma unroll
            for (int i = 0; i < RB; ++i) lds_codeword<DP>(cw, k + (i0 / 4) * 8 + row_of(j + i), c[i]);
#pragma unroll
            for (int i = 0; i < RB; ++i) {
              const float dist = sq_dist<DP>(pv, c[i]);
              bk = dist < best ? (uint32_t)(k + (i0 / 4) * 8 + row_of(j + i)) : bk;
              best = dist < best ? dist : best;
            }
          }
        }
      }
      const float ob = __shfl_xor(best, 32, kWave);
      const uint32_t ok = (uint32_t)__shfl_xor((int)bk, 32, kWave);
      if (ob < best || (ob == best && ok < bk)) bk = ok;
      if (p < P && h == 0 && !(open[f] >> col & 1)) assign[p] = bk;
    }
    if (some) {
      uint64_t lo = 0, hi = 0;  // the open points of tiles 0 and 1, and 2 and 3
#pragma unroll
      for (int f = 0; f < FN; ++f) (f < 2 ? lo : hi) |= (uint64_t)open[f] << (f % 2 * 32);
      enc_open_points<DP, ONE>(w, d, cb, C, assign, p0, bad, lo, hi);
    }
  }
}

// Cluster sums (values times 2^24: exact integers) and counts of the assigned
// points.  Workgroup (x, y) takes its share x of the points and the clusters
// [y cap, y cap + cap), gathers them in LDS (`copies` tables, dealt to the
// waves, where few clusters would make many lanes meet in one) and adds its
// table to the global sums.  cap = 0: every point straight to global memory.
// 4096 x 4096, d = 4, C = 4096: 60 us in one table per CU, 270 us with every
// point's atomics in global memory.
// D: d as a compile-time constant, with w aligned to D halves; 0: any d.
template <int D>
__global__ __launch_bounds__(kEncSumThreads) void k_enc_sum(const half_t* __restrict__ w, int64_t P, int rt_d, int C,
                                                            int cap, int copies, const uint32_t* __restrict__ assign,
                                                            unsigned long long* __restrict__ sums,
                                                            unsigned long long* __restrict__ counts) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int d = D > 0 ? D : rt_d;
  const int k0 = blockIdx.y * cap;
  const int nk = C - k0 < cap ? C - k0 : cap;
  unsigned long long* tsum = reinterpret_cast<unsigned long long*>(smem);            // [copies][cap][d]
  uint32_t* tcnt = reinterpret_cast<uint32_t*>(smem + (size_t)copies * cap * d * 8);  // [copies][cap]
  for (int i = threadIdx.x; i < copies * cap * d; i += blockDim.x) tsum[i] = 0;
  for (int i = threadIdx.x; i < copies * cap; i += blockDim.x) tcnt[i] = 0;
  __syncthreads();
  const int mine = cap > 0 ? (int)(threadIdx.x / kWave) % copies * cap : 0;
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < P; p += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t k = assign[p];
    half_t v[D > 0 ? D : 16];
    if constexpr (D == 2) *reinterpret_cast<uint32_t*>(v) = reinterpret_cast<const uint32_t*>(w)[p];
    else if constexpr (D == 4) *reinterpret_cast<u32x2*>(v) = reinterpret_cast<const u32x2*>(w)[p];
    else if constexpr (D == 8) *reinterpret_cast<u32x4*>(v) = reinterpret_cast<const u32x4*>(w)[p];
    else {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (i < d) v[i] = w[p * d + i];
    }
    const uint32_t t = k - (uint32_t)k0;
    if (cap > 0 && t >= (uint32_t)nk) continue;
#pragma unroll
    for (int i = 0; i < (D > 0 ? D : 16); ++i) {
      if (i >= d) continue;
      const unsigned long long q = (unsigned long long)(int64_t)(static_cast<float>(v[i]) * kQScale);  // exact
      if (cap > 0) atomicAdd(&tsum[(mine + (int)t) * d + i], q);
      else atomicAdd(&sums[(int64_t)k * d + i], q);
    }
    if (cap > 0) atomicAdd(&tcnt[mine + (int)t], 1u);
    else atomicAdd(&counts[k], 1ull);
  }
  if (cap == 0) return;
  __syncthreads();
  for (int i = threadIdx.x; i < nk * (d + 1); i += blockDim.x) {
    unsigned long long v = 0;
    if (i < nk * d) {
      for (int c = 0; c < copies; ++c) v += tsum[c * cap * d + i];
      if (v != 0) atomicAdd(&sums[(int64_t)k0 * d + i], v);
    } else {
      for (int c = 0; c < copies; ++c) v += tcnt[c * cap + i - nk * d];
      if (v != 0) atomicAdd(&counts[k0 + i - nk * d], v);
    }
  }
}

// New codewords: each non-empty cluster's rounded mean; empty ones are kept.
// The sums and counts are cleared for the next iteration.  A thread takes one
// component (a thread per codeword read its components one after the other,
// about 0.5 us each), a workgroup whole codewords, so that a count is cleared
// when all of its readers have it.
__global__ __launch_bounds__(kEncUpdateThreads) void k_enc_update(uint16_t* __restrict__ cb, int64_t* __restrict__ sums,
                                                                  int64_t* __restrict__ counts, int C, int d) {
  const int per = kEncUpdateThreads / d;  // codewords per workgroup
  const int local = threadIdx.x / d;
  const int k = blockIdx.x * per + local;
  const bool live = local < per && k < C;
  const int64_t t = live ? (int64_t)k * d + (threadIdx.x - local * d) : 0;
  const int64_t cnt = live ? counts[k] : 0;
  const int64_t sum = sums[t];
  __syncthreads();
  if (cnt == 0) return;
  sums[t] = 0;
  if (threadIdx.x == local * d) counts[k] = 0;
  cb[t] = f64_to_f16_rne((static_cast<double>(sum) * kQInv) / static_cast<double>(cnt));
}

// ids [N x S] (uint32) -> packed rows of R bytes.  One thread per id pair
// for 12-bit ids (three bytes), per id otherwise.
template <int BITS>
__global__ void k_enc_pack(const uint32_t* __restrict__ ids, int64_t N, int64_t S, int64_t R,
                           uint8_t* __restrict__ idx) {
  const int64_t per_row = BITS == 12 ? (S + 1) / 2 : S;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < N * per_row;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t n = t / per_row;
    const int64_t j = t - n * per_row;
    uint8_t* row = idx + n * R;
    const uint32_t* u = ids + n * S;
    if constexpr (BITS == 8) {
      row[j] = (uint8_t)u[j];
    } else if constexpr (BITS == 16) {
      row[2 * j] = (uint8_t)(u[j] & 0xFF);
      row[2 * j + 1] = (uint8_t)(u[j] >> 8);
    } else {
      const uint32_t a = u[2 * j];
      const uint32_t b = 2 * j + 1 < S ? u[2 * j + 1] : 0u;  // the pad nibble of an odd row is 0
      row[3 * j] = (uint8_t)(a & 0xFF);
      if (3 * j + 1 < R) row[3 * j + 1] = (uint8_t)((a >> 8) | ((b & 0xF) << 4));
      if (3 * j + 2 < R) row[3 * j + 2] = (uint8_t)(b >> 4);
    }
  }
}

inline unsigned grid_for(int64_t n, int threads) {
  const int64_t g = (n + threads - 1) / threads;
  return (unsigned)(g < 65536 ? (g > 0 ? g : 1) : 65536);
}

template <int DP>
hipError_t launch_direct(const half_t* w, int64_t P, int d, const half_t* cb, int C, uint32_t* assign, int64_t* sums,
                         int64_t* counts, bool accum, const DeviceInfo& dev, hipStream_t stream) {
  const int64_t per = (int64_t)kEncDirectThreads * kEncDirectPoints;
  const int64_t groups = (P + per - 1) / per, slots = 4 * (int64_t)dev.num_cus;
  const dim3 grid((unsigned)(groups < slots ? groups : slots));
  unsigned long long* s = reinterpret_cast<unsigned long long*>(sums);
  unsigned long long* c = reinterpret_cast<unsigned long long*>(counts);
  if (accum) return launch_kernel(k_enc_direct<DP, true>, grid, dim3(kEncDirectThreads), 0, stream, w, P, d, cb, C, assign, s, c);
  return launch_kernel(k_enc_direct<DP, false>, grid, dim3(kEncDirectThreads), 0, stream, w, P, d, cb, C, assign, s, c);
}

template <int DP>
hipError_t launch_assign_dp(const half_t* w, int64_t P, int d, const half_t* cb, int C, uint32_t* assign,
                            const DeviceInfo& dev, hipStream_t stream) {
  using Tile = EncTile<DP>;
  const bool one = C <= Tile::MAX;
  const int cap = one ? (C + kEncSuper - 1) / kEncSuper * kEncSuper : Tile::MAX;
  const int lds = (cap / kEncSuper * Tile::SB + 15) / 16 * 16 + cap * 4 + 16;
  // four point tiles per wave where that still gives every CU two workgroups,
  // else one; never more workgroups than two per CU (more would only repeat
  // the codebook staging)
  const int64_t slots = 2 * (int64_t)dev.num_cus;
  auto groups_of = [&](int fn) { return (P + (int64_t)kEncWaves * fn * 32 - 1) / ((int64_t)kEncWaves * fn * 32); };
  const bool wide = groups_of(4) >= slots;
  const int64_t groups = groups_of(wide ? 4 : 1);
  const int64_t blocks = groups < slots ? groups : slots;
  auto go = [&](auto kern) {
    hipError_t e = prepare_kernel(kern);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3((unsigned)blocks), dim3(kEncThreads), lds, stream, w, P, d, cb, C, assign);
  };
  if (!one) return wide ? go(k_enc_assign<DP, 4, 1, false>) : go(k_enc_assign<DP, 1, 1, false>);
  if (C <= kEncFineMax) return wide ? go(k_enc_assign<DP, 4, 2, true>) : go(k_enc_assign<DP, 1, 2, true>);
  return wide ? go(k_enc_assign<DP, 4, 1, true>) : go(k_enc_assign<DP, 1, 1, true>);
}

hipError_t launch_sum(const half_t* w, int64_t P, int d, int C, const uint32_t* assign, int64_t* sums,
                      int64_t* counts, const DeviceInfo& dev, hipStream_t stream) {
  const int per = 8 * d + 4;                 // table bytes per cluster
  int cap = kEncSumBytes / per;              // clusters per table
  int ranges = 1, copies = 1;
  if (cap >= C) {
    copies = cap / C < kEncSumThreads / kWave ? cap / C : kEncSumThreads / kWave;
    cap = C;
  } else {
    ranges = (C + cap - 1) / cap;
    cap = (C + ranges - 1) / ranges;
    if (ranges > kEncSumMaxRanges) ranges = 1, cap = 0;
  }
  // tables: about one workgroup per CU in all, each with at least a table's
  // worth of points; without tables enough threads to fill the chip
  const int64_t per_wg = cap > 0 && copies == 1 ? 4 * (int64_t)cap : 4 * kEncSumThreads;
  int64_t blocks = (P + per_wg - 1) / per_wg;
  const int64_t most = (cap > 0 ? 1 : 2) * (int64_t)dev.num_cus / ranges;
  if (blocks > most) blocks = most;
  if (blocks < 1) blocks = 1;
  const int lds = copies * cap * per;
  unsigned long long* s = reinterpret_cast<unsigned long long*>(sums);
  unsigned long long* c = reinterpret_cast<unsigned long long*>(counts);
  auto go = [&](auto kern) {
    hipError_t e = prepare_kernel(kern);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3((unsigned)blocks, (unsigned)ranges), dim3(kEncSumThreads), lds, stream, w, P, d, C,
                         cap, copies, assign, s, c);
  };
  const uintptr_t at = reinterpret_cast<uintptr_t>(w);
  if (d == 2 && at % 4 == 0) return go(k_enc_sum<2>);
  if (d == 4 && at % 8 == 0) return go(k_enc_sum<4>);
  if (d == 8 && at % 16 == 0) return go(k_enc_sum<8>);
  return go(k_enc_sum<0>);
}

// Assignment of every point, and with accum the cluster sums and counts.
hipError_t launch_assign(const half_t* w, int64_t P, int d, const half_t* cb, int C, uint32_t* assign, int64_t* sums,
                         int64_t* counts, bool accum, const DeviceInfo& dev, hipStream_t stream) {
  if (C <= kEncDirectMax) {
    if (d == 1) return launch_direct<1>(w, P, d, cb, C, assign, sums, counts, accum, dev, stream);
    if (d <= 2) return launch_direct<2>(w, P, d, cb, C, assign, sums, counts, accum, dev, stream);
    if (d <= 4) return launch_direct<4>(w, P, d, cb, C, assign, sums, counts, accum, dev, stream);
    if (d <= 8) return launch_direct<8>(w, P, d, cb, C, assign, sums, counts, accum, dev, stream);
    return launch_direct<16>(w, P, d, cb, C, assign, sums, counts, accum, dev, stream);
  }
  hipError_t e;
  if (d <= 2) e = launch_assign_dp<2>(w, P, d, cb, C, assign, dev, stream);
  else if (d <= 4) e = launch_assign_dp<4>(w, P, d, cb, C, assign, dev, stream);
  else if (d <= 8) e = launch_assign_dp<8>(w, P, d, cb, C, assign, dev, stream);
  else e = launch_assign_dp<16>(w, P, d, cb, C, assign, dev, stream);
  if (e != hipSuccess || !accum) return e;
  return launch_sum(w, P, d, C, assign, sums, counts, dev, stream);
}

}  // namespace

int64_t encode_workspace_bytes(int64_t N, int64_t K, int d, int64_t C) {
  const int64_t P = N * (K / d);
  const int64_t head = ((C * d + C) * 8 + 255) / 256 * 256;
  return head + P * 4;
}

hipError_t launch_encode(const EncodeProblem& e, const DeviceInfo& dev, hipStream_t stream) {
  const int64_t S = e.K / e.d;
  const int64_t P = e.N * S;
  const int d = e.d;
  const int C = (int)e.C;
  uint8_t* ws = static_cast<uint8_t*>(e.workspace);
  int64_t* sums = reinterpret_cast<int64_t*>(ws);
  int64_t* counts = sums + (int64_t)C * d;
  uint32_t* assign = reinterpret_cast<uint32_t*>(ws + ((e.C * d + e.C) * 8 + 255) / 256 * 256);
  const half_t* w = static_cast<const half_t*>(e.w);
  uint16_t* cb = static_cast<uint16_t*>(e.codebook);
  const int64_t cbn = (int64_t)C * d;
  hipError_t err;
  if (e.init != e.codebook) {
    err = launch_kernel(k_enc_copy, dim3(grid_for(cbn, 256)), dim3(256), 0, stream,
                        static_cast<const uint16_t*>(e.init), cb, cbn);
    if (err != hipSuccess) return err;
  }
  if (e.iters > 0) {
    err = launch_kernel(k_enc_zero, dim3(grid_for(cbn + C, 256)), dim3(256), 0, stream, sums, cbn + C);
    if (err != hipSuccess) return err;
  }
  for (int it = 0; it < e.iters; ++it) {
    err = launch_assign(w, P, d, reinterpret_cast<const half_t*>(cb), C, assign, sums, counts, true, dev, stream);
    if (err != hipSuccess) return err;
    err = launch_kernel(k_enc_update, dim3((unsigned)((C + kEncUpdateThreads / d - 1) / (kEncUpdateThreads / d))),
                        dim3(kEncUpdateThreads), 0, stream, cb, sums, counts, C, d);
    if (err != hipSuccess) return err;
  }
  err = launch_assign(w, P, d, reinterpret_cast<const half_t*>(cb), C, assign, sums, counts, false, dev, stream);
  if (err != hipSuccess) return err;
  const int64_t per_row = e.idx_bits == 12 ? (S + 1) / 2 : S;
  const unsigned g = grid_for(e.N * per_row, 256);
  uint8_t* idx = static_cast<uint8_t*>(e.idx);
  switch (e.idx_bits) {
    case 8: return launch_kernel(k_enc_pack<8>, dim3(g), dim3(256), 0, stream, assign, e.N, S, e.R, idx);
    case 12: return launch_kernel(k_enc_pack<12>, dim3(g), dim3(256), 0, stream, assign, e.N, S, e.R, idx);
    default: return launch_kernel(k_enc_pack<16>, dim3(g), dim3(256), 0, stream, assign, e.N, S, e.R, idx);
  }
}

}  // namespace fasq
