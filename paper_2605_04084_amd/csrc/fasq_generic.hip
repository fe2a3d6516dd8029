// Reconstruction kernel and the general-purpose PQ matmul kernel.
//
// The general kernel handles every valid argument combination (any M, K, N,
// d, C, id width, pointer alignment); the tuned GEMV/GEMM kernels cover the
// common shapes and fall back to it for the rest.
#include <type_traits>

#include "fasq_codebook.h"
#include "fasq_device.h"
#include "fasq_internal.h"

namespace fasq {

// W_hat[n, s*d + i] = codebook[u(n, s)*d + i], moved as raw 16-bit patterns.
// One thread per (n, s); grid-stride over all N*S sub-vectors.
template <int BITS>
__global__ __launch_bounds__(256) void k_reconstruct(const uint8_t* __restrict__ idx, int64_t N, int64_t S,
                                                     int64_t R, int d, const uint16_t* __restrict__ cb,
                                                     int64_t cbs, uint16_t* __restrict__ w) {
  const int64_t total = N * S;
  const int64_t K = S * d;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t n = t / S;
    const int64_t s = t - n * S;
    const uint32_t u = load_id_bytes<BITS>(idx + n * R, s, R);
    const uint16_t* src = cb + s * cbs + (int64_t)u * d;
    uint16_t* dst = w + n * K + s * d;
    for (int i = 0; i < d; ++i) dst[i] = src[i];
  }
}

// y[m, n] = sum_s dot(x[m, s*d:(s+1)*d], codebook[u(n, s)]), fp32 accumulation
// (codebook s of subspace s at cb + s * cbs when the books are per subspace),
// for every valid call: any d, alignment and row length, any M.
//
// A workgroup owns up to 16 output features and FM tiles of 16 tokens; its
// waves deal the K spans of 128 among themselves (v_mfma_f32_16x16x32_f16,
// operands straight to registers) and their partial tiles are added in wave
// order in LDS: deterministic, no workspace.  Lane l holds feature l % 16 and
// the 32 consecutive K values of group l / 16 of each span (whole codewords), so it reads its
// ids as one run and the gathered codewords serve every token of the
// workgroup.  The K order inside a span is permuted identically for both
// operands.
// Bound by the gathers: at most one lane per cycle and CU from global memory
// (half of that from L2), where LDS serves ten and more, hence LCB: a shared codebook of up to
// kGenericLdsBytes is staged in LDS.  With a codebook per subspace the 16
// features of a group share the few cache lines of one book, so a workgroup
// draws about every book through its L1 once (2 MB for 4096 x 4096 at d = 2,
// C = 256).  Measured against one wave per feature with scalar products:
// 48 tokens of that layer 694 -> 30 us, one token 52 -> 18 us; 1003 x 1516,
// d = 4, 37 tokens 84 -> 5 us.
// D: d as a compile-time constant, or 0 for any other d.
constexpr int kGenericRun = 32;     // K values per lane and wave step, at most
constexpr int kGenericWaves = 16;   // most waves per workgroup
constexpr int kGenericLdsBytes = 64 * 1024;

// K values per lane and wave step for a run-time d: whole codewords.
__host__ __device__ constexpr int generic_run(int d) { return d <= kGenericRun ? kGenericRun / d * d : kGenericRun; }

struct GenericArgs {
  const half_t* x;
  int64_t M, K, N;
  const uint8_t* idx;
  int64_t R;
  int d;
  const half_t* cb;
  int64_t cbs;
  half_t* y;
  int64_t ldy;   // elements between the outputs of consecutive tokens
  int cols;      // features per workgroup, at most 16
  int cb_bytes;  // LCB: bytes of the codebook
};

template <int BITS, int D, int FM, bool LCB>
__global__ __launch_bounds__(kGenericWaves * kWave) void k_pq_generic(GenericArgs a) {
  constexpr int RB = D > 0 ? kGenericRun / (D > 0 ? D : 1) * BITS / 8 : 4;  // id bytes per run
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // the codebook, then the partial tiles
  float* part = reinterpret_cast<float*>(smem);                   // [waves][FM * 16][16]
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int waves = blockDim.x / kWave;
  const int g = lane >> 4, l16 = lane & 15;
  const int64_t n0 = (int64_t)blockIdx.x * a.cols;
  const int64_t m0 = (int64_t)blockIdx.y * (FM * 16);
  const bool active = l16 < a.cols && n0 + l16 < a.N;  // the other lanes feed zeros
  const uint8_t* row = a.idx + (active ? n0 + l16 : n0) * a.R;
  const uint8_t* table_end = a.idx + a.N * a.R;
  const half_t* xrow[FM];  // tokens past M repeat the last one; they are not stored
#pragma unroll
  for (int f = 0; f < FM; ++f) {
    const int64_t m = m0 + f * 16 + l16;
    xrow[f] = a.x + (m < a.M ? m : a.M - 1) * a.K;
  }
  float4_t acc[FM];
#pragma unroll
  for (int f = 0; f < FM; ++f) acc[f] = float4_t{0.f, 0.f, 0.f, 0.f};
  const int d = D > 0 ? D : a.d;
  const int64_t S = a.K / d;
  const int run = D > 0 ? kGenericRun : generic_run(d);  // K values per lane and wave step
  const int span = 4 * run;
  const int64_t spans = (a.K + span - 1) / span;

  if constexpr (LCB) {
    const int words = a.cb_bytes / 4;
    for (int i = threadIdx.x; i < words; i += blockDim.x)
      __builtin_memcpy(smem + 4 * i, reinterpret_cast<const uint8_t*>(a.cb) + 4 * i, 4);
    if (a.cb_bytes % 4 && threadIdx.x == 0)
      *reinterpret_cast<half_t*>(smem + 4 * words) = a.cb[2 * words];
    __syncthreads();
  }
  const half_t* lcb = reinterpret_cast<const half_t*>(smem);

  for (int64_t sp = wave; sp < spans; sp += waves) {
    const int64_t k0 = sp * span + g * run;
    half8_t b[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) b[t] = half8_t{};
    const bool whole = run == kGenericRun && (sp + 1) * span <= a.K;
    if constexpr (D > 0) {
      constexpr int DD = D > 0 ? D : 1;
      auto read = [&](auto id, int64_t left) {  // the run's codewords; those from `left` values on are zero
        const half_t* books = a.cb + k0 / DD * a.cbs;
        auto codeword = [&](int i, uint32_t* out) {
          const bool live = i * DD < left;
          if constexpr (LCB) {
            read_codeword_lds<DD>(id(i) * (2 * DD), out);
          } else {  // (any alignment)
            out[0] = 0;
            __builtin_memcpy(out, books + (live ? i : 0) * a.cbs + (int64_t)id(i) * DD, 2 * DD);
          }
#pragma unroll
          for (int q = 0; q < (DD + 1) / 2; ++q) out[q] = live ? out[q] : 0u;
        };
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          uint32_t o[4];
          if constexpr (DD == 1) {
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
              uint32_t c0[1], c1[1];
              codeword(t * 8 + e, c0);
              codeword(t * 8 + e + 1, c1);
              o[e / 2] = (c0[0] & 0xFFFFu) | (c1[0] << 16);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 8 / DD; ++e) codeword(t * (8 / DD) + e, o + e * (DD / 2));
          }
          b[t] = __builtin_bit_cast(half8_t, u32x4{o[0], o[1], o[2], o[3]});
        }
      };
      if (active && whole) {
        uint32_t w[(RB + 3) / 4];
        w[(RB + 3) / 4 - 1] = 0;
        __builtin_memcpy(w, row + k0 / DD * BITS / 8, RB);
        read([&](int i) { return stream_id<BITS>(w, i); }, kGenericRun);
      } else if (active && k0 < a.K) {  // past the row's end its first id of the run, whose codeword is dropped
        uint32_t u[kGenericRun / DD];
        const int64_t s0 = k0 / DD;
#pragma unroll
        for (int i = 0; i < kGenericRun / DD; ++i)
          u[i] = load_id_bytes<BITS>(row, k0 + i * DD < a.K ? s0 + i : s0, a.R);
        read([&](int i) { return u[i]; }, a.K - k0);
      }
    } else {
      // Value by value, two at a time for even d.  A run holds whole codewords
      // (run = 32 / d * d values, so every lane starts a codeword at the same
      // place), or 32 values of longer ones.  Its ids (at most 10) come as one
      // window of WN words, shifted down by one id at every codeword, so that
      // no read waits for another; windows past the table's end id by id.
      if (active && k0 < a.K) {
        constexpr int WN = (12 * BITS + 4 + 31) / 32;
        const int64_t s0 = k0 / d;
        const uint8_t* at = row + s0 * BITS / 8;
        uint32_t w[WN];
        if (at + WN * 4 <= table_end) {
          __builtin_memcpy(w, at, WN * 4);
          if (BITS == 12 && (s0 & 1)) {
#pragma unroll
            for (int j = 0; j < WN - 1; ++j) w[j] = __builtin_amdgcn_alignbit(w[j + 1], w[j], 4);
          }
        } else {
#pragma unroll
          for (int j = 0; j < WN; ++j) w[j] = 0;
          for (int e = 0; e < 11 && s0 + e < S; ++e) {
            const uint64_t u = (uint64_t)load_id_bytes<BITS>(row, s0 + e, a.R) << (e * BITS % 32);
#pragma unroll
            for (int j = 0; j < WN; ++j) {
              if (j == e * BITS / 32) w[j] |= (uint32_t)u;
              if (j == e * BITS / 32 + 1) w[j] |= (uint32_t)(u >> 32);
            }
          }
        }
        const half_t* book = a.cb + s0 * a.cbs;
        // first half of the codeword in its book
        auto first = [&]() { return (uint64_t)(w[0] & ((1u << BITS) - 1u)) * (uint32_t)d; };
        uint64_t c = first();
        const int nrun = (int)(a.K - k0 < run ? a.K - k0 : run);  // values of the run
        auto walk = [&](auto step, int i0) {
          constexpr int ST = decltype(step)::value;
          uint32_t r[32 / ST];
          int i = i0;
#pragma unroll
          for (int j = 0; j < 32; j += ST) {
            r[j / ST] = 0;
            if (j >= run) continue;
            if constexpr (ST == 2) {
              if constexpr (LCB) r[j / 2] = *reinterpret_cast<const uint32_t*>(lcb + (uint32_t)c + i);
              else __builtin_memcpy(&r[j / 2], book + c + i, 4);
            } else {
              r[j] = LCB ? reinterpret_cast<const uint16_t*>(lcb)[(uint32_t)c + i] : reinterpret_cast<const uint16_t*>(book)[c + i];
            }
            i += ST;
            if (i == d) {
              i = 0;
              if (j + ST < nrun) {  // past the run the codeword stays: its values are dropped below
                book += a.cbs;
#pragma unroll
                for (int q = 0; q < WN - 1; ++q) w[q] = __builtin_amdgcn_alignbit(w[q + 1], w[q], BITS);
                w[WN - 1] >>= BITS;
                c = first();
              }
            }
          }
#pragma unroll
          for (int j = 0; j < 32; ++j) {
            const uint32_t h = ST == 2 ? r[j / ST] >> (j % 2 * 16) : r[j / ST];
            b[j / 8][j % 8] = __builtin_bit_cast(half_t, (uint16_t)(j < nrun ? h : 0u));
          }
        };
        // (one phase for all lanes as a scalar; codewords longer than a run start anywhere)
        if (d > 32) walk(std::integral_constant<int, 1>{}, (int)(k0 - s0 * d));
        else if (d % 2 == 0) walk(std::integral_constant<int, 2>{}, 0);
        else walk(std::integral_constant<int, 1>{}, 0);
      }
    }
    if (whole) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int f = 0; f < FM; ++f) {
          half8_t v;
          __builtin_memcpy(&v, xrow[f] + k0 + t * 8, 16);
          acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v, b[t], acc[f], 0, 0, 0);
        }
      }
    } else {  // values of x past the run, or the row's end, are zero
#pragma unroll
      for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int f = 0; f < FM; ++f) {
          half8_t v = half8_t{};
          const int64_t k = k0 + t * 8;
          if (k + 8 <= a.K) {
            __builtin_memcpy(&v, xrow[f] + k, 16);
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (k + j < a.K) v[j] = xrow[f][k + j];
          }
#pragma unroll
          for (int j = 0; j < 8; ++j) v[j] = t * 8 + j < run ? v[j] : static_cast<half_t>(0.f);
          acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v, b[t], acc[f], 0, 0, 0);
        }
      }
    }
  }

  if constexpr (LCB) __syncthreads();  // everyone is done with the codebook
  // lane l holds tokens 4 g .. 4 g + 3 of feature l16 of each tile
#pragma unroll
  for (int f = 0; f < FM; ++f)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[((wave * FM + f) * 16 + 4 * g + i) * 16 + l16] = acc[f][i];
  __syncthreads();
  for (int o = threadIdx.x; o < FM * 256; o += blockDim.x) {
    const int64_t m = m0 + o / 16, n = n0 + o % 16;
    if (m >= a.M || n >= a.N || o % 16 >= a.cols) continue;
    float sum = 0.f;
    for (int p = 0; p < waves; ++p) sum += part[p * FM * 256 + o];
    a.y[m * a.ldy + n] = static_cast<half_t>(sum);
  }
}

// The same for calls of few values, a wave per output feature: the lanes take
// the S sub-vectors, up to kRowsTokens tokens at once, scalar products in fp32.
// Bound by the latency of its few serial loads, where k_pq_generic issues an
// unrolled span whatever part of it is there (2500 instructions at a run-time
// d).  Replayed from a graph, this / k_pq_generic (K x N): 1 token, 110 x 478,
// d = 5 3.2 / 5.8 us, 336 x 848, d = 6, 12-bit ids 3.7 / 7.1; 2 tokens, 8 x 7,
// d = 4 3.1 / 4.0; 4 tokens, 203 x 23, d = 7 5.1 / 6.4; but 8 tokens, 6 x 36,
// d = 6 6.3 / 5.3 and 4 tokens, 112 x 1529, d = 4 4.4 / 3.4.
constexpr int kRowsTokens = 8;
constexpr int kRowsThreads = 256;

template <int BITS>
__global__ __launch_bounds__(kRowsThreads) void k_pq_generic_rows(const half_t* __restrict__ x, int M, int64_t K,
                                                                  int64_t N, const uint8_t* __restrict__ idx,
                                                                  int64_t R, int d, const half_t* __restrict__ cb,
                                                                  int64_t cbs, half_t* __restrict__ y) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t S = K / d;
  const int64_t n = blockIdx.x * (int64_t)(kRowsThreads / kWave) + threadIdx.x / kWave;
  if (n >= N) return;
  const uint8_t* row = idx + n * R;
  for (int m0 = 0; m0 < M; m0 += kRowsTokens) {
    const int mb = M - m0 < kRowsTokens ? M - m0 : kRowsTokens;
    float acc[kRowsTokens];
#pragma unroll
    for (int j = 0; j < kRowsTokens; ++j) acc[j] = 0.f;
    for (int64_t s = lane; s < S; s += kWave) {
      const uint32_t u = load_id_bytes<BITS>(row, s, R);
      const half_t* c = cb + s * cbs + (int64_t)u * d;
      for (int i = 0; i < d; ++i) {
        const float cv = static_cast<float>(c[i]);
        const half_t* xp = x + m0 * K + s * d + i;
#pragma unroll
        for (int j = 0; j < kRowsTokens; ++j)
          if (j < mb) acc[j] = __builtin_fmaf(static_cast<float>(xp[j * K]), cv, acc[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < kRowsTokens; ++j) {
      if (j < mb) {
        const float v = wave_sum(acc[j]);
        if (lane == 0) y[(m0 + j) * N + n] = static_cast<half_t>(v);
      }
    }
  }
}

static int grid_for(int64_t items, int per_block, int max_blocks) {
  int64_t b = (items + per_block - 1) / per_block;
  if (b > max_blocks) b = max_blocks;
  if (b < 1) b = 1;
  return (int)b;
}

hipError_t launch_reconstruct(const Problem& p, void* w, hipStream_t stream) {
  const int64_t S = p.K / p.d;
  const int blocks = grid_for(p.N * S, 256, 65536);
  const uint8_t* idx = static_cast<const uint8_t*>(p.idx);
  const uint16_t* cb = static_cast<const uint16_t*>(p.codebook);
  uint16_t* out = static_cast<uint16_t*>(w);
  switch (p.idx_bits) {
    case 8: return launch_kernel(k_reconstruct<8>, dim3(blocks), dim3(256), 0, stream, idx, p.N, S, p.R, p.d, cb, p.cb_stride, out);
    case 12: return launch_kernel(k_reconstruct<12>, dim3(blocks), dim3(256), 0, stream, idx, p.N, S, p.R, p.d, cb, p.cb_stride, out);
    default: return launch_kernel(k_reconstruct<16>, dim3(blocks), dim3(256), 0, stream, idx, p.N, S, p.R, p.d, cb, p.cb_stride, out);
  }
}

namespace {

template <int BITS, int D, int FM>
hipError_t launch_generic_fm(const GenericArgs& a, hipStream_t stream) {
  const int span = 4 * generic_run(a.d);
  const int64_t spans = (a.K + span - 1) / span;
  const int waves = (int)(spans < kGenericWaves ? spans : kGenericWaves);
  const dim3 grid((unsigned)((a.N + a.cols - 1) / a.cols), (unsigned)((a.M + FM * 16 - 1) / (FM * 16)));
  size_t lds = (size_t)waves * FM * 256 * 4;
  if (a.cb_bytes == 0) return launch_kernel(k_pq_generic<BITS, D, FM, false>, grid, dim3(waves * kWave), lds, stream, a);
  if ((size_t)a.cb_bytes > lds) lds = (size_t)a.cb_bytes;
  auto kern = k_pq_generic<BITS, D, FM, true>;  // reads its codebook from LDS address 0
  hipError_t e = prepare_kernel(kern);
  if (e != hipSuccess) return e;
  return launch_kernel(kern, grid, dim3(waves * kWave), lds, stream, a);
}

template <int BITS, int D>
hipError_t launch_generic_d(const GenericArgs& a, int fm, hipStream_t stream) {
  switch (fm) {
    case 1: return launch_generic_fm<BITS, D, 1>(a, stream);
    case 2: return launch_generic_fm<BITS, D, 2>(a, stream);
    case 3: return launch_generic_fm<BITS, D, 3>(a, stream);
    default: return launch_generic_fm<BITS, D, 4>(a, stream);
  }
}

template <int BITS>
hipError_t launch_generic_bits(const GenericArgs& a, int fm, hipStream_t stream) {
  switch (a.d) {
    case 1: return launch_generic_d<BITS, 1>(a, fm, stream);
    case 2: return launch_generic_d<BITS, 2>(a, fm, stream);
    case 4: return launch_generic_d<BITS, 4>(a, fm, stream);
    case 8: return launch_generic_d<BITS, 8>(a, fm, stream);
    default: return launch_generic_d<BITS, 0>(a, fm, stream);
  }
}

// Steps of k_pq_generic_rows (rounds of sub-vectors x d x 5/4 of the tokens and
// three more for the id and the codeword), weighted by the features beyond a
// round of its waves, up to which it is the faster one: 24 where k_pq_generic
// has d as a constant (32 with 12-bit ids), 76 where it takes a run-time d or
// 12-bit ids at d = 1 (whose runs start at half bytes).  Of 1350 random calls
// around the line 30 were on the slower side, by 20 % at most.
bool rows_faster(const Problem& p) {
  if (p.M > 2 * kRowsTokens || p.N > 16384 || p.d > 16) return false;
  const bool constant_d = p.d == 2 || p.d == 4 || p.d == 8 || (p.d == 1 && p.idx_bits != 12);
  const int64_t most = !constant_d ? 76 : p.idx_bits == 12 ? 32 : 24;
  const int64_t passes = (p.M + kRowsTokens - 1) / kRowsTokens;
  const int64_t tokens = p.M < kRowsTokens ? p.M : kRowsTokens;
  const int64_t steps = passes * ((p.S + kWave - 1) / kWave) * p.d * (tokens * 5 / 4 + 3);
  return steps <= most && steps * p.N <= most * 2048;
}

}  // namespace

hipError_t launch_generic(const Problem& p, const DeviceInfo& dev, hipStream_t stream) {
  if (rows_faster(p)) {
    if (plan_record("k_pq_generic_rows", {p.idx_bits})) return hipSuccess;
    const dim3 grid((unsigned)((p.N + kRowsThreads / kWave - 1) / (kRowsThreads / kWave)));
    const half_t* x = static_cast<const half_t*>(p.x);
    const uint8_t* idx = static_cast<const uint8_t*>(p.idx);
    const half_t* cb = static_cast<const half_t*>(p.codebook);
    half_t* y = static_cast<half_t*>(p.y);
    const int M = (int)p.M;
    switch (p.idx_bits) {
      case 8: return launch_kernel(k_pq_generic_rows<8>, grid, dim3(kRowsThreads), 0, stream, x, M, p.K, p.N, idx, p.R, p.d, cb, p.cb_stride, y);
      case 12: return launch_kernel(k_pq_generic_rows<12>, grid, dim3(kRowsThreads), 0, stream, x, M, p.K, p.N, idx, p.R, p.d, cb, p.cb_stride, y);
      default: return launch_kernel(k_pq_generic_rows<16>, grid, dim3(kRowsThreads), 0, stream, x, M, p.K, p.N, idx, p.R, p.d, cb, p.cb_stride, y);
    }
  }
  if (plan_record("k_pq_generic", {p.idx_bits})) return hipSuccess;
  // token tiles per workgroup: up to four share the gathers, fewer where the
  // grid would leave compute units idle
  const int64_t cols = (p.N + 15) / 16, tiles = (p.M + 15) / 16;
  int fm = (int)(tiles < 4 ? tiles : 4);
  while (fm > 1 && cols * ((tiles + fm - 1) / fm) < dev.num_cus) --fm;
  // then fewer features per workgroup (the gathers are bound per CU)
  int per = 16;
  while (per > 4 && (p.N + per - 1) / per * ((tiles + fm - 1) / fm) <= dev.num_cus / 2) per /= 2;
  // a shared codebook in LDS where a workgroup gathers at least four ids for
  // each 16-byte word it stages (20000 x 24, d = 3: 12 us staged, 6 us from
  // global memory)
  const int64_t cb_bytes = p.C * p.d * 2;
  const bool lcb = p.cb_stride == 0 && cb_bytes <= kGenericLdsBytes && per * p.S >= cb_bytes / 4;
  // calls beyond the grid's limits (65535 in y, 2^32 threads in x) go in pieces
  const int64_t most_m = int64_t(65535) * fm * 16, most_n = (int64_t)per << 20;
  for (int64_t m0 = 0; m0 < p.M; m0 += most_m) {
    for (int64_t n0 = 0; n0 < p.N; n0 += most_n) {
      GenericArgs a;
      a.x = static_cast<const half_t*>(p.x) + m0 * p.K;
      a.M = p.M - m0 < most_m ? p.M - m0 : most_m;
      a.K = p.K;
      a.N = p.N - n0 < most_n ? p.N - n0 : most_n;
      a.idx = static_cast<const uint8_t*>(p.idx) + n0 * p.R;
      a.R = p.R;
      a.d = p.d;
      a.cb = static_cast<const half_t*>(p.codebook);
      a.cbs = p.cb_stride;
      a.y = static_cast<half_t*>(p.y) + m0 * p.N + n0;
      a.ldy = p.N;
      a.cols = per;
      a.cb_bytes = lcb ? (int)cb_bytes : 0;
      hipError_t e;
      switch (p.idx_bits) {
        case 8: e = launch_generic_bits<8>(a, fm, stream); break;
        case 12: e = launch_generic_bits<12>(a, fm, stream); break;
        default: e = launch_generic_bits<16>(a, fm, stream); break;
      }
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace fasq
