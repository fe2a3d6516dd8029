// Prefill GEMM for codebooks gathered from global memory (L2): Y[M x N] =
// X[M x K] . W_hat^T with every W_hat tile decoded once per workgroup.
//
// Bound by the gathers: a CU's address units take one lane of a random read per
// cycle, and from L2 the card serves about half of that (278 G reads/s in a
// probe, 0.45 per cycle and CU).  k_gemm_mfma gathers each B operand
// in every wave row that uses it; here the workgroup decodes the BN x 64 tile
// of each K chunk once into LDS, all waves read their operands from there,
// and a tall tile (BM rows of X for few columns) re-gathers W_hat for few
// row tiles.  4096 x 4096, 65536 entries, d = 4, 512 tokens: 244 -> 61 us; the
// address units are then busy 73 % of the time (half of it the gathers, most
// of the rest the X copy).  Address cycles per chunk and workgroup: BN * 64 / d
// for the gathers plus BM * 128 / 64 for the X copy; the launcher takes the
// tile with the smallest sum over its rounds (a ranking of tiles: the time
// itself is that of the reads from L2).
//
// Pipeline, one chunk of 64 K values per step, NS slots: at step c the
// codewords of chunk c + 1 (gathered since step c + 1 - NS) go to LDS, the
// gathers of chunk c + 1 + NS and the id loads of chunk c + 1 + 2 NS are
// issued, then the X copy of chunk c + NS - 1 (global_load_lds, ring of NS),
// then the MFMAs of chunk c; one barrier per step.  Loads return in order, so
// waiting for the X copy of the next chunk leaves the loads of NS - 2 steps
// in flight.  Chunks past the last one read codeword 0, and the last chunks
// that fill no turn of the ring run without loads.  KG wave groups share the k-steps of a chunk
// where the tile has fewer than eight 32 x 32 blocks; their accumulators are
// added through LDS in group order.
#pragma once

#include "fasq_gemm_mfma.h"

namespace fasq {

constexpr int kGatherWaves = 8;
constexpr int kGatherThreads = kGatherWaves * kWave;
constexpr int kGatherBuffers = 2;   // decoded W_hat tiles

struct GatherTile {
  int bm, bn, kg, ns;
};
constexpr GatherTile kGatherTiles[] = {{256, 64, 1, 4}, {256, 32, 1, 4}, {128, 32, 2, 6}, {64, 32, 4, 8}};
constexpr int kGatherNumTiles = 4;

__host__ __device__ constexpr int gather_lds_bytes(int bm, int bn, int kg, int ns) {
  const int ring = ns * bm * 128 + kGatherBuffers * bn * 128;
  const int dump = (kg - 1) * bm * bn * 4;
  return ring > dump ? ring : dump;
}

hipError_t launch_gemm_gather(const GemmArgs& a, int bits, int d, int tile, hipStream_t stream);

// NB: kGatherBuffers (named in the plan).
template <int BITS, int D, int BM, int BN, int KG, int NS, int NB>
__global__ __launch_bounds__(kGatherThreads) void k_gemm_gather(GemmArgs a) {
  constexpr int WGN = BN / 32;                 // waves over the columns
  constexpr int WGM = kGatherWaves / KG / WGN; // waves over the rows
  constexpr int FM = BM / 32 / WGM;            // 32 x 32 blocks per wave, one below the other
  constexpr int STEPS = 4 / KG;                // k-steps of 16 per wave and chunk
  constexpr int XI = BM / 64;                  // X copies per wave and chunk (8 rows each)
  constexpr int RUN = BN / 8;                  // halves of W_hat each thread decodes per chunk
  constexpr int TPC = 64 / RUN;                // threads per column
  constexpr int IPT = RUN / D > 0 ? RUN / D : 1;       // ids per thread and chunk
  constexpr int HPI = RUN < D ? RUN : D;               // halves taken of each codeword
  constexpr int NW = HPI == 1 ? RUN : RUN / 2;         // dwords per run in flight (single halves: one each)
  constexpr int IDB = (IPT * BITS + 7) / 8;            // id bytes per run (12-bit ids: of an even id, or one id's two)
  static_assert((NS - 2) * (IPT + 1 + XI) < 64, "more loads in flight than the counter holds");
  static_assert(FM >= 1 && RUN % HPI == 0 && RUN * kGatherThreads == BN * 64, "tile does not split over the threads");

  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  uint8_t* xring = smem;
  uint8_t* btile = smem + NS * BM * 128;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const int kg = wave / (kGatherWaves / KG), wk = wave % (kGatherWaves / KG);
  const int wm = wk / WGN, wn = wk % WGN;
  const int h = lane >> 5, l32 = lane & 31;
  const int64_t m0 = (int64_t)blockIdx.y * BM;
  const int64_t n0 = (int64_t)blockIdx.x * BN;
  const int all_chunks = (int)(a.K / kGemmKC);
  const int c_begin = (int)((int64_t)blockIdx.z * all_chunks / a.ksplit);
  const int nchunks = (int)((int64_t)(blockIdx.z + 1) * all_chunks / a.ksplit) - c_begin;
  auto chunk_of = [&](int c) { return c_begin + (c < nchunks ? c : nchunks - 1); };

  // X copies: rows past M read row M - 1 (computed, never stored)
  const half_t* xsrc[XI];
#pragma unroll
  for (int j = 0; j < XI; ++j) {
    const int r = (wave * XI + j) * 8 + lane / 8;
    const int g = (lane % 8) ^ ((r >> 1) & 7);
    const int64_t m = m0 + r;
    xsrc[j] = a.x + (m < a.M ? m : a.M - 1) * a.K + g * 8;
  }
  auto copy_x = [&](int c, int stage) {
    const int64_t k = (int64_t)chunk_of(c) * kGemmKC;
#pragma unroll
    for (int j = 0; j < XI; ++j)
      copy16_to_lds(xsrc[j] + k, xring + stage * (BM * 128) + (wave * XI + j) * 8 * 128);
  };

  // W_hat: this thread decodes halves [part * RUN, part * RUN + RUN) of column
  // `col` of each chunk (columns past N read column 0)
  const int col = tid / TPC, part = tid % TPC;
  const uint8_t* idrow = a.idx + (n0 + col < a.N ? n0 + col : 0) * a.R;
  const int bdst = col * 128 + (((part * RUN) / 8) ^ ((col >> 1) & 7)) * 16 + (part * RUN) % 8 * 2;
  // Ids and codewords stay as their loads leave them until they are used, steps
  // later: arithmetic on them here would wait for the load.
  struct Ids {
    uint32_t w[IDB == 3 ? 2 : (IDB + 3) / 4];
  };
  const int odd = BITS == 12 && IPT == 1 ? (part * RUN / D & 1) * 4 : 0;  // the id starts at half a byte
  auto load_ids = [&](Ids& o, int c) {
    const int s = chunk_of(c) * (kGemmKC / D) + part * RUN / D;  // first id of the run
    const uint8_t* at = idrow + (int64_t)s * BITS / 8;
    if constexpr (IDB == 3) {
      o.w[0] = 0;
      __builtin_memcpy(o.w, at, 2);
      o.w[1] = at[2];
    } else {
      o.w[(IDB + 3) / 4 - 1] = 0;
      __builtin_memcpy(o.w, at, IDB);
    }
  };
  struct Words {
    uint32_t w[NW];
  };
  // The codewords of chunk c.  Past the last chunk every lane reads codeword 0:
  // the loads the waits count stay, the random reads don't.
  auto gather_run = [&](Words& o, const Ids& ids, int c) {
    uint32_t w[(IDB + 3) / 4];
#pragma unroll
    for (int i = 0; i < (IDB + 3) / 4; ++i) {
      const uint32_t raw = IDB == 3 ? ids.w[0] | (ids.w[1] << 16) : ids.w[i] >> odd;
      w[i] = raw & (c < nchunks ? ~0u : 0u);
    }
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const half_t* src = a.cb + (size_t)stream_id<BITS>(w, i) * D + (RUN < D ? part * RUN % D : 0);
      if constexpr (HPI == 1) {
        o.w[i] = *reinterpret_cast<const uint16_t*>(src);
      } else if constexpr (HPI == 2) {
        o.w[i] = *reinterpret_cast<const uint32_t*>(src);
      } else if constexpr (HPI == 4) {
        const u32x2 v = *reinterpret_cast<const u32x2*>(src);
        o.w[2 * i] = v[0]; o.w[2 * i + 1] = v[1];
      } else {
        const u32x4 v = *reinterpret_cast<const u32x4*>(src);
        o.w[0] = v[0]; o.w[1] = v[1]; o.w[2] = v[2]; o.w[3] = v[3];
      }
    }
  };
  auto store_run = [&](const Words& o, int buffer) {
    uint8_t* p = btile + buffer * (BN * 128) + bdst;
    uint32_t v[RUN / 2];
#pragma unroll
    for (int i = 0; i < RUN / 2; ++i) v[i] = HPI == 1 ? o.w[2 * i] | (o.w[2 * i + 1] << 16) : o.w[i];
    if constexpr (RUN == 4) *reinterpret_cast<u32x2*>(p) = u32x2{v[0], v[1]};
    else *reinterpret_cast<u32x4*>(p) = u32x4{v[0], v[1], v[2], v[3]};
  };

  float16_t acc[FM];
#pragma unroll
  for (int f = 0; f < FM; ++f)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[f][i] = 0.f;

  // prologue: chunk 0 goes to LDS; then slot q % NS of the codewords holds
  // chunk q for q = 1 .. NS, that of the ids chunk q + NS
  Ids ids[NS];
  Words cw[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) load_ids(ids[q], q);
#pragma unroll
  for (int q = 0; q < NS - 1; ++q) copy_x(q, q);
#pragma unroll
  for (int q = 0; q < NS; ++q) {
    gather_run(cw[q], ids[q], q);
    load_ids(ids[q], q + NS);
  }
  store_run(cw[0], 0);
  gather_run(cw[0], ids[0], NS);
  load_ids(ids[0], 2 * NS);
  wait_vmcnt<0>();
  wait_lgkmcnt0();
  __builtin_amdgcn_s_barrier();

  // chunk c from ring slot u = c % NS
  auto multiply = [&](int c, int u) __attribute__((always_inline)) {
    const uint8_t* xb = xring + u * (BM * 128);
    const uint8_t* bb = btile + (c % NB) * (BN * 128);
    const int bc = wn * 32 + l32;
    half8_t av[STEPS][FM], bv[STEPS];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int g = (s * KG + kg) * 2 + h;  // 16-byte granule of the row
      bv[s] = *reinterpret_cast<const half8_t*>(bb + bc * 128 + (g ^ ((bc >> 1) & 7)) * 16);
#pragma unroll
      for (int f = 0; f < FM; ++f) {
        const int r = (wm * FM + f) * 32 + l32;
        av[s][f] = *reinterpret_cast<const half8_t*>(xb + r * 128 + (g ^ ((r >> 1) & 7)) * 16);
      }
    }
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int f = 0; f < FM; ++f)
        acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[s][f], bv[s], acc[f], 0, 0, 0);
  };
  int c0 = 0;
  for (; c0 + NS <= nchunks; c0 += NS) {  // whole turns of the ring
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int c = c0 + u;
      const int slot = (u + 1) % NS;  // of chunks c + 1, c + 1 + NS, c + 1 + 2 NS
      store_run(cw[slot], (c + 1) % NB);
      gather_run(cw[slot], ids[slot], c + 1 + NS);
      load_ids(ids[slot], c + 1 + 2 * NS);
      copy_x(c + NS - 1, (u + NS - 1) % NS);
      __builtin_amdgcn_sched_barrier(0);
      multiply(c, u);
      __builtin_amdgcn_sched_barrier(0);
      // this wave's X copies of chunk c + 1 (after them each of NS - 2 steps
      // issued at least IPT gathers, one id load and XI copies) and its
      // decoded run
      wait_vmcnt<(NS - 2) * (IPT + 1 + XI)>();
      wait_lgkmcnt0();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  wait_vmcnt<0>();  // what is left is in the ring and the registers (the clamped copies past it too)
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int u = 0; u < NS - 1; ++u) {  // fewer chunks than a turn
    if (c0 + u >= nchunks) break;
    store_run(cw[u + 1], (c0 + u + 1) % NB);
    multiply(c0 + u, u);
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
  }

  if constexpr (KG > 1) {
    // groups 1 .. KG - 1 leave their accumulators in LDS, group 0 adds them in order
    float4_t* dump = reinterpret_cast<float4_t*>(smem);
    constexpr int GW = kGatherWaves / KG;
    auto slot = [&](int g, int f, int i4) { return ((((g - 1) * GW + wk) * FM + f) * 4 + i4) * kWave + lane; };
    __syncthreads();
    if (kg > 0) {
#pragma unroll
      for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          dump[slot(kg, f, i4)] = float4_t{acc[f][4 * i4], acc[f][4 * i4 + 1], acc[f][4 * i4 + 2], acc[f][4 * i4 + 3]};
    }
    __syncthreads();
    if (kg > 0) return;
    for (int g = 1; g < KG; ++g) {
#pragma unroll
      for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const float4_t v = dump[slot(g, f, i4)];
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[f][4 * i4 + k] += v[k];
        }
    }
  }

  float* partial = a.ws + (int64_t)blockIdx.z * a.M * a.N;
  const int64_t n = n0 + wn * 32 + l32;
  if (n >= a.N) return;
#pragma unroll
  for (int f = 0; f < FM; ++f) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int64_t m = m0 + (wm * FM + f) * 32 + (i / 4) * 8 + h * 4 + (i % 4);
      if (m >= a.M) continue;
      if (a.ksplit > 1) partial[m * a.N + n] = acc[f][i];
      else a.y[m * a.N + n] = static_cast<half_t>(acc[f][i]);
    }
  }
}

}  // namespace fasq
