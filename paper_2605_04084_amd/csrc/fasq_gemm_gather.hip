// Prefill GEMM over codebooks in global memory: instantiations and launch.
#include "fasq_gemm_gather.h"

namespace fasq {

namespace {

template <int BITS, int D, int T>
hipError_t launch_tile(const GemmArgs& a, hipStream_t stream) {
  constexpr GatherTile t = kGatherTiles[T];
  auto kern = k_gemm_gather<BITS, D, t.bm, t.bn, t.kg, t.ns, kGatherBuffers>;
  if (plan_record("k_gemm_gather", {BITS, D, t.bm, t.bn, t.kg, t.ns, kGatherBuffers})) return hipSuccess;
  hipError_t e = prepare_kernel(kern);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((a.N + t.bn - 1) / t.bn), (unsigned)((a.M + t.bm - 1) / t.bm), (unsigned)a.ksplit);
  return launch_kernel(kern, grid, dim3(kGatherThreads), gather_lds_bytes(t.bm, t.bn, t.kg, t.ns), stream, a);
}

template <int BITS, int D>
hipError_t launch_d(const GemmArgs& a, int tile, hipStream_t stream) {
  switch (tile) {
    case 0: return launch_tile<BITS, D, 0>(a, stream);
    case 1: return launch_tile<BITS, D, 1>(a, stream);
    case 2: return launch_tile<BITS, D, 2>(a, stream);
    default: return launch_tile<BITS, D, 3>(a, stream);
  }
}

template <int BITS>
hipError_t launch_bits(const GemmArgs& a, int d, int tile, hipStream_t stream) {
  switch (d) {
    case 1: return launch_d<BITS, 1>(a, tile, stream);
    case 2: return launch_d<BITS, 2>(a, tile, stream);
    case 4: return launch_d<BITS, 4>(a, tile, stream);
    default:
      if constexpr (BITS == 12) return hipErrorNotSupported;  // the GEMM's plan declines d = 8 with 12-bit ids
      else return launch_d<BITS, 8>(a, tile, stream);
  }
}

}  // namespace

hipError_t launch_gemm_gather(const GemmArgs& a, int bits, int d, int tile, hipStream_t stream) {
  switch (bits) {
    case 8: return launch_bits<8>(a, d, tile, stream);
    case 12: return launch_bits<12>(a, d, tile, stream);
    default: return launch_bits<16>(a, d, tile, stream);
  }
}

}  // namespace fasq
