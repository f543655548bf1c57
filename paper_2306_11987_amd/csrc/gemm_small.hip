// GEMMs of HQ-MM and LSS-MM on 64-row tiles, for products too small to fill the device with
// the 128-row tiles of gemm.hip (short batches, small layers).
//
// Such a product is bound by latency: a CU holds one workgroup, which waits for every stage
// of its operands.  Tiles of 64 x 64 (64 x 128 for Hadamard blocks of 128, which a wave's
// tile must hold) give up to four times as many workgroups of two waves, and six stage
// buffers (four for 64 x 128 int8 tiles; 48 to 72 KB of LDS) keep five stages of loads (three)
// in flight instead of one or two
// (16 x 1024 -> 4096, b = 128, eight stages: 8.1 -> 5.9 us; 128 x 256 -> 256: forward 5.1 ->
// 4.5, dX 6.0 -> 5.4, dW 5.2 -> 4.5 us).
// Kernel, epilogues and results are those of gemm_kernel.h.
#include "gemm_kernel.h"

namespace hqlss {

namespace {

template <bool A4, int EPI, int DT, bool TRA>
hipError_t small_b(hipStream_t s, const GemmArgs& g, int id) {
  if constexpr (EPI == kEpiFwd || EPI == kEpiAcc) {
    return gemm_t<kSmallBM, A4, EPI, DT, 0, kNarrowBN, false, 0, TRA>(s, g, 1, id);
  } else {
    switch (g.log2b) {
      case 0: return gemm_t<kSmallBM, A4, EPI, DT, 0, kNarrowBN, false, 0, TRA>(s, g, 1, id);
      case 1: return gemm_t<kSmallBM, A4, EPI, DT, 1, kNarrowBN, false, 0, TRA>(s, g, 1, id);
      case 2: return gemm_t<kSmallBM, A4, EPI, DT, 2, kNarrowBN, false, 0, TRA>(s, g, 1, id);
      case 3: return gemm_t<kSmallBM, A4, EPI, DT, 3, kNarrowBN, false, 0, TRA>(s, g, 1, id);
      case 4: return gemm_t<kSmallBM, A4, EPI, DT, 4, kNarrowBN, false, 0, TRA>(s, g, 1, id);
      case 5: return gemm_t<kSmallBM, A4, EPI, DT, 5, kNarrowBN, false, 0, TRA>(s, g, 1, id);
      case 6: return gemm_t<kSmallBM, A4, EPI, DT, 6, kNarrowBN, false, 0, TRA>(s, g, 1, id);
      case 7: return gemm_t<kSmallBM, A4, EPI, DT, 7, kMidBN, false, 0, TRA>(s, g, 1, id);
    }
    return hipErrorInvalidValue;
  }
}

template <bool A4, int EPI, bool TRA = false>
hipError_t small_dt(hipStream_t s, int dt, const GemmArgs& g, int id) {
  switch (dt) {
    case kF32: return small_b<A4, EPI, kF32, TRA>(s, g, id);
    case kF16: return small_b<A4, EPI, kF16, TRA>(s, g, id);
    case kBF16: return small_b<A4, EPI, kBF16, TRA>(s, g, id);
  }
  return hipErrorInvalidValue;
}

}  // namespace

int gemm_small_bn(int log2b) { return log2b == 7 ? kMidBN : kNarrowBN; }

hipError_t launch_gemm_small(hipStream_t s, int epi, int dt, bool a_int4, const GemmArgs& g) {
  if (a_int4) {
    if (epi == kEpiFwd) return small_dt<true, kEpiFwd>(s, dt, g, kKGemmFwd);
    return epi == kEpiAcc ? small_b<true, kEpiAcc, kF32, false>(s, g, kKGemmAcc) : hipErrorInvalidValue;
  }
  switch (epi) {
    case kEpiAcc:
      return g.a_kmajor ? small_b<false, kEpiAcc, kF32, true>(s, g, kKGemmAcc)
                        : small_b<false, kEpiAcc, kF32, false>(s, g, kKGemmAcc);
    case kEpiDx: return small_dt<false, kEpiDx>(s, dt, g, kKGemmDx);
    case kEpiDxL: return small_dt<false, kEpiDxL>(s, dt, g, kKGemmDx);
    case kEpiDw: return small_dt<false, kEpiDw, true>(s, dt, g, kKGemmDw);
    case kEpiDwL: return small_dt<false, kEpiDwL, true>(s, dt, g, kKGemmDw);
  }
  return hipErrorInvalidValue;
}

}  // namespace hqlss
