// Kernels of one order (DG_ORDER, 1-7) and their launchers, in several units
// per order (DG_PART).
#include "dg_launch.hpp"

#if !defined(DG_ORDER) || !defined(DG_PART)
#error "compile with -DDG_ORDER=<order> -DDG_PART=<part>"
#endif

namespace dgl {

template <int N, bool F32>
hipError_t stage_bx(const dgb::BxArgs& A, unsigned grid, hipStream_t st) {
  dgb::stage_bx<N, F32><<<dim3(grid), dim3(dgb::kThreads), 0, st>>>(A);
  return hipGetLastError();
}

template <int N>
hipError_t stage_bx_p(const dgb::BxArgs& A, unsigned grid, hipStream_t st) {
  dgb::stage_bx_p<N><<<dim3(grid), dim3(dgb::kThreads), 0, st>>>(A);
  return hipGetLastError();
}

template <int N>
hipError_t stage_bx_r(const dgb::BxArgs& A, unsigned grid, hipStream_t st) {
  dgb::stage_bx_r<N><<<dim3(grid), dim3(dgb::kThreads), 0, st>>>(A);
  return hipGetLastError();
}

template <int N>
hipError_t stage_bx_d(const dgb::BxArgsT<double>& A, unsigned grid, hipStream_t st) {
  dgb::stage_bx_d<N><<<dim3(grid), dim3(dgb::kThreads), 0, st>>>(A);
  return hipGetLastError();
}

template <int N>
hipError_t adj_tile(const dgt::TileArgs& A, unsigned grid, hipStream_t st) {
  dgt::adj_tile<N, true><<<dim3(grid), dim3(dgt::kThreads), 0, st>>>(A);
  return hipGetLastError();
}

template <int N, bool F32>
hipError_t stage_be(const dgb::BeArgs& A, unsigned grid, hipStream_t st) {
  dgb::stage_be<N, F32><<<dim3(grid), dim3(dgb::kThreads), 0, st>>>(A);
  return hipGetLastError();
}

template <int N, bool F32>
hipError_t stage_bt(const dgb::BeArgs& A, unsigned grid, hipStream_t st) {
  if constexpr (F32 && N > 6) {
    return hipErrorInvalidValue;
  } else {
    constexpr int P = F32 ? 3 : 2;
    dgb::stage_bt<N, P><<<dim3(grid), dim3(dgb::TOrd<N, P>::TH), 0, st>>>(A);
    return hipGetLastError();
  }
}

template <int N>
hipError_t stage_be_d(const dgb::BeArgsT<double>& A, unsigned grid, hipStream_t st) {
  dgb::stage_be_d<N><<<dim3(grid), dim3(dgb::kThreads), 0, st>>>(A);
  return hipGetLastError();
}

template <int N, bool F32>
hipError_t stage_batch(const dgb::BatchSlot* table, int n, unsigned grid, bool tiles,
                       hipStream_t st, int par, float a, float b) {
  if constexpr (N <= 4) {
    if (!tiles) return hipErrorInvalidValue;
    dgb::stage_bx_batch<N, F32><<<dim3(grid), dim3(dgb::kThreads), 0, st>>>(table, n, par, a, b);
  } else if (!tiles) {
    dgb::stage_be_batch<N, F32><<<dim3(grid), dim3(dgb::kThreads), 0, st>>>(table, n, par, a, b);
  } else if constexpr (F32 && N > 6) {
    return hipErrorInvalidValue;
  } else {
    constexpr int P = F32 ? 3 : 2;
    dgb::stage_bt_batch<N, P>
        <<<dim3(grid), dim3(dgb::TOrd<N, P>::TH), 0, st>>>(table, n, par, a, b);
  }
  return hipGetLastError();
}

// DG_PART picks the kernels of a unit: 0 BF16x3, 1 FP32, 2 FP64, 3 the stages
// and the tile kernel of the adjoint
#define DG_INST template hipError_t
#if DG_PART < 2
DG_INST stage_batch<DG_ORDER, DG_PART == 1>(const dgb::BatchSlot*, int, unsigned, bool, hipStream_t,
                                            int, float, float);
#elif DG_PART == 2 && DG_ORDER >= 2
DG_INST stage_be_d<DG_ORDER>(const dgb::BeArgsT<double>&, unsigned, hipStream_t);
#endif
#if DG_ORDER <= 4
#if DG_PART < 2
DG_INST stage_bx<DG_ORDER, DG_PART == 1>(const dgb::BxArgs&, unsigned, hipStream_t);
#elif DG_PART == 2
DG_INST stage_bx_d<DG_ORDER>(const dgb::BxArgsT<double>&, unsigned, hipStream_t);
#else
#if DG_ORDER >= 3
DG_INST stage_bx_p<DG_ORDER>(const dgb::BxArgs&, unsigned, hipStream_t);
#endif
DG_INST stage_bx_r<DG_ORDER>(const dgb::BxArgs&, unsigned, hipStream_t);
DG_INST adj_tile<DG_ORDER>(const dgt::TileArgs&, unsigned, hipStream_t);
#endif
#elif DG_PART < 2
DG_INST stage_be<DG_ORDER, DG_PART == 1>(const dgb::BeArgs&, unsigned, hipStream_t);
DG_INST stage_bt<DG_ORDER, DG_PART == 1>(const dgb::BeArgs&, unsigned, hipStream_t);
#endif
#undef DG_INST

}  // namespace dgl
