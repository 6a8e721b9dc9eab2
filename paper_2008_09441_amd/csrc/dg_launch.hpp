// Launchers of the order-templated kernels.  Each order's kernels are
// compiled in a translation unit of their own (dg_stage.hip with DG_ORDER
// set), so that a build compiles the orders in parallel; callers see only
// these declarations.
#pragma once
#include <hip/hip_runtime.h>

#include "dg_adjt.hpp"
#include "dg_batch.hpp"
#include "dg_be.hpp"
#include "dg_bt.hpp"
#include "dg_bx.hpp"

namespace dgl {

// orders 1-4: `grid` element tiles
template <int N, bool F32>
hipError_t stage_bx(const dgb::BxArgs& A, unsigned grid, hipStream_t st);
template <int N>
hipError_t stage_bx_p(const dgb::BxArgs& A, unsigned grid, hipStream_t st);
template <int N>
hipError_t stage_bx_r(const dgb::BxArgs& A, unsigned grid, hipStream_t st);
template <int N>
hipError_t stage_bx_d(const dgb::BxArgsT<double>& A, unsigned grid, hipStream_t st);
template <int N>
hipError_t adj_tile(const dgt::TileArgs& A, unsigned grid, hipStream_t st);
// `grid` elements: orders 5-7 (FP64: 2-7)
template <int N, bool F32>
hipError_t stage_be(const dgb::BeArgs& A, unsigned grid, hipStream_t st);
template <int N>
hipError_t stage_be_d(const dgb::BeArgsT<double>& A, unsigned grid, hipStream_t st);
// orders 5-7 (FP32: 5 and 6): `grid` element tiles
template <int N, bool F32>
hipError_t stage_bt(const dgb::BeArgs& A, unsigned grid, hipStream_t st);
// one stage of a batch of order N over `grid` launch positions: slots whose
// stage runs on element tiles, or (orders 5-7) on one element per workgroup
template <int N, bool F32>
hipError_t stage_batch(const dgb::BatchSlot* table, int n, unsigned grid, bool tiles,
                       hipStream_t st, int par, float a, float b);

}  // namespace dgl
