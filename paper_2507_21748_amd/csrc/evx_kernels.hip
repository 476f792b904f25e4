// __global__ wrappers of the pass bodies for one transform length.  This file is compiled once
// per supported length (EVX_INST_N) so the instantiations build in parallel; each object exports
// evx_launch_col_<N> and evx_launch_row_<N> (and their batched forms evx_launch_colb_<N>,
// evx_launch_rowb_<N>).
#include "evx_launch.hpp"

#ifndef EVX_INST_N
#error "compile with -DEVX_INST_N=<transform length>"
#endif

namespace evx {

// Workgroups of 8192 points (length 1024: 512 lanes of 16) fit a compute unit twice only below 129
// VGPRs, four waves a SIMD; the compiler is held to that (at most five registers spill, in the rarer
// forms), since one workgroup alone waits for its own loads.  Length 512 (512 lanes of 8 points) is
// left alone: held to it, a 512 x 256 x 256 zero-flux step took 230.2 us, without 228.2.
// Lanes of 20 points in the periodic family are held to three waves a SIMD, 168 VGPRs: with the update's
// coefficients shared (one or two registers more) they fell to two, and the z pass of 100 x 256 x 256
// took 29.1 us instead of 23.3, of 320 x 256 x 256 64.1 instead of 57.9.  (The cosine family, which does
// not share, spills when it is held: Allen-Cahn steps of 400 x 100 x 400 5% slower.  So do lanes of 12
// points held to five waves instead of four: 192 x 256 x 256 36 -> 41 us.)
template <int N, int BC>
constexpr int col_min_waves() {
  if (ColCfg<N>::B * N >= 8192) return 4;
  return ColCfg<N>::E == 20 && BC == BC_PERIODIC ? 3 : 1;
}

template <int N, int BC, int MODE, int SEQS = ColCfg<N>::B>
__global__ __launch_bounds__((ColCfg<N, SEQS>::THREADS), (col_min_waves<N, BC>())) void col_kernel(
    ColArgs a) {
  __shared__ float2 lds[ColCfg<N, SEQS>::LDS];
  colpass_body<N, BC, MODE, SEQS>(a, threadIdx.x, blockIdx.x, gridDim.x, lds);
}

// the same passes over a batch of buffer pairs (grid.y = pair)
template <int N, int BC, int MODE>
__global__ __launch_bounds__(ColCfg<N>::THREADS) void col_kernel_batch(ColArgs a, PassBatch p) {
  __shared__ float2 lds[ColCfg<N>::LDS];
  bind_batch(a, p, blockIdx.y);
  colpass_body<N, BC, MODE>(a, threadIdx.x, blockIdx.x, gridDim.x, lds);
}

template <int NH, int BC>
constexpr int row_threads() {
  return RowCfg<NH, BC>::THREADS;
}

template <int NH, int BC, int MODE, bool STAGED = false>
__global__ __launch_bounds__((row_threads<NH, BC>())) void row_kernel(RowArgs a) {
  __shared__ float2 lds[RowCfg<NH, BC>::LDS];
  rowpass_body<NH, BC, MODE, STAGED>(a, threadIdx.x, blockIdx.x, gridDim.x, lds);
}

template <int NH, int BC, int MODE>
__global__ __launch_bounds__((row_threads<NH, BC>())) void row_kernel_batch(RowArgs a, PassBatch p) {
  __shared__ float2 lds[RowCfg<NH, BC>::LDS];
  bind_batch(a, MODE == ROW_INV, p, blockIdx.y);
  rowpass_body<NH, BC, MODE>(a, threadIdx.x, blockIdx.x, gridDim.x, lds);
}

// the two-species fused x pass (RowArgs::gs)
template <int NH, int BC, int MODE>
__global__ __launch_bounds__((row_threads<NH, BC>())) void row_gs_kernel(RowArgs a) {
  __shared__ float2 lds[RowCfg<NH, BC>::LDS];
  rowpass_gs_body<NH, BC, MODE>(
      a, threadIdx.x, (long long)remap_block(blockIdx.x, gridDim.x, a.remap) * RowCfg<NH, BC>::B,
      lds);
}

// the adjoint step's inverse x pass (RowArgs::comb)
template <int NH>
__global__ __launch_bounds__((row_threads<NH, BC_PERIODIC>())) void row_comb_kernel(RowArgs a) {
  __shared__ float2 lds[RowCfg<NH, BC_PERIODIC>::LDS];
  rowpass_comb_body<NH>(
      a, threadIdx.x,
      (long long)remap_block(blockIdx.x, gridDim.x, a.remap) * RowCfg<NH, BC_PERIODIC>::ROWS, lds);
}

// One workgroup per z plane (small periodic grids; see planepass_body).
template <int NY, int NH>
constexpr int plane_threads() {
  return PlaneCfg<NY, NH>::THREADS;
}

template <int NY, int NH>
__global__ __launch_bounds__((plane_threads<NY, NH>())) void plane_kernel(PlaneArgs a) {
  __shared__ float2 lds[PlaneCfg<NY, NH>::LDS];
  planepass_body<NY, NH>(a, threadIdx.x, blockIdx.x, lds);
}

template <int NY>
static hipError_t plane_go(const PlaneArgs& a, hipStream_t s) {
  using C = PlaneCfg<NY, NY / 2>;
  if (a.nz <= 0) return hipSuccess;
  if (a.sg.ny != NY || a.ngx != (NY / 2 + 1 + 7) / 8) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((plane_kernel<NY, NY / 2>), dim3(unsigned(a.nz)), dim3(C::THREADS), 0, s, a);
  return hipGetLastError();
}

// the forward z pass that goes on with the spectral work (ColArgs::sp)
// (two waves a SIMD at least: length 100 zero flux took one register too many for that)
template <int N, int BC, int MODE>
__global__ __launch_bounds__(ColCfg<N>::THREADS, 2) void colspec_kernel(ColArgs a) {
  __shared__ float2 lds[ColCfg<N>::LDS];
  colspec_body<N, BC, MODE>(a, threadIdx.x, blockIdx.x, gridDim.x, lds);
}

template <int N, int BC, int MODE>
static hipError_t col_go(const ColArgs& a, hipStream_t s) {
  using C = ColCfg<N>;
  if constexpr (MODE == COL_Z_VM) {
    if (a.state) return col_go<N, BC, COL_Z_GS>(a, s);
  }
  const long long nblk = (a.nseq + C::B - 1) / C::B;
  if (nblk <= 0) return hipSuccess;
  constexpr int WIDE = wide_seqs<N>();
  if constexpr (WIDE != C::B) {
    if (col_wide<N>(a) && a.sp.mode == SP_NONE) {
      const long long lane_bytes = col_lane_bytes<N, WIDE>(a), nwide = (a.nseq + WIDE - 1) / WIDE;
      if (nwide > 0x7fffffffLL || a.nseq > 0x7fffffffLL || lane_bytes >= (long long)kDeadLane)
        return hipErrorInvalidConfiguration;
      ColArgs b = a;
      b.lane_bytes = unsigned(lane_bytes);
      hipLaunchKernelGGL((col_kernel<N, BC, MODE, WIDE>), dim3(unsigned(nwide)),
                         dim3(ColCfg<N, WIDE>::THREADS), 0, s, b);
      return hipGetLastError();
    }
  }
  // 32-bit sequence numbers and lane byte offsets (ColTile)
  const long long lane_bytes = col_lane_bytes<N>(a);
  if (nblk > 0x7fffffffLL || a.nseq > 0x7fffffffLL || lane_bytes >= (long long)kDeadLane)
    return hipErrorInvalidConfiguration;
  ColArgs b = a;
  b.lane_bytes = unsigned(lane_bytes);
  if constexpr (MODE == COL_FWD) {
    if (a.sp.mode != SP_NONE) {
      if (a.vlen || a.in != a.out) return hipErrorInvalidValue;
      if (a.sp.mode == SP_ADJOINT)
        hipLaunchKernelGGL((colspec_kernel<N, BC, SP_ADJOINT>), dim3(unsigned(nblk)),
                           dim3(C::THREADS), 0, s, b);
      else
        hipLaunchKernelGGL((colspec_kernel<N, BC, SP_ENERGY>), dim3(unsigned(nblk)),
                           dim3(C::THREADS), 0, s, b);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((col_kernel<N, BC, MODE>), dim3(unsigned(nblk)), dim3(C::THREADS), 0, s, b);
  return hipGetLastError();
}

template <int NH, int BC, int MODE>
static hipError_t row_go(const RowArgs& a, hipStream_t s) {
  using C = RowCfg<NH, BC>;
  const long long nblk = (a.nrows + C::ROWS - 1) / C::ROWS;
  if (nblk <= 0) return hipSuccess;
  if (nblk > 0x7fffffffLL || !row_fits32<NH, BC>(a)) return hipErrorInvalidConfiguration;
  if constexpr (MODE == ROW_FUSED_POLY || MODE == ROW_FWD) {
    if (a.gs) {
      const long long ngs = (a.nrows + C::B - 1) / C::B;
      if (ngs > 0x7fffffffLL) return hipErrorInvalidConfiguration;
      hipLaunchKernelGGL((row_gs_kernel<NH, BC, MODE>), dim3(unsigned(ngs)), dim3(C::THREADS), 0,
                         s, a);
      return hipGetLastError();
    }
  }
  if constexpr (MODE == ROW_INV) {
    if (a.comb) {
      if (BC != BC_PERIODIC || a.vx) return hipErrorInvalidValue;
      hipLaunchKernelGGL((row_comb_kernel<NH>), dim3(unsigned(nblk)),
                         dim3(RowCfg<NH, BC_PERIODIC>::THREADS), 0, s, a);
      return hipGetLastError();
    }
  }
  if constexpr (C::SHORT) {
    if (row_staged<NH, BC>(a)) {
      hipLaunchKernelGGL((row_kernel<NH, BC, MODE, true>), dim3(unsigned(nblk)), dim3(C::THREADS), 0,
                         s, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((row_kernel<NH, BC, MODE>), dim3(unsigned(nblk)), dim3(C::THREADS), 0, s, a);
  return hipGetLastError();
}

// Batched launches check every pair's buffers like the single ones (the geometry is shared).
template <int N, int BC, int MODE>
static hipError_t col_go_batch(const ColArgs& a, const PassBatch& p, hipStream_t s) {
  using C = ColCfg<N>;
  if constexpr (MODE == COL_Z_VM) {
    if (p.state[0]) return col_go_batch<N, BC, COL_Z_GS>(a, p, s);
  }
  const long long nblk = (a.nseq + C::B - 1) / C::B;
  if (nblk <= 0) return hipSuccess;
  if (p.n < 1 || p.n > kMaxBatch) return hipErrorInvalidValue;
  const long long lane_bytes = col_lane_bytes<N>(a);
  if (nblk > 0x7fffffffLL || a.nseq > 0x7fffffffLL || lane_bytes >= (long long)kDeadLane)
    return hipErrorInvalidConfiguration;
  ColArgs b = a;
  b.lane_bytes = unsigned(lane_bytes);
  hipLaunchKernelGGL((col_kernel_batch<N, BC, MODE>), dim3(unsigned(nblk), unsigned(p.n)),
                     dim3(C::THREADS), 0, s, b, p);
  return hipGetLastError();
}

template <int NH, int BC, int MODE>
static hipError_t row_go_batch(const RowArgs& a, const PassBatch& p, hipStream_t s) {
  using C = RowCfg<NH, BC>;
  const long long nblk = (a.nrows + C::ROWS - 1) / C::ROWS;
  if (nblk <= 0) return hipSuccess;
  if (p.n < 1 || p.n > kMaxBatch) return hipErrorInvalidValue;
  if (nblk > 0x7fffffffLL || !row_fits32<NH, BC>(a)) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((row_kernel_batch<NH, BC, MODE>), dim3(unsigned(nblk), unsigned(p.n)),
                     dim3(C::THREADS), 0, s, a, p);
  return hipGetLastError();
}

template <int N, int BC>
static hipError_t col_mode(int mode, const ColArgs& a, hipStream_t s) {
  switch (mode) {
    case COL_FWD: return col_go<N, BC, COL_FWD>(a, s);
    case COL_INV: return col_go<N, BC, COL_INV>(a, s);
    case COL_Z_INIT: return col_go<N, BC, COL_Z_INIT>(a, s);
    case COL_Z_UPDATE: return col_go<N, BC, COL_Z_UPDATE>(a, s);
    case COL_Z_INV_STATE: return col_go<N, BC, COL_Z_INV_STATE>(a, s);
    case COL_Z_ETD: return col_go<N, BC, COL_Z_ETD>(a, s);
    case COL_Z_AC: return col_go<N, BC, COL_Z_AC>(a, s);
    case COL_Z_AC_ETD: return col_go<N, BC, COL_Z_AC_ETD>(a, s);
    case COL_Z_VM: return col_go<N, BC, COL_Z_VM>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int NH, int BC>
static hipError_t row_mode(int mode, const RowArgs& a, hipStream_t s) {
  switch (mode) {
    case ROW_FUSED: return row_go<NH, BC, ROW_FUSED>(a, s);
    case ROW_FWD: return row_go<NH, BC, ROW_FWD>(a, s);
    case ROW_INV: return row_go<NH, BC, ROW_INV>(a, s);
    case ROW_INV_ADD: return row_go<NH, BC, ROW_INV_ADD>(a, s);
    case ROW_FUSED_REC: return row_go<NH, BC, ROW_FUSED_REC>(a, s);
    case ROW_FUSED_POLY: return row_go<NH, BC, ROW_FUSED_POLY>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int N, int BC>
static hipError_t col_mode_batch(int mode, const ColArgs& a, const PassBatch& p, hipStream_t s) {
  switch (mode) {
    case COL_FWD: return col_go_batch<N, BC, COL_FWD>(a, p, s);
    case COL_INV: return col_go_batch<N, BC, COL_INV>(a, p, s);
    case COL_Z_VM: return col_go_batch<N, BC, COL_Z_VM>(a, p, s);
    default: return hipErrorInvalidValue;
  }
}

template <int NH, int BC>
static hipError_t row_mode_batch(int mode, const RowArgs& a, const PassBatch& p, hipStream_t s) {
  switch (mode) {
    case ROW_FWD: return row_go_batch<NH, BC, ROW_FWD>(a, p, s);
    case ROW_INV: return row_go_batch<NH, BC, ROW_INV>(a, p, s);
    default: return hipErrorInvalidValue;
  }
}

#define EVX_PASTE2(a, b) a##b
#define EVX_PASTE(a, b) EVX_PASTE2(a, b)

hipError_t EVX_PASTE(evx_launch_col_, EVX_INST_N)(int bc, int mode, const ColArgs& a,
                                                  hipStream_t s) {
  return bc == BC_PERIODIC ? col_mode<EVX_INST_N, BC_PERIODIC>(mode, a, s)
                           : col_mode<EVX_INST_N, BC_ZERO_FLUX>(mode, a, s);
}

hipError_t EVX_PASTE(evx_launch_row_, EVX_INST_N)(int bc, int mode, const RowArgs& a,
                                                  hipStream_t s) {
  return bc == BC_PERIODIC ? row_mode<EVX_INST_N, BC_PERIODIC>(mode, a, s)
                           : row_mode<EVX_INST_N, BC_ZERO_FLUX>(mode, a, s);
}

hipError_t EVX_PASTE(evx_launch_colb_, EVX_INST_N)(int bc, int mode, const ColArgs& a,
                                                   const PassBatch& p, hipStream_t s) {
  return bc == BC_PERIODIC ? col_mode_batch<EVX_INST_N, BC_PERIODIC>(mode, a, p, s)
                           : col_mode_batch<EVX_INST_N, BC_ZERO_FLUX>(mode, a, p, s);
}

hipError_t EVX_PASTE(evx_launch_rowb_, EVX_INST_N)(int bc, int mode, const RowArgs& a,
                                                   const PassBatch& p, hipStream_t s) {
  return bc == BC_PERIODIC ? row_mode_batch<EVX_INST_N, BC_PERIODIC>(mode, a, p, s)
                           : row_mode_batch<EVX_INST_N, BC_ZERO_FLUX>(mode, a, p, s);
}

#if EVX_INST_N == 32 || EVX_INST_N == 64
hipError_t EVX_PASTE(evx_launch_plane_, EVX_INST_N)(const PlaneArgs& a, hipStream_t s) {
  return plane_go<EVX_INST_N>(a, s);
}
#endif

}  // namespace evx
