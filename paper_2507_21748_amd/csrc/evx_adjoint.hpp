// Pass schedules of the adjoint step and of the diagnostics (shared by the HIP launcher and the
// host emulator).  A launcher L additionally provides col_batch / row_batch (one pass over a
// PassBatch of buffer pairs), realsum(RealSumArgs), final(FinalArgs) and combine(CombineArgs).
//
// Adjoint of one step c^{n+1} = A c^n - B f'(c^n), A = T^{-1} diag(G P) T,
// B = T^{-1} diag(dt M K2 G) T (both symmetric):
//   lam^n = A lam^{n+1} - f''(c^n) (B lam^{n+1}),
//   dL/dkappa += <lam^{n+1}, T^{-1}[-dt M K2^2 G C^{n+1}]>,
//   dL/dM     += <lam^{n+1}, T^{-1}[-dt kappa K2^2 G C^{n+1} - dt K2 G F^n]>,
// with C^{n+1} = G (P T[c^n] - dt M K2 T[f'(c^n)]) recomputed from c^n.
#pragma once

#include "evx_aux.hpp"
#include "evx_schedule.hpp"

namespace evx {

struct AdjointBufs {
  float2 *A, *B, *Lm;  // spectral scratch
  float* v;            // real scratch
  double* partial;     // 2 * AUX_BLOCKS
  float* v2;           // second real scratch (variable mobility's right-hand side)
};

struct AdjointCoef {
  StepCoef step;
  float dt, dt_kappa;
};

// The z pass over T_xy[c] in A that goes on with the spectral work (colspec_body), and the reduction
// of the sums its blocks leave.
inline ColArgs spec_z_args(const Geom& g, const TablePtrs& t, const AdjointBufs& b,
                           const AdjointCoef& c, int mode, int remap) {
  ColArgs a = z_args(g, t, b.A, b.A, nullptr, c.step, remap);
  a.sp = SpecPass{mode, g.nx, g.ny, g.nz, g.bcy, g.bcz, g.xcplx, b.B, b.Lm, b.B, b.Lm, c.dt,
                  c.dt_kappa};
  return a;
}
inline FinalArgs spec_sums(const Geom& g, const ColArgs& a, double* out0, double* out1, double scale0,
                           double scale1, int add0, int add1) {
  const int seqs = col_block_seqs(g.fz);
  return FinalArgs{reinterpret_cast<const double*>(a.out), int((a.nseq + seqs - 1) / seqs), out0,
                   out1, scale0, scale1, add0, add1, seqs, a.n_lo, a.stride_lo, a.stride_hi};
}

// lam (in: dL/dc^{n+1}, out: dL/dc^n); dk, dM accumulate (device doubles).
template <class L>
void sched_adjoint(L& l, const Geom& g, const TablePtrs& t, const float* c, float* lam,
                   const AdjointBufs& b, const AdjointCoef& co, double* dk, double* dM,
                   int remap) {
  // forward transforms of c, f'(c) and lam (A, B, Lm), each pass batched over the buffers
  PassBatch rows_fwd{{c, lam, c}, {b.A, b.Lm, b.B}, 3};
  rows_fwd.fp[2] = 1;
  l.row_batch(g.row_len, g.bc, ROW_FWD, x_args(g, t, nullptr, c, b.A, nullptr), rows_fwd);
  const PassBatch spec3{{b.A, b.B, b.Lm}, {b.A, b.B, b.Lm}, 3};
  l.col_batch(g.fy, g.bcy, COL_FWD, y_args(g, t, b.A, b.A, remap), spec3);
  const ColArgs za = spec_z_args(g, t, b, co, SP_ADJOINT, remap);
  l.col(g.fz, g.bcz, COL_FWD, za);
  const double norm = (g.bc == BC_PERIODIC || g.xcplx) ? 1.0 / double(g.V) : 1.0;
  l.final(spec_sums(g, za, dk, dM, norm, norm, 1, 1));
  // inverse transforms: Lm -> lam, B -> v
  const PassBatch spec2{{b.Lm, b.B, nullptr}, {b.Lm, b.B, nullptr}, 2};
  l.col_batch(g.fy, g.bcy, COL_INV, y_args(g, t, b.Lm, b.Lm, remap), spec2);
  RowArgs xa = x_args(g, t, b.Lm, nullptr, nullptr, lam);
  if (g.bc == BC_PERIODIC) {  // both inverse transforms and the f'' term in one pass
    xa.comb = 1;
    xa.in_c2 = b.B;
    xa.in_r = c;
    l.row(g.row_len, g.bc, ROW_INV, xa);
  } else {
    // a cosine row shares its transform with the next row of the same buffer
    const PassBatch rows_inv{{b.Lm, b.B, nullptr}, {lam, b.v, nullptr}, 2};
    l.row_batch(g.row_len, g.bc, ROW_INV, xa, rows_inv);
    l.combine(CombineArgs{lam, c, b.v, g.V});
  }
}

// out[0] = mass dx^3 sum c, out[1] = energy dx^3 [sum f(c) + (kappa/2) sum c (-L c)].
template <class L>
void sched_diagnostics(L& l, const Geom& g, const TablePtrs& t, const float* c, double kappa,
                       const AdjointBufs& b, double* out, int remap) {
  l.row(g.row_len, g.bc, ROW_FWD, x_args(g, t, nullptr, c, b.A, nullptr));
  l.col(g.fy, g.bcy, COL_FWD, y_args(g, t, b.A, b.A, remap));
  const ColArgs za = spec_z_args(g, t, b, AdjointCoef{}, SP_ENERGY, remap);
  l.col(g.fz, g.bcz, COL_FWD, za);
  const double norm = (g.bc == BC_PERIODIC || g.xcplx) ? 1.0 / double(g.V) : 1.0;
  const double dx3 = g.dx * g.dx * g.dx;
  // out[1] <- dx^3 (kappa/2) sum w K2 |C|^2, then the real-space sums add f(c) and set the mass
  l.final(spec_sums(g, za, out + 1, nullptr, dx3 * 0.5 * kappa * norm, 0.0, 0, 0));
  l.realsum(RealSumArgs{c, g.V, b.partial, nullptr});
  l.final(FinalArgs{b.partial, AUX_BLOCKS, out + 1, out, dx3, dx3, 1, 0});
}

// out[0] = sum (a - b)^2, out[1] = sum b^2 (relative L2 distance = sqrt(out[0] / out[1])).
template <class L>
void sched_distance(L& l, const Geom& g, const float* a, const float* b, const AdjointBufs& bufs,
                    double* out) {
  l.realsum(RealSumArgs{a, g.V, bufs.partial, b});
  l.final(FinalArgs{bufs.partial, AUX_BLOCKS, out, out + 1, 1.0, 1.0, 0, 0});
}

// Gray-Scott: nsteps of both species in the real fields u, v.  Diffusion is implicit and the
// reaction explicit, U' = T[u + dt R_u] / (1 + dt Du K2): the transform is linear, so each species
// transforms its field and reaction together, and the multiplier needs no spectral state.  Between
// steps both species stay spectral (A and B hold F_z^{-1} of them): a step is the two y passes, the
// two-species x pass with the reaction, and one z pass with the multiplier, 64 bytes a voxel.  The
// species' means travel beside the buffers (spec_mean): adding the reaction to the whole field
// instead rounded relative to the mean at every step (relative error of 20 steps at 64^3 and 128^3
// 4.0e-7 against 2.7e-7 with separately transformed reactions, 1.5e-7 with the means apart).  A
// Dirichlet axis has no mean mode: there the species are spectral states (Lm and W), the x pass
// transforms the reactions alone and the z pass adds them, 80 bytes a voxel.
struct GsCoef {
  float dt, dt_du, dt_dv, F, k;
};
// The diffusion multipliers' common scale (coef_scale).
inline float gs_scale(const Geom& g, const GsCoef& co) {
  const double d = co.dt_du > co.dt_dv ? co.dt_du : co.dt_dv;
  return coef_scale(1.0 + d * k2_bound(g));
}

template <class L>
void sched_gray_scott(L& l, const Geom& g, const TablePtrs& t, float* u, float* v,
                      const AdjointBufs& b, float2* W, const GsCoef& co, int nsteps, int remap) {
  if (nsteps <= 0) return;
  const bool states = g.flip != 0;
  // a single step with states takes its reactions from the real fields, beside the states' own
  // transforms: seven launches instead of ten (48 x 384 x 50 110 -> 78 us)
  const bool one = states && nsteps == 1;
  const PassBatch two{{b.A, b.B}, {b.A, b.B}, 2};
  const ColArgs ya = y_args(g, t, b.A, b.A, remap);
  const float sc = gs_scale(g, co);
  const StepCoef zc{0.0f, 0.0f, sc * (states ? co.dt : 1.0f), sc};  // a_dt comes with the batch
  ColArgs za = z_args(g, t, b.A, b.A, nullptr, zc, remap);
  PassBatch upd{{b.A, b.B}, {b.A, b.B}, 2, {sc * co.dt_du, sc * co.dt_dv}};
  RowArgs xa = x_args(g, t, b.A, u, b.A, nullptr);
  xa.gs = 1;
  xa.in_c2 = b.B;
  xa.in_r2 = v;
  xa.out_c2 = b.B;
  xa.gs_dt = co.dt;
  xa.gs_F = co.F;
  xa.gs_k = co.k;
  if (states) {
    upd.state[0] = b.Lm;
    upd.state[1] = W;
    xa.rate = 1;
    const PassBatch rows{{u, v}, {b.Lm, W}, 2}, st{{b.Lm, W}, {b.Lm, W}, 2};
    l.row_batch(g.row_len, g.bc, ROW_FWD, x_args(g, t, nullptr, u, b.Lm, nullptr), rows);
    if (one) {
      const PassBatch all{{b.A, b.B, b.Lm, W}, {b.A, b.B, b.Lm, W}, 4};
      l.row(g.row_len, g.bc, ROW_FWD, xa);
      l.col_batch(g.fy, g.bcy, COL_FWD, ya, all);
      l.col_batch(g.fz, g.bcz, COL_FWD, za, st);
      l.col_batch(g.fz, g.bcz, COL_Z_VM, za, upd);
    } else {
      const PassBatch out{{b.Lm, W}, {b.A, b.B}, 2};
      l.col_batch(g.fy, g.bcy, COL_FWD, ya, st);
      l.col_batch(g.fz, g.bcz, COL_FWD, za, st);
      l.col_batch(g.fz, g.bcz, COL_INV, za, out);
    }
  }
  for (int n = one ? 1 : 0; n < nsteps; ++n) {
    const bool spectral = states || n > 0;  // the species' form on entry
    if (spectral) l.col_batch(g.fy, g.bcy, COL_INV, ya, two);
    if (!states) {
      xa.mean = n > 0 ? MEAN_IN : 0;
      za.mean = xa.mean | (n + 1 < nsteps ? MEAN_OUT : 0);
    }
    l.row(g.row_len, g.bc, spectral ? ROW_FUSED_POLY : ROW_FWD, xa);
    l.col_batch(g.fy, g.bcy, COL_FWD, ya, two);
    l.col_batch(g.fz, g.bcz, COL_Z_VM, za, upd);
  }
  l.col_batch(g.fy, g.bcy, COL_INV, y_args(g, t, b.A, b.A, remap), two);
  const PassBatch back{{b.A, b.B}, {u, v}, 2};
  l.row_batch(g.row_len, g.bc, ROW_INV, x_args(g, t, b.A, nullptr, nullptr, u), back);
}

// Variable-mobility Cahn-Hilliard in the paper's increment form (appendix "Semi-implicit
// timestepping"): phi <- phi + T^{-1}[dt / (1 + c4 K2^2) T[div(M grad mu)]], the right-hand side
// from the stencil pass; the multiplier sits between the forward and inverse z transforms
// of one column pass, and the inverse x pass adds the increment to phi.  Scratch: v2 (the right-hand
// side), A.
struct VmCoef {
  float dt, c4, c_g, c_lap, c_flux;
};

template <class L>
void sched_varmob(L& l, const Geom& g, const TablePtrs& t, float* phi, const AdjointBufs& b,
                  const VmCoef& co, int nsteps, int remap) {
  const int per = (g.bc == BC_PERIODIC ? 1 : 0) | (g.bcy == BC_PERIODIC ? 2 : 0) |
                  (g.bcz == BC_PERIODIC ? 4 : 0);
  // the z pass reads dt from dt_m, c4 from dt_m_kappa
  const StepCoef zc = implicit_coef(g, 0.0, co.c4, co.dt, false);
  // mu and the fluxes in one z-marching pass (mu stays in LDS)
  const VmStencilArgs fused{phi, b.v2, g.nx, g.ny, g.nz, per, co.c_g, co.c_lap, co.c_flux};
  for (int n = 0; n < nsteps; ++n) {
    l.vm_fused(fused);
    l.row(g.row_len, g.bc, ROW_FWD, x_args(g, t, nullptr, b.v2, b.A, nullptr));
    l.col(g.fy, g.bcy, COL_FWD, y_args(g, t, b.A, b.A, remap));
    l.col(g.fz, g.bcz, COL_Z_VM, z_args(g, t, b.A, b.A, nullptr, zc, remap));
    l.col(g.fy, g.bcy, COL_INV, y_args(g, t, b.A, b.A, remap));
    l.row(g.row_len, g.bc, ROW_INV_ADD, x_args(g, t, b.A, nullptr, nullptr, phi));
  }
}

}  // namespace evx
