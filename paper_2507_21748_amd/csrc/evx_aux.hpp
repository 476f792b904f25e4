// Element-wise and reduction passes used by the adjoint step and by the diagnostics.  Like the
// transform passes, each body is the work of one workgroup (gfx950 kernel or host emulator).
//
// Inner products of real fields are evaluated in the spectral domain (Parseval):
//   periodic, half spectrum:  sum_x a b = (1/V) sum_k w(kx) Re(A_k conj B_k),
//                             w = 1 for kx = 0 and kx = nx/2, else 2;
//   zero flux, DCT-II D_k = 2 sum_n x_n cos(pi k (2n+1) / 2N) per axis:
//                             sum_x a b = sum_k prod_axes w(k) A_k B_k,
//                             w(0) = 1/(4N), w(k > 0) = 1/(2N).
// Partial sums are FP64 and reduced in a fixed order, so results are bit-reproducible.
#pragma once

#include "evx_passes.hpp"

namespace evx {

constexpr int AUX_THREADS = 256;
// Fixed grid (fixed summation order).  The loops are grid-stride, so a test build may shrink it.
#ifndef EVX_AUX_BLOCKS
#define EVX_AUX_BLOCKS 1024
#endif
constexpr int AUX_BLOCKS = EVX_AUX_BLOCKS;

template <int T>
EVX_DEV void block_sum2(double& s0, double& s1, int tid, double* red) {
  red[2 * tid] = s0;
  red[2 * tid + 1] = s1;
  evx_sync();
  for (int h = T / 2; h > 0; h >>= 1) {
    if (tid < h) {
      red[2 * tid] += red[2 * (tid + h)];
      red[2 * tid + 1] += red[2 * (tid + h) + 1];
    }
    evx_sync();
  }
  s0 = red[0];
  s1 = red[1];
}

// Real-space sums.  Diagnostics (b == null): partial[2b] = sum f(c), partial[2b+1] = sum c.
// Distance (b != null): partial[2b] = sum (c - b)^2, partial[2b+1] = sum b^2.
struct RealSumArgs {
  const float* c;
  long long n;
  double* partial;
  const float* b;
};

EVX_DEV void realsum_body(const RealSumArgs& a, int tid, int bid, int nblk, double* red) {
  double s0 = 0.0, s1 = 0.0;
  const long long stride = (long long)nblk * AUX_THREADS;
  auto term = [&](double c, double r) {
    if (a.b) {
      s0 += (c - r) * (c - r);
      s1 += r * r;
    } else {
      const double q = c * c - 1.0;
      s0 += 0.25 * q * q;
      s1 += c;
    }
  };
  // four points in flight a lane: one at a time it waited for each (256^3: 26 -> 12 us)
  long long i = (long long)bid * AUX_THREADS + tid;
  for (; i + 3 * stride < a.n; i += 4 * stride) {
    float c[4], r[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < 4; ++k) c[k] = a.c[i + k * stride];
    if (a.b)
      for (int k = 0; k < 4; ++k) r[k] = a.b[i + k * stride];
    for (int k = 0; k < 4; ++k) term(c[k], r[k]);
  }
  for (; i < a.n; i += stride) term(a.c[i], a.b ? a.b[i] : 0.f);
  block_sum2<AUX_THREADS>(s0, s1, tid, red);
  if (tid == 0) {
    a.partial[2 * bid] = s0;
    a.partial[2 * bid + 1] = s1;
  }
}

// Single block: out_j <- (add_j ? out_j : 0) + scale_j * sum_b partial[2b + j] (j = 0, 1),
// summed in a fixed order.  add_j = 1 accumulates (gradients), 0 overwrites.  Null outputs are
// skipped.
struct FinalArgs {
  const double* partial;
  int nparts;
  double* out0;
  double* out1;
  double scale0, scale1;
  int add0, add1;
  // sums that a spectral z pass left in its columns (col_sums_at): seqs > 0
  int seqs, n_lo;
  long long stride_lo, stride_hi;
};

EVX_DEV void final_body(const FinalArgs& a, int tid, double* red) {
  double s0 = 0.0, s1 = 0.0;
  for (int b = tid; b < a.nparts; b += AUX_THREADS) {
    const double* const p =
        a.partial + (a.seqs ? col_sums_at(b, a.seqs, a.n_lo, a.stride_lo, a.stride_hi) : 2LL * b);
    s0 += p[0];
    s1 += p[1];
  }
  block_sum2<AUX_THREADS>(s0, s1, tid, red);
  if (tid == 0) {
    if (a.out0) *a.out0 = (a.add0 ? *a.out0 : 0.0) + a.scale0 * s0;
    if (a.out1) *a.out1 = (a.add1 ? *a.out1 : 0.0) + a.scale1 * s1;
  }
}

// Non-finite check of a spectral buffer (the stepper's optional failure check): block b writes
// flag[b] = 1 if one of its grid-stride elements (live columns only: row padding is skipped) has
// an all-ones exponent (Inf or NaN), else 0.  Every block writes its own slot, so no clearing and
// no atomics are needed, and the host ORs the AUX_BLOCKS slots.
struct FiniteArgs {
  const float2* w;
  long long n;     // float2 elements (grouped spectral layout)
  int ny, ypitch, nz, ncols;
  int* flag;       // AUX_BLOCKS slots
};

EVX_DEV bool evx_nonfinite(float v) {
  unsigned u;
  __builtin_memcpy(&u, &v, 4);
  return (u & 0x7f800000u) == 0x7f800000u;
}

template <int T>
EVX_DEV void finite_body(const FiniteArgs& a, int tid, int bid, int nblk, int* red) {
  int bad = 0;
  const long long stride = (long long)nblk * T;
  for (long long i = (long long)bid * T + tid; i < a.n; i += stride) {
    if (!spec_pos(i, a.ny, a.ypitch, a.nz, a.ncols).live) continue;
    const float2 v = a.w[i];
    bad |= int(evx_nonfinite(v.x) || evx_nonfinite(v.y));
  }
  red[tid] = bad;
  evx_sync();
  for (int h = T / 2; h > 0; h >>= 1) {
    if (tid < h) red[tid] |= red[tid + h];
    evx_sync();
  }
  if (tid == 0) a.flag[bid] = red[0];
}

// Variable-mobility Cahn-Hilliard (paper, appendix "Phase transformations of first and second
// order", eq. cahn-hilliard, stepped as in "Semi-implicit timestepping"): the finite-difference
// right-hand side div(M grad mu), mu = gamma0 g(phi) - 2 gamma0 eps lap phi, M = D0 phi (1 - phi),
// g = (18 / eps) phi (1 - phi) (1 - 2 phi), in one real-space pass over the natural (z, y, x)
// layout.  Periodic axes wrap; zero-flux axes mirror the edge cell into its ghost, so mu's ghost
// equals the edge value and a boundary face carries no flux.
struct VmStencilArgs {
  const float* phi;
  float* out;       // div(M grad mu)
  int nx, ny, nz;
  int per;          // periodic axes: bit 0 x, bit 1 y, bit 2 z
  float c_g;        // gamma0 * 18 / eps
  float c_lap;      // 2 gamma0 eps / dx^2
  float c_flux;     // D0 / (2 dx^2): the face mobility is the mean of the two cells'
};

// mu and div(M grad mu) in one pass: a block owns a VF_X x VF_Y column and marches up lz of its
// z planes:
//   mu = c_g p (1 - p)(1 - 2 p) - c_lap (sum of the 6 neighbours' phi - 6 p),
//   div(M grad mu) = c_flux sum_faces (p (1 - p) + q (1 - q)) (mu_q - mu_p),
// the neighbours and faces taken in the order +x, -x, +y, -y, +z, -z; mu never leaves the block (8
// bytes per voxel).  On a zero-flux axis phi is loaded clamped (the ghost is the edge cell) and a
// boundary face carries no flux.
//
// What bounds it: with one point a lane and all six neighbours read from LDS rings it was
// instruction issue (119 VALU and 104 scalar instructions a voxel, 75 us at 256^3, 1.8 TB/s).  A
// lane owns VF_R consecutive rows of one x: its z neighbours are registers, its y neighbours mostly
// too, a y or z face is evaluated once for the two voxels it joins, and the planes' LDS images
// (phi with a 2-point halo, mu with a 1-point halo, two of each) are addressed by constants: 52 us,
// 2.6 TB/s.  What remains is two barriers a plane and the 128-byte rows of a 32-wide column.
constexpr int VF_X = 32, VF_Y = 32, VF_R = 4, VF_THREADS = VF_X * VF_Y / VF_R;
constexpr int VF_P = 40;  // row pitch of both images: rows VF_R apart fall in opposite bank halves
constexpr int VF_PP = VF_P * (VF_Y + 4), VF_MP = VF_P * (VF_Y + 2);
constexpr int VF_LDS = 2 * (VF_PP + VF_MP);  // floats

EVX_DEV int vf_mod(int v, int n) {
  const int r = v % n;
  return r < 0 ? r + n : r;
}
// grid index of point v on an axis of n points: periodic wrap, or the zero-flux clamp
EVX_DEV int vf_map(int v, int n, bool per) {
  return per ? vf_mod(v, n) : (v < 0 ? 0 : (v >= n ? n - 1 : v));
}

// z planes per block of the fused pass: long runs (few re-read halo planes), but about four
// blocks per CU
inline int vm_fused_lz(const VmStencilArgs& a, int cus) {
  const long long ncols = (long long)((a.nx + VF_X - 1) / VF_X) * ((a.ny + VF_Y - 1) / VF_Y);
  long long lz = (a.nz * ncols + 4LL * cus - 1) / (4LL * cus);
  if (lz < 4) lz = 4;
  if (lz > a.nz) lz = a.nz;
  return int(lz);
}

// Point q of the square ring of half-open box [-h, VF_X + h) x [-h, VF_Y + h): its top and bottom
// rows, then its left and right columns between them.
EVX_DEV void vf_ring(int q, int h, int& x, int& y) {
  const int w = VF_X + 2 * h, c = VF_Y + 2 * h - 2;
  if (q < 2 * w) {
    y = q < w ? -h : VF_Y + h - 1;
    x = (q < w ? q : q - w) - h;
  } else {
    q -= 2 * w;
    x = q < c ? -h : VF_X + h - 1;
    y = (q < c ? q : q - c) - h + 1;
  }
}

// Launch: ceil(nx / VF_X) ceil(ny / VF_Y) columns times ceil(nz / lz) z ranges, VF_THREADS each.
EVX_DEV void vm_fused_body(const VmStencilArgs& a, int lz, int tid, int bid, float* lds) {
  constexpr int R = VF_R, P = VF_P;
  constexpr int RING1 = 2 * (VF_X + 2) + 2 * VF_Y, RING2 = 2 * (VF_X + 4) + 2 * (VF_Y + 2);
  static_assert(RING1 <= VF_THREADS && RING2 <= VF_THREADS, "one halo point of each ring a lane");
  const int ntx = (a.nx + VF_X - 1) / VF_X, nty = (a.ny + VF_Y - 1) / VF_Y;
  const int ncols = ntx * nty;
  const int col = bid % ncols, chunk = bid / ncols;
  const int x0 = (col % ntx) * VF_X, y0 = (col / ntx) * VF_Y;
  const int z0 = chunk * lz, z1 = z0 + lz < a.nz ? z0 + lz : a.nz;
  const bool px = a.per & 1, py = a.per & 2, pz = a.per & 4;
  const int tx = tid % VF_X, ty = R * (tid / VF_X);
  // the lane's points: R own rows, one of the 1-point ring (mu there too), one of the 2-point ring;
  // lanes past a ring repeat its first point
  auto src = [&](int x, int y) {
    return unsigned(vf_map(y0 + y, a.ny, py) * a.nx + vf_map(x0 + x, a.nx, px)) * 4u;
  };
  unsigned own[R];
  static_for<R>([&](auto r) { own[r] = src(tx, ty + decltype(r)::value); });
  int x1, y1, x2, y2;
  vf_ring(tid < RING1 ? tid : 0, 1, x1, y1);
  vf_ring(tid < RING2 ? tid : 0, 2, x2, y2);
  const unsigned src1 = src(x1, y1), src2 = src(x2, y2);
  const int p0 = (ty + 2) * P + tx + 2, m0 = (ty + 1) * P + tx + 1;  // own first point: phi, mu
  const int p1 = (y1 + 2) * P + x1 + 2, m1 = (y1 + 1) * P + x1 + 1;
  const int p2 = (y2 + 2) * P + x2 + 2;
  // boundary faces of zero-flux axes, by whether the lane's face carries flux
  const bool fxp = px || x0 + tx + 1 < a.nx, fxm = px || x0 + tx > 0;
  const int ylast = py ? 0x7fffffff : a.ny - 1 - (y0 + ty);  // own row with no +y face
  const bool fym = py || y0 + ty > 0;
  const unsigned plane = unsigned(a.nx) * unsigned(a.ny) * 4u;
  const long long pstep = (long long)a.nx * a.ny;
  struct Plane {
    float o[R], e, c;  // own rows, 1-point ring, 2-point ring
  };
  auto fetch = [&](int z, Plane& q) {
    const evx_buf b = evx_make_buf(a.phi + vf_map(z, a.nz, pz) * pstep, plane);
    static_for<R>([&](auto r) { q.o[r] = evx_buf_load1(b, own[r]); });
    q.e = evx_buf_load1(b, src1);
    q.c = evx_buf_load1(b, src2);
  };
  auto mu_of = [&](float p, float xp, float xm, float yp, float ym, float zp, float zm) {
    float s = 0.0f;
    s += xp;
    s += xm;
    s += yp;
    s += ym;
    s += zp;
    s += zm;
    return a.c_g * p * (1.0f - p) * (1.0f - 2.0f * p) - a.c_lap * (s - 6.0f * p);
  };
  Plane dn, cur, up, nxt;  // phi of planes k - 1, k, k + 1, k + 2
  fetch(z0 - 2, dn);
  fetch(z0 - 1, cur);
  fetch(z0, up);
  float md[R], mud[R], fz[R], acc[R];  // plane k - 1: p (1 - p), mu, its lower face's flux, sum
  static_for<R>([&](auto r) { md[r] = mud[r] = fz[r] = acc[r] = 0.0f; });
  for (int k = z0 - 1; k <= z1; ++k) {
    float* const ph = lds + (k & 1) * VF_PP;
    float* const mu = lds + 2 * VF_PP + (k & 1) * VF_MP;
    static_for<R>([&](auto r) { ph[p0 + P * decltype(r)::value] = cur.o[r]; });
    if (tid < RING1) ph[p1] = cur.e;
    if (tid < RING2) ph[p2] = cur.c;
    fetch(k + 2, nxt);  // past the range on the last planes: a mapped plane, loaded and unused
    evx_sync();
    float xp[R], xm[R], u[R], m[R];
    const float yl = ph[p0 - P], yh = ph[p0 + P * R];
    static_for<R>([&](auto r) {
      constexpr int j = decltype(r)::value;
      xp[j] = ph[p0 + P * j + 1];
      xm[j] = ph[p0 + P * j - 1];
    });
    static_for<R>([&](auto r) {
      constexpr int j = decltype(r)::value;
      const float p = cur.o[j];
      u[j] = mu_of(p, xp[j], xm[j], j + 1 < R ? cur.o[j + 1 < R ? j + 1 : j] : yh,
                   j > 0 ? cur.o[j > 0 ? j - 1 : j] : yl, up.o[j], dn.o[j]);
      m[j] = p * (1.0f - p);
      mu[m0 + P * j] = u[j];
    });
    if (tid < RING1)
      mu[m1] = mu_of(cur.e, ph[p1 + 1], ph[p1 - 1], ph[p1 + P], ph[p1 - P], up.e, dn.e);
    evx_sync();
    // the +z faces of plane k - 1 (the -z faces of plane k), which complete plane k - 1
    const bool face = pz || (k > 0 && k < a.nz);
    static_for<R>([&](auto r) {
      constexpr int j = decltype(r)::value;
      const float f = face ? (md[j] + m[j]) * (u[j] - mud[j]) : 0.0f;
      const float sum = (acc[j] + f) - fz[j];
      fz[j] = f;
      acc[j] = sum;
    });
    if (k > z0) {
      const evx_buf b = evx_make_buf(a.out + (long long)(k - 1) * pstep, plane);
      const bool in = x0 + tx < a.nx;
      static_for<R>([&](auto r) {
        constexpr int j = decltype(r)::value;
        evx_buf_store1(b, in && y0 + ty + j < a.ny ? own[j] : 0xfffffff0u, a.c_flux * acc[j]);
      });
    }
    // the x and y faces of plane k
    const float ul = mu[m0 - P], uh = mu[m0 + P * R];
    float fy = fym ? (m[0] + yl * (1.0f - yl)) * (ul - u[0]) : 0.0f;  // -y face of row 0
    static_for<R>([&](auto r) {
      constexpr int j = decltype(r)::value;
      const float up_ = mu[m0 + P * j + 1], um_ = mu[m0 + P * j - 1];
      const float mp = xp[j] * (1.0f - xp[j]), mm = xm[j] * (1.0f - xm[j]);
      const float mh = j + 1 < R ? m[j + 1 < R ? j + 1 : j] : yh * (1.0f - yh);
      const float hi = j + 1 < R ? u[j + 1 < R ? j + 1 : j] : uh;
      const float fyp = j < ylast ? (m[j] + mh) * (hi - u[j]) : 0.0f;
      float s = 0.0f;
      s += fxp ? (m[j] + mp) * (up_ - u[j]) : 0.0f;
      s += fxm ? (m[j] + mm) * (um_ - u[j]) : 0.0f;
      s += fyp;
      s += fy;
      fy = -fyp;
      acc[j] = s;
      md[j] = m[j];
      mud[j] = u[j];
    });
    dn = cur;
    cur = up;
    up = nxt;
  }
}

// lam <- lam - f''(c) v  (f'' = 3c^2 - 1)
struct CombineArgs {
  float* lam;
  const float* c;
  const float* v;
  long long n;
};

EVX_DEV void combine_body(const CombineArgs& a, int tid, int bid, int nblk) {
  const long long stride = (long long)nblk * AUX_THREADS;
  for (long long i = (long long)bid * AUX_THREADS + tid; i < a.n; i += stride) {
    const float c = a.c[i];
    a.lam[i] = a.lam[i] - (3.0f * c * c - 1.0f) * a.v[i];
  }
}

}  // namespace evx
