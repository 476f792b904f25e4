// Pass bodies of the Cahn-Hilliard spectral step.  Each body is the work of one workgroup; it
// is wrapped by a __global__ kernel for gfx950 and by a threaded host emulator in the CPU tests.
//
// Spectral layout ("grouped").  The x columns of a spectral buffer -- periodic: the nx/2+1
// complex bins of the half spectrum; zero flux: the DCT-II spectrum is real, and its nx bins are
// handled as nx/2 float2 "column pairs" -- form groups of 8 (64 bytes), and a buffer is ordered
// [group][z][y'][8] with y' over ny + kSpecYPad rows: float2 index
//   (((x / 8) nz + z) ypitch + y) 8 + x % 8,   ypitch = ny + kSpecYPad.
// A y column pass then reads one contiguous ny x 64-byte run per (group, z); a z column pass
// reads 64-byte pieces (ny + 2) x 64 bytes apart, a stride that does not alias the memory
// channels the way a power of two does; the x pass reads 8 rows x 64 bytes per group.  Measured
// on 1024^3 with plain data-movement kernels, these patterns move a step's bytes 0.5 ms faster
// than the row-major half spectrum (rows of nx/2 + 1 values padded to 8), whose y passes read
// 64-byte pieces 4 KB apart and whose z pass 64-byte pieces 4.3 MB apart.  Ordering z outside
// the groups instead helps the x pass (its groups then lie 66 KB apart) but costs the z pass
// more.  Columns
// of the last group past the live count and the two pad rows per (group, z) hold no data: the
// column passes never address them and the x pass writes the dead columns as zeros.  Real fields
// stay in natural C order (z, y, x).  Two spectral buffers exist: S (spectral state, tile-major,
// see ColTile) and W (work).
//
// One time step is four passes over W (and one over S):
//   inverse y  ->  x: inverse x, f'(c) = c^3 - c, forward x  ->  forward y  ->
//   z: forward z, k-space update of S, inverse z.
// The real-space field is never stored between steps.
#pragma once

#include <type_traits>

#include "evx_fft.hpp"

namespace evx {

enum : int { BC_PERIODIC = 0, BC_ZERO_FLUX = 1, BC_DIRICHLET = 2, BC_VERTEX = 3 };

// Pad rows per (group, z) slab of a spectral buffer.
constexpr int kSpecYPad = 2;

// Float2 strides of the grouped spectral layout.
struct SpecGeom {
  long long xstride;  // between x groups: nz * ypitch * 8
  long long zstride;  // between z planes of a group: ypitch * 8
  int ny;
};

// Element i of a grouped spectral buffer: its x column, y and z, and whether it holds data (not a
// pad row, not a dead column of the last group).
struct SpecPos {
  int x, y, z;
  bool live;
};
EVX_HD SpecPos spec_pos(long long i, int ny, int ypitch, int nz, int ncols) {
  const long long q = i >> 3;
  const long long zq = q / ypitch;  // group nz + z
  const long long g = zq / nz;
  SpecPos p;
  p.y = int(q - zq * ypitch);
  p.z = int(zq - g * nz);
  p.x = int(g) * 8 + int(i & 7);
  p.live = p.y < ny && p.x < ncols;
  return p;
}

// Float2 offset (x group 0, column 0) of the row j rows past (z0, y0) (0 <= y0 < ny, j >= 0,
// y0 + j < 2^31), without a branch: an unsigned division.  (A carry loop would be a divergent region,
// into which the compiler sinks the loads that use the offset, each then waited for before the region
// ends.)
EVX_HD long long spec_row_offset_from(const SpecGeom& s, long long z0, int y0, int j) {
  const unsigned y = unsigned(y0 + j), ny = unsigned(s.ny);
  const unsigned dz = y / ny;
  return (z0 + dz) * s.zstride + (long long)(y - dz * ny) * 8;
}

// column (y or z) pass modes
enum : int {
  COL_FWD = 0,         // in -> forward transform -> out
  COL_INV = 1,         // in -> inverse transform -> out
  COL_Z_INIT = 2,      // in -> forward -> state; -> inverse -> out
  COL_Z_UPDATE = 3,    // in -> forward -> k-space update of state -> inverse -> out
  COL_Z_INV_STATE = 4, // state -> inverse -> out
  COL_Z_ETD = 5,       // as COL_Z_UPDATE with the exponential (ETD1) update
  COL_Z_AC = 6,        // as COL_Z_UPDATE for the Allen-Cahn model (semi-implicit)
  COL_Z_AC_ETD = 7,    // Allen-Cahn, exponential (ETD1) update
  COL_Z_VM = 8,        // in -> forward -> x dt / (1 + c2 K2 + c4 K2^2) -> inverse -> out (no state)
  COL_Z_GS = 9         // COL_Z_VM launched with a state (in the work buffers' own layout):
                       // C <- (C + dt x) / (1 + c2 K2 + c4 K2^2) -> state; -> inverse -> out
};

// row (x) pass modes
enum : int {
  ROW_FUSED = 0,  // complex row -> inverse x -> f' -> forward x -> complex row
  ROW_FWD = 1,    // real row -> forward x -> complex row
  ROW_INV = 2,    // complex row -> inverse x -> real row
  ROW_FUSED_REC = 3, // ROW_FUSED that also stores the real row it passes through (out_r)
  ROW_INV_ADD = 4,   // ROW_INV that adds the real row to out_r instead of storing it
  ROW_FUSED_POLY = 5 // ROW_FUSED with the cubic poly(c) of RowArgs in place of f'(c)
};

// What a forward z pass does with the finished spectrum of its columns instead of storing it
// (colspec_body): SP_ADJOINT the adjoint step's multipliers and gradient sums over three buffers,
// then their inverse z transforms; SP_ENERGY the gradient energy's sum.
enum : int { SP_NONE = 0, SP_ADJOINT = 1, SP_ENERGY = 2 };
struct SpecPass {
  int mode;
  int nx, ny, nz;          // points per axis
  int bcy, bcz, xcplx;     // y and z families; one complex column per cosine bin
  const float2* f;         // SP_ADJOINT: T[f'(c)] and T[lam] next to `in` = T[c] (z pass pending),
  const float2* l;         // and where the inverse z transforms of their images go
  float2* f_out;
  float2* l_out;
  float dt, dt_kappa;
};

// A column pass transforms nseq = 8 nouter sequences: sequence s is column s % 8 of outer index
// o = s / 8 = o_hi n_lo + o_lo, o_hi the x group (x = 8 o_hi + s % 8) and o_lo the other axis
// (z for the y pass, y for the z pass); x_lo = 1 would make o_lo the x group instead.
struct ColArgs {
  const float2* in;
  float2* out;
  float2* state;
  long long nseq;          // sequences = 8 * nouter
  int n_lo;                // outer indices per x group
  int nlive;               // x columns holding data (8 o_hi + column < nlive)
  long long stride_lo;     // float2 stride of o_lo
  long long stride_hi;     // float2 stride of o_hi (>= (n_lo - 1) stride_lo: offsets increase)
  int x_lo;                // 1: o_lo is the x group, 0: o_hi is
  int vlen;                // vertex-centred axis: its data length n (the transform length is
                           // 2(n - 1)): loads mirror point k > n - 1 to row 2(n - 1) - k, stores
                           // keep points below n; 0 otherwise
  long long row_stride;    // float2 stride between consecutive points of the transform axis
  const float2* tw;        // exp(-2 pi i j / N), j < N
  const float2* mk;        // zero flux: exp(-i pi k / (2N)), k < N
  const float* k2c;        // K2 along x: nx/2+1 entries, or nx for zero flux
  const float* k2o;        // K2 along the o_lo axis
  const float* k2r;        // K2 along the transform axis
  float a_dt;              // A dt
  float dt_m_kappa;        // dt M kappa
  float dt_m;              // dt M
  float one;               // 1, or the power of two that a_dt, dt_m_kappa and dt_m carry (coef_scale)
  int remap;               // XCD-aware block order
  int xcomplex;            // z pass: a column is one complex x bin (else two real x bins)
  int mean;                // COL_Z_VM: MEAN_* (the buffer's mean travels beside it, see spec_mean)
  unsigned lane_bytes;     // bytes addressable from a point's block base (col_lane_bytes)
  SpecPass sp;             // COL_FWD along z that goes on with the spectral work (SP_*)
};

struct RowArgs {
  const float2* in_c;  // spectral rows (grouped layout, SpecGeom sg)
  const float* in_r;   // real rows (natural order)
  float2* out_c;
  float* out_r;
  SpecGeom sg;
  long long nrows;     // rows of nx real points (ny * nz)
  const float2* tw;    // row FFT twiddles
  const float2* post;  // periodic: exp(-2 pi i k / nx), k <= nx/2; zero flux: exp(-i pi k/(2 nx))
  float scale;         // 1/V (periodic) or 1/(8V) (zero flux), applied after the inverse
  int flip;            // Dirichlet axes (bit 0 x, 1 y, 2 z): real rows carry (-1)^(their index)
  int ny;              // rows r = j + ny l (for the sign)
  int remap;           // XCD-aware block order (consecutive row blocks on one XCD)
  int xcplx;           // cosine x: spectral columns are complex, one per bin (real data)
  int vx;              // vertex-centred x: real rows of vx = NH + 1 points, extended evenly
  float poly[4];       // ROW_FUSED_POLY: poly(c) = poly[0] + poly[1] c + poly[2] c^2 + poly[3] c^3
  // Two-species pass (ROW_FUSED_POLY or ROW_FWD with gs set): in_c / in_r and out_c belong to u,
  // these to v; the pointwise part is one explicit reaction step of Gray-Scott (gs_react).
  int gs;
  const float2* in_c2;
  const float* in_r2;
  float2* out_c2;
  float gs_dt, gs_F, gs_k;
  int mean;            // MEAN_IN: in_c and in_c2 lack their means (spec_mean)
  int rate;            // the results are the reaction terms alone (the species are in states)
  int comb;            // ROW_INV of two buffers: out_r <- row of in_c - f''(in_r) (row of in_c2)
  int fp;              // ROW_FWD: transform f'(c) instead of c (one of a batch)
};

// A spectral buffer may lack its mean: its bin 0 is then zero and the bin's value, an FP64 number,
// lies in the first pad row of (group 0, plane 0), which no pass addresses otherwise.  A nearly
// uniform field then rounds relative to its fluctuations instead of its mean.
enum : int { MEAN_IN = 1, MEAN_OUT = 2 };
EVX_HD double* spec_mean(const float2* p, int ny) {
  return reinterpret_cast<double*>(const_cast<float2*>(p) + 8 * (long long)ny);
}

// (-1)^(i [x Dirichlet] + j [y Dirichlet] + l [z Dirichlet]) of point i of row r = j + ny l
EVX_HD float dirichlet_sign(long long r, int i, int ny, int mask) {
  const long long l = r / ny;
  const int j = int(r - l * ny);
  const int par = ((mask & 1) ? i : 0) + ((mask & 2) ? j : 0) + ((mask & 4) ? int(l & 1) : 0);
  return (par & 1) ? -1.0f : 1.0f;
}

// One launch of the same transform pass over up to four independent (in, out) buffer pairs: the
// grid's y index selects the pair (the small-grid adjoint and the two-species model run their
// transforms this way, which halves their launches).
constexpr int kMaxBatch = 4;
struct PassBatch {
  const void* in[kMaxBatch];
  void* out[kMaxBatch];
  int n;
  float a_dt[kMaxBatch];  // ColArgs::a_dt and state of each pair (the two-species z pass)
  float2* state[kMaxBatch];
  int fp[kMaxBatch];      // RowArgs::fp of each pair
};
EVX_HD void bind_batch(ColArgs& a, const PassBatch& b, int k) {
  a.in = static_cast<const float2*>(b.in[k]);
  a.out = static_cast<float2*>(b.out[k]);
  a.a_dt = b.a_dt[k];
  a.state = b.state[k];
}
// forward modes read real rows and write complex ones; the inverse does the opposite
EVX_HD void bind_batch(RowArgs& a, bool inverse, const PassBatch& b, int k) {
  if (inverse) {
    a.in_c = static_cast<const float2*>(b.in[k]);
    a.out_r = static_cast<float*>(b.out[k]);
  } else {
    a.in_r = static_cast<const float*>(b.in[k]);
    a.out_c = static_cast<float2*>(b.out[k]);
    a.fp = b.fp[k];
  }
}

// Block order: consecutive logical blocks (neighbouring columns, sharing 128-byte lines) are
// placed on the same XCD.  Hardware dispatches block i to XCD i % 8.
EVX_DEV int remap_block(int bid, int nblk, int on) {
  if (!on) return bid;
  const int per = nblk / 8;
  if (bid >= per * 8) return bid;
  return (bid % 8) * per + bid / 8;
}

// Index of the cell-centred input point that becomes point n of Makhoul's reordered sequence
// (v_n = x_{2n} for 2n < N, else x_{2N-2n-1}).
template <int N>
constexpr int makhoul_src(int n) {
  return (2 * n < N) ? 2 * n : 2 * N - 2 * n - 1;
}

// ------------------------------------------------------------------ column pass
template <int N, int SEQS = seqs_per_block<N>()>
struct ColCfg {
  static constexpr int E = FftPlan<N>::E;
  static constexpr int TPS = FftPlan<N>::TPS;
  static constexpr int B = SEQS;
  static constexpr int THREADS = B * TPS;
  static constexpr int TW = B * N;             // twiddle table offset (after the exchange area)
  static constexpr int K2 = TW + N;             // z update: K2 along the transform axis (floats)
  static constexpr int LDS = K2 + (N + 1) / 2;  // float2 slots
};

// src[i] if ok, else zero, with the load outside any branch: a load inside a divergent branch is
// waited for before the branch joins, which would make a lane's loads one round trip each.  The
// address is clamped to element 0 (which every caller guarantees valid) when ok is false, and the
// value is cleared with a bit mask rather than a select (the compiler turns a select of a loaded
// value into a branch around the load).
EVX_DEV float evx_keep(float v, unsigned mask) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, v) & mask);
}
EVX_DEV float2 load_or_zero(const float2* EVX_RESTRICT src, long long i, bool ok) {
  const float2 v = src[ok ? i : 0];
  const unsigned m = ok ? ~0u : 0u;
  return make_float2(evx_keep(v.x, m), evx_keep(v.y, m));
}

// A block's copy of a small constant table (COUNT entries) staged in LDS: every lane issues its
// table loads before the data loads (load) and writes them to LDS after (store), so the table
// latency overlaps the data latency.  Readers come after a barrier.
template <int COUNT, int T, class V>
struct TableStage {
  static constexpr int IT = (COUNT + T - 1) / T;
  V r[IT > 0 ? IT : 1];
  EVX_DEV void load(const V* EVX_RESTRICT src, int tid) {
    static_for<IT>([&](auto I) {
      const int i = tid + T * decltype(I)::value;
      r[I] = src[i < COUNT ? i : 0];
    });
  }
  EVX_DEV void store(V* dst, int tid) const {
    static_for<IT>([&](auto I) {
      const int i = tid + T * decltype(I)::value;
      if (i < COUNT) dst[i] = r[I];
    });
  }
};

// The N-entry FFT twiddle table; a single-stage transform reads none (its first read is in the
// second stage, which follows a barrier).
template <int N, int T>
using TwStage = TableStage<(FftPlan<N>::S > 1 ? N : 0), T, float2>;

// Zero flux, after a forward FFT of packed columns (a + i b): x holds Z[k], k = t + TPS e.
// Produces (Da[k], Db[k]) with D[k] = 2 sum_n x_n cos(pi k (2n+1) / 2N) (Makhoul).
template <int N, int B>
EVX_DEV void makhoul_post(float2 (&x)[FftPlan<N>::E], float2* lds, int b, int t,
                          const float2* EVX_RESTRICT mk) {
  constexpr int E = FftPlan<N>::E, TPS = FftPlan<N>::TPS;
  static_for<E>([&](auto e) { lds[lidx<B>(t + TPS * decltype(e)::value, b)] = x[e]; });
  evx_sync();
  static_for<E>([&](auto e) {
    const int k = t + TPS * decltype(e)::value;
    const int kr = (k == 0) ? 0 : N - k;
    const float2 P = x[e];
    const float2 Q = cconj(lds[lidx<B>(kr, b)]);
    const float2 w = mk[k];
    const float2 sp = cmul(w, cadd(P, Q));
    const float2 sm = cmul(w, csub(P, Q));
    x[e] = make_float2(sp.x, sm.y);
  });
  evx_sync();
}

// Zero flux, before an inverse FFT: x holds (Da[k], Db[k]); produces
// Z[k] = Va[k] + i Vb[k],  V[k] = exp(i pi k / 2N) (D[k] - i D[N-k]),  D[N] = 0.
template <int N, int B>
EVX_DEV void makhoul_pre(float2 (&x)[FftPlan<N>::E], float2* lds, int b, int t,
                         const float2* EVX_RESTRICT mk) {
  constexpr int E = FftPlan<N>::E, TPS = FftPlan<N>::TPS;
  static_for<E>([&](auto e) { lds[lidx<B>(t + TPS * decltype(e)::value, b)] = x[e]; });
  evx_sync();
  static_for<E>([&](auto e) {
    const int k = t + TPS * decltype(e)::value;
    const float2 D = x[e];
    const float2 Dr = (k == 0) ? make_float2(0.f, 0.f) : lds[lidx<B>(N - k, b)];
    const float2 w = cconj(mk[k]);
    const float2 va = cmul(w, make_float2(D.x, -Dr.x));
    const float2 vb = cmul(w, make_float2(D.y, -Dr.y));
    x[e] = make_float2(va.x - vb.y, va.y + vb.x);
  });
  evx_sync();
}

// Addressing of one block's B sequences.  For each point index e the block has a uniform base
// (scalar registers: a buffer resource) and every lane adds one 32-bit byte offset, the same for
// all its points.  A lane without data gets an offset past the resource's range, so its loads
// read zero and its stores are dropped without touching memory: no branches and no shared
// addresses.  Zero-flux reordered accesses (row makhoul_src(n) for point n) use the lowest row of
// the point group as base and a non-negative lane-dependent row shift.
constexpr unsigned kDeadLane = 0xfffffff0u;

// Bound on the bytes any lane addresses from a point base; the launchers check that it is below
// kDeadLane and that sequence numbers fit in 31 bits.
template <int N, int B = ColCfg<N>::B>
inline long long col_lane_bytes(const ColArgs& a) {
  constexpr int TPS = ColCfg<N>::TPS;
  static_assert(B % 8 == 0, "a block covers whole outer indices");
  // outer indices o0 .. o0 + qmax of one block: at most qmax / n_lo + 1 group steps and qmax
  // steps of o_lo (offsets increase with o, see ColArgs)
  const long long qmax = B / 8 - 1;
  const long long cmax = qmax == 0 ? 7 : (qmax / a.n_lo + 1) * a.stride_hi + qmax * a.stride_lo + 7;
  // a point base plus t rows, a Makhoul row shift (< 2 TPS rows), or a vertex axis's data row
  // (< N / 2 + 1 rows) from the point-0 base: N rows cover all of them (N >= 2 TPS)
  return (cmax + (long long)N * a.row_stride + 2) * 8;
}

// Whether a column pass runs on wide_seqs workgroups.  A z pass of length 64 or 128 from 64 MiB a buffer
// on (below, the caches merge the half lines): 128 x 512 x 512 periodic 117 -> 86 us, 128 x 1024 x 1024
// 479 -> 422, 64 x 1024 x 1024 229 -> 187, but 64 x 384 x 384, 38 MiB, 74 -> 76 us a step.  Lengths 50
// and 100 from 8 MiB on: 100 x 256 x 256 zero flux 32.5 -> 24.9, 100 x 128 x 128 mixed 20.0 -> 18.6, but
// 100 x 64 x 64 10.7 -> 11.1 and the y pass of 48 x 100 x 96 8.0 -> 8.4.
constexpr long long kWideHalfLines = kEmulated ? 1 << 16 : 64 << 20;
constexpr long long kWideIdleLanes = kEmulated ? 1 << 16 : 8 << 20;
template <int N>
inline bool col_wide(const ColArgs& a) {
  if constexpr (wide_seqs<N>() == ColCfg<N>::B) return false;
  const long long bytes = a.nseq * N * 8;
  if constexpr (ColCfg<N>::B == 8) return a.row_stride > 8 && bytes >= kWideHalfLines;
  return bytes >= kWideIdleLanes;
}

template <int N>
constexpr int makhoul_group_min(int e) {
  int m = N;
  for (int t = 0; t < FftPlan<N>::TPS; ++t) {
    const int r = makhoul_src<N>(t + FftPlan<N>::TPS * e);
    m = r < m ? r : m;
  }
  return m;
}

template <int N, int B>
struct ColTile {
  static constexpr int TPS = FftPlan<N>::TPS;
  static constexpr int SB = state_cols<N>();
  long long tb = 0;  // float2 offset of the block's first sequence (uniform)
  unsigned lo = 0;   // lane byte offset of point 0 relative to tb, or kDeadLane
  unsigned lc = 0;   // lane byte offset of its column (row 0) relative to tb
  int olo = 0, x = 0, t = 0;  // the lane's o_lo index and x column
  long long tile = 0;
  unsigned so = 0;   // lane byte offset in the tile-major state (or kDeadLane)
  bool live = false;
  EVX_DEV void locate(const ColArgs& a, long long tile_, int b, int t_) {
    static_assert(B % 8 == 0, "a block covers whole outer indices");
    t = t_;
    tile = tile_;
    const unsigned n_lo = unsigned(a.n_lo);
    const unsigned s0 = unsigned(tile) * unsigned(B);
    const unsigned o0 = s0 >> 3;                 // first outer index of the block (column 0)
    const unsigned h0 = o0 / n_lo, l0 = o0 - h0 * n_lo;
    tb = (long long)h0 * a.stride_hi + (long long)l0 * a.stride_lo;
    const unsigned o = o0 + (unsigned(b) >> 3);  // the lane's outer index and column
    const unsigned c = unsigned(b) & 7u;
    const unsigned h = o / n_lo, l = o - h * n_lo;
    olo = int(l);
    x = int((a.x_lo ? l : h) * 8 + c);
    live = (long long)s0 + b < a.nseq && x < a.nlive;
    const long long cofs = (long long)(h - h0) * a.stride_hi +
                           ((long long)l - (long long)l0) * a.stride_lo + c;
    lc = unsigned(cofs * 8);
    lo = live ? unsigned((cofs + (long long)t * a.row_stride) * 8) : kDeadLane;
    so = live ? unsigned((t * SB + int(s0 % unsigned(SB)) + b) * 8) : kDeadLane;
  }
  // The spectral state is stored tile-major: tile of SB sequences, then transform point k, then
  // column, at (tile N + k) SB + column (read and written only by the z pass).  A block's state is
  // one contiguous N B run where B = SB, else N runs of B.  Point t + TPS e of lane (t, b): uniform
  // base plus the lane offset `so`.
  EVX_DEV evx_buf sres(const float2* state, int e) const {
    static_assert(SB % B == 0, "a block lies within one tile of the state");
    return evx_make_buf(state + tile / (SB / B) * ((long long)N * SB) + (long long)(TPS * e) * SB,
                        unsigned(TPS * SB * 8));
  }
  // vertex-centred axis: lane offset of data row `row` from the point-0 base
  EVX_DEV unsigned voff(long long row_stride, int row) const {
    return live ? lc + unsigned((long long)row * row_stride * 8) : kDeadLane;
  }
  // point t + TPS e (natural order)
  EVX_DEV evx_buf res(const float2* base, long long row_stride, int e, unsigned nbytes) const {
    return evx_make_buf(base + tb + (long long)(TPS * e) * row_stride, nbytes);
  }
  // point t + TPS e stored at row makhoul_src(t + TPS e): base row of the group and lane shift
  template <int E_>
  EVX_DEV evx_buf res_m(const float2* base, long long row_stride, unsigned nbytes) const {
    constexpr int gmin = makhoul_group_min<N>(E_);
    return evx_make_buf(base + tb + (long long)gmin * row_stride, nbytes);
  }
  template <int E_>
  EVX_DEV unsigned off_m(long long row_stride) const {
    constexpr int gmin = makhoul_group_min<N>(E_);
    const int sh = makhoul_src<N>(t + TPS * E_) - gmin;
    return live ? lc + unsigned((long long)sh * row_stride * 8) : kDeadLane;
  }
};

// Per-axis Parseval weight of the zero-flux (DCT-II) coefficient k on an axis of n cells.
EVX_DEV double dct_weight(int k, int n) { return (k == 0 ? 0.25 : 0.5) / double(n); }

// One component of a spectral bin in the adjoint step: with C1 = G (P C - dt M K2 F),
//   dkappa += w Re(conj Lam (-dt M K2^2 G C1)),  dM += w Re(conj Lam (-dt kappa K2^2 G C1
//   - dt K2 G F)),  l <- G P Lam,  f <- dt M K2 G Lam.
// (Re(conj(L) X) = L.x X.x + L.y X.y, both components with the same weight; under a cosine x they
// are two independent real coefficients.)
EVX_DEV void adjoint_bin(float one, float a_dt, float dt_m_kappa, float dt_m, float dt,
                         float dt_kappa, float k2, double w, float c, float& f, float& l, double& s0,
                         double& s1) {
  const float k4 = k2 * k2;
  const float P = one + a_dt * k2;
  const float G = evx_rcp(one + dt_m_kappa * k4 + a_dt * k2);
  const float c1 = G * (P * c - dt_m * k2 * f);
  s0 += w * double(-dt_m * k4 * G) * double(l) * double(c1);
  s1 += w * (double(-dt_kappa * k4 * G) * double(l) * double(c1) +
             double(-dt * k2 * G) * double(l) * double(f));
  f = dt_m * k2 * G * l;
  l = G * P * l;
}

// Sums s0 and s1 over the block's T lanes in a fixed order; lane 0 ends with the totals.
template <int T>
EVX_DEV void block_sums(double& s0, double& s1, int tid, double* red) {
  red[2 * tid] = s0;
  red[2 * tid + 1] = s1;
  evx_sync();
  for (int n = T; n > 1;) {
    const int h = (n + 1) / 2;
    if (tid < n - h) {
      red[2 * tid] += red[2 * (tid + h)];
      red[2 * tid + 1] += red[2 * (tid + h) + 1];
    }
    evx_sync();
    n = h;
  }
  s0 = red[0];
  s1 = red[1];
}

template <int N, int BC, int MODE>
EVX_DEV void colspec_body(const ColArgs& a, int tid, int bid, int nblk, float2* lds);

template <int N, int BC, int MODE, int SEQS = ColCfg<N>::B>
EVX_DEV void colpass_body(const ColArgs& a, int tid, int bid, int nblk, float2* lds) {
  if constexpr (kEmulated && MODE == COL_FWD) {  // on the GPU kernels of their own
    if (a.sp.mode == SP_ADJOINT) return colspec_body<N, BC, SP_ADJOINT>(a, tid, bid, nblk, lds);
    if (a.sp.mode == SP_ENERGY) return colspec_body<N, BC, SP_ENERGY>(a, tid, bid, nblk, lds);
  }
  using C = ColCfg<N, SEQS>;
  constexpr int E = C::E, TPS = C::TPS, B = C::B;
  constexpr bool upd =
      MODE == COL_Z_UPDATE || MODE == COL_Z_ETD || MODE == COL_Z_AC || MODE == COL_Z_AC_ETD;
  if constexpr (kEmulated && MODE == COL_Z_VM) {
    if (a.state) return colpass_body<N, BC, COL_Z_GS, SEQS>(a, tid, bid, nblk, lds);  // GPU: a kernel
  }
  constexpr bool vm = MODE == COL_Z_VM || MODE == COL_Z_GS;
  constexpr bool kt = upd || vm;  // needs the K2 tables
  constexpr bool has_fwd = MODE == COL_FWD || MODE == COL_Z_INIT || kt;
  constexpr bool has_inv = MODE != COL_FWD;
  constexpr bool zf = BC == BC_ZERO_FLUX;
  const int b = tid % B;
  const int t = tid / B;
  const unsigned nb = a.lane_bytes;
  ColTile<N, B> ct;
  ct.locate(a, remap_block(bid, nblk, a.remap), b, t);

  // Tables first (they go to LDS after the data loads), then the data and for the update the
  // column K2, all in flight together.
  float2* const twl = lds + C::TW;
  TwStage<N, C::THREADS> tws;
  tws.load(a.tw, tid);
  float* const k2l = reinterpret_cast<float*>(lds + C::K2);
  TableStage<(kt ? N : 0), C::THREADS, float> k2s;
  if constexpr (kt) k2s.load(a.k2r, tid);

  float2 x[E];
  if constexpr (MODE == COL_Z_INV_STATE) {
    static_for<E>([&](auto e) { x[e] = evx_buf_load2(ct.sres(a.state, e), ct.so); });
  } else if constexpr (zf && has_fwd) {
    static_for<E>([&](auto e) {
      constexpr int ev = decltype(e)::value;
      x[e] = evx_buf_load2(ct.template res_m<ev>(a.in, a.row_stride, nb),
                           ct.template off_m<ev>(a.row_stride));
    });
  } else if (!zf && a.vlen) {
    // vertex-centred axis: the even extension about both end points, point n > vlen - 1 read
    // from data row N - n (N = 2 (vlen - 1))
    const evx_buf r0 = ct.res(a.in, a.row_stride, 0, nb);
    static_for<E>([&](auto e) {
      const int n = t + TPS * decltype(e)::value;
      x[e] = evx_buf_load2(r0, ct.voff(a.row_stride, n < a.vlen ? n : N - n));
    });
  } else {
    static_for<E>([&](auto e) { x[e] = evx_buf_load2(ct.res(a.in, a.row_stride, e, nb), ct.lo); });
  }
  // vertex-centred axis: keep points k < vlen (the rest of the extension mirrors them)
  auto store_points = [&](float2* out) {
    if (!zf && a.vlen) {
      const evx_buf r0 = ct.res(out, a.row_stride, 0, nb);
      static_for<E>([&](auto e) {
        const int k = t + TPS * decltype(e)::value;
        evx_buf_store2(r0, k < a.vlen ? ct.voff(a.row_stride, k) : kDeadLane, x[e]);
      });
    } else {
      static_for<E>([&](auto e) {
        evx_buf_store2(ct.res(out, a.row_stride, e, nb), ct.lo, x[e]);
      });
    }
  };
  float kca = 0.f, kcb = 0.f;
  if constexpr (kt) {
    const int o = ct.live ? ct.olo : 0, cc = ct.live ? ct.x : 0;
    const float ko = a.k2o[o];
    // Pair columns (two real x bins) occur under a cosine x whose y and z spectra stay real: a
    // cosine z, or a vertex-centred z (periodic transform of an even extension).
    if (a.xcomplex) {  // both components belong to x bin cc
      kca = a.k2c[cc] + ko;
      kcb = kca;
    } else {           // two real x bins per column
      kca = a.k2c[2 * cc] + ko;
      kcb = a.k2c[2 * cc + 1] + ko;
    }
  }
  tws.store(twl, tid);
  k2s.store(k2l, tid);

  if constexpr (has_fwd) {
    fft_regs<N, -1, B>(x, lds, b, t, twl);
    if constexpr (zf) makhoul_post<N, B>(x, lds, b, t, a.mk);
  }

  if constexpr (MODE == COL_FWD) {
    if constexpr (zf) {
      static_for<E>([&](auto e) {
        evx_buf_store2(ct.res(a.out, a.row_stride, e, nb), ct.lo, x[e]);
      });
    } else {
      store_points(a.out);
    }
    return;
  }

  if constexpr (MODE == COL_Z_INIT) {
    static_for<E>([&](auto e) {
      evx_buf_store2(ct.sres(a.state, e), ct.so, x[e]);
    });
  }

  if constexpr (vm) {
    // Implicit multiplier without a state, x <- dt x / (1 + c2 K2 + c4 K2^2) (c2 in a_dt, c4 in
    // dt_m_kappa, dt in dt_m): the variable-mobility increment (c4 = 2 dt gamma0 eps M0) and
    // Gray-Scott's diffusion (c2 = dt D, dt_m = 1).  One reciprocal a bin: an FP32 division costs
    // about ten VALU instructions, and two of them a point were a fifth of this pass's.
    evx_sync();  // K2 table visible
    auto mult = [&](float K2) {
      return a.dt_m * evx_rcp(a.one + a.a_dt * K2 + a.dt_m_kappa * K2 * K2);
    };
    if constexpr (MODE == COL_Z_GS) {
      float2 cs[E];
      const evx_buf r0 = ct.res(a.state, a.row_stride, 0, nb);
      static_for<E>([&](auto e) {
        const int k = t + TPS * decltype(e)::value;
        if (!zf && a.vlen)
          cs[e] = evx_buf_load2(r0, ct.voff(a.row_stride, k < a.vlen ? k : N - k));
        else
          cs[e] = evx_buf_load2(ct.res(a.state, a.row_stride, e, nb), ct.lo);
      });
      static_for<E>([&](auto e) {
        const float kr = k2l[t + TPS * decltype(e)::value];
        const float Ka = kca + kr, Kb = kcb + kr;
        const float ga = evx_rcp(a.one + a.a_dt * Ka + a.dt_m_kappa * Ka * Ka);
        const float gb = evx_rcp(a.one + a.a_dt * Kb + a.dt_m_kappa * Kb * Kb);
        x[e] = make_float2((a.one * cs[e].x + a.dt_m * x[e].x) * ga,
                           (a.one * cs[e].y + a.dt_m * x[e].y) * gb);
      });
      // a vertex-centred axis reads each state row twice, once as its mirror, which another lane owns:
      // every lane has its states before any lane stores new ones
      if (!zf && a.vlen) evx_sync();
      store_points(a.state);
    } else if (a.mean && ct.tile == 0 && b == 0 && t == 0) {  // bin 0, whose multiplier is dt
      double* const m = spec_mean(a.out, a.n_lo);
      const double v = double(x[0].x) + ((a.mean & MEAN_IN) ? *m : 0.0);
      x[0].x = (a.mean & MEAN_OUT) ? 0.0f : float(v);
      if (a.mean & MEAN_OUT) *m = v;
    }
    if constexpr (MODE == COL_Z_GS) {
    } else if (a.xcomplex) {
      static_for<E>([&](auto e) {
        x[e] = cscale(x[e], mult(kca + k2l[t + TPS * decltype(e)::value]));
      });
    } else {
      static_for<E>([&](auto e) {
        const float kr = k2l[t + TPS * decltype(e)::value];
        x[e] = make_float2(x[e].x * mult(kca + kr), x[e].y * mult(kcb + kr));
      });
    }
  }

  if constexpr (upd) {
    // C' = G (P C - dt M K2 F), P = 1 + A dt K2, G = 1 / (1 + dt M kappa K2^2 + A dt K2).
    // The library is built without FP contraction, so the rounded C' stored in the state is
    // exactly the value the inverse transform consumes, and every kernel that transforms the
    // same data rounds identically (resume from a stored state is bit-exact).
    evx_sync();  // K2 table visible (a single-stage periodic transform has no barrier of its own)
    // The state is read only now: loading it with the data would hold 32 more registers
    // through the forward transform and cost a block per compute unit.
    float2 cs[E];
    static_for<E>([&](auto e) {
      cs[e] = evx_buf_load2(ct.sres(a.state, e), ct.so);
    });
    // one bin: C' from C, F and its K2.  The coefficients of a complex bin's two components are the
    // same and evaluated once: in the periodic family, where pair columns are the exception, and in
    // workgroups below 8192 points (512^3 step 1099.5 -> 1096.6 us).  Length 1024 has that many, 16 a
    // lane on 512 lanes, and no registers left for it (and waits for memory).  Length 384, 12 points
    // a lane and 8 sequences, falls from six waves a SIMD to four by it and only loses (384 x 128 x 128
    // z pass 22.2 -> 23.8 us, 384 x 256 x 256 70.9 -> 72.2).
    constexpr bool share = !zf && B * N < 8192 && !(E == 12 && B == 8);
    struct Coef {
      float p, q, r;
    };
    auto coef = [&](float K2) {
      if constexpr (MODE == COL_Z_ETD) {
        // C' = C + phi1(dt S) dt R, dt S = -(dt M kappa K2^2 + A dt K2),
        // dt R = -(dt M K2 F + dt M kappa K2^2 C); phi1(0) = 1 keeps the DC bin exact
        return Coef{evx_phi1(-(a.dt_m_kappa * K2 * K2 + a.a_dt * K2)), a.dt_m * K2,
                    a.dt_m_kappa * K2 * K2};
      } else if constexpr (MODE == COL_Z_AC) {
        // Allen-Cahn: C' = G (P C - dt M F), P = 1 + A dt, G = 1 / (1 + A dt + dt M kappa K2)
        const float P = a.one + a.a_dt;
        return Coef{evx_rcp(P + a.dt_m_kappa * K2), P, a.dt_m};
      } else if constexpr (MODE == COL_Z_AC_ETD) {
        // Allen-Cahn ETD1: C' = C + phi1(dt S) dt R, dt S = -(dt M kappa K2 + A dt),
        // dt R = -(dt M F + dt M kappa K2 C)
        return Coef{evx_phi1(-(a.dt_m_kappa * K2 + a.a_dt)), a.dt_m, a.dt_m_kappa * K2};
      } else {
        return Coef{evx_rcp(a.one + a.dt_m_kappa * K2 * K2 + a.a_dt * K2), a.one + a.a_dt * K2,
                    a.dt_m * K2};
      }
    };
    auto update = [&](const Coef& c, float C, float F) {
      if constexpr (MODE == COL_Z_ETD || MODE == COL_Z_AC_ETD)
        return C + c.p * -(c.q * F + c.r * C);
      else
        return c.p * (c.q * C - c.r * F);
    };
    static_for<E>([&](auto e) {
      const float kr = k2l[t + TPS * decltype(e)::value];
      const Coef ca = coef(kca + kr);
      Coef cb = ca;
      if (!share || !a.xcomplex) cb = coef(kcb + kr);
      x[e] = make_float2(update(ca, cs[e].x, x[e].x), update(cb, cs[e].y, x[e].y));
      evx_buf_store2(ct.sres(a.state, e), ct.so, x[e]);
    });
  }

  if constexpr (has_inv) {
    if constexpr (zf) makhoul_pre<N, B>(x, lds, b, t, a.mk);
    fft_regs<N, +1, B>(x, lds, b, t, twl);
    if constexpr (zf) {
      static_for<E>([&](auto e) {
        constexpr int ev = decltype(e)::value;
        evx_buf_store2(ct.template res_m<ev>(a.out, a.row_stride, nb),
                       ct.template off_m<ev>(a.row_stride), x[e]);
      });
    } else {
      store_points(a.out);
    }
  }
}

// The forward z pass with the spectral work behind it (SpecPass).  A block leaves its two FP64 sums
// in the first two float2 of its own columns of `out` (= `in`), which nothing reads as a spectrum
// any more; col_sums_at gives their place.  For the adjoint step this one pass replaces the forward
// z passes of three buffers, a spectral kernel and the inverse z passes of two: 5 instead of 15
// buffer passes (128^3: 33 -> 16 us), bound at that size by the latency of its chain, on larger
// grids by memory.  The transforms and the per-bin arithmetic are those of the separate kernels.
EVX_HD long long col_sums_at(long long block, int seqs, int n_lo, long long stride_lo,
                             long long stride_hi) {
  const long long o = block * (seqs / 8), h = o / n_lo;
  return h * stride_hi + (o - h * n_lo) * stride_lo;
}

template <int N, int BC, int MODE>
EVX_DEV void colspec_body(const ColArgs& a, int tid, int bid, int nblk, float2* lds) {
  using C = ColCfg<N>;
  constexpr int E = C::E, TPS = C::TPS, B = C::B, T = C::THREADS;
  constexpr bool zf = BC == BC_ZERO_FLUX, adj = MODE == SP_ADJOINT;
  static_assert(B * N * 8 >= T * 16, "the block's sums fit the exchange area");
  const SpecPass& q = a.sp;
  const int b = tid % B, t = tid / B;
  const unsigned nb = a.lane_bytes;
  ColTile<N, B> ct;
  ct.locate(a, remap_block(bid, nblk, a.remap), b, t);
  auto load = [&](const float2* p, float2 (&x)[E]) {
    static_for<E>([&](auto e) {
      constexpr int ev = decltype(e)::value;
      if constexpr (zf)
        x[e] = evx_buf_load2(ct.template res_m<ev>(p, a.row_stride, nb),
                             ct.template off_m<ev>(a.row_stride));
      else
        x[e] = evx_buf_load2(ct.res(p, a.row_stride, ev, nb), ct.lo);
    });
  };
  float2* const twl = lds + C::TW;
  float* const k2l = reinterpret_cast<float*>(lds + C::K2);
  TwStage<N, T> tws;
  tws.load(a.tw, tid);
  TableStage<N, T, float> k2s;
  k2s.load(a.k2r, tid);
  float2 c[E], f[adj ? E : 1], l[adj ? E : 1];
  load(a.in, c);
  if constexpr (adj) {
    load(q.f, f);
    load(q.l, l);
  }
  const int y = ct.live ? ct.olo : 0, xc = ct.live ? ct.x : 0;
  const float ko = a.k2o[y];
  const bool complex_bin = a.xcomplex;
  const float kxa = a.k2c[complex_bin ? xc : 2 * xc];
  const float kxb = complex_bin ? kxa : a.k2c[2 * xc + 1];
  tws.store(twl, tid);
  k2s.store(k2l, tid);
  auto forward = [&](float2 (&x)[E]) {
    fft_regs<N, -1, B>(x, lds, b, t, twl);
    if constexpr (zf) makhoul_post<N, B>(x, lds, b, t, a.mk);
  };
  forward(c);
  if constexpr (adj) {
    forward(f);
    forward(l);
  }
  evx_sync();  // K2 table visible (a single-stage periodic transform has no barrier of its own)
  // sums per component without the weights; bin 0 of a cosine z weighs half of the others
  const bool cosz = q.bcz != BC_PERIODIC;
  double sa[2] = {0.0, 0.0}, sb[2] = {0.0, 0.0};
  static_for<E>([&](auto e) {
    const float kyz = ko + k2l[t + TPS * decltype(e)::value];
    const float ka = kxa + kyz, kb = kxb + kyz;
    double w = 1.0;
    if constexpr (decltype(e)::value == 0) w = cosz && t == 0 ? 0.5 : 1.0;
    if constexpr (adj) {
      adjoint_bin(a.one, a.a_dt, a.dt_m_kappa, a.dt_m, q.dt, q.dt_kappa, ka, w, c[e].x, f[e].x,
                  l[e].x, sa[0], sa[1]);
      adjoint_bin(a.one, a.a_dt, a.dt_m_kappa, a.dt_m, q.dt, q.dt_kappa, kb, w, c[e].y, f[e].y,
                  l[e].y, sb[0], sb[1]);
      // one bin's FP64 terms at a time: left to the end of the pass they hold 100 registers more
      evx_here(sa[0], sa[1], sb[0], sb[1]);
    } else {
      sa[0] += w * double(ka) * double(c[e].x) * double(c[e].x);
      sb[0] += w * double(kb) * double(c[e].y) * double(c[e].y);
    }
  });
  if constexpr (adj) {
    auto back = [&](float2 (&x)[E], float2* p) {
      if constexpr (zf) makhoul_pre<N, B>(x, lds, b, t, a.mk);
      fft_regs<N, +1, B>(x, lds, b, t, twl);
      static_for<E>([&](auto e) {
        constexpr int ev = decltype(e)::value;
        if constexpr (zf)
          evx_buf_store2(ct.template res_m<ev>(p, a.row_stride, nb),
                         ct.template off_m<ev>(a.row_stride), x[e]);
        else
          evx_buf_store2(ct.res(p, a.row_stride, ev, nb), ct.lo, x[e]);
      });
    };
    back(l, q.l_out);
    back(f, q.f_out);
  }
  // Parseval weights.  A complex bin weighs 1 on the x half spectrum's ends, else 2, and 1/4 or 1/2
  // per cosine axis (the 1/V normalisation is applied to the sums).
  double wa, wb;
  if (complex_bin) {
    wa = q.xcplx ? (xc == 0 ? 0.25 : 0.5) : ((xc == 0 || 2 * xc == q.nx) ? 1.0 : 2.0);
    wa *= q.bcy == BC_PERIODIC ? 1.0 : (y == 0 ? 0.25 : 0.5);
    wa *= cosz ? 0.5 : 1.0;
    wb = wa;
  } else {
    const double wyz = dct_weight(y, q.ny) * dct_weight(1, q.nz);
    wa = dct_weight(2 * xc, q.nx) * wyz;
    wb = dct_weight(2 * xc + 1, q.nx) * wyz;
  }
  double s0 = wa * sa[0] + wb * sb[0], s1 = wa * sa[1] + wb * sb[1];
  evx_sync();
  block_sums<T>(s0, s1, tid, reinterpret_cast<double*>(lds));
  if (tid == 0) {
    double* const p = reinterpret_cast<double*>(a.out + ct.tb);
    p[0] = s0;
    p[1] = s1;
  }
}

// ------------------------------------------------------------------ row pass
// Spectral rows (grouped layout) <-> registers.  Lane (t, b) of a block whose first row is r0
// holds columns k = t + TPS e of row r0 + ROWMUL b (+ 1 for the second row of a packed pair).
// Eight consecutive t of the eight b of a wave are one contiguous 512-byte piece of a group (eight
// rows x 64 bytes), so the rows need no staging in LDS.  Column k lies in group k / 8; over
// P = 8 / gcd(TPS, 8) consecutive e the lanes' (group, column) offsets repeat, STEP groups
// further on, so a lane keeps P byte offsets and every P points advance a wave-uniform base.
//
// A lane without a row gets an offset past the resources' range, which stays past it when a
// point's constant offset is added (kDeadLane would wrap); live offsets span at most 8 groups and
// the planes of one block's rows (under 0.6 GB at 1024^3; row_fits32 checks it on the host).
constexpr unsigned kDeadRow = 0x80000000u, kRowRange = 0x7fffffffu;

constexpr int ct_gcd(int a, int b) { return b == 0 ? a : ct_gcd(b, a % b); }

template <int TPS>
struct SpecLane {
  static constexpr int P = 8 / ct_gcd(TPS, 8);
  static constexpr int STEP = TPS * P / 8;
  long long base;   // float2 offset of the z plane of the block's first row (uniform)
  long long gstep;  // float2 stride of STEP groups (uniform)
  unsigned off[P];  // lane byte offset of point e from base + (e / P) gstep, or kDeadRow
  unsigned row;     // lane byte offset of the row's column 0 from base, or kDeadRow
  EVX_DEV SpecLane(const SpecGeom& sg, long long r0, int j, bool live, int t) {
    const long long z0 = r0 / sg.ny;
    const int y0 = int(r0 - z0 * sg.ny);
    base = z0 * sg.zstride;
    gstep = STEP * sg.xstride;
    const unsigned gbytes = unsigned(sg.xstride * 8);
    row = live ? unsigned(spec_row_offset_from(sg, 0, y0, j) * 8) : kDeadRow;
    static_for<P>([&](auto R) {
      const unsigned k = unsigned(t + TPS * decltype(R)::value);
      off[R] = live ? row + (k >> 3) * gbytes + (k & 7u) * 8u : kDeadRow;
    });
  }
};

// Applies f(e, buffer resource, lane byte offset) to points e = 0 .. COUNT - 1.
template <int COUNT, int TPS, class F>
EVX_DEV void spec_points(const float2* p, const SpecLane<TPS>& ln, F&& f) {
  constexpr int P = SpecLane<TPS>::P;
  const float2* q = p + ln.base;
  static_for<(COUNT + P - 1) / P>([&](auto M) {
    const evx_buf r = evx_make_buf(q, kRowRange);
    static_for<P>([&](auto R) {
      constexpr int e = decltype(M)::value * P + decltype(R)::value;
      if constexpr (e < COUNT) f(std::integral_constant<int, e>{}, r, ln.off[R]);
    });
    q += ln.gstep;
  });
}

// The columns from LAST on, after the lanes' points: the value of column LAST (if its lane, t = 0,
// has one to store) and zeros in the dead columns of its group, so that a buffer is always written
// in whole 64-byte pieces.  LAST is periodic: the Nyquist column NH; cosine: the first dead column.
template <int LAST, bool VALUE, int TPS>
EVX_DEV void spec_tail_out(float2* p, const SpecGeom& sg, const SpecLane<TPS>& ln, int t,
                           float2 v) {
  constexpr int C0 = LAST % 8, ND = (VALUE || C0 != 0) ? 8 - C0 : 0;
  const evx_buf r = evx_make_buf(p + ln.base + (LAST / 8) * sg.xstride, kRowRange);
  static_for<(ND + TPS - 1) / TPS>([&](auto J) {
    const int d = t + TPS * decltype(J)::value;
    const bool ok = ln.row != kDeadRow && d < ND;
    evx_buf_store2(r, ok ? ln.row + unsigned((C0 + d) * 8) : kDeadRow,
                   VALUE && d == 0 ? v : make_float2(0.f, 0.f));
  });
}

// Spectral rows of a periodic block through LDS, for rows of one, two or four lanes (TPS) on many rows
// (row_staged): there the lanes' own points are pieces of 8 TPS bytes, which the caches have to put
// together to lines.  Eight consecutive lanes move the eight columns of a row's group instead, and a
// wave whole lines; lds holds column k of row b at b S + k.  The transform's mirrored points come from
// there too, so the way in costs no barrier more than row_c2r's.
template <int B, int NH, int S, int TPS>
struct SpecRows {
  static constexpr int NG = NH / 8 + 1;   // groups of the NH + 1 columns
  static constexpr int RPL = 8 / TPS;     // rows a lane moves of each group
  static constexpr int STEP = B / RPL;    // between them
  static_assert(8 % TPS == 0 && B % RPL == 0 && S > NH, "a lane's rows and columns");
  const SpecGeom& sg;
  long long base;      // float2 offset of the z plane of the block's first row (uniform)
  int row, c;          // the lane's first row and its column within a group
  unsigned off[RPL];   // lane byte offsets of its rows' column c, or kDeadRow
  float2 r[NG * RPL];
  EVX_DEV SpecRows(const SpecGeom& g, long long r0, long long nrows, int tid)
      : sg(g), row(tid >> 3), c(tid & 7) {
    const long long z0 = r0 / sg.ny;
    const int y0 = int(r0 - z0 * sg.ny);
    base = z0 * sg.zstride;
    static_for<RPL>([&](auto K) {
      const int j = row + STEP * decltype(K)::value;
      off[K] = r0 + j < nrows ? unsigned((spec_row_offset_from(sg, 0, y0, j) + c) * 8) : kDeadRow;
    });
  }
  // f(index, group, byte offset, lds slot, whether the column holds data)
  template <class F>
  EVX_DEV void each(F&& f) const {
    static_for<NG * RPL>([&](auto I) {
      constexpr int g = decltype(I)::value / RPL, k = decltype(I)::value % RPL;
      const int col = 8 * g + c;
      f(I, std::integral_constant<int, g>{}, off[k], (row + STEP * k) * S + col,
        8 * g + 7 <= NH || col <= NH);
    });
  }
  EVX_DEV void load(const float2* p) {
    each([&](auto I, auto G, unsigned o, int, bool live) {
      r[I] = evx_buf_load2(evx_make_buf(p + base + decltype(G)::value * sg.xstride, kRowRange),
                           live ? o : kDeadRow);
    });
  }
  EVX_DEV void stage(float2* lds) const {
    each([&](auto I, auto, unsigned, int at, bool live) {
      if (live) lds[at] = r[I];
    });
  }
  // the staged columns, and zeros in the dead ones of the last group
  EVX_DEV void store(float2* p, const float2* lds) const {
    each([&](auto, auto G, unsigned o, int at, bool live) {
      const float2 v = lds[live ? at : 0];
      evx_buf_store2(evx_make_buf(p + base + decltype(G)::value * sg.xstride, kRowRange), o,
                     live ? v : make_float2(0.f, 0.f));
    });
  }
};

// LDS row stride for B rows read by lanes (t, b) at row b, column t + const: the smallest
// S >= need with S = q (mod 2q), q = 32 / min(B, 32), so that the 32 lanes of a half wave touch
// distinct 64-bit bank pairs.
constexpr int row_lds_stride(int need, int b) {
  const int q = 32 / (b < 32 ? b : 32);
  int s = need;
  while (s % (2 * q) != q % (2 * q)) ++s;
  return s;
}

// Periodic real rows <-> registers: the block's rows are one contiguous run of the field, moved in
// 8 V byte pieces by consecutive lanes (a row pitch that is a power of two would put lanes of
// different rows on one memory channel: 1.87 against 1.76 ms for a pass over 1024^3) and staged in
// LDS at a row stride of S.
template <int B, int NH, int S, int V, int T>
struct RealRows {
  static constexpr int NP = NH / V, COUNT = B * NP, IT = (COUNT + T - 1) / T;
  evx_buf buf;  // the rows that exist: pieces past them read zero and are not stored
  float4 r[IT];
  EVX_DEV RealRows(const float* rows, long long r0, long long nrows) {
    const long long left = nrows - r0;
    buf = evx_make_buf(rows + r0 * (2 * NH), unsigned(left < B ? left : B) * unsigned(NH * 8));
  }
  template <class F>
  EVX_DEV void pieces(int tid, F&& f) {
    static_for<IT>([&](auto I) {
      const int i = tid + T * decltype(I)::value;
      const int row = i / NP;
      if (COUNT % T == 0 || i < COUNT) f(I, unsigned(i * 8 * V), row * S + (i - row * NP) * V);
    });
  }
  EVX_DEV void load(int tid) {
    static_for<IT>([&](auto I) {  // no branch around the loads: pieces past COUNT are out of range
      const unsigned off = unsigned(tid + T * decltype(I)::value) * unsigned(8 * V);
      if constexpr (V == 2) {
        r[I] = evx_buf_load4(buf, off);
      } else {
        const float2 v = evx_buf_load2(buf, off);
        r[I] = make_float4(v.x, v.y, 0.f, 0.f);
      }
    });
  }
  EVX_DEV void stage(int tid, float2* lds) {
    pieces(tid, [&](auto I, unsigned, int at) {
      lds[at] = make_float2(r[I].x, r[I].y);
      if constexpr (V == 2) lds[at + 1] = make_float2(r[I].z, r[I].w);
    });
  }
  // the staged rows into the lane's pieces
  EVX_DEV void unstage(int tid, const float2* lds) {
    pieces(tid, [&](auto I, unsigned, int at) {
      const float2 u = lds[at], v = V == 2 ? lds[at + V - 1] : u;
      r[I] = make_float4(u.x, u.y, v.x, v.y);
    });
  }
  // stores the staged rows, or adds them to the rows loaded before
  template <bool ADD>
  EVX_DEV void store(int tid, const float2* lds) {
    pieces(tid, [&](auto I, unsigned off, int at) {
      float2 u = lds[at], v = V == 2 ? lds[at + V - 1] : u;
      if constexpr (ADD) {
        u = make_float2(r[I].x + u.x, r[I].y + u.y);
        v = make_float2(r[I].z + v.x, r[I].w + v.y);
      }
      if constexpr (V == 2)
        evx_buf_store4(buf, off, make_float4(u.x, u.y, v.x, v.y));
      else
        evx_buf_store2(buf, off, u);
    });
  }
};

// Rows take the fewest sequences per workgroup that fill a wave, and at least 8 (64-byte pieces
// of the real rows, 512-byte ones of the spectral rows per wave).
template <int N>
constexpr int row_seqs_per_block() {
  int b = 8;
  while (b * FftPlan<N>::TPS < 64) b *= 2;
  return b;
}

// Zero flux: LDS area in which whole rows meet packed pairs of rows.  A lane moves bins of row r
// (r = b, then B + b: a wave's accesses are then whole 128-byte lines of the grouped layout, which
// two half-line accesses of rows 2b and 2b + 1 are not: 45 against 34 us a pass at 256^3), while
// sequence b carries rows 2b and 2b + 1 as a + i b.  Bin n of row r is float 2B n + r plus a pad,
// which spreads bins 2t (t of one wave) over distinct banks.
template <int N, int B>
struct RowXch {
  static constexpr int SH = B == 8 ? 2 : 1;
  static constexpr int SLOTS = B * N + B / 2 * (((N - 1) >> SH) + 1);
  EVX_DEV static int at(int n) { return n * (2 * B) + (n >> SH) * B; }
  // at(n0 + C), given at0 = at(n0): a constant away where C keeps the pad's phase
  template <int C>
  EVX_DEV static int at(int n0, int at0) {
    if constexpr (C % (1 << SH) == 0) return at0 + C * (2 * B) + (C >> SH) * B;
    return at(n0 + C);
  }
};

// Lane tid of a row block: sequence b and part t in the transforms and their exchange area, and row
// b, part t when rows move to and from memory.
// Transforms: sequences fastest, so that sixteen lanes address 128 consecutive bytes of LDS.  Their
// memory accesses are then 16-byte pieces of eight rows (four 128-byte lines).  A 512-lane block
// (periodic x of 1024, a grid far beyond the caches) orders four parts, the sequences, then more
// parts instead: 32-byte pieces of four rows, two lines, for two-way bank conflicts (forward pass
// 1.77 -> 1.70 ms, fused 2.22 -> 2.18; smaller blocks lose more to the conflicts than they gain).
template <int B, int TPS>
EVX_DEV void row_lane(int tid, int& b, int& t) {
  if constexpr (B == 8 && TPS >= 64) {
    b = (tid >> 2) & 7;
    t = (tid & 3) + 4 * (tid >> 5);
  } else {
    b = tid % B;
    t = tid / B;
  }
}
// Memory, where rows meet the packed pairs of the cosine transforms in LDS anyway: sixteen lanes are
// whole 64-byte pieces of two rows, or where the parts are no multiple of 8, 32-byte pieces of four
// (256^3 zero flux, forward and inverse 30 -> 27 us, fused 34.5 -> 33.2).
template <int B, int TPS>
EVX_DEV void row_io_lane(int tid, int& b, int& t) {
  if constexpr (B == 8 && TPS % 8 == 0) {
    b = (tid >> 3) & 7;
    t = (tid & 7) + 8 * (tid >> 6);
  } else if constexpr (B == 8 && TPS % 4 == 0) {
    b = (tid >> 2) & 7;
    t = (tid & 3) + 4 * (tid >> 5);
  } else {
    b = tid % B;
    t = tid / B;
  }
}

// Periodic: template length NH = nx/2, the complex FFT length of the packed real row; the row
// has NH+1 complex points.  Zero flux: NH = nx, one sequence carries two rows packed as a + i b.
template <int NH, int BC>
struct RowCfg {
  static constexpr int E = FftPlan<NH>::E;
  static constexpr int TPS = FftPlan<NH>::TPS;
  static constexpr int B = row_seqs_per_block<NH>();   // sequences per block
  static constexpr int THREADS = B * TPS;
  static constexpr int ROWS = (BC == BC_PERIODIC) ? B : 2 * B;  // rows per block
  // real rows move in 16-byte pieces (V = 2 pairs of reals) where the row length, its LDS stride
  // (periodic) and the lane's points (zero flux) allow it
  static constexpr int SROW = row_lds_stride(NH, B);    // periodic: LDS stride of real rows
  static constexpr int V =
      (BC == BC_PERIODIC ? (NH % 2 == 0 && SROW % 2 == 0) : E % 4 == 0) ? 2 : 1;
  // the staging area of whole rows is a little larger than the transform's exchange area
  static constexpr int TW = (BC == BC_PERIODIC) ? B * SROW : RowXch<NH, B>::SLOTS;  // twiddles
  // post-processing twiddles come from a table in LDS; a lane of a short row (few lanes, many points
  // each) holds its own in registers instead.  Loaded a point each by every lane they doubled the
  // pass's loads (1024^3: fused 2.18 -> 2.10 ms, inverse 1.85 -> 1.70, forward 1.70 -> 1.62 with the
  // table; 128^3 and 256^3 1% a step).
  static constexpr bool PL = BC == BC_PERIODIC && TPS >= 8;
  static constexpr int PO = TW + (FftPlan<NH>::S > 1 ? NH : 0);
  static constexpr bool SHORT = TPS <= 4;  // rows that SpecRows (periodic) or CosRows can move
  static constexpr int NPO = PL ? NH / 2 + 1 : 0;  // exp(-2 pi i (NH - k) / nx) = -conj(entry k)
  static constexpr int LDS = PO + NPO;
};

// Whether every live lane offset of a row block (SpecLane: at most 8 groups, the planes its rows
// reach, one 64-byte piece) is below kDeadRow with room for a constant offset.
template <int NH, int BC>
inline bool row_fits32(const RowArgs& a) {
  const long long planes = RowCfg<NH, BC>::ROWS / a.sg.ny + 2;
  return (8 * a.sg.xstride + planes * a.sg.zstride + 8) * 8 < (long long)kDeadRow;
}

// Whether a row pass stages its spectral rows (SpecRows, CosRows): short rows on grids of many.  Fused
// pass direct -> staged: 1024 x 1024 x 16 87.6 -> 40.9 us, 512 x 512 x 16 29.5 -> 14.4, 512 x 512 x 40
// 42.7 -> 23.6, 1024 x 1024 x 64 170 -> 135; but 128 x 128 x 16 7.2 -> 7.7, 64 x 64 x 20 6.8 -> 7.7 and,
// four lanes a row, 256 x 256 x 96 16.8 -> 17.5 (512 x 512 x 96 42.2 either way).
// Cosine rows keep their bins in LDS anyway and lose by the direct way only with complex columns, of
// whose 8 bytes it takes 4 (512 x 512 x 20 mixed 44.3 -> 21.9, 1024 x 1024 x 40 177 -> 117), and with pair
// columns on rows of one lane (1024 x 1024 x 12 zero flux 49.4 -> 29.4); 256 x 256 rows lose by neither.
constexpr long long kStagedRows = kEmulated ? 64 : 32768;
template <int NH, int BC>
inline bool row_staged(const RowArgs& a) {
  using C = RowCfg<NH, BC>;
  if (!C::SHORT || a.gs || a.comb) return false;
  if (BC != BC_PERIODIC) return (a.xcplx || C::TPS == 1) && a.nrows >= 4 * kStagedRows;
  return a.nrows >= (C::TPS == 4 ? 4 : 1) * kStagedRows;
}

// Post-processing twiddles exp(-2 pi i k / nx) of a lane's points k = t + TPS e (RowCfg::PL).
template <int NH, bool PL>
struct PostTw {
  static constexpr int E = FftPlan<NH>::E, TPS = FftPlan<NH>::TPS;
  float2 w[PL ? 1 : E];
  const float2* po;
  int t;
  template <int e>
  EVX_DEV float2 at() const {
    if constexpr (PL) {
      const int k = t + TPS * e;
      const float2 v = po[k <= NH / 2 ? k : NH - k];
      return k <= NH / 2 ? v : make_float2(-v.x, v.y);
    } else {
      return w[e];
    }
  }
};

// C2R pre-processing, Z[k] = (X[k] + conj X[NH-k]) + i (X[k] - conj X[NH-k]) e^{+2 pi i k / nx}:
// X = X[k], Xr = conj X[NH-k], w = e^{-2 pi i k / nx}.
EVX_DEV float2 c2r_pre(float2 X, float2 Xr, float2 w) {
  const float2 Ev = cadd(X, Xr);
  const float2 Od = cmulc(csub(X, Xr), w);
  return make_float2(Ev.x - Od.y, Ev.y + Od.x);
}
// R2C post-processing of the transform of half the real row (the factor 1/2 of the even and odd
// parts travels with the input, where it is free): P = Z[k], Q = conj Z[NH-k].
EVX_DEV float2 r2c_post(float2 P, float2 Q, float2 w) {
  const float2 d = csub(P, Q);
  return cadd(cadd(P, Q), cmul(w, make_float2(d.y, -d.x)));
}

// The pointwise part of the fused x pass on an inverse transform's output v (real values scale v):
// h f'(c) or h poly(c) with c = scale v, h = 1/2 under a periodic x (r2c_post), 1 under a cosine
// one.  Scaling by 1/2 is exact, so h changes no rounding.
template <int MODE, bool HALF>
EVX_DEV float row_nonlin1(float scale, const float* poly, float v) {
  const float c = scale * v;
  if constexpr (MODE == ROW_FUSED_POLY) {
    constexpr float h = HALF ? 0.5f : 1.0f;
    return __builtin_fmaf(__builtin_fmaf(__builtin_fmaf(h * poly[3], c, h * poly[2]), c,
                                         h * poly[1]), c, h * poly[0]);
  } else {
    const float hc = HALF ? (0.5f * scale) * v : c;
    return c * c * hc - hc;
  }
}
template <int MODE, bool HALF>
EVX_DEV float2 row_nonlin(float scale, const float* poly, float2 v) {
  return make_float2(row_nonlin1<MODE, HALF>(scale, poly, v.x),
                     row_nonlin1<MODE, HALF>(scale, poly, v.y));
}

// A periodic row's half spectrum x (Nyquist column nyq, held by lane t = 0) to the input of the
// inverse transform, and back; w: post-processing twiddles of the lane's points.  The exchange
// area must be free on entry; row_c2r leaves it free, row_r2c does not.
template <int NH, int B, class W>
EVX_DEV void row_c2r(float2 (&x)[FftPlan<NH>::E], float2 nyq, const W& w, float2* lds, int b,
                     int t) {
  constexpr int E = FftPlan<NH>::E, TPS = FftPlan<NH>::TPS;
  static_for<E>([&](auto e) { lds[lidx<B>(t + TPS * decltype(e)::value, b)] = x[e]; });
  evx_sync();
  static_for<E>([&](auto e) {
    const int k = t + TPS * decltype(e)::value;
    float2 m = lds[lidx<B>(decltype(e)::value == 0 && t == 0 ? 0 : NH - k, b)];
    if constexpr (decltype(e)::value == 0) m = t == 0 ? nyq : m;
    x[e] = c2r_pre(x[e], cconj(m), w.template at<decltype(e)::value>());
  });
  evx_sync();
}
template <int NH, int B, class W>
EVX_DEV float2 row_r2c(float2 (&x)[FftPlan<NH>::E], const W& w, float2* lds, int b, int t) {
  constexpr int E = FftPlan<NH>::E, TPS = FftPlan<NH>::TPS;
  float2 nyq = make_float2(0.f, 0.f);
  static_for<E>([&](auto e) { lds[lidx<B>(t + TPS * decltype(e)::value, b)] = x[e]; });
  evx_sync();
  static_for<E>([&](auto e) {
    const int k = t + TPS * decltype(e)::value;
    const float2 Q = cconj(lds[lidx<B>(decltype(e)::value == 0 && t == 0 ? 0 : NH - k, b)]);
    // k = NH: w = -1 on the pair of k = 0
    if constexpr (decltype(e)::value == 0) nyq = make_float2(2.0f * (x[e].x - x[e].y), 0.f);
    x[e] = r2c_post(x[e], Q, w.template at<decltype(e)::value>());
  });
  return nyq;
}

// A periodic block's spectral rows: the lane's points and, for lane t = 0, the Nyquist column.
template <int NH>
EVX_DEV float2 spec_row_in(const float2* p, const SpecGeom& sg, const SpecLane<FftPlan<NH>::TPS>& ln,
                           int t, float2 (&x)[FftPlan<NH>::E]) {
  spec_points<FftPlan<NH>::E>(p, ln, [&](auto e, evx_buf r, unsigned off) {
    x[e] = evx_buf_load2(r, off);
  });
  return evx_buf_load2(evx_make_buf(p + ln.base + (NH / 8) * sg.xstride, kRowRange),
                       ln.row != kDeadRow && t == 0 ? ln.row + unsigned(NH % 8 * 8) : kDeadRow);
}
template <int NH>
EVX_DEV void spec_row_out(float2* p, const SpecGeom& sg, const SpecLane<FftPlan<NH>::TPS>& ln,
                          int t, const float2 (&x)[FftPlan<NH>::E], float2 nyq) {
  spec_points<FftPlan<NH>::E>(p, ln, [&](auto e, evx_buf r, unsigned off) {
    evx_buf_store2(r, off, x[e]);
  });
  spec_tail_out<NH, true>(p, sg, ln, t, nyq);
}

// One explicit Gray-Scott reaction step of a point, scaled by h (r2c_post's half): u, v are scale
// times the given values plus their means mu, mv, which the results lack too; sg is the point's
// Dirichlet sign (the fields then carry it, and of the reaction's terms only the constant feed does
// not).
EVX_DEV void gs_react(const RowArgs& a, float scale, float h, float sg, float mu, float mv, float& u,
                      float& v) {
  const float du = scale * u, dv = scale * v;
  const float cu = du + mu, cv = dv + mv;
  const float uv2 = cu * cv * cv;
  const float ru = a.gs_F * (sg - cu) - uv2, rv = uv2 - a.gs_k * cv;
  u = h * (a.rate ? ru : __builtin_fmaf(a.gs_dt, ru, du));
  v = h * (a.rate ? rv : __builtin_fmaf(a.gs_dt, rv, dv));
}
// The means of the two species of a block's input.
EVX_DEV float2 gs_means(const RowArgs& a) {
  if (!(a.mean & MEAN_IN)) return make_float2(0.f, 0.f);
  return make_float2(float(*spec_mean(a.in_c, a.sg.ny) * a.scale),
                     float(*spec_mean(a.in_c2, a.sg.ny) * a.scale));
}

// A periodic block's tables: FFT twiddles to LDS, post-processing twiddles to where w keeps them.
template <int NH, int T, bool PL>
EVX_DEV void row_tables(const RowArgs& a, int tid, int t, float2* twl, PostTw<NH, PL>& w) {
  using C = RowCfg<NH, BC_PERIODIC>;
  TwStage<NH, T> tws;
  tws.load(a.tw, tid);
  if constexpr (PL) {
    TableStage<C::NPO, T, float2> pos;
    pos.load(a.post, tid);
    pos.store(twl + (C::PO - C::TW), tid);
  } else {
    static_for<C::E>([&](auto e) { w.w[e] = a.post[t + C::TPS * decltype(e)::value]; });
  }
  tws.store(twl, tid);
}

// Real rows of a periodic-family block to the lane's points x (pairs of reals), with the Dirichlet
// sign of y / z; `tables` runs once the loads are issued.  Leaves the exchange area free.
template <int NH, int B, class F>
EVX_DEV void real_row_in(const RowArgs& a, const float* in, long long r0, int tid, F&& tables,
                         float2* lds, float2 (&x)[FftPlan<NH>::E]) {
  using C = RowCfg<NH, BC_PERIODIC>;
  constexpr int E = C::E, TPS = C::TPS;
  int b, t;
  row_lane<B, TPS>(tid, b, t);
  const long long row = r0 + b;
  if (a.vx) {
    // vertex-centred x: rows of NH + 1 points, extended evenly about both end points to the 2 NH
    // points the real transform takes: point j > NH is point 2 NH - j
    const evx_buf src = evx_make_buf(in + r0 * (NH + 1), kRowRange);
    auto at = [&](int j) {
      return row < a.nrows ? unsigned((b * (NH + 1) + (j <= NH ? j : 2 * NH - j)) * 4) : kDeadRow;
    };
    static_for<E>([&](auto e) {
      const int j = 2 * (t + TPS * decltype(e)::value);
      x[e] = make_float2(evx_buf_load1(src, at(j)), evx_buf_load1(src, at(j + 1)));
    });
    tables();
  } else {
    RealRows<B, NH, C::SROW, C::V, C::THREADS> rr(in, r0, a.nrows);
    rr.load(tid);
    tables();
    rr.stage(tid, lds);
    evx_sync();
    static_for<E>([&](auto e) { x[e] = lds[b * C::SROW + t + TPS * decltype(e)::value]; });
    evx_sync();
  }
  if (a.flip) {  // Dirichlet y / z: one sign per row
    const float sg = dirichlet_sign(row, 0, a.ny, a.flip);
    static_for<E>([&](auto e) { x[e] = cscale(x[e], sg); });
  }
}

// The same for the 2 B cosine rows of a block and COLS columns, pairs of bins or (CPLX) one complex
// column a bin whose real part counts: bin n of row j is float X::at(n) + j of lds.
template <int B, int COLS, bool CPLX, int TPS, class X>
struct CosRows {
  static constexpr int NG = (COLS + 7) / 8, RPL = 16 / TPS, STEP = 2 * B / RPL;
  static_assert(16 % TPS == 0 && 2 * B % RPL == 0, "a lane's rows");
  const SpecGeom& sg;
  long long base;
  int row, c, ate, ato;  // ate, ato: float offsets of column c's bins
  unsigned off[RPL];
  float2 r[NG * RPL];
  EVX_DEV CosRows(const SpecGeom& g, long long r0, long long nrows, int tid)
      : sg(g), row(tid >> 3), c(tid & 7), ate(X::at(CPLX ? c : 2 * c)), ato(X::at(2 * c + 1)) {
    const long long z0 = r0 / sg.ny;
    const int y0 = int(r0 - z0 * sg.ny);
    base = z0 * sg.zstride;
    static_for<RPL>([&](auto K) {
      const int j = row + STEP * decltype(K)::value;
      off[K] = r0 + j < nrows ? unsigned((spec_row_offset_from(sg, 0, y0, j) + c) * 8) : kDeadRow;
    });
  }
  template <class F>
  EVX_DEV void each(F&& f) const {
    static_for<NG * RPL>([&](auto I) {
      constexpr int g = decltype(I)::value / RPL, k = decltype(I)::value % RPL, n0 = (CPLX ? 8 : 16) * g;
      const int j = row + STEP * k;
      f(I, std::integral_constant<int, g>{}, off[k], X::template at<n0>(CPLX ? c : 2 * c, ate) + j,
        X::template at<n0>(2 * c + 1, ato) + j, 8 * g + 7 < COLS || 8 * g + c < COLS);
    });
  }
  EVX_DEV void load(const float2* p) {
    each([&](auto I, auto G, unsigned o, int, int, bool live) {
      const evx_buf b = evx_make_buf(p + base + decltype(G)::value * sg.xstride, kRowRange);
      if constexpr (CPLX)
        r[I].x = evx_buf_load1(b, live ? o : kDeadRow);
      else
        r[I] = evx_buf_load2(b, live ? o : kDeadRow);
    });
  }
  EVX_DEV void stage(float* lds) const {
    each([&](auto I, auto, unsigned, int e, int o, bool live) {
      if (!live) return;
      lds[e] = r[I].x;
      if constexpr (!CPLX) lds[o] = r[I].y;
    });
  }
  EVX_DEV void store(float2* p, const float* lds) const {
    each([&](auto, auto G, unsigned off_, int e, int o, bool live) {
      float2 v = make_float2(0.f, 0.f);
      if (live) v = make_float2(lds[e], CPLX ? 0.f : lds[o]);
      evx_buf_store2(evx_make_buf(p + base + decltype(G)::value * sg.xstride, kRowRange), off_, v);
    });
  }
};

// Cosine rows.  GS = false: sequence b packs rows r0 + 2b and r0 + 2b + 1 as a + i b, and lane (t, b)
// moves bins of rows r0 + b and r0 + B + b (RowXch).  GS = true: sequence b packs row r0 + b of the
// two species as u + i v.  A spectral column is a pair of real bins (2c, 2c + 1), or with xcplx one
// complex column per bin.
template <int NH, int MODE, bool GS, bool STAGED = false>
EVX_DEV void cos_rows(const RowArgs& a, int tid, long long r0, float2* lds) {
  using C = RowCfg<NH, BC_ZERO_FLUX>;
  constexpr int E = C::E, TPS = C::TPS, B = C::B, T = C::THREADS;
  constexpr bool real_in = MODE == ROW_FWD;
  constexpr bool real_out =
      MODE == ROW_INV || MODE == ROW_INV_ADD || MODE == ROW_FUSED_REC;
  constexpr bool add = MODE == ROW_INV_ADD;
  const int b = tid % B, t = tid / B;
  int bo, to;
  row_io_lane<B, TPS>(tid, bo, to);
  float2 x[E], w[E];
  float2* const twl = lds + C::TW;
  TwStage<NH, T> tws;
  tws.load(a.tw, tid);
  static_for<E>([&](auto e) { w[e] = a.post[t + TPS * decltype(e)::value]; });
  auto put = [&](int n, float2 v) { lds[lidx<B>(n, b)] = v; };
  auto get = [&](int n) { return lds[lidx<B>(n, b)]; };
  static_assert(E % 2 == 0, "a lane's bins come in pairs");
  using X = RowXch<NH, B>;
  constexpr int NX = NH, H = E / 2, V = C::V, HV = H / V;
  float* const st = reinterpret_cast<float*>(lds);
  // float offsets of the lane's bin t, its mirror, and the row it moves; bins come as base + C
  const int atp = X::at(t), atm = X::at(-t);
  const int ate = X::at(2 * to), ato = X::at(2 * to + 1), ats = X::at(V * to), atn = X::at(-V * to);
  const int atx = X::at(to);
  float2* const prs = lds + b;   // pair b of bin n: prs[at(n) / 2]
  float* const rwa = st + (GS ? 2 * bo : bo);           // the lane's first row of bin n: rwa[at(n)]
  float* const rwb = st + (GS ? 2 * bo + 1 : B + bo);   // and its second
  const float2* const in_b = GS ? a.in_c2 : a.in_c;
  float2* const out_b = GS ? a.out_c2 : a.out_c;
  const long long ra = r0 + bo, rb = GS ? ra : ra + B;  // rows whose bins the lane moves
  const bool va = ra < a.nrows, vb = rb < a.nrows;
  const SpecLane<TPS> la(a.sg, r0, bo, va, to);
  const SpecLane<TPS> lb(a.sg, r0, int(rb - r0), vb, to);
  // real rows: lane offsets of its first pairs from the block's first row
  const unsigned oa = va ? unsigned((bo * NX + 2 * V * to) * 4) : kDeadRow;
  const unsigned ob = vb ? unsigned((int(rb - r0) * NX + 2 * V * to) * 4) : kDeadRow;
  // pairs c = V (t + TPS i) .. + V - 1 of a real row
  auto row_in = [&](evx_buf r, unsigned off, float2 (&p)[H]) {
    static_for<HV>([&](auto i) {
      constexpr int iv = decltype(i)::value;
      if constexpr (V == 2) {
        const float4 q = evx_buf_load4i<TPS * iv * 16>(r, off);
        p[2 * iv] = make_float2(q.x, q.y);
        p[2 * iv + 1] = make_float2(q.z, q.w);
      } else {
        p[iv] = evx_buf_load2i<TPS * iv * 8>(r, off);
      }
    });
  };
  auto row_out = [&](evx_buf r, unsigned off, const float2 (&p)[H]) {
    static_for<HV>([&](auto i) {
      constexpr int iv = decltype(i)::value;
      if constexpr (V == 2)
        evx_buf_store4i<TPS * iv * 16>(
            r, off, make_float4(p[2 * iv].x, p[2 * iv].y, p[2 * iv + 1].x, p[2 * iv + 1].y));
      else
        evx_buf_store2i<TPS * iv * 8>(r, off, p[iv]);
    });
  };
  // pair c holds points 2c = src(c) and 2c + 1 = src(N - 1 - c) of Makhoul's order
  // Dirichlet signs: of the rows the lane moves and of the one it transforms (two species) at even
  // points, and of odd points against even ones
  float sa = 1.0f, sb = 1.0f, sx = 1.0f;
  if (a.flip) {
    sa = dirichlet_sign(ra, 0, a.ny, a.flip);
    sb = dirichlet_sign(rb, 0, a.ny, a.flip);
    if constexpr (GS) sx = dirichlet_sign(r0 + b, 0, a.ny, a.flip);
  }
  const float sodd = (a.flip & 1) ? -1.0f : 1.0f;
  auto flip = [&](float sg, float2 v) { return make_float2(v.x * sg, v.y * (sg * sodd)); };
  // the two-species reaction
  const float2 mean = GS && !real_in ? gs_means(a) : make_float2(0.f, 0.f);
  auto react = [&](float scale) {
    static_for<E>([&](auto e) {
      // (the first half of the order are the row's even points, the second its odd ones)
      gs_react(a, scale, 1.0f, decltype(e)::value < H ? sx : sx * sodd, mean.x, mean.y, x[e].x,
               x[e].y);
    });
  };
  static_assert(!STAGED || (C::SHORT && !GS), "rows that are staged are short, of one species");
  // f(rows) with the block's rows as CosRows
  auto staged = [&](auto&& f) {
    if constexpr (STAGED) {
      if (a.xcplx)
        f(CosRows<B, NX, true, TPS, X>(a.sg, r0, a.nrows, tid));
      else
        f(CosRows<B, NX / 2, false, TPS, X>(a.sg, r0, a.nrows, tid));
    }
  };
  float2 pa[H], pb[H];
  if constexpr (real_in) {
    const evx_buf src = evx_make_buf(a.in_r + r0 * NX, kRowRange);
    row_in(src, oa, pa);
    row_in(GS ? evx_make_buf(a.in_r2 + r0 * NX, kRowRange) : src, ob, pb);
    tws.store(twl, tid);
    static_for<H>([&](auto m) {
      constexpr int c0 = V * TPS * (decltype(m)::value / V) + decltype(m)::value % V;
      if (a.flip) {
        pa[m] = flip(sa, pa[m]);
        pb[m] = flip(sb, pb[m]);
      }
      const int lo = X::template at<c0>(V * to, ats), hi = X::template at<NX - 1 - c0>(-V * to, atn);
      rwa[lo] = pa[m].x;
      rwa[hi] = pa[m].y;
      rwb[lo] = pb[m].x;
      rwb[hi] = pb[m].y;
    });
    evx_sync();
    static_for<E>([&](auto e) { x[e] = prs[X::template at<TPS * decltype(e)::value>(t, atp) / 2]; });
    if (!GS && a.fp)
      static_for<E>([&](auto e) { x[e] = row_nonlin<ROW_FUSED, false>(1.0f, nullptr, x[e]); });
    evx_sync();
    if constexpr (GS) react(1.0f);
  } else {
    if constexpr (STAGED) {
      staged([&](auto rows) {
        rows.load(a.in_c);
        tws.store(twl, tid);
        rows.stage(st);
      });
    } else if (a.xcplx) {  // complex columns, one per bin (a periodic y or z follows): real parts
      float qa[E], qb[E];
      spec_points<E>(a.in_c, la, [&](auto e, evx_buf r, unsigned off) {
        qa[e] = evx_buf_load1(r, off);
      });
      spec_points<E>(in_b, lb, [&](auto e, evx_buf r, unsigned off) {
        qb[e] = evx_buf_load1(r, off);
      });
      tws.store(twl, tid);
      static_for<E>([&](auto e) {
        const int k = X::template at<TPS * decltype(e)::value>(to, atx);
        rwa[k] = qa[e];
        rwb[k] = qb[e];
      });
    } else {
      spec_points<H>(a.in_c, la, [&](auto i, evx_buf r, unsigned off) {
        pa[i] = evx_buf_load2(r, off);
      });
      spec_points<H>(in_b, lb, [&](auto i, evx_buf r, unsigned off) {
        pb[i] = evx_buf_load2(r, off);
      });
      tws.store(twl, tid);
      static_for<H>([&](auto i) {
        const int ev = X::template at<2 * TPS * decltype(i)::value>(2 * to, ate);
        const int od = X::template at<2 * TPS * decltype(i)::value>(2 * to + 1, ato);
        rwa[ev] = pa[i].x;
        rwa[od] = pa[i].y;
        rwb[ev] = pb[i].x;
        rwb[od] = pb[i].y;
      });
    }
    evx_sync();
    static_for<E>([&](auto e) {
      const float2 D = prs[X::template at<TPS * decltype(e)::value>(t, atp) / 2];
      const int m = X::template at<NX - TPS * decltype(e)::value>(-t, atm);
      float2 Dr = prs[decltype(e)::value == 0 && t == 0 ? 0 : m / 2];
      if constexpr (decltype(e)::value == 0) Dr = t == 0 ? make_float2(0.f, 0.f) : Dr;
      const float2 wc = cconj(w[e]);
      const float2 za = cmul(wc, make_float2(D.x, -Dr.x));
      const float2 zb = cmul(wc, make_float2(D.y, -Dr.y));
      x[e] = make_float2(za.x - zb.y, za.y + zb.x);
    });
    evx_sync();
    if constexpr (add) {  // real rows to add to: in flight during the transform
      const evx_buf dst = evx_make_buf(a.out_r + r0 * NX, kRowRange);
      row_in(dst, oa, pa);
      row_in(dst, ob, pb);
    }
    fft_regs<NX, +1, B>(x, lds, b, t, twl);
    if constexpr (real_out) {
      static_for<E>([&](auto e) {
        prs[X::template at<TPS * decltype(e)::value>(t, atp) / 2] = cscale(x[e], a.scale);
      });
      evx_sync();
      static_for<H>([&](auto m) {
        constexpr int c0 = V * TPS * (decltype(m)::value / V) + decltype(m)::value % V;
        const int lo = X::template at<c0>(V * to, ats);
        const int hi = X::template at<NX - 1 - c0>(-V * to, atn);
        float2 u = make_float2(rwa[lo], rwa[hi]), v = make_float2(rwb[lo], rwb[hi]);
        if (a.flip) {
          u = flip(sa, u);
          v = flip(sb, v);
        }
        pa[m] = add ? cadd(pa[m], u) : u;
        pb[m] = add ? cadd(pb[m], v) : v;
      });
      const evx_buf dst = evx_make_buf(a.out_r + r0 * NX, kRowRange);
      row_out(dst, oa, pa);
      row_out(dst, ob, pb);
      if constexpr (MODE != ROW_FUSED_REC) return;
      evx_sync();  // the forward transform reuses the exchange area
    }
    if constexpr (GS) {
      react(a.scale);
    } else {
      static_for<E>([&](auto e) { x[e] = row_nonlin<MODE, false>(a.scale, a.poly, x[e]); });
    }
  }
  fft_regs<NX, -1, B>(x, lds, b, t, twl);
  static_for<E>([&](auto e) { put(t + TPS * decltype(e)::value, x[e]); });
  evx_sync();
  static_for<E>([&](auto e) {
    const int k = t + TPS * decltype(e)::value;
    const float2 Q = cconj(get(decltype(e)::value == 0 && t == 0 ? 0 : NX - k));
    const float2 sp = cmul(w[e], cadd(x[e], Q));
    const float2 sm = cmul(w[e], csub(x[e], Q));
    x[e] = make_float2(sp.x, sm.y);
  });
  evx_sync();
  static_for<E>([&](auto e) {
    prs[X::template at<TPS * decltype(e)::value>(t, atp) / 2] = x[e];
  });
  evx_sync();
  if constexpr (STAGED) {
    staged([&](auto rows) { rows.store(a.out_c, st); });
    return;
  }
  if (a.xcplx) {
    spec_points<E>(a.out_c, la, [&](auto e, evx_buf r, unsigned off) {
      evx_buf_store2(r, off, make_float2(rwa[X::template at<TPS * decltype(e)::value>(to, atx)], 0.f));
    });
    spec_points<E>(out_b, lb, [&](auto e, evx_buf r, unsigned off) {
      evx_buf_store2(r, off, make_float2(rwb[X::template at<TPS * decltype(e)::value>(to, atx)], 0.f));
    });
    spec_tail_out<NX, false>(a.out_c, a.sg, la, to, make_float2(0.f, 0.f));
    spec_tail_out<NX, false>(out_b, a.sg, lb, to, make_float2(0.f, 0.f));
    return;
  }
  static_for<H>([&](auto i) {
    const int ev = X::template at<2 * TPS * decltype(i)::value>(2 * to, ate);
    const int od = X::template at<2 * TPS * decltype(i)::value>(2 * to + 1, ato);
    pa[i] = make_float2(rwa[ev], rwa[od]);
    pb[i] = make_float2(rwb[ev], rwb[od]);
  });
  spec_points<H>(a.out_c, la, [&](auto i, evx_buf r, unsigned off) {
    evx_buf_store2(r, off, pa[i]);
  });
  spec_points<H>(out_b, lb, [&](auto i, evx_buf r, unsigned off) {
    evx_buf_store2(r, off, pb[i]);
  });
  spec_tail_out<NX / 2, false>(a.out_c, a.sg, la, to, make_float2(0.f, 0.f));
  spec_tail_out<NX / 2, false>(out_b, a.sg, lb, to, make_float2(0.f, 0.f));
}

// What bounds this pass: with spectral rows staged through LDS it was VALU issue (87% of the SIMD
// cycles at 1024^3 periodic, 96% at 400^3 zero flux, rocprofv3 SQ counters), a third to a half of it
// the staging's addresses.  Spectral rows now move between memory and registers directly (994 ->
// 777 VALU instructions a wave at length 512, about 4000 -> 2300 at 400 zero flux) and their
// mirrored points through the transform's own exchange area.  Measured a pass, before -> after: 400^3
// zero flux 184 -> 151 us, 256^3 zero flux 39.5 -> 34.7, 128^3 10.5 -> 9.0, 48 x 100 x 96 mixed 7.6 ->
// 5.9; forward from real rows at 256^3 37 -> 26 us (1.3 -> 2.6 TB/s each way out of cache); at 1024^3
// it is bound by its access pattern (65 pieces of 512 bytes a block) and stays at 2.1 ms.
template <int NH, int BC, int MODE>
EVX_DEV void rowpass_gs_body(const RowArgs& a, int tid, long long r0, float2* lds);
template <int NH>
EVX_DEV void rowpass_comb_body(const RowArgs& a, int tid, long long r0, float2* lds);

template <int NH, int BC, int MODE, bool STAGED = false>
EVX_DEV void rowpass_body(const RowArgs& a, int tid, int bid, int nblk, float2* lds) {
  using C = RowCfg<NH, BC>;
  constexpr int E = C::E, TPS = C::TPS, B = C::B, T = C::THREADS;
  constexpr bool real_in = MODE == ROW_FWD;
  constexpr bool real_out =
      MODE == ROW_INV || MODE == ROW_INV_ADD || MODE == ROW_FUSED_REC;
  constexpr bool add = MODE == ROW_INV_ADD;
  if constexpr (kEmulated && (MODE == ROW_FUSED_POLY || MODE == ROW_FWD)) {
    if (a.gs) {  // on the GPU a kernel of its own
      const long long r0 = (long long)bid * C::ROWS;
      for (long long r = r0; r < r0 + C::ROWS && r < a.nrows; r += B) {
        rowpass_gs_body<NH, BC, MODE>(a, tid, r, lds);
        evx_sync();
      }
      return;
    }
  }
  if constexpr (kEmulated && BC == BC_PERIODIC && MODE == ROW_INV) {
    if (a.comb) {
      rowpass_comb_body<NH>(a, tid, (long long)bid * C::ROWS, lds);
      return;
    }
  }
  // consecutive row blocks (their 8-row pieces of each x group are neighbours) on one XCD
  const long long r0 = (long long)remap_block(bid, nblk, a.remap) * C::ROWS;
  if constexpr (BC == BC_PERIODIC) {
    int b, t;
    row_lane<B, TPS>(tid, b, t);
    float2 x[E];
    float2* const twl = lds + C::TW;
    PostTw<NH, C::PL> w;
    w.po = lds + C::PO;
    w.t = t;
    // the tables' loads are issued after the data's, and staged once those are in flight
    auto tables = [&] { row_tables<NH, T>(a, tid, t, twl, w); };
    const long long row = r0 + b;
    const bool live = row < a.nrows;
    const SpecLane<TPS> ln(a.sg, r0, b, live, t);
    static_assert(!STAGED || C::SHORT, "rows that are staged are short");
    using SR = SpecRows<B, NH, C::SROW, STAGED ? TPS : 8>;
    using RR = RealRows<B, NH, C::SROW, C::V, T>;
    float2* const rowl = lds + b * C::SROW + t;  // the lane's points of its staged real row
    // vertex-centred x: rows of NH + 1 points, 4 (b (NH + 1) + j) bytes from the block's first
    auto voff = [&](int j) { return live ? unsigned((b * (NH + 1) + j) * 4) : kDeadRow; };
    if constexpr (real_in) {
      real_row_in<NH, B>(a, a.in_r, r0, tid, tables, lds, x);
      static_for<E>([&](auto e) {  // with the halves r2c_post leaves out
        if (a.fp) {
          x[e] = row_nonlin<ROW_FUSED, true>(1.0f, nullptr, x[e]);
        } else {
          x[e] = cscale(x[e], 0.5f);
        }
      });
    } else {
      if constexpr (STAGED) {
        SR sr(a.sg, r0, a.nrows, tid);
        sr.load(a.in_c);
        tables();
        sr.stage(lds);
        evx_sync();
        static_for<E>([&](auto e) {
          const int k = t + TPS * decltype(e)::value;
          x[e] = c2r_pre(rowl[TPS * decltype(e)::value], cconj(lds[b * C::SROW + NH - k]),
                         w.template at<decltype(e)::value>());
        });
        evx_sync();
      } else {
        const float2 nyq = spec_row_in<NH>(a.in_c, a.sg, ln, t, x);
        tables();
        row_c2r<NH, B>(x, nyq, w, lds, b, t);
      }
      // real rows to add to: in flight during the transform
      RR rr(a.out_r, r0, a.nrows);
      if constexpr (add) {
        if (!a.vx) rr.load(tid);
      }
      fft_regs<NH, +1, B>(x, lds, b, t, twl);
      if constexpr (real_out) {
        const float sg =
            a.scale * (a.flip ? dirichlet_sign(row, 0, a.ny, a.flip) : 1.0f);
        if (a.vx) {  // the first NH + 1 of the extension's points are the field's
          const evx_buf dst = evx_make_buf(a.out_r + r0 * (NH + 1), kRowRange);
          static_for<E>([&](auto e) {
            const int j = 2 * (t + TPS * decltype(e)::value);
            const unsigned o0 = j <= NH ? voff(j) : kDeadRow;
            const unsigned o1 = j + 1 <= NH ? voff(j + 1) : kDeadRow;
            float2 v = cscale(x[e], sg);
            if constexpr (add) v = cadd(make_float2(evx_buf_load1(dst, o0), evx_buf_load1(dst, o1)), v);
            evx_buf_store1(dst, o0, v.x);
            evx_buf_store1(dst, o1, v.y);
          });
        } else {
          static_for<E>([&](auto e) { rowl[TPS * decltype(e)::value] = cscale(x[e], sg); });
          evx_sync();
          rr.template store<add>(tid, lds);
        }
        if constexpr (MODE == ROW_FUSED_REC) evx_sync();  // the forward transform reuses the area
        if constexpr (MODE != ROW_FUSED_REC) return;
      }
      static_for<E>([&](auto e) { x[e] = row_nonlin<MODE, true>(a.scale, a.poly, x[e]); });
    }
    // ---------------------------------------------------------------- forward x (R2C)
    fft_regs<NH, -1, B>(x, lds, b, t, twl);
    const float2 nyq = row_r2c<NH, B>(x, w, lds, b, t);
    if constexpr (STAGED) {
      evx_sync();  // the mirrored points are read
      static_for<E>([&](auto e) { rowl[TPS * decltype(e)::value] = x[e]; });
      if (t == 0) rowl[NH] = nyq;
      evx_sync();
      SR(a.sg, r0, a.nrows, tid).store(a.out_c, lds);
    } else {
      spec_row_out<NH>(a.out_c, a.sg, ln, t, x, nyq);
    }
  } else {
    cos_rows<NH, MODE, false, STAGED>(a, tid, r0, lds);
  }
}

// The adjoint step's inverse x pass on a periodic x: rows of in_c (the A operator's image) and in_c2
// (the B operator's, v) become lam = A image - f''(c) v in one pass, c the field in in_r.  Storing
// both and combining them in a kernel of its own moved seven fields instead of four: 9.1 + 6.1 us at
// 128^3, here 9.5, bound like the other 128^3 passes by a launch's chain of loads and exchanges.
template <int NH>
EVX_DEV void rowpass_comb_body(const RowArgs& a, int tid, long long r0, float2* lds) {
  using C = RowCfg<NH, BC_PERIODIC>;
  constexpr int E = C::E, TPS = C::TPS, B = C::B, T = C::THREADS;
  using RR = RealRows<B, NH, C::SROW, C::V, T>;
  int b, t;
  row_lane<B, TPS>(tid, b, t);
  float2 x[E], y[E];
  float2* const twl = lds + C::TW;
  float2* const rowl = lds + b * C::SROW + t;
  PostTw<NH, C::PL> w;
  w.po = lds + C::PO;
  w.t = t;
  const SpecLane<TPS> ln(a.sg, r0, b, r0 + b < a.nrows, t);
  const float2 ny = spec_row_in<NH>(a.in_c2, a.sg, ln, t, y);
  const float2 nx = spec_row_in<NH>(a.in_c, a.sg, ln, t, x);
  row_tables<NH, T>(a, tid, t, twl, w);
  const float sg = a.scale * (a.flip ? dirichlet_sign(r0 + b, 0, a.ny, a.flip) : 1.0f);
  auto back = [&](float2 (&z)[E], float2 nyq) {
    row_c2r<NH, B>(z, nyq, w, lds, b, t);
    fft_regs<NH, +1, B>(z, lds, b, t, twl);
    static_for<E>([&](auto e) { rowl[TPS * decltype(e)::value] = cscale(z[e], sg); });
    evx_sync();
  };
  RR c(a.in_r, r0, a.nrows), v(a.out_r, r0, a.nrows);
  back(y, ny);
  v.unstage(tid, lds);
  evx_sync();
  c.load(tid);  // in flight during the second transform
  back(x, nx);
  auto lam = [](float l, float cc, float vv) { return l - (3.0f * cc * cc - 1.0f) * vv; };
  v.pieces(tid, [&](auto I, unsigned off, int at) {
    const float2 p = lds[at], q = C::V == 2 ? lds[at + C::V - 1] : p;
    const float4 cc = c.r[I], vv = v.r[I];
    const float2 o = make_float2(lam(p.x, cc.x, vv.x), lam(p.y, cc.y, vv.y));
    if constexpr (C::V == 2)
      evx_buf_store4(v.buf, off, make_float4(o.x, o.y, lam(q.x, cc.z, vv.z), lam(q.y, cc.w, vv.w)));
    else
      evx_buf_store2(v.buf, off, o);
  });
}

// The two-species fused x pass: u and v to real rows, one explicit reaction step, and back (MODE
// ROW_FUSED_POLY; ROW_FWD starts from real rows) for the B rows from r0.  Periodic rows: a lane
// holds its points of both species.  Cosine rows: one sequence holds a row of both.
// Bound by memory traffic and occupancy (71 to 235 VGPRs for both species' points, 84 at 256^3, five
// waves a SIMD): 65 us at 256^3 periodic, 4.2 TB/s.  With a reaction kernel, four fields' forward
// transforms and an update kernel of its own a step took 0.61 ms at 256^3; with this pass and the
// multiplier in the z pass 0.19 ms.
template <int NH, int BC, int MODE>
EVX_DEV void rowpass_gs_body(const RowArgs& a, int tid, long long r0, float2* lds) {
  using C = RowCfg<NH, BC>;
  if constexpr (BC != BC_PERIODIC) {
    cos_rows<NH, MODE, true>(a, tid, r0, lds);
  } else {
    constexpr int E = C::E, TPS = C::TPS, B = C::B, T = C::THREADS;
    int b, t;
    row_lane<B, TPS>(tid, b, t);
    const long long row = r0 + b;
    float2 u[E], v[E];
    float2* const twl = lds + C::TW;
    PostTw<NH, C::PL> w;
    w.po = lds + C::PO;
    w.t = t;
    auto tables = [&] { row_tables<NH, T>(a, tid, t, twl, w); };
    const SpecLane<TPS> ln(a.sg, r0, b, row < a.nrows, t);
    if constexpr (MODE == ROW_FWD) {
      real_row_in<NH, B>(a, a.in_r, r0, tid, tables, lds, u);
      real_row_in<NH, B>(a, a.in_r2, r0, tid, [] {}, lds, v);
    } else {
      const float2 nu = spec_row_in<NH>(a.in_c, a.sg, ln, t, u);
      const float2 nv = spec_row_in<NH>(a.in_c2, a.sg, ln, t, v);
      tables();
      row_c2r<NH, B>(u, nu, w, lds, b, t);
      fft_regs<NH, +1, B>(u, lds, b, t, twl);
      row_c2r<NH, B>(v, nv, w, lds, b, t);
      fft_regs<NH, +1, B>(v, lds, b, t, twl);
    }
    const float sg = a.flip ? dirichlet_sign(row, 0, a.ny, a.flip) : 1.0f;
    const float scale = MODE == ROW_FWD ? 1.0f : a.scale;
    const float2 mean = MODE == ROW_FWD ? make_float2(0.f, 0.f) : gs_means(a);
    static_for<E>([&](auto e) {
      gs_react(a, scale, 0.5f, sg, mean.x, mean.y, u[e].x, v[e].x);
      gs_react(a, scale, 0.5f, sg, mean.x, mean.y, u[e].y, v[e].y);
    });
    fft_regs<NH, -1, B>(u, lds, b, t, twl);
    const float2 nu = row_r2c<NH, B>(u, w, lds, b, t);
    spec_row_out<NH>(a.out_c, a.sg, ln, t, u, nu);
    evx_sync();  // the mirrored points are read
    fft_regs<NH, -1, B>(v, lds, b, t, twl);
    const float2 nv = row_r2c<NH, B>(v, w, lds, b, t);
    spec_row_out<NH>(a.out_c2, a.sg, ln, t, v, nv);
  }
}

// ------------------------------------------------------------------ plane pass (small grids)
// On a grid whose xy spectral plane fits in LDS, one workgroup per z plane runs the step's first
// three passes on that plane in place: it reads the plane's NH + 1 complex x bins of NY rows once,
// runs the inverse y transforms, the fused x pass (inverse x, f', forward x) and the forward y
// transforms, and writes the plane back once.  Three launches and three trips through memory
// become one, which is what bounds a step on such grids (every launch carries a few microseconds
// of load-transform-store latency).  The transforms use the same twiddle tables and operation
// order as the column and row passes they replace (and their FFT plans where PlanePlans says so).
// Periodic x and y (and z) only.
struct PlaneArgs {
  float2* W;            // work buffer (grouped layout), read and written in place
  SpecGeom sg;
  int nz, ngx;
  const float2* tw_y;   // exp(-2 pi i j / NY)
  const float2* tw_x;   // exp(-2 pi i j / NH)
  const float2* post;   // exp(-2 pi i k / (2 NH)), k < NH
  float scale;          // 1 / (nx ny nz), applied after the inverse x transform
};

// Per plane size: the FFT plans of the y and x transforms (those of the column and row passes, so
// the results are bitwise theirs) and the lanes of the workgroup, chosen so that one batch covers
// all NH + 1 columns and all NY rows (every lane is a (sequence, part) pair in both) and the
// exchange area fits beside the plane.  Measured on 128 x 128 planes the pass lost to the three
// separate ones (27 us against about 22 us for the three: 128 workgroups fill half the chip), so
// it stops at 64 x 64.
template <int NY, int NH>
struct PlanePlans;
template <>
struct PlanePlans<32, 16> {  // 32 columns (17 live) x 4 lanes, 32 rows x 4 lanes
  using PY = FftPlan<32>;
  using PX = FftPlan<16>;
  static constexpr int THREADS = 128;
};
template <>
struct PlanePlans<64, 32> {  // 64 columns x 16 lanes, 256 rows x 4 lanes
  using PY = FftPlan<64>;
  using PX = FftPlan<32>;
  static constexpr int THREADS = 1024;
};

template <int NY, int NH>
struct PlaneCfg {
  using PY = typename PlanePlans<NY, NH>::PY;
  using PX = typename PlanePlans<NY, NH>::PX;
  static constexpr int THREADS = PlanePlans<NY, NH>::THREADS;
  static constexpr int EY = PY::E, TY = PY::TPS;
  static constexpr int EX = PX::E, TX = PX::TPS;
  static_assert(THREADS % TY == 0 && THREADS % TX == 0, "lanes split into whole sequences");
  static constexpr int NC = NH + 1;                       // live x bins
  // sequences per batch: every lane takes part in every transform (they hold barriers), and
  // lanes past the live columns or rows work on zeros and store nothing
  static constexpr int BY = THREADS / TY;                 // y columns per batch
  static constexpr int BX = THREADS / TX;                 // x rows per batch
  static constexpr int PW = NC % 2 ? NC : NC + 1;        // plane row pitch (odd: rows in distinct banks)
  static constexpr int PLANE = NY * PW;
  static constexpr int XCH = BY * NY > BX * NH ? BY * NY : BX * NH;  // FFT exchange area
  static constexpr int TWY = PLANE + XCH, TWX = TWY + NY, PO = TWX + NH;
  static constexpr int NPOST = NH;
  static constexpr int LDS = PO + NPOST;  // float2 slots
  static constexpr int LOADS = (((NC + 7) / 8) * NY * 8 + THREADS - 1) / THREADS;
};

template <int NY, int NH>
EVX_DEV void planepass_body(const PlaneArgs& a, int tid, int bid, float2* lds) {
  using C = PlaneCfg<NY, NH>;
  constexpr int T = C::THREADS, PW = C::PW, NC = C::NC;
  float2* const P = lds;
  float2* const xch = lds + C::PLANE;
  float2* const twy = lds + C::TWY;
  float2* const twx = lds + C::TWX;
  float2* const pol = lds + C::PO;
  const long long zoff = (long long)bid * a.sg.zstride;  // plane z = bid, group 0
  // tables and the plane, all loads in flight together; group g's rows are one contiguous run
  TableStage<NY, T, float2> sty;
  sty.load(a.tw_y, tid);
  TableStage<NH, T, float2> stx;
  stx.load(a.tw_x, tid);
  TableStage<C::NPOST, T, float2> spo;
  spo.load(a.post, tid);
  constexpr int GRUN = NY * 8;  // float2 of one group's rows of the plane
  float2 r[C::LOADS];
  static_for<C::LOADS>([&](auto I) {
    const int f = tid + T * decltype(I)::value;
    const int g = f / GRUN, rem = f - g * GRUN;
    const bool ok = g < a.ngx;
    r[I] = load_or_zero(a.W, g * a.sg.xstride + zoff + rem, ok);
  });
  sty.store(twy, tid);
  stx.store(twx, tid);
  spo.store(pol, tid);
  static_for<C::LOADS>([&](auto I) {
    const int f = tid + T * decltype(I)::value;
    const int g = f / GRUN, rem = f - g * GRUN;
    const int col = g * 8 + (rem & 7), y = rem >> 3;
    if (g < a.ngx && col < NC) P[y * PW + col] = r[I];
  });
  evx_sync();

  // y transforms of the live columns, C::BY at a time (dir +1 inverse, -1 forward)
  auto y_pass = [&](auto dir_) {
    constexpr int DIR = decltype(dir_)::value;
    constexpr int B = C::BY, E = C::EY, TPS = C::TY;
    const int b = tid % B, t = tid / B;
    for (int c0 = 0; c0 < NC; c0 += B) {  // uniform
      const int col = c0 + b;
      const bool live = col < NC;
      float2 x[E];
      static_for<E>([&](auto e) {
        const int yy = t + TPS * decltype(e)::value;
        x[e] = live ? P[yy * PW + (live ? col : 0)] : make_float2(0.f, 0.f);
      });
      fft_regs<NY, DIR, B, typename C::PY>(x, xch, b, t, twy);
      if (live)
        static_for<E>([&](auto e) { P[(t + TPS * decltype(e)::value) * PW + col] = x[e]; });
      evx_sync();  // the next batch reuses the exchange area
    }
  };
  y_pass(std::integral_constant<int, +1>{});

  // fused x pass on rows of NH + 1 complex bins (the periodic row pass's arithmetic)
  {
    constexpr int B = C::BX, E = C::EX, TPS = C::TX;
    const int b = tid % B, t = tid / B;
    for (int y0 = 0; y0 < NY; y0 += B) {  // uniform
      const bool act = y0 + b < NY;
      float2* const row = P + (act ? y0 + b : 0) * PW;
      float2 x[E];
      // C2R pre-processing: Z[k] = (X[k] + conj X[NH-k]) + i (X[k] - conj X[NH-k]) e^{+2pi i k/NX}
      static_for<E>([&](auto e) {
        const int k = t + TPS * decltype(e)::value;
        if (act) {
          const float2 X = row[k];
          const float2 Xr = cconj(row[NH - k]);
          x[e] = c2r_pre(X, Xr, pol[k]);
        } else {
          x[e] = make_float2(0.f, 0.f);
        }
      });
      fft_regs<NH, +1, B, typename C::PX>(x, xch, b, t, twx);
      static_for<E>([&](auto e) { x[e] = row_nonlin<ROW_FUSED, true>(a.scale, nullptr, x[e]); });
      fft_regs<NH, -1, B, typename C::PX>(x, xch, b, t, twx);
      static_for<E>([&](auto e) { xch[lidx<B>(t + TPS * decltype(e)::value, b)] = x[e]; });
      evx_sync();
      float2 yv[E];
      float2 ynyq = make_float2(0.f, 0.f);
      static_for<E>([&](auto e) {
        const int k = t + TPS * decltype(e)::value;
        const float2 Pk = x[e];
        const float2 Q = cconj(xch[lidx<B>(k == 0 ? 0 : NH - k, b)]);
        yv[e] = r2c_post(Pk, Q, pol[k]);
        if (k == 0) ynyq = make_float2(2.0f * (Pk.x - Pk.y), 0.f);
      });
      evx_sync();  // the exchange area is read; the next batch (or y pass) may write it
      if (act) {
        static_for<E>([&](auto e) { row[t + TPS * decltype(e)::value] = yv[e]; });
        if (t == 0) row[NH] = ynyq;
      }
    }
    evx_sync();
  }
  y_pass(std::integral_constant<int, -1>{});

  // write the plane back; the dead columns of the last group are written as zeros
  static_for<C::LOADS>([&](auto I) {
    const int f = tid + T * decltype(I)::value;
    const int g = f / GRUN, rem = f - g * GRUN;
    const int col = g * 8 + (rem & 7), y = rem >> 3;
    if (g < a.ngx)
      a.W[g * a.sg.xstride + zoff + rem] = col < NC ? P[y * PW + col] : make_float2(0.f, 0.f);
  });
}

}  // namespace evx
