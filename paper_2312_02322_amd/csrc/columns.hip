// Coordinate-list coupling tables and the columns schedule: decoupled (AT)
// dynamics of many initial states per classical path on truncated coupling
// matrices -- the paper's production form (Section III: AT-MQCT with 100
// initial states of water per trajectory, on matrices of about 14.6 M kept
// elements for 206,350 states).
//
// Tables: the stored elements in row order (CSR, each row's columns ascending),
// their values and natural-spline second derivatives per knot, [K][nnz]
// (complex interleaved).  A group of columns that shares a path (at most
// COL_MAX) keeps its amplitudes in column tiles: tile k holds columns k TW ..
// k TW + tw - 1 of every row, [N][tw] complex, so the product's gather of a
// coupled row m reads tw contiguous values.
//
// One launch per RK4 stage: a wave takes one row of one tile.  A row's elements
// are read 64 at a time, one per lane, turned into the spline value at the stage's
// R in FP64 and left in LDS; then LPT lanes (two columns each) per element gather
// the coupled row's phased amplitudes c_m = e^{-iE_m t} a_m, 64 / LPT elements
// side by side, whose sums meet at the end of the row.  The J_x term, the row's
// phase, the RK4 update and the phased amplitudes of the next stage follow in the
// same kernel (Eq. 5).  The classical path is driven by U(R) alone (AT), so it is
// integrated once per group beforehand (Eqs. 7-9 with the driver's force), one
// thread per group.
#include "device.h"

#include <math.h>

#include <algorithm>

namespace mqct {

namespace {

constexpr int CB = 512;         // threads of the row kernels
constexpr int CW = CB / 64;
constexpr int ROWS_PER_WG = CW; // one row per wave
constexpr int OUT_ROWS = 64;    // rows per workgroup of col_out
constexpr int NXCD = 8;         // dies of the device; workgroups are dealt to them round-robin
constexpr int COL_JX = 2;        // entries of a J_x row requested ahead of the product
constexpr int COL_TILE = 64;     // most columns of a tile (two per lane, 32 lanes)
constexpr int COL_GU32 = 8, COL_GU64 = 4;   // gathers in flight per lane, FP32 / FP64

inline size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- loading -----------------------------------------------------------------

// v64[k][e] = values[k][perm[e]] (NC reals per element), counting non-finite values.
__global__ void coo_gather(const double* __restrict__ values, int64_t ld, const int32_t* __restrict__ perm,
                           int64_t nnz, int K, int NC, double* __restrict__ v64,
                           unsigned long long* __restrict__ nonfinite) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const int64_t src = perm[e];
  int bad = 0;
  for (int k = 0; k < K; ++k)
    for (int c = 0; c < NC; ++c) {
      const double v = values[((int64_t)k * ld + src) * NC + c];
      bad += !isfinite(v);
      v64[((int64_t)k * nnz + e) * NC + c] = v;
    }
  if (bad) atomicAdd(nonfinite, (unsigned long long)bad);
}

// Natural cubic spline second derivatives of ncol real columns stored knot-major,
// y[k * ncol + col]: Thomas elimination along the grid.  The elimination factors
// depend on the grid only and are formed once per workgroup in LDS; the forward
// sweep's values are held in y2 until the backward sweep overwrites them.
constexpr int SPL_KMAX = 2048;
__global__ void __launch_bounds__(256)
csr_spline(const double* __restrict__ y, const double* __restrict__ x, int K, int64_t ncol,
           double* __restrict__ y2) {
  __shared__ double den[SPL_KMAX], cp[SPL_KMAX];
  if (threadIdx.x == 0) {
    double cprev = 0.0;
    for (int k = 1; k <= K - 2; ++k) {
      const double hl = x[k] - x[k - 1], hr = x[k + 1] - x[k];
      const double dn = (hl + hr) / 3.0 - (k > 1 ? hl / 6.0 * cprev : 0.0);
      den[k] = dn;
      cprev = hr / 6.0 / dn;
      cp[k] = cprev;
    }
  }
  __syncthreads();
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncol) return;
  y2[c] = 0.0;
  y2[(int64_t)(K - 1) * ncol + c] = 0.0;
  double dprev = 0.0;
  for (int k = 1; k <= K - 2; ++k) {
    const double hl = x[k] - x[k - 1], hr = x[k + 1] - x[k];
    const double yl = y[(int64_t)(k - 1) * ncol + c], y0 = y[(int64_t)k * ncol + c],
                 yr = y[(int64_t)(k + 1) * ncol + c];
    const double rhs = (yr - y0) / hr - (y0 - yl) / hl;
    const double dk = (rhs - (k > 1 ? hl / 6.0 * dprev : 0.0)) / den[k];
    y2[(int64_t)k * ncol + c] = dk;
    dprev = dk;
  }
  double nxt = 0.0;
  for (int k = K - 2; k >= 1; --k) {
    const double v = y2[(int64_t)k * ncol + c] - cp[k] * nxt;
    y2[(int64_t)k * ncol + c] = v;
    nxt = v;
  }
}

// The largest |M_e - conj(M_p)| (p: the partner (m, n) of element e = (n, m))
// and the largest |M| over every knot, as the bit patterns of non-negative doubles.
__global__ void csr_partner_check(const double* __restrict__ v64, const int32_t* __restrict__ partner,
                                  int64_t nnz, int K, int NC,
                                  unsigned long long* __restrict__ maxdiff,
                                  unsigned long long* __restrict__ maxabs) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double dm = 0.0, am = 0.0;
  if (e < nnz) {
    const int64_t p = partner[e];
    for (int k = 0; k < K; ++k) {
      const double* a = v64 + ((int64_t)k * nnz + e) * NC;
      const double* b = v64 + ((int64_t)k * nnz + p) * NC;
      double d = fabs(a[0] - b[0]), m = fabs(a[0]);
      if (NC == 2) {
        d = fmax(d, fabs(a[1] + b[1]));
        m = fmax(m, fabs(a[1]));
      }
      dm = fmax(dm, d);
      am = fmax(am, m);
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    dm = fmax(dm, __shfl_xor(dm, off, 64));
    am = fmax(am, __shfl_xor(am, off, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    atomicMax(maxdiff, (unsigned long long)__double_as_longlong(dm));
    atomicMax(maxabs, (unsigned long long)__double_as_longlong(am));
  }
}

template <typename S>
__global__ void csr_cast(const double* __restrict__ in, int64_t n, S* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (S)in[i];
}

// ---- columns schedule ------------------------------------------------------------

struct ColStage {
  double om;       // dPhi/dt at the stage
  double w[4];     // spline value weights at the stage's R
  int32_t k;       // spline interval
  int32_t pad[5];
};

struct ColArgs {
  const DevSystem* systems;
  const TrajIn* traj;       // records in group order
  const ColGroup* groups;   // [G]
  int G, N, CT;
  int TW;                   // columns per tile (even); the last tile holds the rest
  int nt;                   // tiles of a group
  int64_t nchunk;           // row chunks of one tile in the stage kernel
  int64_t nout;             // row chunks of one group in col_out
  ColStage* st;             // stage records, group g from groups[g].stage_off
  double* fin;              // [G][8]: R, Phi, P_R, P_Phi, theta, P_theta, E0, E1
  int* gstatus;             // [G]
  // [G][tiles][N][tw]:
  double2* A0;              // amplitudes at the start of the step (the input of stage 0)
  double2* ACC;             // RK4 accumulator
  double2* CUR[2];          // amplitudes of stages 2 (buffer 0) and 1, 3 (buffer 1)
  void* C[2];               // phased stage amplitudes in the table precision
  double* part;             // [G][nout][CT] partial norms
};

// Columns of tile k, and where its rows start.
__device__ __forceinline__ int tile_w(const ColArgs& a, int k) { return min(a.TW, a.CT - k * a.TW); }
__device__ __forceinline__ int64_t tile_at(const ColArgs& a, int g, int k) {
  return (int64_t)a.N * ((int64_t)g * a.CT + (int64_t)k * a.TW);
}

// Stage times of step j: t_j + cf_s h with t_j = t0 + j h (Eq. 4's time, RK4 stages).
__device__ __forceinline__ double col_cf(int s) { return s == 0 ? 0.0 : (s == 3 ? 1.0 : 0.5); }

// The classical path of every group (AT: Eqs. 7-9 with the driving potential's
// force, no torque), RK4 with the records of every stage; one thread per group.
__global__ void col_path(ColArgs a) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= a.G) return;
  const ColGroup gr = a.groups[g];
  const TrajIn tj = a.traj[gr.first];
  const DevSystem sy = a.systems[tj.sys];
  const double mu = sy.mu, h = tj.dt;
  double y[4], theta = 0.5 * M_PI, ptheta = 0.0;
  if (tj.flags & TRAJ_HAS_C0) {
    y[0] = tj.c0[0]; theta = tj.c0[1]; y[1] = tj.c0[2]; y[2] = tj.c0[3]; ptheta = tj.c0[4];
    y[3] = tj.c0[5];
  } else {
    const double kk = sqrt(2.0 * mu * tj.E_coll);
    const double pphi = tj.b * kk;
    y[0] = tj.R0; y[1] = 0.0;
    y[2] = -sqrt(2.0 * mu * tj.E_coll - pphi * pphi / (tj.R0 * tj.R0));
    y[3] = pphi;
  }
  int status = 0;
  auto U_of = [&](const Spl& sp) {
    const int k = sp.k;
    return sp.w0 * sy.drv[k] + sp.w1 * sy.drv[k + 1] + sp.w2 * sy.drv2[k] + sp.w3 * sy.drv2[k + 1];
  };
  auto energy = [&](const double (&ys)[4]) {
    const Spl sp = spline_at(sy.R, sy.K, ys[0], sy.R_inv_h);
    return ys[2] * ys[2] / (2.0 * mu) + ys[3] * ys[3] / (2.0 * mu * ys[0] * ys[0]) + U_of(sp);
  };
  auto deriv = [&](const double (&ys)[4], double (&ky)[4], ColStage* rec) {
    const Spl sp = spline_at(sy.R, sy.K, ys[0], sy.R_inv_h);
    if (sp.below) status |= ST_BELOW_GRID;
    const int k = sp.k;
    const double dU = sp.d0 * sy.drv[k] + sp.d1 * sy.drv[k + 1] + sp.d2 * sy.drv2[k] +
                      sp.d3 * sy.drv2[k + 1];
    const double R = ys[0];
    ky[0] = ys[2] / mu;
    ky[1] = ys[3] / (mu * R * R);
    ky[2] = -dU + ys[3] * ys[3] / (mu * R * R * R);
    ky[3] = 0.0;
    ColStage r{};
    r.om = ky[1];
    r.w[0] = sp.w0; r.w[1] = sp.w1; r.w[2] = sp.w2; r.w[3] = sp.w3;
    r.k = k;
    *rec = r;
  };
  const double E0 = energy(y);
  ColStage* rec = a.st + gr.stage_off;
  for (int64_t j = 0; j < gr.n_steps; ++j) {
    double k1[4], k2[4], k3[4], k4[4], ys[4];
    deriv(y, k1, rec + 4 * j);
    for (int i = 0; i < 4; ++i) ys[i] = fma(0.5 * h, k1[i], y[i]);
    deriv(ys, k2, rec + 4 * j + 1);
    for (int i = 0; i < 4; ++i) ys[i] = fma(0.5 * h, k2[i], y[i]);
    deriv(ys, k3, rec + 4 * j + 2);
    for (int i = 0; i < 4; ++i) ys[i] = fma(h, k3[i], y[i]);
    deriv(ys, k4, rec + 4 * j + 3);
    for (int i = 0; i < 4; ++i) {
      const double acc = k1[i] + 2.0 * k2[i] + 2.0 * k3[i] + k4[i];
      y[i] = fma(h / 6.0, acc, y[i]);
    }
  }
  // the end state's interval is checked too (the results are evaluated there)
  if (spline_at(sy.R, sy.K, y[0], sy.R_inv_h).below) status |= ST_BELOW_GRID;
  double* f = a.fin + (int64_t)g * 8;
  f[0] = y[0]; f[1] = y[1]; f[2] = y[2]; f[3] = y[3]; f[4] = theta; f[5] = ptheta;
  f[6] = E0; f[7] = energy(y);
  a.gstatus[g] = status;
}

template <typename CS> struct CV;
template <> struct CV<double> {
  using T = double2;
  __device__ static double2 make(double x, double y) { return make_double2(x, y); }
};
template <> struct CV<float> {
  using T = float2;
  __device__ static float2 make(double x, double y) { return make_float2((float)x, (float)y); }
};

// Start amplitudes of every column (a0, or the initial channel), the stage-0
// input and its phased form at t0.
template <typename CS>
__global__ void __launch_bounds__(CB) col_init(ColArgs a, const double* __restrict__ a0_all) {
  const int64_t item = (int64_t)blockIdx.x * CW + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int g = (int)(item / a.N), n = (int)(item % a.N);
  if (g >= a.G) return;
  const ColGroup gr = a.groups[g];
  const TrajIn t0r = a.traj[gr.first];
  const DevSystem sy = a.systems[t0r.sys];
  double sn, cs;
  sincos(sy.E[n] * t0r.t0, &sn, &cs);
  using C2 = typename CV<CS>::T;
  C2* c = (C2*)a.C[0];
  for (int col = lane; col < a.CT; col += 64) {
    double2 v = make_double2(0.0, 0.0);
    if (col < gr.count) {
      const TrajIn tj = a.traj[gr.first + col];
      if (tj.flags & TRAJ_HAS_A0) v = ((const double2*)a0_all)[tj.amp_off + n];
      else if (n == tj.init_channel) v = make_double2(1.0, 0.0);
    }
    const int k = col / a.TW;
    const int64_t o = tile_at(a, g, k) + (int64_t)n * tile_w(a, k) + (col - k * a.TW);
    a.A0[o] = v;
    c[o] = CV<CS>::make(cs * v.x + sn * v.y, cs * v.y - sn * v.x);
  }
}

__device__ __forceinline__ double rl(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

// Loads and stores of data that is used once per stage.
typedef double dnt2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double2 load_once(const double2* p) {
  const dnt2 v = __builtin_nontemporal_load((const dnt2*)p);
  return make_double2(v.x, v.y);
}
__device__ __forceinline__ void store_once(double2* p, double2 v) {
  __builtin_nontemporal_store(dnt2{v.x, v.y}, (dnt2*)p);
}

// One element of a row in LDS: its column and its spline value in the precision of
// the products.
template <typename CS, bool CPLX> struct ColEnt;
template <> struct alignas(8) ColEnt<float, false> { int m; float v; };
template <> struct alignas(16) ColEnt<float, true> { int m; float v, w; int pad; };
template <> struct alignas(16) ColEnt<double, false> { double v; int m; int pad; };
template <> struct alignas(16) ColEnt<double, true> { double v, w; int m; int pad[3]; };

// One RK4 stage s of step j for every group still running (see the top of the
// file).  S: table precision; CPLX: complex tables; CS: precision of the phased
// amplitudes (and of the products: FP32 products over one 64-element chunk,
// then FP64 sums).
//
// Bound by the round trips of the gathers, which read a kept element's
// coupled row, 8 or 16 B x columns, which stays in a die's 4 MB L2 only if the rows
// of one m-block do.  With all 100 columns side by side the largest blocks (5,300
// rows x 800 B) did not, and the misses bound the kernel; a tile's do (206,350 states,
// FP32, L2 misses of requests a stage: 22 M of 104 M, with the columns side by side 38 M
// of 136 M; the vector units are busy a third of the time, and the gathered bytes are a
// fraction of what L1 and L2 can deliver), for the price of reading the tables once per
// tile.  Rows are dealt to the dies in contiguous ranges of one tile.  Lanes beyond
// a tile's columns would idle, so 64 / LPT elements run side by side.  What the
// row's update reads, and the next chunk's elements, are requested before the
// products (a wave's life is a chain of such round trips); the step's start and
// the accumulator, read once, stay out of the caches.  206,700 states, 13.1 M
// elements, 100 columns: FP32 1.38 ms a stage before, 1.10 now, FP64 2.35 and 1.80;
// N = 30,000, 2 x 37 columns, FP64: 0.288 and 0.158.
template <typename S, bool CPLX, typename CS, int LPT>
__global__ void __launch_bounds__(CB)
col_stage(ColArgs a, int64_t j, int s) {
  constexpr int EP = 64 / LPT;      // elements side by side
  constexpr int GU = sizeof(CS) == 4 ? COL_GU32 : COL_GU64;   // gathers in flight per lane
  using Ent = ColEnt<CS, CPLX>;
  __shared__ Ent ents[CW][64];
  const int64_t items = (int64_t)a.G * a.nt * a.nchunk;
  const int64_t per = (items + NXCD - 1) / NXCD;
  const int64_t pos = (int64_t)(blockIdx.x % NXCD) * per + blockIdx.x / NXCD;
  if (blockIdx.x / NXCD >= per || pos >= items) return;
  const int gt = (int)(pos / a.nchunk);
  const int64_t chunk = pos - (int64_t)gt * a.nchunk;
  const int g = gt / a.nt, k = gt - g * a.nt;
  const ColGroup gr = a.groups[g];
  if (j >= gr.n_steps) return;
  const TrajIn t0r = a.traj[gr.first];
  const DevSystem sy = a.systems[t0r.sys];
  const ColStage rec = a.st[gr.stage_off + 4 * j + s];
  const double h = t0r.dt;
  const double tj = t0r.t0 + (double)j * h;
  const double t = tj + col_cf(s) * h;
  const double tn = s < 3 ? tj + col_cf(s + 1) * h : t0r.t0 + (double)(j + 1) * h;
  using C2 = typename CV<CS>::T;
  const int64_t base = tile_at(a, g, k);
  const int tw = tile_w(a, k);
  const C2* __restrict__ cin = (const C2*)a.C[s & 1] + base;
  C2* __restrict__ cout = (C2*)a.C[(s & 1) ^ 1] + base;
  const double2* __restrict__ curin = (s == 0 ? a.A0 : a.CUR[s & 1]) + base;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nl = chunk * ROWS_PER_WG + wave;
  if (nl >= a.N) return;
  const int n = (int)nl;
  const int grp = lane / LPT;
  const int c0 = 2 * (lane % LPT);
  const bool act = c0 < tw;
  const int64_t nnz = sy.knot_stride;
  constexpr int NC = CPLX ? 2 : 1;
  const S* __restrict__ V0 = (const S*)sy.M + (int64_t)rec.k * nnz * NC;
  const S* __restrict__ V1 = V0 + nnz * NC;
  const S* __restrict__ D0 = (const S*)sy.M2 + (int64_t)rec.k * nnz * NC;
  const S* __restrict__ D1 = D0 + nnz * NC;
  const double w0 = rec.w[0], w1 = rec.w[1], w2 = rec.w[2], w3 = rec.w[3];
  const C2* cg = cin + (act ? c0 : 0);
  Ent* ent = ents[wave];
  const int rs = sy.csr_row[n], re = sy.csr_row[n + 1];
  // what the row's update reads -- this lane's column of the step's start, of the
  // accumulator and of the rows coupled by J_x -- is requested before the product
  const bool upd = act && grp < 2;      // lane group 0 updates a pair's first column, 1 its second
  const int col = c0 + (grp & 1);
  const int64_t o = (int64_t)n * tw + col, ob = base + o;
  const int jw = sy.jx_w;
  double2 av0 = make_double2(0.0, 0.0), ac = av0, jav[COL_JX];
  double jv[COL_JX];
#pragma unroll
  for (int w = 0; w < COL_JX; ++w) {
    jav[w] = av0;
    jv[w] = 0.0;
    if (upd && w < jw) {
      jv[w] = sy.jx_val[(int64_t)n * jw + w];
      jav[w] = curin[(int64_t)sy.jx_col[(int64_t)n * jw + w] * tw + col];
    }
  }
  if (upd) {
    av0 = load_once(a.A0 + ob);
    if (s > 0) ac = load_once(a.ACC + ob);
  }
  // the row's phases at t (even lanes) and tn (odd lanes)
  double sns, css;
  sincos(sy.E[n] * ((lane & 1) ? tn : t), &sns, &css);
  // a chunk's elements, one per lane; the next chunk's are requested before the
  // current one's products
  auto fetch = [&](int e, int& m, S (&x)[4], S (&xi)[4]) {
    m = n;         // entries past the row's end read the row's own amplitudes and add zero
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = xi[q] = 0;
    if (e < re) {
      m = sy.csr_col[e];
      const S* const T[4] = {V0, V1, D0, D1};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        x[q] = T[q][(int64_t)e * NC];
        if constexpr (CPLX) xi[q] = T[q][(int64_t)e * NC + 1];
      }
    }
  };
  int mq;
  S xq[4], xiq[4];
  fetch(rs + lane, mq, xq, xiq);
  double y0x = 0.0, y0y = 0.0, y1x = 0.0, y1y = 0.0;
  for (int e0 = rs; e0 < re; e0 += 64) {
    Ent en{};
    en.m = mq;
    en.v = (CS)(w0 * (double)xq[0] + w1 * (double)xq[1] + w2 * (double)xq[2] + w3 * (double)xq[3]);
    if constexpr (CPLX)
      en.w = (CS)(w0 * (double)xiq[0] + w1 * (double)xiq[1] + w2 * (double)xiq[2] +
                  w3 * (double)xiq[3]);
    __builtin_amdgcn_wave_barrier();   // the previous chunk's entries are consumed (in order)
    ent[lane] = en;
    __builtin_amdgcn_wave_barrier();
    if (e0 + 64 < re) fetch(e0 + 64 + lane, mq, xq, xiq);
    const int steps = (min(64, re - e0) + EP - 1) / EP;
    CS p0x = 0, p0y = 0, p1x = 0, p1y = 0;
    for (int i = 0; i < steps; i += GU) {
      // i + u < LPT (a multiple of GU), so the entries stay within the 64
      C2 g0[GU], g1[GU];
      CS br[GU], bi[GU];
#pragma unroll
      for (int u = 0; u < GU; ++u) {
        const Ent x = ent[(i + u) * EP + grp];
        br[u] = x.v;
        if constexpr (CPLX) bi[u] = x.w;
        const C2* src = cg + (int64_t)x.m * tw;
        if constexpr (sizeof(CS) == 4) {
          // the pair's 16 bytes at once (tw and c0 are even, the arrays 256-byte aligned)
          const float4 v = *(const float4*)src;
          g0[u] = C2{v.x, v.y};
          g1[u] = C2{v.z, v.w};
        } else {
          g0[u] = src[0];
          g1[u] = src[1];
        }
      }
#pragma unroll
      for (int u = 0; u < GU; ++u) {
        p0x += br[u] * g0[u].x; p0y += br[u] * g0[u].y;
        p1x += br[u] * g1[u].x; p1y += br[u] * g1[u].y;
        if constexpr (CPLX) {
          p0x -= bi[u] * g0[u].y; p0y += bi[u] * g0[u].x;
          p1x -= bi[u] * g1[u].y; p1y += bi[u] * g1[u].x;
        }
      }
    }
    y0x += (double)p0x; y0y += (double)p0y; y1x += (double)p1x; y1y += (double)p1y;
  }
  // the side-by-side sums of each column pair, then one column per lane
#pragma unroll
  for (int x = LPT; x < 64; x <<= 1) {
    y0x += __shfl_xor(y0x, x, 64); y0y += __shfl_xor(y0y, x, 64);
    y1x += __shfl_xor(y1x, x, 64); y1y += __shfl_xor(y1y, x, 64);
  }
  const double sn = rl(sns, 0), cs = rl(css, 0), sn2 = rl(sns, 1), cs2 = rl(css, 1);
  if (!upd) return;
  const double yx = grp ? y1x : y0x, yy = grp ? y1y : y0y;
  // J_x a of this row (couples states of equal energy, Eq. 5)
  double xx = 0.0, xy = 0.0;
#pragma unroll
  for (int w = 0; w < COL_JX; ++w) {
    xx = fma(jv[w], jav[w].x, xx);
    xy = fma(jv[w], jav[w].y, xy);
  }
  for (int w = COL_JX; w < jw; ++w) {
    const double2 av = curin[(int64_t)sy.jx_col[(int64_t)n * jw + w] * tw + col];
    const double jvw = sy.jx_val[(int64_t)n * jw + w];
    xx = fma(jvw, av.x, xx);
    xy = fma(jvw, av.y, xy);
  }
  // da/dt = -i (e^{iE_n t} (M c)_n + Phidot (J_x a)_n)
  const double Gx = cs * yx - sn * yy + rec.om * xx;
  const double Gy = cs * yy + sn * yx + rec.om * xy;
  const double fx = Gy, fy = -Gx;
  double2 nx;
  if (s == 0) {
    store_once(a.ACC + ob, make_double2(fx, fy));
    nx = make_double2(fma(0.5 * h, fx, av0.x), fma(0.5 * h, fy, av0.y));
    a.CUR[1][ob] = nx;
  } else if (s < 3) {
    store_once(a.ACC + ob, make_double2(fma(2.0, fx, ac.x), fma(2.0, fy, ac.y)));
    const double cfn = s == 1 ? 0.5 * h : h;
    nx = make_double2(fma(cfn, fx, av0.x), fma(cfn, fy, av0.y));
    a.CUR[(s & 1) ^ 1][ob] = nx;
  } else {
    // the next step's stage 0 reads its input from A0 (no other row reads A0 here)
    nx = make_double2(fma(h / 6.0, ac.x + fx, av0.x), fma(h / 6.0, ac.y + fy, av0.y));
    store_once(a.A0 + ob, nx);
  }
  cout[o] = CV<CS>::make(cs2 * nx.x + sn2 * nx.y, cs2 * nx.y - sn2 * nx.x);
}

// Final probabilities and amplitudes of every column, and its norm over OUT_ROWS
// rows (summed by col_fin).  The results are stored column after column, the
// amplitudes row after row: 64 rows x 32 columns turn in LDS, so both sides are
// read and written in whole lines (0.58 ms for 206,350 x 100 by strided stores).
constexpr int OUT_COLS = 32;
__global__ void __launch_bounds__(256) col_out(ColArgs a, TrajOut out) {
  __shared__ double2 buf[OUT_COLS][OUT_ROWS + 1];
  const int64_t item = blockIdx.x;
  const int nsub = (a.CT + OUT_COLS - 1) / OUT_COLS;
  const int sub = (int)(item % nsub);
  const int64_t gc = item / nsub;
  const int g = (int)(gc / a.nout);
  const int64_t chunk = gc - (int64_t)g * a.nout;
  const ColGroup gr = a.groups[g];
  const int64_t n0 = chunk * OUT_ROWS;
  const int rows = (int)min((int64_t)OUT_ROWS, a.N - n0);
  const int cl = threadIdx.x % OUT_COLS, col = sub * OUT_COLS + cl;
  if (col < a.CT) {
    const int k = col / a.TW, tw = tile_w(a, k);
    const double2* src = a.A0 + tile_at(a, g, k) + (col - k * a.TW);
    for (int r = threadIdx.x / OUT_COLS; r < rows; r += 256 / OUT_COLS)
      buf[cl][r] = src[(n0 + r) * tw];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  for (int c = threadIdx.x >> 6; c < OUT_COLS; c += 4) {
    const int cc = sub * OUT_COLS + c;
    if (cc >= a.CT) break;
    double p[1] = {0.0};
    if (lane < rows) {
      const double2 v = buf[c][lane];
      p[0] = v.x * v.x + v.y * v.y;
      if (cc < gr.count) {
        const int64_t o = a.traj[gr.first + cc].amp_off + n0 + lane;
        if (out.P) out.P[o] = p[0];
        if (out.a_final) ((double2*)out.a_final)[o] = v;
      }
    }
    wave_sum<1>(p);
    if (lane == 0) a.part[((int64_t)g * a.nout + chunk) * a.CT + cc] = p[0];
  }
}

// Per column: the norm (16 runs of partials, then the runs in order), the path's
// end state and diagnostics (AT: the driven energy P_R^2/2mu + P_Phi^2/(2 mu R^2) +
// U(R) and P_Phi).  One workgroup per group and 64 columns.
constexpr int FIN_SEG = 16;
__global__ void __launch_bounds__(64 * FIN_SEG) col_fin(ColArgs a, TrajOut out) {
  __shared__ double seg[FIN_SEG][64];
  const int g = blockIdx.x, lane = threadIdx.x & 63, sg = threadIdx.x >> 6;
  const int col = blockIdx.y * 64 + lane;
  const ColGroup gr = a.groups[g];
  const bool real = col < gr.count;
  double s = 0.0;
  if (real) {
    const int64_t c1 = a.nout * (sg + 1) / FIN_SEG;
#pragma unroll 8
    for (int64_t c = a.nout * sg / FIN_SEG; c < c1; ++c)
      s += a.part[((int64_t)g * a.nout + c) * a.CT + col];
  }
  seg[sg][lane] = s;
  __syncthreads();
  if (sg > 0 || !real) return;
  const TrajIn tj = a.traj[gr.first + col];
  double nrm = 0.0;
  for (int q = 0; q < FIN_SEG; ++q) nrm += seg[q][lane];
  const double* f = a.fin + (int64_t)g * 8;
  const int64_t id = tj.id;
  if (out.classical) {
    double* o = out.classical + id * 6;
    o[0] = f[0]; o[1] = f[4]; o[2] = f[1]; o[3] = f[2]; o[4] = f[5]; o[5] = f[3];
  }
  if (out.t_final) out.t_final[id] = tj.t0 + (double)gr.n_steps * tj.dt;
  if (out.steps) out.steps[id] = gr.n_steps;
  if (out.rejects) out.rejects[id] = 0;
  if (out.status) out.status[id] = a.gstatus[g];
  if (out.norm_err) out.norm_err[id] = nrm - 1.0;
  if (out.energy_err) out.energy_err[id] = (f[7] - f[6]) / fabs(f[6]);
  if (out.angmom_err) out.angmom_err[id] = 0.0;   // no torque: P_Phi is constant
}

// Columns per tile: tiles of equal width, even (two columns per lane), as few as
// hold COL_TILE columns each.  Narrower tiles waste lanes and repeat the row's
// fixed work: 100 columns, 206,700 states, per 32 stages, FP32 35.6 ms as 2 x 50,
// 43.1 as one, 46.3 as 4 x 25; FP64 58.0 as 2 x 50, 75.6 as 3 x 34; N = 30,000 and
// 37 columns, FP64, 48 stages: 7.9 ms as one, 10.3 as 2 x 20.
int col_tile(int CT) {
  const int nt = (CT + COL_TILE - 1) / COL_TILE;
  return ((CT + nt - 1) / nt + 1) & ~1;
}

template <typename S, bool CPLX, typename CS>
void launch_stage(const ColArgs& a, unsigned grid, int64_t j, int st, hipStream_t s) {
  if (a.TW <= 16) col_stage<S, CPLX, CS, 8><<<grid, CB, 0, s>>>(a, j, st);
  else if (a.TW <= 32) col_stage<S, CPLX, CS, 16><<<grid, CB, 0, s>>>(a, j, st);
  else col_stage<S, CPLX, CS, 32><<<grid, CB, 0, s>>>(a, j, st);
}

}  // namespace

// ---- host ------------------------------------------------------------------------

hipError_t launch_coo_gather(const double* values, int64_t ld, const int32_t* perm, int64_t nnz,
                             int K, int NC, double* v64, unsigned long long* nonfinite,
                             hipStream_t s) {
  coo_gather<<<(unsigned)((nnz + 255) / 256), 256, 0, s>>>(values, ld, perm, nnz, K, NC, v64,
                                                           nonfinite);
  return hipGetLastError();
}

hipError_t launch_csr_spline(const double* y, const double* x, int K, int64_t ncol, double* y2,
                             hipStream_t s) {
  csr_spline<<<(unsigned)((ncol + 255) / 256), 256, 0, s>>>(y, x, K, ncol, y2);
  return hipGetLastError();
}

hipError_t launch_csr_partner_check(const double* v64, const int32_t* partner, int64_t nnz, int K,
                                    int NC, unsigned long long* maxdiff,
                                    unsigned long long* maxabs, hipStream_t s) {
  csr_partner_check<<<(unsigned)((nnz + 255) / 256), 256, 0, s>>>(v64, partner, nnz, K, NC,
                                                                  maxdiff, maxabs);
  return hipGetLastError();
}

hipError_t launch_csr_cast_f32(const double* in, int64_t n, float* out, hipStream_t s) {
  csr_cast<float><<<(unsigned)((n + 255) / 256), 256, 0, s>>>(in, n, out);
  return hipGetLastError();
}

size_t columns_workspace_bytes(int G, int N, int CT, int64_t stages, bool fp32) {
  const size_t v = (size_t)G * N * CT;
  const int64_t nout = (N + OUT_ROWS - 1) / OUT_ROWS;
  size_t b = 0;
  b += al((size_t)G * sizeof(ColGroup));
  b += al((size_t)std::max<int64_t>(stages, 1) * sizeof(ColStage));
  b += al((size_t)G * 8 * 8) + al((size_t)G * 4);
  b += 4 * al(v * 16);
  b += 2 * al(v * (fp32 ? 8 : 16));
  b += al((size_t)G * nout * CT * 8);
  return b;
}

hipError_t run_columns(const DevSystem* d_systems, const DevSystem& hs, const TrajIn* d_traj,
                       const std::vector<ColGroup>& groups, int CT, const double* d_a0,
                       TrajOut out, void* wsp, hipStream_t s) {
  const int G = (int)groups.size();
  const int N = hs.N;
  const bool fp32 = dtype_fp32(hs.dtype);
  int64_t stages = 0, nmax = 0;
  for (const ColGroup& g : groups) {
    stages = std::max(stages, g.stage_off + 4 * g.n_steps);
    nmax = std::max(nmax, g.n_steps);
  }
  ColArgs a{};
  a.systems = d_systems;
  a.traj = d_traj;
  a.G = G;
  a.N = N;
  a.CT = CT;
  a.TW = col_tile(CT);
  a.nt = (CT + a.TW - 1) / a.TW;
  a.nchunk = (N + ROWS_PER_WG - 1) / ROWS_PER_WG;
  a.nout = (N + OUT_ROWS - 1) / OUT_ROWS;
  char* p = (char*)wsp;
  auto take = [&](size_t bytes) { void* q = p; p += al(bytes); return q; };
  ColGroup* dg = (ColGroup*)take((size_t)G * sizeof(ColGroup));
  a.groups = dg;
  a.st = (ColStage*)take((size_t)std::max<int64_t>(stages, 1) * sizeof(ColStage));
  a.fin = (double*)take((size_t)G * 8 * 8);
  a.gstatus = (int*)take((size_t)G * 4);
  const size_t v = (size_t)G * N * CT;
  a.A0 = (double2*)take(v * 16);
  a.ACC = (double2*)take(v * 16);
  a.CUR[0] = (double2*)take(v * 16);
  a.CUR[1] = (double2*)take(v * 16);
  a.C[0] = take(v * (fp32 ? 8 : 16));
  a.C[1] = take(v * (fp32 ? 8 : 16));
  a.part = (double*)take((size_t)G * a.nout * CT * 8);
  hipError_t e;
  if ((e = hipMemcpyAsync(dg, groups.data(), (size_t)G * sizeof(ColGroup), hipMemcpyHostToDevice,
                          s)) != hipSuccess)
    return e;
  col_path<<<(G + 63) / 64, 64, 0, s>>>(a);
  const unsigned init_grid = (unsigned)(((int64_t)G * N + CW - 1) / CW);
  if (fp32) col_init<float><<<init_grid, CB, 0, s>>>(a, d_a0);
  else col_init<double><<<init_grid, CB, 0, s>>>(a, d_a0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t items = (int64_t)G * a.nt * a.nchunk;
  const int64_t outs = (int64_t)G * a.nout * ((CT + OUT_COLS - 1) / OUT_COLS);
  if (items + NXCD > 0x7fffffffLL || outs > 0x7fffffffLL) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((items + NXCD - 1) / NXCD * NXCD);
  for (int64_t j = 0; j < nmax; ++j)
    for (int st = 0; st < 4; ++st) {
      if (hs.dtype == R64) launch_stage<double, false, double>(a, grid, j, st, s);
      else if (hs.dtype == C128) launch_stage<double, true, double>(a, grid, j, st, s);
      else if (hs.dtype == R32) launch_stage<float, false, float>(a, grid, j, st, s);
      else launch_stage<float, true, float>(a, grid, j, st, s);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  col_out<<<(unsigned)outs, 256, 0, s>>>(a, out);
  col_fin<<<dim3((unsigned)G, COL_MAX / 64), 64 * FIN_SEG, 0, s>>>(a, out);
  return hipGetLastError();
}

}  // namespace mqct
