// Shared-stream form of the right-hand side and of the steppers: one workgroup per
// trajectory, for trajectories that have a compute unit (nearly) to themselves --
// small batches, and the last trajectories of a large one.  There nothing is
// bound by bandwidth or arithmetic: an evaluation is one chain of dependent round
// trips, reductions and FP64 operations, and the form is built to shorten it.
//
// * Thread t owns row t (amplitude, phases, J_x, derivative).  The stream over the
//   stored rows is shared out differently: the threads form BLOCK / (Npad / VEC)
//   shares of one thread per 16-byte column group, each share streams its part of
//   the rows with two batches of SB rows in flight per lane, and the shares' partial
//   sums meet in LDS, where the row's owner adds them in share order.
// * The phases e^{-iEt} of all stage times of a step are formed together before the
//   step by all threads (they depend on the times only), not one after the other in
//   the stages.
// * E, the grid and 1/h of its intervals sit in LDS, a row's J_x entries in
//   registers; the interval search starts from the last evaluation's interval.
// * One division per evaluation (1/R); the reductions run through DPP and carry
//   only what the stage uses.
// * The adaptive stepper accumulates the inputs of all later stages and the error
//   estimate as each stage derivative appears (the same sums in the same order as
//   reading the stored derivatives back), so no derivative leaves the registers.
//
// Precision as in rhs.h: FP64 tables FP64 throughout; FP32 tables multiply in FP32
// and add SB-row partial sums into FP64.
//
// Measured, microseconds per evaluation against the row-split form: N = 49 FP64, 64
// trajectories 3.5 (7.3), 512 trajectories 4.5 (8.8); N = 100, 64 trajectories 6.6
// (12.1); N = 256 sparse (36 slots) FP64, 64 trajectories 6.4 (10.9).  What is left is
// about 2.6 us of dependent FP64 operations, LDS trips, reductions and barriers and
// the stream (295 KB per evaluation at N = 256, 2 us at the L1 rate).
#pragma once

#include "rhs.h"

namespace mqct {
namespace shared {

using rhs::Sums;
using rhs::Tr;

// Multiply-adds are written out, so that every kernel built from this code (one
// attempt per launch or several) rounds alike.
#pragma clang fp contract(off)

constexpr int GRID_LDS = 512;   // grids up to this many knots are held in LDS
constexpr int NPH = 5;          // stage times whose phases are held
constexpr int JXB = 4;          // J_x entries of a row held in registers

// LDS layout: [Npad] CS (FP32 tables), [Npad] double2 c, red 2 x [16][8], part
// 2 x [BLOCK * VEC] double2, E [Npad], ph [NPH][Npad] double2, x [GRID_LDS], 1/h [GRID_LDS]
__host__ __device__ inline size_t lds_bytes(int npad, bool fp32, int block, int vec) {
  return (fp32 ? (size_t)npad * 8 : 0) + (size_t)npad * 16 + 2 * 16 * 8 * 8 +
         (size_t)block * vec * 32 + (size_t)npad * 8 + (size_t)NPH * npad * 16 +
         2 * GRID_LDS * 8;
}
// Whether a workgroup of `block` threads can run the form: a thread for every row, at
// least two shares.
__host__ __device__ inline bool fits(int npad, int vec, int block) {
  return npad <= block && 2 * (npad / vec) <= block;
}

// Sum over one wave by DPP shifts (lane 63 holds the total), identical in every lane.
template <int CTRL, int MASK>
__device__ __forceinline__ double dpp_get(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, MASK, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <int NV>
__device__ __forceinline__ void wave_total(double (&v)[NV]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_get<0x111, 0xf>(v[i]);   // row_shr:1
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_get<0x112, 0xf>(v[i]);   // row_shr:2
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_get<0x114, 0xf>(v[i]);   // row_shr:4
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_get<0x118, 0xf>(v[i]);   // row_shr:8
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_get<0x142, 0xa>(v[i]);   // row_bcast:15
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_get<0x143, 0xc>(v[i]);   // row_bcast:31
}

template <int DT, int BLOCK>
struct SK {
  using T = Tr<DT>;
  using S = typename T::S;
  using L = typename T::L;
  using CS = typename T::CS;
  static constexpr int VEC = T::VEC;
  static constexpr int NW = BLOCK / 64;
  static constexpr bool FP32 = (DT == C64 || DT == R32);
  static constexpr bool CPLX = T::CPLX;
  static constexpr int NCOMP = CPLX ? 2 : 1;
  static constexpr int SB = 2;   // rows per batch, two batches in flight
  using F = typename std::conditional<FP32, float, double>::type;
  using F2 = typename std::conditional<FP32, float2, double2>::type;

  // What a workgroup keeps of its trajectory's system.
  struct Own {
    int npad;          // what the LDS areas are sized for (offsets below)
    // byte offsets, so that every access is known to be to LDS
    template <typename X>
    __device__ static X* at(int off) {
      extern __shared__ __align__(16) unsigned char smem[];
      return (X*)(smem + off);
    }
    __device__ int o64() const { return FP32 ? npad * 8 : 0; }
    __device__ int ored() const { return o64() + npad * 16; }
    __device__ int opart() const { return ored() + 2 * 16 * 8 * 8; }
    __device__ int oE() const { return opart() + BLOCK * VEC * 32; }
    __device__ int oph() const { return oE() + npad * 8; }
    __device__ int ox() const { return oph() + NPH * npad * 16; }
    __device__ CS* c() const { return at<CS>(0); }
    __device__ double2* c64() const { return at<double2>(o64()); }
    __device__ double* red() const { return at<double>(ored()); }    // two areas, used in turn
    __device__ double2* part() const { return at<double2>(opart()); }   // u, then v
    __device__ double* E() const { return at<double>(oE()); }
    __device__ double2* ph() const { return at<double2>(oph()); }
    __device__ double* x() const { return at<double>(ox()); }        // grid, 1/h (if it fits)
    __device__ double* rh() const { return at<double>(ox() + GRID_LDS * 8); }
    int n, N, Npad, K, k;
    bool row, lds_grid;
    int jw, jc[JXB];
    double jv[JXB];
    double En, mu, imu, x0, xl;
    int ngroups, shares, grp, sb, se;
    bool on;
    int side;          // reduction area of the next reduction
  };

  __device__ static void setup(Own& o, const DevSystem& sy, int npad) {
    o.npad = npad;
    const int t = threadIdx.x;
    o.N = sy.N; o.Npad = sy.Npad; o.K = sy.K;
    o.n = min(t, sy.N - 1);
    o.row = t < sy.N;
    o.jw = sy.jx_w;
#pragma unroll
    for (int q = 0; q < JXB; ++q) {
      const bool in = q < o.jw && o.jw <= JXB;
      o.jc[q] = in ? sy.jx_col[(int64_t)o.n * o.jw + q] : o.n;
      o.jv[q] = in ? sy.jx_val[(int64_t)o.n * o.jw + q] : 0.0;
    }
    o.En = sy.E[o.n];
    if (t < sy.Npad) o.E()[t] = o.row ? o.En : 0.0;
    o.lds_grid = sy.K <= GRID_LDS;
    if (o.lds_grid)
      for (int i = t; i < sy.K; i += BLOCK) {
        const double xi = sy.R[i];
        o.x()[i] = xi;
        o.rh()[i] = i + 1 < sy.K ? 1.0 / (sy.R[i + 1] - xi) : 0.0;
      }
    o.x0 = sy.R[0];
    o.xl = sy.R[sy.K - 1];
    o.mu = sy.mu;
    o.imu = 1.0 / sy.mu;
    o.k = -1;
    o.side = 0;
    o.ngroups = sy.Npad / VEC;
    o.shares = BLOCK / o.ngroups;
    const int q = t / o.ngroups;
    o.grp = t - q * o.ngroups;
    o.on = q < o.shares;
    const int nst = sy.ell_w > 0 ? sy.ell_w : sy.N;
    o.shares = min(o.shares, nst);
    o.on = q < o.shares;
    o.sb = o.on ? nst * q / o.shares : 0;
    o.se = o.on ? nst * (q + 1) / o.shares : 0;
    __syncthreads();
  }

  // Phases of the owned rows at the times ts[0 .. np): (cos E t, sin E t) in LDS.
  __device__ static void phases(const Own& o, const double (&ts)[NPH], int np) {
    for (int i = threadIdx.x; i < np * o.Npad; i += BLOCK) {
      const int p = i / o.Npad, n = i - p * o.Npad;
      const double t = p == 0 ? ts[0] : p == 1 ? ts[1] : p == 2 ? ts[2] : p == 3 ? ts[3] : ts[4];
      double sn, cs;
      sincos(o.E()[n] * t, &sn, &cs);
      o.ph()[i] = make_double2(cs, sn);
    }
    __syncthreads();
  }

  // Sum NV values over the workgroup, identical in every lane; one barrier.  The two
  // areas alternate, so a reduction never overwrites one that a slower wave reads.
  template <int NV>
  __device__ static void reduce(Own& o, double (&v)[NV]) {
    wave_total<NV>(v);
    double* red = o.red() + o.side * 16 * 8;
    o.side ^= 1;
    if ((threadIdx.x & 63) == 63) {
#pragma unroll
      for (int i = 0; i < NV; ++i) red[i * NW + (threadIdx.x >> 6)] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      double s = red[i * NW];
#pragma unroll
      for (int q = 1; q < NW; ++q) s += red[i * NW + q];
      v[i] = uni(s);
    }
  }

  // Interval and weights (device.h spline_at, with 1/h from LDS and the search
  // started at the last evaluation's interval).  The off-grid cases are selects, so
  // that the weights stay in registers.
  __device__ static Spl spline(Own& o, const DevSystem& sy, double R) {
    int k = o.k;
    double xa, xb, r;
    if (o.lds_grid) {
      if (k < 0) {
        k = 0;
        int hi = o.K - 2;
        while (k < hi) {
          const int mid = (k + hi + 1) >> 1;
          if (o.x()[mid] <= R) k = mid; else hi = mid - 1;
        }
      }
      xa = o.x()[k]; xb = o.x()[k + 1]; r = o.rh()[k];
      // bounded by the grid: each turn moves one interval towards R (a NaN stays put)
      for (int q = 0; q < o.K; ++q) {
        if (R < xa && k > 0) --k;
        else if (R >= xb && k < o.K - 2) ++k;
        else break;
        xa = o.x()[k]; xb = o.x()[k + 1]; r = o.rh()[k];
      }
    } else {
      k = 0;
      int hi = o.K - 2;
      while (k < hi) {
        const int mid = (k + hi + 1) >> 1;
        if (sy.R[mid] <= R) k = mid; else hi = mid - 1;
      }
      xa = sy.R[k]; xb = sy.R[k + 1]; r = 1.0 / (xb - xa);
    }
    k = __builtin_amdgcn_readfirstlane(k);
    o.k = k;
    Spl s;
    s.k = k;
    s.below = R < o.x0;
    const bool above = R > o.xl;
    const double h = xb - xa, h6 = h * (1.0 / 6.0);
    const double A = (xb - R) * r, B = 1.0 - A, h26 = h * h6;
    const double A2 = A * A, B2 = B * B, dR = R - o.x0;
    const double d2 = fma(-3.0, A2, 1.0) * h6, d3 = fma(3.0, B2, -1.0) * h6;
    s.d0 = above ? 0.0 : -r;
    s.d1 = above ? 0.0 : r;
    s.d2 = above ? 0.0 : s.below ? -2.0 * h6 : d2;
    s.d3 = above ? 0.0 : s.below ? -h6 : d3;
    s.w0 = above ? 0.0 : s.below ? fma(dR, s.d0, 1.0) : A;
    s.w1 = above ? 1.0 : s.below ? dR * s.d1 : B;
    s.w2 = above ? 0.0 : s.below ? dR * s.d2 : fma(A2, A, -A) * h26;
    s.w3 = above ? 0.0 : s.below ? dR * s.d3 : fma(B2, B, -B) * h26;
    return s;
  }

  __device__ static void split(const L& v, F (&re)[VEC], F (&im)[VEC]) {
    if constexpr (DT == C128) { re[0] = v.x; im[0] = v.y; }
    else if constexpr (DT == C64) { re[0] = v.x; im[0] = v.y; re[1] = v.z; im[1] = v.w; }
    else { re[0] = v.x; re[1] = v.y; im[0] = im[1] = (F)0; }
  }

  struct Batch {
    int ci[SB][VEC];
    L tv[SB][4];
  };

  // The owned row's derivative da/dt at the amplitude a (all other rows alike), phases
  // ph[p], classical R and P_Phi.  tot: force, torque and norm; with full also the
  // sums of the diagnostics.
  __device__ static double2 eval(Own& o, const DevSystem& sy, int p, double R, double pphi,
                                 double2 a, Sums& tot, bool& below, double& phidot, bool at,
                                 bool full) {
    const Spl sp = spline(o, sy, R);
    below |= sp.below;
    const double iR = 1.0 / R;
    phidot = pphi * o.imu * iR * iR;
    double2 f = make_double2(1.0, 0.0), c = make_double2(0.0, 0.0);
    if (o.row) {
      f = o.ph()[p * o.Npad + o.n];
      c = make_double2(fma(f.x, a.x, f.y * a.y), fma(f.x, a.y, -(f.y * a.x)));
      if constexpr (FP32) o.c()[o.n] = make_float2((float)c.x, (float)c.y);
      o.c64()[o.n] = c;
    }
    __syncthreads();
    const int64_t ks = sy.knot_stride;
    const uint32_t sbytes = (uint32_t)(ks * NCOMP * (int64_t)sizeof(S));
    const auto rs0 = slice_rsrc((const S*)sy.M + (int64_t)sp.k * ks * NCOMP, sbytes);
    const auto rs1 = slice_rsrc((const S*)sy.M + (int64_t)(sp.k + 1) * ks * NCOMP, sbytes);
    const auto rs2 = slice_rsrc((const S*)sy.M2 + (int64_t)sp.k * ks * NCOMP, sbytes);
    const auto rs3 = slice_rsrc((const S*)sy.M2 + (int64_t)(sp.k + 1) * ks * NCOMP, sbytes);
    const auto rcol = slice_rsrc(sy.ell_col, (uint32_t)((int64_t)sy.ell_w * o.Npad * 4));
    const F w[4] = {(F)uni(sp.w0), (F)uni(sp.w1), (F)uni(sp.w2), (F)uni(sp.w3)};
    const F d[4] = {(F)uni(sp.d0), (F)uni(sp.d1), (F)uni(sp.d2), (F)uni(sp.d3)};
    double2 U[VEC], V[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) U[v] = V[v] = make_double2(0.0, 0.0);
    auto stream = [&](auto sparse) {
      constexpr bool ELL = decltype(sparse)::value;
      // indices first, then the table elements (loads retire in order)
      auto load = [&](Batch& b, int m0) {
        if constexpr (ELL) {
#pragma unroll
          for (int u = 0; u < SB; ++u) {
            if (m0 + u >= o.se) break;
            const uint32_t off = ((uint32_t)(m0 + u) * (uint32_t)o.Npad + (uint32_t)o.grp * VEC) * 4u;
            if constexpr (VEC == 2) {
              const int2 cc = __builtin_bit_cast(
                  int2, __builtin_amdgcn_raw_buffer_load_b64(rcol, off, 0, 0));
              b.ci[u][0] = cc.x;
              b.ci[u][1] = cc.y;
            } else {
              b.ci[u][0] = (int)__builtin_amdgcn_raw_buffer_load_b32(rcol, off, 0, 0);
            }
          }
        }
#pragma unroll
        for (int u = 0; u < SB; ++u) {
          if (m0 + u >= o.se) break;
          const uint32_t off = ((uint32_t)(m0 + u) * (uint32_t)o.ngroups + (uint32_t)o.grp) *
                               (uint32_t)sizeof(L);
          b.tv[u][0] = load16<L>(rs0, off);
          b.tv[u][1] = load16<L>(rs1, off);
          b.tv[u][2] = load16<L>(rs2, off);
          b.tv[u][3] = load16<L>(rs3, off);
        }
      };
      auto use = [&](const Batch& b, int m0) {
        F2 pu[VEC], pv[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) pu[v].x = pu[v].y = pv[v].x = pv[v].y = (F)0;
#pragma unroll
        for (int u = 0; u < SB; ++u) {
          if (m0 + u >= o.se) break;
          F r0[VEC], i0[VEC], r1[VEC], i1[VEC], r2[VEC], i2[VEC], r3[VEC], i3[VEC];
          split(b.tv[u][0], r0, i0); split(b.tv[u][1], r1, i1);
          split(b.tv[u][2], r2, i2); split(b.tv[u][3], r3, i3);
#pragma unroll
          for (int v = 0; v < VEC; ++v)
            rhs::elem<CPLX, F, F2>(pu[v], pv[v], r0[v], i0[v], r1[v], i1[v], r2[v], i2[v], r3[v],
                                   i3[v], w, d, o.c()[ELL ? b.ci[u][v] : m0 + u]);
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          U[v].x += (double)pu[v].x; U[v].y += (double)pu[v].y;
          V[v].x += (double)pv[v].x; V[v].y += (double)pv[v].y;
        }
      };
      Batch A, B;
      load(A, o.sb);
      for (int m0 = o.sb; m0 < o.se; m0 += 2 * SB) {
        load(B, m0 + SB);
        use(A, m0);
        load(A, m0 + 2 * SB);
        use(B, m0 + SB);
      }
    };
    if (sy.ell_w > 0) stream(std::true_type{});
    else stream(std::false_type{});
    if (o.on) {
      double2* pu = o.part() + (int)threadIdx.x * VEC;
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        pu[v] = U[v];
        pu[v + BLOCK * VEC] = V[v];
      }
    }
    __syncthreads();
    double sums[3] = {0.0, 0.0, 0.0}, more[3] = {0.0, 0.0, 0.0};
    double2 k = make_double2(0.0, 0.0);
    if (o.row) {
      // thread t = share * (Npad / VEC) + group wrote its VEC rows at t * VEC, which
      // is share * Npad + row
      const double2* pu = o.part() + o.n;
      double2 u = pu[0], v = pu[BLOCK * VEC];
      for (int q = 1; q < o.shares; ++q) {
        const double2 x = pu[q * o.Npad], z = pu[q * o.Npad + BLOCK * VEC];
        u.x += x.x; u.y += x.y; v.x += z.x; v.y += z.y;
      }
      double2 xc = make_double2(0.0, 0.0);
      if (o.jw <= JXB) {
#pragma unroll
        for (int q = 0; q < JXB; ++q) {
          if (q >= o.jw) break;
          const double2 cm = o.c64()[o.jc[q]];
          xc.x = fma(o.jv[q], cm.x, xc.x);
          xc.y = fma(o.jv[q], cm.y, xc.y);
        }
      } else {
        for (int q = 0; q < o.jw; ++q) {
          const double jv = sy.jx_val[(int64_t)o.n * o.jw + q];
          const double2 cm = o.c64()[sy.jx_col[(int64_t)o.n * o.jw + q]];
          xc.x = fma(jv, cm.x, xc.x);
          xc.y = fma(jv, cm.y, xc.y);
        }
      }
      const double pn = fma(a.x, a.x, a.y * a.y);
      sums[0] = fma(c.x, v.x, c.y * v.y);
      sums[1] = fma(xc.x, u.y, -(xc.y * u.x));
      sums[2] = pn;
      if (full) {
        more[0] = fma(c.x, u.x, c.y * u.y);
        more[1] = o.En * pn;
        more[2] = fma(c.x, xc.x, c.y * xc.y);
      }
      // da/dt = -i e^{iE_n t} (u + Phidot J_x c)
      const double gx = fma(phidot, xc.x, u.x), gy = fma(phidot, xc.y, u.y);
      k = make_double2(fma(f.x, gy, f.y * gx), fma(f.y, gy, -(f.x * gx)));
    }
    reduce(o, sums);
    tot.force = sums[0];
    tot.torque = sums[1];
    tot.norm = sums[2];
    if (full) {
      reduce(o, more);
      tot.vexp = more[0];
      tot.erot = more[1];
      tot.jx = more[2];
    }
    if (at) {
      // decoupled (AT) dynamics: the driving potential in place of the mean field
      const int kk = sp.k;
      tot.force = uni(sp.d0 * sy.drv[kk] + sp.d1 * sy.drv[kk + 1] + sp.d2 * sy.drv2[kk] +
                      sp.d3 * sy.drv2[kk + 1]);
      tot.torque = 0.0;
      if (full) {
        tot.vexp = uni(sp.w0 * sy.drv[kk] + sp.w1 * sy.drv[kk + 1] + sp.w2 * sy.drv2[kk] +
                       sp.w3 * sy.drv2[kk + 1]);
        tot.erot = 0.0;
        tot.jx = 0.0;
      }
    }
    return k;
  }

  // One evaluation at time t with the sums of the diagnostics.
  __device__ static void eval_at(Own& o, const DevSystem& sy, double t, const double (&y)[4],
                                 double2 a, Sums& tot, bool& below, bool at) {
    const double ts[NPH] = {t, t, t, t, t};
    __syncthreads();      // the phases of an earlier step are consumed
    phases(o, ts, 1);
    double om;
    eval(o, sy, 0, y[0], y[3], a, tot, below, om, at, true);
  }

  __device__ static double kinetic(double mu, const double (&y)[4]) {
    return y[2] * y[2] / (2.0 * mu) + y[3] * y[3] / (2.0 * mu * y[0] * y[0]);
  }

  // The classical variables (R, Phi, P_R, P_Phi) run one per lane: lane l carries
  // component l mod 4.
  __device__ static double pick(double v0, double v1, double v2, double v3) {
    const double x = (threadIdx.x & 1) ? v1 : v0, y = (threadIdx.x & 1) ? v3 : v2;
    return (threadIdx.x & 2) ? y : x;
  }
  __device__ static double lane_val(double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
  }
  // This lane's component of the classical derivative at the state whose components
  // R, P_R, P_Phi are given, om = P_Phi / (mu R^2) (Eqs. 7-10).
  __device__ static double classical_rhs(const Own& o, double R, double PR, double PPhi, double om,
                                         const Sums& s) {
    return pick(PR * o.imu, om, fma(PPhi * om, 1.0 / R, -s.force), 2.0 * s.torque);
  }

  // One classical RK4 step at time t (stage times t, t + h/2, t + h), or (nst = 1) only
  // the first stage's evaluation: a and y stay.  full: with the diagnostics' sums of
  // the first stage.  y: this lane's classical component.
  __device__ static void rk4_step(Own& o, const DevSystem& sy, double t, double h, double2& a,
                                  double& y, Sums& tot, bool& below, bool at, int nst, bool full) {
    const double ts[NPH] = {t, t + 0.5 * h, t + h, t, t};
    phases(o, ts, nst == 1 ? 1 : 3);
    double2 k = make_double2(0.0, 0.0), acc = k;
    double ky = 0.0, ay = 0.0;
    for (int st = 0; st < nst; ++st) {
      const double cf = st == 0 ? 0.0 : (st == 3 ? h : 0.5 * h);
      const double wgt = (st == 0 || st == 3) ? 1.0 : 2.0;
      const double ys = fma(cf, ky, y);
      const double R = lane_val(ys, 0), PR = lane_val(ys, 2), PPhi = lane_val(ys, 3);
      double om;
      const double2 in = make_double2(fma(cf, k.x, a.x), fma(cf, k.y, a.y));
      k = eval(o, sy, (st + 1) >> 1, R, PPhi, in, tot, below, om, at, full && st == 0);
      ky = classical_rhs(o, R, PR, PPhi, om, tot);
      acc.x = fma(wgt, k.x, acc.x);
      acc.y = fma(wgt, k.y, acc.y);
      ay = fma(wgt, ky, ay);
    }
    if (nst == 1) return;
    const double h6 = h / 6.0;
    a.x = fma(h6, acc.x, a.x);
    a.y = fma(h6, acc.y, a.y);
    y = fma(h6, ay, y);
  }

  __device__ static bool bad(const Sums& tot, double y) {
    return !isfinite(tot.force) || !isfinite(tot.torque) || !isfinite(tot.norm) ||
           !isfinite(lane_val(y, 0)) || !isfinite(lane_val(y, 2)) || !isfinite(lane_val(y, 3));
  }

  __device__ static void write_out(const Own& o, const TrajIn& tj, const TrajOut& out, double2 a,
                                   const double (&y)[4], double theta, double ptheta, double tend,
                                   int64_t steps, int64_t rejects, int32_t status,
                                   const Sums& tot, double E0, double J0) {
    if (!out.P) return;   // timing runs of the autotuner write no results
    if (o.row) {
      out.P[tj.amp_off + o.n] = a.x * a.x + a.y * a.y;
      if (out.a_final) ((double2*)out.a_final)[tj.amp_off + o.n] = a;
      if (out.st_amp) out.st_amp[tj.amp_off + o.n] = a;
    }
    if (threadIdx.x == 0) {
      const int64_t id = tj.id;
      if (out.classical) {
        double* q = out.classical + id * 6;
        q[0] = y[0]; q[1] = theta; q[2] = y[1]; q[3] = y[2]; q[4] = ptheta; q[5] = y[3];
      }
      if (out.t_final) out.t_final[id] = tend;
      if (out.steps) out.steps[id] = steps;
      if (out.rejects) out.rejects[id] = rejects;
      if (out.status) out.status[id] = status;
      if (out.norm_err) out.norm_err[id] = tot.norm - 1.0;
      if (out.energy_err) out.energy_err[id] = (kinetic(o.mu, y) + tot.erot + tot.vexp - E0) / fabs(E0);
      if (out.angmom_err) out.angmom_err[id] = (y[3] - tot.jx) - J0;
    }
  }

  // Fixed-step RK4 of one trajectory, the whole step loop (as Kern::run_rk4).
  __device__ static void run_rk4(Own& o, const DevSystem& sy, const TrajIn& tj,
                                 const double* __restrict__ a0_all, const TrajOut& out) {
    double2 a = make_double2(0.0, 0.0);
    if (o.row) {
      if (tj.flags & TRAJ_HAS_A0) a = ((const double2*)a0_all)[tj.amp_off + o.n];
      else if (o.n == tj.init_channel) a = make_double2(1.0, 0.0);
    }
    double y[4], theta = 0.5 * M_PI, ptheta = 0.0;
    if (tj.flags & TRAJ_HAS_C0) {
      y[0] = tj.c0[0]; theta = tj.c0[1]; y[1] = tj.c0[2]; y[2] = tj.c0[3]; ptheta = tj.c0[4];
      y[3] = tj.c0[5];
    } else {
      const double k = sqrt(2.0 * sy.mu * tj.E_coll);
      const double pphi = tj.b * k;
      y[0] = tj.R0; y[1] = 0.0;
      y[2] = -sqrt(2.0 * sy.mu * tj.E_coll - pphi * pphi / (tj.R0 * tj.R0));
      y[3] = pphi;
    }
    const double R_exit = start_exit_radius(tj, y[0]);
    const double ekin0 = uni(kinetic(o.mu, y)), pphi0 = uni(y[3]);
    double yl = pick(y[0], y[1], y[2], y[3]);
    const double h = tj.dt, t0 = tj.t0;
    const bool resume = (tj.flags & TRAJ_RESUME) != 0, at = (tj.flags & TRAJ_AT) != 0;
    const int64_t j0 = tj.step0;
    bool below = false, b2 = false;
    int32_t status = tj.status0;
    double E0 = tj.E0, J0 = tj.J0;
    Sums tot{};
    // the steps, then the evaluation of the end state; the diagnostics take their
    // references from the very first evaluation
    int64_t j = 0;
    bool last = false, fin = tj.n_steps <= 0;
    while (!last) {
      last = fin;
      rk4_step(o, sy, t0 + (double)(j0 + j) * h, h, a, yl, tot, last ? b2 : below, at, last ? 1 : 4,
               last || (j == 0 && !resume));
      if (j == 0 && !resume) {
        E0 = ekin0 + tot.erot + tot.vexp;
        J0 = pphi0 - tot.jx;
      }
      if (last) break;
      ++j;
      if (bad(tot, yl)) {
        status |= ST_NONFINITE;
        fin = true;
      }
      fin = fin || j >= tj.n_steps;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = lane_val(yl, i);
    const double tend = t0 + (double)(j0 + j) * h;
    if (below) status |= ST_BELOW_GRID;
    const int64_t steps = tj.steps0 + j;
    write_out(o, tj, out, a, y, theta, ptheta, tend, steps, tj.rejects0, status, tot, E0, J0);
    if (threadIdx.x == 0)
      put_traj_state(out, tj, sy.N, tend, t0, j0 + j, h, y, theta, ptheta, E0, J0, R_exit, steps,
                     tj.rejects0, tj.attempts0 + j, status, tj.dflags);
  }
};

#pragma clang fp contract(fast)

}  // namespace shared
}  // namespace mqct
