// Coupling-matrix builder for an asymmetric-top rotor + linear rotor (paper
// Section II, Eqs. 12-18).
//
// The potential is expanded over the angular functions tau_t of Eq. 13 with
// radial coefficients v_t(R) (Eq. 12), so the matrix of Eq. 6 between coupled
// states |n m> = |j1 tau1 j2 j m> (Eq. 3) is M(R) = sum_t v_t(R) G_t with
//
//   G_t(n'', n') = F_t(j1' j2' j', j1'' j2'' j'') * K_t(r'', r') * C(j' m lam 0 | j'' m)
//
// for m'' = m' (zero otherwise).  K_t is the rotor-1 factor of Eq. 17 (the sum
// over k1'', k1' of b b [C(j1' k1' lam1 mu1 | j1'' k1'') + s C(j1' k1' lam1 -mu1 |
// j1'' k1'')], s = (-1)^(lam1+mu1+lam2+lam)).  The sums over m1', m1'' and eta of
// Eq. 17, five Clebsch-Gordan coefficients, recouple into one 9j symbol times a
// coefficient in m (Wigner-Eckart theorem for the rank-lam tensor tau_t):
//
//   F_t = sqrt((2j1'+1)(2j2'+1)(2j'+1)(2lam+1)) sqrt((2lam1+1)(2lam2+1)) / (4 pi)
//         * C(j2' 0 lam2 0 | j2'' 0) * {j1' j2' j'; lam1 lam2 lam; j1'' j2'' j''}
//
// which is what makes the build cheap: F depends on the angular momenta only
// (not on m or tau1), K on the rotor-1 states only.  Kernels:
//   cpl_lfact  log-factorials (the Racah sums below run in the log domain);
//   cpl_zero   the outputs cleared with 16-byte stores (most elements couple
//              channels of different m and stay zero), while the host lays out the
//              build;
//   cpl_rotor  K_t for every pair of rotor-1 states;
//   cpl_jlevel F_t for every pair of (j1, j2, j) levels (9j from three 6j);
//   cpl_cgm    the coefficients C(j' m lam 0 | j'' m) for every j', j'', m and lam
//              that occur;
//   cpl_fill   one work item per row n'' and 256 of the channels n' that share its
//              m: M[k][n''][n'] = sum_t v_t(R_k) g_t as a product (knots x terms) x
//              (terms x channels) on the FP64 matrix cores, each lane forming g_t =
//              F K C of its channel for four consecutive terms at a time.  With
//              channels ordered by m the lanes of a work item write consecutive
//              columns.
#include "internal.h"

#include <math.h>

#include <algorithm>

namespace mqct {

namespace {

constexpr int LF_N = 256;        // log-factorial table: arguments up to 255
constexpr int FILL_BLOCK = 256;
constexpr int VAL_KC = CPL_KNOT_CHUNK;    // knots per accumulation chunk (registers)
constexpr int JL_ITEMS = 2048;   // level factors per workgroup
constexpr int NXCD = 8;          // accelerator dies of the device, each with its own L2
constexpr int GATHER_TC = 8;     // terms whose factors are gathered together

__device__ inline bool tri(int a, int b, int c) { return c >= abs(a - b) && c <= a + b; }

// <j1 m1 j2 m2 | J M> by Racah's sum, each term formed in the log domain
__device__ double cg_dev(const double* __restrict__ lf, int j1, int m1, int j2, int m2, int J,
                         int M) {
  if (m1 + m2 != M || !tri(j1, j2, J) || abs(m1) > j1 || abs(m2) > j2 || abs(M) > J) return 0.0;
  const double lpre = 0.5 * (log((double)(2 * J + 1)) + lf[J + j1 - j2] + lf[J - j1 + j2] +
                             lf[j1 + j2 - J] - lf[j1 + j2 + J + 1] + lf[J + M] + lf[J - M] +
                             lf[j1 - m1] + lf[j1 + m1] + lf[j2 - m2] + lf[j2 + m2]);
  const int kmin = max(0, max(j2 - J - m1, j1 - J + m2));
  const int kmax = min(j1 + j2 - J, min(j1 - m1, j2 + m2));
  double s = 0.0;
  for (int k = kmin; k <= kmax; ++k) {
    const double t = exp(lpre - (lf[k] + lf[j1 + j2 - J - k] + lf[j1 - m1 - k] + lf[j2 + m2 - k] +
                                 lf[J - j2 + m1 + k] + lf[J - j1 - m2 + k]));
    s += (k & 1) ? -t : t;
  }
  return s;
}

__device__ inline double ldelta(const double* lf, int a, int b, int c) {
  return lf[a + b - c] + lf[a - b + c] + lf[b + c - a] - lf[a + b + c + 1];
}

// {a b c; d e f} by Racah's sum
__device__ double sixj_dev(const double* __restrict__ lf, int a, int b, int c, int d, int e,
                           int f) {
  if (!tri(a, b, c) || !tri(a, e, f) || !tri(d, b, f) || !tri(d, e, c)) return 0.0;
  const int a1 = a + b + c, a2 = a + e + f, a3 = d + b + f, a4 = d + e + c;
  const int b1 = a + b + d + e, b2 = b + c + e + f, b3 = c + a + f + d;
  const double ld = 0.5 * (ldelta(lf, a, b, c) + ldelta(lf, a, e, f) + ldelta(lf, d, b, f) +
                           ldelta(lf, d, e, c));
  const int tmin = max(max(a1, a2), max(a3, a4)), tmax = min(b1, min(b2, b3));
  double s = 0.0;
  for (int t = tmin; t <= tmax; ++t) {
    const double x = exp(ld + lf[t + 1] - lf[t - a1] - lf[t - a2] - lf[t - a3] - lf[t - a4] -
                         lf[b1 - t] - lf[b2 - t] - lf[b3 - t]);
    s += (t & 1) ? -x : x;
  }
  return s;
}

// {a b c; d e f; g h i} as a sum over x of (2x+1) {a b c; f i x}{d e f; b x h}{g h i; x a d}
__device__ double ninej_dev(const double* __restrict__ lf, int a, int b, int c, int d, int e,
                            int f, int g, int h, int i) {
  const int xmin = max(abs(a - i), max(abs(b - f), abs(d - h)));
  const int xmax = min(a + i, min(b + f, d + h));
  double s = 0.0;
  for (int x = xmin; x <= xmax; ++x)
    s += (2 * x + 1) * sixj_dev(lf, a, b, c, f, i, x) * sixj_dev(lf, d, e, f, b, x, h) *
         sixj_dev(lf, g, h, i, x, a, d);
  return s;
}

__global__ void cpl_lfact(double* __restrict__ lf) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < LF_N) lf[i] = lgamma((double)i + 1.0);
}

// K[rb][ra][t]: the rotor-1 factor between rotor-1 states ra (initial) and rb (final)
__global__ void cpl_rotor(CouplingDev d) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nn = (int64_t)d.n1 * d.n1;
  if (i >= (int64_t)d.T * nn) return;
  const int t = (int)(i % d.T);
  const int64_t pr = i / d.T;
  const int rb = (int)(pr / d.n1), ra = (int)(pr - (int64_t)rb * d.n1);
  const int l1 = d.t_l1[t], mu = d.t_mu[t], l2 = d.t_l2[t], l = d.t_l[t];
  const double s = ((l1 + mu + l2 + l) & 1) ? -1.0 : 1.0;
  const int ja = d.rot_j[ra], jb = d.rot_j[rb];
  const double* ba = d.b + (int64_t)ra * d.b_stride;
  const double* bb = d.b + (int64_t)rb * d.b_stride;
  double acc = 0.0;
  for (int ka = -ja; ka <= ja; ++ka) {
    const double x = ba[ka + ja];
    if (x == 0.0) continue;
    int kb = ka + mu;
    if (abs(kb) <= jb) acc += bb[kb + jb] * x * cg_dev(d.lf, ja, ka, l1, mu, jb, kb);
    kb = ka - mu;
    if (abs(kb) <= jb) acc += s * bb[kb + jb] * x * cg_dev(d.lf, ja, ka, l1, -mu, jb, kb);
  }
  d.Kr[pr * d.TP + t] = acc;
}

// F[Jb][Ja][t] between (j1, j2, j) levels Ja (initial) and Jb (final).  Triangle rules
// and C(j2' 0 lam2 0 | j2'' 0) leave few of a workgroup's JL_ITEMS factors nonzero: those
// are listed first, so that the 9j sums run in full waves.
__global__ void __launch_bounds__(256) cpl_jlevel(CouplingDev d) {
  __shared__ int list[JL_ITEMS];
  __shared__ int count;
  if (threadIdx.x == 0) count = 0;
  __syncthreads();
  const int64_t nn = (int64_t)d.nJ * d.nJ, total = (int64_t)d.T * nn;
  const int64_t i0 = (int64_t)blockIdx.x * JL_ITEMS;
  for (int q = threadIdx.x; q < JL_ITEMS; q += 256) {
    const int64_t i = i0 + q;
    if (i >= total) break;
    const int t = (int)(i % d.T);
    const int64_t pr = i / d.T;
    const int Jb = (int)(pr / d.nJ), Ja = (int)(pr - (int64_t)Jb * d.nJ);
    const int j2a = d.jl_j2[Ja], j2b = d.jl_j2[Jb], l2 = d.t_l2[t];
    if (tri(d.jl_j1[Ja], d.t_l1[t], d.jl_j1[Jb]) && tri(d.jl_j[Ja], d.t_l[t], d.jl_j[Jb]) &&
        cg_dev(d.lf, j2a, 0, l2, 0, j2b, 0) != 0.0)
      list[atomicAdd(&count, 1)] = q;
    else
      d.F[pr * d.TP + t] = 0.0;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < count; q += 256) {
    const int64_t i = i0 + list[q];
    const int t = (int)(i % d.T);
    const int64_t pr = i / d.T;
    const int Jb = (int)(pr / d.nJ), Ja = (int)(pr - (int64_t)Jb * d.nJ);
    const int l1 = d.t_l1[t], l2 = d.t_l2[t], l = d.t_l[t];
    const int j1a = d.jl_j1[Ja], j2a = d.jl_j2[Ja], ja = d.jl_j[Ja];
    const int j1b = d.jl_j1[Jb], j2b = d.jl_j2[Jb], jb = d.jl_j[Jb];
    const double c2 = cg_dev(d.lf, j2a, 0, l2, 0, j2b, 0);
    const double nj = ninej_dev(d.lf, j1a, j2a, ja, l1, l2, l, j1b, j2b, jb);
    d.F[pr * d.TP + t] =
        sqrt((double)(2 * j1a + 1) * (2 * j2a + 1) * (2 * ja + 1) * (2 * l + 1)) *
        sqrt((double)(2 * l1 + 1) * (2 * l2 + 1)) * (0.25 / M_PI) * c2 * nj;
  }
}

// zero n doubles (9.3 GB: 1.31 ms, 7.1 TB/s; in one launch with the factors, which hold
// four times the registers, the two took 1.73 ms instead of 1.60), one 16-byte store per thread from the first 16-byte boundary
// (single elements before it and after the last pair)
__global__ void __launch_bounds__(256) cpl_zero(double* __restrict__ p, int64_t n) {
  typedef double dv2 __attribute__((ext_vector_type(2)));
  const int64_t head = ((uintptr_t)p & 15) ? 1 : 0;
  const int64_t pairs = (n - head) >> 1;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < pairs) ((dv2*)(p + head))[i] = dv2{0.0, 0.0};
  if (i == 0) {
    if (head) p[0] = 0.0;
    if ((n - head) & 1) p[n - 1] = 0.0;
  }
}

// C(ja m lam 0 | jb m) for ja, jb <= JM, |m| <= JM, lam <= LM: cgt[((ja * (JM+1) +
// jb) * (2 JM + 1) + m + JM) * (LM + 1) + lam]
__global__ void cpl_cgm(CouplingDev d) {
  const int JM = d.cg_jmax, LM = d.cg_lmax;
  const int64_t total = (int64_t)(JM + 1) * (JM + 1) * (2 * JM + 1) * (LM + 1);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int lam = (int)(i % (LM + 1));
  int64_t r = i / (LM + 1);
  const int m = (int)(r % (2 * JM + 1)) - JM;
  r /= (2 * JM + 1);
  const int jb = (int)(r % (JM + 1)), ja = (int)(r / (JM + 1));
  d.cgt[i] = cg_dev(d.lf, ja, m, lam, 0, jb, m);
}

// Per element (nb, na) of equal m: pointers to its level factors F[Jb][Ja][.],
// rotor-1 factors K[rb][ra][.] and m-coefficients C(ja m . 0 | jb m); g_t is
// F[t] K[t] C[lam_t] for every kernel that forms it.
struct GPtr {
  const double* F;
  const double* Kr;
  const double* C;
};
__device__ __forceinline__ GPtr gptr(const CouplingDev& d, int nb, int na) {
  const int TP = d.TP, JM = d.cg_jmax, mb = d.chan_m[nb];
  const int Jb = d.chan_J[nb], rb = d.chan_r[nb], jb = d.chan_j[nb];
  const int Ja = d.chan_J[na], ra = d.chan_r[na], ja = d.chan_j[na];
  GPtr p;
  p.F = d.F + ((int64_t)Jb * d.nJ + Ja) * TP;
  p.Kr = d.Kr + ((int64_t)rb * d.n1 + ra) * TP;
  p.C = d.cgt + (((int64_t)ja * (JM + 1) + jb) * (2 * JM + 1) + mb + JM) * (d.cg_lmax + 1);
  return p;
}
// g_t for the GATHER_TC terms from t0 (indices past the last term repeat it)
__device__ __forceinline__ void gather_g(const CouplingDev& d, const GPtr& p, int t0,
                                         double (&gv)[GATHER_TC]) {
#pragma unroll
  for (int i = 0; i < GATHER_TC; ++i) {
    const int t = min(t0 + i, d.T - 1);
    gv[i] = p.F[t] * p.Kr[t] * p.C[d.t_l[t]];
  }
}

// Workgroup ids go to the dies round-robin: each die gets one contiguous share of the
// work list (ordered by the rows' levels), so that its L2 holds the level-factor rows
// those items read.  False for the ids beyond the list.
__device__ __forceinline__ bool work_item(const CouplingDev& d, int2& w) {
  const int64_t per = (d.n_work + NXCD - 1) / NXCD;
  const int64_t wi = (int64_t)(blockIdx.x % NXCD) * per + blockIdx.x / NXCD;
  if (blockIdx.x / NXCD >= per || wi >= d.n_work) return false;
  w = d.work[wi];
  return true;
}

// One work item = (row nb, FILL_BLOCK consecutive entries of the list of channels
// that share nb's m).  M[k][nb][na] (and G[t][nb][na] when asked) for those na, as
// v_mfma_f64_16x16x4 products: lane l holds the column of channel l % 16 of a tile and
// the terms t0 + 4 (l / 16) + i, i = 0..3, of a step of 16 (a permutation of the sum over
// t), so 64 lanes touch 16 rows of F and of K with 32 consecutive bytes each; v of up to
// FILL_TC terms and 64 knots is in LDS, rows padded so that the four term groups of a
// read fall into different banks, and the row's m-coefficients beside it.  The next
// step's factors are requested before this step's products.
// N = 4,290, 83 terms, 63 knots (9.3 GB, of it 0.74 GB written here): one channel per
// lane, terms one by one and the knots in two passes, 1.29 ms (its loads touch 64 rows
// each); this form 0.69 ms.  What is left is neither its products (0.56 without) nor its
// stores (0.60 without) but the latency of the gathers at three waves per SIMD; two tiles
// a wave (230 registers) take 0.74 ms, a persistent grid 0.68.
// Beyond FILL_TC terms v is staged again for each 16 channels of a wave, beyond FILL_KC
// knots the factors are read again, and both stay ahead of the per-lane form (whole builds,
// N = 2,475: 97 terms 1.51 -> 1.20 ms, 240 terms 2.43 -> 1.56, 83 terms and 200 knots 3.80
// -> 2.66, 192 and 200 6.14 -> 3.86).
typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));
constexpr int FILL_TC = 96, FILL_KC = 64, FILL_LD = FILL_KC + 4;

__global__ void __launch_bounds__(FILL_BLOCK)
cpl_fill(CouplingDev d, double* __restrict__ M, double* __restrict__ G) {
  extern __shared__ __align__(16) double vl[];      // [FILL_TC][FILL_LD] v
  double* cl = vl + FILL_TC * FILL_LD;              // [cg_jmax + 1][cg_lmax + 1] C(ja m lam 0 | jb m)
  __shared__ int tl[FILL_TC];
  int2 w;
  if (!work_item(d, w)) return;
  const int nb = w.x, g = d.chan_grp[nb];
  const int g0 = d.grp_off[g], cnt = d.grp_off[g + 1] - g0;
  const int N = d.N, T = d.T, K = d.K, KP = d.KP, L1 = d.cg_lmax + 1;
  const int64_t NN = (int64_t)N * N;
  const int wave = threadIdx.x >> 6, col = threadIdx.x & 15, grp = (threadIdx.x & 63) >> 4;
  {
    const int JM = d.cg_jmax, jb = d.chan_j[nb], mb = d.chan_m[nb];
    for (int i = threadIdx.x; i < (JM + 1) * L1; i += FILL_BLOCK)
      cl[i] = d.cgt[(((int64_t)(i / L1) * (JM + 1) + jb) * (2 * JM + 1) + mb + JM) * L1 + i % L1];
  }
  const int kend = M ? K : 1;          // G alone: one pass over the terms
  for (int k0 = 0; k0 < kend; k0 += FILL_KC) {
    const int ntile = min(FILL_KC, K - k0 + 15) >> 4;
    for (int h = 0; h < 4; ++h) {      // a wave's 64 channels, 16 at a time
      const int q = w.y * FILL_BLOCK + wave * 64 + h * 16 + col;
      const bool work = q - col < cnt;
      const int na = d.grp_list[g0 + min(q, cnt - 1)];
      const GPtr gp = gptr(d, nb, na);
      const double* cj = cl + d.chan_j[na] * L1;
      const int64_t pos = (int64_t)nb * N + na;
      v4d acc[4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) acc[mt] = v4d{0.0, 0.0, 0.0, 0.0};
      for (int c0 = 0; c0 < T; c0 += FILL_TC) {
        const int nt = min(FILL_TC, T - c0);
        if (h == 0 || T > FILL_TC) {
          __syncthreads();
          if (M)
            for (int i = threadIdx.x; i < FILL_TC * FILL_KC; i += FILL_BLOCK) {
              const int t = i / FILL_KC, k = i % FILL_KC;
              vl[t * FILL_LD + k] = t < nt && k0 + k < K ? d.v[(int64_t)(c0 + t) * KP + k0 + k] : 0.0;
            }
          if (threadIdx.x < FILL_TC) tl[threadIdx.x] = d.t_l[min(c0 + (int)threadIdx.x, T - 1)];
          __syncthreads();
        }
        if (!work) continue;
        const double *F = gp.F + c0, *Kr = gp.Kr + c0;
        v2d f[2], kr[2];
        auto load = [&](int t0) {
          const int tq = t0 + 4 * grp;
          if (t0 + 16 <= nt) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              f[i] = *(const v2d*)(F + tq + 2 * i);
              kr[i] = *(const v2d*)(Kr + tq + 2 * i);
            }
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              f[i >> 1][i & 1] = F[min(tq + i, nt - 1)];
              kr[i >> 1][i & 1] = Kr[min(tq + i, nt - 1)];
            }
          }
        };
        load(0);
        for (int t0 = 0; t0 < nt; t0 += 16) {
          const int tq = t0 + 4 * grp;
          double gv[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) gv[i] = f[i >> 1][i & 1] * kr[i >> 1][i & 1] * cj[tl[tq + i]];
          if (t0 + 16 < nt) load(t0 + 16);
          if (G && k0 == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (tq + i < nt && q < cnt) G[(int64_t)d.t_user[c0 + tq + i] * NN + pos] = gv[i];
          }
          if (!M) continue;
          const double* vr = vl + tq * FILL_LD + col;
#pragma unroll
          for (int mt = 0; mt < 4; ++mt) {
            if (mt >= ntile) break;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              acc[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(vr[i * FILL_LD + mt * 16], gv[i],
                                                             acc[mt], 0, 0, 0);
          }
        }
      }
      if (!M || q >= cnt) continue;
      double* out = M + (int64_t)(k0 + grp) * NN + pos;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = mt * 16 + 4 * r;
          if (k0 + grp + k < K) out[k * NN] = acc[mt][r];
        }
    }
  }
}

// Screening: an element of equal m is kept when max_s |M(R_s)| > thr over the
// screening radii, M(R_s) = sum_t vs[t][s] g_t.  Kept elements take slots of
// (rows, cols) in the order the per-wave atomics give (one atomic per wave);
// slots past the capacity are counted but not written.
__global__ void __launch_bounds__(FILL_BLOCK)
cpl_screen(CouplingDev d, int S, const double* __restrict__ vs,
           double thr, int64_t capacity, unsigned long long* __restrict__ count,
           int32_t* __restrict__ rows, int32_t* __restrict__ cols) {
  int2 w;
  if (!work_item(d, w)) return;
  const int nb = w.x;
  const int g = d.chan_grp[nb];
  const int g0 = d.grp_off[g], cnt = d.grp_off[g + 1] - g0;
  const int q = w.y * FILL_BLOCK + threadIdx.x;
  const bool act = q < cnt;
  const int na = act ? d.grp_list[g0 + q] : nb;
  bool keep = false;
  if (act) {
    // the element is symmetric, so the decision is taken from one ordering of the
    // pair: (n, m) and (m, n) are kept or dropped together
    const GPtr gp = gptr(d, min(nb, na), max(nb, na));
    double acc[CPL_MAX_SCREEN];
#pragma unroll
    for (int u = 0; u < CPL_MAX_SCREEN; ++u) acc[u] = 0.0;
    for (int t0 = 0; t0 < d.T; t0 += GATHER_TC) {
      double gv[GATHER_TC];
      gather_g(d, gp, t0, gv);
#pragma unroll
      for (int i = 0; i < GATHER_TC; ++i) {
        if (t0 + i >= d.T) break;
        const double* vt = vs + (int64_t)(t0 + i) * S;
#pragma unroll
        for (int u = 0; u < CPL_MAX_SCREEN; ++u)
          if (u < S) acc[u] = fma(vt[u], gv[i], acc[u]);
      }
    }
    double mx = 0.0;
#pragma unroll
    for (int u = 0; u < CPL_MAX_SCREEN; ++u)
      if (u < S) mx = fmax(mx, fabs(acc[u]));
    keep = mx > thr;
  }
  const unsigned long long bal = __ballot(keep);
  const int lane = threadIdx.x & 63;
  unsigned long long base = 0;
  if (lane == 0 && bal) base = atomicAdd(count, (unsigned long long)__popcll(bal));
  const int lo = __shfl((int)(base & 0xffffffffull), 0, 64);
  const int hi = __shfl((int)(base >> 32), 0, 64);
  base = ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
  if (keep) {
    const int64_t idx = (int64_t)(base + __popcll(bal & ((1ull << lane) - 1ull)));
    if (idx < capacity) {
      rows[idx] = nb;
      cols[idx] = na;
    }
  }
}

// Values of the kept elements at every knot: values[k * capacity + i] for the
// element (rows[i], cols[i]), one thread per element.
__global__ void __launch_bounds__(256)
cpl_values(CouplingDev d, int64_t n, const int32_t* __restrict__ rows,
           const int32_t* __restrict__ cols, int64_t capacity, double* __restrict__ values) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const GPtr gp = gptr(d, rows[i], cols[i]);
  const int T = d.T, K = d.K, KP = d.KP;
  const double* __restrict__ v = d.v;
  for (int k0 = 0; k0 < K; k0 += VAL_KC) {
    double acc[VAL_KC];
#pragma unroll
    for (int u = 0; u < VAL_KC; ++u) acc[u] = 0.0;
    for (int t0 = 0; t0 < T; t0 += GATHER_TC) {
      double gv[GATHER_TC];
      gather_g(d, gp, t0, gv);
#pragma unroll
      for (int j = 0; j < GATHER_TC; ++j) {
        if (t0 + j >= T) break;
        const double* vt = v + (int64_t)(t0 + j) * KP + k0;
#pragma unroll
        for (int u = 0; u < VAL_KC; ++u) acc[u] = fma(vt[u], gv[j], acc[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < VAL_KC; ++u)
      if (k0 + u < K) values[(int64_t)(k0 + u) * capacity + i] = acc[u];
  }
}

}  // namespace

namespace {

hipError_t launch_factors(const CouplingDev& d, hipStream_t s) {
  cpl_lfact<<<1, LF_N, 0, s>>>(d.lf);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t ncg = (int64_t)(d.cg_jmax + 1) * (d.cg_jmax + 1) * (2 * d.cg_jmax + 1) *
                      (d.cg_lmax + 1);
  cpl_cgm<<<(unsigned)((ncg + 255) / 256), 256, 0, s>>>(d);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t nr = (int64_t)d.T * d.n1 * d.n1;
  cpl_rotor<<<(unsigned)((nr + 255) / 256), 256, 0, s>>>(d);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t nj = (int64_t)d.T * d.nJ * d.nJ;
  cpl_jlevel<<<(unsigned)((nj + JL_ITEMS - 1) / JL_ITEMS), 256, 0, s>>>(d);
  return hipGetLastError();
}

}  // namespace

bool coupling_launchable(int64_t N, int64_t T, int64_t K, int64_t n1, int64_t nJ, bool M, bool G) {
  // as doubles: the products may pass 2^63
  const double lim = 256.0 * 0x7fffffff, NN = (double)N * N;
  return (!M || NN * K / 2 <= lim) && (!G || NN * T / 2 <= lim) && (double)T * n1 * n1 <= lim &&
         (double)T * nJ * nJ <= lim;
}

hipError_t launch_coupling_zero(double* p, int64_t n, hipStream_t s) {
  const int64_t blocks = ((n + 1) / 2 + 255) / 256;
  cpl_zero<<<(unsigned)blocks, 256, 0, s>>>(p, n);
  return hipGetLastError();
}

hipError_t launch_coupling(const CouplingDev& d, double* M, double* G, Prof* prof,
                           hipStream_t s) {
  const size_t lds = (FILL_TC * FILL_LD + (size_t)(d.cg_jmax + 1) * (d.cg_lmax + 1)) * 8;
  hipError_t e = hipSuccess;
  if (lds + FILL_TC * 4 > 65536)      // (the terms' lam beside it)
    e = hipFuncSetAttribute((const void*)cpl_fill, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
  if (e != hipSuccess || (e = launch_factors(d, s)) != hipSuccess) return e;
  const int64_t blocks = (d.n_work + NXCD - 1) / NXCD * NXCD;
  if (prof) prof->join();      // one timed launch with the clearing of the outputs
  hipEvent_t e0 = prof ? prof->next() : nullptr, e1 = prof ? prof->next() : nullptr;
  prof_mark(prof, e0, s);
  cpl_fill<<<(unsigned)blocks, FILL_BLOCK, lds, s>>>(d, M, G);
  prof_mark(prof, e1, s);
  return hipGetLastError();
}

hipError_t launch_coupling_screen(const CouplingDev& d, int S, const double* vs, double thr,
                                  int64_t capacity, unsigned long long* count, int32_t* rows,
                                  int32_t* cols, hipStream_t s) {
  if (S < 1 || S > CPL_MAX_SCREEN) return hipErrorInvalidValue;
  hipError_t e = launch_factors(d, s);
  if (e != hipSuccess) return e;
  const int64_t blocks = (d.n_work + NXCD - 1) / NXCD * NXCD;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  cpl_screen<<<(unsigned)blocks, FILL_BLOCK, 0, s>>>(d, S, vs, thr, capacity, count, rows, cols);
  return hipGetLastError();
}

hipError_t launch_coupling_values(const CouplingDev& d, int64_t n, const int32_t* rows,
                                  const int32_t* cols, int64_t capacity, double* values,
                                  hipStream_t s) {
  const int64_t blocks = (n + 255) / 256;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  cpl_values<<<(unsigned)blocks, 256, 0, s>>>(d, n, rows, cols, capacity, values);
  return hipGetLastError();
}

}  // namespace mqct
