// The FP64 local-energy contraction in the trial's virtual space (arXiv:1711.02242, Sec.
// III.D.3, eq:localenergy3; force-bias traces of eq:precomputing2): the FP64 mode, and the FP64
// pass of the mixed modes' precision guard.
//
// Theta_s = U (V^T U)^-1 satisfies V_s^T Theta_s = 1, so with V0 = V (V^T V)^-1 and the
// orthonormal complement Q of V's columns (M x nv, nv = M - N)
//   Theta = V0 + Q X,   X = Q^T Theta   (nv x N),
// and only the d = N nv amplitudes x_e = X_ac, e = c nv + a, depend on the walker.  With the
// half-rotated Cholesky vectors Lh^g = V^T L^g, Om0^g = Lh^g V0 and B^g = Lh^g Q (N x nv):
//   t_g             = tr Om0^g + sum_e B^g_e x_e,
//   sum_g tr(Om Om) = c0 + 2 sum_e f_e x_e + x^T K x,
//     c0 = sum_g tr(Om0^g Om0^g),  f_{(c,a)} = sum_g (Om0^g B^g)_{ca},
//     K_{(c,a),(c',a')} = sum_g B^g_{c'a} B^g_{ca'}   (d x d, symmetric, built once).
// Per walker-spin that is 2 d^2 + 4 G d real operations (Re and Im planes, the symmetric half
// of K) instead of the 4 G N^2 M of Omega^g = Lh^g Theta for every g; with G = 6 M and N = M / 4
// ten times fewer.
//
// Both are one GEMM over columns = walkers x {Re, Im}: the rows of B (traces) and, per block
// row I of K, Z_I = sum_{J <= I} K_IJ X_J followed by x_I . (Z_I + f_I) (the diagonal blocks
// stored halved, the whole counted twice).  k_pair walks units of 128 rows x 128 k x 64
// walkers.  Every workgroup first takes whole trace tiles, then a contiguous run of K units
// sized so that all workgroups do the same number of units; a run may start and end inside a
// block row, since the quadratic form is a sum over units, and leaves one partial sum per
// column tile.
#pragma once

#include <algorithm>

#include "common.hpp"
#include "kernels_mfma.hpp"

constexpr int PAIR_B = 128;        // rows and k of a unit
constexpr int PAIR_W = 64;         // walkers of a column tile
constexpr int PAIR_KC = 16;        // k of one LDS chunk
constexpr size_t PAIR_MAX_BYTES = size_t(16) << 30;   // of the K tables

// Sizes of the tables of one system (host and device).
struct PairDims {
  int n_det, G, Gt;                // Gt = ceil(G / 128) trace row tiles
  int Mp;                          // M rounded up to 16
  int N[2], nv[2], d[2], dp[2];    // amplitudes, padded to a multiple of 128
  int T[2], P[2];                  // block rows dp / 128, units T (T + 1) / 2
};

struct PairTables {
  bool on = false;
  PairDims dim{};
  double* Qt = nullptr;   // [n_det][nv_up + nv_dn][Mp]: the complements, rows a (zero past M)
  double* f = nullptr;    // [n_det][dp_up + dp_dn], zero past d_s
  double* t0 = nullptr;   // [n_det][2][G]: tr Om0^g
  double* c0 = nullptr;   // [n_det][2]
  double* B = nullptr;    // [n_det][s][G][dp_s], then 128 rows of slack (trace tiles past G)
  double* K = nullptr;    // [n_det][s][P_s][128][128]; the start of the one allocation
  size_t bytes = 0;       // of all of them
};

inline size_t pair_b_elems(const PairDims& p) {
  return (size_t)p.n_det * p.G * (p.dp[0] + p.dp[1]) +
         (size_t)PAIR_B * std::max(p.dp[0], p.dp[1]);
}
inline size_t pair_k_elems(const PairDims& p) {
  return (size_t)p.n_det * (p.P[0] + p.P[1]) * PAIR_B * PAIR_B;
}
// X of one (walker, determinant): [s][plane][dp_s] elements.
__host__ __device__ inline size_t pair_x_elems(const PairDims& p) {
  return 2 * (size_t)(p.dp[0] + p.dp[1]);
}

// Sizes, and whether the form is used: it needs Cholesky vectors, at least one virtual orbital
// per occupied spin, fewer operations than the products Omega^g (G small against M - N favours
// those: at M = 200, N = 50 the two meet near G = 50), and K tables within PAIR_MAX_BYTES.
inline void pair_plan(PairTables& t, int M, int nup, int ndn, int G, int n_det) {
  PairDims& p = t.dim;
  t.on = false;
  t.bytes = 0;
  p.n_det = n_det;
  p.G = G;
  p.Mp = (M + 15) / 16 * 16;
  p.Gt = (G + PAIR_B - 1) / PAIR_B;
  double fp = 0.0, fo = 0.0;
  bool ok = G > 0;
  for (int s = 0; s < 2; ++s) {
    const int N = s ? ndn : nup;
    p.N[s] = N;
    p.nv[s] = N > 0 ? M - N : 0;
    if (N > 0 && p.nv[s] < 1) ok = false;
    const long long d = (long long)N * p.nv[s];
    if (d > 1000000) {
      ok = false;
      p.d[s] = p.dp[s] = p.T[s] = p.P[s] = 0;
      continue;
    }
    p.d[s] = (int)d;
    p.T[s] = (p.d[s] + PAIR_B - 1) / PAIR_B;
    p.dp[s] = p.T[s] * PAIR_B;
    p.P[s] = p.T[s] * (p.T[s] + 1) / 2;
    fp += 2.0 * p.d[s] * (double)p.d[s] + 4.0 * G * p.d[s];
    fo += 4.0 * G * N * (double)N * M;
  }
  if (!ok || fp > fo) return;
  const size_t k = pair_k_elems(p);
  if (k * 8 > PAIR_MAX_BYTES) return;
  const size_t nv = (size_t)p.nv[0] + p.nv[1];
  t.bytes = (k + pair_b_elems(p) + n_det * (nv * p.Mp + p.dp[0] + p.dp[1] + 2 * (size_t)G + 2)) * 8;
  t.on = true;
}

inline void pair_free_tables(PairTables& t) {
  (void)hipFree(t.K);
  t = PairTables();
}

// ---------------------------------------------------------------------------
// Setup: B^g = Lh^g Q of one (determinant, spin), rows (g, c) of Lh at Lh + g gst + c M, on
// v_mfma_f64_16x16x4_f64: one wavefront per 16 rows and 64 virtuals.  B [G][dp] zeroed before.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_pair_b(int M, int Mp, int N, int nv, int G, int dp, size_t gst,
                                               const double* __restrict__ Lh,
                                               const double* __restrict__ Qt,
                                               double* __restrict__ B) {
  const int lane = threadIdx.x, l16 = lane & 15, q = lane >> 4;
  const long long rows = (long long)G * N, r = (long long)blockIdx.x * 16 + l16;
  const long long rc = r < rows ? r : rows - 1;
  const double* lrow = Lh + (size_t)(rc / N) * gst + (size_t)(rc % N) * M;
  const double* qrow[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int a = blockIdx.y * 64 + 16 * b + l16;
    qrow[b] = Qt + (size_t)(a < nv ? a : nv - 1) * Mp;
  }
  f64x4 acc[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) acc[b] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < M; k0 += 16)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + 4 * q + u, kk = k < M ? k : M - 1;
      const double v = lrow[kk], l = k < M ? v : 0.0;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(l, qrow[b][k], acc[b], 0, 0, 0);
    }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const long long row = (long long)blockIdx.x * 16 + q + 4 * v;
    if (row >= rows) continue;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int a = blockIdx.y * 64 + 16 * b + l16;
      if (a < nv) B[(size_t)(row / N) * dp + (size_t)(row % N) * nv + a] = acc[b][v];
    }
  }
}

// ---------------------------------------------------------------------------
// Setup: the K units of one (determinant, spin) from B [G][dp] on v_mfma_f64_16x16x4_f64.
// C[r][q] = sum_g B^g_r B^g_q with r = (c', a), q = (c, a') is K_{(c,a),(c',a')}: a wavefront
// computes 32 x 32 of C straight from global memory (64-lane rows of B are contiguous) and
// stores what lies in block rows I >= J.  The units must be zeroed before (padding).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_pair_build(int d, int dp, int nv, int G,
                                                    const double* __restrict__ B,
                                                    double* __restrict__ K) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, q = lane >> 4;
  const int r0 = blockIdx.x * 64 + (wave >> 1) * 32, c0 = blockIdx.y * 64 + (wave & 1) * 32;
  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  // rows r0 + 31 and columns c0 + 31 stay below dp (a multiple of 128); g past G reads the
  // last vector and is zeroed
  for (int g0 = 0; g0 < G; g0 += 4) {
    const int g = g0 + q, gg = g < G ? g : G - 1;
    double fa[2], fb[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double v = B[(size_t)gg * dp + r0 + 16 * a + l16];
      fa[a] = g < G ? v : 0.0;
      fb[a] = B[(size_t)gg * dp + c0 + 16 * a + l16];
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb[b], acc[a][b], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = r0 + 16 * a + q + 4 * v, col = c0 + 16 * b + l16;
        if (r >= d || col >= d) continue;
        const int e = (col / nv) * nv + r % nv, f = (r / nv) * nv + col % nv;
        const int I = e >> 7, J = f >> 7;
        if (J > I) continue;
        K[((size_t)(I * (I + 1) / 2 + J) * PAIR_B + (e & 127)) * PAIR_B + (f & 127)] =
            I == J ? 0.5 * acc[a][b][v] : acc[a][b][v];
      }
}

// ---------------------------------------------------------------------------
// X = Q^T Theta of every (walker, determinant, spin) on v_mfma_f64_16x16x4_f64.  One
// wavefront per 16 orbitals c (the A operand, rows of Theta^T) and AB <= 6 blocks of 16 virtuals a (the accumulators of both planes take 16 AB VGPRs; the
// host picks AB so that the groups of blocks are even); the four wavefronts of a workgroup
// read the same rows of Q close in time, so they come from the L1.  Each lane takes four
// consecutive p per step in both operands.
// M = 128, N = 32 + 32, 1024 walkers: 0.125 ms, 234 MB read and written (0.154 ms without the
// loads ahead and the padded rows of Q).
// With thmax != NULL only the walker-spins whose max |Theta| exceeds `guard`.
// Grid: (walkers, 4-wavefront groups of (c block, a group) per spin, n_det).
// ---------------------------------------------------------------------------
constexpr int PV_AB = 6;   // most blocks of 16 virtuals per wavefront

template <int AB>
__global__ void __launch_bounds__(256, 2) k_pair_virtual(
    PairDims p, int M, const double* __restrict__ Qt, const cd* __restrict__ thetaT,
    const double* __restrict__ weight, double* __restrict__ x,
    const double* __restrict__ thmax, double guard, int g0 /*groups of spin 0*/) {
  const int w = blockIdx.x, d = blockIdx.z;
  const int s = (int)blockIdx.y >= g0 ? 1 : 0;
  if (!(weight[w] > 0.0)) return;
  const int N = p.N[s], nv = p.nv[s], ntot = p.N[0] + p.N[1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nab = (nv + 15) / 16, nag = (nab + AB - 1) / AB, ncb = (N + 15) / 16;
  const int job = 4 * ((int)blockIdx.y - (s ? g0 : 0)) + wave;
  if (job >= nag * ncb) return;
  const int cb = job / nag, ag = job % nag;
  const int wd = w * p.n_det + d;
  if (thmax && !(thmax[2 * wd + s] > guard)) return;
  const int l16 = lane & 15, q = lane >> 4;
  const int c_in = 16 * cb + l16, cc = c_in < N ? c_in : N - 1;
  const cd* Th = thetaT + ((size_t)wd * ntot + (s ? p.N[0] : 0) + cc) * M;
  const double* Qs = Qt + ((size_t)d * (p.nv[0] + p.nv[1]) + (s ? p.nv[0] : 0)) * p.Mp;
  const double* qrow[AB];
#pragma unroll
  for (int b = 0; b < AB; ++b) {
    const int a = 16 * (ag * AB + b) + l16;
    qrow[b] = Qs + (size_t)(a < nv ? a : nv - 1) * p.Mp + 4 * q;
  }
  f64x4 ar[AB], ai[AB];
#pragma unroll
  for (int b = 0; b < AB; ++b) ar[b] = ai[b] = f64x4{0.0, 0.0, 0.0, 0.0};
  // the next 16 p go out before the MFMAs of these; p past M reads Theta at M - 1 against the
  // zeros of Q's padding
  cd th[4], tn[4];
  f64x2 qv[AB][2], qn[AB][2];
  auto load = [&](int k0, cd (&t)[4], f64x2 (&v)[AB][2]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + 4 * q + u;
      t[u] = Th[k < M ? k : M - 1];
    }
#pragma unroll
    for (int b = 0; b < AB; ++b) {
      v[b][0] = *reinterpret_cast<const f64x2*>(qrow[b] + k0);
      v[b][1] = *reinterpret_cast<const f64x2*>(qrow[b] + k0 + 2);
    }
  };
  load(0, th, qv);
  for (int k0 = 0; k0 < M; k0 += 16) {
    load(k0 + 16 < M ? k0 + 16 : k0, tn, qn);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int b = 0; b < AB; ++b) {
        const double v = qv[b][u >> 1][u & 1];
        ar[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(th[u].re, v, ar[b], 0, 0, 0);
        ai[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(th[u].im, v, ai[b], 0, 0, 0);
      }
#pragma unroll
    for (int u = 0; u < 4; ++u) th[u] = tn[u];
#pragma unroll
    for (int b = 0; b < AB; ++b) {
      qv[b][0] = qn[b][0];
      qv[b][1] = qn[b][1];
    }
  }
  const size_t o = (size_t)wd * pair_x_elems(p) + (s ? 2 * (size_t)p.dp[0] : 0);
  const int dp = p.dp[s];
#pragma unroll
  for (int b = 0; b < AB; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 16 * cb + q + 4 * v, a = 16 * (ag * AB + b) + l16;
      if (c >= N || a >= nv) continue;
      x[o + (size_t)c * nv + a] = ar[b][v];
      x[o + dp + (size_t)c * nv + a] = ai[b][v];
    }
  // the padding of both planes
  if (job == 0)
    for (int e = p.d[s] + lane; e < dp; e += 64) x[o + e] = x[o + dp + e] = 0.0;
}

// ---------------------------------------------------------------------------
// Which units a workgroup takes.  C[s] column tiles of 64 walkers per spin.  Trace tiles
// (determinant, spin, column tile, k split, row tile) are dealt evenly: k each and one more to
// nhi of them, spread over the launch (packed at its start, they left the XCDs with unlike work:
// 13 % of the wavefronts' time idle).  The K units, in the order (determinant, spin, column
// tile, unit), are cut into contiguous runs in proportion to what each workgroup has left of an
// equal share.  Where a whole trace tile is more than that share (few walkers: at M = 150,
// N = 37, 64 walkers it was 33 units against 3, and 0.64 ms instead of 0.17), its k range is
// split ts ways, the parts go to scratch (at most PAIR_SPLIT of them) and k_pair_reduce adds them.
// ---------------------------------------------------------------------------
constexpr int PAIR_SPLIT = 64;

struct PairSched {
  int C[2], nwg, nhi, k, ts;
  long long tr, units, a, b;   // trace tiles; K units; run weights with and without the extra tile
};

__host__ __device__ inline PairSched pair_sched(const PairDims& p, int C0, int C1, int nwg) {
  PairSched r;
  r.C[0] = p.N[0] > 0 ? C0 : 0;
  r.C[1] = p.N[1] > 0 ? C1 : 0;
  r.nwg = nwg;
  const long long cols = (long long)p.n_det * (r.C[0] + r.C[1]);
  r.tr = cols * p.Gt;
  r.units = (long long)p.n_det * ((long long)r.C[0] * p.P[0] + (long long)r.C[1] * p.P[1]);
  const long long tu =
      (long long)p.n_det * p.Gt * ((long long)r.C[0] * p.T[0] + (long long)r.C[1] * p.T[1]);
  long long per = r.tr > 0 ? (tu + r.tr - 1) / r.tr : 0;   // units of a trace tile
  const long long cap = (r.units + tu + nwg - 1) / nwg;
  r.ts = 1;
  if (per > cap && cols > 0) {
    const int T = r.C[0] == 0 ? p.T[1] : r.C[1] == 0 ? p.T[0] : p.T[0] < p.T[1] ? p.T[0] : p.T[1];
    long long ts = (per + cap - 1) / cap;
    if (ts > PAIR_SPLIT / cols) ts = PAIR_SPLIT / cols;
    if (ts > T) ts = T;
    r.ts = ts < 1 ? 1 : (int)ts;
  }
  per = (per + r.ts - 1) / r.ts;
  r.tr *= r.ts;
  r.k = (int)(r.tr / nwg);
  r.nhi = (int)(r.tr % nwg);
  r.a = cap - (r.k + 1) * per;
  r.b = cap - r.k * per;
  if (r.a < 0) r.a = 0;
  if (r.b < 1) r.b = 1;
  return r;
}
// Workgroups below wg with an extra trace tile, and the first K unit of wg's run.
__host__ __device__ inline int pair_hi(const PairSched& r, int wg) {
  return (int)((long long)wg * r.nhi / r.nwg);
}
__host__ __device__ inline long long pair_cum(const PairSched& r, int wg) {
  return wg * r.b - pair_hi(r, wg) * (r.b - r.a);
}
__host__ __device__ inline long long pair_start(const PairSched& r, int wg) {
  return r.units * pair_cum(r, wg) / pair_cum(r, r.nwg);
}
// Column tile (counted over determinants and spins) and first unit of tile (d, s, c).
__host__ __device__ inline long long pair_tile_unit(const PairDims& p, const PairSched& r, int d,
                                                    int s, int c) {
  return (long long)d * ((long long)r.C[0] * p.P[0] + (long long)r.C[1] * p.P[1]) +
         (s ? (long long)r.C[0] * p.P[0] : 0) + (long long)c * p.P[s];
}
__host__ __device__ inline int pair_tile_index(const PairSched& r, int d, int s, int c) {
  return d * (r.C[0] + r.C[1]) + (s ? r.C[0] : 0) + c;
}
// Workgroups of a launch: two per compute unit, no more than there is work for and at most two for
// each of the MI355X's 256, for which the scratch is laid out (its size is host arithmetic alone).
constexpr int PAIR_WG = 512;
inline int pair_grid(const PairDims& p, int nw, int cus) {
  const int C = (nw + PAIR_W - 1) / PAIR_W;
  const PairSched r = pair_sched(p, C, C, 1);   // one workgroup: r.b is all there is to do
  const long long n = std::min(2 * cus, PAIR_WG), most = r.b > 0 ? r.b + r.tr * std::max(p.T[0], p.T[1]) : 1;
  return (int)(most < n ? most : n);
}
inline size_t pair_part_elems(const PairDims& p, int nw) {
  const int C = (nw + PAIR_W - 1) / PAIR_W;
  return ((size_t)PAIR_WG + (size_t)p.n_det * 2 * C) * PAIR_W;
}
// Scratch of split traces: column tiles times splits of what pair_sched makes of all nw walkers, or
// (any) of any part of them.  There ts < per / cap + 1 with per <= T and cap >= cols (P + Gt T) / nwg,
// so cols ts is at most T nwg / (P + Gt T) + cols, and ts > 1 needs cols <= PAIR_SPLIT / 2.
inline size_t pair_split_elems(const PairDims& p, int nw, bool any) {
  const int C = (nw + PAIR_W - 1) / PAIR_W, nwg = pair_grid(p, nw, PAIR_WG / 2);
  long long tiles = 0;
  if (any) {
    long long cols = 0, T = 1, unit = 0;
    for (int s = 0; s < 2; ++s) {
      if (p.N[s] == 0) continue;
      const long long u = p.P[s] + (long long)p.Gt * p.T[s];
      cols += (long long)p.n_det * C;
      unit = unit == 0 ? u : std::min(unit, u);
      T = std::max(T, (long long)p.T[s]);
    }
    cols = std::min(cols, (long long)PAIR_SPLIT / 2);
    if (T > 1) tiles = std::min({(long long)PAIR_SPLIT, cols * T, T * nwg / unit + cols});
  } else {
    const PairSched r = pair_sched(p, C, C, nwg);
    if (r.ts > 1) tiles = (long long)p.n_det * (r.C[0] + r.C[1]) * r.ts;
  }
  return (size_t)tiles * PAIR_W * p.G;
}

struct PairArgs {
  PairDims p;
  int nw;
  const double *K, *B, *f, *t0, *X;
  cd* tpart;                 // [nw][n_det][2][G]
  cd* part;                  // [workgroup + column tile][64] partial sums
  cd* split;                 // [column tile][split][64][G] parts of split traces
  long long* start;          // [workgroups + 1] first K unit of each workgroup's run
  // the precision guard: walkers list[s][0 .. cnt[s]) instead of 0 .. nw, of which only the
  // determinants with thmax above guard are written
  const int* list;           // [2][nw]
  const int* cnt;            // [2]
  const double* thmax;       // [nw][n_det][2]
  double guard;
};

// One run of 16-k chunks with the same row tile and 128-k block.
struct PairSeg {
  int kind;        // 0: trace rows, 1: K unit, -1: nothing left
  int d, s, c;     // determinant, spin, column tile
  int I, J;        // row tile and k block
  int Je, sp;      // trace: end of its k blocks, and which split it is
  int nch;         // chunks
  bool last;       // the row tile's accumulators are complete (for this workgroup) after it
};

// Workgroup: 128 rows x 64 walkers x {Re, Im}, four wavefronts of 64 rows x 32 walkers (16
// blocks of v_mfma_f64_16x16x4_f64, 128 accumulator VGPRs), chunks of 16 k double-buffered in
// LDS (74 KB: two workgroups per CU), the next chunk's loads ahead of this one's MFMAs also
// across units and tiles.  A lane takes two consecutive k of its row in both operands.
// M = 128, N = 32 + 32, G = 800, 1024 walkers: 1.13 ms, 55 TFLOP/s (77 % of the matrix cores'
// cycles at the 2.2 GHz the card holds in FP64; 62 TFLOP/s on all-zero data; eight wavefronts
// of half the columns gave the same).
constexpr int PAIR_LD = PAIR_KC + 2;
constexpr int PAIR_LDS = 4 * PAIR_B * PAIR_LD * 8;

__global__ void __launch_bounds__(256, 2) k_pair(PairArgs g) {
  constexpr int LD = PAIR_LD, NP = 4, RSTEP = 32;    // 16-byte pieces per thread; row step
  extern __shared__ __attribute__((aligned(16))) double pair_smem[];
  double* const As = pair_smem;                       // [2][128][LD]
  double* const Bs = As + 2 * PAIR_B * LD;            // [2][128][LD]
  __shared__ cd red[2][PAIR_W];
  const PairDims& p = g.p;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = wave >> 1, cw = wave & 1;
  // contiguous runs of logical workgroups per XCD (they are dispatched round-robin): the
  // column tiles of a run stay in one L2
  const int nwg = gridDim.x;
  int wg = blockIdx.x;
  {
    const int x = wg & 7, j = wg >> 3, q8 = nwg >> 3, r8 = nwg & 7;
    wg = x * q8 + (x < r8 ? x : r8) + j;
  }
  const int n0 = __builtin_amdgcn_readfirstlane(g.list ? g.cnt[0] : g.nw);
  const int n1 = __builtin_amdgcn_readfirstlane(g.list ? g.cnt[1] : g.nw);
  const PairSched sc = pair_sched(p, (n0 + PAIR_W - 1) / PAIR_W, (n1 + PAIR_W - 1) / PAIR_W, nwg);
  const size_t xst = pair_x_elems(p);
  auto walker = [&](int s, int n) {   // walker n of spin s (past the end: the last one)
    const int cnt = s ? n1 : n0;
    n = n < cnt ? n : cnt - 1;
    return g.list ? g.list[(size_t)s * g.nw + n] : n;
  };

  // ---- the workgroup's sequence of segments
  int tk = 0;                                  // trace tiles taken
  const int hi = pair_hi(sc, wg), nt = sc.k + (pair_hi(sc, wg + 1) > hi ? 1 : 0);
  long long u = pair_start(sc, wg), u1 = pair_start(sc, wg + 1);
  if (tid == 0) {
    g.start[wg] = u;
    if (wg == nwg - 1) g.start[nwg] = u1;
  }
  PairSeg ls;
  ls.kind = -1;
  int left = 0;                                // K units left in the column tile
  auto chunks = [&](int s, int J) {            // 16-k chunks of block J that hold amplitudes
    const int n = (p.d[s] - PAIR_B * J + PAIR_KC - 1) / PAIR_KC;
    return n < PAIR_B / PAIR_KC ? n : PAIR_B / PAIR_KC;
  };
  auto next = [&]() {
    if (ls.kind == 0 && !ls.last) {            // the trace tile's next k block
      ++ls.J;
      ls.last = ls.J + 1 == ls.Je;
      ls.nch = chunks(ls.s, ls.J);
      return;
    }
    if (tk < nt) {
      const long long tt = tk < sc.k ? wg + (long long)tk * nwg : (long long)sc.k * nwg + hi;
      const int gts = p.Gt * sc.ts, per_det = (sc.C[0] + sc.C[1]) * gts;
      int r = (int)(tt % per_det);
      ls.kind = 0;
      ls.d = (int)(tt / per_det);
      ls.s = r >= sc.C[0] * gts ? 1 : 0;
      r -= ls.s ? sc.C[0] * gts : 0;
      ls.c = r / gts;
      r %= gts;
      ls.sp = r / p.Gt;
      ls.I = r % p.Gt;
      ls.J = p.T[ls.s] * ls.sp / sc.ts;
      ls.Je = p.T[ls.s] * (ls.sp + 1) / sc.ts;
      ls.last = ls.J + 1 == ls.Je;
      ls.nch = chunks(ls.s, ls.J);
      ++tk;
      return;
    }
    if (u >= u1) {
      ls.kind = -1;
      return;
    }
    if (ls.kind == 1 && left > 0) {            // the next unit of the same column tile
      if (ls.J == ls.I) {
        ++ls.I;
        ls.J = 0;
      } else {
        ++ls.J;
      }
    } else {
      const long long per_det =
          (long long)sc.C[0] * p.P[0] + (long long)sc.C[1] * p.P[1];
      long long r = u % per_det;
      ls.kind = 1;
      ls.d = (int)(u / per_det);
      ls.s = r >= (long long)sc.C[0] * p.P[0] ? 1 : 0;
      r -= ls.s ? (long long)sc.C[0] * p.P[0] : 0;
      ls.c = (int)(r / p.P[ls.s]);
      const int m = (int)(r % p.P[ls.s]);
      int I = (int)((sqrtf(8.f * (float)m + 1.f) - 1.f) * 0.5f);
      while (I * (I + 1) / 2 > m) --I;
      while ((I + 1) * (I + 2) / 2 <= m) ++I;
      ls.I = __builtin_amdgcn_readfirstlane(I);
      ls.J = m - ls.I * (ls.I + 1) / 2;
      left = p.P[ls.s] - m;
    }
    --left;
    ++u;
    ls.last = ls.J == ls.I || u >= u1;
    ls.nch = chunks(ls.s, ls.J);
  };

  // ---- staging: piece i of a thread is row prow + 32 i of the tile, two k from pk.  Row r of
  // the column tile: wavefront column block r / 64, plane (r / 32) % 2, walker r % 32.
  const int prow = tid >> 3, pk = (tid & 7) * 2;
  const char* ab = nullptr;       // uniform: the A tile at k block J
  unsigned aoff = 0, astep = 0;   // this thread's piece 0, and the step to the next (bytes)
  const char* bp[NP];             // the column rows at k = 0
  unsigned kb = 0;                // uniform: byte offset of k block J
  auto point = [&](const PairSeg& was) {
    if (ls.kind == 0) {
      ab = reinterpret_cast<const char*>(
          g.B + (size_t)ls.d * p.G * (p.dp[0] + p.dp[1]) + (ls.s ? (size_t)p.G * p.dp[0] : 0) +
          (size_t)PAIR_B * ls.I * p.dp[ls.s] + PAIR_B * ls.J);
      aoff = (unsigned)(prow * p.dp[ls.s] + pk) * 8u;
      astep = RSTEP * (unsigned)p.dp[ls.s] * 8u;
    } else {
      const size_t unit = (size_t)ls.d * (p.P[0] + p.P[1]) + (ls.s ? p.P[0] : 0) +
                          ls.I * (ls.I + 1) / 2 + ls.J;
      ab = reinterpret_cast<const char*>(g.K + unit * PAIR_B * PAIR_B);
      aoff = (unsigned)(prow * PAIR_B + pk) * 8u;
      astep = RSTEP * PAIR_B * 8u;
    }
    kb = (unsigned)(PAIR_B * ls.J) * 8u;
    if (was.kind < 0 || was.d != ls.d || was.s != ls.s || was.c != ls.c) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int r = prow + RSTEP * i;
        const int w = walker(ls.s, PAIR_W * ls.c + 32 * (r >> 6) + (r & 31));
        bp[i] = reinterpret_cast<const char*>(
            g.X + ((size_t)w * p.n_det + ls.d) * xst + (ls.s ? 2 * (size_t)p.dp[0] : 0) +
            ((r >> 5) & 1) * (size_t)p.dp[ls.s] + pk);
      }
    }
  };
  u32x4 sa[NP], sb[NP];
  auto gload = [&](int ch) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      sa[i] = *reinterpret_cast<const u32x4*>(ab + (size_t)i * astep + PAIR_KC * 8 * ch + aoff);
      sb[i] = *reinterpret_cast<const u32x4*>(bp[i] + (kb + PAIR_KC * 8 * ch));
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      *reinterpret_cast<u32x4*>(&As[(buf * PAIR_B + prow + RSTEP * i) * LD + pk]) = sa[i];
      *reinterpret_cast<u32x4*>(&Bs[(buf * PAIR_B + prow + RSTEP * i) * LD + pk]) = sb[i];
    }
  };

  f64x4 acc[4][2][2];                      // [row block of 16][walker block of 16][plane]
  auto clear = [&]() {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b][0] = acc[a][b][1] = f64x4{0.0, 0.0, 0.0, 0.0};
  };
  double er[2] = {0.0, 0.0}, ei[2] = {0.0, 0.0};   // walkers 32 cw + 16 b + l16
  clear();
  next();
  if (ls.kind < 0) return;
  PairSeg cs = ls;
  cs.kind = -1;
  point(cs);
  int lch = 0, buf = 0;
  gload(0);
  lstore(0);
  __syncthreads();
  cs = ls;
  int cch = 0;
  while (cs.kind >= 0) {
    // the chunk after this one goes out first
    if (++lch == ls.nch) {
      next();
      lch = 0;
      if (ls.kind >= 0) point(cs);
    }
    const bool more = ls.kind >= 0;
    if (more) gload(lch);
    {
      const double* A = As + (buf * PAIR_B + 64 * rw + l16) * LD + 2 * q;
      const double* B = Bs + (buf * PAIR_B + 64 * cw + l16) * LD + 2 * q;
#pragma unroll
      for (int kk = 0; kk < PAIR_KC; kk += 8) {
        f64x2 fa[4], fb[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          fa[a] = *reinterpret_cast<const f64x2*>(A + 16 * a * LD + kk);
          fb[a] = *reinterpret_cast<const f64x2*>(B + 16 * a * LD + kk);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int pl = 0; pl < 2; ++pl)
                acc[a][b][pl] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                    fa[a][e], fb[2 * pl + b][e], acc[a][b][pl], 0, 0, 0);
      }
    }
    if (more) lstore(buf ^ 1);
    if (++cch == cs.nch) {
      if (cs.last) {
        const int cnt = cs.s ? n1 : n0;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int n = PAIR_W * cs.c + 32 * cw + 16 * b + l16;
          const int w = walker(cs.s, n);
          const size_t wds = ((size_t)w * p.n_det + cs.d) * 2 + cs.s;
          const int row = PAIR_B * cs.I + 64 * rw + q;   // + 16 a + 4 v
          if (cs.kind == 0) {
            if (n >= cnt || (g.list && !(g.thmax[wds] > g.guard))) continue;
            cd* t = sc.ts == 1
                        ? g.tpart + wds * p.G
                        : g.split + (((size_t)pair_tile_index(sc, cs.d, cs.s, cs.c) * sc.ts + cs.sp) *
                                         PAIR_W + (n - PAIR_W * cs.c)) * p.G;
            const double* t0 = g.t0 + ((size_t)cs.d * 2 + cs.s) * p.G;
            const double f0 = cs.sp == 0 ? 1.0 : 0.0;
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int gg = row + 16 * a + 4 * v;
                if (gg < p.G) t[gg] = mkc(fma(f0, t0[gg], acc[a][b][0][v]), acc[a][b][1][v]);
              }
          } else {
            const int dp = p.dp[cs.s];
            const double* x = g.X + ((size_t)w * p.n_det + cs.d) * xst +
                              (cs.s ? 2 * (size_t)p.dp[0] : 0) + row;
            // the linear term, with the block row's last unit
            const double* f = g.f + (size_t)cs.d * (p.dp[0] + p.dp[1]) + (cs.s ? p.dp[0] : 0) + row;
            const double ff = cs.J == cs.I ? 1.0 : 0.0;
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int o = 16 * a + 4 * v;
                const double xr = x[o], xi = x[dp + o];
                const double zr = fma(ff, f[o], acc[a][b][0][v]), zi = acc[a][b][1][v];
                er[b] = fma(xr, zr, fma(-xi, zi, er[b]));
                ei[b] = fma(xr, zi, fma(xi, zr, ei[b]));
              }
          }
        }
        clear();
      }
      // the column tile's partial sum, when the next segment is in another one
      if (cs.kind == 1 && (ls.kind != 1 || ls.c != cs.c || ls.s != cs.s || ls.d != cs.d)) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          double r = er[b], i = ei[b];
          r += __shfl_xor(r, 16);
          i += __shfl_xor(i, 16);
          r += __shfl_xor(r, 32);
          i += __shfl_xor(i, 32);
          if (lane < 16) red[rw][32 * cw + 16 * b + lane] = mkc(r, i);
          er[b] = ei[b] = 0.0;
        }
        __syncthreads();
        if (tid < PAIR_W)
          g.part[((size_t)wg + pair_tile_index(sc, cs.d, cs.s, cs.c)) * PAIR_W + tid] =
              cadd(red[0][tid], red[1][tid]);
      }
      cs = ls;
      cch = 0;
    }
    buf ^= 1;
    __syncthreads();
  }
}

// blockIdx.z == 0: exch[w][d][s] = c0 + 2 (sum over the workgroups whose run meets the walker's
// column tile, in a fixed order); zero exchange and traces of an empty spin.  One workgroup per
// column tile, one lane per walker; wavefront v searches the runs (start) of 64 workgroups at a
// time.  blockIdx.z > 0: the sums of split traces, 128 rows g per workgroup.
__global__ void __launch_bounds__(1024) k_pair_reduce(PairDims p, int nw, int nwg,
                                                      const cd* __restrict__ part,
                                                      const cd* __restrict__ split,
                                                      const long long* __restrict__ start,
                                                      const double* __restrict__ c0,
                                                      cd* __restrict__ exch, cd* __restrict__ tpart,
                                                      const int* __restrict__ list,
                                                      const int* __restrict__ cnt,
                                                      const double* __restrict__ thmax,
                                                      double guard, int nz, size_t xst) {
  __shared__ cd red[16][PAIR_W];
  const int c = blockIdx.x, s = blockIdx.y & 1, d = blockIdx.y >> 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (p.N[s] == 0) {
    if (list || blockIdx.z) return;
    for (int j = wave; j < PAIR_W && c * PAIR_W + j < nw; j += 16) {
      const size_t wds = ((size_t)(c * PAIR_W + j) * p.n_det + d) * 2 + s;
      for (int e = lane; e < p.G; e += 64) tpart[wds * p.G + e] = mkc(0.0, 0.0);
      if (lane == 0) exch[wds] = mkc(0.0, 0.0);
    }
    return;
  }
  const int n0 = __builtin_amdgcn_readfirstlane(list ? cnt[0] : nw);
  const int n1 = __builtin_amdgcn_readfirstlane(list ? cnt[1] : nw);
  const int ns = s ? n1 : n0;
  if (c * PAIR_W >= ns) return;
  const PairSched sc = pair_sched(p, (n0 + PAIR_W - 1) / PAIR_W, (n1 + PAIR_W - 1) / PAIR_W, nwg);
  const int tile = pair_tile_index(sc, d, s, c);
  auto slot = [&](int n) {   // (walker, determinant, spin) of walker n, or -1 if it is not written
    if (n >= ns) return (long long)-1;
    const long long w = list ? list[(size_t)s * nw + n] : n;
    const long long wds = (w * p.n_det + d) * 2 + s;
    return list && !(thmax[wds] > guard) ? (long long)-1 : wds;
  };
  if (blockIdx.z) {
    if (sc.ts == 1) return;
    const int g = ((int)blockIdx.z - 1) * PAIR_B + (tid & 127);
    if (g >= p.G) return;
    for (int j = tid >> 7; j < PAIR_W; j += 8) {
      const long long wds = slot(c * PAIR_W + j);
      if (wds < 0) continue;
      cd t = mkc(0.0, 0.0);
      for (int k = 0; k < sc.ts; ++k)
        t = cadd(t, split[(((size_t)tile * sc.ts + k) * PAIR_W + j) * p.G + g]);
      tpart[wds * p.G + g] = t;
    }
    return;
  }
  const long long a = pair_tile_unit(p, sc, d, s, c), b = a + p.P[s];
  // workgroups with a run inside [a, b): consecutive but for empty runs
  cd x = mkc(0.0, 0.0);
  for (int g0 = 64 * wave; g0 < nwg; g0 += 1024) {
    const int gl = g0 + lane;
    const long long s0 = gl < nwg ? start[gl] : b, s1 = gl < nwg ? start[gl + 1] : b;
    const unsigned long long m = __ballot(s0 < b && s1 > a && s1 > s0);
    if (!m) continue;
    const int lo = __builtin_ctzll(m), hi = 63 - __builtin_clzll(m);
#pragma unroll 8
    for (int i = lo; i <= hi; ++i) {
      const cd v = part[((size_t)(g0 + i) + tile) * PAIR_W + lane];
      if ((m >> i) & 1ull) x = cadd(x, v);
    }
  }
  red[wave][lane] = x;
  __syncthreads();
  if (wave) return;
  for (int v = 1; v < 16; ++v) x = cadd(x, red[v][lane]);
  const long long wds = slot(c * PAIR_W + lane);
  if (wds < 0) return;
  exch[wds] = mkc(fma(2.0, x.re, c0[2 * d + s]), 2.0 * x.im);
  // the partial sums of a split low-precision contraction of the same walker-spin
  for (int z = 1; z < nz; ++z) exch[z * xst + wds] = mkc(0.0, 0.0);
}

// ---------------------------------------------------------------------------
// Precision guard of the mixed modes.  glist: the live walkers whose largest |Theta_pc| over
// spins and determinants exceeds `limit`, in walker order, their number in gcount[0] (added to
// counts[CAP_GUARD] when counts != NULL); slist[s]: those whose spin s does (over
// determinants), gcount[1 + s] of them; ulist[s]: the live walkers with a determinant whose spin
// s does not, gcount[3 + s] of them (the low-precision contraction takes only these).  One workgroup; every 1024 walkers one ballot per
// wavefront and a prefix over the 16 wavefronts (a scan by one thread took 13.7 us).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024) k_guard_list(int nw, int nd, double limit,
                                                     const double* __restrict__ weight,
                                                     const double* __restrict__ thmax,
                                                     int* __restrict__ glist, int* __restrict__ slist,
                                                     int* __restrict__ ulist,
                                                     int* __restrict__ gcount,
                                                     unsigned long long* __restrict__ counts) {
  constexpr int NL = 5;
  __shared__ int wsum[NL][16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int* const out[NL] = {glist, slist, slist + nw, ulist, ulist + nw};
  int base[NL] = {};
  for (int w0 = 0; w0 < nw; w0 += 1024) {
    const int w = w0 + tid;
    bool f[NL] = {};
    if (w < nw && weight[w] > 0.0) {
      double m0 = 0.0, m1 = 0.0;
      bool u0 = false, u1 = false;
      for (int i = 0; i < nd; ++i) {
        const double a = thmax[(size_t)w * 2 * nd + 2 * i], b = thmax[(size_t)w * 2 * nd + 2 * i + 1];
        m0 = fmax(m0, a);
        m1 = fmax(m1, b);
        u0 = u0 || !(a > limit);
        u1 = u1 || !(b > limit);
      }
      f[1] = m0 > limit;
      f[2] = m1 > limit;
      f[0] = f[1] || f[2];
      f[3] = u0;
      f[4] = u1;
    }
    unsigned long long m[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      m[i] = __ballot(f[i]);
      if (lane == 0) wsum[i][wv] = __popcll(m[i]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      int before = base[i], all = 0;
      for (int k = 0; k < 16; ++k) {
        const int v = wsum[i][k];
        before += k < wv ? v : 0;
        all += v;
      }
      if (f[i]) out[i][before + __popcll(m[i] & ((1ull << lane) - 1ull))] = w;
      base[i] += all;
    }
    __syncthreads();
  }
  if (tid == 0) {
    for (int i = 0; i < NL; ++i) gcount[i] = base[i];
    if (counts && base[0] > 0) atomicAdd(&counts[CAP_GUARD], (unsigned long long)base[0]);
  }
}

// k_pair and the sums of its partials (part: pair_part_elems, split: pair_split_elems, start:
// PAIR_WG + 1).
inline hipError_t pair_contract(const PairTables& t, hipStream_t st, int nw, int cus,
                                const double* X, cd* tpart, cd* exch, cd* part, cd* split,
                                long long* start, const int* list = nullptr, const int* cnt = nullptr,
                                const double* thmax = nullptr, double guard = 0.0, int nz = 1,
                                size_t xst = 0) {
  const PairArgs a{t.dim, nw,    t.K,   t.B,  t.f, t.t0,  X,
                   tpart, part,  split, start, list, cnt, thmax, guard};
  const int nwg = pair_grid(t.dim, nw, cus);
  (void)hipFuncSetAttribute((const void*)k_pair, hipFuncAttributeMaxDynamicSharedMemorySize,
                            PAIR_LDS);
  hipLaunchKernelGGL(k_pair, dim3(nwg), dim3(256), PAIR_LDS, st, a);
  hipLaunchKernelGGL(k_pair_reduce, dim3((nw + PAIR_W - 1) / PAIR_W, 2 * t.dim.n_det, 1 + t.dim.Gt),
                     dim3(1024), 0, st, t.dim, nw, nwg, (const cd*)part, (const cd*)split,
                     (const long long*)start,
                     (const double*)t.c0, exch, tpart, list, cnt, thmax, guard, nz, xst);
  return hipGetLastError();
}

inline void pair_virtual(const PairTables& t, hipStream_t st, int nw, int M, const cd* thetaT,
                         const double* weight, double* x, const double* thmax, double guard) {
  const int nab = (std::max(t.dim.nv[0], t.dim.nv[1]) + 15) / 16;
  const int nag = (nab + PV_AB - 1) / PV_AB, ab = (nab + nag - 1) / nag;
  auto groups = [&](int s) {
    const int n = ((t.dim.nv[s] + 15) / 16 + ab - 1) / ab;
    return t.dim.N[s] > 0 ? (n * ((t.dim.N[s] + 15) / 16) + 3) / 4 : 0;
  };
  const int g0 = groups(0), g1 = groups(1);
  const dim3 grid(nw, g0 + g1, t.dim.n_det);
#define PAIR_VIRTUAL(ABV)                                                                      \
  case ABV:                                                                                    \
    hipLaunchKernelGGL(k_pair_virtual<ABV>, grid, dim3(256), 0, st, t.dim, M,                  \
                       (const double*)t.Qt, thetaT, weight, x, thmax, guard, g0);       \
    break;
  switch (ab) {
    PAIR_VIRTUAL(1) PAIR_VIRTUAL(2) PAIR_VIRTUAL(3) PAIR_VIRTUAL(4) PAIR_VIRTUAL(5)
    default: PAIR_VIRTUAL(6)
  }
#undef PAIR_VIRTUAL
}
