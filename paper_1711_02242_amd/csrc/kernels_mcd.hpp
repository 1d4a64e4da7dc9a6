// Modified Cholesky decomposition of the two-electron tensor on the GPU
// (arXiv:1711.02242, Sec. II.B.2, eq:chol, eq:chol2).
//
// V_{mu nu} = v_pqrs with mu = p M + r, nu = q M + s, v stored as eri[p][q][r][s].
// Only the diagonal of the residual, D_mu = (V - sum_g L^g L^g^T)_{mu mu}, is kept:
// the pivot column of the residual is rebuilt from the tensor and the previous
// vectors, c_mu = V_{mu nu0} - sum_g L^g_mu L^g_nu0.  Per vector, one launch of k_mcd_vector:
//   nu0 = argmax D (first index on ties), Dmax; stop when Dmax < delta;
//   damped prescreening sqrt(|D_mu| Dmax) <= min(1e-9, delta) -> mu dead (D_mu = 0);
//   L_mu = c_mu / sqrt(Dmax) (0 for dead mu), D_mu -= L_mu^2.
// What bounds it: the previous vectors are read once per vector (n M^2 doubles, mostly from the
// L2 of the XCD that wrote them) behind a chain of a launch, the pivot and one latency per batch
// of loads.  So a workgroup takes 64 mu with 16 wavefronts, wavefront v the vectors g = v, v + 16,
// ...; L^g_nu0 is gathered into LDS by all threads at once; and each workgroup leaves the
// argmax of its 64 new D for the next launch, where every workgroup reduces all of them.  (One
// thread per mu running over all g, and a pivot launch of its own: 66 us per vector at M = 64
// and up to 512 vectors, 33.7 ms in all; now 9.1 us per vector, 4.65 ms.)
#pragma once

#include "common.hpp"

struct McdState {
  int done;       // 1 once converged or out of vectors
  int count;      // number of vectors when done
  int piv, pad;   // unused
  double dmax;    // largest residual diagonal when done
};

constexpr int MCD_B = 64;          // mu per workgroup
constexpr int MCD_G = 1024;        // L^g_nu0 staged in LDS at a time

// Largest D of a workgroup's mu (ties to the smallest mu).
struct McdBest {
  double d;
  int mu, pad;
};

// Per workgroup b: dead bits of its 64 mu, and two McdBest (by parity of the vector), in the
// M^2 bytes (rounded up to 256) that the workspace holds behind D: 40 bytes per 64 of them.
__host__ __device__ inline int mcd_blocks(int MM) { return (MM + MCD_B - 1) / MCD_B; }

__device__ __forceinline__ void mcd_best_of_wave(double d, int mu, McdBest* out, int lane) {
  wave_argmax(d, mu);
  if (lane == 0) *out = McdBest{d, mu, 0};
}

// One wavefront per 64 mu.
__global__ void __launch_bounds__(64) k_mcd_init(int M, const double* __restrict__ eri,
                                                 double* __restrict__ D,
                                                 unsigned long long* __restrict__ dead,
                                                 McdBest* __restrict__ best,
                                                 McdState* __restrict__ st) {
  const int MM = M * M, lane = threadIdx.x, mu = blockIdx.x * MCD_B + lane;
  double d = -INFINITY;
  if (mu < MM) {
    const int p = mu / M, r = mu % M;
    d = eri[(((size_t)p * M + p) * M + r) * M + r];
    D[mu] = d;
  }
  // strict comparison with -infinity: a NaN diagonal is never chosen
  mcd_best_of_wave(d > -INFINITY ? d : -INFINITY, d > -INFINITY ? mu : MM, &best[blockIdx.x], lane);
  if (lane == 0) dead[blockIdx.x] = 0ull;
  if (mu == 0) {
    st->done = 0;
    st->count = 0;
    st->piv = -1;
    st->pad = 0;
    st->dmax = 0.0;
  }
}

// Vector n.  best: [2][blocks], parity n & 1 read, the other written.
__global__ void __launch_bounds__(1024) k_mcd_vector(int M, int n, double delta, int max_vectors,
                                                     const double* __restrict__ eri,
                                                     double* __restrict__ L /*[..][MM]*/,
                                                     double* __restrict__ D,
                                                     unsigned long long* __restrict__ dead,
                                                     McdBest* __restrict__ best,
                                                     McdState* __restrict__ st) {
  __shared__ double s_l[MCD_G];
  __shared__ double s_c[16][MCD_B];
  __shared__ McdBest s_b[16];
  const int MM = M * M, nb = mcd_blocks(MM);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // ---- the pivot, from what the launch before left: the same for every wavefront of every block.
  // `st` is not asked (a block of this launch may be writing it): a launch past the end finds the
  // maxima that the last one handed on.
  const McdBest* in = best + (size_t)(n & 1) * nb;
  McdBest* out = best + (size_t)((n + 1) & 1) * nb + blockIdx.x;
  {
    double d = -INFINITY;
    int mu = MM;
    for (int b = tid; b < nb; b += 1024) {
      const McdBest x = in[b];
      if (x.d > d || (x.d == d && x.mu < mu)) {
        d = x.d;
        mu = x.mu;
      }
    }
    mcd_best_of_wave(d, mu, &s_b[wave], lane);
  }
  __syncthreads();
  double dmax = -INFINITY;
  int nu0 = MM;
  for (int v = 0; v < 16; ++v) {
    const McdBest x = s_b[v];
    if (x.d > dmax || (x.d == dmax && x.mu < nu0)) {
      dmax = x.d;
      nu0 = x.mu;
    }
  }
  if (!(dmax >= delta) || n >= max_vectors) {
    if (tid == 0) *out = in[blockIdx.x];
    if (blockIdx.x == 0 && tid == 0 && !st->done) {
      st->count = n;
      st->dmax = dmax;
      st->done = 1;
    }
    return;
  }
  // ---- c_mu: sums over the previous vectors, 16 wavefronts of 64 mu
  const int mu = blockIdx.x * MCD_B + lane, muc = mu < MM ? mu : MM - 1;
  double acc = 0.0;
  for (int g0 = 0; g0 < n; g0 += MCD_G) {
    __syncthreads();
    if (g0 + tid < n) s_l[tid] = L[(size_t)(g0 + tid) * MM + nu0];
    __syncthreads();
    const int ng = n - g0 < MCD_G ? n - g0 : MCD_G;
    const double* Lg = L + (size_t)g0 * MM + muc;
#pragma unroll 8
    for (int g = wave; g < ng; g += 16) acc = fma(Lg[(size_t)g * MM], s_l[g], acc);
  }
  s_c[wave][lane] = acc;
  __syncthreads();
  if (wave) return;
  for (int v = 1; v < 16; ++v) acc += s_c[v][lane];
  double d = -INFINITY;
  bool gone = false;
  if (mu < MM) {
    const int p = mu / M, r = mu % M, q = nu0 / M, s = nu0 % M;
    d = D[mu];
    gone = (dead[blockIdx.x] >> lane) & 1ull;
    if (!gone && sqrt(fabs(d) * dmax) <= fmin(1e-9, delta)) {
      gone = true;
      d = 0.0;
    }
    double l = 0.0;
    if (!gone) {
      l = (eri[(((size_t)p * M + q) * M + r) * M + s] - acc) / sqrt(dmax);
      d = mu == nu0 ? 0.0 : d - l * l;
    }
    L[(size_t)n * MM + mu] = l;
    D[mu] = d;
  }
  const unsigned long long bits = __ballot(gone);
  if (lane == 0) dead[blockIdx.x] = bits;
  mcd_best_of_wave(d > -INFINITY ? d : -INFINITY, d > -INFINITY ? mu : MM, out, lane);
}
