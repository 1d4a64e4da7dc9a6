// FP32 MFMA kernels of the propagation (arXiv:1711.02242, Sec. III.D.2, Theorem 1.4,
// eq:primitive):
//
//   A_w = i s sum_g y_wg L^g                       (propagator exponent, y = x - xbar)
//   U_w <- E_h T_n(A_w) E_h U_w,   T_n(A) = sum_{k<=n} A^k / k!,   E_h = exp(-dtau/2 v0)
//
// Walker orbitals are rows (U^T, orbital-major), so the propagation multiplies
// the rows from the right: u' = u E_h T_n(A) E_h, using E_h^T = E_h and
// A^T = A (every L^g is symmetric).  Both MFMA operands are then contiguous
// along the contraction index.
#pragma once

#include "common.hpp"
#include "kernels_mfma.hpp"

// ---------------------------------------------------------------------------
// Block-packed storage of the FP32 exponent A_w (symmetric, one Re and one Im plane per
// walker): the 8 x 8 blocks (QB, PB), PB <= QB, of the lower block triangle, block row by
// block row, each block whole and row-major (a diagonal block holds both of its halves).
// A_w[q][p] for p in the upper block triangle is read as A_w[p][q].  Entries past M (the last
// block row and column when 8 does not divide M) hold zero.
// ---------------------------------------------------------------------------
__host__ __device__ inline int apk_size(int M) {
  const int nb = (M + 7) / 8;
  return 32 * nb * (nb + 1);   // 64 entries per block, nb (nb + 1) / 2 blocks
}
__host__ __device__ inline int apk_index(int q, int p) {
  int QB = q >> 3, PB = p >> 3, qi = q & 7, pi = p & 7;
  if (PB > QB) {
    const int t = QB, ti = qi;
    QB = PB, qi = pi;
    PB = t, pi = ti;
  }
  return 64 * (QB * (QB + 1) / 2 + PB) + 8 * qi + pi;
}
// The (q, p) of packed entry k (inverse of apk_index on the lower block triangle).
inline void apk_entry(int k, int& q, int& p) {
  const int blk = k >> 6, e = k & 63;
  int QB = 0;
  while ((QB + 1) * (QB + 2) / 2 <= blk) ++QB;
  const int PB = blk - QB * (QB + 1) / 2;
  q = 8 * QB + (e >> 3);
  p = 8 * PB + (e & 7);
}

// Workgroup tile of a gx x gy grid renumbered for the 8 XCDs (workgroups go to them
// round-robin by linear id, each XCD with an L2 of its own).  Where gx is even and 4 divides
// gy, XCD x takes the block of half the rows (x & 1) and a quarter of the columns (x >> 1),
// rows fastest: its share of the row operand stays small enough for its L2 while the column
// operand streams through once.  Otherwise each XCD takes a contiguous run of tiles in
// x-fastest order.
__device__ __forceinline__ int2 xcd_tile(int gx, int gy) {
  const int n = gx * gy, L = blockIdx.x + gx * blockIdx.y;
  const int x = L & 7, j = L >> 3;
  if ((gx & 1) == 0 && (gy & 3) == 0) {
    const int hx = gx >> 1, qy = gy >> 2;   // block of hx x qy tiles = n / 8
    return make_int2((x & 1) * hx + j % hx, (x >> 1) * qy + j / hx);
  }
  const int q = n >> 3, r = n & 7;
  const int t = x * q + (x < r ? x : r) + j;
  return make_int2(t % gx, t / gx);
}

// Four consecutive entries A[q][p0 .. p0 + 3] (p0 a multiple of 4, q < M) of a block-packed
// plane, zero past M: one 16-byte load inside the lower block triangle, four loads of a
// column of the block (p0, q) above it.
__device__ __forceinline__ f32x4 apk_load4(const float* __restrict__ Ap, int M, int q, int p0) {
  if ((p0 >> 3) <= (q >> 3)) return *reinterpret_cast<const f32x4*>(Ap + apk_index(q, p0));
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (p0 + e < M) v[e] = Ap[apk_index(q, p0 + e)];
  return v;
}

// ---------------------------------------------------------------------------
// A-build as a tiled MFMA GEMM:  C[r][col] = sum_k Y[r][k] Lt[col][k]
//   r = 2w + (0: Re y, 1: Im y),  col = block-packed entry of A (apk_index; MA = apk_size(M)
//   columns, about half of M^2 since A is symmetric),  k = g (padded to Gp, zeros).
//   Re A_w[col] = -s C[2w+1][col],  Im = s C[2w][col]: planar FP32 output of MA entries per
//   walker, each written once (a tile's columns are whole block rows: contiguous stores).
// Tile 128 rows x 16 CB columns per workgroup, two workgroups per CU; four wavefronts of
// 32 rows x 16 CB columns (2 x CB blocks of v_mfma_f32_16x16x4_f32); K chunks of 16
// double-buffered in LDS, Y rows first, then the Lt rows of the tile's columns.  The host
// picks CB (abuild_cb) so that the workgroups fill whole rounds of the device's slots: at
// M = 128 the 8704 packed columns make 32 tiles of 272 (CB = 17), and 1024 walkers 16 row
// tiles, 512 workgroups in all, one round on 256 CUs.  A lane holds four consecutive k of
// its row in each operand and MFMA e takes the e-th of them: a permutation of the k of the
// chunk, the same in both operands.
// ---------------------------------------------------------------------------
constexpr int AB_BM = 128, AB_BK = 16, AB_LD = AB_BK + 4;

template <int CB>
__global__ void __launch_bounds__(256, 2) k_abuild_f32(int rows /*2 nw*/, int MA, int Gp, float s,
                                                       const float* __restrict__ Y,
                                                       const float* __restrict__ Lt,
                                                       float* __restrict__ Are,
                                                       float* __restrict__ Aim) {
  constexpr int BN = 16 * CB, TR = AB_BM + BN;
  constexpr int NLD = TR * (AB_BK / 4);           // 16-byte pieces of one K chunk
  constexpr int PER = (NLD + 255) / 256;
  static_assert(2 * TR * AB_LD * 4 <= 65536, "tile exceeds the static LDS of a workgroup");
  __shared__ __attribute__((aligned(16))) float Ls[2][TR * AB_LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int2 tile = xcd_tile(gridDim.x, gridDim.y);
  const int r0 = tile.x * AB_BM, c0 = tile.y * BN;
  const int wr = wave * 32;
  const int col = lane & 15, kg = lane >> 4;
  // piece e of a chunk: tile row e / 4 (rows below AB_BM are Y rows, the rest Lt rows), k
  // offset 4 (e % 4); with 256 threads, pass c covers rows 64 c .. 64 c + 63, so the Y / Lt
  // choice is uniform per pass.  Rows past the walkers and columns past the packed triangle
  // re-read row / column 0: they only feed accumulator rows / columns that are never stored.
  f32x4 stg[PER];
  auto gload = [&](int k0) {
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      const int e = tid + c * 256;
      if ((c + 1) * 256 <= NLD || e < NLD) {
        const int rr = e >> 2, kk = (e & 3) * 4;
        const float* src;
        if (c * 64 + 63 < AB_BM) {
          const int gr = r0 + rr;
          src = Y + (size_t)(gr < rows ? gr : 0) * Gp;
        } else {
          const int gc = c0 + rr - AB_BM;
          src = Lt + (size_t)(gc < MA ? gc : 0) * Gp;
        }
        stg[c] = *reinterpret_cast<const f32x4*>(src + k0 + kk);
      }
    }
  };
  auto lstore = [&](float* dst) {
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      const int e = tid + c * 256;
      if ((c + 1) * 256 <= NLD || e < NLD)
        *reinterpret_cast<f32x4*>(dst + (e >> 2) * AB_LD + (e & 3) * 4) = stg[c];
    }
  };
  f32x4 acc[2][CB];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < CB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nk = Gp / AB_BK;
  gload(0);
  lstore(Ls[0]);
  __syncthreads();
  for (int kc = 0; kc < nk; ++kc) {
    const float* Lb = Ls[kc & 1];
    if (kc + 1 < nk) gload((kc + 1) * AB_BK);
    const f32x4 fa0 = *reinterpret_cast<const f32x4*>(Lb + (wr + col) * AB_LD + 4 * kg);
    const f32x4 fa1 = *reinterpret_cast<const f32x4*>(Lb + (wr + 16 + col) * AB_LD + 4 * kg);
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const f32x4 fb = *reinterpret_cast<const f32x4*>(Lb + (AB_BM + 16 * b + col) * AB_LD + 4 * kg);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[0][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa0[e], fb[e], acc[0][b], 0, 0, 0);
        acc[1][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa1[e], fb[e], acc[1][b], 0, 0, 0);
      }
    }
    if (kc + 1 < nk) lstore(Ls[(kc + 1) & 1]);
    __syncthreads();
  }
  // epilogue: lane holds column 16 b + col, rows 16 a + 4 kg + v of the wave's 32; v = 0, 1
  // are the Re and Im rows of one walker, v = 2, 3 of the next
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const int cc = c0 + 16 * b + col;
      if (cc >= MA) continue;
#pragma unroll
      for (int v = 0; v < 4; v += 2) {
        const int r = r0 + wr + 16 * a + 4 * kg + v;   // even
        if (r >= rows) continue;
        const size_t o = (size_t)(r >> 1) * MA + cc;
        Are[o] = -s * acc[a][b][v + 1];
        Aim[o] = s * acc[a][b][v];
      }
    }
}

// Column blocks of 16 per A-build tile, from those compiled (FN: the kernel of each, block
// threads, dynamic LDS): the least MFMA time, counted as (rounds of the device's workgroup
// slots) x (workgroups per CU) x CB, with the workgroups per CU of each instance from the
// runtime's occupancy (queried once per device); ties go to the wider tile.
constexpr int AB_CBS[] = {17, 16, 12, 8, 4};
constexpr int AB_NCB = sizeof(AB_CBS) / sizeof(AB_CBS[0]);
struct AbuildFn {
  const void* fn;
  int threads, lds;
};
inline int abuild_pick(const AbuildFn* fns, int (&per_cu)[64][AB_NCB], int rows, int MA) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  const long long cus = device_cu_count(), nrow = (rows + AB_BM - 1) / AB_BM;
  int best = AB_CBS[0];
  long long best_cost = -1;
  for (int i = 0; i < AB_NCB; ++i) {
    if (per_cu[dev][i] <= 0) {
      int n = 0;
      if (fns[i].lds > 0)
        (void)hipFuncSetAttribute(fns[i].fn, hipFuncAttributeMaxDynamicSharedMemorySize, fns[i].lds);
      per_cu[dev][i] = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                           &n, fns[i].fn, fns[i].threads, fns[i].lds) == hipSuccess && n > 0
                           ? n
                           : 1;
    }
    const long long cb = AB_CBS[i], n = per_cu[dev][i];
    const long long wgs = nrow * ((MA + 16 * cb - 1) / (16 * cb));
    const long long cost = (wgs + n * cus - 1) / (n * cus) * n * cb;
    if (best_cost < 0 || cost < best_cost) best = (int)cb, best_cost = cost;
  }
  return best;
}
inline int abuild_cb(int rows, int MA) {
  static int per_cu[64][AB_NCB] = {};
  static const AbuildFn fns[AB_NCB] = {
      {(const void*)k_abuild_f32<17>, 256, 0}, {(const void*)k_abuild_f32<16>, 256, 0},
      {(const void*)k_abuild_f32<12>, 256, 0}, {(const void*)k_abuild_f32<8>, 256, 0},
      {(const void*)k_abuild_f32<4>, 256, 0}};
  return abuild_pick(fns, per_cu, rows, MA);
}

// ---------------------------------------------------------------------------
// Fused propagation of one walker per workgroup: u' = u E_h T_n(A) E_h for all
// its orbitals u (rows).  One wavefront per 16 output columns q; the wave keeps
// its columns of A (Re, Im) and of E_h in registers as the MFMA B operand for
// the whole Taylor series, while the current term (rows c, FP32 Re/Im planes)
// lives in LDS as the A operand.  Sum Y of the series accumulates in registers.
// v_mfma_f32_16x16x4_f32; output lane layout: column j = lane % 16, rows 4*(lane/16) + v.
// Requirements: M <= 128, ntot <= 64.
// ---------------------------------------------------------------------------
constexpr int PR_RB = 4;  // row blocks of 16 (ntot <= 64)

// NKC = K_P / 16 wavefronts (K chunks of 16), NRB = ceil(ntot / 16) row blocks: both compile
// time, so the chunk loops carry no branches and the LDS reads can run ahead of the MFMAs.
template <int NKC, int NRB>
__global__ void __launch_bounds__(64 * NKC, 1) k_propagate_f32(
    int M, int ntot, int Kp_arg, int n_taylor, const float* __restrict__ Eh32 /*[M][M]*/,
    const float* __restrict__ Are, const float* __restrict__ Aim, cd* __restrict__ U,
    const double* __restrict__ weight) {
  extern __shared__ __attribute__((aligned(16))) float tsm[];
  const int w = blockIdx.x;
  if (!(weight[w] > 0.0)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int Kp = 16 * NKC;
  (void)Kp_arg;
  constexpr int ldt = Kp + 4;
  constexpr int RP = 16 * NRB;   // term rows held in LDS
  float* Tr = tsm;             // [RP][ldt]
  float* Ti = tsm + RP * ldt;  // [RP][ldt]
  const int j = lane & 15, q4 = lane >> 4;
  const int qcol = 16 * wave + j;  // output column owned by the lane
  const size_t MA = (size_t)apk_size(M);

  // load U rows (FP64 complex) into the term planes, zero padding: all loads of a thread go
  // out before the first store (padding positions read a valid element and store zero)
  const cd* Uw = U + (size_t)w * ntot * M;
  {
    constexpr int NT = 64 * NKC, NIT = RP * Kp / NT;   // = 4 NRB
    cd uv[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int e = tid + it * NT, c = e / Kp, p = e % Kp;
      uv[it] = Uw[(size_t)(c < ntot ? c : 0) * M + (p < M ? p : 0)];
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int e = tid + it * NT, c = e / Kp, p = e % Kp;
      const bool ok = c < ntot && p < M;
      Tr[c * ldt + p] = ok ? (float)uv[it].re : 0.f;
      Ti[c * ldt + p] = ok ? (float)uv[it].im : 0.f;
    }
  }
  // B operands: lane holds rows q = qcol, k = 16*kc + 4*q4 .. +3 (16-byte loads where the
  // four are inside the row and aligned)
  f32x4 be[NKC], bar_[NKC], bai[NKC], bas[NKC];
  const bool colok = qcol < M;
  auto load_eh = [&]() {
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      be[kc] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int p0 = 16 * kc + 4 * q4;
      if (colok) {
        if ((M & 3) == 0 && p0 + 4 <= M) {
          be[kc] = *reinterpret_cast<const f32x4*>(Eh32 + (size_t)qcol * M + p0);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (p0 + e < M) be[kc][e] = Eh32[(size_t)qcol * M + p0 + e];
        }
      }
    }
  };
  load_eh();
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc) {
    bar_[kc] = f32x4{0.f, 0.f, 0.f, 0.f};
    bai[kc] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int p0 = 16 * kc + 4 * q4;
    if (colok) {
      bar_[kc] = apk_load4(Are + (size_t)w * MA, M, qcol, p0);
      bai[kc] = apk_load4(Aim + (size_t)w * MA, M, qcol, p0);
    }
    bas[kc] = bar_[kc] + bai[kc];
  }
  __syncthreads();

  f32x4 yre[NRB], yim[NRB], cre[NRB], cim[NRB];
  // X = U E_h  (real B operand)
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    cre[rb] = f32x4{};
    cim[rb] = f32x4{};
  }
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      const f32x4 ar = *reinterpret_cast<const f32x4*>(&Tr[(16 * rb + j) * ldt + 16 * kc + 4 * q4]);
      const f32x4 ai = *reinterpret_cast<const f32x4*>(&Ti[(16 * rb + j) * ldt + 16 * kc + 4 * q4]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        cre[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[e], be[kc][e], cre[rb], 0, 0, 0);
        cim[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[e], be[kc][e], cim[rb], 0, 0, 0);
      }
    }
  }
  __syncthreads();
  // write X back as the first term, Y = X
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    yre[rb] = cre[rb];
    yim[rb] = cim[rb];
    if (qcol < Kp) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        Tr[(16 * rb + 4 * q4 + v) * ldt + qcol] = cre[rb][v];
        Ti[(16 * rb + 4 * q4 + v) * ldt + qcol] = cim[rb][v];
      }
    }
  }
  __syncthreads();
  // Taylor terms: T <- T A / n, Y += T.  The complex product takes three real ones,
  // P1 = Tr Ar, P2 = Ti Ai, P3 = (Tr + Ti)(Ar + Ai): Re = P1 - P2, Im = P3 - P1 - P2.
  for (int n = 1; n <= n_taylor; ++n) {
    f32x4 p1[NRB], p2[NRB], p3[NRB];
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        const f32x4 ar = *reinterpret_cast<const f32x4*>(&Tr[(16 * rb + j) * ldt + 16 * kc + 4 * q4]);
        const f32x4 ai = *reinterpret_cast<const f32x4*>(&Ti[(16 * rb + j) * ldt + 16 * kc + 4 * q4]);
        const f32x4 as = ar + ai;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool first = kc == 0 && e == 0;
          p1[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[e], bar_[kc][e], first ? f32x4{} : p1[rb], 0, 0, 0);
          p2[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[e], bai[kc][e], first ? f32x4{} : p2[rb], 0, 0, 0);
          p3[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(as[e], bas[kc][e], first ? f32x4{} : p3[rb], 0, 0, 0);
        }
      }
    }
    const float inv = 1.0f / (float)n;
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      cre[rb] = (p1[rb] - p2[rb]) * inv;
      cim[rb] = (p3[rb] - p1[rb] - p2[rb]) * inv;
      yre[rb] += cre[rb];
      yim[rb] += cim[rb];
      if (qcol < Kp) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          Tr[(16 * rb + 4 * q4 + v) * ldt + qcol] = cre[rb][v];
          Ti[(16 * rb + 4 * q4 + v) * ldt + qcol] = cim[rb][v];
        }
      }
    }
    __syncthreads();
  }
  // Y into the planes, then U' = Y E_h (E_h read again: the Taylor loop does not hold it)
  load_eh();
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    if (qcol < Kp) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        Tr[(16 * rb + 4 * q4 + v) * ldt + qcol] = yre[rb][v];
        Ti[(16 * rb + 4 * q4 + v) * ldt + qcol] = yim[rb][v];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    cre[rb] = f32x4{};
    cim[rb] = f32x4{};
  }
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      const f32x4 ar = *reinterpret_cast<const f32x4*>(&Tr[(16 * rb + j) * ldt + 16 * kc + 4 * q4]);
      const f32x4 ai = *reinterpret_cast<const f32x4*>(&Ti[(16 * rb + j) * ldt + 16 * kc + 4 * q4]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        cre[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[e], be[kc][e], cre[rb], 0, 0, 0);
        cim[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[e], be[kc][e], cim[rb], 0, 0, 0);
      }
    }
  }
  cd* Uo = U + (size_t)w * ntot * M;
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    if (!colok) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 16 * rb + 4 * q4 + v;
      if (c < ntot) Uo[(size_t)c * M + qcol] = mkc((double)cre[rb][v], (double)cim[rb][v]);
    }
  }
}

// ---------------------------------------------------------------------------
// Fused propagation for the wide shapes (M up to 224, up to 64 orbitals per spin):
// u' = u E_h T_n(A) E_h for the orbitals of one spin of one walker per workgroup
// (grid: walkers x 2 spins).  As in k_propagate_f32, one wavefront per 16 output
// columns q and the current term (rows c, FP32 Re/Im planes) in LDS as the A operand;
// the B operands (columns q of E_h and of A, read as rows since both are symmetric)
// are E_h's a 16-wide K chunk ahead from memory, and A's in registers for the whole series where
// they fit (prop_wide_reg: 8 NKC of the 512 / ceil(NKC / 4) VGPRs a wave has), else streamed too.
// NRB = ceil(max(N_up, N_dn) / 16) row blocks.  The products of a row block wait for each other,
// so those of RS row blocks alternate (two where the registers are short).  M = 143, N = 35+33,
// 701 walkers, six terms: 0.95 ms, 49 TFLOP/s; with A streamed in every term, four scattered
// loads above the diagonal: 1.50 ms.  M = 220, N = 60, 512 walkers (streamed): 2.51 against 2.83 ms
// without the compile-time row blocks.
// ---------------------------------------------------------------------------
constexpr bool prop_wide_reg(int nkc, int nrb) { return nkc <= 8 || (nkc <= 10 && nrb <= 3); }

template <int NKC, int NRB>
__global__ void __launch_bounds__(64 * NKC) k_propagate_f32_wide(
    int M, int nup, int ndn, int Kp, int n_taylor, const float* __restrict__ Eh32 /*[M][M]*/,
    const float* __restrict__ Are, const float* __restrict__ Aim, cd* __restrict__ U,
    const double* __restrict__ weight) {
  extern __shared__ __attribute__((aligned(16))) float tsm[];
  constexpr int RB = NRB;                       // row blocks of 16
  constexpr bool REG = prop_wide_reg(NKC, NRB);
  constexpr int RS = NKC <= 8 || (NKC <= 12 && RB <= 3) ? RB : 2;   // row blocks that alternate
  const int w = blockIdx.x, s = blockIdx.y;
  const int N = s ? ndn : nup, off = s ? nup : 0, ntot = nup + ndn;
  if (N == 0 || !(weight[w] > 0.0)) return;     // uniform over the workgroup
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ldt = Kp + 4;
  float* Tr = tsm;                  // [16 RB][ldt]
  float* Ti = tsm + 16 * RB * ldt;  // [16 RB][ldt]
  const int j = lane & 15, q4 = lane >> 4;
  const int qcol = 16 * wave + j;   // output column owned by the lane
  const bool colok = qcol < M;
  const size_t MA = (size_t)apk_size(M);
  const float* Eq = Eh32 + (size_t)(colok ? qcol : 0) * M;
  const float* Aw_re = Are + (size_t)w * MA;
  const float* Aw_im = Aim + (size_t)w * MA;
  // B operand of K chunk kc: rows p = 16 kc + 4 q4 + e of column qcol (zero beyond M), of
  // E_h (full) and of A (block-packed)
  auto lda4 = [&](const float* Ap, int kc) {
    return colok ? apk_load4(Ap, M, qcol, 16 * kc + 4 * q4) : f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto ld4 = [&](const float* row, int kc) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    const int p0 = 16 * kc + 4 * q4;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (colok && p0 + e < M) v[e] = row[p0 + e];
    return v;
  };

  const cd* Uw = U + ((size_t)w * ntot + off) * M;
  for (int e = tid; e < 16 * RB * Kp; e += blockDim.x) {
    const int c = e / Kp, p = e % Kp;
    cd v = mkc(0.0, 0.0);
    if (c < N && p < M) v = Uw[(size_t)c * M + p];
    Tr[c * ldt + p] = (float)v.re;
    Ti[c * ldt + p] = (float)v.im;
  }
  f32x4 bar_[REG ? NKC : 1], bai[REG ? NKC : 1];
  if constexpr (REG) {
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      bar_[kc] = lda4(Aw_re, kc);
      bai[kc] = lda4(Aw_im, kc);
    }
  }
  __syncthreads();

  f32x4 yre[RB], yim[RB], cre[RB], cim[RB];
  // real B (E_h): C = T E_h
  auto mul_real = [&](const float* Bq) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      cre[rb] = f32x4{};
      cim[rb] = f32x4{};
    }
    f32x4 b = ld4(Bq, 0);
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      const f32x4 bn = kc + 1 < NKC ? ld4(Bq, kc + 1) : b;
      f32x4 ar[RB], ai[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        ar[rb] = *reinterpret_cast<const f32x4*>(&Tr[(16 * rb + j) * ldt + 16 * kc + 4 * q4]);
        ai[rb] = *reinterpret_cast<const f32x4*>(&Ti[(16 * rb + j) * ldt + 16 * kc + 4 * q4]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          cre[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[rb][e], b[e], cre[rb], 0, 0, 0);
          cim[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[rb][e], b[e], cim[rb], 0, 0, 0);
        }
      b = bn;
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto store_planes = [&](const f32x4* pr, const f32x4* pi) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      if (qcol < Kp) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          Tr[(16 * rb + 4 * q4 + v) * ldt + qcol] = pr[rb][v];
          Ti[(16 * rb + 4 * q4 + v) * ldt + qcol] = pi[rb][v];
        }
      }
    }
  };

  // X = U E_h; the first term and Y = X
  mul_real(Eq);
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    yre[rb] = cre[rb];
    yim[rb] = cim[rb];
  }
  store_planes(cre, cim);
  __syncthreads();
  // Taylor terms: T <- T A / n, Y += T
  for (int n = 1; n <= n_taylor; ++n) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      cre[rb] = f32x4{};
      cim[rb] = f32x4{};
    }
    f32x4 br, bi;
    const float *are = Aw_re, *aim = Aw_im;
    if constexpr (!REG) {
      asm volatile("" : "+s"(are), "+s"(aim));   // opaque: not the whole of A ahead of the series
      br = lda4(are, 0);
      bi = lda4(aim, 0);
    }
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      f32x4 brn, bin;
      if constexpr (REG) {
        br = bar_[REG ? kc : 0];
        bi = bai[REG ? kc : 0];
      } else {
        brn = kc + 1 < NKC ? lda4(are, kc + 1) : br;
        bin = kc + 1 < NKC ? lda4(aim, kc + 1) : bi;
      }
#pragma unroll
      for (int r0 = 0; r0 < RB; r0 += RS) {
        f32x4 ar[RS], ai[RS], an[RS];
#pragma unroll
        for (int i = 0; i < RS; ++i) {
          const int at = (16 * (r0 + i < RB ? r0 + i : r0) + j) * ldt + 16 * kc + 4 * q4;
          ar[i] = *reinterpret_cast<const f32x4*>(&Tr[at]);
          ai[i] = *reinterpret_cast<const f32x4*>(&Ti[at]);
          an[i] = -ai[i];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int i = 0; i < RS; ++i) {
            if (r0 + i >= RB) continue;
            f32x4 &cr = cre[r0 + i < RB ? r0 + i : 0], &ci = cim[r0 + i < RB ? r0 + i : 0];
            cr = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[i][e], br[e], cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[i][e], bi[e], ci, 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < RS; ++i) {
            if (r0 + i >= RB) continue;
            f32x4 &cr = cre[r0 + i < RB ? r0 + i : 0], &ci = cim[r0 + i < RB ? r0 + i : 0];
            cr = __builtin_amdgcn_mfma_f32_16x16x4f32(an[i][e], bi[e], cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[i][e], br[e], ci, 0, 0, 0);
          }
        }
        if (RS < RB) __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (!REG) {
        br = brn;
        bi = bin;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    const float inv = 1.0f / (float)n;
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      cre[rb] *= inv;
      cim[rb] *= inv;
      yre[rb] += cre[rb];
      yim[rb] += cim[rb];
    }
    store_planes(cre, cim);
    __syncthreads();
  }
  // Y into the planes, then U' = Y E_h
  store_planes(yre, yim);
  __syncthreads();
  mul_real(Eq);
  cd* Uo = U + ((size_t)w * ntot + off) * M;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    if (!colok) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 16 * rb + 4 * q4 + v;
      if (c < N) Uo[(size_t)c * M + qcol] = mkc((double)cre[rb][v], (double)cim[rb][v]);
    }
  }
}

// ---------------------------------------------------------------------------
// FP64 A-build for M <= 128 on v_mfma_f64_16x16x4_f64: the GEMM of k_abuild_f32 (rows of Y,
// block-packed columns of A, planar output of MA doubles per walker and plane).  Tile 128 rows
// x 16 CB columns per workgroup of eight wavefronts, each 16 rows x 16 CB columns (CB blocks of
// accumulators, 136 VGPRs at CB = 17, so two wavefronts per SIMD), K chunks of 16
// double-buffered in LDS, 144-byte rows.  A lane takes two consecutive k of its row in both
// operands.  Each MFMA reads one B fragment: 32 B per clock and CU from LDS at the full rate.
// At M = 128, 1024 walkers: 512 tiles of 272 columns, two full rounds on 256 CUs, 0.50 ms, 57
// TFLOP/s (64 x 64 tiles with mirrored stores of the whole A: 0.64 ms; a library FP64 product
// of 4096^3 runs at 60 on this card).
// ---------------------------------------------------------------------------
constexpr int AB64_LDP = AB_BK + 2;
template <int CB>
constexpr int abuild_f64_lds() {
  return 2 * (AB_BM + 16 * CB) * AB64_LDP * 8;
}

template <int CB>
__global__ void __launch_bounds__(512, 2) k_abuild_f64(int rows /*2 nw*/, int MA, int Gp, double s,
                                                       const double* __restrict__ Y,
                                                       const double* __restrict__ Lt,
                                                       double* __restrict__ Are,
                                                       double* __restrict__ Aim) {
  constexpr int BN = 16 * CB, TR = AB_BM + BN, LD = AB64_LDP;
  constexpr int NLD = TR * (AB_BK / 2);           // 16-byte pieces of one K chunk
  constexpr int PER = (NLD + 511) / 512;
  extern __shared__ __attribute__((aligned(16))) double ab64_smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int2 tile = xcd_tile(gridDim.x, gridDim.y);
  const int r0 = tile.x * AB_BM, c0 = tile.y * BN;
  const int l16 = lane & 15, q = lane >> 4;
  // piece e of a chunk: tile row e / 8 (rows below AB_BM are Y rows, the rest Lt rows), k
  // offset 2 (e % 8); pass c covers rows 64 c .. 64 c + 63, so the Y / Lt choice is uniform.
  // Rows past the walkers and columns past the packed triangle re-read row / column 0: they
  // only feed accumulator rows / columns that are never stored.
  f64x2 stg[PER];
  auto gload = [&](int k0) {
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      const int e = tid + c * 512;
      if ((c + 1) * 512 <= NLD || e < NLD) {
        const int rr = e >> 3, kk = (e & 7) * 2;
        const double* src;
        if (c * 64 + 63 < AB_BM) {
          const int gr = r0 + rr;
          src = Y + (size_t)(gr < rows ? gr : 0) * Gp;
        } else {
          const int gc = c0 + rr - AB_BM;
          src = Lt + (size_t)(gc < MA ? gc : 0) * Gp;
        }
        stg[c] = *reinterpret_cast<const f64x2*>(src + k0 + kk);
      }
    }
  };
  auto lstore = [&](double* dst) {
#pragma unroll
    for (int c = 0; c < PER; ++c) {
      const int e = tid + c * 512;
      if ((c + 1) * 512 <= NLD || e < NLD)
        *reinterpret_cast<f64x2*>(dst + (e >> 3) * LD + (e & 7) * 2) = stg[c];
    }
  };
  f64x4 acc[CB];
#pragma unroll
  for (int b = 0; b < CB; ++b) acc[b] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int nk = Gp / AB_BK;
  gload(0);
  lstore(ab64_smem);
  __syncthreads();
  for (int kc = 0; kc < nk; ++kc) {
    const double* Lb = ab64_smem + (size_t)(kc & 1) * TR * LD;
    if (kc + 1 < nk) gload((kc + 1) * AB_BK);
    const double* A = Lb + (16 * wave + l16) * LD + 2 * q;
    const double* B = Lb + (AB_BM + l16) * LD + 2 * q;
#pragma unroll
    for (int kk = 0; kk < AB_BK; kk += 8) {
      const f64x2 fa = *reinterpret_cast<const f64x2*>(A + kk);
      // four column blocks at a time, so that an accumulator is used again four MFMAs later
#pragma unroll
      for (int b0 = 0; b0 < CB; b0 += 4) {
        f64x2 fb[4];
#pragma unroll
        for (int b = b0; b < b0 + 4 && b < CB; ++b)
          fb[b - b0] = *reinterpret_cast<const f64x2*>(B + 16 * b * LD + kk);
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int b = b0; b < b0 + 4 && b < CB; ++b)
            acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[e], fb[b - b0][e], acc[b], 0, 0, 0);
      }
    }
    if (kc + 1 < nk) lstore(ab64_smem + (size_t)((kc + 1) & 1) * TR * LD);
    __syncthreads();
  }
  // lane: column 16 b + l16, rows q + 4 v of the wavefront's 16; even rows are Re y (the Im
  // part of A), odd rows Im y
  double* out = q & 1 ? Are : Aim;
  const double f = q & 1 ? -s : s;
#pragma unroll
  for (int b = 0; b < CB; ++b) {
    const int cc = c0 + 16 * b + l16;
    if (cc >= MA) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = r0 + 16 * wave + q + 4 * v;
      if (r < rows) out[(size_t)(r >> 1) * MA + cc] = f * acc[b][v];
    }
  }
}

inline int abuild_f64_cb(int rows, int MA) {
  static int per_cu[64][AB_NCB] = {};
  static const AbuildFn fns[AB_NCB] = {
      {(const void*)k_abuild_f64<17>, 512, abuild_f64_lds<17>()},
      {(const void*)k_abuild_f64<16>, 512, abuild_f64_lds<16>()},
      {(const void*)k_abuild_f64<12>, 512, abuild_f64_lds<12>()},
      {(const void*)k_abuild_f64<8>, 512, abuild_f64_lds<8>()},
      {(const void*)k_abuild_f64<4>, 512, abuild_f64_lds<4>()}};
  return abuild_pick(fns, per_cu, rows, MA);
}

// Four consecutive entries A[q][p0 .. p0 + 3] of a block-packed FP64 plane (as apk_load4).
__device__ __forceinline__ void apk_load4(const double* __restrict__ Ap, int M, int q, int p0,
                                          double (&v)[4]) {
  if ((p0 >> 3) <= (q >> 3)) {
    const double* a = Ap + apk_index(q, p0);
    const f64x2 x = *reinterpret_cast<const f64x2*>(a), y = *reinterpret_cast<const f64x2*>(a + 2);
    v[0] = x[0], v[1] = x[1], v[2] = y[0], v[3] = y[1];
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = p0 + e < M ? Ap[apk_index(q, p0 + e)] : 0.0;
}

// ---------------------------------------------------------------------------
// FP64 propagation for M <= 128: u' = u E_h T_n(A) E_h on v_mfma_f64_16x16x4_f64 with A_w in
// registers.  One wavefront per 16 output columns q; a wavefront's columns of A (Re and Im, 16
// NKC VGPRs each half: 128 at M = 128) stay in registers for every row block of the walker and
// every Taylor term, so A is read once per walker (k_propagate_f64 below streams it for each
// term, row block and spin).  The current term, 16 NRB rows, is in LDS as the A operand.  The
// complex product T A takes three real ones.  Job: 16 NRB rows of one spin; workgroup (w, y) of the
// grid takes jobs y, y + gridDim.y, ... of walker w.  Operand lanes and output layout as in
// k_propagate_f64.  Bound by the FP64 matrix cores (about 57 TFLOP/s on real data): M = 128,
// N = 32 + 32, 1024 walkers 0.91 ms (four products and A streamed: 1.28; four products with A in
// registers: 1.05).
// ---------------------------------------------------------------------------
template <int NKC, int NRB>
__global__ void __launch_bounds__(64 * NKC, 2) k_propagate_f64r(
    int M, int nup, int ndn, int n_taylor, const double* __restrict__ Eh /*[M][M]*/,
    const double* __restrict__ Are, const double* __restrict__ Aim, cd* __restrict__ U,
    const double* __restrict__ weight) {
  extern __shared__ __attribute__((aligned(16))) double dsm[];
  constexpr int Kp = 16 * NKC, ldt = Kp + 2, RP = 16 * NRB;
  const int w = blockIdx.x;
  if (!(weight[w] > 0.0)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* Tr = dsm;                 // [RP][ldt]
  double* Ti = dsm + RP * ldt;      // [RP][ldt]
  const int j = lane & 15, q4 = lane >> 4;
  const int qcol = 16 * wave + j;
  const bool colok = qcol < M;
  const size_t MA = (size_t)apk_size(M);
  const double* Ehq = Eh + (size_t)(colok ? qcol : 0) * M;
  double ar[NKC][4], ai[NKC][4];
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc) {
#pragma unroll
    for (int e = 0; e < 4; ++e) ar[kc][e] = ai[kc][e] = 0.0;
    if (colok && n_taylor > 0) {
      apk_load4(Are + (size_t)w * MA, M, qcol, 16 * kc + 4 * q4, ar[kc]);
      apk_load4(Aim + (size_t)w * MA, M, qcol, 16 * kc + 4 * q4, ai[kc]);
    }
  }
  const int jup = (nup + RP - 1) / RP, jobs = jup + (ndn + RP - 1) / RP;
  for (int job = blockIdx.y; job < jobs; job += gridDim.y) {
    const int s = job >= jup ? 1 : 0, rblk = job - (s ? jup : 0);
    const int off = (s ? nup : 0) + RP * rblk, nrows = min(RP, (s ? ndn : nup) - RP * rblk);
    cd* Uw = U + ((size_t)w * (nup + ndn) + off) * M;
    {
      constexpr int NIT = RP * Kp / (64 * NKC);   // = 4 NRB
      cd uv[NIT];
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int e = tid + it * 64 * NKC, c = e / Kp, p = e % Kp;
        uv[it] = Uw[(size_t)(c < nrows ? c : 0) * M + (p < M ? p : 0)];
      }
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int e = tid + it * 64 * NKC, c = e / Kp, p = e % Kp;
        const bool ok = c < nrows && p < M;
        Tr[c * ldt + p] = ok ? uv[it].re : 0.0;
        Ti[c * ldt + p] = ok ? uv[it].im : 0.0;
      }
    }
    __syncthreads();
    f64x4 yre[NRB], yim[NRB], cre[NRB], cim[NRB];
    auto mul_real = [&]() {   // C = T E_h, E_h streamed (shared by all walkers)
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) cre[rb] = cim[rb] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) {
        double b[4];
        const int p0 = 16 * kc + 4 * q4;
#pragma unroll
        for (int e = 0; e < 4; ++e) b[e] = (colok && p0 + e < M) ? Ehq[p0 + e] : 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb) {
            cre[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(Tr[(16 * rb + j) * ldt + p0 + e], b[e], cre[rb], 0, 0, 0);
            cim[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(Ti[(16 * rb + j) * ldt + p0 + e], b[e], cim[rb], 0, 0, 0);
          }
      }
    };
    auto store_planes = [&](const f64x4* pr, const f64x4* pi) {
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          Tr[(16 * rb + q4 + 4 * v) * ldt + qcol] = pr[rb][v];
          Ti[(16 * rb + q4 + 4 * v) * ldt + qcol] = pi[rb][v];
        }
    };
    mul_real();   // X = U E_h: the first term and Y = X
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      yre[rb] = cre[rb];
      yim[rb] = cim[rb];
    }
    store_planes(cre, cim);
    __syncthreads();
    for (int n = 1; n <= n_taylor; ++n) {
      // P1 = Tr Ar, P2 = Ti Ai, P3 = (Tr + Ti)(Ar + Ai): Re = P1 - P2, Im = P3 - P1 - P2
      f64x4 p3[NRB];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) cre[rb] = cim[rb] = p3[rb] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) {
        const int p0 = 16 * kc + 4 * q4;
        // Ar + Ai is formed again for every term: held across the loop it would take 64 more
        // registers (the opaque use of Ar keeps the compiler from hoisting it)
        double as[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          asm volatile("" : "+v"(ar[kc][e]));
          as[e] = ar[kc][e] + ai[kc][e];
        }
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
          const f64x2* tr = reinterpret_cast<const f64x2*>(&Tr[(16 * rb + j) * ldt + p0]);
          const f64x2* ti = reinterpret_cast<const f64x2*>(&Ti[(16 * rb + j) * ldt + p0]);
          const f64x2 t0 = tr[0], t1 = tr[1], u0 = ti[0], u1 = ti[1];
          const f64x2 w0 = t0 + u0, w1 = t1 + u1;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            cre[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(e < 2 ? t0[e & 1] : t1[e & 1], ar[kc][e], cre[rb], 0, 0, 0);
            cim[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(e < 2 ? u0[e & 1] : u1[e & 1], ai[kc][e], cim[rb], 0, 0, 0);
            p3[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(e < 2 ? w0[e & 1] : w1[e & 1], as[e], p3[rb], 0, 0, 0);
          }
        }
      }
      const double inv = 1.0 / (double)n;
      __syncthreads();
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        p3[rb] = (p3[rb] - cre[rb] - cim[rb]) * inv;
        cre[rb] = (cre[rb] - cim[rb]) * inv;
        cim[rb] = p3[rb];
        yre[rb] += cre[rb];
        yim[rb] += cim[rb];
      }
      store_planes(cre, cim);
      __syncthreads();
    }
    store_planes(yre, yim);   // U' = Y E_h
    __syncthreads();
    mul_real();
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = 16 * rb + q4 + 4 * v;
        if (colok && c < nrows) Uw[(size_t)c * M + qcol] = mkc(cre[rb][v], cim[rb][v]);
      }
    __syncthreads();   // the next job's rows overwrite the planes
  }
}

// ---------------------------------------------------------------------------
// FP64 A-build on v_mfma_f64_16x16x4_f64, lower triangle only (A_w is symmetric):
//   C[r][col] = sum_g Y[r][g] Lt[col][g],  r = 2w + (0: Re y, 1: Im y) read straight from the
//   interleaved complex y [nw][G],  col = packed pair p <= q,  Lt FP64 [MMh][Gp] (zero beyond G).
//   A_w[q][p] = A_w[p][q] = (-s C[2w+1][col], s C[2w][col])  (complex128 [nw][M][M]).
// Tile 64 x 64 per workgroup, K chunks of 16 double-buffered in LDS, 4 waves of 32 x 32
// (2 x 2 blocks).  Operand lanes: A[i][k] at lane i + 16k, B[k][j] at lane j + 16k;
// output lane l, item v holds D[l/16 + 4v][l%16], so rows 2w and 2w + 1 of a walker sit in
// lanes l and l + 16 (same v) and meet through one shuffle.
// ---------------------------------------------------------------------------
constexpr int AB64_B = 64, AB64_K = 16, AB64_LD = AB64_K + 2;

__global__ void __launch_bounds__(256) k_abuild_f64mfma(int nw, int G, int MMh, int MA, int Gp,
                                                        double s, const double* __restrict__ y,
                                                        const double* __restrict__ Lt,
                                                        const int2* __restrict__ pairs,
                                                        cd* __restrict__ A) {
  __shared__ __attribute__((aligned(16))) double As[2][AB64_B * AB64_LD];
  __shared__ __attribute__((aligned(16))) double Bs[2][AB64_B * AB64_LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rows = 2 * nw;
  const int r0 = blockIdx.x * AB64_B, c0 = blockIdx.y * AB64_B;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  const int l16 = lane & 15, q = lane >> 4;
  // each thread moves 4 doubles of A and 4 of B per K chunk: element e = tid + 256 i
  double pa[4], pb[4];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + 256 * i;
      const int rr = e >> 4, kk = e & 15;
      const int r = r0 + rr, c = c0 + rr, g = k0 + kk;
      pa[i] = (r < rows && g < G) ? y[((size_t)(r >> 1) * G + g) * 2 + (r & 1)] : 0.0;
      pb[i] = (c < MMh && g < Gp) ? Lt[(size_t)c * Gp + g] : 0.0;
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + 256 * i;
      const int rr = e >> 4, kk = e & 15;
      As[buf][rr * AB64_LD + kk] = pa[i];
      Bs[buf][rr * AB64_LD + kk] = pb[i];
    }
  };
  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int nk = (G + AB64_K - 1) / AB64_K;
  gload(0);
  lstore(0);
  __syncthreads();
  for (int kc = 0; kc < nk; ++kc) {
    const int buf = kc & 1;
    if (kc + 1 < nk) gload((kc + 1) * AB64_K);
#pragma unroll
    for (int ks = 0; ks < AB64_K / 4; ++ks) {
      double fa[2], fb[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) fa[a] = As[buf][(wr + 16 * a + l16) * AB64_LD + 4 * ks + q];
#pragma unroll
      for (int b = 0; b < 2; ++b) fb[b] = Bs[buf][(wc + 16 * b + l16) * AB64_LD + 4 * ks + q];
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
    if (kc + 1 < nk) lstore(buf ^ 1);
    __syncthreads();
  }
  // epilogue: lane (q even) holds row 2w's value, lane + 16 row 2w + 1's
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int cc = c0 + wc + 16 * b + l16;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double mine = acc[a][b][v];
        const double odd = __shfl_down(mine, 16, 64);
        const int r = r0 + wr + 16 * a + q + 4 * v;   // even for even q
        if ((q & 1) || cc >= MMh || r >= rows) continue;
        const int2 pq = pairs[cc];
        const int w = r >> 1;
        const cd val = mkc(-s * odd, s * mine);
        A[(size_t)w * MA + pq.x] = val;
        if (pq.y != pq.x) A[(size_t)w * MA + pq.y] = val;
      }
    }
}

// ---------------------------------------------------------------------------
// FP64 propagation on v_mfma_f64_16x16x4_f64: u' = u E_h T_n(A) E_h for up to 32 orbitals
// (one row block) of one spin of one walker per workgroup (grid: walkers x 2 spins x row
// blocks), one wavefront per 16 output columns q.  The current term (Re / Im planes) sits
// in LDS as the A operand; the B operands (rows q of the symmetric A_w, complex128, and of
// E_h) are streamed per 16-wide K chunk.  Inside a chunk lane group q4 = lane / 16 takes
// k = 16 kc + 4 q4 + e for its four MFMAs e, on both operands, so each lane's operands are
// contiguous (the sum over k is unchanged).  Output lane l, item v: row l/16 + 4v, column l%16.
// ---------------------------------------------------------------------------
template <int NKC>
__global__ void __launch_bounds__(64 * NKC) k_propagate_f64(
    int M, int nup, int ndn, int Kp, int n_taylor, const double* __restrict__ Eh /*[M][M]*/,
    const cd* __restrict__ A /*[nw][M][M]*/, cd* __restrict__ U,
    const double* __restrict__ weight) {
  extern __shared__ __attribute__((aligned(16))) double dsm[];
  constexpr int RB = 2;                          // 16-row blocks per workgroup (32 rows)
  const int w = blockIdx.x, s = blockIdx.y, rblk = blockIdx.z;
  const int N = s ? ndn : nup, off = (s ? nup : 0) + 32 * rblk, ntot = nup + ndn;
  const int nrows = min(32, N - 32 * rblk);
  if (nrows <= 0 || !(weight[w] > 0.0)) return;  // uniform over the workgroup
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ldt = Kp + 2;
  double* Tr = dsm;                 // [32][ldt]
  double* Ti = dsm + 32 * ldt;      // [32][ldt]
  const int j = lane & 15, q4 = lane >> 4;
  const int qcol = 16 * wave + j;
  const bool colok = qcol < M;
  const size_t MM = (size_t)M * M;
  const int nrb = (nrows + 15) / 16;
  const double* Ehq = Eh + (size_t)(colok ? qcol : 0) * M;
  const cd* Aq = A + (size_t)w * MM + (size_t)(colok ? qcol : 0) * M;

  const cd* Uw = U + ((size_t)w * ntot + off) * M;
  for (int e = tid; e < 32 * Kp; e += blockDim.x) {
    const int c = e / Kp, p = e % Kp;
    cd v = mkc(0.0, 0.0);
    if (c < nrows && p < M) v = Uw[(size_t)c * M + p];
    Tr[c * ldt + p] = v.re;
    Ti[c * ldt + p] = v.im;
  }
  __syncthreads();

  f64x4 yre[RB], yim[RB], cre[RB], cim[RB];
  auto zero = [&](f64x4* a) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) a[rb] = f64x4{0.0, 0.0, 0.0, 0.0};
  };
  // real B (E_h): C = T E_h
  auto mul_real = [&]() {
    zero(cre);
    zero(cim);
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      double b[4];
      const int p0 = 16 * kc + 4 * q4;
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = (colok && p0 + e < M) ? Ehq[p0 + e] : 0.0;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        if (rb >= nrb) break;
        const double* tr = &Tr[(16 * rb + j) * ldt + p0];
        const double* ti = &Ti[(16 * rb + j) * ldt + p0];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          cre[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(tr[e], b[e], cre[rb], 0, 0, 0);
          cim[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ti[e], b[e], cim[rb], 0, 0, 0);
        }
      }
    }
  };
  auto store_planes = [&](const f64x4* pr, const f64x4* pi) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      if (rb < nrb && qcol < Kp) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          Tr[(16 * rb + q4 + 4 * v) * ldt + qcol] = pr[rb][v];
          Ti[(16 * rb + q4 + 4 * v) * ldt + qcol] = pi[rb][v];
        }
      }
    }
  };

  mul_real();   // X = U E_h: the first term and Y = X
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    yre[rb] = cre[rb];
    yim[rb] = cim[rb];
  }
  store_planes(cre, cim);
  __syncthreads();
  for (int n = 1; n <= n_taylor; ++n) {
    zero(cre);
    zero(cim);
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      double br[4], bi[4];
      const int p0 = 16 * kc + 4 * q4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const cd a = (colok && p0 + e < M) ? Aq[p0 + e] : mkc(0.0, 0.0);
        br[e] = a.re;
        bi[e] = a.im;
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        if (rb >= nrb) break;
        const double* tr = &Tr[(16 * rb + j) * ldt + p0];
        const double* ti = &Ti[(16 * rb + j) * ldt + p0];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          cre[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(tr[e], br[e], cre[rb], 0, 0, 0);
          cre[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ti[e], bi[e], cre[rb], 0, 0, 0);
          cim[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(tr[e], bi[e], cim[rb], 0, 0, 0);
          cim[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ti[e], br[e], cim[rb], 0, 0, 0);
        }
      }
    }
    const double inv = 1.0 / (double)n;
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      cre[rb] *= inv;
      cim[rb] *= inv;
      yre[rb] += cre[rb];
      yim[rb] += cim[rb];
    }
    store_planes(cre, cim);
    __syncthreads();
  }
  store_planes(yre, yim);   // U' = Y E_h
  __syncthreads();
  mul_real();
  cd* Uo = U + ((size_t)w * ntot + off) * M;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    if (rb >= nrb || !colok) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 16 * rb + q4 + 4 * v;
      if (c < nrows) Uo[(size_t)c * M + qcol] = mkc(cre[rb][v], cim[rb][v]);
    }
  }
}
