// Shared-row form of the FP32 MFMA local-energy contraction (arXiv:1711.02242, Sec. III.D.3,
// eq:localenergy3; force-bias traces of eq:precomputing2), in the place of the wide, the flattened
// and the stacked-row kernels.
//
// Those kernels give a workgroup one walker-spin and every wavefront its own copy of the rows of
// Lh^g from the caches.  Two or three wavefronts per SIMD were all that the registers for two
// column sets and the row prefetch left, and the matrix cores were busy 54 - 60 % of the time.
// Here
//   columns   wavefront cb of a walker holds 16 columns of [Re Theta | Im Theta] (2N of them
//             padded to 16, not 2 N_P), all K, in registers: 4 NK registers instead of 8 NK;
//   rows      q consecutive blocks Lh^g stacked into RT row tiles of 16 (the padding of N is paid
//             once per group), 32 k a step in LDS for the W walkers of the workgroup, two buffers:
//             the wavefronts fetch step n + 2 into registers and store step n + 1 while all of
//             them multiply step n; a fragment is read in lane order;
//   Omega'    of each walker as [Re | Im] columns in LDS;
//   exchange  tr(Omega Omega) = sum_i Omega_ii^2 + 2 sum_(i < j) Omega_ij Omega_ji: a lane takes
//             row j of a block and the partners i = j + d (mod N) of a range of d, so every pair
//             is read once.
// One workgroup of 12 to 16 wavefronts per CU, so that the four SIMDs get the same number (ten
// wavefronts: three on two of them, and a second workgroup does not fit beside).  The exchange
// sums of a group run in the first step of the next one, after the first set of its products: the
// matrix core has another wavefront's products meanwhile, and the barriers of the later steps (there
// is at least one) come between these reads of Omega' and the stores of the next.
//
// Each element of Omega, and each trace, is the same chain of v_mfma_f32_16x16x4_f32 over k (and sum
// over lanes) as in those kernels; the FP32 terms of the exchange are grouped otherwise.
// M = 143, N = 35+33, N_g = 859, 701 walkers: 14.4 -> 9.1 ms (matrix cores 73 % busy; of the rest
// 6 % each are the 15 wavefronts of 16 slots, the exchange, the row fetch and the barriers).
#pragma once

constexpr int SHARE_MAX_WAVES = 16;
constexpr int SHARE_MAX_RT = 7;
constexpr int SHARE_MIN_NK = 3, SHARE_MAX_NK = 14;   // at least two steps per group
constexpr size_t SHARE_LDS_CAP = 163840;

// Column length of Omega' in LDS: 16-byte stores, and LDR + 1 odd for the reads along a diagonal.
__host__ __device__ constexpr int share_ldr(int RT) { return 16 * RT + 4; }
inline size_t share_lds_bytes(int W, int NWV, int RT, int nmax) {
  return (size_t)4 * RT * 1024 + (size_t)2 * W * NWV * 8 +
         (size_t)W * 2 * nmax * share_ldr(RT) * 4;
}

template <int NK, int RT>
__global__ void __launch_bounds__(64 * SHARE_MAX_WAVES, 4) k_contract_share(
    int nw, int G, int nup, int ndn, int NP, int KP, int qup, int qdn, int NWV,
    const float* __restrict__ Lp, const float* __restrict__ thp,
    const double* __restrict__ weight, cd* __restrict__ tpart, cd* __restrict__ exch,
    ContractSel sel) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int LDR = share_ldr(RT);
  const int s = blockIdx.y & 1, dd = blockIdx.y >> 1, n_det = gridDim.y >> 1;
  const int N = s ? ndn : nup;
  const int q = s ? qdn : qup;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nwaves = blockDim.x >> 6, W = nwaves / NWV;
  const int slot = wave / NWV, cb = wave - slot * NWV;   // walker of the workgroup, column block
  const int w0 = blockIdx.x * W;
  if (N == 0) {
    contract_empty_spin(N, w0 + slot, cb == 0 ? nw : 0, n_det, dd, s, G, lane, tpart, exch, sel);
    return;
  }
  if (sel.none_left(w0, s)) return;
  auto taken = [&](int i) {   // the walker of a slot, -1: none, lost, or left to the guard
    const int w = sel.walker(i, s, nw);
    return w >= 0 && weight[w] > 0.0 && sel.takes(w * n_det + dd, s) ? w : -1;
  };
  bool any = false;
  for (int i = w0; i < w0 + W; ++i) any = any || taken(i) >= 0;
  if (!any) return;
  const int w = taken(w0 + slot);
  const bool live = w >= 0;
  const int wd = (live ? w : 0) * n_det + dd;

  float* const As = reinterpret_cast<float*>(smem);                 // [2][2 RT][64 lanes][4]
  double* const red = reinterpret_cast<double*>(As + 4 * RT * 256);   // [2][nwaves]
  float* const ep =
      reinterpret_cast<float*>(red + 2 * nwaves) + (size_t)slot * 2 * max(nup, ndn) * LDR;

  const size_t per = (size_t)NP * KP;
  const float* const Lbase = Lp + ((size_t)dd * 2 + s) * G * per;
  const int col = lane & 15, kg = lane >> 4;
  const int cc = 16 * cb + col;          // column of [Re Theta | Im Theta] held by the lane
  const bool col_ok = live && cc < 2 * N;
  const bool im_col = cc >= N;
  const int j = im_col ? cc - N : cc;

  f32x4 b[NK];
  {
    const float* tb = thp + ((size_t)wd * 2 + s) * 2 * per + (im_col ? per : 0) +
                      (size_t)(col_ok ? j : 0) * KP + 4 * kg;
#pragma unroll
    for (int c = 0; c < NK; ++c)
      b[c] = col_ok ? *reinterpret_cast<const f32x4*>(tb + 16 * c) : f32x4{0.f, 0.f, 0.f, 0.f};
  }

  const int ngroups = (G + q - 1) / q;
  const GRange kr = sel.range(ngroups);   // whole groups
  // This wavefront fetches the fragments (row tile, 16 k of the step) wave and wave + nwaves; per
  // lane its row and k; rows past a group's end read its first row.
  constexpr int NS = (NK + 1) / 2;
  uint32_t ro[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int x = wave + f * nwaves, rho = 16 * (x % RT) + col, gl = rho / N;
    ro[f] = (uint32_t)(gl * per + (size_t)(rho - gl * N) * KP + 4 * kg);
  }
  const int half0 = wave / RT;   // 16-k half of the first fragment, of the second: 1
  const bool has0 = wave < 2 * RT, has1 = wave + nwaves < 2 * RT;
  float* const my = As + wave * 256 + lane * 4;   // this lane's place in the first buffer
  f32x4 stg0 = {0.f, 0.f, 0.f, 0.f}, stg1 = {0.f, 0.f, 0.f, 0.f};
  auto fetch = [&](const float* gb, uint32_t lim, int st) {
    gb += 32 * st;
    if (has0)
      stg0 = *reinterpret_cast<const f32x4*>(gb + (ro[0] < lim ? ro[0] : (uint32_t)(4 * kg)) +
                                             16 * half0);
    if (has1)
      stg1 = *reinterpret_cast<const f32x4*>(gb + (ro[1] < lim ? ro[1] : (uint32_t)(4 * kg)) + 16);
  };
  auto glim = [&](int k) { return (uint32_t)(min(q, G - k * q) * per); };
  auto store = [&](int buf) {
    if (has0) *reinterpret_cast<f32x4*>(my + buf) = stg0;
    if (has1) *reinterpret_cast<f32x4*>(my + buf + nwaves * 256) = stg1;
  };

  double xr = 0.0, xi = 0.0;
  const float* const ei = ep + N * LDR;              // the Im columns
  const uint32_t invN = 65536u / (uint32_t)N + 1u;   // u / N = u invN >> 16 for u < 112
  // Pairs: lane (row u = gl N + j of the group, part p of np of the distances d = 1 .. N / 2).
  const int rows = q * N, np = max(1, 64 * NWV / rows), nd = ((N >> 1) + np - 1) / np;
  auto exchange = [&](int k) {
    const int qk = min(q, G - k * q);
    int ln = lane;   // opaque: addresses kept from group to group would take registers
    asm volatile("" : "+v"(ln));
    for (int t = 64 * cb + ln; t < rows * np; t += 64 * NWV) {
      int p = 0, u = t;
      while (u >= rows) {
        u -= rows;
        ++p;
      }
      const int gl = (int)((u * invN) >> 16), jj = u - gl * N;
      if (gl >= qk) continue;
      const float* const oth = ep + jj * LDR + gl * N;   // Omega_ij, i = 0 .. N - 1
      const float* const own = ep + u;                   // Omega_ji, column i
      float pr = 0.f, pi = 0.f;
      if (p == 0) {
        const float R = oth[jj], I = oth[N * LDR + jj];
        pr = 0.5f * (R * R - I * I);
        pi = R * I;
      }
      int i = jj + p * nd, n = min(nd, (N >> 1) - p * nd);
      if (i >= N) i -= N;
      // an even N: the pairs at d = N / 2 once
      if (!(N & 1) && p * nd + n == (N >> 1) && 2 * jj >= N) --n;
#pragma unroll 2
      for (int d = 0; d < n; ++d) {
        i = i + 1 == N ? 0 : i + 1;
        exch_term(own[i * LDR], own[(N + i) * LDR], oth[i], oth[N * LDR + i], pr, pi);
      }
      xr += 2.0 * (double)pr;
      xi += 2.0 * (double)pi;
    }
    for (int gl = cb; gl < qk; gl += NWV) {
      float dr = 0.f, di = 0.f;
      if (lane < N) {
        dr = ep[lane * LDR + gl * N + lane];
        di = ei[lane * LDR + gl * N + lane];
      }
      dr = dpp_wave_sum(dr);
      di = dpp_wave_sum(di);
      if (lane == 0)
        tpart[((size_t)wd * 2 + s) * G + k * q + gl] = mkc((double)dr, (double)di);
    }
  };

  int cur = 0;   // buffer of the step at hand, in floats
  if (kr.b < kr.e) {
    fetch(Lbase + (size_t)kr.b * q * per, glim(kr.b), 0);
    store(0);
    fetch(Lbase + (size_t)kr.b * q * per, glim(kr.b), 1);
  }
  for (int k = kr.b; k < kr.e; ++k) {
    const int kn = k + 1 < kr.e ? k + 1 : k;
    const float* const gb = Lbase + (size_t)k * q * per;
    const float* const gn = Lbase + (size_t)kn * q * per;
    const uint32_t lim = glim(k), limn = glim(kn);
    f32x4 acc[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      __syncthreads();   // this step's rows are stored, the other buffer's are used up
      // sets of up to GT row tiles (a tile's products wait for each other), the halves of k
      // outside; the fragments of the next set read ahead
      constexpr int NG = RT > 5 || NK > 10 ? (RT + 1) / 2 - (RT == 7) : (RT + 2) / 3, GT = (RT + NG - 1) / NG;
      const int U = (2 * st + 1 < NK ? 2 : 1) * NG;
      const f32x4* const a_s = reinterpret_cast<const f32x4*>(As + cur) + lane;
      f32x4 an[GT];
      auto frags = [&](int u) {
#pragma unroll
        for (int i = 0; i < GT; ++i) {
          const int r = RT * (u % NG) / NG + i;
          if (r < RT * (u % NG + 1) / NG) an[i] = a_s[64 * (RT * (u / NG) + r)];
        }
      };
      if (live) frags(0);
      __builtin_amdgcn_sched_barrier(0);
      store(4 * RT * 128 - cur);
      if (st + 2 < NS) fetch(gb, lim, st + 2);
      else fetch(gn, limn, st + 2 - NS);
      __builtin_amdgcn_sched_barrier(0);
      if (live) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          f32x4 a[GT];
#pragma unroll
          for (int i = 0; i < GT; ++i) a[i] = an[i];
          if (u + 1 < U) frags(u + 1);
          __builtin_amdgcn_sched_barrier(0);
          const f32x4 bb = b[2 * st + u / NG];
#pragma unroll
          for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int i = 0; i < GT; ++i) {
              const int r = RT * (u % NG) / NG + i;
              if (r < RT * (u % NG + 1) / NG)
                acc[r < RT ? r : 0] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    a[i][m], bb[m], acc[r < RT ? r : 0], 0, 0, 0);
            }
          __builtin_amdgcn_sched_barrier(0);
          if (st == 0 && u == 0) {
            if (k > kr.b) exchange(k - 1);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      cur = 4 * RT * 128 - cur;
    }
    // lane holds Omega'[16 r + 4 kg + v][cc]; the last group's was read before this step's barrier
    if (col_ok) {
#pragma unroll
      for (int r = 0; r < RT; ++r) *reinterpret_cast<f32x4*>(ep + cc * LDR + 16 * r + 4 * kg) = acc[r];
    }
  }
  __syncthreads();
  if (live && kr.b < kr.e) exchange(kr.e - 1);

  xr = wave_sum(xr);
  xi = wave_sum(xi);
  if (lane == 0) {
    red[wave] = xr;
    red[nwaves + wave] = xi;
  }
  __syncthreads();
  if (live && cb == 0 && lane == 0) {
    double sr = 0.0, si = 0.0;
    for (int i = 0; i < NWV; ++i) {
      sr += red[wave + i];
      si += red[nwaves + wave + i];
    }
    exch[sel.part() + 2 * (size_t)wd + s] = mkc(sr, si);
  }
}

// Launch geometry: wavefronts per walker, walkers per workgroup, row tiles and blocks per group.
struct ShareLaunch {
  bool ok = false;
  int NWV = 1, W = 1, RT = 1, qup = 1, qdn = 1;
  size_t lds = 0;
};
// The RT of the least padded work; walkers per workgroup: those that fill the most wavefront slots
// of a round of four SIMDs, then the most.
inline ShareLaunch share_launch(int nup, int ndn, int M, int G) {
  ShareLaunch f;
  const int nmax = nup > ndn ? nup : ndn, nk = (M + 15) / 16;
  if (nmax < 1 || nmax > 64 || nk < SHARE_MIN_NK || nk > SHARE_MAX_NK) return f;
  f.NWV = (2 * nmax + 15) / 16;
  const int g1 = G > 1 ? G : 1;
  double best = 1e300;
  for (int rt = (nmax + 15) / 16; rt <= SHARE_MAX_RT; ++rt) {
    const int qu = nup > 0 ? std::min(g1, 16 * rt / nup) : 1;
    const int qd = ndn > 0 ? std::min(g1, 16 * rt / ndn) : 1;
    // products of one row tile wait for each other: with two tiles 133 of 151 TFLOP/s
    const double work =
        (rt == 1 ? 1.5 : rt == 2 ? 1.15 : 1.0) * rt *
        ((nup > 0 ? (g1 + qu - 1) / qu : 0) + (ndn > 0 ? (g1 + qd - 1) / qd : 0));
    if (work < best * 0.99) best = work, f.RT = rt, f.qup = qu, f.qdn = qd;
  }
  best = 0.0;
  for (int w = 1; w * f.NWV <= SHARE_MAX_WAVES; ++w) {
    const int waves = w * f.NWV;
    if (waves < f.RT || share_lds_bytes(w, f.NWV, f.RT, nmax) > SHARE_LDS_CAP) continue;
    const double fill = (double)waves / ((waves + 3) / 4 * 4);
    if (fill >= best) best = fill, f.W = w, f.ok = true;
  }
  f.lds = share_lds_bytes(f.W, f.NWV, f.RT, nmax);
  return f;
}
