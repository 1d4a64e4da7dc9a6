// Launches of the per-vector local-energy contraction: one kernel instance per precision, tile
// variant and K chunk count.
#include <hip/hip_runtime.h>

#include "../../include/afqmc.h"
#include "kernels_mfma.hpp"

hipError_t mfma_contract(const MfmaTables& t, hipStream_t st, int nw, int n_det, int G,
                         const void* thetaP, const double* weight, cd* tpart, cd* exch, int tile,
                         ContractSel sel, int nz) {
  if (t.precision == AFQMC_FP64) {
    const size_t shm = mfma_f64_contract_lds_bytes(t);
    dim3 grid((nw + 1) / 2, 2 * n_det);
    // one instantiation per K chunk count (K_P = 32 .. 128 in steps of 32)
    if (t.KP % 32 != 0 || t.KP < 32 || t.KP > MFMA_KMAX) return hipErrorInvalidValue;
#define LAUNCH_F64(NPV, NKV)                                                                   \
  do {                                                                                         \
    (void)hipFuncSetAttribute((const void*)k_contract_f64mfma<NPV, NKV>,                       \
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);           \
    hipLaunchKernelGGL((k_contract_f64mfma<NPV, NKV>), grid, dim3(256), shm, st, nw, G, t.nup, \
                       t.ndn, t.KP, (const double*)t.Lp, (const double*)thetaP, weight, tpart, \
                       exch, sel.list, sel.cnt, sel.thmax, sel.guard);                         \
  } while (0)
#define LAUNCH_F64_NP(NPV)                                                                     \
  do {                                                                                         \
    switch (t.KP / 8) {                                                                        \
      case 4: LAUNCH_F64(NPV, 4); break;                                                       \
      case 8: LAUNCH_F64(NPV, 8); break;                                                       \
      case 12: LAUNCH_F64(NPV, 12); break;                                                     \
      default: LAUNCH_F64(NPV, 16); break;                                                     \
    }                                                                                          \
  } while (0)
    if (t.NP == 32) LAUNCH_F64_NP(32);
    else LAUNCH_F64_NP(16);
#undef LAUNCH_F64_NP
#undef LAUNCH_F64
    return hipGetLastError();
  }
  const bool bf = t.precision == AFQMC_BF16X3;
  if (!mfma_tile_valid(t, tile)) tile = TILE_DEFAULT;
  // FP32 chunks of 16 k past M hold only zeros and are left out (the same bits)
  const int nk16 = (t.M + 15) / 16;
  // default at N_P = 32: the block-exchange kernel (fewest LDS and vector instructions per g),
  // eight walkers per workgroup when the workgroups with work (walkers, active spins,
  // determinants) still cover every CU
  if (tile == TILE_DEFAULT && !t.wide && t.NP == 32) {
    const int spins = (t.nup > 0 ? 1 : 0) + (t.ndn > 0 ? 1 : 0);
    tile = (size_t)((nw + 7) / 8) * spins * n_det * nz >= (size_t)device_cu_count() ? TILE_BX8
                                                                                      : TILE_BX;
  }
  if (const ShareLaunch f = share_of(t, tile); f.ok)
    return mfma_contract_share(t, st, nw, n_det, G, thetaP, weight, tpart, exch, f, sel, nz);
  if (tile == TILE_FLAT || tile == TILE_STACK)
    return mfma_contract_flat(t, st, nw, n_det, G, thetaP, weight, tpart, exch, tile == TILE_STACK,
                              sel, nz, bf ? t.KP / 32 : nk16);
  if (t.wide || tile == TILE_WIDE) {
    dim3 grid(nw, 2 * n_det, nz);
#define LAUNCH_WIDE_K(NPV, BFV, KM)                                                             \
  do {                                                                                          \
    const size_t shm_ = wide_contract_lds_bytes_t<NPV, BFV>(t.KP);                              \
    hipLaunchKernelGGL((k_contract_mfma_wide<NPV, BFV, KM>), grid, dim3(4 * NPV), shm_, st, nw, \
                       G, t.nup, t.ndn, t.KP, (const void*)t.Lp, thetaP, weight, tpart, exch, sel); \
  } while (0)
  // one instantiation per K chunk count (FP32 of 16, BF16x3 of 32, up to K_P = 224)
#define LAUNCH_WIDE(NPV, BFV)                                                                   \
  do {                                                                                          \
    switch (BFV ? t.KP / 32 : nk16) {                                                           \
      case 1: LAUNCH_WIDE_K(NPV, BFV, 1); break;                                                \
      case 2: LAUNCH_WIDE_K(NPV, BFV, 2); break;                                                \
      case 3: LAUNCH_WIDE_K(NPV, BFV, 3); break;                                                \
      case 4: LAUNCH_WIDE_K(NPV, BFV, 4); break;                                                \
      case 5: LAUNCH_WIDE_K(NPV, BFV, 5); break;                                                \
      case 6: LAUNCH_WIDE_K(NPV, BFV, 6); break;                                                \
      case 7: LAUNCH_WIDE_K(NPV, BFV, 7); break;                                                \
      case 8: LAUNCH_WIDE_K(NPV, BFV, BFV ? 7 : 8); break;                                      \
      case 9: LAUNCH_WIDE_K(NPV, BFV, BFV ? 7 : 9); break;                                      \
      case 10: LAUNCH_WIDE_K(NPV, BFV, BFV ? 7 : 10); break;                                    \
      case 11: LAUNCH_WIDE_K(NPV, BFV, BFV ? 7 : 11); break;                                    \
      case 12: LAUNCH_WIDE_K(NPV, BFV, BFV ? 7 : 12); break;                                    \
      case 13: LAUNCH_WIDE_K(NPV, BFV, BFV ? 7 : 13); break;                                    \
      case 14: LAUNCH_WIDE_K(NPV, BFV, BFV ? 7 : 14); break;                                    \
      default: return hipErrorInvalidValue;                                                     \
    }                                                                                           \
  } while (0)
    if (t.NP == 64) {
      if (bf) LAUNCH_WIDE(64, true);
      else LAUNCH_WIDE(64, false);
    } else if (t.NP == 48) {
      if (bf) LAUNCH_WIDE(48, true);
      else LAUNCH_WIDE(48, false);
    } else {
      if (bf) LAUNCH_WIDE(32, true);
      else LAUNCH_WIDE(32, false);
    }
#undef LAUNCH_WIDE
#undef LAUNCH_WIDE_K
    return hipGetLastError();
  }
  const int wpb = tile == TILE_W2 ? 2 : 4;
  // the kernels are instantiated for K_P = 32, 64, 96, 128
  if (t.KP % 32 != 0 || t.KP < 32 || t.KP > MFMA_KMAX) return hipErrorInvalidValue;
  if (tile == TILE_BX || tile == TILE_BX8) {
    const int wb = tile == TILE_BX8 ? 8 : 4;
    const size_t shm = bx_contract_lds_bytes(t.KP, bf, wb);
    dim3 grid((nw + wb - 1) / wb, 2 * n_det, nz);
#define LAUNCH_BX(BFV, NKV, WBV)                                                               \
  do {                                                                                         \
    (void)hipFuncSetAttribute((const void*)k_contract_mfma_bx<BFV, NKV, WBV>,                  \
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);           \
    hipLaunchKernelGGL((k_contract_mfma_bx<BFV, NKV, WBV>), grid, dim3(64 * WBV), shm, st, nw, \
                       G, t.nup, t.ndn, (const void*)t.Lp, thetaP, weight, tpart, exch, sel);  \
  } while (0)
#define LAUNCH_BX_W(BFV, NKV)                                                                  \
  case NKV:                                                                                    \
    if (wb == 8) LAUNCH_BX(BFV, NKV, 8);                                                       \
    else LAUNCH_BX(BFV, NKV, 4);                                                               \
    break;
    // one instantiation per K chunk count (16 < N <= M, so FP32 has at least two chunks of 16)
    if (bf) {
      switch (t.KP / 32) { LAUNCH_BX_W(true, 1) LAUNCH_BX_W(true, 2) LAUNCH_BX_W(true, 3)
                           default: LAUNCH_BX_W(true, 4) }
    } else {
      switch (nk16) { LAUNCH_BX_W(false, 2) LAUNCH_BX_W(false, 3) LAUNCH_BX_W(false, 4)
                      LAUNCH_BX_W(false, 5) LAUNCH_BX_W(false, 6) LAUNCH_BX_W(false, 7)
                      LAUNCH_BX_W(false, 8)
                      default: return hipErrorInvalidValue; }
    }
#undef LAUNCH_BX_W
#undef LAUNCH_BX
    return hipGetLastError();
  }
  if (tile == TILE_PP) {
    const size_t shm = pp_contract_lds_bytes(t.NP, t.KP, bf);
    dim3 grid((nw + 7) / 8, 2 * n_det, nz);
#define LAUNCH_PP_K(NPV, BFV, NKV)                                                             \
  do {                                                                                         \
    (void)hipFuncSetAttribute((const void*)k_contract_mfma_pp<NPV, BFV, NKV>,                  \
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);           \
    hipLaunchKernelGGL((k_contract_mfma_pp<NPV, BFV, NKV>), grid, dim3(512), shm, st, nw, G,   \
                       t.nup, t.ndn, (const void*)t.Lp, thetaP, weight, tpart, exch, sel);     \
  } while (0)
#define LAUNCH_PP(NPV, BFV)                                                                    \
  do {                                                                                         \
    constexpr int KCH_ = contract_kch<NPV, BFV>();                                             \
    switch (t.KP / KCH_) {                                                                     \
      case 32 / KCH_: LAUNCH_PP_K(NPV, BFV, 32 / KCH_); break;                                 \
      case 64 / KCH_: LAUNCH_PP_K(NPV, BFV, 64 / KCH_); break;                                 \
      case 96 / KCH_: LAUNCH_PP_K(NPV, BFV, 96 / KCH_); break;                                 \
      default: LAUNCH_PP_K(NPV, BFV, 128 / KCH_); break;                                       \
    }                                                                                          \
  } while (0)
    if (t.NP == 32) {
      if (bf) LAUNCH_PP(32, true);
      else LAUNCH_PP(32, false);
    } else {
      if (bf) LAUNCH_PP(16, true);
      else LAUNCH_PP(16, false);
    }
#undef LAUNCH_PP
#undef LAUNCH_PP_K
    return hipGetLastError();
  }
  const size_t shm = mfma_contract_lds_bytes(t, wpb);
  dim3 grid((nw + wpb - 1) / wpb, 2 * n_det, nz);
#define LAUNCH_CONTRACT_K(NPV, BFV, WPBV, NKV)                                                  \
  do {                                                                                          \
    (void)hipFuncSetAttribute((const void*)k_contract_mfma<NPV, BFV, WPBV, NKV>,                \
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);            \
    hipLaunchKernelGGL((k_contract_mfma<NPV, BFV, WPBV, NKV>), grid, dim3(64 * WPBV), shm, st,  \
                       nw, G, t.nup, t.ndn, t.KP, (const void*)t.Lp, thetaP, weight, tpart,     \
                       exch, sel);                                                                \
  } while (0)
  // one instantiation per K chunk count (K_P = 32 .. 128 in steps of 32)
#define LAUNCH_CONTRACT(NPV, BFV, WPBV)                                                         \
  do {                                                                                          \
    constexpr int KCH_ = contract_kch<NPV, BFV>();                                              \
    switch (t.KP / KCH_) {                                                                      \
      case 32 / KCH_: LAUNCH_CONTRACT_K(NPV, BFV, WPBV, 32 / KCH_); break;                      \
      case 64 / KCH_: LAUNCH_CONTRACT_K(NPV, BFV, WPBV, 64 / KCH_); break;                      \
      case 96 / KCH_: LAUNCH_CONTRACT_K(NPV, BFV, WPBV, 96 / KCH_); break;                      \
      default: LAUNCH_CONTRACT_K(NPV, BFV, WPBV, 128 / KCH_); break;                            \
    }                                                                                           \
  } while (0)
  if (wpb == 4) {
    if (t.NP == 32) {
      if (bf) LAUNCH_CONTRACT(32, true, 4);
      else LAUNCH_CONTRACT(32, false, 4);
    } else {
      if (bf) LAUNCH_CONTRACT(16, true, 4);
      else
        switch (nk16) {
          case 1: LAUNCH_CONTRACT_K(16, false, 4, 1); break;
          case 3: LAUNCH_CONTRACT_K(16, false, 4, 3); break;
          case 5: LAUNCH_CONTRACT_K(16, false, 4, 5); break;
          case 7: LAUNCH_CONTRACT_K(16, false, 4, 7); break;
          default: LAUNCH_CONTRACT(16, false, 4);
        }
    }
  } else {
    if (t.NP == 32) {
      if (bf) LAUNCH_CONTRACT(32, true, 2);
      else LAUNCH_CONTRACT(32, false, 2);
    } else {
      if (bf) LAUNCH_CONTRACT(16, true, 2);
      else LAUNCH_CONTRACT(16, false, 2);
    }
  }
#undef LAUNCH_CONTRACT
#undef LAUNCH_CONTRACT_K
  return hipGetLastError();
}
