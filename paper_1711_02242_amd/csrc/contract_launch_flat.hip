// Launches of the stacked-row contraction kernels: one instance per precision, row-tile count and
// K chunk count.
#include <hip/hip_runtime.h>

#include "../../include/afqmc.h"
#include "kernels_mfma.hpp"

hipError_t mfma_contract_flat(const MfmaTables& t, hipStream_t st, int nw, int n_det, int G,
                              const void* thetaP, const double* weight, cd* tpart, cd* exch,
                              bool stk, ContractSel sel, int nz, int nk) {
  const bool bf = t.precision == AFQMC_BF16X3;
  const FlatLaunch f = flat_launch(t.nup, t.ndn, G, bf, stk);
  dim3 grid(nw, 2 * n_det, nz);
#define LAUNCH_FLAT_KR(BFV, KM, RTV)                                                              \
  do {                                                                                            \
    if (stk)                                                                                      \
      hipLaunchKernelGGL((k_contract_mfma_stack<KM, BFV, ((RTV) > (BFV ? 3 : STACK_MAX_RT)        \
                                                              ? (BFV ? 3 : STACK_MAX_RT)          \
                                                              : (RTV))>),                         \
                         grid, dim3(64 * f.waves), f.lds, st, nw, G, t.nup, t.ndn, t.NP, t.KP,    \
                         f.qup, f.qdn, f.LDR, (const void*)t.Lp, thetaP, weight, tpart, exch, sel); \
    else                                                                                          \
      hipLaunchKernelGGL((k_contract_mfma_flat<KM, BFV, (RTV)>), grid, dim3(64 * f.waves), f.lds, \
                         st, nw, G, t.nup, t.ndn, t.NP, t.KP, f.qup, f.qdn, f.LDR,                \
                         (const void*)t.Lp, thetaP, weight, tpart, exch, sel);                    \
  } while (0)
  // one instantiation per row-tile count (flat 1 .. 7, BF16x3 1 .. 4; stack 1 .. 7, BF16x3
  // 1 .. 3)
#define LAUNCH_FLAT_K(BFV, KM)                                                                    \
  do {                                                                                            \
    switch (f.RT) {                                                                               \
      case 1: LAUNCH_FLAT_KR(BFV, KM, 1); break;                                                  \
      case 2: LAUNCH_FLAT_KR(BFV, KM, 2); break;                                                  \
      case 3: LAUNCH_FLAT_KR(BFV, KM, 3); break;                                                  \
      case 4: LAUNCH_FLAT_KR(BFV, KM, 4); break;                                                  \
      case 5: LAUNCH_FLAT_KR(BFV, KM, BFV ? 4 : 5); break;                                        \
      case 6: LAUNCH_FLAT_KR(BFV, KM, BFV ? 4 : 6); break;                                        \
      default: LAUNCH_FLAT_KR(BFV, KM, BFV ? 4 : 7); break;                                       \
    }                                                                                             \
  } while (0)
  // and per K chunk count (FP32 chunks of 16: chunks past M hold only zeros; BF16x3 of 32)
  if (bf) {
    switch (nk) {
      case 1: LAUNCH_FLAT_K(true, 1); break;
      case 2: LAUNCH_FLAT_K(true, 2); break;
      case 3: LAUNCH_FLAT_K(true, 3); break;
      case 4: LAUNCH_FLAT_K(true, 4); break;
      case 5: LAUNCH_FLAT_K(true, 5); break;
      case 6: LAUNCH_FLAT_K(true, 6); break;
      case 7: LAUNCH_FLAT_K(true, 7); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (nk) {
      case 1: LAUNCH_FLAT_K(false, 1); break;
      case 2: LAUNCH_FLAT_K(false, 2); break;
      case 3: LAUNCH_FLAT_K(false, 3); break;
      case 4: LAUNCH_FLAT_K(false, 4); break;
      case 5: LAUNCH_FLAT_K(false, 5); break;
      case 6: LAUNCH_FLAT_K(false, 6); break;
      case 7: LAUNCH_FLAT_K(false, 7); break;
      case 8: LAUNCH_FLAT_K(false, 8); break;
      case 9: LAUNCH_FLAT_K(false, 9); break;
      case 10: LAUNCH_FLAT_K(false, 10); break;
      case 11: LAUNCH_FLAT_K(false, 11); break;
      case 12: LAUNCH_FLAT_K(false, 12); break;
      case 13: LAUNCH_FLAT_K(false, 13); break;
      case 14: LAUNCH_FLAT_K(false, 14); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef LAUNCH_FLAT_K
#undef LAUNCH_FLAT_KR
  return hipGetLastError();
}
