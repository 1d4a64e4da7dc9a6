// Launches of the shared-row contraction kernel: one instance per K chunk count and row-tile count.
#include <hip/hip_runtime.h>

#include "../../include/afqmc.h"
#include "kernels_mfma.hpp"

namespace {

template <int NK, int RT>
hipError_t launch(const MfmaTables& t, hipStream_t st, dim3 grid, int G, int nw, const void* thetaP,
                  const double* weight, cd* tpart, cd* exch, const ShareLaunch& f, ContractSel sel) {
  if (f.lds > 65536)
    (void)hipFuncSetAttribute((const void*)k_contract_share<NK, RT>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)f.lds);
  hipLaunchKernelGGL((k_contract_share<NK, RT>), grid, dim3(64 * f.NWV * f.W), f.lds, st, nw, G,
                     t.nup, t.ndn, t.NP, t.KP, f.qup, f.qdn, f.NWV, (const float*)t.Lp, (const float*)thetaP, weight, tpart, exch, sel);
  return hipGetLastError();
}

template <int NK, typename... Args>
hipError_t launch_rt(int rt, Args&&... a) {
  switch (rt) {
    case 1: return launch<NK, 1>(a...);
    case 2: return launch<NK, 2>(a...);
    case 3: return launch<NK, 3>(a...);
    case 4: return launch<NK, 4>(a...);
    case 5: return launch<NK, 5>(a...);
    case 6: return launch<NK, 6>(a...);
    case 7: return launch<NK, 7>(a...);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t mfma_contract_share(const MfmaTables& t, hipStream_t st, int nw, int n_det, int G,
                               const void* thetaP, const double* weight, cd* tpart, cd* exch,
                               const ShareLaunch& f, ContractSel sel, int nz) {
  const dim3 grid((nw + f.W - 1) / f.W, 2 * n_det, nz);
#define SHARE_NK(NK) \
  case NK: return launch_rt<NK>(f.RT, t, st, grid, G, nw, thetaP, weight, tpart, exch, f, sel);
  switch ((t.M + 15) / 16) {
    SHARE_NK(3) SHARE_NK(4) SHARE_NK(5) SHARE_NK(6) SHARE_NK(7) SHARE_NK(8) SHARE_NK(9)
    SHARE_NK(10) SHARE_NK(11) SHARE_NK(12) SHARE_NK(13) SHARE_NK(14)
    default: return hipErrorInvalidValue;
  }
#undef SHARE_NK
}
