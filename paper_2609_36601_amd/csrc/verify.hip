// One part of the verification kernel's instantiations (SAKI_PART, see verify.hpp).
#include <algorithm>

#include "verify.hpp"

namespace saki {

template <>
hipError_t launch_verify_part<SAKI_PART>(const VerifyParams& P, int cus, bool bf16, hipStream_t hs) {
  constexpr bool K34 = SAKI_PART != 0;
  const bool cached = bf16 && (P.V + CHUNK - 1) / CHUNK <= CACHED_MAXC;
  const int64_t n_items = P.n_blocks * P.k;
  const int grid = static_cast<int>(std::min<int64_t>(n_items, static_cast<int64_t>(cus) * WG_PER_CU));
  if (P.n_blocks <= cus) {
    // no more blocks than CUs: 512-thread workgroups, one per CU (see verify_kernel)
    const dim3 g1(static_cast<unsigned>(std::min<int64_t>(n_items, cus))), b1(512);
    if (cached)
      hipLaunchKernelGGL((verify_kernel<uint16_t, CACHE_KC, 512, K34>), g1, b1, 0, hs, P);
    else if (bf16)
      hipLaunchKernelGGL((verify_kernel<uint16_t, 0, 512, K34>), g1, b1, 0, hs, P);
    else
      hipLaunchKernelGGL((verify_kernel<float, 0, 512, K34>), g1, b1, 0, hs, P);
  } else if (cached) {
    hipLaunchKernelGGL((verify_kernel<uint16_t, CACHE_KC, 256, K34>), dim3(grid), dim3(256), 0, hs, P);
  } else if (bf16) {
    hipLaunchKernelGGL((verify_kernel<uint16_t, 0, 256, K34>), dim3(grid), dim3(256), 0, hs, P);
  } else {
    hipLaunchKernelGGL((verify_kernel<float, 0, 256, K34>), dim3(grid), dim3(256), 0, hs, P);
  }
  return hipGetLastError();
}

}  // namespace saki
