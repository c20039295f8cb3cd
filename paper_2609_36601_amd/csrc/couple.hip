// One part of the coupling kernel's instantiations (SAKI_PART, see couple.hpp).
#include "couple.hpp"

namespace saki {
namespace {

constexpr bool K34 = (SAKI_PART & 1) != 0;
using T = std::conditional_t<(SAKI_PART & 2) != 0, float, uint16_t>;

template <typename G, bool ROUTE, bool GRAD>
void launch(const CoupleParams& P, int grid, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    if ((P.V + CHUNK - 1) / CHUNK <= CACHED_MAXC) {
      hipLaunchKernelGGL((couple_kernel<T, G, ROUTE, GRAD, CACHE_KC, K34>), dim3(grid), dim3(NT), 0, st, P);
      return;
    }
  }
  hipLaunchKernelGGL((couple_kernel<T, G, ROUTE, GRAD, 0, K34>), dim3(grid), dim3(NT), 0, st, P);
}

}  // namespace

template <>
hipError_t launch_couple_part<SAKI_PART>(const CoupleParams& P, bool route, bool grad, bool grad_bf16, int grid,
                                         hipStream_t st) {
  if (!route)
    launch<float, false, false>(P, grid, st);
  else if (!grad)
    launch<float, true, false>(P, grid, st);
  else if (grad_bf16)
    launch<uint16_t, true, true>(P, grid, st);
  else
    launch<float, true, true>(P, grid, st);
  return hipGetLastError();
}

}  // namespace saki
