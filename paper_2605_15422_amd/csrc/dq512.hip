// Launch of the head-dim 512 dQ kernel (dq512.h) on its own.
#include "dq512.h"
#include "launch.h"

namespace dkv {
namespace {

using namespace dq512;

template <bool LOCAL>
__global__ __launch_bounds__(512) void dq512_kernel(const AttnParams p) {
  const int bid = blockIdx.x, nblk = gridDim.x;
  constexpr bool STATS = true;
#include "dq512_body.h"
}

template <bool LOCAL>
hipError_t launch_t(AttnParams p, hipStream_t st) {
  fill_packing(p, NSUB);
  hipError_t e = ensure_dynamic_lds<dq512_kernel<LOCAL>>(SMEM_BYTES);
  if (e != hipSuccess) return e;
  return launch_sequences(p, (int64_t)p.MB * p.HC * p.Hk, 512, [&](const AttnParams& q, unsigned n) {
    hipLaunchKernelGGL(dq512_kernel<LOCAL>, dim3(n), dim3(512), SMEM_BYTES, st, q);
    return hipGetLastError();
  });
}

}  // namespace

hipError_t launch_dq512(const AttnParams& p, hipStream_t st) {
  if (p.window > 0) return hipErrorInvalidValue;   // (the interface offers no window at this head dim)
  return launch_t<false>(p, st);
}

}  // namespace dkv
