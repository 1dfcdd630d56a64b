// Launch of the head-dim 192 / 256 dQ kernel (dq256.h) on its own.
#include "dq256.h"
#include "launch.h"

namespace dkv {
namespace {

using namespace dq256;

template <int D, bool LOCAL>
__global__ __launch_bounds__(512) void dq256_kernel(const AttnParams p) {
  const int bid = blockIdx.x, nblk = gridDim.x;
  constexpr bool STATS = true;
#include "dq256_body.h"
}

template <int D, bool LOCAL>
hipError_t launch_t(AttnParams p, hipStream_t st) {
  fill_packing(p, NSUB);
  auto kern = dq256_kernel<D, LOCAL>;
  hipError_t e = ensure_dynamic_lds<dq256_kernel<D, LOCAL>>(Cfg<D>::SMEM_BYTES);
  if (e != hipSuccess) return e;
  return launch_sequences(p, (int64_t)p.MB * p.HC * p.Hk, 512, [&](const AttnParams& q, unsigned n) {
    hipLaunchKernelGGL(kern, dim3(n), dim3(512), Cfg<D>::SMEM_BYTES, st, q);
    return hipGetLastError();
  });
}

}  // namespace

hipError_t launch_dq256(const AttnParams& p, int head_dim, hipStream_t st) {
  const bool local = p.window > 0;
  switch (head_dim) {
    case 192: return local ? launch_t<192, true>(p, st) : launch_t<192, false>(p, st);
    case 256: return local ? launch_t<256, true>(p, st) : launch_t<256, false>(p, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace dkv
