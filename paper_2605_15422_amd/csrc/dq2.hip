// Launch of the head-dim 64 / 96 / 128 dQ kernel (dq2.h) on its own.
#include "dq2.h"
#include "launch.h"

namespace dkv {

template <int D, int NW, bool LOCAL>
__global__ __launch_bounds__(NW * 64, D == 64 && NW == 4 ? 3 : 2) void dq2_kernel(const AttnParams p) {
  dq2_workgroup<D, NW, LOCAL, true>(p, blockIdx.x, gridDim.x);
}

template <int D, int NW, bool LOCAL>
static hipError_t launch_dq2_t(AttnParams p, bool pair, hipStream_t st) {
  fill_packing(p, NW);
  constexpr size_t alone = 96 << 10;   // (of a CU's 160 KB: one workgroup)
  const size_t smem = pair ? kDq2Smem<D, NW> : std::max(kDq2Smem<D, NW>, alone);
  auto kern = dq2_kernel<D, NW, LOCAL>;
  hipError_t e = ensure_dynamic_lds<dq2_kernel<D, NW, LOCAL>>(std::max(kDq2Smem<D, NW>, alone));
  if (e != hipSuccess) return e;
  return launch_sequences(p, (int64_t)p.MB * p.HC * p.Hk, NW * 64, [&](const AttnParams& q, unsigned n) {
    hipLaunchKernelGGL(kern, dim3(n), dim3(NW * 64), smem, st, q);
    return hipGetLastError();
  });
}

template <int D>
static hipError_t launch_dq2_d(const AttnParams& p, hipStream_t st) {
  const bool local = p.window > 0;
  const rules::Waves w = choose_waves(p, D, true);
  if (w.n == 8) return local ? launch_dq2_t<D, 8, true>(p, w.pair, st) : launch_dq2_t<D, 8, false>(p, w.pair, st);
  return local ? launch_dq2_t<D, 4, true>(p, w.pair, st) : launch_dq2_t<D, 4, false>(p, w.pair, st);
}

hipError_t launch_dq2(const AttnParams& p, int head_dim, hipStream_t st) {
  switch (head_dim) {
    case 64:  return launch_dq2_d<64>(p, st);
    case 96:  return launch_dq2_d<96>(p, st);
    case 128: return launch_dq2_d<128>(p, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace dkv
