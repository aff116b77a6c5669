// One CG-stage kernel with a generated, register-resident contraction body
// for a single L_max.  Built once per L with -DCGCONV_TU_L=<L> and
// -DCGCONV_BODY="cg_body_L<L>.inc".  See cg.hip for the stage itself.
#include <hip/hip_runtime.h>

#include "cg_common.h"

namespace cgconv {
namespace cgdev {
#include CGCONV_BODY
}  // namespace cgdev

namespace {

// Up to L_max = 6 the inputs of a point (2K complex values) fit one lane's
// 256-register budget (two waves per SIMD) with at most a few spills.
template <int L>
__global__ __launch_bounds__(cgdev::kCgThreads, 2) void cg_gen_kernel(CgArgs a) {
  using namespace cgdev;
  constexpr int K = (L + 1) * (L + 1);
  const long long p = (long long)blockIdx.x * kCgThreads + threadIdx.x;
  const Point pt = point_of(p, a);
  float2 qa[K], ka[K];
  load_unpack<K>(a, pt, qa, ka);
  PairStore st = make_store(a, pt, K);
  CgBody<L>::run(qa, ka, st);
}

// L_max 7 and 8: one point per pair of lanes (CgMirrorBody), so that two
// waves share a SIMD (179 and 215 VGPRs, no scratch): a single wave issues at
// most one instruction every ~4.8 cycles, two waves one every ~2.4.  Bound by
// the vector instruction stream, 31.5k operations per lane at L_max = 8; the
// lane pair that held q in one lane and k in the other took 39.8k.  Measured,
// L_max = 8, B = 2, N = 65536, C = 64: 7.42 -> 6.36 ms; L_max = 7, B = 4, N =
// 16384, C = 32: 1.19 -> 1.03 ms.  Below L_max = 7 one point per lane stays
// faster, as its fewer instructions per point count for more than the third
// wave a lane pair would allow (588 against 626 us at L_max = 6, 311 against
// 344 at 5, B = 4, N = 16384, C = 32).
template <int L>
__global__ __launch_bounds__(cgdev::kCgThreads, 2) void cg_split_kernel(CgArgs a) {
  using namespace cgdev;
  constexpr int K = (L + 1) * (L + 1), H = (L + 1) * (L + 2) / 2;
  const long long lane = (long long)blockIdx.x * kCgThreads + threadIdx.x;
  const int half = (int)(lane & 1);
  const float g = half ? -1.f : 1.f;
  const Point pt = point_of(lane >> 1, a);
  float2 q[H], k[H];
  load_unpack_mirror<L>(a, pt, half, g, q, k);
  SplitPairStore st = make_split_store(a, pt, half, g, K);
  CgMirrorBody<L>::run(q, k, st);
}

}  // namespace

template <>
hipError_t launch_cg_gen<CGCONV_TU_L>(const CgArgs& a, hipStream_t s) {
  if constexpr (CGCONV_TU_L >= 7) {
    const long long blocks = (2 * a.npts + cgdev::kCgThreads - 1) / cgdev::kCgThreads;
    hipLaunchKernelGGL(cg_split_kernel<CGCONV_TU_L>, dim3((unsigned)blocks), dim3(cgdev::kCgThreads), 0, s, a);
  } else {
    const long long blocks = (a.npts + cgdev::kCgThreads - 1) / cgdev::kCgThreads;
    hipLaunchKernelGGL(cg_gen_kernel<CGCONV_TU_L>, dim3((unsigned)blocks), dim3(cgdev::kCgThreads), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace cgconv
