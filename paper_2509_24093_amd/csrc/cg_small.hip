// The whole CG convolution of one batch element and one channel group in a
// single block, for short token axes (DFT length Nf <= 256) on gfx950
// (arXiv 2509.24093: §4.1 convolution theorem, §4.3 sparsity).
//
// At the small shapes (n-body, molecule sizes) the three-kernel pipeline is
// latency-bound: every kernel waits for its loads, runs a short dependent
// chain and ends, and the intermediate spectra go through memory twice.  Here
// one block keeps its channel group's spectra in LDS from the load to the
// store:
//   1. load q + i k of cc channels, all Nf rows and K components, into an LDS
//      tile [row][k][c] (rows >= in_rows of a zero-padded plan are zero; a
//      padding channel of odd C repeats channel C-1, whose spectrum is again
//      that of a real signal);
//   2. forward DFT along the rows of every column (k, c), in place: Nf =
//      R1 x R2 (R1, R2 <= 16), a radix-R1 DFT in registers per (column, n2),
//      the twiddle W_Nf^(n2 f1), a radix-R2 DFT per (column, f1); frequency
//      f1 + R1 f2 ends at row R2 f1 + f2;
//   3. one point (frequency pair w, N-w; channel) per pair of lanes: both
//      gather the spectra at w and N-w, half 0 keeps the complex-m components
//      m >= 0 of 2Q and 2K, half 1 the mirrored ones, and the lane-pair
//      contraction CgMirrorBody runs on registers;
//   4. every output component, packed with the neighbouring channel
//      (W = U_c + i U_{c+1} at row w, conj U_c + i conj U_{c+1} at row N-w),
//      goes to an LDS tile [row][k][pair] that aliases the first one;
//   5. inverse DFT of every column (k, pair) in the same way (time n1 + R1 n2
//      at row R2 n1 + n2), x 1/Nf, and the store of the real and imaginary
//      parts as channels c and c+1.
// HBM traffic is q, k in and out out; the kernel is one launch, also for the
// two gradients of a backward (the adjoint form, one problem each).
// Bound by latency: one lane's chain of loads, LDS exchanges and dependent
// operations (of 47k cycles at B=32, N=32, L_max=4, C=32 with one lane group
// per point, 20k were the contraction's 2.6k operations, which two groups
// halve).  Measured at that shape: forward 17.5 us (23.6 with the lane pair
// that held q in one lane and k in the other), both gradients 21.1 us (52.7 in
// the six launches of the three kernels).
#include <hip/hip_runtime.h>

#include "cg_common.h"
#include "fft_reg.h"

namespace cgconv {
namespace cgdev {
#include CGCONV_BODY
}  // namespace cgdev

namespace {

using namespace cgdev;

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmulf(float2 a, float2 b) {
  return make_float2(fnma(a.y, b.y, a.x * b.x), fmaf(a.y, b.x, a.x * b.y));
}

// fp32 -> bfloat16 bits, round to nearest even (NaN stays a quiet NaN)
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// floor(x / d) for x * d < 2^32, with m = floor((2^32 - 1) / d) + 1 taken
// modulo 2^32 (d = 1 gives m = 0: the identity)
__device__ __forceinline__ int divm(int x, uint32_t m) { return m ? (int)__umulhi((uint32_t)x, m) : x; }

// In-place DFT of `cols` interleaved columns of length Nf = R1 * R2 (element
// (n, col) at Z[n * cols + col]), natural order in; frequency f1 + R1 f2 out
// at row R2 f1 + f2.  tw[j] = exp(-2 pi i j / Nf), j < Nf; DIR = +1: inverse
// (conjugate twiddles).  mc = the division magic of cols.
template <int R1, int R2, int DIR>
__device__ __forceinline__ void dft_columns(float2* Z, const float2* tw, int cols, uint32_t mc, int tid,
                                            int nthreads) {
  __syncthreads();
  // stage 1: per (column, n2), rows R2 n1 + n2 -> radix R1 -> x W^(n2 f1)
  for (int it = tid; it < R2 * cols; it += nthreads) {
    const int n2 = divm(it, mc), col = it - n2 * cols;
    float2* z = Z + n2 * cols + col;
    float2 x[R1];
#pragma unroll
    for (int t = 0; t < R1; ++t) x[t] = z[t * R2 * cols];
    dft::dft_reg<R1, DIR>(x);
#pragma unroll
    for (int f = 0; f < R1; ++f) {
      float2 w = tw[n2 * f];
      if (DIR > 0) w.y = -w.y;
      z[f * R2 * cols] = f == 0 ? x[0] : cmulf(x[f], w);
    }
  }
  if constexpr (R2 > 1) {
    __syncthreads();
    // stage 2: per (column, f1), rows R2 f1 .. R2 f1 + R2 - 1 -> radix R2, in place
    for (int it = tid; it < R1 * cols; it += nthreads) {
      const int f1 = divm(it, mc), col = it - f1 * cols;
      float2* z = Z + f1 * R2 * cols + col;
      float2 x[R2];
#pragma unroll
      for (int t = 0; t < R2; ++t) x[t] = z[t * cols];
      dft::dft_reg<R2, DIR>(x);
#pragma unroll
      for (int f = 0; f < R2; ++f) z[f * cols] = x[f];
    }
  }
  __syncthreads();
}

template <int DIR>
__device__ __forceinline__ void dft_any(int lg, float2* Z, const float2* tw, int cols, uint32_t mc, int tid,
                                        int nthreads) {
  switch (lg) {  // uniform: Nf = R1 * R2
    case 1: dft_columns<2, 1, DIR>(Z, tw, cols, mc, tid, nthreads); break;
    case 2: dft_columns<4, 1, DIR>(Z, tw, cols, mc, tid, nthreads); break;
    case 3: dft_columns<8, 1, DIR>(Z, tw, cols, mc, tid, nthreads); break;
    case 4: dft_columns<16, 1, DIR>(Z, tw, cols, mc, tid, nthreads); break;
    case 5: dft_columns<8, 4, DIR>(Z, tw, cols, mc, tid, nthreads); break;
    case 6: dft_columns<8, 8, DIR>(Z, tw, cols, mc, tid, nthreads); break;
    case 7: dft_columns<16, 8, DIR>(Z, tw, cols, mc, tid, nthreads); break;
    default: dft_columns<16, 16, DIR>(Z, tw, cols, mc, tid, nthreads); break;
  }
}

// second radix of Nf = 2^lg as split above
__device__ __forceinline__ int radix2_of(int lg) { return lg <= 4 ? 1 : (lg == 5 ? 4 : (lg <= 7 ? 8 : 16)); }

// Outputs of a lane pair: half 0 stores component (J, +mu), half 1 (J, -mu);
// both hold the same value of (J, 0) and write it to the same slot.  The
// channel partner is lane ^ 2.
struct SmallStore {
  float2* V;    // LDS output tile [row][K][cq], row Nf = trash
  int K, cq, ci;
  int row;      // destination row of this lane (w, N - w), or Nf
  float g;      // the half's sign
  bool even;
  __device__ __forceinline__ void put(int J, int mu, float2 acc) const {
    const float2 u = mirror_out(J, mu, acc, g);
    const float2 v = make_float2(swap_quad_pair(u.x), swap_quad_pair(u.y));
    V[(row * K + J * J + J + (g < 0.f ? -mu : mu)) * cq + ci] =
        even ? make_float2(u.x - v.y, u.y + v.x) : make_float2(v.x + u.y, u.x - v.y);
  }
  __device__ __forceinline__ void end_phase(int) const {}
};

// Waves per SIMD the registers must allow: up to L_max 3 the radix-16 DFTs hold
// the most, 70 VGPRs, seven waves, when held to it; left alone the forward takes
// 85, and blocks of five or nine waves no longer share a CU (B=512 N=64 L=0 C=8:
// 6.5 us held, 9.4 not).  Above, the contraction's registers decide (at L_max 4
// six waves would spill).
constexpr int small_waves(int L) { return L <= 3 ? 6 : 1; }

// ADJ: the adjoint form, one or two problems; otherwise the forward of problem
// 0, without the reversed rows, the scales and the choice of a problem (L=0,
// B=1 N=8 C=3, where the launch is all there is: 4.9 us for one kernel of both
// forms, 4.1 us).
template <int L, bool ADJ>
__global__ __launch_bounds__(small_max_threads(L), small_waves(L)) void cg_small_kernel(SmallArgs a) {
  constexpr int K = (L + 1) * (L + 1);
  extern __shared__ __attribute__((aligned(16))) float2 smem[];
  const int Nf = a.Nf, lg = a.lg, cc = a.cc, cq = cc >> 1;
  const int tid = threadIdx.x, nthreads = blockDim.x;
  const int b = blockIdx.x / a.groups, grp = blockIdx.x % a.groups;
  const int c0 = grp * cc;  // first channel of the group
  const SmallProblem pr = a.problem[ADJ ? blockIdx.y : 0];
  float2* Z = smem;                 // [Nf][K][cc]
  float2* tw = smem + Nf * K * cc;  // [Nf]
  const int colsZ = K * cc, colsV = K * cq;

  for (int j = tid; j < Nf; j += nthreads) tw[j] = a.tw[j];
  // 1. load q + i k: kInFlight elements per thread at a time.  The adjoint
  // form scales both operands per component and reads the rows of the second
  // one reversed.
  // (eight: the same with many elements per thread, but with few the code that
  // finds nothing to load is what a block runs, 4-7% of a launch at L_max 0, 1; two
  // wait more often, up to 5% above L_max 2)
  constexpr int kInFlight = 4;
  const long long in_b = (long long)b * a.in_rows * K * a.C;
  const int totalZ = Nf * colsZ;
  for (int base = 0; base < totalZ; base += kInFlight * nthreads) {
    float2 z[kInFlight];
    [[maybe_unused]] float2 sc[kInFlight];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const int it = base + u * nthreads + tid;
      const int n = divm(it, a.mz), col = it - n * colsZ;
      const int k = col >> a.lcc, c = col & (cc - 1);
      const int ch = c0 + c < a.C ? c0 + c : a.C - 1;
      const int n1 = ADJ ? (-n) & (Nf - 1) : n;
      z[u] = make_float2(0.f, 0.f);
      const bool in0 = it < totalZ && n < a.in_rows, in1 = it < totalZ && n1 < a.in_rows;
      const uint32_t off0 = ((uint32_t)n * K + k) * (uint32_t)a.C + ch;
      const uint32_t off1 = ((uint32_t)n1 * K + k) * (uint32_t)a.C + ch;
      const float* q32 = static_cast<const float*>(pr.q) + in_b;
      const float* k32 = static_cast<const float*>(pr.k) + in_b;
      if constexpr (ADJ) {
        if (in0) z[u].x = q32[off0];
        if (in1) z[u].y = k32[off1];
        if (it < totalZ) sc[u] = make_float2(pr.scales[k], pr.scales[K + k]);
      } else if (in0) {
        if (a.bf16) {
          const uint16_t* q16 = static_cast<const uint16_t*>(pr.q) + in_b;
          const uint16_t* k16 = static_cast<const uint16_t*>(pr.k) + in_b;
          z[u] = make_float2(__uint_as_float((uint32_t)q16[off0] << 16), __uint_as_float((uint32_t)k16[off0] << 16));
        } else {
          z[u] = make_float2(q32[off0], k32[off0]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const int it = base + u * nthreads + tid;
      if (it < totalZ) Z[it] = ADJ ? make_float2(z[u].x * sc[u].x, z[u].y * sc[u].y) : z[u];
    }
  }
  // 2. forward DFT of every column
  dft_any<-1>(lg, Z, tw, colsZ, a.mz, tid, nthreads);
  const int R1 = Nf / radix2_of(lg), R2 = radix2_of(lg);
  auto row_of = [&](int f) { return R2 * (f & (R1 - 1)) + (f / R1); };  // row of frequency f

  // 3. gather and contract: point p = (w, c) on lanes 2p, 2p + 1 of each
  // part (a part has a lane for every point; lanes past the last point repeat
  // point 0 and write the trash row).  Every part gathers the same inputs and
  // takes its own phases |M|: a lane's chain of dependent operations is what
  // the block waits for here.
  {
    const int npts = ((Nf >> 1) + 1) * cc;
    // (compared, not divided: two integer divisions ahead of the gather cost
    // 0.5 us of a launch)
    const int lanes = a.lanes;  // whole waves
    const int part = __builtin_amdgcn_readfirstlane((tid >= lanes) + (tid >= 2 * lanes) + (tid >= 3 * lanes));
    const uint32_t phases = part < 2 ? (part == 0 ? a.phases[0] : a.phases[1]) : (part == 2 ? a.phases[2] : a.phases[3]);
    const int lt = tid - part * lanes;
    const int half = lt & 1;
    const int p = lt >> 1;
    const bool valid = p < npts;
    const int pc = valid ? p : 0;
    const int w = pc >> a.lcc, c = pc & (cc - 1);
    const int wn = (Nf - w) & (Nf - 1);
    const float g = half ? -1.f : 1.f;
    constexpr int H = (L + 1) * (L + 2) / 2;
    float2 q[H], k[H];
    {
      const float2* zv = Z + row_of(half ? wn : w) * colsZ + c;
      const float2* zu = Z + row_of(half ? w : wn) * colsZ + c;
#pragma unroll
      for (int l = 0; l <= L; ++l) {
        mirror_unpack0(l, g, zv[(l * l + l) * cc], zu[(l * l + l) * cc], q[l * (l + 1) / 2], k[l * (l + 1) / 2]);
#pragma unroll
        for (int m = 1; m <= l; ++m) {
          const int ic = (l * l + l + m) * cc, is = (l * l + l - m) * cc, h = l * (l + 1) / 2 + m;
          mirror_unpack(l, g, zv[ic], zu[ic], zv[is], zu[is], q[h], k[h]);
        }
      }
#pragma unroll
      for (int h = 0; h < H; ++h)  // opaque: not recomputed from the LDS values
        asm volatile("" : "+v"(q[h].x), "+v"(q[h].y), "+v"(k[h].x), "+v"(k[h].y));
    }
    __syncthreads();  // every lane has gathered: the output tile may overwrite Z
    SmallStore st;
    st.V = Z;
    st.K = K;
    st.cq = cq;
    st.ci = c >> 1;
    st.even = (c & 1) == 0;
    st.g = g;
    // the odd channel of the self-paired frequencies 0 and Nf/2 would write
    // row w again with the conjugate: it writes the trash row instead
    const bool write = valid && (st.even || wn != w);
    st.row = write ? (st.even ? w : wn) : Nf;
    CgMirrorBody<L>::run(q, k, st, phases);
  }
  // 5. inverse DFT of every packed column, scale and store (time n at row
  // R2 (n mod R1) + n / R1)
  dft_any<1>(lg, Z, tw, colsV, a.mv, tid, nthreads);
  const float inv = 1.0f / (float)Nf;
  const long long out_b = (long long)b * a.out_rows * K * a.C;
  const int totalV = a.out_rows * colsV;
  const bool even_c = (a.C & 1) == 0;
#pragma unroll 1  // four at a time: 0.1 us more per launch, nothing gained at any length
  for (int it = tid; it < totalV; it += nthreads) {
    const int n = divm(it, a.mv), col = it - n * colsV;
    const int k = col >> (a.lcc - 1), pi = col & (cq - 1);
    float2 v = Z[row_of(n) * colsV + col];
    v.x *= inv;
    v.y *= inv;
    if constexpr (ADJ) {
      const float so = pr.scales[2 * K + k];
      v.x *= so;
      v.y *= so;
    }
    const int ch = c0 + 2 * pi;
    const uint32_t off = ((uint32_t)n * K + k) * (uint32_t)a.C + ch;
    if (a.bf16) {
      uint16_t* o16 = static_cast<uint16_t*>(pr.out) + out_b;
      if (ch < a.C) o16[off] = f32_to_bf16_rne(v.x);
      if (ch + 1 < a.C) o16[off + 1] = f32_to_bf16_rne(v.y);
    } else {
      float* o = static_cast<float*>(pr.out) + out_b;
      if (even_c) {
        if (ch < a.C) *reinterpret_cast<float2*>(o + off) = v;  // ch and off are even
      } else {
        if (ch < a.C) o[off] = v.x;
        if (ch + 1 < a.C) o[off + 1] = v.y;
      }
    }
  }
}

}  // namespace

template <>
hipError_t launch_cg_small<CGCONV_TU_L>(const SmallArgs& a, hipStream_t s) {
  constexpr int K = (CGCONV_TU_L + 1) * (CGCONV_TU_L + 1);
  const int cc = 1 << a.lcc;
  if (a.Nf < 2 || a.Nf > kSmallMaxNf || (1 << a.lg) != a.Nf || a.lcc < 1 || a.lcc > 4 || a.cc != cc ||
      a.threads < 64 || a.threads > small_max_threads(CGCONV_TU_L) || (a.threads & 63) ||
      a.parts < 1 || a.parts > kSmallMaxParts || a.lanes * a.parts != a.threads || (a.lanes & 63) ||
      2 * ((a.Nf / 2 + 1) * cc) > a.lanes || a.problems < 1 || a.problems > 2 || a.groups != (a.C + cc - 1) / cc || a.in_rows > a.Nf ||
      a.out_rows > a.Nf || a.mz != 0xFFFFFFFFu / (uint32_t)(K * cc) + 1 || a.mv != 0xFFFFFFFFu / (uint32_t)(K * cc / 2) + 1)
    return hipErrorInvalidValue;
  const bool adjoint = a.problem[0].scales != nullptr;  // (fp32 only; a forward is one problem)
  if (adjoint ? a.bf16 || (a.problems == 2 && !a.problem[1].scales) : a.problems != 1) return hipErrorInvalidValue;
  const size_t lds = ((size_t)a.Nf * K * cc + a.Nf) * sizeof(float2);
  if (lds > kSmallMaxLds) return hipErrorInvalidValue;
  // the phases of each part: the longest first, each to the part with the
  // least work so far
  SmallArgs args = a;
  using Body = cgdev::CgMirrorBody<CGCONV_TU_L>;
  long work[kSmallMaxParts] = {};
  unsigned left = (2u << CGCONV_TU_L) - 1;
  for (int i = 0; i < kSmallMaxParts; ++i) args.phases[i] = 0;
  while (left) {
    int mu = -1, part = 0;
    for (int m = 0; m <= CGCONV_TU_L; ++m)
      if ((left >> m & 1) && (mu < 0 || Body::kPhaseOps[m] > Body::kPhaseOps[mu])) mu = m;
    for (int i = 1; i < a.parts; ++i)
      if (work[i] < work[part]) part = i;
    work[part] += Body::kPhaseOps[mu];
    args.phases[part] |= 1u << mu;
    left &= ~(1u << mu);
  }
  const dim3 grid((unsigned)(a.B * a.groups), a.problems);
  if (adjoint)
    hipLaunchKernelGGL((cg_small_kernel<CGCONV_TU_L, true>), grid, dim3(a.threads), lds, s, args);
  else
    hipLaunchKernelGGL((cg_small_kernel<CGCONV_TU_L, false>), grid, dim3(a.threads), lds, s, args);
  return hipGetLastError();
}

// More dynamic LDS than the default 64 KB limit must be allowed once per
// device before the launch; the plan does it when it is created.
template <>
hipError_t prepare_cg_small<CGCONV_TU_L>(int lds_bytes) {
  for (const void* f : {reinterpret_cast<const void*>(&cg_small_kernel<CGCONV_TU_L, false>),
                        reinterpret_cast<const void*>(&cg_small_kernel<CGCONV_TU_L, true>)}) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace cgconv
