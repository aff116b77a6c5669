// Register-resident small DFTs shared by the FFT passes and the fused CG
// kernel.
#pragma once

#include <hip/hip_runtime.h>

namespace cgconv {
namespace dft {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}

// exp(2 pi i k / 32) for k = 0..31 is (c32[k], s32[k]); forward DFTs use the
// conjugate.  Used for the radix <= 32 register DFTs.
__device__ __forceinline__ constexpr float c32(int k) {
  constexpr float t[32] = {1.0f, 0.98078528040323044f, 0.92387953251128674f, 0.83146961230254524f,
                           0.70710678118654752f, 0.55557023301960222f, 0.38268343236508977f, 0.19509032201612826f,
                           0.0f, -0.19509032201612826f, -0.38268343236508977f, -0.55557023301960222f,
                           -0.70710678118654752f, -0.83146961230254524f, -0.92387953251128674f, -0.98078528040323044f,
                           -1.0f, -0.98078528040323044f, -0.92387953251128674f, -0.83146961230254524f,
                           -0.70710678118654752f, -0.55557023301960222f, -0.38268343236508977f, -0.19509032201612826f,
                           0.0f, 0.19509032201612826f, 0.38268343236508977f, 0.55557023301960222f,
                           0.70710678118654752f, 0.83146961230254524f, 0.92387953251128674f, 0.98078528040323044f};
  return t[k & 31];
}
__device__ __forceinline__ constexpr float s32(int k) { return c32(k - 8); }

constexpr int bitrev(int x, int bits) {
  int r = 0;
  for (int i = 0; i < bits; ++i) r |= ((x >> i) & 1) << (bits - 1 - i);
  return r;
}
constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// cos and sin of 2 pi k / R, folded to constants once k is one
__device__ __forceinline__ float cosr(int k, int R) { return (float)__builtin_cos(6.283185307179586476925 * k / R); }
__device__ __forceinline__ float sinr(int k, int R) { return (float)__builtin_sin(6.283185307179586476925 * k / R); }

// DFT of an odd prime length P from the sums and differences of x_j and
// x_{P-j}: (P-1)/2 pairs of outputs share their products.
template <int P, int DIR>
__device__ __forceinline__ void dft_prime(float2 (&x)[P]) {
  constexpr int H = (P - 1) / 2;
  float2 s[H], d[H];
  float2 sum = x[0];
#pragma unroll
  for (int j = 1; j <= H; ++j) {
    s[j - 1] = make_float2(x[j].x + x[P - j].x, x[j].y + x[P - j].y);
    d[j - 1] = make_float2(x[j].x - x[P - j].x, x[j].y - x[P - j].y);
    sum.x += s[j - 1].x;
    sum.y += s[j - 1].y;
  }
  float2 y[P];
#pragma unroll
  for (int f = 1; f <= H; ++f) {
    float2 a = x[0], b = make_float2(0.f, 0.f);  // a + DIR i b, a - DIR i b
#pragma unroll
    for (int j = 1; j <= H; ++j) {
      const float c = cosr(j * f % P, P), n = sinr(j * f % P, P);
      a.x = fmaf(c, s[j - 1].x, a.x);
      a.y = fmaf(c, s[j - 1].y, a.y);
      b.x = fmaf(n, d[j - 1].x, b.x);
      b.y = fmaf(n, d[j - 1].y, b.y);
    }
    const float g = DIR > 0 ? 1.f : -1.f;
    y[f] = make_float2(a.x - g * b.y, a.y + g * b.x);
    y[P - f] = make_float2(a.x + g * b.y, a.y - g * b.x);
  }
  x[0] = sum;
#pragma unroll
  for (int f = 1; f < P; ++f) x[f] = y[f];
}

// In-place DFT of R <= 32 values held in registers, natural order in and out:
// X[f] = sum_e x[e] exp(DIR * 2 pi i e f / R).  Powers of two: radix-2
// decimation in time with constant twiddles; multiplications by 1 and +-i
// are not emitted.  R = P Q with P = 3, 5 or 7 and Q a power of two: e = P e1
// + e0, f = f1 + Q f0, length-Q DFTs, the twiddles W_R^(e0 f1), length-P DFTs.
template <int R, int DIR>
__device__ __forceinline__ void dft_reg(float2 (&x)[R]) {
  if constexpr (R == 1) {
    return;
  } else if constexpr ((R & (R - 1)) != 0) {
    constexpr int P = R % 3 == 0 ? 3 : (R % 5 == 0 ? 5 : 7), Q = R / P;
    static_assert(R % P == 0 && (Q & (Q - 1)) == 0);
    float2 t[P][Q];
#pragma unroll
    for (int e0 = 0; e0 < P; ++e0) {
#pragma unroll
      for (int e1 = 0; e1 < Q; ++e1) t[e0][e1] = x[P * e1 + e0];
      dft_reg<Q, DIR>(t[e0]);
    }
#pragma unroll
    for (int f1 = 0; f1 < Q; ++f1) {
      float2 u[P];
#pragma unroll
      for (int e0 = 0; e0 < P; ++e0) {
        u[e0] = t[e0][f1];
        if (e0 * f1 > 0)
          u[e0] = cmul(u[e0], make_float2(cosr(e0 * f1, R), DIR > 0 ? sinr(e0 * f1, R) : -sinr(e0 * f1, R)));
      }
      dft_prime<P, DIR>(u);
#pragma unroll
      for (int f0 = 0; f0 < P; ++f0) x[f1 + Q * f0] = u[f0];
    }
  } else {
    constexpr int B = ilog2(R);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int r = bitrev(i, B);
      if (r > i) {
        const float2 t = x[i];
        x[i] = x[r];
        x[r] = t;
      }
    }
#pragma unroll
    for (int len = 2; len <= R; len <<= 1) {
      const int half = len / 2;
#pragma unroll
      for (int i = 0; i < R; i += len) {
#pragma unroll
        for (int k = 0; k < half; ++k) {
          const int tk = k * (32 / len);  // exp(DIR 2 pi i k / len) = w32^(DIR tk)
          float2 b = x[i + k + half];
          if (tk == 0) {
          } else if (tk == 8) {
            // multiply by DIR * i
            b = DIR > 0 ? make_float2(-b.y, b.x) : make_float2(b.y, -b.x);
          } else {
            const float2 w = make_float2(c32(tk), DIR > 0 ? s32(tk) : -s32(tk));
            b = cmul(b, w);
          }
          const float2 a = x[i + k];
          x[i + k] = make_float2(a.x + b.x, a.y + b.y);
          x[i + k + half] = make_float2(a.x - b.x, a.y - b.y);
        }
      }
    }
  }
}

}  // namespace dft
}  // namespace cgconv
