// Inter-channel CG stage with a per-degree channel reduction, for gfx950
// (arXiv 2509.24093 §4.1: within a head every query channel c1 meets every
// key channel c2, (2J+1) m m components per degree, and the multiplicity is
// reduced by a learned equivariant map, read as one matrix per head and
// output degree):
//
//   out[(J,M), h m_o + o] = sum_{c1,c2} W[h][J][o][c1 m + c2] u[(J,M), h, c1, c2]
//
// at every frequency, u being the CG product of the spectra of query channel
// h m + c1 and key channel h m + c2 (the reduction is linear, so it commutes
// with the inverse transform).  Runs between the unfused forward passes and
// the unfused inverse passes.
//
// Block = one batch element, one head and 8 frequency points w in [0, N/2];
// wave = point, lane = pair slot c2*8 + c1 (m <= 8; a slot with c1 or c2 >= m
// holds zeros and meets zero weights).  The block loads the head's spectra at
// w and N - w of its points into LDS once; each lane keeps 2Q of query channel
// c1 and one part (real or imaginary) of 2K of key channel c2, both in the
// complex-m basis, and the generated CgPairsBody contracts every pair: the
// coefficients are applied once per key channel and the sums over the query
// components run as 4x4x1 outer products on the matrix cores, in fp32.
// Bound by the issue of those 2424 matrix instructions and 2.8k vector
// operations per wave (L_max = 6), two waves per SIMD; one pair per lane took
// 18.9k vector operations.  The two kinds share the FMA hardware and alternate
// at about 1.2 times the sum of their own times.  Measured, stage alone, one
// pair per lane -> this form (B=8 N=16384, 4 heads of 8 channels): L_max = 6
// 7.11 -> 6.82 ms, 3 1.01 -> 0.99 ms, 1 259 -> 192 us; B=1 N=512 L_max = 6
// 76 -> 55 us.
// Every output component is parked in LDS per output phase; after the phase
// the matrix cores reduce the 64 pair values of each component with the
// degree's matrix, v_mfma_f32_16x16x4f32 in fp32 (A: rows o padded to 16,
// columns 4 pair slots per step, 16 steps; B: the parked values, columns
// (point, sign of M, re/im)), and the packed output W = U_o + i U_{o+1}
// goes to row w, conj U_o + i conj U_{o+1} to row N - w.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cg_common.h"

namespace cgconv {
namespace cgdev {
typedef float v4f __attribute__((ext_vector_type(4)));
#define CGCONV_PAIRS_BODY
#include CGCONV_BODY
}  // namespace cgdev

namespace {

using cgdev::CgPairsBody;
using cgdev::swap_pair;
using cgdev::v4f;

constexpr int kPts = 8;      // frequency points per block, one per wave
constexpr int kSlots = 64;   // channel-pair slots per point
constexpr int kThreadsI = kPts * kSlots;
constexpr int kWRows = kInterMmax;  // rows o of the reduction matrices held in LDS (m_out <= m)
// floats of a row of 64 pair slots (parked values, matrices): four more, so
// that the reduction's reads of neighbouring rows fall on distinct banks
constexpr int kPitch = kSlots + 4;

// This lane's column of the coefficient table in LDS: entry e holds four
// consecutive coefficients of each of the four lane roles.
typedef __attribute__((address_space(3))) const v4f lds_cv4;
struct LdsTable {
  lds_cv4* p;  // this lane's role of entry 0
  __device__ __forceinline__ v4f at(int e) const { return p[4 * e]; }
  // an opaque copy per pipeline step: its loads stay in the step
  __device__ __forceinline__ LdsTable fresh() const {
    LdsTable r = *this;
    asm volatile("" : "+v"(r.p));
    return r;
  }
};

template <int L>
struct InterGeo {
  static constexpr int K = (L + 1) * (L + 1);
  // most components of an even and of an odd output phase
  static constexpr int EVEN = L < 3 ? L + 1 : 2 * (L - 1), ODD = 2 * L;
  static constexpr int ROW = 2 * kPts * kPitch;  // floats of a component: [re, im][point][slot]
};

template <int L>
struct InterStore {
  static constexpr int K = InterGeo<L>::K, ROW = InterGeo<L>::ROW;
  float* T;         // LDS [EVEN + ODD][2][kPts][kPitch]: parked outputs, even phases first
  const float* Wl;  // LDS [L+1][kWRows][kPitch]: the head's matrices
  char* Wb;         // packed output spectra of this batch element (bytes)
  int N;
  RowMap rows;
  int F, w0, Cpo, co0, mo;
  int slot, pt, lane, wave;

  // Phases alternate between two areas, so that one barrier per phase is
  // enough: the area of phase mu is written again two phases on, after a
  // barrier that every wave reaches past its reduction of phase mu.
  __device__ __forceinline__ float* area(int mu) const { return T + ((mu & 1) ? InterGeo<L>::EVEN * ROW : 0); }

  // component kout = J^2 + J + M of phase mu = |M|: row ci within the
  // phase is J for mu = 0, 2 (J - mu) + (M < 0) otherwise
  __device__ __forceinline__ void operator()(int kout, float2 u) const {
    const int J = (int)__builtin_sqrtf((float)kout + 0.5f);
    const int M = kout - J * J - J, mu = M < 0 ? -M : M;
    const int ci = mu == 0 ? J : 2 * (J - mu) + (M < 0 ? 1 : 0);
    float* d = area(mu) + ci * ROW + pt * kPitch + slot;
    d[0] = u.x;
    d[kPts * kPitch] = u.y;
  }

  // Reduction of the phase's 64 pair values per component and point by the
  // degree's matrix, one degree and four points at a time per wave:
  // D[o][col] += A[o][pair] B[pair][col], columns (point, sign of M, re/im).
  // Step i of lane group kq takes pair 16 kq + i, so that a lane's operands of
  // the 16 steps are consecutive.  Rows o >= 8 of A repeat rows o - 8 and
  // columns of a missing sign (mu = 0) repeat another's: their results are not
  // stored.
  __device__ __forceinline__ void end_phase(int mu) const {
    __syncthreads();  // every lane has parked its outputs
    const int col = lane & 15, cpt = (wave & 4) + (col >> 2), sgn = (col >> 1) & 1, ri = col & 1;
    const int kq = lane >> 4;
    const int w = w0 + cpt, wn = w ? N - w : 0;
    const bool has = mu > 0 || sgn == 0;
    const bool store = has && w < F && !(ri == 1 && wn == w);  // one row for w = 0, N/2
    for (int J = mu + (wave & 3); J <= L; J += 4) {
      const int ci = mu == 0 ? J : 2 * (J - mu) + sgn;
      const v4f* wa = reinterpret_cast<const v4f*>(Wl + (J * kWRows + (col & 7)) * kPitch + 16 * kq);
      const v4f* tb = reinterpret_cast<const v4f*>(area(mu) + ci * ROW + (ri * kPts + cpt) * kPitch + 16 * kq);
      v4f av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        av[i] = wa[i];
        bv[i] = tb[i];
      }
      // two chains, even and odd steps
      v4f acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][0], bv[i][0], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][1], bv[i][1], acc1, 0, 0, 0);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][2], bv[i][2], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][3], bv[i][3], acc1, 0, 0, 0);
      }
      const v4f acc = acc0 + acc1;
      // this lane holds D[o = 4 kq + i][col], i = 0..3; lane ^ 1 holds the
      // other part (re/im) of the same complex value
      float other[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) other[i] = swap_pair(acc[i]);
      if (!store) continue;
      const int kout = J * J + J + (sgn ? -mu : mu);
      const long long row = rows.row(ri == 0 ? w : wn);
      float2* dst = reinterpret_cast<float2*>(Wb) + (row * K + kout) * Cpo;
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        const int o = 4 * kq + i;  // even: the channel pair (o, o + 1)
        if (o >= mo) continue;
        const float2 u0 = ri == 0 ? make_float2(acc[i], other[i]) : make_float2(other[i], acc[i]);
        const float2 u1 = ri == 0 ? make_float2(acc[i + 1], other[i + 1]) : make_float2(other[i + 1], acc[i + 1]);
        // row w: U_o + i U_{o+1};  row N - w: conj U_o + i conj U_{o+1}
        const float2 v = ri == 0 ? make_float2(u0.x - u1.y, u0.y + u1.x) : make_float2(u0.x + u1.y, u1.x - u0.y);
        dst[(co0 + o) >> 1] = v;
      }
    }
  }
};

// Highest L_max whose block takes several groups of points, keeping the table
// and the matrices and loading the next group's spectra during the
// contraction (L_max = 4, B=4 N=16384, 4 heads of 8: 1.16 -> 1.07 ms).  Above,
// those spectra no longer fit the registers (201 spilled at L_max = 6).
constexpr int kLoopLmax = 4;
constexpr long long kMinBlocks = 8 * 256;  // at least eight blocks per CU before a block takes a second group

template <int L>
__global__ __launch_bounds__(kThreadsI, L <= 3 ? 4 : 2) void cg_inter_kernel(InterArgs a) {
  constexpr int K = InterGeo<L>::K;
  using Body = CgPairsBody<L>;
  // the spectra of the block's points ([pt][w or N - w][k][channel of the
  // head], 2 kPts K kInterMmax values) until every lane has gathered its
  // own, then the parked outputs of the output phases
  constexpr int ZE = 2 * kPts * K * kInterMmax, TE = (InterGeo<L>::EVEN + InterGeo<L>::ODD) * InterGeo<L>::ROW;
  __shared__ __attribute__((aligned(16))) float sO[TE > 2 * ZE ? TE : 2 * ZE];
  __shared__ __attribute__((aligned(16))) float sW[(L + 1) * kWRows * kPitch];
  float2* const sT = reinterpret_cast<float2*>(sO);
  __shared__ __attribute__((aligned(16))) float sTab[Body::kEntries * 16];
  const int tid = threadIdx.x;
  const int ngroups = (a.F + kPts - 1) / kPts;
  const int nblocks = (ngroups + a.loop - 1) / a.loop;  // blocks of a (batch element, head)
  const int g0 = blockIdx.x % nblocks * a.loop, bh = blockIdx.x / nblocks;
  const int g1 = min(g0 + a.loop, ngroups);
  const int h = bh % a.H, b = bh / a.H;
  const int slot = tid & (kSlots - 1), pt = tid / kSlots;
  const int c1 = slot & 7, c2 = slot >> 3;
  const float2* Zb = a.Z + (long long)b * a.N * K * a.C + (long long)h * a.m;
  // the head's spectra at w and N - w of a group's points (64 contiguous
  // bytes per row and component; points past N/2 read row 0, channels past m
  // read zero)
  constexpr int NZ = (ZE + kThreadsI - 1) / kThreadsI;
  float2 z[NZ];
  auto load = [&](int g) {
    int t = tid;  // opaque: the addresses are computed here, not held across the loop
    if constexpr (L <= kLoopLmax) asm volatile("" : "+v"(t));
#pragma unroll
    for (int u = 0; u < NZ; ++u) {
      const int idx = u * kThreadsI + t;
      const int ch = idx % kInterMmax, k = (idx / kInterMmax) % K, side = (idx / (kInterMmax * K)) & 1,
                pl = idx / (2 * kInterMmax * K);
      const int wp = g * kPts + pl, wf = wp < a.F ? wp : 0;
      const long long row = a.rows.row(side && wf ? (int)a.N - wf : wf);
      z[u] = (idx < ZE && ch < a.m) ? Zb[(row * K + k) * a.C + ch] : make_float2(0.f, 0.f);
    }
  };
  // The first group's spectra, the coefficient table and the head's matrices
  // (rows o < mo and slots of real pairs, zeros elsewhere): every load is
  // issued before the first LDS store, so the block waits for one round trip
  // to memory.
  load(g0);
  {
    constexpr int NT = (Body::kEntries * 4 + kThreadsI - 1) / kThreadsI;
    constexpr int WE = (L + 1) * kWRows * kSlots, NW = (WE + kThreadsI - 1) / kThreadsI;
    const float* wh = a.wt + (long long)h * (L + 1) * a.mo * a.m * a.m;
    const v4f* tg = reinterpret_cast<const v4f*>(Body::table());
    float wv[NW];
    v4f tv[NT];
#pragma unroll
    for (int u = 0; u < NW; ++u) {
      const int idx = u * kThreadsI + tid;
      const int J = idx / (kWRows * kSlots), o = (idx / kSlots) % kWRows, s = idx % kSlots;
      const int s1 = s & 7, s2 = s >> 3;
      wv[u] = (idx < WE && o < a.mo && s1 < a.m && s2 < a.m) ? wh[((J * a.mo + o) * a.m + s1) * a.m + s2] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int idx = u * kThreadsI + tid;
      tv[u] = tg[idx < Body::kEntries * 4 ? idx : 0];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int idx = u * kThreadsI + tid;
      if (idx < Body::kEntries * 4) reinterpret_cast<v4f*>(sTab)[idx] = tv[u];
    }
#pragma unroll
    for (int u = 0; u < NW; ++u) {
      const int idx = u * kThreadsI + tid;
      if (idx < WE) sW[idx / kSlots * kPitch + idx % kSlots] = wv[u];
    }
  }
  for (int g = g0;;) {
    // the previous group's reductions have read the parked values
    if constexpr (L <= kLoopLmax) __syncthreads();
#pragma unroll
    for (int u = 0; u < NZ; ++u) {
      const int idx = u * kThreadsI + tid;
      if (idx < ZE) sT[idx] = z[u];
    }
    __syncthreads();
    // this lane's operands in the complex-m basis, degrees of odd l times i:
    // 2Q of channel c1, and of 2K of channel c2 the part of its row (real for
    // even lanes, imaginary for odd ones).  Channels past m hold zeros;
    // points past N/2 compute on row 0 and are not stored.
    float2 q[K];
    float kp[K];
    {
      const float2* za = sT + (pt * 2 + 0) * K * kInterMmax;
      const float2* zb = sT + (pt * 2 + 1) * K * kInterMmax;
      const bool im = (tid & 1) != 0;
      auto q2 = [&](int k) {
        const float2 A = za[k * kInterMmax + c1], B = zb[k * kInterMmax + c1];
        return make_float2(A.x + B.x, A.y - B.y);
      };
      auto k2 = [&](int k) {
        const float2 A = za[k * kInterMmax + c2], B = zb[k * kInterMmax + c2];
        return make_float2(A.y + B.y, B.x - A.x);
      };
      auto put = [&](int l, int k, float2 qv, float2 kv) {
        q[k] = (l & 1) ? make_float2(-qv.y, qv.x) : qv;
        kp[k] = (l & 1) ? (im ? kv.x : -kv.y) : (im ? kv.y : kv.x);
      };
#pragma unroll
      for (int l = 0; l <= L; ++l) {
        put(l, l * l + l, q2(l * l + l), k2(l * l + l));
#pragma unroll
        for (int m = 1; m <= l; ++m) {
          const int c = l * l + l + m, s = l * l + l - m;
          const float2 qc = q2(c), qs = q2(s), kc = k2(c), ks = k2(s);
          put(l, s, make_float2(qc.x - qs.y, qc.y + qs.x), make_float2(kc.x - ks.y, kc.y + ks.x));
          put(l, c, make_float2(qc.x + qs.y, qc.y - qs.x), make_float2(kc.x + ks.y, kc.y - ks.x));
        }
      }
#pragma unroll
      for (int k = 0; k < K; ++k) asm volatile("" : "+v"(q[k].x), "+v"(q[k].y), "+v"(kp[k]));
    }
    __syncthreads();  // every lane has gathered: the output phases reuse sT
    if constexpr (L <= kLoopLmax) {  // the next group's spectra load during the contraction
      if (g + 1 < g1) load(g + 1);
    }
    // role of this lane in the table: which x of a pair its half computes, and
    // which degree of a row pair
    const LdsTable tab{(lds_cv4*)(sTab) + ((tid >> 2) & 1) * 2 + ((tid >> 1) & 1)};
    InterStore<L> st;
    st.T = sO;
    st.Wl = sW;
    st.Wb = reinterpret_cast<char*>(a.W + (long long)b * a.N * K * a.Cpo);
    st.N = (int)a.N;
    st.rows = a.rows;
    st.F = a.F;
    st.Cpo = a.Cpo;
    st.co0 = h * a.mo;
    st.mo = a.mo;
    st.slot = slot;
    st.pt = pt;
    st.lane = tid & 63;
    st.wave = tid >> 6;
    st.w0 = g * kPts;
    Body::run(q, kp, tab, st);
    if (L > kLoopLmax || ++g == g1) break;
  }
}

}  // namespace

template <>
hipError_t launch_cg_inter<CGCONV_TU_L>(const InterArgs& a, hipStream_t s) {
  if (a.m < 1 || a.m > kInterMmax || a.mo < 2 || a.mo > kWRows || (a.mo & 1) || a.C != a.H * a.m || a.F < 1)
    return hipErrorInvalidValue;
  // groups of points per block: a block keeps the table and the matrices for
  // several groups while that leaves every CU several blocks
  const long long ngroups = (a.F + kPts - 1) / kPts, units = (long long)a.B * a.H * ngroups;
  InterArgs args = a;
  args.loop = CGCONV_TU_L > kLoopLmax ? 1 : (int)std::max(1LL, std::min(8LL, units / kMinBlocks));
  const long long blocks = (long long)a.B * a.H * ((ngroups + args.loop - 1) / args.loop);
  hipLaunchKernelGGL(cg_inter_kernel<CGCONV_TU_L>, dim3((unsigned)blocks), dim3(kThreadsI), 0, s, args);
  return hipGetLastError();
}

}  // namespace cgconv
