"""The generated contraction bodies evaluated on the CPU (no GPU): the code
generator's output is compiled as host C++ with double precision in place of
float and compared with the plan's host contraction of the same table
(cgconv_contract_host), which is itself pinned to the oracle's dense tensor.
The mirror lane-pair body runs with both lanes of a point side by side: a
value is a pair of doubles, one per lane, and the lane swap exchanges them.
The channel-pairs body runs with the 64 lanes of a wave side by side: a value
is 64 doubles, the 4x4x1 matrix instruction its 16 outer products.
"""

import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2509_24093_amd as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_24093_amd", "csrc")

pytestmark = pytest.mark.skipif(not os.path.exists(P.LIB_PATH), reason="libcgconv.so not built")

PRELUDE = r"""
#include <cmath>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_sched_barrier(x)
struct V { double a, b; V() = default; V(double x) : a(x), b(x) {} V(double x, double y) : a(x), b(y) {} };
static inline V operator*(V x, V y) { return V(x.a * y.a, x.b * y.b); }
static inline V operator+(V x, V y) { return V(x.a + y.a, x.b + y.b); }
static inline V operator-(V x, V y) { return V(x.a - y.a, x.b - y.b); }
static inline V operator-(V x) { return V(-x.a, -x.b); }
static inline V vfma(V x, V y, V z) { return x * y + z; }
template <int ID> static inline V mul_here(V x, V y) { return x * y; }
static inline V fnma(V x, V y, V z) { return z - x * y; }
#define float V
#define fmaf vfma
struct float2 { V x, y; };
static inline float2 make_float2(V x, V y) { return {x, y}; }
static inline V sw(V v) { return V(v.b, v.a); }
static inline V lane_partner(V v) { return sw(v); }
static inline float2 lane_partner2(float2 v) { return {sw(v.x), sw(v.y)}; }
static inline void lane_partner4(float2 a, float2 b, float2& pa, float2& pb) { pa = lane_partner2(a); pb = lane_partner2(b); }
template <int L> struct CgBody;
template <int L> struct CgRealBody;
template <int L> struct CgMirrorBody;
template <int L> struct CgPathSplitBody;
"""

DRIVER = r"""
// mirror body: x = qa, ka in the complex-m basis (K complex values each), out = U (K complex values)
struct MStore {
  double* out;
  void put(int J, int mu, float2 acc) {
    const double s = (J & 1) ? -1 : 1;
    const double wpx = acc.x.a, wpy = acc.y.a, wmx = s * acc.x.b, wmy = s * acc.y.b;
    double* p = out + 2 * (J * J + J + mu);
    if (mu == 0) { p[0] = wpx + wmx; p[1] = wpy + wmy; return; }
    double* n = out + 2 * (J * J + J - mu);
    p[0] = wpx + wmx; p[1] = wpy + wmy;
    n[0] = -(wpy - wmy); n[1] = wpx - wmx;
  }
  void end_phase(int) {}
};
extern "C" void mirror(const double* qa, const double* ka, double* out) {
  constexpr int H = (LL + 1) * (LL + 2) / 2;
  float2 q[H], k[H];
  for (int l = 0; l <= LL; ++l)
    for (int m = 0; m <= l; ++m) {
      const int p = 2 * (l * l + l + m), n = 2 * (l * l + l - m), h = l * (l + 1) / 2 + m;
      const double s = (l & 1) ? -1 : 1;
      q[h] = {V(qa[p], s * qa[n]), V(qa[p + 1], s * qa[n + 1])};
      k[h] = {V(ka[p], s * ka[n]), V(ka[p + 1], s * ka[n + 1])};
    }
  MStore st{out};
  CgMirrorBody<LL>::run(q, k, st);
}
// token-wise product of real components
extern "C" void real(const double* a, const double* b, double* f) {
  constexpr int K = (LL + 1) * (LL + 1);
  V x[K], y[K], z[K];
  for (int i = 0; i < K; ++i) { x[i] = V(a[i]); y[i] = V(b[i]); }
  CgRealBody<LL>::run(x, y, z);
  for (int i = 0; i < K; ++i) f[i] = z[i].a;
}
"""


@pytest.fixture(scope="module")
def bodies(tmp_path_factory):
    d = tmp_path_factory.mktemp("bodies")
    subprocess.run(["g++", "-O1", "-std=c++17", os.path.join(CSRC, "codegen", "gen_cg.cpp"),
                    os.path.join(CSRC, "cg_table.cpp"), "-o", str(d / "gen")], check=True)
    subprocess.run([str(d / "gen"), str(d), "8"], check=True, capture_output=True)

    def load(L):
        src = d / f"b{L}.cpp"
        src.write_text(PRELUDE + f'#define LL {L}\n#include "cg_body_L{L}.inc"\n#undef float\n' + DRIVER)
        so = d / f"b{L}.so"
        subprocess.run(["g++", "-O0", "-std=c++17", "-w", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
        return ctypes.CDLL(str(so))

    return load


def _complex_basis(L, x):
    """2x in the complex-m basis: a[l,-mu] = x_c + i x_s, a[l,+mu] = x_c - i x_s."""
    a = np.array(2 * x)
    for l in range(1, L + 1):
        for mu in range(1, l + 1):
            c, s = l * l + l + mu, l * l + l - mu
            a[s], a[c] = 2 * (x[c] + 1j * x[s]), 2 * (x[c] - 1j * x[s])
    return a


def _ptr(a):
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))


@pytest.mark.parametrize("L", [0, 1, 2, 5, 7, 8])
def test_mirror_body_is_the_host_contraction(L, bodies):
    lib = bodies(L)
    rng = np.random.default_rng(40 + L)
    K = (L + 1) ** 2
    for _ in range(2):
        q = rng.normal(size=K) + 1j * rng.normal(size=K)
        k = rng.normal(size=K) + 1j * rng.normal(size=K)
        qa, ka = _complex_basis(L, q), _complex_basis(L, k)
        out = np.zeros(K, dtype=np.complex128)
        lib.mirror(_ptr(qa), _ptr(ka), _ptr(out))
        ref = P.cgconv_contract_host(L, q, k)
        # the emitted coefficients are rounded to float (2^-24 each)
        assert np.abs(out - ref).max() < 2e-7 * np.abs(ref).max() * np.sqrt(K)


@pytest.mark.parametrize("L", [0, 1, 2, 3, 5, 6, 8])
def test_real_body_is_the_real_table(L, bodies):
    lib = bodies(L)
    rng = np.random.default_rng(70 + L)
    K = (L + 1) ** 2
    idx, coef = P.cgconv_cg_table(L)
    x = idx[:, 0] ** 2 + idx[:, 0] + idx[:, 1]
    y = idx[:, 2] ** 2 + idx[:, 2] + idx[:, 3]
    o = idx[:, 4] ** 2 + idx[:, 4] + idx[:, 5]
    for _ in range(2):
        a, b = rng.normal(size=K), rng.normal(size=K)
        f = np.zeros(K)
        lib.real(_ptr(a), _ptr(b), _ptr(f))
        ref = np.bincount(o, weights=coef * a[x] * b[y], minlength=K)
        assert np.abs(f - ref).max() < 2e-7 * np.abs(ref).max() * np.sqrt(K)


# A wave of the inter-channel kernel: lane = c2 * 8 + c1.  The matrix
# instruction's blocks are groups of four lanes; A holds a row per lane, B a
# column per lane, D[r] row r of the lane's column.  cbsz = 1 takes A from block
# abid of each pair of blocks.
PAIRS_PRELUDE = r"""
#include <array>
#include <vector>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_sched_barrier(x)
#define __builtin_amdgcn_mfma_f32_4x4x1f32 mfma441
struct W {
  std::vector<double> v;
  W() : v(64) {}
  W(double x) : v(64, x) {}
};
template <class F> static W each(F f) { W r; for (int i = 0; i < 64; ++i) r.v[i] = f(i); return r; }
static W operator*(const W& x, const W& y) { return each([&](int i) { return x.v[i] * y.v[i]; }); }
static W operator+(const W& x, const W& y) { return each([&](int i) { return x.v[i] + y.v[i]; }); }
static W operator-(const W& x, const W& y) { return each([&](int i) { return x.v[i] - y.v[i]; }); }
static W operator-(const W& x) { return each([&](int i) { return -x.v[i]; }); }
static W vfma(const W& x, const W& y, const W& z) { return each([&](int i) { return x.v[i] * y.v[i] + z.v[i]; }); }
#define float W
#define fmaf vfma
struct float2 { W x, y; };
static float2 make_float2(const W& x, const W& y) { return {x, y}; }
struct v4f {
  std::array<W, 4> e;
  v4f() {}
  v4f(double a, double b, double c, double d) : e{W(a), W(b), W(c), W(d)} {}
  W& operator[](int i) { return e[i]; }
};
static v4f mfma441(const W& a, const W& b, v4f c, int cbsz, int abid, int) {
  for (int r = 0; r < 4; ++r)
    for (int l = 0; l < 64; ++l) {
      const int block = l / 4, from = (block >> cbsz << cbsz) + (cbsz ? abid : block & ((1 << cbsz) - 1));
      c.e[r].v[l] += a.v[4 * from + r] * b.v[l];
    }
  return c;
}
template <int L> struct CgBody;
template <int L> struct CgRealBody;
template <int L> struct CgMirrorBody;
template <int L> struct CgPathSplitBody;
template <int L> struct CgPairsBody;
#define CGCONV_PAIRS_BODY
"""

PAIRS_DRIVER = r"""
struct Tab {  // entry e: four coefficients of each of the four lane roles
  const double* t;
  Tab fresh() const { return *this; }
  v4f at(int e) const {
    v4f r;
    for (int i = 0; i < 4; ++i)
      r.e[i] = each([&](int l) { return t[16 * e + 4 * (((l >> 2) & 1) * 2 + ((l >> 1) & 1)) + i]; });
    return r;
  }
};
struct PStore {
  double* out;  // [K][64] complex
  int phases = 0;
  void operator()(int k, const float2& u) {
    for (int l = 0; l < 64; ++l) { out[2 * (64 * k + l)] = u.x.v[l]; out[2 * (64 * k + l) + 1] = u.y.v[l]; }
  }
  void end_phase(int mu) { phases = phases == mu ? mu + 1 : -1000; }
};
// q, k: [8 channels][K] complex, 2Q and 2K in the complex-m basis; degrees of odd l times i
extern "C" int pairs(const double* q, const double* k, const double* table, double* out) {
  constexpr int K = (LL + 1) * (LL + 1);
  float2 qa[K];
  W kp[K];
  for (int l = 0; l <= LL; ++l)
    for (int i = l * l; i < (l + 1) * (l + 1); ++i)
      for (int lane = 0; lane < 64; ++lane) {
        const double *a = q + 2 * (K * (lane & 7) + i), *b = k + 2 * (K * (lane >> 3) + i);
        const bool im = lane & 1, odd = l & 1;
        qa[i].x.v[lane] = odd ? -a[1] : a[0];
        qa[i].y.v[lane] = odd ? a[0] : a[1];
        kp[i].v[lane] = odd ? (im ? b[0] : -b[1]) : (im ? b[1] : b[0]);
      }
  PStore st{out};
  CgPairsBody<LL>::run(qa, kp, Tab{table}, st);
  return st.phases == LL + 1 ? CgPairsBody<LL>::kEntries : -1;
}
"""


@pytest.mark.parametrize("L", [0, 1, 2, 3, 6])
def test_pairs_body_is_the_host_contraction_of_every_pair(L, tmp_path):
    subprocess.run(["g++", "-O1", "-std=c++17", os.path.join(CSRC, "codegen", "gen_cg.cpp"),
                    os.path.join(CSRC, "cg_table.cpp"), "-o", str(tmp_path / "gen")], check=True)
    subprocess.run([str(tmp_path / "gen"), str(tmp_path), "8"], check=True, capture_output=True)
    body = (tmp_path / f"cg_body_L{L}.inc").read_text().split("#ifdef CGCONV_PAIRS_BODY")[1].split("\n", 1)[1]
    code, rest = body.split("static __device__ __attribute__((aligned(16))) const float pairs_table", 1)
    numbers = rest[rest.index("{") + 1:rest.index("}")].replace("f", "").replace("\n", "")
    table = np.array([float(x) for x in numbers.split(",") if x.strip()])
    src, so = tmp_path / "pairs.cpp", tmp_path / "pairs.so"
    src.write_text(PAIRS_PRELUDE + f"#define LL {L}\n" + code + "\n#undef float\n" + PAIRS_DRIVER)
    subprocess.run(["g++", "-O0", "-std=c++17", "-w", "-fno-exceptions", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    rng = np.random.default_rng(90 + L)
    K = (L + 1) ** 2
    q = rng.normal(size=(8, K)) + 1j * rng.normal(size=(8, K))
    k = rng.normal(size=(8, K)) + 1j * rng.normal(size=(8, K))
    qa, ka = (np.array([_complex_basis(L, x) for x in a]) for a in (q, k))
    out = np.zeros((K, 64), dtype=np.complex128)
    assert lib.pairs(_ptr(qa), _ptr(ka), _ptr(table), _ptr(out)) == len(table) // 16
    for c1 in range(8):
        for c2 in range(8):
            ref = P.cgconv_contract_host(L, q[c1], k[c2])
            # the coefficients are rounded to float (2^-24 each)
            assert np.abs(out[:, 8 * c2 + c1] - ref).max() < 2e-7 * np.abs(ref).max() * np.sqrt(K), (c1, c2)


def test_pairs_bodies_end_at_the_inter_channel_kernels(tmp_path):
    from paper_2509_24093_amd import build
    subprocess.run(["g++", "-O1", "-std=c++17", os.path.join(CSRC, "codegen", "gen_cg.cpp"),
                    os.path.join(CSRC, "cg_table.cpp"), "-o", str(tmp_path / "gen")], check=True)
    subprocess.run([str(tmp_path / "gen"), str(tmp_path), "8"], check=True, capture_output=True)
    emitted = [L for L in range(9) if "CgPairsBody" in (tmp_path / f"cg_body_L{L}.inc").read_text()]
    assert emitted == list(range(build.INTER_LMAX + 1))
