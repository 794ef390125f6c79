// Workgroup-cooperative complex FFT in LDS for gfx950 (wave64).
//
// Stockham auto-sort (each pass reads with stride L/R and writes with stride
// Ns, so the result lands in natural order without a bit-reversal pass).  A
// pass loads every butterfly input of the thread into registers, waits at a
// barrier, then writes its outputs back over the same LDS buffer, so one
// L-point buffer is enough.  Radices: 8, 4, 2 for the power-of-two part
// (as many 8s as possible, the remainder as 4s), then 5 and 3; 4096 and 5120
// take three passes of radix 16 (16, 20).  Twiddles
// come from a table of exp(-2 pi i m/L), m < L, computed in float64 on the
// host and rounded once to float32.
#pragma once

#include <hip/hip_runtime.h>

// Buffers in global memory are typed as such in device code, which keeps
// their loads and stores off the flat path (the host pass sees plain pointers).
#ifdef __HIP_DEVICE_COMPILE__
#define NR_G __attribute__((address_space(1)))
#else
#define NR_G
#endif
using TwPtr = const NR_G float2*;

namespace nrk {

__device__ __forceinline__ float2 c_add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 c_sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 c_mul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 c_scale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 c_conj(float2 a) { return make_float2(a.x, -a.y); }

// multiply by -i (forward transform) or +i (inverse transform)
template <bool INV>
__device__ __forceinline__ float2 mul_i(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// ---------------------------------------------------------------------------
// compile-time radix plan
// ---------------------------------------------------------------------------

constexpr int pow2_exponent(int v) {
  int e = 0;
  while (v > 1 && (v & 1) == 0) {
    v >>= 1;
    ++e;
  }
  return e;
}

// A transform is named by its length, plus kAdjointPlan for the adjoint's
// radices: 640 = 8 8 10 and 16 16 L/256 from 1024 to 2560 points, three passes
// through LDS where the general plan takes four.  Columns and rows in us per
// slice, four passes and three: 2560 10.0 + 6.4 and 8.8 + 6.1, 2048 6.9 + 3.5
// and 6.4 + 3.4, 1280 3.1 + 2.3 and 2.8 + 2.0, 1024 1.85 + 1.2 and 1.63 + 1.1,
// 640 1.75 + 1.17 and 1.62 + 1.12.  Shorter ones have too few butterflies of
// such a radix for a wavefront; 8192 points keep the general plan unmeasured.
// The adjoint's relative L2 error against 64 bits, four passes and three (means
// of six inputs, 1e-7): 640 points 5.11 and 5.10, 1024 5.18 and 5.24, 1280 5.17
// and 5.22, 2048 5.19 and 5.24, 2560 5.15 and 5.13 (a radix-16 butterfly
// multiplies by rounded roots where a radix-8 one mostly adds).  The forward
// keeps the general plan: other radices would change its last bits, and with
// them those of float64 objectives, which is a choice.
constexpr int kAdjointPlan = 1 << 20;
constexpr int fft_len(int L) { return L & (kAdjointPlan - 1); }
constexpr bool adjoint_plan_differs(int L) { return L == 640 || L == 1024 || L == 1280 || L == 2048 || L == 2560; }

constexpr int radix_of(int L, int p) {
  if (L & kAdjointPlan) {
    L = fft_len(L);
    if (adjoint_plan_differs(L)) {
      const int first = L == 640 ? 8 : 16;
      return p < 2 ? first : (p == 2 ? L / (first * first) : 1);
    }
  }
  // three passes for the two longest transforms of the 2560^2 and 2048^2
  // workloads: radix 16 and 20 butterflies in registers, one LDS round trip
  // per pass
  if (L == 5120) return p == 0 ? 16 : (p == 1 ? 16 : (p == 2 ? 20 : 1));
  if (L == 4096) return p < 3 ? 16 : 1;
  int r[24] = {};
  int n = 0;
  const int e = pow2_exponent(L);
  const int k = e / 3, rem = e % 3;
  if (rem == 0) {
    for (int i = 0; i < k; ++i) r[n++] = 8;
  } else if (rem == 1) {
    if (k >= 1) {
      for (int i = 0; i < k - 1; ++i) r[n++] = 8;
      r[n++] = 4;
      r[n++] = 4;
    } else {
      r[n++] = 2;
    }
  } else {
    for (int i = 0; i < k; ++i) r[n++] = 8;
    r[n++] = 4;
  }
  int o = L >> e;
  while (o % 5 == 0) {
    r[n++] = 5;
    o /= 5;
  }
  while (o % 3 == 0) {
    r[n++] = 3;
    o /= 3;
  }
  return p < n ? r[p] : 1;
}

constexpr int num_passes(int L) {
  int n = 0;
  while (radix_of(L, n) > 1) ++n;
  return n;
}

constexpr int span_before(int L, int p) {
  int s = 1;
  for (int i = 0; i < p; ++i) s *= radix_of(L, i);
  return s;
}

constexpr bool radix_plan_complete(int L) { return span_before(L, num_passes(L)) == fft_len(L); }

// ---------------------------------------------------------------------------
// small DFTs, X_k = sum_n x_n exp(-+2 pi i n k / R)
// ---------------------------------------------------------------------------

// HALF: only the inputs n < R/4 and n >= 3R/4 are non-zero (the others are
// not read).
template <int R, bool INV, bool HALF = false>
struct Dft;

template <bool INV>
struct Dft<2, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    const float2 a = v[0], b = v[1];
    v[0] = c_add(a, b);
    v[1] = c_sub(a, b);
  }
};

template <bool INV>
struct Dft<4, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    const float2 a0 = c_add(v[0], v[2]), a1 = c_sub(v[0], v[2]);
    const float2 a2 = c_add(v[1], v[3]), a3 = mul_i<INV>(c_sub(v[1], v[3]));
    v[0] = c_add(a0, a2);
    v[2] = c_sub(a0, a2);
    v[1] = c_add(a1, a3);
    v[3] = c_sub(a1, a3);
  }
};

template <bool INV>
struct Dft<4, INV, true> {
  __device__ __forceinline__ static void run(float2* v) {
    const float2 a = v[0];
    // (inputs that are products are rounded here, by the addition of zero, and
    // enter fused only where they did in the transform with zeros: v[1], v[3])
    const float2 r = round_product(v[0]), d = round_product(v[3]), q = mul_i<INV>(d);
    v[0] = c_add(r, d);
    v[2] = c_sub(r, d);
    v[1] = c_sub(a, q);
    v[3] = c_add(a, q);
  }
  __device__ __forceinline__ static float2 round_product(float2 x) { return make_float2(x.x + 0.f, x.y + 0.f); }
};

template <bool INV, bool HALF>
struct Dft<8, INV, HALF> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 e[4] = {v[0], v[2], v[4], v[6]};
    float2 o[4] = {v[1], v[3], v[5], v[7]};
    Dft<4, INV, HALF>::run(e);
    Dft<4, INV, HALF>::run(o);
    const float h = 0.70710678118654752440f;
    // W^1 = (1 -+ i)/sqrt(2), W^2 = -+i, W^3 = W^2 W^1
    const float2 o1 = INV ? make_float2((o[1].x - o[1].y) * h, (o[1].x + o[1].y) * h)
                          : make_float2((o[1].x + o[1].y) * h, (o[1].y - o[1].x) * h);
    const float2 o2 = mul_i<INV>(o[2]);
    const float2 o3t = INV ? make_float2((o[3].x - o[3].y) * h, (o[3].x + o[3].y) * h)
                           : make_float2((o[3].x + o[3].y) * h, (o[3].y - o[3].x) * h);
    const float2 o3 = mul_i<INV>(o3t);
    v[0] = c_add(e[0], o[0]);
    v[4] = c_sub(e[0], o[0]);
    v[1] = c_add(e[1], o1);
    v[5] = c_sub(e[1], o1);
    v[2] = c_add(e[2], o2);
    v[6] = c_sub(e[2], o2);
    v[3] = c_add(e[3], o3);
    v[7] = c_sub(e[3], o3);
  }
};

template <bool INV>
struct Dft<3, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    const float s3 = 0.86602540378443864676f;  // sin(2 pi/3)
    const float2 b = c_add(v[1], v[2]);
    const float2 t = make_float2(v[0].x - 0.5f * b.x, v[0].y - 0.5f * b.y);
    const float2 u = mul_i<INV>(c_scale(c_sub(v[1], v[2]), s3));
    v[0] = c_add(v[0], b);
    v[1] = c_add(t, u);
    v[2] = c_sub(t, u);
  }
};

template <bool INV>
struct Dft<5, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    const float c1 = 0.30901699437494742410f;   // cos(2 pi/5)
    const float c2 = -0.80901699437494742410f;  // cos(4 pi/5)
    const float s1 = 0.95105651629515357212f;   // sin(2 pi/5)
    const float s2 = 0.58778525229247312917f;   // sin(4 pi/5)
    const float2 b1 = c_add(v[1], v[4]), b2 = c_add(v[2], v[3]);
    const float2 d1 = c_sub(v[1], v[4]), d2 = c_sub(v[2], v[3]);
    const float2 t1 = make_float2(v[0].x + c1 * b1.x + c2 * b2.x, v[0].y + c1 * b1.y + c2 * b2.y);
    const float2 t2 = make_float2(v[0].x + c2 * b1.x + c1 * b2.x, v[0].y + c2 * b1.y + c1 * b2.y);
    const float2 u1 = mul_i<INV>(make_float2(s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y));
    const float2 u2 = mul_i<INV>(make_float2(s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y));
    v[0] = c_add(v[0], c_add(b1, b2));
    v[1] = c_add(t1, u1);
    v[4] = c_sub(t1, u1);
    v[2] = c_add(t2, u2);
    v[3] = c_sub(t2, u2);
  }
};

// cos and sin of 2 pi m / N for the composite butterflies below
template <int N>
struct UnitRoots;
template <>
struct UnitRoots<16> {
  static constexpr float c[16] = {1.f, 0.92387953251128674f, 0.70710678118654757f, 0.38268343236508984f,
                                  0.f, -0.38268343236508984f, -0.70710678118654757f, -0.92387953251128674f,
                                  -1.f, -0.92387953251128674f, -0.70710678118654757f, -0.38268343236508984f,
                                  0.f, 0.38268343236508984f, 0.70710678118654757f, 0.92387953251128674f};
  static constexpr float s[16] = {0.f, 0.38268343236508984f, 0.70710678118654757f, 0.92387953251128674f,
                                  1.f, 0.92387953251128674f, 0.70710678118654757f, 0.38268343236508984f,
                                  0.f, -0.38268343236508984f, -0.70710678118654757f, -0.92387953251128674f,
                                  -1.f, -0.92387953251128674f, -0.70710678118654757f, -0.38268343236508984f};
};
template <>
struct UnitRoots<10> {
  static constexpr float c[10] = {1.f, 0.80901699437494742f, 0.30901699437494742f, -0.30901699437494742f,
                                  -0.80901699437494742f, -1.f, -0.80901699437494742f, -0.30901699437494742f,
                                  0.30901699437494742f, 0.80901699437494742f};
  static constexpr float s[10] = {0.f, 0.58778525229247313f, 0.95105651629515357f, 0.95105651629515357f,
                                  0.58778525229247313f, 0.f, -0.58778525229247313f, -0.95105651629515357f,
                                  -0.95105651629515357f, -0.58778525229247313f};
};
template <>
struct UnitRoots<20> {
  static constexpr float c[20] = {1.f, 0.95105651629515357f, 0.80901699437494742f, 0.58778525229247313f,
                                  0.30901699437494742f, 0.f, -0.30901699437494742f, -0.58778525229247313f,
                                  -0.80901699437494742f, -0.95105651629515357f, -1.f, -0.95105651629515357f,
                                  -0.80901699437494742f, -0.58778525229247313f, -0.30901699437494742f, 0.f,
                                  0.30901699437494742f, 0.58778525229247313f, 0.80901699437494742f,
                                  0.95105651629515357f};
  static constexpr float s[20] = {0.f, 0.30901699437494742f, 0.58778525229247313f, 0.80901699437494742f,
                                  0.95105651629515357f, 1.f, 0.95105651629515357f, 0.80901699437494742f,
                                  0.58778525229247313f, 0.30901699437494742f, 0.f, -0.30901699437494742f,
                                  -0.58778525229247313f, -0.80901699437494742f, -0.95105651629515357f, -1.f,
                                  -0.95105651629515357f, -0.80901699437494742f, -0.58778525229247313f,
                                  -0.30901699437494742f};
};

// a * exp(-+2 pi i m/N) for an index m that is a constant once the calling
// loops are unrolled (the quarter turns are sign swaps)
template <int N, bool INV>
__device__ __forceinline__ float2 mul_root(float2 a, int m) {
  m %= N;
  if (m == 0) return a;
  if (4 * m == N) return mul_i<INV>(a);
  if (2 * m == N) return make_float2(-a.x, -a.y);
  if (4 * m == 3 * N) return mul_i<!INV>(a);
  const float c = UnitRoots<N>::c[m], sn = INV ? UnitRoots<N>::s[m] : -UnitRoots<N>::s[m];
  return make_float2(a.x * c - a.y * sn, a.x * sn + a.y * c);
}

// N = P*Q point DFT from P- and Q-point ones: input n = Q*n1 + n2, output
// k = k1 + P*k2; DFT_P over n1 for each n2, twiddles W_N^(n2*k1), DFT_Q over
// n2 for each k1.
template <int P, int Q, bool INV, bool HALF = false>
struct DftPQ {
  static_assert(!HALF || P == 4, "the zero inputs are whole quarters of the first stage");
  __device__ __forceinline__ static void run(float2* v) {
    float2 y[Q][P];
#pragma unroll
    for (int n2 = 0; n2 < Q; ++n2) {
      float2 t[P];
#pragma unroll
      for (int n1 = 0; n1 < P; ++n1) t[n1] = v[Q * n1 + n2];
      Dft<P, INV, HALF>::run(t);
#pragma unroll
      for (int k1 = 0; k1 < P; ++k1) y[n2][k1] = mul_root<P * Q, INV>(t[k1], n2 * k1);
    }
#pragma unroll
    for (int k1 = 0; k1 < P; ++k1) {
      float2 t[Q];
#pragma unroll
      for (int n2 = 0; n2 < Q; ++n2) t[n2] = y[n2][k1];
      Dft<Q, INV>::run(t);
#pragma unroll
      for (int k2 = 0; k2 < Q; ++k2) v[k1 + P * k2] = t[k2];
    }
  }
};

template <bool INV, bool HALF>
struct Dft<16, INV, HALF> : DftPQ<4, 4, INV, HALF> {};
template <bool INV>
struct Dft<10, INV> : DftPQ<5, 2, INV> {};
template <bool INV>
struct Dft<20, INV> : DftPQ<5, 4, INV> {};

// ---------------------------------------------------------------------------
// LDS buffer of one transform.  Element i lives at i ^ ((i >> 4) & 15): an
// XOR swizzle within blocks of 16 elements (128 bytes), so that the stride-R
// writes of the early passes (R = 8, 16: lanes 64 or 128 bytes apart, all on
// the same banks unswizzled) and the contiguous reads of the others both
// spread over the banks.  Counters put bank conflicts at 56 % of the LDS
// cycles of the 5120-point column transform unswizzled; swizzled, the
// transforms run 0-2 % faster (LDS is not their limit).  A bijection within
// each block, so L (a multiple of 16) elements still fill L slots.
// ---------------------------------------------------------------------------

template <int L>
constexpr int lds_elems() {
  return fft_len(L);
}

struct Lds {
  float2* p;
  __device__ __forceinline__ float2& operator[](int i) const { return p[i ^ ((i >> 4) & 15)]; }
  // Element base + c with c a constant once the calling loop is unrolled, a
  // multiple of 16: the swizzle of base + c depends on c only through
  // c / 16 mod 16, so the accesses of one butterfly (or of one thread's strided
  // loop) share one address per such class and take the rest of c as the
  // instruction's immediate offset.
  __device__ __forceinline__ float2& at(int base, int c) const {
    const int x = (base & ~15) | ((base ^ ((base >> 4) + (c >> 4))) & 15);
    return p[x + c];
  }
  // The same when base and c have no bits in common (and c may be any
  // constant): the swizzle is linear in the bits of the index, so the low byte
  // of c enters by one exclusive or and the rest is the immediate offset.
  __device__ __forceinline__ float2& at_disjoint(int base, int c) const {
    const int x = ((base ^ ((base >> 4) & 15)) * 8) ^ (((c & 255) ^ ((c >> 4) & 15)) * 8);   // bytes
    return *reinterpret_cast<float2*>(reinterpret_cast<char*>(p) + x + (c & ~255) * 8);
  }
};

constexpr bool is_pow2(int v) { return (v & (v - 1)) == 0; }

// element base + r STEP of a butterfly; DISJOINT: base shares no bits with any r STEP
template <int STEP, bool DISJOINT>
__device__ __forceinline__ float2& butterfly_elem(Lds s, int base, int r) {
  if constexpr (DISJOINT)
    return s.at_disjoint(base, r * STEP);
  else if constexpr (STEP % 16 == 0)
    return s.at(base, r * STEP);
  else
    return s[base + r * STEP];
}

// ---------------------------------------------------------------------------
// one Stockham pass and the whole transform
// ---------------------------------------------------------------------------

// Twiddles of a radix-R pass: w^r for r = 1..R-1 with w = e^{-2 pi i k/(Ns R)}.
// For R >= 8 only w and w^B are read from the table (B = ceil(sqrt(R))):
// w^b (b < B) and w^{aB} follow by repeated products, and w^{aB+b} =
// w^{aB} w^b, so a twiddle carries at most (B - 2) + (A - 2) + 1 extra
// roundings, A = ceil(R / B) (5 at R = 16, 6 at R = 20; parity at 2560^2
// does not change).  The table loads were most of a transform's
// vector-memory instructions: all R - 1 per butterfly ran the 5120-point
// column transforms at 53 us per slice, 2 run them at 45.5.
constexpr int tw_split(int R) {
  int b = 1;
  while (b * b < R) ++b;
  return b;
}

// w[r - 1] = tw[r st], r = 1..R-1 (w = tw[st] is e^{-2 pi i st/L}), as above
template <int R>
__device__ __forceinline__ void radix_twiddles(TwPtr __restrict__ tw, int st, float2 (&w)[R - 1]) {
  if constexpr (R >= 8) {
    constexpr int B = tw_split(R);
    constexpr int A = (R - 1) / B + 1;
    float2 lo[B], hi[A];
    lo[1] = tw[st];
    hi[1] = tw[B * st];
#pragma unroll
    for (int b = 2; b < B; ++b) lo[b] = c_mul(lo[b - 1], lo[1]);
#pragma unroll
    for (int a = 2; a < A; ++a) hi[a] = c_mul(hi[a - 1], hi[1]);
#pragma unroll
    for (int r = 1; r < R; ++r) {
      const int a = r / B, b = r % B;
      w[r - 1] = a == 0 ? lo[b] : (b == 0 ? hi[a] : c_mul(hi[a], lo[b]));
    }
  } else {
#pragma unroll
    for (int r = 1; r < R; ++r) w[r - 1] = tw[r * st];
  }
}

template <int L, int T, int P, bool INV>
__device__ __forceinline__ void fft_pass(Lds s, TwPtr __restrict__ tw, int tid) {
  constexpr int R = radix_of(L, P);
  constexpr int Ns = span_before(L, P);
  constexpr int NB = fft_len(L) / R;
  constexpr int PER = (NB + T - 1) / T;
  float2 v[PER][R];
  float2 w[PER][R - 1];
  // twiddles first (clamped index, no branch): their global loads overlap the
  // LDS reads and the barrier
  if constexpr (Ns > 1) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int j = (NB % T == 0 || tid + i * T < NB) ? tid + i * T : 0;
      const int k = j % Ns;
      radix_twiddles<R>(tw, k * (fft_len(L) / (Ns * R)), w[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = tid + i * T;
    if (NB % T == 0 || j < NB) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[i][r] = butterfly_elem<NB, is_pow2(NB)>(s, j, r);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = tid + i * T;
    if (NB % T == 0 || j < NB) {
      const int k = j % Ns;
      if constexpr (Ns > 1) {
#pragma unroll
        for (int r = 1; r < R; ++r) v[i][r] = c_mul(v[i][r], INV ? c_conj(w[i][r - 1]) : w[i][r - 1]);
      }
      Dft<R, INV>::run(v[i]);
      // base = k mod Ns below r Ns, a multiple of Ns R above it (0 in the last pass)
      const int base = (j - k) * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) butterfly_elem<Ns, is_pow2(Ns) && (is_pow2(R) || Ns * R == fft_len(L))>(s, base, r) = v[i][r];
    }
  }
  __syncthreads();
}

template <int L, int T, bool INV, int P = 0, int END = num_passes(L)>
__device__ __forceinline__ void fft_passes(Lds s, TwPtr __restrict__ tw, int tid) {
  if constexpr (P < END) {
    fft_pass<L, T, P, INV>(s, tw, tid);
    fft_passes<L, T, INV, P + 1, END>(s, tw, tid);
  }
}

// In-place length-L transform of the LDS buffer s by T threads.  Forward:
// X_k = sum_n x_n exp(-2 pi i nk/L); inverse: the + sign, unnormalised.
// The caller must have synchronised after filling s; on return s holds the
// result and the workgroup has synchronised.
template <int L, int T, bool INV>
__device__ __forceinline__ void fft_lds(Lds s, TwPtr __restrict__ tw, int tid) {
  static_assert(radix_plan_complete(L), "FFT length must be 2^a * 3^b * 5^c");
  fft_passes<L, T, INV>(s, tw, tid);
}

// A thread's butterflies of pass P in registers.
template <int L, int T, int P>
struct Regs {
  static constexpr int R = radix_of(L, P), NB = fft_len(L) / R, PER = (NB + T - 1) / T;
  float2 v[PER][R];
};

// The first pass takes its inputs from load(j, r) (input r of butterfly j,
// natural index j + r L/R; r is a constant once the loop is unrolled) straight
// into registers, and the workgroup synchronises after it.  With HALF, the
// input is a length-L/2 signal zero-padded to L and centred (non-zero only at
// natural indices [0, L/4) and [3L/4, L)): the zeros of each first-pass
// butterfly sit at fixed positions (inputs R/4 .. 3R/4 - 1), are not loaded and
// take no additions.

// Inputs of the first pass in registers.
template <int L, int T, class Load>
__device__ __forceinline__ void first_inputs(Regs<L, T, 0>& a, int tid, Load&& load) {
  constexpr int R = radix_of(L, 0), NB = fft_len(L) / R;
#pragma unroll
  for (int i = 0; i < Regs<L, T, 0>::PER; ++i) {
    const int j = tid + i * T;
    if (NB % T == 0 || j < NB) {
#pragma unroll
      for (int r = 0; r < R; ++r) a.v[i][r] = load(j, r);
    }
  }
}

// The first pass of the inputs in a, written to the LDS buffer.
template <int L, int T, bool INV>
__device__ __forceinline__ void first_pass_to_lds(Lds s, int tid, Regs<L, T, 0>& a) {
  constexpr int R = radix_of(L, 0), NB = fft_len(L) / R;
#pragma unroll
  for (int i = 0; i < Regs<L, T, 0>::PER; ++i) {
    const int j = tid + i * T;
    if (NB % T == 0 || j < NB) {
      Dft<R, INV>::run(a.v[i]);
#pragma unroll
      for (int r = 0; r < R; ++r) butterfly_elem<1, is_pow2(R)>(s, j * R, r) = a.v[i][r];
    }
  }
  __syncthreads();
}

// Both in one, a butterfly's loads next to its additions: a load that returns a
// product is then fused into them.
template <int L, int T, bool INV, bool HALF, class Load>
__device__ __forceinline__ void fft_first_pass_from(Lds s, int tid, Load&& load) {
  constexpr int R = radix_of(L, 0), NB = fft_len(L) / R;
  static_assert(!HALF || (R % 4 == 0 && fft_len(L) % 4 == 0), "the first radix must split the zero padding evenly");
#pragma unroll
  for (int i = 0; i < (NB + T - 1) / T; ++i) {
    const int j = tid + i * T;
    if (NB % T == 0 || j < NB) {
      float2 v[R];
#pragma unroll
      for (int r = 0; r < R; ++r)
        v[r] = (!HALF || r < R / 4 || r >= 3 * R / 4) ? load(j, r) : make_float2(0.f, 0.f);
      Dft<R, INV, HALF>::run(v);
#pragma unroll
      for (int r = 0; r < R; ++r) butterfly_elem<1, is_pow2(R)>(s, j * R, r) = v[r];
    }
  }
  __syncthreads();
}

// Transform of a length-L/2 signal zero-padded to L and centred, its input
// from load(j, r): the first pass as fft_first_pass_from with HALF, the rest as
// in fft_lds.  No LDS fill precedes it; on return s holds the result and the
// workgroup has synchronised.
template <int L, int T, bool INV, class Load>
__device__ __forceinline__ void fft_lds_halfzero(Lds s, TwPtr __restrict__ tw, int tid, Load&& load) {
  static_assert(radix_plan_complete(L), "FFT length must be 2^a * 3^b * 5^c");
  fft_first_pass_from<L, T, INV, true>(s, tid, load);
  fft_passes<L, T, INV, 1>(s, tw, tid);
}

// store(j, r, v[r]) for the outputs j + r NS of a last-pass butterfly; with
// HALF only those at [0, L/4) and [3L/4, L)
template <int L, int NS, int R, bool HALF, class Store>
__device__ __forceinline__ void store_kept(int j, const float2 (&v)[R], Store&& store) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if constexpr (HALF && R % 4 == 0) {
      if (r < R / 4 || r >= R - R / 4) store(j, r, v[r]);
    } else {
      const int n = j + r * NS;
      if (!HALF || n < fft_len(L) / 4 || n >= fft_len(L) - fft_len(L) / 4) store(j, r, v[r]);
    }
  }
}

// Transform whose last pass hands its outputs straight from registers to
// store(j, r, value) (natural index j + r Ns, Ns the span of the last pass,
// r a constant once the loop is unrolled) instead of writing the LDS buffer;
// with HALF only the outputs at [0, L/4) and [3L/4, L) (the centred half of
// the result) are handed over.  Passes START to the last but one run as in
// fft_lds (START = 1 after fft_first_pass_from).  Expects s to hold the
// input of pass START and the workgroup synchronised; leaves s holding the
// input of the last pass, and the caller must synchronise before writing s
// again.
template <int L, int T, bool INV, int START = 0, bool HALF = true, class Store>
__device__ __forceinline__ void fft_lds_store_out(Lds s, TwPtr __restrict__ tw, int tid, Store&& store) {
  static_assert(radix_plan_complete(L), "FFT length must be 2^a * 3^b * 5^c");
  constexpr int P = num_passes(L) - 1;
  constexpr int R = radix_of(L, P);
  constexpr int Ns = span_before(L, P);
  static_assert(Ns * R == fft_len(L) && P >= 1 && START <= P, "a transform of at least two passes");
  fft_passes<L, T, INV, START, P>(s, tw, tid);
  constexpr int PER = (Ns + T - 1) / T;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    // butterfly j of the last pass reads j + r Ns and yields outputs j + r Ns
    const int j = tid + i * T;
    if (Ns % T == 0 || j < Ns) {
      float2 v[R], w[R - 1];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = butterfly_elem<Ns, is_pow2(Ns)>(s, j, r);
      radix_twiddles<R>(tw, j, w);
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = c_mul(v[r], INV ? c_conj(w[r - 1]) : w[r - 1]);
      Dft<R, INV>::run(v);
      store_kept<L, Ns, R, HALF>(j, v, store);
    }
  }
}

// ---------------------------------------------------------------------------
// Split exchange: passes that keep the data in registers and hand it on
// through an L-float buffer, the real parts first and then the imaginary ones.
// Half the LDS of Lds for twice the barriers, so that more workgroups are
// resident.  For the transforms that end in registers (the adjoint's), whose
// 32 or 40 KB buffers otherwise admit five or four workgroups per CU.
// Measured on 2560^2 and 2048^2 slices, eight per launch (us per slice):
// adjoint columns 35.5 -> 33.3 and 21.9 -> 20.0, adjoint rows 24.8 -> 23.0 and
// 14.4 -> 14.1; shorter lengths, already at the wavefront limit, gain nothing.
// 8192 points (64 KB, two workgroups per CU) exchange whole values: the split is
// not measured there.
// Element i lives at i ^ ((i >> 5) & 15): the banks of 4-byte elements.
// ---------------------------------------------------------------------------
constexpr bool split_exchange_length(int L) { return L == 4096 || L == 5120; }

struct LdsF {
  float* p;
  __device__ __forceinline__ float& operator[](int i) const { return p[i ^ ((i >> 5) & 15)]; }
  // as Lds::at and Lds::at_disjoint; c of at() a multiple of 32
  __device__ __forceinline__ float& at(int base, int c) const {
    const int x = (base & ~15) | ((base ^ ((base >> 5) + (c >> 5))) & 15);
    return p[x + c];
  }
  __device__ __forceinline__ float& at_disjoint(int base, int c) const {
    const int x = ((base ^ ((base >> 5) & 15)) * 4) ^ (((c & 511) ^ ((c >> 5) & 15)) * 4);   // bytes
    return *reinterpret_cast<float*>(reinterpret_cast<char*>(p) + x + (c & ~511) * 4);
  }
};
template <int STEP, bool DISJOINT>
__device__ __forceinline__ float& butterfly_elem(LdsF s, int base, int r) {
  if constexpr (DISJOINT)
    return s.at_disjoint(base, r * STEP);
  else if constexpr (STEP % 32 == 0)
    return s.at(base, r * STEP);
  else
    return s[base + r * STEP];
}

// outputs of pass P (in a) -> inputs of pass P + 1 (in u)
template <int L, int T, int P>
__device__ __forceinline__ void split_exchange(LdsF s, int tid, const Regs<L, T, P>& a, Regs<L, T, P + 1>& u) {
  constexpr int R = radix_of(L, P), Ns = span_before(L, P), NB = fft_len(L) / R;
  constexpr int R1 = radix_of(L, P + 1), NB1 = fft_len(L) / R1;
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    if (part) __syncthreads();
#pragma unroll
    for (int i = 0; i < Regs<L, T, P>::PER; ++i) {
      const int j = tid + i * T;
      if (NB % T == 0 || j < NB) {
        const int k = j % Ns;
        const int base = (j - k) * R + k;
#pragma unroll
        for (int r = 0; r < R; ++r)
          butterfly_elem<Ns, is_pow2(Ns) && (is_pow2(R) || Ns * R == fft_len(L))>(s, base, r) = part ? a.v[i][r].y : a.v[i][r].x;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < Regs<L, T, P + 1>::PER; ++i) {
      const int j = tid + i * T;
      if (NB1 % T == 0 || j < NB1) {
#pragma unroll
        for (int r = 0; r < R1; ++r) {
          const float t = butterfly_elem<NB1, is_pow2(NB1)>(s, j, r);
          if (part) u.v[i][r].y = t;
          else u.v[i][r].x = t;
        }
      }
    }
  }
}

// passes P .. last on the outputs a of pass P - 1, then store(j, r, value) as
// in fft_lds_store_out
template <int L, int T, int P, bool INV, bool HALF, class Store>
__device__ __forceinline__ void split_passes(LdsF s, TwPtr __restrict__ tw, int tid, const Regs<L, T, P - 1>& a,
                                             Store&& store) {
  constexpr int R = radix_of(L, P), Ns = span_before(L, P), NB = fft_len(L) / R;
  Regs<L, T, P> u;
  split_exchange<L, T, P - 1>(s, tid, a, u);
#pragma unroll
  for (int i = 0; i < Regs<L, T, P>::PER; ++i) {
    const int j = tid + i * T;
    if (NB % T == 0 || j < NB) {
      const int k = j % Ns;
      float2 w[R - 1];
      radix_twiddles<R>(tw, k * (fft_len(L) / (Ns * R)), w);
#pragma unroll
      for (int r = 1; r < R; ++r) u.v[i][r] = c_mul(u.v[i][r], INV ? c_conj(w[r - 1]) : w[r - 1]);
      Dft<R, INV>::run(u.v[i]);
      if constexpr (P + 1 == num_passes(L)) store_kept<L, NB, R, HALF>(j, u.v[i], store);
    }
  }
  if constexpr (P + 1 < num_passes(L)) {
    __syncthreads();   // the exchange's last reads are done
    split_passes<L, T, P + 1, INV, HALF>(s, tw, tid, u, store);
  }
}

// The whole transform of the first pass's inputs a, its outputs handed to
// store(j, r, value) from registers, through lds (L float2; the split exchange
// uses half of it).
template <int L, int T, bool INV, bool SPLIT, class Store>
__device__ __forceinline__ void fft_store_out(float2* lds, TwPtr __restrict__ tw, int tid, Regs<L, T, 0>& a, Store&& store) {
  static_assert(radix_plan_complete(L), "FFT length must be 2^a * 3^b * 5^c");
  if constexpr (SPLIT) {
#pragma unroll
    for (int i = 0; i < Regs<L, T, 0>::PER; ++i) Dft<radix_of(L, 0), INV>::run(a.v[i]);
    split_passes<L, T, 1, INV, true>(LdsF{reinterpret_cast<float*>(lds)}, tw, tid, a, store);
  } else {
    first_pass_to_lds<L, T, INV>(Lds{lds}, tid, a);
    fft_lds_store_out<L, T, INV, 1>(Lds{lds}, tw, tid, store);
  }
}
template <int L, bool SPLIT>
constexpr int store_out_lds_elems() {
  return SPLIT ? fft_len(L) / 2 : lds_elems<L>();
}

// threads per transform for a length-L FFT.  For 5·2^a lengths five
// wavefronts split the radix-8 and radix-4 passes evenly (2560: 320 radix-8
// butterflies per pass; 5120: 640 and 1280), where four would leave the last
// round of each pass partly idle.
constexpr int fft_threads(int L) {
  return (L == 2560 || L == 5120) ? 320 : (L >= 2048 ? 256 : (L >= 512 ? 128 : 64));
}

// threads per transform of the adjoint's grid transforms: one or two of its
// wider butterflies a thread and pass
constexpr int adj_threads(int L) { return L == 1024 ? 64 : (L == 2048 ? 128 : (L == 2560 ? 256 : fft_threads(L))); }

}  // namespace nrk
