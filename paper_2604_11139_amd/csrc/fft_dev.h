// Device building blocks of the LDS-resident FFTs: DFTs of up to 15 points in
// registers, one Stockham stage over a set of pencils held in LDS, a 1D FFT
// from a radix plan, twiddle loading; and the host rule for the thread count
// of a stage.  Shared by the single-system passes and the batched passes.
#pragma once

#include <type_traits>
#include <utility>

#include "cplx.h"
#include "internal.h"

namespace chebfi {
namespace {

// butterflies per thread in one runtime-size stage of radix R: at most 20
// complex values held per thread (radix 2: 10, 3: 6, 4: 5, 5: 4), which takes
// every plane up to 96 x 96 in 512 threads
constexpr int kStageValues = 20;
__host__ __device__ constexpr int max_butterflies(int r) { return kStageValues / r; }

// Radix-R DFT in registers; sgn = -1 forward (e^{-}), +1 inverse (e^{+}).
template <typename T, int R> struct Dft;

template <typename T> struct Dft<T, 2> {
  static __device__ __forceinline__ void run(C2<T> *x, int) {
    C2<T> a = x[0], b = x[1];
    x[0] = cadd(a, b);
    x[1] = csub(a, b);
  }
};

template <typename T> struct Dft<T, 4> {
  static __device__ __forceinline__ void run(C2<T> *x, int sgn) {
    C2<T> s02 = cadd(x[0], x[2]), d02 = csub(x[0], x[2]);
    C2<T> s13 = cadd(x[1], x[3]), d13 = cmul_i(csub(x[1], x[3]), sgn);
    x[0] = cadd(s02, s13);
    x[2] = csub(s02, s13);
    x[1] = cadd(d02, d13);
    x[3] = csub(d02, d13);
  }
};

template <typename T> struct Dft<T, 3> {
  static __device__ __forceinline__ void run(C2<T> *x, int sgn) {
    const T h = (T)0.86602540378443864676;  // sin(2 pi / 3)
    C2<T> t1 = cadd(x[1], x[2]);
    C2<T> t2 = cmul_i(cscale(csub(x[1], x[2]), h), sgn);
    C2<T> m = csub(x[0], cscale(t1, (T)0.5));
    x[0] = cadd(x[0], t1);
    x[1] = cadd(m, t2);
    x[2] = csub(m, t2);
  }
};

template <typename T> struct Dft<T, 5> {
  static __device__ __forceinline__ void run(C2<T> *x, int sgn) {
    const T c1 = (T)0.30901699437494742410;   // cos(2 pi / 5)
    const T c2 = (T)-0.80901699437494742410;  // cos(4 pi / 5)
    const T s1 = (T)0.95105651629515357212;   // sin(2 pi / 5)
    const T s2 = (T)0.58778525229247312917;   // sin(4 pi / 5)
    C2<T> t1 = cadd(x[1], x[4]), t2 = cadd(x[2], x[3]);
    C2<T> t3 = csub(x[1], x[4]), t4 = csub(x[2], x[3]);
    C2<T> a1 = cadd(x[0], cadd(cscale(t1, c1), cscale(t2, c2)));
    C2<T> a2 = cadd(x[0], cadd(cscale(t1, c2), cscale(t2, c1)));
    C2<T> b1 = cmul_i(cadd(cscale(t3, s1), cscale(t4, s2)), sgn);
    C2<T> b2 = cmul_i(csub(cscale(t3, s2), cscale(t4, s1)), sgn);
    x[0] = cadd(x[0], cadd(t1, t2));
    x[1] = cadd(a1, b1);
    x[4] = csub(a1, b1);
    x[2] = cadd(a2, b2);
    x[3] = csub(a2, b2);
  }
};

template <typename T> struct Dft<T, 6> {
  // even/odd split: two radix-3 DFTs combined with w6^k = e^{sgn i pi k/3}
  static __device__ __forceinline__ void run(C2<T> *x, int sgn) {
    C2<T> e[3] = {x[0], x[2], x[4]}, o[3] = {x[1], x[3], x[5]};
    Dft<T, 3>::run(e, sgn);
    Dft<T, 3>::run(o, sgn);
    const T h = (T)0.86602540378443864676;
    const C2<T> w1{(T)0.5, (T)sgn * h}, w2{(T)-0.5, (T)sgn * h};
    const C2<T> t1 = cmul(o[1], w1), t2 = cmul(o[2], w2);
    x[0] = cadd(e[0], o[0]);
    x[3] = csub(e[0], o[0]);
    x[1] = cadd(e[1], t1);
    x[4] = csub(e[1], t1);
    x[2] = cadd(e[2], t2);
    x[5] = csub(e[2], t2);
  }
};

template <typename T> struct Dft<T, 9> {
  // 3 x 3: radix-3 DFTs of x[n2], x[n2+3], x[n2+6], twiddles w9^(n2 k1), then
  // radix-3 DFTs across n2 (output k1 + 3 k2), w9 = e^{sgn 2 pi i / 9}
  static __device__ __forceinline__ void run(C2<T> *x, int sgn) {
    C2<T> a[3][3];
#pragma unroll
    for (int n2 = 0; n2 < 3; ++n2) {
      a[n2][0] = x[n2];
      a[n2][1] = x[n2 + 3];
      a[n2][2] = x[n2 + 6];
      Dft<T, 3>::run(a[n2], sgn);
    }
    const T c1 = (T)0.76604444311897803520, s1 = (T)0.64278760968653932632;   // 2 pi / 9
    const T c2 = (T)0.17364817766693034885, s2 = (T)0.98480775301220805936;   // 4 pi / 9
    const T c4 = (T)-0.93969262078590838405, s4 = (T)0.34202014332566873304;  // 8 pi / 9
    a[1][1] = cmul(a[1][1], C2<T>{c1, (T)sgn * s1});
    a[1][2] = cmul(a[1][2], C2<T>{c2, (T)sgn * s2});
    a[2][1] = cmul(a[2][1], C2<T>{c2, (T)sgn * s2});
    a[2][2] = cmul(a[2][2], C2<T>{c4, (T)sgn * s4});
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) {
      C2<T> b[3] = {a[0][k1], a[1][k1], a[2][k1]};
      Dft<T, 3>::run(b, sgn);
      x[k1] = b[0];
      x[k1 + 3] = b[1];
      x[k1 + 6] = b[2];
    }
  }
};

template <typename T> struct Dft<T, 8> {
  // even/odd split: two radix-4 DFTs combined with w8^k = e^{sgn i pi k/4}
  static __device__ __forceinline__ void run(C2<T> *x, int sgn) {
    C2<T> e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
    Dft<T, 4>::run(e, sgn);
    Dft<T, 4>::run(o, sgn);
    const T c = (T)0.70710678118654752440;
    const C2<T> t1{c * (o[1].x - sgn * o[1].y), c * (o[1].y + sgn * o[1].x)};
    const C2<T> t2 = cmul_i(o[2], sgn);
    const C2<T> t3{c * (-o[3].x - sgn * o[3].y), c * (-o[3].y + sgn * o[3].x)};
    x[0] = cadd(e[0], o[0]);
    x[4] = csub(e[0], o[0]);
    x[1] = cadd(e[1], t1);
    x[5] = csub(e[1], t1);
    x[2] = cadd(e[2], t2);
    x[6] = csub(e[2], t2);
    x[3] = cadd(e[3], t3);
    x[7] = csub(e[3], t3);
  }
};

// Radix A*B DFT for coprime A and B without twiddles (Good 1958, Thomas 1963):
// input B n1 + A n2, output k1 eB + k2 eA (mod A B) with eB = 1 mod A, 0 mod B
// and eA = 0 mod A, 1 mod B; all indices are compile-time constants.
constexpr int idempotent(int a, int b) {  // multiple of b that is 1 mod a
  int e = b;
  while (e % a != 1) e += b;
  return e;
}
template <typename T, int A, int B> struct DftCoprime {
  static __device__ __forceinline__ void run(C2<T> *x, int sgn) {
    constexpr int N = A * B, eB = idempotent(A, B), eA = idempotent(B, A);
    C2<T> t[A][B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
      C2<T> a[A];
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) a[n1] = x[(B * n1 + A * n2) % N];
      Dft<T, A>::run(a, sgn);
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) t[k1][n2] = a[k1];
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      Dft<T, B>::run(t[k1], sgn);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) x[(k1 * eB + k2 * eA) % N] = t[k1][k2];
    }
  }
};
template <typename T> struct Dft<T, 10> : DftCoprime<T, 2, 5> {};
template <typename T> struct Dft<T, 12> : DftCoprime<T, 3, 4> {};
template <typename T> struct Dft<T, 15> : DftCoprime<T, 3, 5> {};

// One Stockham stage of radix R over `npen` pencils of length n held in LDS.
// Element e of pencil q sits at buf[q*pstride + e*estride].  p is the product
// of the radices already applied.
template <typename T, int R>
__device__ void stage(C2<T> *buf, int n, int estride, int npen, int pstride, int p,
                      const C2<T> *tw, int sgn) {
  const int nbf = n / R;
  const int total = npen * nbf;
  const int m = n / (p * R);
  constexpr int MB = max_butterflies(R);
  C2<T> y[MB][R];
  int dst[MB];
#pragma unroll
  for (int c = 0; c < MB; ++c) {
    const int i = threadIdx.x + c * blockDim.x;
    dst[c] = -1;
    if (i < total) {
      // consecutive lanes take consecutive pencils: with an odd pencil stride
      // (padded planes) or a unit one their accesses spread over all LDS banks
      const int pen = i % npen, bf = i / npen;
      const int base = pen * pstride;
      C2<T> x[R];
#pragma unroll
      for (int t = 0; t < R; ++t) x[t] = buf[base + (bf + t * nbf) * estride];
      const int k = bf % p;
#pragma unroll
      for (int t = 1; t < R; ++t) {
        C2<T> w = tw[t * k * m];
        if (sgn > 0) w.y = -w.y;
        x[t] = cmul(x[t], w);
      }
      Dft<T, R>::run(x, sgn);
#pragma unroll
      for (int t = 0; t < R; ++t) y[c][t] = x[t];
      dst[c] = base + ((bf - k) * R + k) * estride;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < MB; ++c) {
    if (dst[c] >= 0) {
#pragma unroll
      for (int t = 0; t < R; ++t) buf[dst[c] + t * p * estride] = y[c][t];
    }
  }
  __syncthreads();
}

template <typename T>
__device__ void lds_fft(C2<T> *buf, const Plan1D &pl, int estride, int npen, int pstride,
                        const C2<T> *tw, int sgn) {
  int p = 1;
  for (int s = 0; s < pl.nstage; ++s) {
    const int r = pl.radix[s];
    if (r == 4)
      stage<T, 4>(buf, pl.n, estride, npen, pstride, p, tw, sgn);
    else if (r == 2)
      stage<T, 2>(buf, pl.n, estride, npen, pstride, p, tw, sgn);
    else if (r == 3)
      stage<T, 3>(buf, pl.n, estride, npen, pstride, p, tw, sgn);
    else
      stage<T, 5>(buf, pl.n, estride, npen, pstride, p, tw, sgn);
    p *= r;
  }
}

template <typename T>
__device__ void load_twiddles(C2<T> *dst, const double2 *src, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = to_c2<T>(src[i]);
}


// Smallest multiple of 64 threads with at most max_butterflies(r) butterflies
// per thread in every stage of the plan over npen pencils.
inline int stage_need(const Plan1D &pl, int npen) {
  int need = 64;
  for (int s = 0; s < pl.nstage; ++s) {
    const int total = npen * (pl.n / pl.radix[s]);
    const int mb = max_butterflies(pl.radix[s]);
    const int t = (total + mb - 1) / mb;
    if (t > need) need = t;
  }
  return (need + 63) / 64 * 64;
}

// Threads of the runtime-size passes: 512 (the most a pass may use); the
// extra waves per CU hide the latency of the plane loads and stores.
inline int stage_threads(const Plan1D &pl, int npen) {
  const int need = stage_need(pl, npen);
  return need > 512 ? need : 512;
}

// ---- compile-time specialised passes ------------------------------------------
// Same three passes as above with the transform length N, the radix sequence,
// the pencil strides and the thread count known at compile time, so that all
// index arithmetic reduces to constant multiplies and shifts.  A plane sits in
// LDS with a row stride of N + 1 elements, and the lanes of a wave take
// consecutive pencils in both directions: pencils along a row are then an odd
// stride apart, which spreads a wave's accesses over all LDS banks.
template <int N> struct CPlan;
#define CHEBFI_CPLAN(N_, NS_, R0_, R1_, R2_)                              \
  template <> struct CPlan<N_> {                                          \
    static constexpr int ns = NS_;                                        \
    static constexpr int r[3] = {R0_, R1_, R2_};                          \
  };
CHEBFI_CPLAN(12, 2, 4, 3, 1)
CHEBFI_CPLAN(15, 2, 5, 3, 1)
CHEBFI_CPLAN(16, 2, 4, 4, 1)
CHEBFI_CPLAN(18, 2, 6, 3, 1)
CHEBFI_CPLAN(20, 2, 5, 4, 1)
CHEBFI_CPLAN(24, 2, 8, 3, 1)
CHEBFI_CPLAN(25, 2, 5, 5, 1)
CHEBFI_CPLAN(27, 2, 3, 9, 1)
CHEBFI_CPLAN(30, 2, 6, 5, 1)
CHEBFI_CPLAN(32, 2, 8, 4, 1)
CHEBFI_CPLAN(36, 2, 6, 6, 1)
CHEBFI_CPLAN(40, 2, 8, 5, 1)
CHEBFI_CPLAN(45, 2, 5, 9, 1)
CHEBFI_CPLAN(48, 2, 8, 6, 1)
CHEBFI_CPLAN(50, 2, 5, 10, 1)
CHEBFI_CPLAN(54, 2, 6, 9, 1)
CHEBFI_CPLAN(60, 2, 6, 10, 1)
CHEBFI_CPLAN(64, 2, 8, 8, 1)
CHEBFI_CPLAN(72, 2, 8, 9, 1)
CHEBFI_CPLAN(75, 2, 5, 15, 1)
CHEBFI_CPLAN(80, 2, 8, 10, 1)
CHEBFI_CPLAN(81, 2, 9, 9, 1)
CHEBFI_CPLAN(90, 2, 9, 10, 1)
CHEBFI_CPLAN(96, 2, 8, 12, 1)
#undef CHEBFI_CPLAN

// Threads of a pass over NPEN pencils of length N: one butterfly of the widest
// stage per thread, in as few rounds as keep the workgroup at 576 threads or
// fewer (a 36 x 36 plane has 216 radix-6 butterflies: 256 threads, not 512 of
// which 300 wait at every barrier).
template <int N, int NPEN>
constexpr int cthreads() {
  int w = 0;
  for (int i = 0; i < CPlan<N>::ns; ++i)
    if (NPEN * (N / CPlan<N>::r[i]) > w) w = NPEN * (N / CPlan<N>::r[i]);
  int k = 1;
  while ((w + k - 1) / k > 576) ++k;
  return ((w + k - 1) / k + 63) / 64 * 64;
}

// LDS row pitch of an N x N plane in the specialised passes: odd, so that the
// lanes of a wave walking consecutive pencils across rows (8-byte elements,
// row stride 2 cld dwords) meet every bank pair once: N + 1 for even N, N + 2
// for odd N (an even pitch such as 46 for N = 45 reaches only 16 banks).
template <int N>
constexpr int cld() {
  return N % 2 ? N + 2 : N + 1;
}

// One stage in place over NPEN pencils held in LDS, element e of pencil q at
// buf[q * PS + e * ES], by CT threads.
template <typename T, int N, int R, int P, int NPEN, int ES, int PS, int SGN, int CT>
__device__ __forceinline__ void cstage(C2<T> *buf, const C2<T> *tw) {
  constexpr int NBF = N / R;
  constexpr int TOTAL = NPEN * NBF;
  constexpr int M = N / (P * R);
  constexpr int MAXB = (TOTAL + CT - 1) / CT;
  C2<T> y[MAXB][R];
  int dst[MAXB];
#pragma unroll
  for (int c = 0; c < MAXB; ++c) {
    const int i = threadIdx.x + c * CT;
    dst[c] = -1;
    if (TOTAL % CT == 0 || i < TOTAL) {
      const int pa = i % NPEN, bf = i / NPEN;
      const int base = pa * PS;
      C2<T> x[R];
#pragma unroll
      for (int t = 0; t < R; ++t) x[t] = buf[base + (bf + t * NBF) * ES];
      const int k = bf % P;
      if (P > 1) {
#pragma unroll
        for (int t = 1; t < R; ++t) {
          C2<T> w = tw[t * k * M];
          if (SGN > 0) w.y = -w.y;
          x[t] = cmul(x[t], w);
        }
      }
      Dft<T, R>::run(x, SGN);
#pragma unroll
      for (int t = 0; t < R; ++t) y[c][t] = x[t];
      dst[c] = base + ((bf - k) * R + k) * ES;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < MAXB; ++c) {
    if (TOTAL % CT == 0 || dst[c] >= 0) {
#pragma unroll
      for (int t = 0; t < R; ++t) buf[dst[c] + t * P * ES] = y[c][t];
    }
  }
  __syncthreads();
}

template <typename T, int N, int S, int P, int NPEN, int ES, int PS, int SGN, int CT>
__device__ __forceinline__ void cfft(C2<T> *buf, const C2<T> *tw) {
  if constexpr (S < CPlan<N>::ns) {
    constexpr int R = CPlan<N>::r[S];
    cstage<T, N, R, P, NPEN, ES, PS, SGN, CT>(buf, tw);
    cfft<T, N, S + 1, P * R, NPEN, ES, PS, SGN, CT>(buf, tw);
  }
}

// One stage of the same Stockham FFT over NPEN pencils with its inputs taken
// from ld(pencil, element) and its outputs given to st(pencil, element,
// value): the first stage of a transform can read straight from global memory
// and the last one write straight to it (or fuse a pointwise product into its
// store), saving a pass of the plane through LDS.  SYNC_MID: a barrier
// between the reads and the writes (needed when both are the same LDS plane).
// Position of a thread's c-th butterfly of such a stage: pencil, and the element of
// its output 0 (output t is P elements further on per t); false past the last one.
template <int N, int R, int P, int NPEN, int CT>
__device__ __forceinline__ bool cstage_at(int c, int &pa, int &e0) {
  const int i = threadIdx.x + c * CT, bf = i / NPEN, k = bf % P;
  pa = i % NPEN;
  e0 = (bf - k) * R + k;
  return NPEN * (N / R) % CT == 0 || i < NPEN * (N / R);
}
template <int N, int R, int NPEN, int CT>
constexpr int cstage_rounds() {
  return (NPEN * (N / R) + CT - 1) / CT;
}

// The stage's outputs in registers, y[c][t] = output t of the c-th butterfly.
template <typename T, int N, int R, int P, int NPEN, int SGN, int CT, class Ld>
__device__ __forceinline__ void cstage_vals(const C2<T> *tw, Ld ld,
                                            C2<T> (&y)[cstage_rounds<N, R, NPEN, CT>()][R]) {
  constexpr int NBF = N / R, TOTAL = NPEN * NBF, M = N / (P * R);
#pragma unroll
  for (int c = 0; c < cstage_rounds<N, R, NPEN, CT>(); ++c) {
    const int i = threadIdx.x + c * CT;
    if (TOTAL % CT == 0 || i < TOTAL) {
      const int pa = i % NPEN, bf = i / NPEN, k = bf % P;
      C2<T> x[R];
#pragma unroll
      for (int t = 0; t < R; ++t) x[t] = ld(pa, bf + t * NBF);
      if (P > 1) {
#pragma unroll
        for (int t = 1; t < R; ++t) {
          C2<T> w = tw[t * k * M];
          if (SGN > 0) w.y = -w.y;
          x[t] = cmul(x[t], w);
        }
      }
      Dft<T, R>::run(x, SGN);
#pragma unroll
      for (int t = 0; t < R; ++t) y[c][t] = x[t];
    }
  }
}

// With `pre`, st also gets pre(pencil, element), fetched before the stage reads.
struct NoPre {};
template <class Pre> struct PreValue {
  typedef decltype(std::declval<Pre>()(0, 0)) type;
};
template <> struct PreValue<NoPre> {
  typedef int type;
};
template <typename T, int N, int R, int P, int NPEN, int SGN, bool SYNC_MID, int CT, class Ld,
          class St, class Pre = NoPre>
__device__ __forceinline__ void cstage_io(const C2<T> *tw, Ld ld, St st, Pre pre = Pre()) {
  constexpr bool PRE = !std::is_same<Pre, NoPre>::value;
  constexpr int NBF = N / R;
  constexpr int TOTAL = NPEN * NBF;
  constexpr int M = N / (P * R);
  constexpr int MAXB = (TOTAL + CT - 1) / CT;
  C2<T> y[MAXB][R];
  int eo[MAXB], pp[MAXB];
  typename PreValue<Pre>::type pv[PRE ? MAXB : 1][PRE ? R : 1];
#pragma unroll
  for (int c = 0; c < MAXB; ++c) {
    const int i = threadIdx.x + c * CT;
    eo[c] = -1;
    pp[c] = 0;
    if (TOTAL % CT == 0 || i < TOTAL) {
      const int pa = i % NPEN, bf = i / NPEN;
      const int k = bf % P;
      if constexpr (PRE) {
#pragma unroll
        for (int t = 0; t < R; ++t) pv[c][t] = pre(pa, (bf - k) * R + k + t * P);
      }
      C2<T> x[R];
#pragma unroll
      for (int t = 0; t < R; ++t) x[t] = ld(pa, bf + t * NBF);
      if (P > 1) {
#pragma unroll
        for (int t = 1; t < R; ++t) {
          C2<T> w = tw[t * k * M];
          if (SGN > 0) w.y = -w.y;
          x[t] = cmul(x[t], w);
        }
      }
      Dft<T, R>::run(x, SGN);
#pragma unroll
      for (int t = 0; t < R; ++t) y[c][t] = x[t];
      eo[c] = (bf - k) * R + k;
      pp[c] = pa;
    }
  }
  if (SYNC_MID) __syncthreads();
#pragma unroll
  for (int c = 0; c < MAXB; ++c) {
    if (TOTAL % CT == 0 || eo[c] >= 0) {
#pragma unroll
      for (int t = 0; t < R; ++t) {
        if constexpr (PRE)
          st(pp[c], eo[c] + t * P, y[c][t], pv[c][t]);
        else
          st(pp[c], eo[c] + t * P, y[c][t]);
      }
    }
  }
}

// A whole transform of NPEN pencils: the first stage reads through ld0 (from
// LDS if IN_LDS, else from global memory), the last one writes through stl
// (into LDS if OUT_LDS), the stages between through the LDS accessors ldm /
// stm.  A barrier follows every stage whose output is in LDS.
template <typename T, int N, int S, int P, int NPEN, int SGN, bool IN_LDS, bool OUT_LDS,
          int CT, class Ld0, class StL, class LdM, class StM, class Pre = NoPre>
__device__ __forceinline__ void cfft_io(const C2<T> *tw, Ld0 ld0, StL stl, LdM ldm, StM stm,
                                        Pre pre = Pre()) {
  if constexpr (S < CPlan<N>::ns) {
    constexpr int R = CPlan<N>::r[S];
    constexpr bool first = S == 0, last = S + 1 == CPlan<N>::ns;
    constexpr bool rd = first ? IN_LDS : true, wr = last ? OUT_LDS : true;
    if constexpr (first && last)
      cstage_io<T, N, R, P, NPEN, SGN, rd && wr, CT>(tw, ld0, stl, pre);
    else if constexpr (first)
      cstage_io<T, N, R, P, NPEN, SGN, rd && wr, CT>(tw, ld0, stm);
    else if constexpr (last)
      cstage_io<T, N, R, P, NPEN, SGN, rd && wr, CT>(tw, ldm, stl, pre);
    else
      cstage_io<T, N, R, P, NPEN, SGN, true, CT>(tw, ldm, stm);
    if constexpr (wr) __syncthreads();
    cfft_io<T, N, S + 1, P * R, NPEN, SGN, IN_LDS, OUT_LDS, CT>(tw, ld0, stl, ldm, stm, pre);
  }
}

// ---- whole-plane and pencil bodies of the compile-time passes -----------------------
// One workgroup holds one plane, or 512 bytes' worth of neighbouring z pencils;
// shared by the single-system and the batched kernels.  All are bound by their HBM
// bytes when the waves in flight cover the latency; see cthreads for the thread
// count.  256 36^3 complex64 bands: pass A 44.6 -> 33.4 us (140 MB), B 40.3 -> 32.7
// (191 MB), C 63 -> 55 (277 MB), the first figures with 512 threads a plane.

// Pass A of one plane of edge N: the sphere points [s0, s1) of xb (at box index
// box_index - off inside the plane) -> inverse x and y transforms -> dst.
template <typename T, int N>
__device__ __forceinline__ void pass_a_plane(const C2<T> *__restrict__ xb,
                                             const int32_t *__restrict__ box_index, int s0, int s1,
                                             int off, const double2 *__restrict__ twg,
                                             C2<T> *__restrict__ dst, C2<T> *buf, C2<T> *tw) {
  constexpr int NXY = N * N, LD = cld<N>(), CT = cthreads<N, N>();
  // the plane's sphere rows (a disk: at most pi/4 of it when the sphere fits the
  // box) are fetched before the plane is cleared, all in flight together
  constexpr int FULL = (NXY * 4 / 5 + CT - 1) / CT, U = FULL < 6 ? FULL : 6;
  T xr[U], xi[U];
  int xe[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int idx = min(s0 + (int)threadIdx.x + u * CT, s1 - 1);
    const C2<T> v = xb[idx];
    xr[u] = v.x;
    xi[u] = v.y;
    xe[u] = box_index[idx] - off;
  }
  for (int i = threadIdx.x; i < N; i += CT) tw[i] = to_c2<T>(twg[i]);
  for (int i = threadIdx.x; i < N * LD; i += CT) buf[i] = C2<T>{0, 0};
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (s0 + (int)threadIdx.x + u * CT < s1)
      buf[(xe[u] / N) * LD + xe[u] % N] = C2<T>{xr[u], xi[u]};
  for (int idx = s0 + threadIdx.x + U * CT; idx < s1; idx += CT) {
    const int e = box_index[idx] - off;
    buf[(e / N) * LD + e % N] = xb[idx];
  }
  __syncthreads();
  cfft<T, N, 0, 1, N, 1, LD, +1, CT>(buf, tw);  // x: N pencils of stride-1 elements
  // y: pencil i1, element i2; the last stage writes the box plane
  auto ldm = [&](int pa, int e) { return buf[pa + e * LD]; };
  auto stm = [&](int pa, int e, C2<T> v) { buf[pa + e * LD] = v; };
  auto stg = [&](int pa, int e, C2<T> v) { dst[pa + e * N] = v; };
  cfft_io<T, N, 0, 1, N, +1, true, false, CT>(tw, ldm, stg, ldm, stm);
}

// The transforms of pass C: the box plane src -> forward y and x transforms in buf
// (element (i1, i2) at i2 cld<N>() + i1).
template <typename T, int N>
__device__ __forceinline__ void pass_c_plane(const C2<T> *__restrict__ src,
                                             const double2 *__restrict__ twg, C2<T> *buf,
                                             C2<T> *tw) {
  constexpr int LD = cld<N>(), CT = cthreads<N, N>();
  for (int i = threadIdx.x; i < N; i += CT) tw[i] = to_c2<T>(twg[i]);
  __syncthreads();
  // y: pencil i1, element i2; the first stage reads the box plane
  auto ldm = [&](int pa, int e) { return buf[pa + e * LD]; };
  auto stm = [&](int pa, int e, C2<T> v) { buf[pa + e * LD] = v; };
  auto ldg = [&](int pa, int e) { return src[pa + e * N]; };
  cfft_io<T, N, 0, 1, N, -1, false, true, CT>(tw, ldg, stm, ldm, stm);
  cfft<T, N, 0, 1, N, 1, LD, -1, CT>(buf, tw);
}

// Reciprocal z-planes that hold sphere points, one bit each.
struct ZOcc {
  uint64_t lo, hi;
};

// z pencils per workgroup: 512 bytes of neighbouring pencils (64 complex64, 32
// complex128), so that every element row of a load or store is a whole run of
// 512 contiguous bytes whatever the plane's edges are (the pencils of a box are
// numbered i1 + n1 i2: a slab of one i2 would give rows of n1 elements, 288
// bytes and 216 of 512 threads busy at 36), and an LDS row is one bank sweep.
template <typename T> constexpr int zpencils() { return 512 / (int)sizeof(C2<T>); }

// Loads of a z transform's first stage from the box.  Reciprocal planes g3 without
// sphere points are zero (pass A leaves them unwritten).  Every load is issued: a
// pencil past the end reads the last one, an empty plane's element plane 0's, which
// the workgroup reads anyway; a branch around each load kept them from overlapping,
// 48 against 40 us per 64 64^3 complex64 boxes.
template <int N> __device__ __forceinline__ bool z_occupied(const ZOcc &z, int e) {
  return (((N > 64 && e >= 64 ? z.hi : z.lo) >> (e & 63)) & 1) != 0;
}
template <typename T, int N>
__device__ __forceinline__ C2<T> z_load(const C2<T> *src, const ZOcc &z, int left, int nxy, int pa,
                                        int e) {
  const bool in = z_occupied<N>(z, e);
  const C2<T> x = src[min(pa, left - 1) + (in ? e * nxy : 0)];
  return in ? x : C2<T>{0, 0};
}

// Pass B of the pencils [0, left) (at most zpencils) of a box whose planes hold nxy
// elements: inverse z transform, times V, forward transform; src and v point at the
// first pencil's plane-0 element, twg at the transform's twiddles.
template <typename T, int N>
__device__ __forceinline__ void z_pencils(C2<T> *__restrict__ src, const T *__restrict__ v,
                                          int left, int nxy, const double2 *__restrict__ twg,
                                          ZOcc zocc, C2<T> *buf, C2<T> *tw) {
  constexpr int Q = zpencils<T>(), CT = cthreads<N, Q>();
  for (int i = threadIdx.x; i < N; i += CT) tw[i] = to_c2<T>(twg[i]);
  __syncthreads();
  auto ldm = [&](int pa, int e) { return buf[pa + e * Q]; };
  auto stm = [&](int pa, int e, C2<T> x) { buf[pa + e * Q] = x; };
  auto ldg = [&](int pa, int e) { return z_load<T, N>(src, zocc, left, nxy, pa, e); };
  // V fetched ahead of the stage that multiplies by it
  auto pre = [&](int pa, int e) { return v[min(pa, left - 1) + e * nxy]; };
  auto stv = [&](int pa, int e, C2<T> x, T p) { buf[pa + e * Q] = cscale(x, p); };
  // (pass C does not read planes without sphere points)
  auto stg = [&](int pa, int e, C2<T> x) {
    if (pa < left && z_occupied<N>(zocc, e)) src[pa + e * nxy] = x;
  };
  cfft_io<T, N, 0, 1, Q, +1, false, true, CT>(tw, ldg, stv, ldm, stm, pre);
  cfft_io<T, N, 0, 1, Q, -1, true, false, CT>(tw, ldm, stg, ldm, stm);
}

// Edges with compile-time transforms.
#define CHEBFI_EDGES(X)                                                                         \
  X(12) X(15) X(16) X(18) X(20) X(24) X(25) X(27) X(30) X(32) X(36) X(40) X(45) X(48) X(50) \
  X(54) X(60) X(64) X(72) X(75) X(80) X(81) X(90) X(96)

inline bool listed_edge(int n) {
#define CHEBFI_CASE(N_) case N_:
  switch (n) {
    CHEBFI_EDGES(CHEBFI_CASE)
    return true;
    default:
      return false;
  }
#undef CHEBFI_CASE
}

}  // namespace
}  // namespace chebfi
