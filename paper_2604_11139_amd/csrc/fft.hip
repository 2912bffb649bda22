// Local-potential part of H on a batch of bands: scatter sphere -> box,
// inverse 3D FFT, multiply by V_loc(r), forward 3D FFT, gather sphere.
//
// The paper applies V_loc to all bands with one batched FFT call instead of a
// per-band loop (arXiv 2604.11139, section "Batch processing", Algorithms
// "Per-band kernel execution" / "Batched bands kernel execution").  Here the
// batched 3D transform is split in three HBM passes, each holding one 2D slab
// of one band in LDS:
//   pass A  (band, i3 plane): scatter the plane's sphere rows into a zeroed
//           n1 x n2 plane, inverse FFT along x then y, store the plane;
//   pass B  (band, run of z pencils or i2 slab): load, inverse FFT along z,
//           multiply by V(r), forward FFT along z, store;
//   pass C  (band, i3 plane): load, forward FFT along y then x, gather the
//           sphere rows, scale 1/(n1 n2 n3) and combine with the kinetic term
//           and the Chebyshev recurrence:
//           out = alpha (local + (kin - cshift) yk) - beta yprev.
// Each 1D transform is a Stockham autosort FFT executed in place in LDS (every
// thread holds its butterflies' outputs in registers across a barrier): two stages
// of radix 3 to 15 with compile-time lengths where the plane is square and its edge,
// or for pass B the z edge, is a {2,3,5}-smooth one from 12 to 96; radix-2/3/4/5
// stages of runtime length otherwise (a 54^3 pass B took 234 us in those, 40 in
// these).  Twiddles are FP64 tables built on the host.
#include <cstdlib>

#include "cplx.h"
#include "internal.h"
#include "kernels.h"
#include "fft_dev.h"

namespace chebfi {

namespace {

// ---- pass A: sphere plane -> inverse xy FFT -> box plane -------------------
// bf16 planes of the complex64 values a pass writes (the operand layout of the
// split-BF16 projection: planes re_hi, im_hi, re_lo, im_lo of ps elements each,
// band b at b * ld): hi = bf16(v) and lo = bf16(v - hi), both rounded to
// nearest even, the same values as the planes made by a separate split pass.
struct PlanesOut {
  unsigned short *p;
  int64_t ld, ps;
};
// Out[idx] = value(idx) over the sphere rows [s0, s1) with nt threads, and with
// po.p (T = float) the bf16 planes of each value.  (Pairing neighbouring
// lanes' planes into 32-bit stores by a shuffle measured slower: the pass is
// bound by its HBM bytes, which the planes raise by a fifth either way.)
template <typename T, class F>
__device__ __forceinline__ void sphere_store(int s0, int s1, int nt, const PlanesOut &po,
                                             int64_t b, C2<T> *out, F value) {
  if constexpr (std::is_same<T, float>::value) {
    if (po.p) {
      unsigned short *pb = po.p + b * po.ld;
      for (int idx = s0 + threadIdx.x; idx < s1; idx += nt) {
        const C2<T> o = value(idx);
        out[idx] = o;
        const unsigned short hr = bf16_bits(o.x), hi = bf16_bits(o.y);
        unsigned short *q = pb + idx;
        q[0] = hr;
        q[po.ps] = hi;
        q[2 * po.ps] = bf16_bits(o.x - bf16_float(hr));
        q[3 * po.ps] = bf16_bits(o.y - bf16_float(hi));
      }
      return;
    }
  }
  for (int idx = s0 + threadIdx.x; idx < s1; idx += nt) out[idx] = value(idx);
}

template <typename T>
__global__ __launch_bounds__(512) void pass_a_kernel(const C2<T> *__restrict__ X, int64_t ldx, int band0,
                              const int32_t *__restrict__ box_index,
                              const int32_t *__restrict__ plane, BoxPlan plan,
                              const double2 *__restrict__ twg, C2<T> *__restrict__ box) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C2<T> *buf = reinterpret_cast<C2<T> *>(smem_raw);
  const int n1 = plan.d[0].n, n2 = plan.d[1].n, n3 = plan.d[2].n;
  const int nxy = n1 * n2, L1 = n1 + 1;  // LDS plane rows padded to n1 + 1
  C2<T> *tw1 = buf + n2 * L1;
  C2<T> *tw2 = tw1 + n1;
  const int i3 = blockIdx.x;
  const int bl = blockIdx.y;
  load_twiddles<T>(tw1, twg, n1);
  load_twiddles<T>(tw2, twg + kMaxN, n2);
  for (int i = threadIdx.x; i < n2 * L1; i += blockDim.x) buf[i] = C2<T>{0, 0};
  __syncthreads();
  const int s0 = plane[i3], s1 = plane[i3 + 1];
  const C2<T> *xb = X + (int64_t)(band0 + bl) * ldx;
  const int off = i3 * nxy;
  for (int idx = s0 + threadIdx.x; idx < s1; idx += blockDim.x) {
    const int e = box_index[idx] - off;
    buf[e + e / n1] = xb[idx];
  }
  __syncthreads();
  lds_fft<T>(buf, plan.d[0], 1, n2, L1, tw1, +1);
  lds_fft<T>(buf, plan.d[1], L1, n1, 1, tw2, +1);
  C2<T> *dst = box + (int64_t)bl * nxy * n3 + off;
  for (int i = threadIdx.x; i < nxy; i += blockDim.x) dst[i] = buf[i + i / n1];
}

// ---- pass B: z pencils of one i2 slab, inverse FFT, * V, forward FFT -------
template <typename T, typename VT>
__global__ __launch_bounds__(512) void pass_b_kernel(C2<T> *__restrict__ box, const VT *__restrict__ V, BoxPlan plan,
                              const double2 *__restrict__ twg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C2<T> *buf = reinterpret_cast<C2<T> *>(smem_raw);
  const int n1 = plan.d[0].n, n2 = plan.d[1].n, n3 = plan.d[2].n;
  const int nxz = n1 * n3, L1 = n1 + 1;  // LDS slab rows padded to n1 + 1
  C2<T> *tw3 = buf + n3 * L1;
  const int i2 = blockIdx.x;
  const int bl = blockIdx.y;
  load_twiddles<T>(tw3, twg + 2 * kMaxN, n3);
  C2<T> *src = box + (int64_t)bl * n1 * n2 * n3;
  for (int i = threadIdx.x; i < nxz; i += blockDim.x) {
    const int i1 = i % n1, i3 = i / n1;
    buf[i3 * L1 + i1] = src[i1 + n1 * (i2 + n2 * i3)];
  }
  __syncthreads();
  lds_fft<T>(buf, plan.d[2], L1, n1, 1, tw3, +1);
  for (int i = threadIdx.x; i < nxz; i += blockDim.x) {
    const int i1 = i % n1, i3 = i / n1;
    buf[i3 * L1 + i1] = cscale(buf[i3 * L1 + i1], (T)V[i1 + n1 * (i2 + n2 * i3)]);
  }
  __syncthreads();
  lds_fft<T>(buf, plan.d[2], L1, n1, 1, tw3, -1);
  for (int i = threadIdx.x; i < nxz; i += blockDim.x) {
    const int i1 = i % n1, i3 = i / n1;
    src[i1 + n1 * (i2 + n2 * i3)] = buf[i3 * L1 + i1];
  }
}

// a + b rounded on its own (never fused with the multiply that produced a), so
// that adding a precomputed block E equals storing the value and adding E later
template <typename V2> __device__ __forceinline__ V2 add_rounded(V2 a, V2 b) {
#pragma clang fp contract(off)
  return V2{a.x + b.x, a.y + b.y};
}

// ---- pass C: box plane -> forward xy FFT -> gather + recurrence combine ----
template <typename T>
__global__ __launch_bounds__(512) void pass_c_kernel(const C2<T> *__restrict__ box, BoxPlan plan,
                              const double2 *__restrict__ twg,
                              const int32_t *__restrict__ box_index,
                              const int32_t *__restrict__ plane, const double *__restrict__ kin,
                              int band0, const C2<T> *__restrict__ Yk, int64_t ldk,
                              const C2<T> *__restrict__ Yprev, int64_t ldp,
                              C2<T> *__restrict__ Out, int64_t ldo, T alpha, T cshift, T beta,
                              T scale, const C2<T> *__restrict__ E, int64_t lde,
                              const double *__restrict__ coef, PlanesOut po) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C2<T> *buf = reinterpret_cast<C2<T> *>(smem_raw);
  if (coef) {  // (alpha, cshift, beta) of this step from device memory (captured filters)
    alpha = (T)coef[0];
    cshift = (T)coef[1];
    beta = (T)coef[2];
  }
  const int n1 = plan.d[0].n, n2 = plan.d[1].n;
  const int nxy = n1 * n2, L1 = n1 + 1;  // LDS plane rows padded to n1 + 1
  C2<T> *tw1 = buf + n2 * L1;
  C2<T> *tw2 = tw1 + n1;
  const int i3 = blockIdx.x;
  const int bl = blockIdx.y;
  load_twiddles<T>(tw1, twg, n1);
  load_twiddles<T>(tw2, twg + kMaxN, n2);
  const int off = i3 * nxy;
  const C2<T> *src = box + (int64_t)bl * nxy * plan.d[2].n + off;
  for (int i = threadIdx.x; i < nxy; i += blockDim.x) buf[i + i / n1] = src[i];
  __syncthreads();
  lds_fft<T>(buf, plan.d[1], L1, n1, 1, tw2, -1);
  lds_fft<T>(buf, plan.d[0], 1, n2, L1, tw1, -1);
  const int s0 = plane[i3], s1 = plane[i3 + 1];
  const int64_t b = band0 + bl;
  const C2<T> *yk = Yk + b * ldk;
  C2<T> *out = Out + b * ldo;
  const C2<T> *ex = E ? E + b * lde : nullptr;
  if (Yprev != nullptr) {
    const C2<T> *yp = Yprev + b * ldp;
    sphere_store<T>(s0, s1, (int)blockDim.x, po, b, out, [&](int idx) {
      const int e = box_index[idx] - off;
      C2<T> loc = cscale(buf[e + e / n1], scale);
      C2<T> x = yk[idx];
      const T kd = (T)kin[idx] - cshift;
      C2<T> h = cadd(loc, cscale(x, kd));
      C2<T> p = yp[idx];
      C2<T> o{alpha * h.x - beta * p.x, alpha * h.y - beta * p.y};
      if (ex) o = add_rounded(o, ex[idx]);
      return o;
    });
  } else {
    sphere_store<T>(s0, s1, (int)blockDim.x, po, b, out, [&](int idx) {
      const int e = box_index[idx] - off;
      C2<T> loc = cscale(buf[e + e / n1], scale);
      C2<T> x = yk[idx];
      const T kd = (T)kin[idx] - cshift;
      C2<T> h = cadd(loc, cscale(x, kd));
      C2<T> o = cscale(h, alpha);
      if (ex) o = add_rounded(o, ex[idx]);
      return o;
    });
  }
}

// ---- adjoint passes (runtime sizes) -----------------------------------------
// z-inverse FFT only: the box then holds the band in real space.
template <typename T>
__global__ __launch_bounds__(512) void pass_b_inv_kernel(C2<T> *__restrict__ box, BoxPlan plan,
                                                         const double2 *__restrict__ twg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C2<T> *buf = reinterpret_cast<C2<T> *>(smem_raw);
  const int n1 = plan.d[0].n, n2 = plan.d[1].n, n3 = plan.d[2].n;
  const int nxz = n1 * n3, L1 = n1 + 1;  // LDS slab rows padded to n1 + 1
  C2<T> *tw3 = buf + n3 * L1;
  const int i2 = blockIdx.x;
  const int bl = blockIdx.y;
  load_twiddles<T>(tw3, twg + 2 * kMaxN, n3);
  C2<T> *src = box + (int64_t)bl * n1 * n2 * n3;
  for (int i = threadIdx.x; i < nxz; i += blockDim.x) {
    const int i1 = i % n1, i3 = i / n1;
    buf[i3 * L1 + i1] = src[i1 + n1 * (i2 + n2 * i3)];
  }
  __syncthreads();
  lds_fft<T>(buf, plan.d[2], L1, n1, 1, tw3, +1);
  for (int i = threadIdx.x; i < nxz; i += blockDim.x) {
    const int i1 = i % n1, i3 = i / n1;
    src[i1 + n1 * (i2 + n2 * i3)] = buf[i3 * L1 + i1];
  }
}

// Pass B of the adjoint H application: z-inverse of the adjoint band (box),
// the pointwise product Re[conj(adjoint) * forward] written over the forward
// band's real-space box (`fwd`, real part), then * V and the z-forward FFT.
template <typename T>
__global__ __launch_bounds__(512) void pass_b_adj_kernel(C2<T> *__restrict__ box,
                                                         C2<T> *__restrict__ fwd,
                                                         const T *__restrict__ V, BoxPlan plan,
                                                         const double2 *__restrict__ twg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C2<T> *buf = reinterpret_cast<C2<T> *>(smem_raw);
  const int n1 = plan.d[0].n, n2 = plan.d[1].n, n3 = plan.d[2].n;
  const int nxz = n1 * n3, L1 = n1 + 1;  // LDS slab rows padded to n1 + 1
  C2<T> *tw3 = buf + n3 * L1;
  const int i2 = blockIdx.x;
  const int bl = blockIdx.y;
  load_twiddles<T>(tw3, twg + 2 * kMaxN, n3);
  C2<T> *src = box + (int64_t)bl * n1 * n2 * n3;
  C2<T> *fw = fwd + (int64_t)bl * n1 * n2 * n3;
  for (int i = threadIdx.x; i < nxz; i += blockDim.x) {
    const int i1 = i % n1, i3 = i / n1;
    buf[i3 * L1 + i1] = src[i1 + n1 * (i2 + n2 * i3)];
  }
  __syncthreads();
  lds_fft<T>(buf, plan.d[2], L1, n1, 1, tw3, +1);
  for (int i = threadIdx.x; i < nxz; i += blockDim.x) {
    const int i1 = i % n1, i3 = i / n1;
    const int64_t r = i1 + n1 * (i2 + n2 * i3);
    const C2<T> a = buf[i3 * L1 + i1], y = fw[r];
    fw[r] = C2<T>{a.x * y.x + a.y * y.y, (T)0};
    buf[i3 * L1 + i1] = cscale(a, V[r]);
  }
  __syncthreads();
  lds_fft<T>(buf, plan.d[2], L1, n1, 1, tw3, -1);
  for (int i = threadIdx.x; i < nxz; i += blockDim.x) {
    const int i1 = i % n1, i3 = i / n1;
    src[i1 + n1 * (i2 + n2 * i3)] = buf[i3 * L1 + i1];
  }
}

// dV[r] += scale * sum_b prod[b][r].x, bands summed in order.
template <typename T>
__global__ __launch_bounds__(256) void dv_reduce_kernel(int64_t nbox, int nb,
                                                        const C2<T> *__restrict__ prod,
                                                        double scale, double *__restrict__ dV) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nbox) return;
  double acc = 0.0;
  for (int b = 0; b < nb; ++b) acc += (double)prod[(int64_t)b * nbox + r].x;
  dV[r] += scale * acc;
}

// rho[r] += sum_b w[band0 + b] |box_b(r)|^2 * scale, bands summed in order.
template <typename T>
__global__ __launch_bounds__(256) void rho_accum_kernel(int64_t nbox, int nb, int band0,
                                                        const C2<T> *__restrict__ box,
                                                        const double *__restrict__ w,
                                                        double scale, double *__restrict__ rho) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nbox) return;
  double acc = 0.0;
  for (int b = 0; b < nb; ++b) {
    const C2<T> v = box[(int64_t)b * nbox + r];
    const double wb = w ? w[band0 + b] : 1.0;
    acc += wb * ((double)v.x * v.x + (double)v.y * v.y);
  }
  rho[r] += scale * acc;
}

// ---- compile-time specialised passes (bodies in fft_dev.h) --------------------------------
// Passes A and C for square planes of a listed edge N (any n3), the z passes for a
// listed n3 (any plane).

template <typename T, int N>
__global__ __launch_bounds__((cthreads<N, N>())) void cpass_a_kernel(
    const C2<T> *__restrict__ X, int64_t ldx, int band0, const int32_t *__restrict__ box_index,
    const int32_t *__restrict__ plane, const double2 *__restrict__ twg, C2<T> *__restrict__ box) {
  __shared__ C2<T> buf[N * cld<N>()];
  __shared__ C2<T> tw[N];
  const int i3 = blockIdx.x, bl = blockIdx.y, off = i3 * N * N;
  const int s0 = plane[i3], s1 = plane[i3 + 1];
  // a plane with no sphere points is left unwritten: the middle passes read it as zero
  if (s0 == s1) return;
  pass_a_plane<T, N>(X + (int64_t)(band0 + bl) * ldx, box_index, s0, s1, off, twg,
                     box + (int64_t)bl * N * N * gridDim.x + off, buf, tw);
}

template <typename T, int N>
__global__ __launch_bounds__((cthreads<N, zpencils<T>()>())) void zpass_kernel(
    C2<T> *__restrict__ box, const T *__restrict__ V, int nxy, const double2 *__restrict__ twg,
    ZOcc zocc) {
  constexpr int Q = zpencils<T>();
  __shared__ C2<T> buf[N * Q];
  __shared__ C2<T> tw[N];
  const int q0 = blockIdx.x * Q;
  z_pencils<T, N>(box + (int64_t)blockIdx.y * nxy * N + q0, V + q0, nxy - q0, nxy,
                  twg + 2 * kMaxN, zocc, buf, tw);
}

// A partial sum in FP64 kept in one box element.
__device__ __forceinline__ void put_sum(C2<double> &x, double s) { x = C2<double>{s, 0.0}; }
__device__ __forceinline__ void put_sum(C2<float> &x, double s) {
  x = C2<float>{__int_as_float(__double2loint(s)), __int_as_float(__double2hiint(s))};
}
__device__ __forceinline__ double get_sum(const C2<double> &x) { return x.x; }
__device__ __forceinline__ double get_sum(const C2<float> &x) {
  return __hiloint2double(__float_as_int(x.y), __float_as_int(x.x));
}

// Real-space sums over bands without a real-space box in memory.  A workgroup takes
// one run of pencils and `per` bands in turn: the inverse z transform's last stage
// leaves real space in registers, each thread the same points for every band, and
// the workgroup's sums (FP64, bands in order) end up in its first band's box of
// `fwd`, whose pencils no other workgroup reads.
//   ADJ = false, the density: sum_b w_b |psi_b(r)|^2 from the boxes fwd;
//   ADJ = true, the adjoint's pass B: sum_b Re[conj(a_b) y_b] with the adjoint
//   bands a in `box` and the forward bands y in `fwd`, and box <- the forward
//   transform of V a.
// One butterfly of the last stage per thread: with the filter's thread counts the
// sums, V and two bands' values of two or three butterflies spilled (96: 252 B).
template <typename T, int N> constexpr int zaccum_threads() {
  return (zpencils<T>() * (N / CPlan<N>::r[1]) + 63) / 64 * 64;
}
template <typename T, int N, bool ADJ>
__global__ __launch_bounds__((zaccum_threads<T, N>())) void zaccum_kernel(
    C2<T> *__restrict__ box, C2<T> *__restrict__ fwd, const T *__restrict__ V,
    const double *__restrict__ w, int nxy_, const double2 *__restrict__ twg, ZOcc zocc, int nb,
    int per) {
  constexpr int Q = zpencils<T>(), CT = zaccum_threads<T, N>();
  static_assert(CPlan<N>::ns == 2, "two-stage transforms");
  constexpr int R0 = CPlan<N>::r[0], R = CPlan<N>::r[1], MB = cstage_rounds<N, R, Q, CT>();
  __shared__ C2<T> buf[N * Q];
  __shared__ C2<T> tw[N];
  const int q0 = blockIdx.x * Q, left = nxy_ - q0;
  for (int i = threadIdx.x; i < N; i += CT) tw[i] = to_c2<T>(twg[2 * kMaxN + i]);
  __syncthreads();
  auto ldm = [&](int pa, int e) { return buf[pa + e * Q]; };
  auto stm = [&](int pa, int e, C2<T> x) { buf[pa + e * Q] = x; };
  double acc[MB][R];
#pragma unroll
  for (int c = 0; c < MB; ++c)
#pragma unroll
    for (int t = 0; t < R; ++t) acc[c][t] = 0.0;
  const int b1 = min(nb, ((int)blockIdx.y + 1) * per);
  for (int b = blockIdx.y * per; b < b1; ++b) {
    const int64_t o = (int64_t)b * nxy_ * N + q0;
    // opaque per band: otherwise every offset of the box is kept across bands, in
    // more registers than the sums
    int nxy = nxy_;
    asm volatile("" : "+s"(nxy));
    const C2<T> *f = fwd + o;
    auto ldf = [&](int pa, int e) { return z_load<T, N>(f, zocc, left, nxy, pa, e); };
    cstage_io<T, N, R0, 1, Q, +1, false, CT>(tw, ldf, stm);
    __syncthreads();
    C2<T> y[MB][R];
    cstage_vals<T, N, R, R0, Q, +1, CT>(tw, ldm, y);
    __syncthreads();
    if constexpr (!ADJ) {
      const double wb = w ? w[b] : 1.0;
#pragma unroll
      for (int c = 0; c < MB; ++c)
#pragma unroll
        for (int t = 0; t < R; ++t)
          acc[c][t] += wb * ((double)y[c][t].x * y[c][t].x + (double)y[c][t].y * y[c][t].y);
    } else {
      C2<T> *a = box + o;
      auto lda = [&](int pa, int e) { return z_load<T, N>(a, zocc, left, nxy, pa, e); };
      cstage_io<T, N, R0, 1, Q, +1, false, CT>(tw, lda, stm);
      T v[MB][R];
#pragma unroll
      for (int c = 0; c < MB; ++c) {
        int pa, e0;
        cstage_at<N, R, R0, Q, CT>(c, pa, e0);
#pragma unroll
        for (int t = 0; t < R; ++t)
          v[c][t] = V[q0 + min(pa, left - 1) + min(e0 + t * R0, N - 1) * nxy];
      }
      __syncthreads();
      C2<T> x[MB][R];
      cstage_vals<T, N, R, R0, Q, +1, CT>(tw, ldm, x);
      __syncthreads();
#pragma unroll
      for (int c = 0; c < MB; ++c) {
        int pa, e0;
        if (cstage_at<N, R, R0, Q, CT>(c, pa, e0)) {
#pragma unroll
          for (int t = 0; t < R; ++t) {
            acc[c][t] += (double)(x[c][t].x * y[c][t].x + x[c][t].y * y[c][t].y);
            buf[pa + (e0 + t * R0) * Q] = cscale(x[c][t], v[c][t]);
          }
        }
      }
      __syncthreads();
      auto stg = [&](int pa, int e, C2<T> z) {
        if (pa < left && z_occupied<N>(zocc, e)) a[pa + e * nxy] = z;
      };
      cfft_io<T, N, 0, 1, Q, -1, true, false, CT>(tw, ldm, stg, ldm, stm);
      __syncthreads();
    }
  }
  // (the barriers above stand between the last band's loads and these stores)
  C2<T> *out = fwd + (int64_t)blockIdx.y * per * nxy_ * N + q0;
#pragma unroll
  for (int c = 0; c < MB; ++c) {
    int pa, e0;
    if (cstage_at<N, R, R0, Q, CT>(c, pa, e0) && pa < left) {
#pragma unroll
      for (int t = 0; t < R; ++t) put_sum(out[pa + (e0 + t * R0) * nxy_], acc[c][t]);
    }
  }
}

// out[r] += scale * the sum of element r of boxes 0, per, 2 per, ... (in order).
template <typename T>
__global__ __launch_bounds__(256) void zaccum_sum_kernel(int64_t nbox, int groups, int per,
                                                         const C2<T> *__restrict__ part,
                                                         double scale, double *__restrict__ out) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= nbox) return;
  double s = 0.0;
#pragma unroll 8
  for (int g = 0; g < groups; ++g) s += get_sum(part[(int64_t)g * per * nbox + r]);
  out[r] += scale * s;
}

// (Gathering two or three rows per thread at once, all their loads in flight
// together, made this pass slower: 53.5 -> 59.5 us for 256 36^3 complex64 bands,
// 68.6 -> 76.6 us for 64 64^3 ones.)
template <typename T, int N>
__global__ __launch_bounds__((cthreads<N, N>())) void cpass_c_kernel(
    const C2<T> *__restrict__ box, const double2 *__restrict__ twg,
    const int32_t *__restrict__ box_index, const int32_t *__restrict__ plane,
    const double *__restrict__ kin, int band0, const C2<T> *__restrict__ Yk, int64_t ldk,
    const C2<T> *__restrict__ Yprev, int64_t ldp, C2<T> *__restrict__ Out, int64_t ldo, T alpha,
    T cshift, T beta, T scale, const C2<T> *__restrict__ E, int64_t lde,
    const double *__restrict__ coef, PlanesOut po) {
  constexpr int NXY = N * N, LD = cld<N>(), CT = cthreads<N, N>();
  __shared__ C2<T> buf[N * LD];
  __shared__ C2<T> tw[N];
  if (coef) {  // (alpha, cshift, beta) of this step from device memory (captured filters)
    alpha = (T)coef[0];
    cshift = (T)coef[1];
    beta = (T)coef[2];
  }
  const int i3 = blockIdx.x;
  const int bl = blockIdx.y;
  const int s0 = plane[i3], s1 = plane[i3 + 1];
  if (s0 == s1) return;  // no sphere points to gather in this plane
  const int off = i3 * NXY;
  pass_c_plane<T, N>(box + (int64_t)bl * NXY * gridDim.x + off, twg, buf, tw);
  const int64_t b = band0 + bl;
  const C2<T> *yk = Yk + b * ldk;
  C2<T> *out = Out + b * ldo;
  const C2<T> *ex = E ? E + b * lde : nullptr;
  if (Yprev != nullptr) {
    const C2<T> *yp = Yprev + b * ldp;
    sphere_store<T>(s0, s1, CT, po, b, out, [&](int idx) {
      const int e = box_index[idx] - off;
      const C2<T> loc = cscale(buf[(e / N) * LD + e % N], scale);
      const C2<T> x = yk[idx];
      const T kd = (T)kin[idx] - cshift;
      const C2<T> h = cadd(loc, cscale(x, kd));
      const C2<T> p = yp[idx];
      C2<T> o{alpha * h.x - beta * p.x, alpha * h.y - beta * p.y};
      if (ex) o = add_rounded(o, ex[idx]);
      return o;
    });
  } else {
    sphere_store<T>(s0, s1, CT, po, b, out, [&](int idx) {
      const int e = box_index[idx] - off;
      const C2<T> loc = cscale(buf[(e / N) * LD + e % N], scale);
      const C2<T> x = yk[idx];
      const T kd = (T)kin[idx] - cshift;
      C2<T> o = cscale(cadd(loc, cscale(x, kd)), alpha);
      if (ex) o = add_rounded(o, ex[idx]);
      return o;
    });
  }
}

template <typename F> void set_lds(F kernel, size_t bytes) {
  CHEBFI_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
}

// Which passes of a handle are compile-time specialised: the z passes for a
// listed n3, passes A and C for square planes of a listed edge when the z passes
// are too (they leave planes without sphere points unwritten, which only the
// specialised z passes know); the runtime-size ones otherwise.
bool special_z(const abi_system_s *s) { return !s->generic_fft && listed_edge(s->n3); }
bool special_planes(const abi_system_s *s) {
  return special_z(s) && s->n1 == s->n2 && listed_edge(s->n1);
}

// Thread counts and LDS bytes of the runtime-size passes.
template <typename T> struct RuntimeShape {
  int tA, tB;
  size_t ldsA, ldsB;
  explicit RuntimeShape(const BoxPlan &plan) {
    const int n1 = plan.d[0].n, n2 = plan.d[1].n, n3 = plan.d[2].n;
    tA = std::max(stage_threads(plan.d[0], n2), stage_threads(plan.d[1], n1));
    tB = stage_threads(plan.d[2], n1);
    CHEBFI_REQUIRE(tA <= 512 && tB <= 512, ABI_ERR_GRID, "FFT plane too large for one workgroup");
    ldsA = sizeof(C2<T>) * (size_t)(n2 * (n1 + 1) + n1 + n2);
    ldsB = sizeof(C2<T>) * (size_t)(n3 * (n1 + 1) + n3);
  }
};

// Pass A of bands band0 .. band0 + nb - 1 of X into `box`.
template <typename T>
void launch_a(const abi_system_s *s, const void *X, int64_t ldx, int band0, int nb, void *box,
              hipStream_t st) {
  const C2<T> *x = reinterpret_cast<const C2<T> *>(X);
  C2<T> *bx = reinterpret_cast<C2<T> *>(box);
  const double2 *tw = reinterpret_cast<const double2 *>(s->d_tw);
  const dim3 grid(s->n3, nb);
  if (special_planes(s)) {
#define CHEBFI_CASE(N_)                                                                       \
  case N_:                                                                                    \
    hipLaunchKernelGGL((cpass_a_kernel<T, N_>), grid, dim3(cthreads<N_, N_>()), 0, st, x, ldx, \
                       band0, s->d_box, s->d_plane, tw, bx);                                  \
    break;
    switch (s->n1) { CHEBFI_EDGES(CHEBFI_CASE) }
#undef CHEBFI_CASE
  } else {
    const RuntimeShape<T> r(s->plan);
    set_lds(pass_a_kernel<T>, r.ldsA);
    hipLaunchKernelGGL(pass_a_kernel<T>, grid, dim3(r.tA), r.ldsA, st, x, ldx, band0, s->d_box,
                       s->d_plane, s->plan, tw, bx);
  }
  CHEBFI_HIP(hipGetLastError());
}

// Pass B of nb boxes.
template <typename T>
void launch_z(const abi_system_s *s, void *box, const void *V, int nb, hipStream_t st) {
  C2<T> *bx = reinterpret_cast<C2<T> *>(box);
  const T *v = reinterpret_cast<const T *>(V);
  const double2 *tw = reinterpret_cast<const double2 *>(s->d_tw);
  if (special_z(s)) {
    constexpr int Q = zpencils<T>();
    const int nxy = s->n1 * s->n2;
    const dim3 grid((nxy + Q - 1) / Q, nb);
    const ZOcc occ{s->zocc, s->zocc_hi};
#define CHEBFI_CASE(N_)                                                                          \
  case N_:                                                                                       \
    hipLaunchKernelGGL((zpass_kernel<T, N_>), grid, dim3(cthreads<N_, Q>()), 0, st, bx, v, nxy, \
                       tw, occ);                                                                 \
    break;
    switch (s->n3) { CHEBFI_EDGES(CHEBFI_CASE) }
#undef CHEBFI_CASE
  } else {
    const RuntimeShape<T> r(s->plan);
    set_lds(pass_b_kernel<T, T>, r.ldsB);
    hipLaunchKernelGGL((pass_b_kernel<T, T>), dim3(s->n2, nb), dim3(r.tB), r.ldsB, st, bx, v,
                       s->plan, tw);
  }
  CHEBFI_HIP(hipGetLastError());
}

// out += scale * the real-space sums of zaccum_kernel (listed n3 only).
template <typename T, bool ADJ>
void launch_zaccum(const abi_system_s *s, void *box, void *fwd, const void *V, const double *w,
                   int nb, double scale, double *out, hipStream_t st) {
  constexpr int Q = zpencils<T>();
  const double2 *tw = reinterpret_cast<const double2 *>(s->d_tw);
  const int nxy = s->n1 * s->n2, runs = (nxy + Q - 1) / Q;
  const int64_t nbox = (int64_t)nxy * s->n3;
  const ZOcc occ{s->zocc, s->zocc_hi};
  // bands per workgroup: as many as leave six workgroups per CU
  const int per = std::max<int>(1, (int)((int64_t)runs * nb / (6 * device_cus())));
  const int groups = (nb + per - 1) / per;
#define CHEBFI_CASE(N_)                                                                          \
  case N_:                                                                                       \
    hipLaunchKernelGGL((zaccum_kernel<T, N_, ADJ>), dim3(runs, groups),                          \
                       dim3(zaccum_threads<T, N_>()), 0, st, (C2<T> *)box, (C2<T> *)fwd,         \
                       (const T *)V, w, nxy, tw, occ, nb, per);                                  \
    break;
  switch (s->n3) { CHEBFI_EDGES(CHEBFI_CASE) }
#undef CHEBFI_CASE
  CHEBFI_HIP(hipGetLastError());
  hipLaunchKernelGGL(zaccum_sum_kernel<T>, dim3((unsigned)((nbox + 255) / 256)), dim3(256), 0, st,
                     nbox, groups, per, (const C2<T> *)fwd, scale, out);
  CHEBFI_HIP(hipGetLastError());
}

// Pass C of nb boxes into bands band0 .. of Out.
template <typename T>
void launch_c(const abi_system_s *s, const void *box, int band0, int nb, const void *Yk,
              int64_t ldk, const void *Yprev, int64_t ldp, void *Out, int64_t ldo, double alpha,
              double cshift, double beta, const void *E, int64_t lde, const double *coef,
              PlanesOut po, hipStream_t st) {
  typedef const C2<T> *In;
  const double2 *tw = reinterpret_cast<const double2 *>(s->d_tw);
  const T scale = (T)(1.0 / ((double)s->n1 * (double)s->n2 * (double)s->n3));
  const dim3 grid(s->n3, nb);
  if (special_planes(s)) {
#define CHEBFI_CASE(N_)                                                                         \
  case N_:                                                                                      \
    hipLaunchKernelGGL((cpass_c_kernel<T, N_>), grid, dim3(cthreads<N_, N_>()), 0, st, (In)box, \
                       tw, s->d_box, s->d_plane, s->d_kin, band0, (In)Yk, ldk, (In)Yprev, ldp,  \
                       (C2<T> *)Out, ldo, (T)alpha, (T)cshift, (T)beta, scale, (In)E, lde,      \
                       coef, po);                                                               \
    break;
    switch (s->n1) { CHEBFI_EDGES(CHEBFI_CASE) }
#undef CHEBFI_CASE
  } else {
    const RuntimeShape<T> r(s->plan);
    set_lds(pass_c_kernel<T>, r.ldsA);
    hipLaunchKernelGGL(pass_c_kernel<T>, grid, dim3(r.tA), r.ldsA, st, (In)box, s->plan, tw,
                       s->d_box, s->d_plane, s->d_kin, band0, (In)Yk, ldk, (In)Yprev, ldp,
                       (C2<T> *)Out, ldo, (T)alpha, (T)cshift, (T)beta, scale, (In)E, lde, coef,
                       po);
  }
  CHEBFI_HIP(hipGetLastError());
}

}  // namespace

template <typename T>
void launch_local_potential(const abi_system_s *s, const void *Yk, int64_t ldk, const void *Yprev,
                            int64_t ldp, void *Out, int64_t ldo, int band0, int nb, void *box,
                            const void *V, double alpha, double cshift, double beta,
                            hipStream_t st, Profiler *prof, const void *E, int64_t lde,
                            void *ypl, int64_t ldpl, int64_t pspl) {
  const PlanesOut po{std::is_same<T, float>::value ? (unsigned short *)ypl : nullptr, ldpl, pspl};
  // algorithmic HBM bytes of each pass (sphere rows, box planes, V once)
  const double es = (double)sizeof(C2<T>), np = (double)s->npw;
  const double nbx = (double)s->n1 * s->n2 * s->n3;
  int tok = prof ? prof->begin(PROF_FFT_A, nb * (np + nbx) * es, st) : -1;
  launch_a<T>(s, Yk, ldk, band0, nb, box, st);
  if (prof) prof->end(tok, st);
  tok = prof ? prof->begin(PROF_FFT_B, nb * 2.0 * nbx * es + nbx * (double)sizeof(T), st) : -1;
  launch_z<T>(s, box, V, nb, st);
  if (prof) prof->end(tok, st);
  tok = prof ? prof->begin(PROF_FFT_C,
                           nb * (nbx + np * ((Yprev ? 3.0 : 2.0) + (E ? 1.0 : 0.0))) * es, st)
             : -1;
  launch_c<T>(s, box, band0, nb, Yk, ldk, Yprev, ldp, Out, ldo, alpha, cshift, beta, E, lde,
              s->coef_dev, po, st);
  if (prof) prof->end(tok, st);
}

template <typename T>
void launch_adjoint_local(const abi_system_s *s, const void *Ak1, int64_t lda1, const void *Yk,
                          int64_t ldy, const void *Ak2, int64_t lda2, double delta, void *Ak,
                          int64_t ldak, int band0, int nb, void *box1, void *box2, const void *V,
                          double gamma, double cshift, const void *E, int64_t lde, double *dV,
                          hipStream_t st) {
  const int64_t nbox = (int64_t)s->n1 * s->n2 * s->n3;
  launch_a<T>(s, Ak1, lda1, band0, nb, box1, st);
  launch_a<T>(s, Yk, ldy, band0, nb, box2, st);
  if (special_z(s)) {
    launch_zaccum<T, true>(s, box1, box2, V, nullptr, nb, gamma / (double)nbox, dV, st);
  } else {
    const RuntimeShape<T> r(s->plan);
    const double2 *tw = reinterpret_cast<const double2 *>(s->d_tw);
    const dim3 grid(s->n2, nb), threads(r.tB);
    set_lds(pass_b_inv_kernel<T>, r.ldsB);
    set_lds(pass_b_adj_kernel<T>, r.ldsB);
    hipLaunchKernelGGL(pass_b_inv_kernel<T>, grid, threads, r.ldsB, st, (C2<T> *)box2, s->plan, tw);
    hipLaunchKernelGGL(pass_b_adj_kernel<T>, grid, threads, r.ldsB, st, (C2<T> *)box1,
                       (C2<T> *)box2, (const T *)V, s->plan, tw);
    hipLaunchKernelGGL(dv_reduce_kernel<T>, dim3((unsigned)((nbox + 255) / 256)), dim3(256), 0, st,
                       nbox, nb, (const C2<T> *)box2, gamma / (double)nbox, dV);
    CHEBFI_HIP(hipGetLastError());
  }
  // Ak = gamma (local + (kin - c) Ak1) - delta Ak2 + E
  launch_c<T>(s, box1, band0, nb, Ak1, lda1, Ak2, lda2, Ak, ldak, gamma, cshift, delta, E, lde,
              nullptr, PlanesOut{nullptr, 0, 0}, st);
}

template <typename T>
void launch_density(const abi_system_s *s, const void *Psi, int64_t ld, int band0, int nb, void *box,
                    const double *w, double *rho, hipStream_t st) {
  const int64_t nbox = (int64_t)s->n1 * s->n2 * s->n3;
  launch_a<T>(s, Psi, ld, band0, nb, box, st);
  if (special_z(s)) {
    launch_zaccum<T, false>(s, nullptr, box, nullptr, w ? w + band0 : nullptr, nb,
                            1.0 / (double)nbox, rho, st);
    return;
  }
  const RuntimeShape<T> r(s->plan);
  set_lds(pass_b_inv_kernel<T>, r.ldsB);
  hipLaunchKernelGGL(pass_b_inv_kernel<T>, dim3(s->n2, nb), dim3(r.tB), r.ldsB, st, (C2<T> *)box,
                     s->plan, reinterpret_cast<const double2 *>(s->d_tw));
  hipLaunchKernelGGL(rho_accum_kernel<T>, dim3((unsigned)((nbox + 255) / 256)), dim3(256), 0, st,
                     nbox, nb, band0, (const C2<T> *)box, w, 1.0 / (double)nbox, rho);
  CHEBFI_HIP(hipGetLastError());
}

template void launch_density<double>(const abi_system_s *, const void *, int64_t, int, int, void *,
                                     const double *, double *, hipStream_t);
template void launch_density<float>(const abi_system_s *, const void *, int64_t, int, int, void *,
                                    const double *, double *, hipStream_t);

template void launch_adjoint_local<double>(const abi_system_s *, const void *, int64_t, const void *,
                                           int64_t, const void *, int64_t, double, void *, int64_t,
                                           int, int, void *, void *, const void *, double, double,
                                           const void *, int64_t, double *, hipStream_t);
template void launch_adjoint_local<float>(const abi_system_s *, const void *, int64_t, const void *,
                                          int64_t, const void *, int64_t, double, void *, int64_t,
                                          int, int, void *, void *, const void *, double, double,
                                          const void *, int64_t, double *, hipStream_t);

template void launch_local_potential<double>(const abi_system_s *, const void *, int64_t,
                                             const void *, int64_t, void *, int64_t, int, int,
                                             void *, const void *, double, double, double,
                                             hipStream_t, Profiler *, const void *, int64_t,
                                             void *, int64_t, int64_t);
template void launch_local_potential<float>(const abi_system_s *, const void *, int64_t,
                                             const void *, int64_t, void *, int64_t, int, int,
                                             void *, const void *, double, double, double,
                                             hipStream_t, Profiler *, const void *, int64_t,
                                             void *, int64_t, int64_t);

int fft_stage_threads(const Plan1D &pl, int npen) { return stage_need(pl, npen); }

}  // namespace chebfi
