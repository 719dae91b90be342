// Contour-integral filter (Sakurai-Sugiura), FP64 complex.
//
// The paper names a Sakurai-Sugiura eigensolver as a candidate for the fast
// iterations (section 3) without details; this is the published method's
// first moment with Rayleigh-Ritz extraction: for the reduced C = L^{-1} A L^{-H}
// and a circle through a < b on the real axis, the spectral projector onto
// the eigenvalues inside is approximated by the trapezoidal rule
//     Y = sum_j w_j (z_j I - C)^{-1} V,
//     z_j = gamma + rho e^{i t_j},  w_j = rho e^{i t_j} / nq,  t_j = 2 pi (j + 1/2) / nq,
// which acts on an eigenvector with eigenvalue lambda as 1 / (1 + t^nq),
// t = (lambda - gamma) / rho.
//
// Each shifted matrix M_j = z_j I - C is factored once, M_j = L_j U_j, without
// row exchanges: -i M_j has Hermitian part Im(z_j) I, positive definite, so
// every leading block is nonsingular and the growth stays bounded.  The
// factorisation is right-looking by 256-wide panels: inside a panel one
// work-group factors each 64 x 64 diagonal block in registers and writes the
// inverses of its two triangles, the block's column and row pieces are
// products with those inverses, and the trailing matrix gets one FP64
// matrix-core GEMM per panel (K = 256).  The nq factorisations are
// independent and run on four streams (the caller's and three more), so one
// factorisation's latency-bound diagonal blocks overlap another's GEMMs.
// Applying the filter is two triangular solves per node (the existing
// recursive lower solve with the unit-lower block inverses, and an upper solve
// written here), accumulated with the complex weights into one partial sum per
// stream.
//
// The FP32 form takes the nodes in step instead, every launch of the chain
// serving all of them (the solves: up to eight at a time): the chain is bound by
// the latency of its small launches, and nq products in one launch take little
// longer than one.  n = 1100, 8 nodes: 2280 products of 12 us on four streams
// became 285 of 14 us on one, the solve 27.7 -> 12.9 ms.
#include <cmath>
#include <vector>

#include "common.h"

namespace {
constexpr int NB = 64;
constexpr int QSTREAMS = 4;
constexpr int64_t GRID_Y_MAX = 65535;  // column kernels put the column index in grid.y

typedef float2 zf;

// complex element types of the factorisation: FP64 (zd) and FP32 (zf)
template <class T> struct Cx;
template <> struct Cx<zd> {
  typedef double R;
  static __device__ __forceinline__ zd mk(double re, double im) { return make_double2(re, im); }
};
template <> struct Cx<zf> {
  typedef float R;
  static __device__ __forceinline__ zf mk(float re, float im) { return make_float2(re, im); }
};

template <class T>
__device__ __forceinline__ T zmul(T a, T b) {
  return Cx<T>::mk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// One 64 x 64 diagonal block (kb <= 64 rows and columns in use, the rest padded
// with the identity): M = L U in place without row exchanges (L unit lower, stored
// strictly below the diagonal), then inv(L) into DinvL and inv(U) into DinvU (64 x
// 64 each, leading dimension ldi).  *info receives goff + the first failing pivot
// (1-based); one work-group per matrix of a batch.
//
// A chain of 64 pivots, bound by its latency.  Wave 0 factors 16-wide panels of
// all rows in registers (a lane holds its row's 16 entries; the pivot row comes
// from its lane by lane reads, no barrier); the row block right of the panel and
// the trailing update follow from the LDS, on one and on all four waves.  The
// eight 16 x 16 diagonal blocks of the inverses take one wave each for L and for U
// (16 lanes a block, a column each); the blocks off the diagonal are built outward,
// X_IJ = -X_II sum L_IK X_KJ and alike for U, a wave a block.  FP32: 49 us (102 with
// a barrier per pivot and 1024 threads, whose instructions bound it); contour solve
// n = 1100 10.6 -> 9.6 ms.
constexpr int PB = 16, SLD = NB + 1;  // panel width; leading dimension in the LDS

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  const unsigned long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, lane);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), lane);
  return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}
// a - b c, a + b c
template <class T>
__device__ __forceinline__ T sub_mul(T a, T b, T c) {
  return Cx<T>::mk(fma(b.y, c.y, fma(-b.x, c.x, a.x)), fma(-b.y, c.x, fma(-b.x, c.y, a.y)));
}
template <class T>
__device__ __forceinline__ T add_mul(T a, T b, T c) {
  return Cx<T>::mk(fma(-b.y, c.y, fma(b.x, c.x, a.x)), fma(b.y, c.x, fma(b.x, c.y, a.y)));
}
// by value: a conditional between lvalues would be a choice of addresses
template <class T>
__device__ __forceinline__ T pick(bool c, T a, T b) {
  return Cx<T>::mk(c ? a.x : b.x, c ? a.y : b.y);
}

template <class T>
__global__ __launch_bounds__(256) void k_getrf_block(T* M, int64_t ldm, int kb, T* DinvL, T* DinvU,
                                                     int64_t ldi, int* info, int goff, int64_t sM,
                                                     int64_t sD) {
  typedef typename Cx<T>::R R;
  __shared__ T S[NB * SLD];   // the block, then its factors, [column][row]
  __shared__ T X[NB * SLD];   // inv(L) strictly below, inv(U) on and above the diagonal
  __shared__ T W[4][PB * (PB + 1)];
  M += blockIdx.x * sM;
  DinvL += blockIdx.x * sD;
  DinvU += blockIdx.x * sD;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const T zero = Cx<T>::mk(R(0), R(0)), one = Cx<T>::mk(R(1), R(0));
  {
    T v[NB * NB / 256];
#pragma unroll
    for (int q = 0; q < NB * NB / 256; ++q) {
      const int j = wave + 4 * q;
      v[q] = pick(lane == j, one, zero);
      if (lane < kb && j < kb) v[q] = M[lane + (int64_t)j * ldm];
    }
#pragma unroll
    for (int q = 0; q < NB * NB / 256; ++q) S[(wave + 4 * q) * SLD + lane] = v[q];
  }
  __syncthreads();
  for (int p = 0; p < NB / PB; ++p) {
    const int d0 = p * PB, d1 = d0 + PB;
    if (wave == 0) {  // the panel
      T a[PB];
#pragma unroll
      for (int c = 0; c < PB; ++c) a[c] = S[(d0 + c) * SLD + lane];
      int bad = 0;
#pragma unroll
      for (int j = 0; j < PB; ++j) {
        const R pr = lane_value(a[j].x, d0 + j), pi = lane_value(a[j].y, d0 + j);
        const R d = pr * pr + pi * pi;
        if (bad == 0 && (!(d > R(0)) || !isfinite(d))) bad = j + 1;
        const T l = zmul(a[j], Cx<T>::mk(pr / d, -pi / d));
        const bool below = lane > d0 + j;
        a[j] = pick(below, l, a[j]);
        const T lm = pick(below, l, zero);
#pragma unroll
        for (int c = j + 1; c < PB; ++c)
          a[c] = sub_mul(a[c], lm, Cx<T>::mk(lane_value(a[c].x, d0 + j), lane_value(a[c].y, d0 + j)));
      }
      if (bad && lane == 0) atomicMin(info, goff + d0 + bad);
      if (lane >= d0) {
#pragma unroll
        for (int c = 0; c < PB; ++c) S[(d0 + c) * SLD + lane] = a[c];
      }
    }
    __syncthreads();
    if (wave == 0 && d1 + lane < NB) {  // rows of the panel right of it: a lane a column
      T x[PB];
      T* col = S + (d1 + lane) * SLD + d0;
#pragma unroll
      for (int r = 0; r < PB; ++r) x[r] = col[r];
      int o = 0;
#pragma unroll
      for (int k = 0; k < PB - 1; ++k) {
        // the reads' address waits for the step before: all of them at once would
        // not fit the registers
        if (k > 0) asm volatile("" : "+v"(o) : "v"(x[k].x));
        const T* lk = S + (d0 + k) * SLD + d0 + o;
#pragma unroll
        for (int r = k + 1; r < PB; ++r) x[r] = sub_mul(x[r], x[k], lk[r]);
      }
#pragma unroll
      for (int r = 0; r < PB; ++r) col[r] = x[r];
    }
    __syncthreads();
    const int left = NB / PB - 1 - p;  // trailing blocks a side
    for (int t = wave; t < left * left; t += 4) {
      const int I = p + 1 + t % left, J = p + 1 + t / left;
      T* out = S + (J * PB + l16) * SLD + I * PB + 4 * lg;
      T acc[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = out[i];
#pragma unroll
      for (int k = 0; k < PB; ++k) {
        const T u = S[(J * PB + l16) * SLD + d0 + k];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = sub_mul(acc[i], S[(d0 + k) * SLD + I * PB + 4 * lg + i], u);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i] = acc[i];
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NB * NB / 256; ++q) {
    const int j = wave + 4 * q;
    if (lane < kb && j < kb) M[lane + (int64_t)j * ldm] = S[j * SLD + lane];
  }
  if (wave < 2) {  // diagonal blocks of inv(L) (wave 0) and inv(U): block lg, column l16
    T x[PB];
    const T* B = S + lg * PB * SLD + lg * PB;
    int o = 0;
#pragma unroll
    for (int r = 0; r < PB; ++r) x[r] = pick(r == l16, one, zero);
    if (wave == 0) {
#pragma unroll
      for (int k = 0; k < PB - 1; ++k) {
        if (k > 0) asm volatile("" : "+v"(o) : "v"(x[k].x));
        const T* col = B + k * SLD + o;
#pragma unroll
        for (int r = k + 1; r < PB; ++r) x[r] = sub_mul(x[r], x[k], col[r]);
      }
    } else {
#pragma unroll
      for (int k = PB - 1; k >= 0; --k) {
        if (k < PB - 1) asm volatile("" : "+v"(o) : "v"(x[k].x));
        const T* col = B + k * SLD + o;
        const T u = col[k];
        const R d = u.x * u.x + u.y * u.y;
        x[k] = zmul(x[k], Cx<T>::mk(u.x / d, -u.y / d));
#pragma unroll
        for (int r = 0; r < k; ++r) x[r] = sub_mul(x[r], x[k], col[r]);
      }
    }
    T* out = X + (lg * PB + l16) * SLD + lg * PB;
#pragma unroll
    for (int r = 0; r < PB; ++r)
      if ((wave == 0) == (r > l16)) out[r] = x[r];
  }
  __syncthreads();
  for (int d = 1; d < NB / PB; ++d) {
    const int side = NB / PB - d;  // blocks of L at this distance from the diagonal, as many of U
    for (int t = wave; t < 2 * side; t += 4) {
      const bool low = t < side;
      const int q = low ? t : t - side, I = low ? q + d : q, J = low ? q : q + d;
      T acc[4] = {zero, zero, zero, zero};
      // rows 4 lg + i, column l16
      const int K0 = low ? J : I + 1, K1 = low ? I : J + 1;
      for (int K = K0; K < K1; ++K) {
#pragma unroll
        for (int k = 0; k < PB; ++k) {
          T x = X[(J * PB + l16) * SLD + K * PB + k];
          if (K == J) x = low ? pick(k == l16, one, pick(k > l16, x, zero)) : pick(k <= l16, x, zero);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[i] = add_mul(acc[i], S[(K * PB + k) * SLD + I * PB + 4 * lg + i], x);
        }
      }
      T* w = W[wave];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        w[l16 * (PB + 1) + 4 * lg + i] = acc[i];
        acc[i] = zero;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int k = 0; k < PB; ++k) {
        const T v = w[l16 * (PB + 1) + k];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = 4 * lg + i;
          T x = X[(I * PB + k) * SLD + I * PB + m];
          x = low ? pick(k == m, one, pick(k < m, x, zero)) : pick(k >= m, x, zero);
          acc[i] = sub_mul(acc[i], x, v);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) X[(J * PB + l16) * SLD + I * PB + 4 * lg + i] = acc[i];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NB * NB / 256; ++q) {
    const int j = wave + 4 * q;
    const T x = X[j * SLD + lane];
    if (lane < kb) {
      DinvL[lane + (int64_t)j * ldi] = pick(lane > j, x, pick(lane == j, one, zero));
      DinvU[lane + (int64_t)j * ldi] = pick(lane <= j, x, zero);
    }
  }
}

// M = z I - C (n x n, both full storage)
__global__ __launch_bounds__(256) void k_shift_neg(int64_t n, const zd* __restrict__ C, int64_t ldc,
                                                   double zr, double zi, zd* __restrict__ M,
                                                   int64_t ldm) {
  const int64_t j = blockIdx.y;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const zd c = C[i + j * ldc];
    M[i + j * ldm] = (i == j) ? make_double2(zr - c.x, zi - c.y) : make_double2(-c.x, -c.y);
  }
}

// Y = w T (first) or Y += w T, complex scalar w, rows x cols
__global__ __launch_bounds__(256) void k_zaxpy_cols(int64_t rows, double wr, double wi,
                                                    const zd* __restrict__ T, int64_t ldt,
                                                    zd* __restrict__ Y, int64_t ldy, int first) {
  const int64_t j = blockIdx.y;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < rows; i += (int64_t)gridDim.x * 256) {
    const zd t = T[i + j * ldt];
    const zd v = make_double2(wr * t.x - wi * t.y, wr * t.y + wi * t.x);
    if (first) {
      Y[i + j * ldy] = v;
    } else {
      const zd y = Y[i + j * ldy];
      Y[i + j * ldy] = make_double2(y.x + v.x, y.y + v.y);
    }
  }
}

// Y = S1 + S2 + ... (up to QSTREAMS partial sums, column-major rows x cols)
__global__ __launch_bounds__(256) void k_sum_parts(int64_t rows, int parts, const zd* __restrict__ S,
                                                   int64_t lds, int64_t pstride, zd* __restrict__ Y,
                                                   int64_t ldy) {
  const int64_t j = blockIdx.y;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < rows; i += (int64_t)gridDim.x * 256) {
    zd s = S[i + j * lds];
    for (int p = 1; p < parts; ++p) {
      const zd t = S[p * pstride + i + j * lds];
      s.x += t.x;
      s.y += t.y;
    }
    Y[i + j * ldy] = s;
  }
}

// ---- residual-correction form in FP32.  For a Ritz pair (theta, q) with
// residual r = C q - theta q, (z I - C)^{-1} q = [q + (z I - C)^{-1} r] / (z - theta),
// so sum_j w_j (z_j I - C)^{-1} q = f(theta) q + sum_j w_j (z_j I - C)^{-1} r / (z_j - theta)
// with f(theta) = sum_j w_j / (z_j - theta).  Only the second term goes through
// the FP32 factorisations; its rounding error is relative to |r|, which
// shrinks as the pairs converge.

// M_q = z_q I - C in complex64 for every node q (C complex128, full storage)
__global__ __launch_bounds__(256) void k_shift_neg32(int64_t n, const zd* __restrict__ C, int64_t ldc,
                                                     const zd* __restrict__ z, int nq, zf* __restrict__ M,
                                                     int64_t ldm, int64_t stride) {
  const int64_t j = blockIdx.y;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const zd c = C[i + j * ldc];
    for (int q = 0; q < nq; ++q)
      M[q * stride + i + j * ldm] = (i == j) ? make_float2((float)(z[q].x - c.x), (float)(z[q].y - c.y))
                                             : make_float2((float)-c.x, (float)-c.y);
  }
}

// T_q(:, j) = R(:, j) / (z_q - theta_j), rounded to complex64, for nq nodes
__global__ __launch_bounds__(256) void k_scale_to32(int64_t rows, const zd* __restrict__ R, int64_t ldr,
                                                    const double* __restrict__ theta,
                                                    const zd* __restrict__ z, int nq, zf* __restrict__ T,
                                                    int64_t ldt, int64_t stride) {
  const int64_t j = blockIdx.y;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < rows; i += (int64_t)gridDim.x * 256) {
    const zd r = R[i + j * ldr];
    for (int q = 0; q < nq; ++q) {
      const double a = z[q].x - theta[j], b = z[q].y;
      const double d = a * a + b * b;
      const double sr = a / d, si = -b / d;  // 1 / (z - theta_j)
      T[q * stride + i + j * ldt] = make_float2((float)(r.x * sr - r.y * si), (float)(r.x * si + r.y * sr));
    }
  }
}

// S = (S_before unless first) + sum over nodes [q0, q1) of w_q T_q; the last
// call adds f(theta_j) Q(:, j), f(theta) = sum_q w_q / (z_q - theta) (zw: nq nodes,
// then nq weights), and writes Y instead of Acc
__global__ __launch_bounds__(256) void k_contour_sum(int64_t rows, int q0, int q1, int nq,
                                                     const zd* __restrict__ zw, const zf* __restrict__ T,
                                                     int64_t ldt, int64_t stride, zd* __restrict__ Acc,
                                                     int64_t lda, const zd* __restrict__ Q, int64_t ldq,
                                                     const double* __restrict__ theta,
                                                     zd* __restrict__ Y, int64_t ldy) {
  const int64_t j = blockIdx.y;
  double fr = 0.0, fi = 0.0;
  if (q1 == nq)
    for (int q = 0; q < nq; ++q) {
      const zd z = zw[q], w = zw[nq + q];
      const double a = z.x - theta[j], b = z.y, d = a * a + b * b;
      fr += (w.x * a + w.y * b) / d;
      fi += (w.y * a - w.x * b) / d;
    }
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < rows; i += (int64_t)gridDim.x * 256) {
    zd s = make_double2(0.0, 0.0);
    if (q0 > 0) s = Acc[i + j * lda];
    for (int q = q0; q < q1; ++q) {
      const zf t = T[(q - q0) * stride + i + j * ldt];
      const zd w = zw[nq + q];
      s.x += w.x * t.x - w.y * t.y;
      s.y += w.x * t.y + w.y * t.x;
    }
    if (q1 == nq) {
      const zd qv = Q[i + j * ldq];
      Y[i + j * ldy] = make_double2(s.x + (fr * qv.x - fi * qv.y), s.y + (fr * qv.y + fi * qv.x));
    } else {
      Acc[i + j * lda] = s;
    }
  }
}

// R(:, j) = W(:, perm[j]) - theta[perm[j]] Qp(:, j) for j in [s0, m); thp[j] = theta[perm[j]]
__global__ __launch_bounds__(256) void k_contour_residual(int64_t rows, int64_t s0, const int* __restrict__ perm,
                                                          const zd* __restrict__ W, int64_t ldw,
                                                          const double* __restrict__ theta,
                                                          const zd* __restrict__ Qp, int64_t ldq,
                                                          zd* __restrict__ R, int64_t ldr,
                                                          double* __restrict__ thp) {
  const int64_t j = s0 + blockIdx.y;
  const int pj = perm[j];
  const double th = theta[pj];
  if (blockIdx.x == 0 && threadIdx.x == 0) thp[j] = th;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < rows; i += (int64_t)gridDim.x * 256) {
    const zd w = W[i + (int64_t)pj * ldw], q = Qp[i + j * ldq];
    R[i + j * ldr] = make_double2(w.x - th * q.x, w.y - th * q.y);
  }
}

// coefficient columns of the FP32 products: ones, minus ones, zeros (n each)
__global__ void k_fill_coefs(int64_t n, double* co) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    co[i] = 1.0;
    co[n + i] = -1.0;
    co[2 * n + i] = 0.0;
  }
}

inline dim3 grid_cols(int64_t rows, int64_t cols) {
  int64_t gx = (rows + 255) / 256;
  if (gx > 16) gx = 16;
  return dim3((unsigned)gx, (unsigned)cols);
}

inline int64_t split64(int64_t n) { return ((n / 2 + NB - 1) / NB) * NB; }

// quadrature stream i of the handle (created once, non-blocking, default priority)
gevp_status quad_ctx(gevp_ctx* c, int i, gevp_ctx** out) {
  while ((int)c->qctx.size() <= i) {
    gevp_ctx* w = new gevp_ctx();
    w->device = c->device;
    if (hipStreamCreateWithFlags(&w->stream, hipStreamNonBlocking) != hipSuccess) {
      delete w;
      return GEVP_ERR_HIP;
    }
    w->owns_stream = true;
    w->inner_streams = false;
    w->parent = c;
    c->qctx.push_back(w);
    ext_assign(c, w, SLOT_QUAD0 + (int)c->qctx.size() - 1);
  }
  *out = c->qctx[i];
  return GEVP_OK;
}

// The nodes run on c's own stream and up to QSTREAMS - 1 further streams
// (c's stream is idle meanwhile; with four hardware queues per process, more
// streams would share queues and serialise).  The further streams start after
// the work queued on c's stream; every exit waits for them (they write
// workspace the next call reuses).
struct QuadStreams {
  gevp_ctx* c;
  int count = 0;
  gevp_ctx* s[QSTREAMS] = {};
  hipEvent_t fork = nullptr, join[QSTREAMS] = {};
  explicit QuadStreams(gevp_ctx* ctx) : c(ctx) {}
  gevp_status open(int want) {
    s[0] = c;
    count = (!c->inner_streams || want <= 1) ? 1 : (want < QSTREAMS ? want : QSTREAMS);
    if (count == 1) return GEVP_OK;
    GEVP_HIP_TRY(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
    GEVP_HIP_TRY(hipEventRecord(fork, c->stream));
    for (int q = 1; q < count; ++q) {
      GEVP_TRY(quad_ctx(c, q - 1, &s[q]));
      GEVP_HIP_TRY(hipEventCreateWithFlags(&join[q], hipEventDisableTiming));
      GEVP_HIP_TRY(hipStreamWaitEvent(s[q]->stream, fork, 0));
    }
    return GEVP_OK;
  }
  gevp_status close() {
    for (int q = 1; q < count; ++q) {
      GEVP_HIP_TRY(hipEventRecord(join[q], s[q]->stream));
      GEVP_HIP_TRY(hipStreamWaitEvent(c->stream, join[q], 0));
    }
    return GEVP_OK;
  }
  ~QuadStreams() {
    for (int q = 1; q < count; ++q)
      if (s[q]) (void)hipStreamSynchronize(s[q]->stream);
    if (fork) (void)hipEventDestroy(fork);
    for (hipEvent_t e : join)
      if (e) (void)hipEventDestroy(e);
  }
};

struct ContourLayout {
  zd* LU;
  zd* DinvL;
  zd* DinvU;
  zd* T;    // per stream: n x m solve buffer
  zd* Acc;  // per stream: n x m partial sum
  int* info;
  size_t lu_stride, dinv_stride, blk_stride;
};

ContourLayout carve(void* work, int64_t n, int64_t m, int nq) {
  ContourLayout L;
  char* p = (char*)work;
  L.lu_stride = (size_t)n * n;
  L.dinv_stride = (size_t)n * NB;
  L.blk_stride = (size_t)n * m;
  L.LU = (zd*)p;
  p += ws_round(sizeof(zd) * L.lu_stride * nq);
  L.DinvL = (zd*)p;
  p += ws_round(sizeof(zd) * L.dinv_stride * nq);
  L.DinvU = (zd*)p;
  p += ws_round(sizeof(zd) * L.dinv_stride * nq);
  L.T = (zd*)p;
  p += ws_round(sizeof(zd) * L.blk_stride * QSTREAMS);
  L.Acc = (zd*)p;
  p += ws_round(sizeof(zd) * L.blk_stride * QSTREAMS);
  L.info = (int*)p;
  return L;
}

void node(double a, double b, int nq, int j, zd* z, zd* w) {
  const double gamma = 0.5 * (a + b), rho = 0.5 * (b - a);
  const double t = 6.283185307179586476925 * (j + 0.5) / nq;
  const double ct = std::cos(t), st = std::sin(t);
  *z = make_double2(gamma + rho * ct, rho * st);
  *w = make_double2(rho * ct / nq, rho * st / nq);
}

}  // namespace

// ---------------------------------------------------------------------------

gevp_status lu_nopiv(gevp_ctx* c, int64_t n, zd* M, int64_t ldm, zd* DinvL, zd* DinvU,
                     int64_t ldi, int* info_dev) {
  // Panels of PW columns; inside a panel a right-looking LU by 64-wide blocks
  // restricted to the panel's columns; then the panel's row block
  // U12 = L11^{-1} A12 by the recursive lower solve, and one trailing update
  // with K = PW (a K = 64 update per block would re-read and re-write the
  // trailing matrix four times as often: HBM-bound at about 30 TFLOP/s).
  constexpr int64_t PW = 256;
  for (int64_t r0 = 0; r0 < n; r0 += PW) {
    const int64_t kb = std::min<int64_t>(PW, n - r0);
    const int64_t pend = r0 + kb;  // first column after the panel
    for (int64_t s0 = r0; s0 < pend; s0 += NB) {
      const int64_t sb = std::min<int64_t>(NB, pend - s0);
      const int64_t below = n - s0 - sb, pc = pend - s0 - sb;
      zd* Mss = M + s0 + s0 * ldm;
      hipLaunchKernelGGL(k_getrf_block<zd>, dim3(1), dim3(256), 0, c->stream, Mss, ldm, (int)sb,
                         DinvL + s0, DinvU + s0, ldi, info_dev, (int)s0, (int64_t)0, (int64_t)0);
      GEVP_HIP_TRY(hipGetLastError());
      zd* A21 = Mss + sb;
      zd* A12 = Mss + sb * ldm;
      // L21 = A21 U11^{-1} and U12 = L11^{-1} A12 in place (one 64-wide
      // output tile side: every tile reads its whole K range before it writes)
      if (below > 0)
        GEVP_TRY(launch_zgemm(c, 0, 0, below, sb, sb, 1.0, A21, ldm, DinvU + s0, ldi, 0.0, nullptr,
                              0, 0.0, nullptr, 0, nullptr, A21, ldm));
      if (pc > 0) {
        GEVP_TRY(launch_zgemm(c, 0, 0, sb, pc, sb, 1.0, DinvL + s0, ldi, A12, ldm, 0.0, nullptr, 0,
                              0.0, nullptr, 0, nullptr, A12, ldm));
        if (below > 0)
          GEVP_TRY(launch_zgemm(c, 0, 0, below, pc, sb, -1.0, A21, ldm, A12, ldm, 1.0, Mss + sb + sb * ldm,
                                ldm, 0.0, nullptr, 0, nullptr, Mss + sb + sb * ldm, ldm));
      }
    }
    const int64_t rest = n - pend;
    if (rest > 0) {
      zd* Mrr = M + r0 + r0 * ldm;
      zd* A12 = Mrr + kb * ldm;
      GEVP_TRY(trsm_left_lower_n(c, kb, rest, Mrr, ldm, DinvL + r0, ldi, A12, ldm));
      GEVP_TRY(launch_zgemm(c, 0, 0, rest, rest, kb, -1.0, Mrr + kb, ldm, A12, ldm, 1.0,
                            Mrr + kb + kb * ldm, ldm, 0.0, nullptr, 0, nullptr, Mrr + kb + kb * ldm,
                            ldm));
    }
  }
  return GEVP_OK;
}

// R (n x m) <- U^{-1} R, U upper triangular (the upper part of a packed LU)
gevp_status trsm_left_upper_n(gevp_ctx* c, int64_t n, int64_t m, const zd* U, int64_t ldu,
                              const zd* DinvU, int64_t ldi, zd* R, int64_t ldr) {
  if (n <= 0 || m <= 0) return GEVP_OK;
  if (n <= NB)
    return launch_zgemm(c, 0, 0, n, m, n, 1.0, DinvU, ldi, R, ldr, 0.0, nullptr, 0, 0.0, nullptr,
                        0, nullptr, R, ldr);
  const int64_t h = split64(n);
  GEVP_TRY(trsm_left_upper_n(c, n - h, m, U + h + h * ldu, ldu, DinvU + h, ldi, R + h, ldr));
  // R1 -= U12 R2   (U12 = U[:h, h:])
  GEVP_TRY(launch_zgemm(c, 0, 0, h, m, n - h, -1.0, U + h * ldu, ldu, R + h, ldr, 1.0, R, ldr, 0.0,
                        nullptr, 0, nullptr, R, ldr));
  return trsm_left_upper_n(c, h, m, U, ldu, DinvU, ldi, R, ldr);
}

// ---- FP32 factorisation and solves (products on the FP32 matrix cores by the
// general form of the complex64 filter kernel: D = alpha A G + gamma P with
// per-column coefficient vectors taken from co = [ones | minus ones | zeros])

namespace {
struct Co32 {
  const double *one, *mone, *zero;
};

// one matrix of every node, at a constant stride
struct Mats {
  zf* p;
  int64_t ld, stride;
  Mats at(int64_t i, int64_t j) const { return {p + i + j * ld, ld, stride}; }
};

// D = alpha A G (+ P when acc) for every node: m x n, inner dimension k
gevp_status gemm32(gevp_ctx* c, int nodes, int64_t m, int64_t n, int64_t k, Mats A, Mats G, Mats D, bool minus,
                   bool acc, const Co32& co) {
  return launch_cgemm32_filter(c, m, n, k, A.p, A.ld, G.p, G.ld, D.p, D.ld, D.p, D.ld, D.p, D.ld,
                               minus ? co.mone : co.one, co.zero, acc ? co.one : co.zero, co.zero, nodes,
                               A.stride, G.stride, D.stride);
}

gevp_status trsm32_lower(gevp_ctx* c, int nodes, int64_t n, int64_t m, Mats L, Mats Dinv, Mats R,
                         const Co32& co) {
  if (n <= 0 || m <= 0) return GEVP_OK;
  if (n <= NB) return gemm32(c, nodes, n, m, n, Dinv, R, R, false, false, co);
  const int64_t h = split64(n);
  GEVP_TRY(trsm32_lower(c, nodes, h, m, L, Dinv, R, co));
  GEVP_TRY(gemm32(c, nodes, n - h, m, h, L.at(h, 0), R, R.at(h, 0), true, true, co));
  return trsm32_lower(c, nodes, n - h, m, L.at(h, h), Dinv.at(h, 0), R.at(h, 0), co);
}

gevp_status trsm32_upper(gevp_ctx* c, int nodes, int64_t n, int64_t m, Mats U, Mats Dinv, Mats R,
                         const Co32& co) {
  if (n <= 0 || m <= 0) return GEVP_OK;
  if (n <= NB) return gemm32(c, nodes, n, m, n, Dinv, R, R, false, false, co);
  const int64_t h = split64(n);
  GEVP_TRY(trsm32_upper(c, nodes, n - h, m, U.at(h, h), Dinv.at(h, 0), R.at(h, 0), co));
  GEVP_TRY(gemm32(c, nodes, h, m, n - h, U.at(0, h), R.at(h, 0), R, true, true, co));
  return trsm32_upper(c, nodes, h, m, U, Dinv, R, co);
}

// the FP32 counterpart of lu_nopiv (same panels and block kernel) for all nodes
// in step: every launch of the chain serves them all
gevp_status lu_nopiv32(gevp_ctx* c, int nodes, int64_t n, Mats M, Mats DinvL, Mats DinvU, int* info_dev,
                       const Co32& co) {
  constexpr int64_t PW = 256;
  for (int64_t r0 = 0; r0 < n; r0 += PW) {
    const int64_t kb = std::min<int64_t>(PW, n - r0);
    const int64_t pend = r0 + kb;
    for (int64_t s0 = r0; s0 < pend; s0 += NB) {
      const int64_t sb = std::min<int64_t>(NB, pend - s0);
      const int64_t below = n - s0 - sb, pc = pend - s0 - sb;
      const Mats A11 = M.at(s0, s0), dl = DinvL.at(s0, 0), du = DinvU.at(s0, 0);
      hipLaunchKernelGGL(k_getrf_block<zf>, dim3((unsigned)nodes), dim3(256), 0, c->stream, A11.p, M.ld, (int)sb,
                         dl.p, du.p, dl.ld, info_dev, (int)s0, M.stride, dl.stride);
      GEVP_HIP_TRY(hipGetLastError());
      const Mats A21 = A11.at(sb, 0), A12 = A11.at(0, sb), A22 = A11.at(sb, sb);
      if (below > 0) GEVP_TRY(gemm32(c, nodes, below, sb, sb, A21, du, A21, false, false, co));
      if (pc > 0) {
        GEVP_TRY(gemm32(c, nodes, sb, pc, sb, dl, A12, A12, false, false, co));
        if (below > 0) GEVP_TRY(gemm32(c, nodes, below, pc, sb, A21, A12, A22, true, true, co));
      }
    }
    const int64_t rest = n - pend;
    if (rest > 0) {
      const Mats A11 = M.at(r0, r0), A12 = M.at(r0, pend);
      GEVP_TRY(trsm32_lower(c, nodes, kb, rest, A11, DinvL.at(r0, 0), A12, co));
      GEVP_TRY(gemm32(c, nodes, rest, rest, kb, M.at(pend, r0), A12, M.at(pend, pend), true, true, co));
    }
  }
  return GEVP_OK;
}

// nodes solved together in one application (their solve buffers and the partial
// sum take the room of the workspace's four buffers of both kinds)
constexpr int GROUP32 = 8;

struct Contour32Layout {
  zf* LU;
  zf* DinvL;
  zf* DinvU;
  zd* Acc;  // n x m complex128 partial sum
  zf* T;    // per node of a group: n x m complex64 solve buffer
  double* co;
  zd* zw;
  int* info;
  size_t lu_stride, dinv_stride, blk_stride;
};

Contour32Layout carve32(void* work, int64_t n, int64_t m, int nq) {
  Contour32Layout L;
  char* p = (char*)work;
  L.lu_stride = (size_t)n * n;
  L.dinv_stride = (size_t)n * NB;
  L.blk_stride = (size_t)n * m;
  L.LU = (zf*)p;
  p += ws_round(sizeof(zf) * L.lu_stride * nq);
  L.DinvL = (zf*)p;
  p += ws_round(sizeof(zf) * L.dinv_stride * nq);
  L.DinvU = (zf*)p;
  p += ws_round(sizeof(zf) * L.dinv_stride * nq);
  static_assert(sizeof(zd) + GROUP32 * sizeof(zf) <= QSTREAMS * (sizeof(zf) + sizeof(zd)), "");
  L.Acc = (zd*)p;
  L.T = (zf*)(L.Acc + L.blk_stride);
  p += ws_round(sizeof(zf) * L.blk_stride * QSTREAMS);
  p += ws_round(sizeof(zd) * L.blk_stride * QSTREAMS);
  L.co = (double*)p;
  p += ws_round(sizeof(double) * 3 * n);
  L.zw = (zd*)p;
  p += ws_round(sizeof(zd) * 2 * nq);
  L.info = (int*)p;
  return L;
}

// nodes, then weights, in device memory
gevp_status upload_nodes(gevp_ctx* c, double a, double b, int nq, zd* dst) {
  std::vector<zd> zw(2 * nq);
  for (int j = 0; j < nq; ++j) node(a, b, nq, j, &zw[j], &zw[nq + j]);
  GEVP_HIP_TRY(hipMemcpyAsync(dst, zw.data(), sizeof(zd) * 2 * nq, hipMemcpyHostToDevice, c->stream));
  return GEVP_OK;
}
}  // namespace

size_t contour32_work_bytes(int64_t n, int64_t m, int nq) {
  return ws_round(sizeof(zf) * (size_t)n * n * nq) + 2 * ws_round(sizeof(zf) * (size_t)n * NB * nq) +
         ws_round(sizeof(zf) * (size_t)n * m * QSTREAMS) +
         ws_round(sizeof(zd) * (size_t)n * m * QSTREAMS) + ws_round(sizeof(double) * 3 * n) +
         ws_round(sizeof(zd) * 2 * nq) + ws_round(sizeof(int) * 4) + 256;
}

gevp_status contour_factor32(gevp_ctx* c, int64_t n, const zd* C, int64_t ldc, double a, double b,
                             int nq, void* work, int64_t mmax, int* pivot) {
  Contour32Layout L = carve32(work, n, mmax, nq);
  const Co32 co{L.co, L.co + n, L.co + 2 * n};
  hipLaunchKernelGGL(k_fill_coefs, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 64)), dim3(256), 0,
                     c->stream, n, L.co);
  GEVP_HIP_TRY(hipGetLastError());
  const int big = 0x7fffffff;
  GEVP_HIP_TRY(hipMemcpyAsync(L.info, &big, sizeof(int), hipMemcpyHostToDevice, c->stream));
  GEVP_TRY(upload_nodes(c, a, b, nq, L.zw));
  hipLaunchKernelGGL(k_shift_neg32, grid_cols(n, n), dim3(256), 0, c->stream, n, C, ldc, L.zw, nq, L.LU, n,
                     (int64_t)L.lu_stride);
  GEVP_HIP_TRY(hipGetLastError());
  const int64_t ds = (int64_t)L.dinv_stride;
  GEVP_TRY(lu_nopiv32(c, nq, n, Mats{L.LU, n, (int64_t)L.lu_stride}, Mats{L.DinvL, n, ds}, Mats{L.DinvU, n, ds},
                      L.info, co));
  int f = big;
  GEVP_HIP_TRY(hipMemcpyAsync(&f, L.info, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  GEVP_HIP_TRY(hipStreamSynchronize(c->stream));
  *pivot = (f == big) ? 0 : f;
  return GEVP_OK;
}

gevp_status contour_apply32(gevp_ctx* c, int64_t n, int64_t m, const zd* Q, int64_t ldq, const zd* R,
                            int64_t ldr, const double* theta, zd* Y, int64_t ldy, double a, double b,
                            int nq, void* work, int64_t mmax) {
  if (m <= 0) return GEVP_OK;
  Contour32Layout L = carve32(work, n, mmax, nq);
  const Co32 co{L.co, L.co + n, L.co + 2 * n};
  GEVP_TRY(upload_nodes(c, a, b, nq, L.zw));
  const int64_t ls = (int64_t)L.lu_stride, ds = (int64_t)L.dinv_stride, bs = (int64_t)L.blk_stride;
  const Mats T{L.T, n, bs};
  for (int q0 = 0; q0 < nq; q0 += GROUP32) {
    const int g = std::min(GROUP32, nq - q0);
    hipLaunchKernelGGL(k_scale_to32, grid_cols(n, m), dim3(256), 0, c->stream, n, R, ldr, theta, L.zw + q0, g,
                       L.T, n, bs);
    GEVP_HIP_TRY(hipGetLastError());
    const Mats LU{L.LU + ls * q0, n, ls};
    GEVP_TRY(trsm32_lower(c, g, n, m, LU, Mats{L.DinvL + ds * q0, n, ds}, T, co));
    GEVP_TRY(trsm32_upper(c, g, n, m, LU, Mats{L.DinvU + ds * q0, n, ds}, T, co));
    hipLaunchKernelGGL(k_contour_sum, grid_cols(n, m), dim3(256), 0, c->stream, n, q0, q0 + g, nq, L.zw, L.T, n,
                       bs, L.Acc, n, Q, ldq, theta, Y, ldy);
    GEVP_HIP_TRY(hipGetLastError());
  }
  return GEVP_OK;
}

gevp_status contour_residual(gevp_ctx* c, int64_t n, int64_t nb, int64_t s0, const int* perm,
                             const zd* W, int64_t ldw, const double* theta, const zd* Qp, int64_t ldq,
                             zd* R, int64_t ldr, double* thp) {
  if (s0 >= nb) return GEVP_OK;
  hipLaunchKernelGGL(k_contour_residual, grid_cols(n, nb - s0), dim3(256), 0, c->stream, n, s0, perm, W,
                     ldw, theta, Qp, ldq, R, ldr, thp);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

size_t contour_work_bytes(int64_t n, int64_t m, int nq) {
  return ws_round(sizeof(zd) * (size_t)n * n * nq) + 2 * ws_round(sizeof(zd) * (size_t)n * NB * nq) +
         2 * ws_round(sizeof(zd) * (size_t)n * m * QSTREAMS) + ws_round(sizeof(int) * 4) + 256;
}

gevp_status contour_factor(gevp_ctx* c, int64_t n, const zd* C, int64_t ldc, double a, double b,
                           int nq, void* work, int64_t mmax, int* pivot) {
  ContourLayout L = carve(work, n, mmax, nq);
  const int big = 0x7fffffff;
  GEVP_HIP_TRY(hipMemcpyAsync(L.info, &big, sizeof(int), hipMemcpyHostToDevice, c->stream));
  QuadStreams qs(c);
  GEVP_TRY(qs.open(nq));
  for (int j = 0; j < nq; ++j) {
    gevp_ctx* s = qs.s[j % qs.count];
    zd z, w;
    node(a, b, nq, j, &z, &w);
    zd* M = L.LU + L.lu_stride * j;
    hipLaunchKernelGGL(k_shift_neg, dim3((unsigned)((n + 255) / 256 < 16 ? (n + 255) / 256 : 16),
                                         (unsigned)n),
                       dim3(256), 0, s->stream, n, C, ldc, z.x, z.y, M, n);
    GEVP_HIP_TRY(hipGetLastError());
    GEVP_TRY(lu_nopiv(s, n, M, n, L.DinvL + L.dinv_stride * j, L.DinvU + L.dinv_stride * j, n,
                      L.info));
  }
  GEVP_TRY(qs.close());
  int f = big;
  GEVP_HIP_TRY(hipMemcpyAsync(&f, L.info, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  GEVP_HIP_TRY(hipStreamSynchronize(c->stream));
  *pivot = (f == big) ? 0 : f;
  return GEVP_OK;
}

gevp_status contour_apply(gevp_ctx* c, int64_t n, int64_t m, const zd* V, int64_t ldv, zd* Y,
                          int64_t ldy, double a, double b, int nq, void* work, int64_t mmax) {
  if (m <= 0) return GEVP_OK;
  ContourLayout L = carve(work, n, mmax, nq);
  QuadStreams qs(c);
  GEVP_TRY(qs.open(nq));
  std::vector<int> firsts(qs.count, 1);
  for (int j = 0; j < nq; ++j) {
    const int q = j % qs.count;
    gevp_ctx* s = qs.s[q];
    zd z, w;
    node(a, b, nq, j, &z, &w);
    zd* T = L.T + L.blk_stride * q;
    zd* Acc = L.Acc + L.blk_stride * q;
    const zd* LU = L.LU + L.lu_stride * j;
    GEVP_TRY(launch_copy2d(s, n, m, V, ldv, T, n));
    GEVP_TRY(trsm_left_lower_n(s, n, m, LU, n, L.DinvL + L.dinv_stride * j, n, T, n));
    GEVP_TRY(trsm_left_upper_n(s, n, m, LU, n, L.DinvU + L.dinv_stride * j, n, T, n));
    hipLaunchKernelGGL(k_zaxpy_cols, grid_cols(n, m), dim3(256), 0, s->stream, n, w.x, w.y, T, n,
                       Acc, n, firsts[q]);
    GEVP_HIP_TRY(hipGetLastError());
    firsts[q] = 0;
  }
  GEVP_TRY(qs.close());
  hipLaunchKernelGGL(k_sum_parts, grid_cols(n, m), dim3(256), 0, c->stream, n, qs.count, L.Acc, n,
                     (int64_t)L.blk_stride, Y, ldy);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

extern "C" {

gevp_status gevp_k_lu_shifted(gevp_handle h, int64_t n, const void* C, int64_t ldc, double zr,
                              double zi, void* LU, int64_t ldlu, int64_t* pivot) {
  if (!h || n < 1 || n > GRID_Y_MAX || !C || ldc < n || !LU || ldlu < n || !std::isfinite(zr) ||
      !std::isfinite(zi))
    return GEVP_ERR_INVALID;
  GEVP_HIP_TRY(hipSetDevice(h->device));
  GEVP_TRY(ws_reserve(h, 2 * ws_round(sizeof(zd) * n * NB) + ws_round(sizeof(int) * 4) + 256));
  zd* DL = (zd*)ws_take(h, sizeof(zd) * n * NB);
  zd* DU = (zd*)ws_take(h, sizeof(zd) * n * NB);
  int* info = (int*)ws_take(h, sizeof(int) * 4);
  const int big = 0x7fffffff;
  GEVP_HIP_TRY(hipMemcpyAsync(info, &big, sizeof(int), hipMemcpyHostToDevice, h->stream));
  hipLaunchKernelGGL(k_shift_neg, dim3((unsigned)((n + 255) / 256 < 16 ? (n + 255) / 256 : 16),
                                       (unsigned)n),
                     dim3(256), 0, h->stream, n, (const zd*)C, ldc, zr, zi, (zd*)LU, ldlu);
  GEVP_HIP_TRY(hipGetLastError());
  GEVP_TRY(lu_nopiv(h, n, (zd*)LU, ldlu, DL, DU, n, info));
  int f = big;
  GEVP_HIP_TRY(hipMemcpyAsync(&f, info, sizeof(int), hipMemcpyDeviceToHost, h->stream));
  GEVP_HIP_TRY(hipStreamSynchronize(h->stream));
  if (pivot) *pivot = (f == big) ? 0 : f;
  return (f == big) ? GEVP_OK : GEVP_ERR_SINGULAR;
}

gevp_status gevp_k_contour_filter(gevp_handle h, int64_t n, const void* C, int64_t ldc,
                                  const void* V, int64_t ldv, int64_t m, double a, double b, int nq,
                                  void* Y, int64_t ldy) {
  if (!h || n < 1 || n > GRID_Y_MAX || !C || ldc < n || !V || ldv < n || m < 0 ||
      m > GRID_Y_MAX || !Y || ldy < n)
    return GEVP_ERR_INVALID;
  if (!(a < b) || !std::isfinite(a) || !std::isfinite(b) || nq < 1 || nq > 256)
    return GEVP_ERR_INVALID;
  if (m == 0) return GEVP_OK;
  GEVP_HIP_TRY(hipSetDevice(h->device));
  GEVP_TRY(ws_reserve(h, contour_work_bytes(n, m, nq) + 256));
  void* work = ws_take(h, contour_work_bytes(n, m, nq));
  int piv = 0;
  GEVP_TRY(contour_factor(h, n, (const zd*)C, ldc, a, b, nq, work, m, &piv));
  if (piv) return GEVP_ERR_SINGULAR;
  GEVP_TRY(contour_apply(h, n, m, (const zd*)V, ldv, (zd*)Y, ldy, a, b, nq, work, m));
  GEVP_HIP_TRY(hipStreamSynchronize(h->stream));
  return GEVP_OK;
}

}  // extern "C"
