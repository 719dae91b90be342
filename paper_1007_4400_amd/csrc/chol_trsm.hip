// Cholesky factorisation and triangular solves, FP64 complex.
//
// The factorisation is right-looking in outer panels of 384 to 1024 columns, each
// in inner panels of 384, with one panel of lookahead on a second stream (see
// chol_lower); each 64 x 64 diagonal block is factored and inverted by one
// work-group.  The triangular solves
// recurse: every level splits the triangle in two halves (rounded to the
// 64-wide block), so the off-diagonal work is one large GEMM on the FP64
// matrix cores per level, and the base case applies a diagonal block's
// inverse with a GEMM (in place: a 64-wide block fits one output tile of the
// GEMM, so every tile reads its whole K range before it writes).
#include <cfloat>
#include <climits>

#include "common.h"

namespace {
constexpr int NB = 64;

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int PB = 16;       // panel width
constexpr int SLD = NB + 1;  // LDS column stride in complex entries (odd: rows spread over banks)
// L and inv(L) share one array: L in the lower triangle (column-major,
// S[c * SLD + r], r >= c), the strict lower triangle of inv(L) transposed into
// the upper one (X(i, j), i > j, at S[i * SLD + j]), inv(L)'s diagonal in a
// separate vector: 75 KB of LDS, so the factor fits on a compute unit next to
// one work-group of the FP64 trailing-update GEMM.
constexpr int TLD = 33;
struct Block64 {
  zd S[NB * SLD];
  zd Xd[NB];        // diagonal of inv(L)
  zd T[PB * TLD];   // the inverting wave's copy of a panel's columns
};

__device__ __forceinline__ double lane_value(double v, int lane) {
  const unsigned long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, lane);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), lane);
  return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}

// s = sqrt(d) and il = 1 / sqrt(d) for finite d > 0: the hardware estimate (24 bits)
// and one third-order step, a chain of five operations where the library's square
// root and division take over thirty (no product leaves the range for any d,
// subnormal ones included).  Off by 0.5000 and 0.93 units in the last place at most
// (exact rationals, 9000 random d, estimates of 24 to 28 bits); a division by the
// rounded root is off from 1 / sqrt(d) by up to 1.38.
__device__ __forceinline__ void sqrt_and_inverse(double d, double& s, double& il) {
  const double y = __builtin_amdgcn_rsq(d);
  const double e = fma(-(d * y), y, 1.0);
  il = fma(y * e, fma(e, 0.375, 0.5), y);
  const double t = d * il;
  s = fma(fma(-t, t, d), 0.5 * il, t);
}
// by value: a conditional between lvalues would be a choice of addresses, with
// the operands put in memory for it
__device__ __forceinline__ zd pick(bool c, zd a, zd b) {
  return make_double2(c ? a.x : b.x, c ? a.y : b.y);
}
// a - b conj(s), a - b s
__device__ __forceinline__ zd sub_mulc(zd a, zd b, zd s) {
  return make_double2(fma(-b.y, s.y, fma(-b.x, s.x, a.x)), fma(b.x, s.y, fma(-b.y, s.x, a.y)));
}
__device__ __forceinline__ zd sub_mul(zd a, zd b, zd s) {
  return make_double2(fma(b.y, s.y, fma(-b.x, s.x, a.x)), fma(-b.y, s.x, fma(-b.x, s.y, a.y)));
}

// A wave's part of a 16-column panel whose diagonal block starts at lane d0: a
// lane holds its row's 16 entries in registers, so a column is finished by
// every row at once, without a barrier.  The chain from pivot to pivot is what
// counts: the next two columns get their multipliers straight from the lanes
// that hold them; those of the others go through the LDS (broadcast reads of
// the finished columns in buf) and are applied one column later, beside the
// next pivot's chain.  Entries above the diagonal carry values no other row
// reads.  Returns the first failing pivot of the panel, or INT_MAX.
__device__ __forceinline__ int panel16(zd (&a)[PB], int d0, zd* buf, int ld, int slot) {
  const int lane = threadIdx.x & 63;
  zd f[2][PB];  // multipliers of this and the previous column
  double ljj, il;
  int bad = INT_MAX;
  auto pivot = [&](int j) {
    const double d = lane_value(a[j].x, d0 + j);
    const bool ok = d > 0.0 && d <= DBL_MAX;
    bad = ok ? bad : min(bad, j);
    sqrt_and_inverse(d, ljj, il);
    ljj = ok ? ljj : 1.0;
    il = ok ? il : 1.0;
  };
  pivot(0);
#pragma unroll
  for (int j = 0; j < PB; ++j) {
    a[j] = (lane == d0 + j) ? make_double2(ljj, 0.0) : make_double2(a[j].x * il, a[j].y * il);
    zd* col = buf + j * ld;
    col[slot] = a[j];
#pragma unroll
    for (int c = j + 3; c < PB; ++c) f[j & 1][c] = col[d0 + c];
#pragma unroll
    for (int c = j + 1; c < PB && c <= j + 2; ++c) {
      a[c] = sub_mulc(a[c], a[j], make_double2(lane_value(a[j].x, d0 + c), lane_value(a[j].y, d0 + c)));
      if (c == j + 1) pivot(c);
    }
    if (j > 0) {
#pragma unroll
      for (int c = j + 2; c < PB; ++c) a[c] = sub_mulc(a[c], a[j - 1], f[(j - 1) & 1][c]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  return bad;
}

// Block (I, J) of the trailing matrix: A_IJ -= L_Ip L_Jp^H by one wave on the
// matrix cores (above the diagonal of a diagonal block: values nobody reads)
__device__ __forceinline__ void update16(Block64& m, int I, int J, int p) {
  const int l16 = threadIdx.x & 15, lg = (threadIdx.x >> 4) & 3;
  zd* col = m.S + (J * PB + l16) * SLD + I * PB + lg;
  d4 re, im, re2 = {0, 0, 0, 0}, im2 = {0, 0, 0, 0};  // four chains: an MFMA's result takes two slots
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    re[r] = col[4 * r].x;
    im[r] = col[4 * r].y;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const zd* k = m.S + (p * PB + 4 * t + lg) * SLD + l16;
    const zd a = k[I * PB], b = k[J * PB];
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.x, b.x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.x, im, 0, 0, 0);
    re2 = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, re2, 0, 0, 0);
    im2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, im2, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) col[4 * r] = make_double2(re[r] + re2[r], im[r] + im2[r]);
}

// Inverse of diagonal block p by one wave, rd the reciprocals of L's diagonal:
// lane c % 16 substitutes forward for column c, columns of L being broadcast
// reads.
__device__ __forceinline__ void invert16(Block64& m, const zd* rd, int p) {
  const int lane = threadIdx.x & 63, c = lane & 15, p0 = p * PB;
  zd x[PB];
#pragma unroll
  for (int r = 0; r < PB; ++r) x[r] = make_double2(r == c ? 1.0 : 0.0, 0.0);
  int o = 0;
#pragma unroll
  for (int k = 0; k < PB; ++k) {
    const zd d = rd[p0 + k], t = x[k];
    x[k] = make_double2(t.x * d.x - t.y * d.y, t.x * d.y + t.y * d.x);
    // the reads' address waits for the step before: all of them at once would
    // not fit the registers
    if (k > 0) asm volatile("" : "+v"(o) : "v"(__double2loint(x[k - 1].x)));
    const zd* col = m.S + (p0 + k) * SLD + p0 + o;
#pragma unroll
    for (int r = k + 1; r < PB; ++r) {
      x[r] = sub_mul(x[r], x[k], col[r]);
    }
  }
  if (lane < 16) {
#pragma unroll
    for (int r = 0; r < PB; ++r) {
      if (r > c) m.S[(p0 + r) * SLD + p0 + c] = x[r];
      if (r == c) m.Xd[p0 + c] = x[r];
    }
  }
}

// Block (I, J), I > J, of inv(L) by one wave: X_IJ = -X_II sum_{K=J}^{I-1} L_IK
// X_KJ.  The matrix cores leave the sum in the layout their next product takes
// as its right operand, so it never leaves the registers.
struct Sum16 {
  d4 re, im;
};
__device__ __forceinline__ Sum16 offdiag_sum(const Block64& m, int I, int J) {
  const int l16 = threadIdx.x & 15, lg = (threadIdx.x >> 4) & 3;
  const zd zero = make_double2(0.0, 0.0);
  d4 tr = {0, 0, 0, 0}, ti = {0, 0, 0, 0}, t2 = {0, 0, 0, 0}, t3 = {0, 0, 0, 0};
  for (int K = J; K < I; ++K) {
    zd a[4], b[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int k = 4 * t + lg;
      a[t] = m.S[(K * PB + k) * SLD + I * PB + l16];
      b[t] = m.S[(K * PB + k) * SLD + J * PB + l16];
      if (K == J) b[t] = pick(k == l16, m.Xd[J * PB + k], pick(k > l16, b[t], zero));
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      tr = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, b[t].x, tr, 0, 0, 0);
      ti = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].x, b[t].y, ti, 0, 0, 0);
      t2 = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[t].y, b[t].y, t2, 0, 0, 0);
      t3 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].y, b[t].x, t3, 0, 0, 0);
    }
  }
  return {tr + t2, ti + t3};
}
__device__ __forceinline__ void offdiag_finish(Block64& m, int I, int J, const Sum16& s) {
  const int l16 = threadIdx.x & 15, lg = (threadIdx.x >> 4) & 3;
  const zd zero = make_double2(0.0, 0.0);
  d4 xr = {0, 0, 0, 0}, xi = {0, 0, 0, 0}, x2 = {0, 0, 0, 0}, x3 = {0, 0, 0, 0};
  zd a[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int k = 4 * t + lg;
    a[t] = m.S[(I * PB + l16) * SLD + I * PB + k];
    a[t] = pick(k == l16, m.Xd[I * PB + k], pick(k < l16, a[t], zero));
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    xr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[t].x, s.re[t], xr, 0, 0, 0);
    xi = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[t].x, s.im[t], xi, 0, 0, 0);
    x2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t].y, s.im[t], x2, 0, 0, 0);
    x3 = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[t].y, s.re[t], x3, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    m.S[(I * PB + lg + 4 * r) * SLD + J * PB + l16] = make_double2(xr[r] + x2[r], xi[r] + x3[r]);
}

// lower triangle of the n x n block at A (padded with the identity) into LDS,
// all loads in flight before the first store; zeros above the diagonal
__device__ __forceinline__ void load_lower(Block64& m, const zd* A, int64_t lda, int n) {
  zd v[NB * NB / 256];
#pragma unroll
  for (int q = 0; q < NB * NB / 256; ++q) {
    const int e = threadIdx.x + 256 * q, r = e & (NB - 1), c = e >> 6;
    v[q] = make_double2((r == c && r >= n) ? 1.0 : 0.0, 0.0);
    if (r < n && c < n && r >= c) v[q] = A[r + (int64_t)c * lda];
  }
#pragma unroll
  for (int q = 0; q < NB * NB / 256; ++q) {
    const int e = threadIdx.x + 256 * q, r = e & (NB - 1), c = e >> 6;
    m.S[c * SLD + r] = v[q];
  }
}
__device__ __forceinline__ void store_inverse(const Block64& m, int n, zd* Dinv, int64_t ldi) {
  for (int e = threadIdx.x; e < NB * NB; e += 256) {
    const int r = e & (NB - 1), c = e >> 6;
    if (r < n && c < n)
      Dinv[r + (int64_t)c * ldi] =
          pick(r > c, m.S[r * SLD + c], pick(r == c, m.Xd[r], make_double2(0.0, 0.0)));
  }
}

// Factor the n x n (n <= 64) diagonal block at M (lower triangle read), write
// L back (upper part of the block zeroed) and inv(L) to Dinv.  A chain of 64
// columns, bound by its latency: wave 0 factors 16-wide panels of all rows in
// registers; wave 1 runs the same chain on the panel's diagonal block and, below
// it, on the rows of the unit matrix, which become the block's inverse
// (conjugate-transposed); waves 2 and 3 meanwhile apply the previous panel
// beyond the next one and build inv(L)'s blocks below the diagonal on the
// matrix cores as their parts become known.  27-30 us, 11.8 of them the four
// panels' vector instructions (76-81 us when one wave went through the LDS for
// every column and the panels below and the inverse followed in turn); 3001 x
// 3001 factorisation 5.8 -> 3.5 ms.
// Entries past n are the identity, so a ragged block needs no special case.
// A non-positive or non-finite pivot is recorded in *info (atomic min of the
// 1-based global index) and replaced by 1 so the kernel always finishes.
__global__ __launch_bounds__(256) void k_potrf_block(zd* M, int64_t ldm, int n, zd* Dinv,
                                                     int64_t ldi, int* info, int goff) {
  extern __shared__ double block_lds[];
  Block64& m = *reinterpret_cast<Block64*>(block_lds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  load_lower(m, M, ldm, n);
  __syncthreads();
  Sum16 s30 = {}, s31 = {};
  for (int p = 0; p < 4; ++p) {
    const int p0 = p * PB;
    zd a[PB];
    const int i = lane - PB;  // wave 1: row of the unit matrix
    if (wave < 2) {
      const int row = wave == 0 ? lane : p0 + (lane & 15);
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        a[c] = pick(wave == 1 && i >= 0, make_double2(c == i ? 1.0 : 0.0, 0.0), m.S[(p0 + c) * SLD + row]);
      }
    }
    __syncthreads();
    if (wave < 2) {
      const int bad = panel16(a, wave == 0 ? p0 : 0, wave == 0 ? m.S + p0 * SLD : m.T, wave == 0 ? SLD : TLD,
                              wave == 0 ? lane : min(lane, TLD - 1));
      if (threadIdx.x == 0 && bad != INT_MAX && p0 + bad < n) atomicMin(info, goff + p0 + bad + 1);
    } else if (p == 1) {  // blocks right of panel 1 by panel 0
      update16(m, wave, 2, 0);
      if (wave == 3) update16(m, 3, 3, 0);
    } else if (p == 2) {
      if (wave == 2) update16(m, 3, 3, 1);
      else offdiag_finish(m, 1, 0, offdiag_sum(m, 1, 0));
    } else if (p == 3) {
      const int J = wave - 2;
      offdiag_finish(m, 2, J, offdiag_sum(m, 2, J));
      if (wave == 2) s30 = offdiag_sum(m, 3, 0);
      else s31 = offdiag_sum(m, 3, 1);
    }
    __syncthreads();
    if (wave == 1 && i >= 0 && i < PB) {  // X(c, i) = conj of entry c of row i
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        const zd x = make_double2(a[c].x, -a[c].y);
        if (c > i) m.S[(p0 + c) * SLD + p0 + i] = x;
        if (c == i) m.Xd[p0 + c] = x;
      }
    }
    if (p < 3 && wave != 1) {  // the next panel's columns: three, two, one blocks
      const int I = p + 1 + (wave == 0 ? 0 : wave - 1);
      if (I < 4) update16(m, I, p + 1, p);
    }
    __syncthreads();
  }
  if (wave == 2) offdiag_finish(m, 3, 0, s30);
  else if (wave == 3) offdiag_finish(m, 3, 1, s31);
  else if (wave == 0) offdiag_finish(m, 3, 2, offdiag_sum(m, 3, 2));
  __syncthreads();
  // L and inv(L), both from the LDS
#pragma unroll 4
  for (int q = 0; q < NB * NB / 256; ++q) {
    const int e = threadIdx.x + 256 * q, r = e & (NB - 1), c = e >> 6;
    const zd zero = make_double2(0.0, 0.0);
    const zd l = pick(r >= c, m.S[c * SLD + r], zero);
    const zd x = pick(r > c, m.S[r * SLD + c], pick(r == c, m.Xd[r], zero));
    if (r < n && c < n) {
      M[r + (int64_t)c * ldm] = l;
      Dinv[r + (int64_t)c * ldi] = x;
    }
  }
}

// inverse of the lower-triangular 64 x 64 diagonal blocks of L (the last one
// ragged) into Dinv, one work-group each: the four 16 x 16 diagonal blocks at
// once, then the blocks below them (a barrier per column before: 85 us at 15
// blocks).
__global__ __launch_bounds__(256, 2) void k_trtri_block(const zd* L, int64_t ldl, int64_t ntot, zd* Dinv,
                                                     int64_t ldi) {
  extern __shared__ double block_lds[];
  Block64& m = *reinterpret_cast<Block64*>(block_lds);
  const int wave = threadIdx.x >> 6;
  const int64_t off = (int64_t)blockIdx.x * NB;
  const int n = (int)((ntot - off) < NB ? (ntot - off) : NB);
  load_lower(m, L + off + off * ldl, ldl, n);
  __syncthreads();
  if (threadIdx.x < NB) {
    const zd d = m.S[threadIdx.x * SLD + threadIdx.x];
    const double q = d.x * d.x + d.y * d.y;
    m.T[threadIdx.x] = make_double2(d.x / q, -d.y / q);
  }
  __syncthreads();
  invert16(m, m.T, wave);
  __syncthreads();
  for (int I = wave + 1; I < 4; ++I) offdiag_finish(m, I, wave, offdiag_sum(m, I, wave));
  __syncthreads();
  store_inverse(m, n, Dinv + off, ldi);
}

__global__ void k_zero_upper(zd* M, int64_t ldm, int64_t n) {
  const int64_t j = blockIdx.y;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < j && i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    M[i + j * ldm] = make_double2(0.0, 0.0);
}

inline int64_t split64(int64_t n) { return ((n / 2 + NB - 1) / NB) * NB; }

}  // namespace

namespace {
gevp_status panel_ctx(gevp_ctx* c, gevp_ctx** out) {
  if (!c->panel) {
    gevp_ctx* w = new gevp_ctx();
    w->device = c->device;
    if (hipStreamCreateWithFlags(&w->stream, hipStreamNonBlocking) != hipSuccess) {
      delete w;
      return GEVP_ERR_HIP;
    }
    w->owns_stream = true;
    w->parent = c;
    c->panel = w;
    ext_assign(c, w, SLOT_PANEL);
  }
  for (hipEvent_t& e : c->pev)
    if (!e) GEVP_HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  *out = c->panel;
  return GEVP_OK;
}

gevp_status potrf_leaf(gevp_ctx* c, int64_t n, zd* M, int64_t ldm, zd* Dinv, int64_t ldi, int* info,
                       int64_t goff) {
  static const bool attr = [] {
    (void)hipFuncSetAttribute((const void*)k_potrf_block, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)sizeof(Block64));
    return true;
  }();
  (void)attr;
  hipLaunchKernelGGL(k_potrf_block, dim3(1), dim3(256), sizeof(Block64), c->stream, M, ldm, (int)n, Dinv,
                     ldi, info, (int)goff);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}
}  // namespace

namespace {
// out (k x m) = in^H, in (m x k): 32 x 32 tiles through LDS, both sides coalesced
__global__ __launch_bounds__(256) void k_copy_ct(const zd* in, int64_t ldin, zd* out, int64_t ldout,
                                                 int64_t m, int64_t k) {
  __shared__ zd t[32][33];
  const int64_t bi = blockIdx.x, bj = blockIdx.y;  // tile of `in`: rows bi, columns bj
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bi * 32 + tx, j = bj * 32 + r;
    if (i < m && j < k) t[r][tx] = in[i + j * ldin];
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {  // out(j, i) = conj(in(i, j)): j = bj*32 + tx, i = bi*32 + r
    const int64_t j = bj * 32 + tx, i = bi * 32 + r;
    if (i < m && j < k) {
      const zd v = t[tx][r];
      out[j + i * ldout] = make_double2(v.x, -v.y);
    }
  }
}

gevp_status copy_ct(gevp_ctx* c, int64_t m, int64_t k, const zd* in, int64_t ldin, zd* out,
                    int64_t ldout) {
  if (m <= 0 || k <= 0) return GEVP_OK;
  hipLaunchKernelGGL(k_copy_ct, dim3((unsigned)((m + 31) / 32), (unsigned)((k + 31) / 32)),
                     dim3(256), 0, c->stream, in, ldin, out, ldout, m, k);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}
}  // namespace

// Right-looking blocked Cholesky in 384-wide panels, grouped into outer panels,
// with one panel of lookahead.  A panel is factored on the panel stream, 64 columns at a time:
// the diagonal block in LDS (k_potrf_block, which also writes its inverse to
// Dinv), the rows below by an in-place product with that inverse,
// L21 = A21 L11^{-H}, and the panel's remaining columns by a rank-64 update.
// The panel's conjugate transpose is then copied into the upper block row
// (space the factor does not use until it is zeroed at the end), so the
// trailing updates multiply both operands as stored.  An inner panel updates the
// rest of its outer panel; the matrix behind that is updated once per outer panel,
// with its whole width as K: wide enough for the products in residue arithmetic,
// whose conversions and reconstruction cost a pass over the trailing matrix each
// time.  The main
// stream applies the panel first to the next panel's columns, after which
// the panel stream may factor that panel, then to the rest of the lower
// triangle, which overlaps the factorisation.
namespace {
constexpr int64_t IPW = 6 * NB;
// Measured with 384, 768 and 1024 columns (factorisation; one-sweep solve, where the
// left solve is carried along): n = 3000 3.38, 3.45, 3.42 and 12.5, 12.1, 12.2 ms, n =
// 5500 8.62, 8.13, 8.20 and 36.0, 33.6, 33.1 ms, n = 8192 17.9, 15.3, 15.0 and 82.6,
// 71.2, 69.2 ms.
inline int64_t outer_panel(int64_t n) { return n >= 6144 ? 1024 : n >= 3072 ? 768 : IPW; }
}  // namespace
gevp_status chol_lower(gevp_ctx* c, int64_t n, zd* M, int64_t ldm, zd* Dinv, int64_t ldi,
                       int* info_dev, hipEvent_t midpoint, zd* R, int64_t ldr, int64_t m) {
  const int64_t PW = outer_panel(n);
  if (n <= 0) {
    if (midpoint) GEVP_HIP_TRY(hipEventRecord(midpoint, c->stream));
    return GEVP_OK;
  }
  const bool rhs = R != nullptr && m > 0;
  if (n <= NB) {
    GEVP_TRY(potrf_leaf(c, n, M, ldm, Dinv, ldi, info_dev, 0));
    if (rhs) GEVP_TRY(trsm_left_lower_n(c, n, m, M, ldm, Dinv, ldi, R, ldr));
    if (midpoint) GEVP_HIP_TRY(hipEventRecord(midpoint, c->stream));
  } else {
    const int64_t half = ((n + NB - 1) / NB / 2) * NB;  // first row of the second half
    bool mid_done = false;
    gevp_ctx* pc = c;  // without inner streams the panels run in order on c's stream
    if (c->inner_streams) {
      GEVP_TRY(panel_ctx(c, &pc));
      pc->profiling = c->profiling & 4;
    }
    const bool two = pc != c;
    hipEvent_t evp = c->pev[0], evn = c->pev[1];
    // the panel stream starts after the work already queued on the main stream
    if (two) {
      GEVP_HIP_TRY(hipEventRecord(evn, c->stream));
      GEVP_HIP_TRY(hipStreamWaitEvent(pc->stream, evn, 0));
    }
    for (int64_t p0 = 0; p0 < n; p0 += PW) {
      const int64_t pw = std::min<int64_t>(PW, n - p0), pend = p0 + pw;
      // factor the panel (columns p0 .. pend-1, all rows below p0) in inner panels
      for (int64_t q0 = p0; q0 < pend; q0 += IPW) {
        const int64_t qend = std::min<int64_t>(q0 + IPW, pend);
        for (int64_t r0 = q0; r0 < qend; r0 += NB) {
          const int64_t kb = std::min<int64_t>(NB, qend - r0), below = n - r0 - kb;
          zd* Mkk = M + r0 + r0 * ldm;
          GEVP_TRY(potrf_leaf(pc, kb, Mkk, ldm, Dinv + r0, ldi, info_dev, r0));
          if (below <= 0) continue;
          zd* L21 = Mkk + kb;
          GEVP_TRY(launch_zgemm(pc, 0, 1, below, kb, kb, 1.0, L21, ldm, Dinv + r0, ldi, 0.0, nullptr,
                                0, 0.0, nullptr, 0, nullptr, L21, ldm));
          const int64_t w = qend - r0 - kb;  // inner panel columns right of this block
          if (w > 0) {
            zd* A2 = M + (r0 + kb) + (r0 + kb) * ldm;
            GEVP_TRY(launch_zgemm(pc, 0, 1, below, w, kb, -1.0, L21, ldm, L21, ldm, 1.0, A2, ldm, 0.0,
                                  nullptr, 0, nullptr, A2, ldm));
          }
        }
        if (qend < pend) {  // the panel's columns right of the inner panel
          const zd* Lq = M + qend + q0 * ldm;
          zd* A2 = M + qend + qend * ldm;
          GEVP_TRY(launch_zgemm(pc, 0, 1, n - qend, pend - qend, qend - q0, -1.0, Lq, ldm, Lq, ldm, 1.0,
                                A2, ldm, 0.0, nullptr, 0, nullptr, A2, ldm));
        }
      }
      const int64_t rest = n - pend;
      const zd* Lp = M + pend + p0 * ldm;  // rest x pw, below the panel's diagonal block
      zd* LpH = M + p0 + pend * ldm;       // pw x rest, the upper block row
      if (rest > 0) GEVP_TRY(copy_ct(pc, rest, pw, Lp, ldm, LpH, ldm));
      if (two) {
        GEVP_HIP_TRY(hipEventRecord(evp, pc->stream));
        GEVP_HIP_TRY(hipStreamWaitEvent(c->stream, evp, 0));
      }
      if (rest > 0) {
        const int64_t pw1 = std::min<int64_t>(PW, rest);
        zd* A2 = M + pend + pend * ldm;
        // next panel's columns: A2(:, :pw1) -= Lp LpH(:, :pw1)
        GEVP_TRY(launch_zgemm(c, 0, 0, rest, pw1, pw, -1.0, Lp, ldm, LpH, ldm, 1.0, A2, ldm, 0.0,
                              nullptr, 0, nullptr, A2, ldm));
        if (two) {
          GEVP_HIP_TRY(hipEventRecord(evn, c->stream));
          GEVP_HIP_TRY(hipStreamWaitEvent(pc->stream, evn, 0));
        }
        const int64_t rest2 = rest - pw1;
        if (rest2 > 0) {  // the rest of the trailing lower triangle
          zd* A3 = A2 + pw1 + pw1 * ldm;
          GEVP_TRY(launch_zgemm(c, 0, 0, rest2, rest2, pw, -1.0, Lp + pw1, ldm, LpH + pw1 * ldm,
                                ldm, 1.0, A3, ldm, 0.0, nullptr, 0, nullptr, A3, ldm, nullptr, 1));
        }
      }
      if (rhs) {
        // block row of the forward substitution: R_p <- L_pp^{-1} R_p (every
        // earlier panel's update of these rows is queued before it on this
        // stream), then the rows below: R_rest -= L_rest,p R_p
        GEVP_TRY(trsm_left_lower_n(c, pw, m, M + p0 + p0 * ldm, ldm, Dinv + p0, ldi, R + p0, ldr));
        if (rest > 0)
          GEVP_TRY(launch_zgemm(c, 0, 0, rest, m, pw, -1.0, Lp, ldm, R + p0, ldr, 1.0, R + pend, ldr,
                                0.0, nullptr, 0, nullptr, R + pend, ldr));
      }
      if (midpoint && !mid_done && pend >= half) {
        GEVP_HIP_TRY(hipEventRecord(midpoint, c->stream));
        mid_done = true;
      }
    }
  }
  if (n > 1) {
    dim3 g((unsigned)((n + 255) / 256 < 64 ? (n + 255) / 256 : 64), (unsigned)n);
    hipLaunchKernelGGL(k_zero_upper, g, dim3(256), 0, c->stream, M, ldm, n);
    GEVP_HIP_TRY(hipGetLastError());
  }
  return GEVP_OK;
}

gevp_status diag_block_inverses(gevp_ctx* c, int64_t n, const zd* L, int64_t ldl, zd* Dinv,
                                int64_t ldi) {
  if (n <= 0) return GEVP_OK;
  static const bool attr = [] {
    (void)hipFuncSetAttribute((const void*)k_trtri_block, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)sizeof(Block64));
    return true;
  }();
  (void)attr;
  hipLaunchKernelGGL(k_trtri_block, dim3((unsigned)((n + NB - 1) / NB)), dim3(256), sizeof(Block64), c->stream, L,
                     ldl, n, Dinv, ldi);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

// R (n x m) <- L^{-1} R
gevp_status trsm_left_lower_n(gevp_ctx* c, int64_t n, int64_t m, const zd* L, int64_t ldl,
                              const zd* Dinv, int64_t ldi, zd* R, int64_t ldr) {
  if (n <= 0 || m <= 0) return GEVP_OK;
  if (n <= NB)
    return launch_zgemm(c, 0, 0, n, m, n, 1.0, Dinv, ldi, R, ldr, 0.0, nullptr, 0, 0.0, nullptr,
                        0, nullptr, R, ldr);
  const int64_t h = split64(n);
  GEVP_TRY(trsm_left_lower_n(c, h, m, L, ldl, Dinv, ldi, R, ldr));
  GEVP_TRY(launch_zgemm(c, 0, 0, n - h, m, h, -1.0, L + h, ldl, R, ldr, 1.0, R + h, ldr, 0.0,
                        nullptr, 0, nullptr, R + h, ldr));
  return trsm_left_lower_n(c, n - h, m, L + h + h * ldl, ldl, Dinv + h, ldi, R + h, ldr);
}

// R (n x m) <- L^{-H} R
gevp_status trsm_left_lower_c(gevp_ctx* c, int64_t n, int64_t m, const zd* L, int64_t ldl,
                              const zd* Dinv, int64_t ldi, zd* R, int64_t ldr, int lhu) {
  if (n <= 0 || m <= 0) return GEVP_OK;
  if (n <= NB)
    return launch_zgemm(c, 1, 0, n, m, n, 1.0, Dinv, ldi, R, ldr, 0.0, nullptr, 0, 0.0, nullptr,
                        0, nullptr, R, ldr);
  const int64_t h = split64(n);
  GEVP_TRY(trsm_left_lower_c(c, n - h, m, L + h + h * ldl, ldl, Dinv + h, ldi, R + h, ldr, lhu));
  // R1 -= L21^H R2   (L21 is (n-h) x h; with lhu its conjugate transpose is the
  // block above the diagonal, read as stored)
  if (lhu)
    GEVP_TRY(launch_zgemm(c, 0, 0, h, m, n - h, -1.0, L + h * ldl, ldl, R + h, ldr, 1.0, R, ldr,
                          0.0, nullptr, 0, nullptr, R, ldr));
  else
    GEVP_TRY(launch_zgemm(c, 1, 0, h, m, n - h, -1.0, L + h, ldl, R + h, ldr, 1.0, R, ldr, 0.0,
                          nullptr, 0, nullptr, R, ldr));
  return trsm_left_lower_c(c, h, m, L, ldl, Dinv, ldi, R, ldr, lhu);
}

// R (m x n) <- R L^{-H}
gevp_status trsm_right_lower_c(gevp_ctx* c, int64_t n, int64_t m, const zd* L, int64_t ldl,
                               const zd* Dinv, int64_t ldi, zd* R, int64_t ldr) {
  if (n <= 0 || m <= 0) return GEVP_OK;
  if (n <= NB)
    return launch_zgemm(c, 0, 1, m, n, n, 1.0, R, ldr, Dinv, ldi, 0.0, nullptr, 0, 0.0, nullptr,
                        0, nullptr, R, ldr);
  const int64_t h = split64(n);
  GEVP_TRY(trsm_right_lower_c(c, h, m, L, ldl, Dinv, ldi, R, ldr));
  // R2 -= R1 L21^H   (R1 = R[:, :h], L21 is (n-h) x h)
  GEVP_TRY(launch_zgemm(c, 0, 1, m, n - h, h, -1.0, R, ldr, L + h, ldl, 1.0, R + h * ldr, ldr,
                        0.0, nullptr, 0, nullptr, R + h * ldr, ldr));
  return trsm_right_lower_c(c, n - h, m, L + h + h * ldl, ldl, Dinv + h, ldi, R + h * ldr, ldr);
}

namespace {
// rows [c0, n) of columns [c0, c0 + nn) of R <- R L^{-H}
gevp_status trsm_rlc_lower_rec(gevp_ctx* c, int64_t n, int64_t c0, int64_t nn, const zd* L,
                               int64_t ldl, const zd* Dinv, int64_t ldi, zd* R, int64_t ldr,
                               int lhu) {
  const zd* Lb = L + c0 + c0 * ldl;
  zd* Rb = R + c0 + c0 * ldr;
  const int64_t rows = n - c0;
  if (nn <= NB)
    return launch_zgemm(c, 0, 1, rows, nn, nn, 1.0, Rb, ldr, Dinv + c0, ldi, 0.0, nullptr, 0, 0.0,
                        nullptr, 0, nullptr, Rb, ldr);
  const int64_t h = split64(nn);
  GEVP_TRY(trsm_rlc_lower_rec(c, n, c0, h, L, ldl, Dinv, ldi, R, ldr, lhu));
  // R[c0+h:, c0+h : c0+nn] -= R[c0+h:, c0 : c0+h] L21^H,  L21 = L[c0+h : c0+nn, c0 : c0+h]
  // (with lhu, L21^H = L[c0 : c0+h, c0+h : c0+nn] as stored)
  if (lhu)
    GEVP_TRY(launch_zgemm(c, 0, 0, n - c0 - h, nn - h, h, -1.0, Rb + h, ldr, Lb + h * ldl, ldl,
                          1.0, Rb + h + h * ldr, ldr, 0.0, nullptr, 0, nullptr, Rb + h + h * ldr,
                          ldr));
  else
    GEVP_TRY(launch_zgemm(c, 0, 1, n - c0 - h, nn - h, h, -1.0, Rb + h, ldr, Lb + h, ldl, 1.0,
                          Rb + h + h * ldr, ldr, 0.0, nullptr, 0, nullptr, Rb + h + h * ldr, ldr));
  return trsm_rlc_lower_rec(c, n, c0 + h, nn - h, L, ldl, Dinv, ldi, R, ldr, lhu);
}
}  // namespace

gevp_status trsm_right_lower_c_lowerpart(gevp_ctx* c, int64_t n, const zd* L, int64_t ldl,
                                         const zd* Dinv, int64_t ldi, zd* R, int64_t ldr, int lhu) {
  if (n <= 0) return GEVP_OK;
  return trsm_rlc_lower_rec(c, n, 0, n, L, ldl, Dinv, ldi, R, ldr, lhu);
}
