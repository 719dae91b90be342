// Complex64 filter GEMM on the FP32 matrix cores (v_mfma_f32_16x16x4f32)
// for the mixed-precision Chebyshev filter:
//
//   D(:, j) = alpha_j C G(:, j) + beta_j G(:, j) + gamma_j P(:, j) + delta_j R(:, j)
//
// with per-column coefficients (device float64 arrays, one entry per active
// column).  C is the FP32 copy of the reduced matrix, G the current iterate,
// P the previous one (D may alias P) and R the FP32 residual block.  With
// beta_j = 0 the G term is not read, so the kernel also serves general
// products D = alpha A G + gamma P (A of m rows, G of k rows).  Same tiling,
// LDS staging, XCD-aware tile order and three-real-product complex form
// (P1 = Ar Gr, P2 = Ai Gi, P3 = (Ar + Ai)(Gr + Gi); Re = P1 - P2,
// Im = P3 - P1 - P2) as the FP64 kernel; the accumulators are FP32.
//
// Split-K: with few output tiles the K range is cut over several work-groups
// (split32), each writes its raw partial tile to the stream's split-K buffer
// and a second kernel sums them in a fixed order and applies the epilogue.
//
// A batch of products of one shape, each operand at a constant stride (the
// contour filter's nodes), is one launch.
#include "common.h"

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float2 zf;

namespace {
constexpr int BM = 64, BN = 64, KT = 16, NTHR = 256;
constexpr int PADA = BM + 1, PADB = BN + 1;

struct CgemmParams {
  int M, N, K;
  const zf* A;
  int64_t lda;
  const zf* B;
  int64_t ldb;
  const zf* P;
  int64_t ldp;
  const zf* R;
  int64_t ldr;
  zf* D;
  int64_t ldd;
  const double* alpha;  // per column
  const double* beta;
  const double* gamma;
  const double* delta;
  int tiles_n, total, remap;
  int tiles, nks;  // output tiles (of the whole batch); K slices per part
  // a batch of products: tiles of one, element strides of A, B and D (P, R as D)
  int tiles1;
  int64_t sA, sB, sD;
  zf* part;        // split-K partial tiles [part][tile][col][row], or null
};

// the parameters of product b of a batch
__device__ __forceinline__ void select(CgemmParams& p, int b) {
  p.A += b * p.sA;
  p.B += b * p.sB;
  p.P += b * p.sD;
  p.R += b * p.sD;
  p.D += b * p.sD;
}

// D entry from its product, FP32 as the accumulators
__device__ __forceinline__ void epilogue(const CgemmParams& p, int row, int col, float pr, float pi) {
  const float al = (float)p.alpha[col], be = (float)p.beta[col];
  const float ga = (float)p.gamma[col], de = (float)p.delta[col];
  float vr = al * pr, vi = al * pi;
  if (be != 0.f) {  // G(row, col) exists only for square products (the filter's)
    const zf g = p.B[row + (int64_t)col * p.ldb];
    vr += be * g.x;
    vi += be * g.y;
  }
  if (ga != 0.f) {
    const zf q = p.P[row + (int64_t)col * p.ldp];
    vr += ga * q.x;
    vi += ga * q.y;
  }
  if (de != 0.f) {
    const zf q = p.R[row + (int64_t)col * p.ldr];
    vr += de * q.x;
    vi += de * q.y;
  }
  p.D[row + (int64_t)col * p.ldd] = make_float2(vr, vi);
}

__global__ __launch_bounds__(NTHR, 2) void k_cgemm32_filter(CgemmParams p) {
  __shared__ zf As[2][KT][PADA];
  __shared__ zf Bs[2][KT][PADB];
  const int tid = threadIdx.x;
  int L = blockIdx.x;
  if (p.remap) {
    const int per = p.total >> 3;
    L = (L & 7) * per + (L >> 3);
  }
  const int kc = L / p.tiles, tile = L - kc * p.tiles;
  const int bt = tile / p.tiles1, tile1 = tile - bt * p.tiles1;
  select(p, bt);
  const int tm = tile1 / p.tiles_n, tn = tile1 - tm * p.tiles_n;
  const int row0 = tm * BM, col0 = tn * BN;
  const int lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int l16 = lane & 15, lg = lane >> 4;

  f4 acc1[2][2], acc2[2][2], acc3[2][2];  // P1, P2, P3 of the three-product form
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      acc1[i][j] = f4{0, 0, 0, 0};
      acc2[i][j] = f4{0, 0, 0, 0};
      acc3[i][j] = f4{0, 0, 0, 0};
    }
  // PRE slices of operands in flight, in registers (n = 8192, 645 columns with the
  // copy to FP32 3.08 -> 2.82 ms against one, n = 4096, 410 columns 0.61 -> 0.54)
  constexpr int PRE = 4;
  zf sa_[PRE][4], sb_[PRE][4];
  auto load = [&](zf (&ra)[4], zf (&rb)[4], int k0) {
    const int m = tid & 63, gm = row0 + m;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int gk = k0 + (tid >> 6) + 4 * i;
      ra[i] = (gm < p.M && gk < p.K) ? p.A[gm + (int64_t)gk * p.lda] : make_float2(0.f, 0.f);
    }
    const int k = tid & 15, gk = k0 + k;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int gn = col0 + (tid >> 4) + 16 * i;
      rb[i] = (gn < p.N && gk < p.K) ? p.B[gk + (int64_t)gn * p.ldb] : make_float2(0.f, 0.f);
    }
  };
  auto store = [&](const zf (&ra)[4], const zf (&rb)[4], int buf) {
    const int m = tid & 63;
#pragma unroll
    for (int i = 0; i < 4; ++i) As[buf][(tid >> 6) + 4 * i][m] = ra[i];
    const int k = tid & 15;
#pragma unroll
    for (int i = 0; i < 4; ++i) Bs[buf][k][(tid >> 4) + 16 * i] = rb[i];
  };
  const int nk = (p.K + KT - 1) / KT;
  const int t0 = kc * p.nks, t1 = min(nk, t0 + p.nks);
#pragma unroll
  for (int q = 0; q < PRE; ++q)
    if (t0 + q < t1) load(sa_[q], sb_[q], (t0 + q) * KT);
  if (t0 < t1) {
    store(sa_[0], sb_[0], 0);
    if (t0 + PRE < t1) load(sa_[0], sb_[0], (t0 + PRE) * KT);
  }
  __syncthreads();
  // slice t lies in LDS buffer t - t0 mod 2, slice t + 1 in register set t + 1 - t0 mod PRE
  auto slice = [&](zf (&na)[4], zf (&nb)[4], int t, int cur) {
    if (t >= t1) return;  // uniform
#pragma unroll
    for (int ks = 0; ks < KT / 4; ++ks) {
      const int kk = ks * 4 + lg;
      zf a[2], b[2];
      float sa[2], sb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = As[cur][kk][wr * 32 + i * 16 + l16];
        sa[i] = a[i].x + a[i].y;
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        b[j] = Bs[cur][kk][wc * 32 + j * 16 + l16];
        sb[j] = b[j].x + b[j].y;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc1[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].x, b[j].x, acc1[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc2[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].y, b[j].y, acc2[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc3[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(sa[i], sb[j], acc3[i][j], 0, 0, 0);
    }
    if (t + 1 < t1) {
      store(na, nb, cur ^ 1);
      if (t + 1 + PRE < t1) load(na, nb, (t + 1 + PRE) * KT);
    }
    __syncthreads();
  };
  for (int t = t0; t < t1; t += PRE) {
    slice(sa_[1], sb_[1], t, 0);
    slice(sa_[2], sb_[2], t + 1, 1);
    slice(sa_[3], sb_[3], t + 2, 0);
    slice(sa_[0], sb_[0], t + 3, 1);
  }
  f4 accR[2][2], accI[2][2];  // the complex result of the three products
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      accR[i][j] = acc1[i][j] - acc2[i][j];
      accI[i][j] = acc3[i][j] - acc1[i][j] - acc2[i][j];
    }
  // D layout of v_mfma_f32_16x16x4f32: lane l, register r -> row 4 (l/16) + r, col l%16
  if (p.part) {
    zf* pt = p.part + ((int64_t)kc * p.tiles + tile) * (BM * BN);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          pt[(wc * 32 + j * 16 + l16) * BM + wr * 32 + i * 16 + 4 * lg + r] =
              make_float2(accR[i][j][r], accI[i][j][r]);
    return;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = col0 + wc * 32 + j * 16 + l16;
      if (col >= p.N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = row0 + wr * 32 + i * 16 + 4 * lg + r;
        if (row < p.M) epilogue(p, row, col, accR[i][j][r], accI[i][j][r]);
      }
    }
}

// sum of the partial tiles in part order, then the epilogue; one thread per
// entry, consecutive threads on consecutive rows
__global__ __launch_bounds__(256) void k_cgemm32_reduce(CgemmParams p, int parts) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  constexpr int PER = BM * BN;
  if (e >= (int64_t)p.tiles * PER) return;
  const int tile = (int)(e / PER), w = (int)(e - (int64_t)tile * PER);
  const int bt = tile / p.tiles1, tile1 = tile - bt * p.tiles1;
  select(p, bt);
  const int tm = tile1 / p.tiles_n, tn = tile1 - tm * p.tiles_n;
  const int row = tm * BM + (w & (BM - 1)), col = tn * BN + w / BM;
  if (row >= p.M || col >= p.N) return;
  const zf* src = p.part + e;
  const int64_t st = (int64_t)p.tiles * PER;
  float sr = 0.f, si = 0.f;
#pragma unroll 8  // eight loads in flight
  for (int q = 0; q < parts; ++q) {
    const zf v = src[q * st];
    sr += v.x;
    si += v.y;
  }
  epilogue(p, row, col, sr, si);
}

// K splits for T tiles of nk slices on `cus` compute units: the slices of a part
// one after the other, at 3/4 of their time each where several work-groups share a
// unit (one's loads run behind another's products), plus the sum of the partial
// tiles (a hundredth of a slice each, 3 for the launch), keeping at least four
// slices a part.  Measured at 1001 x 116 x 1001 (32 tiles, 63 slices): one
// work-group per tile 92 us, in 8 parts 13.5 + 4.4 us, in 16 14.1 + 4.8 us; at 3000 x
// 300 x 3000 (235 tiles) in one part 305 us, in 2 268 us.
inline int split32(int64_t T, int nk, int64_t cus, int64_t max_parts) {
  auto busy = [&](int64_t groups, int nks) {
    const int64_t q = (groups + cus - 1) / cus;
    return (q == 1 ? 1.0 : 0.75 * (double)q) * nks;
  };
  int best = 1;
  double cost = busy(T, nk);
  for (int s = 2; s <= 16; ++s) {
    const int nks = (nk + s - 1) / s;
    if (nks < 4) break;
    const int se = (nk + nks - 1) / nks;
    if (T * se > max_parts) break;
    const double c = busy(T * se, nks) + 3.0 + 0.01 * (double)(T * se);
    if (c < 0.95 * cost) {
      best = se;
      cost = c;
    }
  }
  return best;
}

// FP64 complex -> FP32 complex copy of an n x n matrix (column-major)
__global__ void k_to_c32(int64_t rows, const zd* S, int64_t lds, zf* D, int64_t ldd) {
  const int64_t j = blockIdx.y;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < rows;
       i += (int64_t)gridDim.x * blockDim.x) {
    const zd v = S[i + j * lds];
    D[i + j * ldd] = make_float2((float)v.x, (float)v.y);
  }
}

// R(:, j) = (W(:, pj) - theta_pj Q(:, pj)) * sc,  G1(:, j) = rho0_j * R(:, j),
// G0(:, j) = 0, with pj = perm[j] (degree-sorted order), sc = 1/e
__global__ void k_resid_start32(int64_t rows, const zd* W, const zd* Q, int64_t ld,
                                const double* theta, const int* perm, const double* rho0,
                                double sc, zf* R, zf* G1, zf* G0, int64_t ldl) {
  const int64_t j = blockIdx.y;
  const int pj = perm[j];
  const double th = theta[pj], r0 = rho0[j];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < rows;
       i += (int64_t)gridDim.x * blockDim.x) {
    const zd w = W[i + (int64_t)pj * ld], q = Q[i + (int64_t)pj * ld];
    const double rx = (w.x - th * q.x) * sc, ry = (w.y - th * q.y) * sc;
    R[i + j * ldl] = make_float2((float)rx, (float)ry);
    G1[i + j * ldl] = make_float2((float)(r0 * rx), (float)(r0 * ry));
    G0[i + j * ldl] = make_float2(0.f, 0.f);
  }
}

// Y(:, j) = Q(:, perm[j]) + G(:, j)  (FP64 result)
__global__ void k_add_correction32(int64_t rows, const zd* Q, int64_t ldq, const int* perm,
                                   const zf* G, int64_t ldg, zd* Y, int64_t ldy) {
  const int64_t j = blockIdx.y;
  const int pj = perm[j];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < rows;
       i += (int64_t)gridDim.x * blockDim.x) {
    const zd q = Q[i + (int64_t)pj * ldq];
    const zf g = G[i + j * ldg];
    Y[i + j * ldy] = make_double2(q.x + (double)g.x, q.y + (double)g.y);
  }
}

inline unsigned gx(int64_t rows) {
  int64_t b = (rows + 255) / 256;
  return (unsigned)(b < 64 ? (b < 1 ? 1 : b) : 64);
}
}  // namespace

gevp_status launch_cgemm32_filter(gevp_ctx* c, int64_t m, int64_t n, int64_t k, const void* A,
                                  int64_t lda, const void* G, int64_t ldg, const void* P,
                                  int64_t ldp, const void* R, int64_t ldr, void* D, int64_t ldd,
                                  const double* al, const double* be, const double* ga,
                                  const double* de, int batch, int64_t sA, int64_t sG, int64_t sD) {
  if (m <= 0 || n <= 0 || batch <= 0) return GEVP_OK;
  CgemmParams p;
  p.M = (int)m;
  p.N = (int)n;
  p.K = (int)k;
  p.A = (const zf*)A;
  p.lda = lda;
  p.B = (const zf*)G;
  p.ldb = ldg;
  p.P = (const zf*)P;
  p.ldp = ldp;
  p.R = (const zf*)R;
  p.ldr = ldr;
  p.D = (zf*)D;
  p.ldd = ldd;
  p.alpha = al;
  p.beta = be;
  p.gamma = ga;
  p.delta = de;
  p.tiles_n = (int)((n + BN - 1) / BN);
  p.tiles1 = (int)(((m + BM - 1) / BM) * p.tiles_n);
  p.sA = sA;
  p.sB = sG;
  p.sD = sD;
  const int64_t total = (int64_t)p.tiles1 * batch;
  const int nk = (p.K + KT - 1) / KT;
  constexpr int64_t MAX_PARTS = (int64_t)(SKW_BYTES / (sizeof(zf) * BM * BN));
  int parts = 1;
  if (splitk_possible(c))
    parts = split32(total, nk,
                    std::max<int64_t>(1, (int64_t)gevp_device_cus(c->device) / std::max(1, c->cu_div)), MAX_PARTS);
  p.part = nullptr;
  if (parts > 1) {
    void* buf = nullptr;
    GEVP_TRY(splitk_buffer(c, (size_t)parts * total * BM * BN * sizeof(zf), &buf));
    p.part = (zf*)buf;
    if (!buf) parts = 1;
  }
  p.tiles = (int)total;
  p.nks = nk > 0 ? (nk + parts - 1) / parts : 1;
  const int64_t blocks = total * parts;
  p.total = (int)blocks;
  p.remap = (blocks % 8 == 0 && blocks >= 64) ? 1 : 0;
  hipLaunchKernelGGL(k_cgemm32_filter, dim3((unsigned)blocks), dim3(NTHR), 0, c->stream, p);
  if (parts > 1)
    hipLaunchKernelGGL(k_cgemm32_reduce, dim3((unsigned)(total * BM * BN / 256)), dim3(256), 0, c->stream, p,
                       parts);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

gevp_status launch_to_c32(gevp_ctx* c, int64_t rows, int64_t cols, const zd* S, int64_t lds,
                          void* D, int64_t ldd) {
  if (rows <= 0 || cols <= 0) return GEVP_OK;
  hipLaunchKernelGGL(k_to_c32, dim3(gx(rows), (unsigned)cols), dim3(256), 0, c->stream, rows, S, lds,
                     (zf*)D, ldd);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

gevp_status launch_resid_start32(gevp_ctx* c, int64_t rows, int64_t cols, const zd* W,
                                 const zd* Q, int64_t ld, const double* theta, const int* perm,
                                 const double* rho0, double sc, void* R, void* G1, void* G0,
                                 int64_t ldl) {
  if (rows <= 0 || cols <= 0) return GEVP_OK;
  hipLaunchKernelGGL(k_resid_start32, dim3(gx(rows), (unsigned)cols), dim3(256), 0, c->stream, rows,
                     W, Q, ld, theta, perm, rho0, sc, (zf*)R, (zf*)G1, (zf*)G0, ldl);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

gevp_status launch_add_correction32(gevp_ctx* c, int64_t rows, int64_t cols, const zd* Q,
                                    int64_t ldq, const int* perm, const void* G, int64_t ldg,
                                    zd* Y, int64_t ldy) {
  if (rows <= 0 || cols <= 0) return GEVP_OK;
  hipLaunchKernelGGL(k_add_correction32, dim3(gx(rows), (unsigned)cols), dim3(256), 0, c->stream,
                     rows, Q, ldq, perm, (const zf*)G, ldg, Y, ldy);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}
