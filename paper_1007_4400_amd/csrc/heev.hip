// Small dense Hermitian eigensolver for the Rayleigh-Ritz step (n up to a few
// thousand), all on the GPU in FP64:
//
//  1. Householder tridiagonalisation H = U T U^H, whole in one launch that
//     keeps H in registers, or one fused kernel per reflector.  Step s
//     finishes the rank-2 update of reflector s-1 on the columns it owns, forms reflector s from column s (which every
//     work-group reconstructs redundantly from the old column and the
//     previous reflector, so no extra grid-wide barrier is needed), and
//     accumulates p = tau H v for reflector s on its columns.  Hermitian
//     symmetry turns each row dot product into a contiguous column dot.
//  2. Eigenvalues of the real tridiagonal T by multisection on Sturm counts,
//     one wave per eigenvalue (64 points per round).
//  3. Eigenvectors of T by inverse iteration (tridiagonal LU with partial
//     pivoting), one thread per eigenvalue, recurrences in registers; members
//     of numerically degenerate clusters are then made orthonormal by
//     modified Gram-Schmidt.
//  4. Z = U Z_T with U = I - V T V^H for all reflectors at once: T^{-1} is
//     diag(1/tau) plus the strict upper triangle of V^H V, so Z <- Z - V (T
//     (V^H Z)) is a Gram product, a triangular solve and two products on the
//     FP64 matrix cores.
#include <cfloat>

#include "exchange.h"

namespace {
constexpr int HT = 256;  // threads per work-group
// Columns whose squares sum to less than 2^-900 (their entries' own may have lost
// digits or be zero) are taken times 2^600 to form their reflector: a rank-deficient
// matrix whose rounding errors are alike in every column, the matrix of ones say,
// shrinks by 2^-50 from step to step, and a reflector from lost digits is not unitary.
constexpr double SMALL_COL = 0x1p-900, COL_UP = 0x1p600;
__device__ __forceinline__ bool small_column(zd a, double sig) {
  return __builtin_expect(a.x * a.x + a.y * a.y + sig < SMALL_COL, 0);
}

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ double bsum(double v, double* sh) {
  v = wsum(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) sh[w] = v;
  __syncthreads();
  const double s = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return s;
}
__device__ __forceinline__ zd cmul(zd a, zd b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ zd cconj(zd a) { return make_double2(a.x, -a.y); }

struct TrdArgs {
  int n;
  zd* H;
  int64_t ldh;
  zd* V;  // reflectors, column s holds v_s (v_s[s+1] = 1)
  int64_t ldv;
  zd* tau;
  double* d;
  double* e;
  zd* pb;       // 2 x n : p of the previous / current reflector
  zd* pp;       // 2 x G : per-work-group partial sums v^H p
  int G;
};

// Reflector s (0 <= s <= n-2); s == n-1 finishes the last diagonal entry.
// One pass over global memory per step: every thread first loads its share
// of column s, v_{s-1} and p_{s-1} (rows s .. n-1, at most QMAX per thread)
// together with one partial sum, everything else is formed in registers and
// LDS: w_{s-1} = p - K v (K from the partials), the updated column s, the
// reflector, and the staged vectors v_s, w_{s-1}, v_{s-1} that the column
// updates read.
// LDS: sm = [v_s | w_{s-1} | v_{s-1}], each n complex; sh: 8 doubles.
constexpr int QMAX = 8;  // rows per thread: n <= QMAX * HT

__device__ __forceinline__ zd bsum2(zd v, double* sh) {
  v.x = wsum(v.x);
  v.y = wsum(v.y);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) {
    sh[2 * w] = v.x;
    sh[2 * w + 1] = v.y;
  }
  __syncthreads();
  const zd r = make_double2(sh[0] + sh[2] + sh[4] + sh[6], sh[1] + sh[3] + sh[5] + sh[7]);
  __syncthreads();
  return r;
}

__device__ void hetrd_body(const TrdArgs& a, int s, zd* sm, double* sh, zd* bc) {
  const int n = a.n, tid = threadIdx.x, wg = blockIdx.x;
  const int prev = s - 1;
  zd* vs = sm;            // v_s
  zd* sw = sm + n;        // w_{s-1}
  zd* sv = sm + 2 * n;    // v_{s-1}
  const zd* vp = (prev >= 0) ? a.V + (int64_t)prev * a.ldv : nullptr;
  const zd* pprev = (prev >= 0) ? a.pb + (int64_t)(prev & 1) * n : nullptr;
  const zd* cs = a.H + (int64_t)s * a.ldh;
  // ---- the one round of global loads
  zd hc[QMAX], vv[QMAX], pv[QMAX];
  zd ppart = make_double2(0.0, 0.0);
#pragma unroll
  for (int q = 0; q < QMAX; ++q) {
    const int i = s + tid + q * HT;
    hc[q] = (i < n) ? cs[i] : make_double2(0.0, 0.0);
    vv[q] = (prev >= 0 && i < n) ? vp[i] : make_double2(0.0, 0.0);
    pv[q] = (prev >= 0 && i < n) ? pprev[i] : make_double2(0.0, 0.0);
  }
  if (prev >= 0 && tid < a.G) ppart = a.pp[(int64_t)(prev & 1) * a.G + tid];
  const zd taup = (prev >= 0) ? a.tau[prev] : make_double2(0.0, 0.0);
  // ---- K = 1/2 conj(tau) sum(partials); w = p - K v
  zd K = make_double2(0.0, 0.0);
  if (prev >= 0) {
    const zd ps = bsum2(ppart, sh);
    const zd k2 = cmul(cconj(taup), ps);
    K = make_double2(0.5 * k2.x, 0.5 * k2.y);
  }
  zd ww[QMAX];
#pragma unroll
  for (int q = 0; q < QMAX; ++q) {
    const zd kv = cmul(K, vv[q]);
    ww[q] = make_double2(pv[q].x - kv.x, pv[q].y - kv.y);
  }
  // v_s and w_s of the previous reflector (row s, owned by thread 0, q = 0)
  if (tid == 0) {
    bc[0] = vv[0];
    bc[1] = ww[0];
  }
  __syncthreads();
  const zd vps = bc[0], wps = bc[1];
  // updated column s: H(i,s) - v_i conj(w_s) - w_i conj(v_s)
  double sig = 0.0;
#pragma unroll
  for (int q = 0; q < QMAX; ++q) {
    const int i = s + tid + q * HT;
    const zd t1 = cmul(vv[q], cconj(wps)), t2 = cmul(ww[q], cconj(vps));
    hc[q].x -= t1.x + t2.x;
    hc[q].y -= t1.y + t2.y;
    if (i >= s + 2 && i < n) sig += hc[q].x * hc[q].x + hc[q].y * hc[q].y;
    if (i == s + 1) bc[2] = hc[q];
    if (i == s) bc[3] = hc[q];
  }
  sig = bsum(sig, sh);  // its barriers also publish bc[2], bc[3]
  if (s == n - 1) {  // finish: last diagonal entry only
    if (wg == 0 && tid == 0) a.d[s] = bc[3].x;
    return;
  }
  zd alpha = bc[2];
  double up = 1.0;
  if (small_column(alpha, sig)) {
    up = COL_UP;
    alpha = make_double2(alpha.x * up, alpha.y * up);
    sig = 0.0;
#pragma unroll
    for (int q = 0; q < QMAX; ++q) {
      const int i = s + tid + q * HT;
      hc[q] = make_double2(hc[q].x * up, hc[q].y * up);
      if (i >= s + 2 && i < n) sig += hc[q].x * hc[q].x + hc[q].y * hc[q].y;
    }
    sig = bsum(sig, sh);
  }
  zd tau = make_double2(0.0, 0.0), scal = make_double2(0.0, 0.0);
  double beta;
  if (sig == 0.0 && alpha.y == 0.0) {
    beta = alpha.x;
  } else {
    const double nrm = sqrt(alpha.x * alpha.x + alpha.y * alpha.y + sig);
    beta = (alpha.x >= 0.0) ? -nrm : nrm;
    tau = make_double2((beta - alpha.x) / beta, -alpha.y / beta);
    const zd den = make_double2(alpha.x - beta, alpha.y);  // scal = 1 / den
    const double dd = den.x * den.x + den.y * den.y;
    scal = make_double2(den.x / dd, -den.y / dd);
  }
  // stage v_s, w_{s-1}, v_{s-1} in LDS
#pragma unroll
  for (int q = 0; q < QMAX; ++q) {
    const int i = s + tid + q * HT;
    if (i < n) {
      vs[i] = (i == s + 1) ? make_double2(1.0, 0.0) : (i > s + 1 ? cmul(hc[q], scal) : make_double2(0.0, 0.0));
      sw[i] = ww[q];
      sv[i] = vv[q];
    }
  }
  __syncthreads();
  if (wg == 0) {
    zd* vcol = a.V + (int64_t)s * a.ldv;
    for (int i = tid; i < n; i += HT) vcol[i] = (i > s) ? vs[i] : make_double2(0.0, 0.0);
    if (tid == 0) {
      a.tau[s] = tau;
      a.e[s] = beta / up;
      a.d[s] = bc[3].x;
    }
  }
  // own columns j >= s+1, j % G == wg: finish the previous update on rows
  // >= s+1 and accumulate p_s[j] = tau sum_i conj(H(i,j)) v_i (Hermitian
  // symmetry turns the row product into a contiguous column product)
  const int lane = tid & 63, wave = tid >> 6;
  zd part = make_double2(0.0, 0.0);
  zd* pcur = a.pb + (int64_t)(s & 1) * n;
  const int j0 = s + 1 + ((wg - (s + 1)) % a.G + a.G) % a.G;
  for (int j = j0 + wave * a.G; j < n; j += 4 * a.G) {
    zd* col = a.H + (int64_t)j * a.ldh;
    const zd vj = sv[j], wj = sw[j];
    double ar = 0.0, ai = 0.0;
    for (int i = s + 1 + lane; i < n; i += 64) {
      zd h = col[i];
      if (prev >= 0) {
        const zd v = sv[i], w = sw[i];
        const zd t1 = cmul(v, cconj(wj)), t2 = cmul(w, cconj(vj));
        h.x -= t1.x + t2.x;
        h.y -= t1.y + t2.y;
        col[i] = h;
      }
      const zd v = vs[i];  // conj(h) * v
      ar += h.x * v.x + h.y * v.y;
      ai += h.x * v.y - h.y * v.x;
    }
    ar = wsum(ar);
    ai = wsum(ai);
    const zd pj = cmul(tau, make_double2(ar, ai));
    if (lane == 0) {
      pcur[j] = pj;
      const zd t = cmul(cconj(vs[j]), pj);
      part.x += t.x;
      part.y += t.y;
    }
  }
  // work-group partial of v_s^H p_s
  const zd pt = bsum2(lane == 0 ? part : make_double2(0.0, 0.0), sh);
  if (tid == 0) a.pp[(int64_t)(s & 1) * a.G + wg] = pt;
}

__global__ __launch_bounds__(HT) void k_hetrd_step(TrdArgs a, int s) {
  extern __shared__ double sm[];
  __shared__ double sh[8];
  __shared__ zd bc[4];
  hetrd_body(a, s, reinterpret_cast<zd*>(sm), sh, bc);
}

// ---- the whole tridiagonalisation in one launch
//
// A wave owns whole columns of H and keeps them in registers (lane l holds rows
// l, l + 64, ...), so H is read once and never written.  What a step exchanges
// is small: every column's owner publishes p_s(j), and the owner of column s +
// 1 that column as it stands, which is all a wave needs to form the next
// reflector by itself, exactly as every other wave forms it (the same operations
// in the same order).  One exchange per reflector, no other communication.

struct Reflector {
  zd tau, scal, K, wps;  // K of the previous reflector and w_{s-1}(s)
  double d, beta;
};
// Reflector s from column s as published (updated through reflector s - 2), p of
// reflector s - 1 (rows >= s) and v_{s-1}, one row a lane: c becomes v_s, w
// becomes w_{s-1}.
__device__ __forceinline__ Reflector reflect(int s, int n, const zd* C, const zd* P, const zd* V, zd taup,
                                             zd& c, zd& w) {
  const int lane = threadIdx.x & 63;
  const zd zero = make_double2(0.0, 0.0);
  Reflector f;
  f.K = f.wps = c = w = zero;
  if (lane >= s && lane < n) c = C[lane];
  zd cs = C[s], ca = zero;  // rows s and s + 1
  if (s + 1 < n) ca = C[s + 1];
  if (s > 0) {
    zd v = zero;
    if (lane >= s && lane < n) {
      v = V[lane];
      w = P[lane];
    }
    const double kr = v.x * w.x + v.y * w.y, ki = v.x * w.y - v.y * w.x;  // conj(v) p
    const zd k2 = cmul(cconj(taup), make_double2(wave_total(kr), wave_total(ki)));
    f.K = make_double2(0.5 * k2.x, 0.5 * k2.y);
    // v_{s-1}(s) = 1
    f.wps = make_double2(P[s].x - f.K.x, P[s].y - f.K.y);
    const zd kv = cmul(f.K, v), t = cmul(v, cconj(f.wps));
    w = make_double2(w.x - kv.x, w.y - kv.y);
    c = make_double2(c.x - (t.x + w.x), c.y - (t.y + w.y));
    cs.x -= 2.0 * f.wps.x;
    if (s + 1 < n) {
      const zd va = V[s + 1], ka = cmul(f.K, va), ta = cmul(va, cconj(f.wps));
      ca.x -= ta.x + (P[s + 1].x - ka.x);
      ca.y -= ta.y + (P[s + 1].y - ka.y);
    }
  }
  f.d = cs.x;
  double sig = wave_total(lane >= s + 2 ? c.x * c.x + c.y * c.y : 0.0), up = 1.0;
  if (small_column(ca, sig)) {
    up = COL_UP;
    ca = make_double2(ca.x * up, ca.y * up);
    c = make_double2(c.x * up, c.y * up);
    sig = wave_total(lane >= s + 2 ? c.x * c.x + c.y * c.y : 0.0);
  }
  f.tau = f.scal = zero;
  if (sig == 0.0 && ca.y == 0.0) {
    f.beta = ca.x;
  } else {
    const double nrm = sqrt(ca.x * ca.x + ca.y * ca.y + sig);
    f.beta = (ca.x >= 0.0) ? -nrm : nrm;
    f.tau = make_double2((f.beta - ca.x) / f.beta, -ca.y / f.beta);
    const zd den = make_double2(ca.x - f.beta, ca.y);  // scal = 1 / den
    const double dd = den.x * den.x + den.y * den.y;
    f.scal = make_double2(den.x / dd, -den.y / dd);
  }
  f.beta /= up;
  const zd x = cmul(c, f.scal);
  c = make_double2(lane == s + 1 ? 1.0 : lane > s + 1 ? x.x : 0.0, lane > s + 1 ? x.y : 0.0);
  return f;
}

// p_s(j) of one column h (row of the lane), after its update by reflector s - 1
__device__ __forceinline__ zd column_step(int s, int j, const Reflector& f, const zd* P, const zd* V, zd vs,
                                          zd w, zd& h) {
  const int lane = threadIdx.x & 63;
  if (s > 0) {
    const zd vj = V[j], kv = cmul(f.K, vj), wj = make_double2(P[j].x - kv.x, P[j].y - kv.y);
    const zd t1 = cmul(V[lane], cconj(wj)), t2 = cmul(w, cconj(vj));
    if (lane >= s) h = make_double2(h.x - (t1.x + t2.x), h.y - (t1.y + t2.y));
  }
  // conj(h) v_s
  return cmul(f.tau, make_double2(wave_total(h.x * vs.x + h.y * vs.y), wave_total(h.x * vs.y - h.y * vs.x)));
}

// n <= 60: one work-group of 16 waves, up to four columns a wave, the exchange
// through the LDS and one barrier per reflector.
__global__ __launch_bounds__(1024) void k_hetrd_one(TrdArgs a) {
  __shared__ zd P[2][64], C[2][64], V[2][64];
  const int n = a.n, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const zd zero = make_double2(0.0, 0.0);
  zd h[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int j = wave + 16 * m;
    h[m] = zero;
    if (lane < n && j < n) h[m] = a.H[lane + (int64_t)j * a.ldh];
  }
  if (threadIdx.x < 64) {
    V[0][threadIdx.x] = V[1][threadIdx.x] = zero;
    if ((int)threadIdx.x < n) C[0][threadIdx.x] = a.H[threadIdx.x];
  }
  __syncthreads();
  zd taup = zero;
  for (int s = 0; s < n; ++s) {
    const int b = s & 1;
    zd c, w;
    const Reflector f = reflect(s, n, C[b], P[b], V[b], taup, c, w);
    if (wave == 0) {
      if (lane == 0) {
        a.d[s] = f.d;
        if (s < n - 1) {
          a.tau[s] = f.tau;
          a.e[s] = f.beta;
        }
      }
      V[b ^ 1][lane] = c;
      if (lane < n && s < n - 1) a.V[lane + (int64_t)s * a.ldv] = c;
    }
    if (s == n - 1) break;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int j = wave + 16 * m;
      if (j <= s || j >= n) continue;
      const zd p = column_step(s, j, f, P[b], V[b], c, w, h[m]);
      if (lane == 0) P[b ^ 1][j] = p;
      if (j == s + 1) C[b ^ 1][lane] = h[m];
    }
    taup = f.tau;
    __syncthreads();
  }
}

// 60 < n <= 2048: eight columns a work-group, a row of each in every thread (R
// rows when there are more than threads), one launch.  The exchange
// goes through device memory (exchange.h).  A work-group publishes its eight p as
// one line of 128 bytes.  When a wait gives up the host takes the launch per
// reflector.
// Latency bounds it: of the 4.4 us a step takes at n = 948 about half is the way
// of p through memory, the rest three sums over the work-group and eight columns
// of FP64 arithmetic.  Measured whole, n = 256, 512, 948: 0.71, 1.82, 4.18 ms,
// against 1.9, 4.1 and 8.8 ms for the launches per reflector.  One column a wave
// and the reflector formed by every wave took 10 us a step at n = 948 (the reads
// of p by 237 work-groups queue up); 256 threads instead of 512 4.9 us.
constexpr int TRDM_MAX = 2048;
struct TrdExchange {
  // step t: p_t, then column t + 1, each as n real and n imaginary parts (a wave's
  // read is one contiguous piece) of ld entries
  unsigned long long* x;
  int64_t ld;
  int* err;
  int spin;               // polls before a wait gives up
};
constexpr int TRD_COLS = 8;
template <int T, int R>
__global__ __launch_bounds__(T) void k_hetrd_all(TrdArgs a, TrdExchange e) {
  constexpr int K = TRD_COLS, W = T / 64;
  __shared__ zd P[T * R + 1], V[2][T * R + 1];
  __shared__ double sums[2 * W], sigs[W], dots[W][2 * K];
  __shared__ zd head[2];  // rows s and s + 1 of column s
  __shared__ int fail;
  const int n = a.n, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j0 = blockIdx.x * K, last = min(n, j0 + K) - 1;  // done after step `last`
  const zd zero = make_double2(0.0, 0.0);
  zd h[K][R], v[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int i = tid + T * q;
    v[q] = V[0][i] = V[1][i] = P[i] = zero;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      h[k][q] = zero;
      if (i < n && j0 + k < n) h[k][q] = a.H[i + (int64_t)(j0 + k) * a.ldh];
    }
  }
  if (tid == 0) {
    fail = 0;
    P[T * R] = V[0][T * R] = V[1][T * R] = head[1] = zero;
  }
  __syncthreads();
  zd taup = zero;
  for (int s = 0; s <= last; ++s) {
    // p of reflector s - 1 and column s, rows >= s
    zd p[R], c[R];
#pragma unroll
    for (int q = 0; q < R; ++q) p[q] = c[q] = zero;
    if (s == 0) {
#pragma unroll
      for (int q = 0; q < R; ++q)
        if (tid + T * q < n) c[q] = a.H[tid + T * q];
    } else {
      const unsigned long long* x = e.x + (s - 1) * 4 * e.ld;
      unsigned long long g[R][4];
#pragma unroll
      for (int q = 0; q < R; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) g[q][u] = HOLE;
      bool miss = true;
      for (int spin = 0; miss && spin < e.spin; ++spin) {
        miss = false;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int i = tid + T * q;
          if (i >= s && i < n && (g[q][0] == HOLE || g[q][1] == HOLE)) {
            g[q][0] = peek(x + i);
            g[q][1] = peek(x + e.ld + i);
          }
          if (i >= s && i < n && (g[q][2] == HOLE || g[q][3] == HOLE)) {
            g[q][2] = peek(x + 2 * e.ld + i);
            g[q][3] = peek(x + 3 * e.ld + i);
          }
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const int i = tid + T * q;
          if (i >= s && i < n)
            miss |= g[q][0] == HOLE || g[q][1] == HOLE || g[q][2] == HOLE || g[q][3] == HOLE;
        }
      }
      if (miss) fail = 1;
#pragma unroll
      for (int q = 0; q < R; ++q)
        if (tid + T * q >= s && tid + T * q < n) {
          p[q] = make_double2(__longlong_as_double(g[q][0]), __longlong_as_double(g[q][1]));
          c[q] = make_double2(__longlong_as_double(g[q][2]), __longlong_as_double(g[q][3]));
        }
    }
    // K = conj(tau) / 2 * v^H p
    double kr = 0.0, ki = 0.0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int i = tid + T * q;
      P[i] = p[q];
      if (i == s) head[0] = c[q];
      if (i == s + 1) head[1] = c[q];
      kr += v[q].x * p[q].x + v[q].y * p[q].y;
      ki += v[q].x * p[q].y - v[q].y * p[q].x;
    }
    kr = wave_total(kr);
    ki = wave_total(ki);
    if (lane == 0) {
      sums[2 * wave] = kr;
      sums[2 * wave + 1] = ki;
    }
    __syncthreads();
    if (fail) {
      if (tid == 0) __hip_atomic_store(e.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    const zd* Vp = V[s & 1];
    kr = ki = 0.0;
#pragma unroll
    for (int u = 0; u < W; ++u) {
      kr += sums[2 * u];
      ki += sums[2 * u + 1];
    }
    const zd k2 = cmul(cconj(taup), make_double2(0.5 * kr, 0.5 * ki));
    // w = p - K v; column s: c - (v conj(w(s)) + w conj(v(s))), v(s) = 1
    const zd ps = P[s], wps = make_double2(ps.x - k2.x, ps.y - k2.y);
    zd cs = head[0], ca = head[1];
    if (s > 0) {
      cs.x -= 2.0 * wps.x;
      const zd va = Vp[s + 1], pa = P[s + 1], kv = cmul(k2, va), t = cmul(va, cconj(wps));
      ca.x -= t.x + (pa.x - kv.x);
      ca.y -= t.y + (pa.y - kv.y);
    }
    double sig = 0.0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const zd kv = cmul(k2, v[q]), t = cmul(v[q], cconj(wps));
      p[q] = make_double2(p[q].x - kv.x, p[q].y - kv.y);  // w from here on
      c[q] = make_double2(c[q].x - (t.x + p[q].x), c[q].y - (t.y + p[q].y));
      if (tid + T * q >= s + 2) sig += c[q].x * c[q].x + c[q].y * c[q].y;
    }
    sig = wave_total(sig);
    if (lane == 0) sigs[wave] = sig;
    __syncthreads();
    sig = 0.0;
#pragma unroll
    for (int u = 0; u < W; ++u) sig += sigs[u];
    // (alike in every thread of every work-group)
    const int small = __builtin_amdgcn_readfirstlane(small_column(ca, sig) ? 1 : 0);
    if (__builtin_expect(small, 0)) {
      ca = make_double2(ca.x * COL_UP, ca.y * COL_UP);
      sig = 0.0;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        c[q] = make_double2(c[q].x * COL_UP, c[q].y * COL_UP);
        if (tid + T * q >= s + 2) sig += c[q].x * c[q].x + c[q].y * c[q].y;
      }
      sig = wave_total(sig);
      __syncthreads();
      if (lane == 0) sigs[wave] = sig;
      __syncthreads();
      sig = 0.0;
#pragma unroll
      for (int u = 0; u < W; ++u) sig += sigs[u];
    }
    zd tau = zero, scal = zero;
    double beta = ca.x;
    if (sig != 0.0 || ca.y != 0.0) {
      const double nrm = sqrt(ca.x * ca.x + ca.y * ca.y + sig);
      beta = (ca.x >= 0.0) ? -nrm : nrm;
      tau = make_double2((beta - ca.x) / beta, -ca.y / beta);
      const zd den = make_double2(ca.x - beta, ca.y);  // scal = 1 / den
      const double dd = den.x * den.x + den.y * den.y;
      scal = make_double2(den.x / dd, -den.y / dd);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {  // v_s
      const int i = tid + T * q;
      const zd t = cmul(c[q], scal);
      c[q] = make_double2(i == s + 1 ? 1.0 : i > s + 1 ? t.x : 0.0, i > s + 1 ? t.y : 0.0);
      V[(s & 1) ^ 1][i] = c[q];
    }
    if (s >= j0) {  // this work-group's column: the reflector goes out
      if (tid == 0) {
        a.d[s] = cs.x;
        if (s < n - 1) {
          a.tau[s] = tau;
          a.e[s] = small ? beta / COL_UP : beta;
        }
      }
      if (s < n - 1) {
#pragma unroll
        for (int q = 0; q < R; ++q)
          if (tid + T * q < n) a.V[tid + T * q + (int64_t)s * a.ldv] = c[q];
      }
    }
    if (s == last) break;
    // the columns' update by reflector s - 1, then conj(h) v_s
    // (a wave's 64 rows that lie above row s are zero in v, w and v_s)
    double dot[2 * K];
    constexpr int KB = R > 2 ? K / 2 : K;  // columns at a time, by the registers left
#pragma unroll
    for (int kb = 0; kb < K; kb += KB) {
      zd vj[KB], wj[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int j = min(j0 + kb + k, n - 1);
        vj[k] = Vp[j];
        const zd kv = cmul(k2, vj[k]);
        wj[k] = make_double2(P[j].x - kv.x, P[j].y - kv.y);
        dot[2 * (kb + k)] = dot[2 * (kb + k) + 1] = 0.0;
      }
#pragma unroll
      for (int q = 0; q < R; ++q) {
        if (64 * wave + T * q + 63 < s) continue;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          double x = h[kb + k][q].x, y = h[kb + k][q].y;
          x = fma(-v[q].x, wj[k].x, x);  // - v conj(w(j)) - w conj(v(j))
          y = fma(-v[q].y, wj[k].x, y);
          x = fma(-v[q].y, wj[k].y, x);
          y = fma(v[q].x, wj[k].y, y);
          x = fma(-p[q].x, vj[k].x, x);
          y = fma(-p[q].y, vj[k].x, y);
          x = fma(-p[q].y, vj[k].y, x);
          y = fma(p[q].x, vj[k].y, y);
          h[kb + k][q] = make_double2(x, y);
          dot[2 * (kb + k)] += x * c[q].x + y * c[q].y;
          dot[2 * (kb + k) + 1] += x * c[q].y - y * c[q].x;
        }
      }
    }
    unsigned long long* x = e.x + s * 4 * e.ld;
    if (s + 1 >= j0) {  // column s + 1 (s < last: it is one of these)
      const int kc = s + 1 - j0;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int i = tid + T * q;
        zd t = h[0][q];
#pragma unroll
        for (int k = 1; k < K; ++k) {
          t.x = kc == k ? h[k][q].x : t.x;
          t.y = kc == k ? h[k][q].y : t.y;
        }
        if (i > s && i < n) {
          publish(x + 2 * e.ld + i, t.x);
          publish(x + 3 * e.ld + i, t.y);
        }
      }
    }
    const double total = wave_totals16(dot);
    if ((lane & 15) < 4) dots[wave][4 * (lane >> 4) + (lane & 3)] = total;
    __syncthreads();
    if (tid < 2 * K) {
      const int k = tid >> 1, j = j0 + k;
      double dr = 0.0, di = 0.0;
#pragma unroll
      for (int u = 0; u < W; ++u) {
        dr += dots[u][2 * k];
        di += dots[u][2 * k + 1];
      }
      const zd pk = cmul(tau, make_double2(dr, di));
      if (j > s && j < n) publish(x + (tid & 1 ? e.ld : 0) + j, tid & 1 ? pk.y : pk.x);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = c[q];
    taup = tau;
  }
}

// 1 / x for a normal x: the vector unit's estimate (24 bits or more) times 1 + e +
// e^2, e = 1 - x r being what it lacks.  As good as the full divide: off by 0.5000
// units in the last place at most for estimates of 24 to 28 bits (exact rationals,
// 9000 random x), the one rounding of the last operation.  The recurrences below are
// one chain of divisions; the full divide's scaling and fix-up double the chain.
__device__ __forceinline__ double recip(double x) {
  const double r = __builtin_amdgcn_rcp(x), e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Sturm count: number of eigenvalues of T smaller than x.  |q| >= pivmin keeps
// both 1 / q and e^2 / q finite.  948 eigenvalues: 820 us with the full divide, now
// 460 us.
__device__ int sturm(const double* d, const double* e2, int n, double x, double pivmin) {
  int cnt = 0;
  double q = d[0] - x;
  if (fabs(q) < pivmin) q = -pivmin;
  cnt += q < 0.0;
  for (int i = 1; i < n; ++i) {
    q = fma(-e2[i - 1], recip(q), d[i] - x);
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0.0;
  }
  return cnt;
}

// largest v of the work-group; sh holds one entry per wave
__device__ double bmax(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

// One wave per row k, whose block of T between zero couplings has rows [b0, b1):
// the block's eigenvalue k - b0.  Every round the 64 lanes evaluate Sturm counts
// at 64 interior points of [lo, hi] and the bracket shrinks to the
// sub-interval where the count passes it (65x per round).
__global__ __launch_bounds__(HT) void k_tri_bisect(const double* d, const double* e, int n,
                                                   double* theta, int2* block) {
  extern __shared__ double sm[];
  double* sd = sm;
  double* se2 = sm + n;
  __shared__ double red[4];
  for (int i = threadIdx.x; i < n; i += HT) {
    sd[i] = d[i];
    se2[i] = (i < n - 1) ? e[i] * e[i] : 0.0;
  }
  __syncthreads();
  double gl = DBL_MAX, gu = -DBL_MAX, emax = 0.0;
  for (int i = threadIdx.x; i < n; i += HT) {
    const double r = (i > 0 ? sqrt(se2[i - 1]) : 0.0) + (i < n - 1 ? sqrt(se2[i]) : 0.0);
    gl = fmin(gl, sd[i] - r);
    gu = fmax(gu, sd[i] + r);
    emax = fmax(emax, se2[i]);
  }
  gl = -bmax(-gl, red);
  gu = bmax(gu, red);
  emax = bmax(emax, red);
  const double tnorm = fmax(fabs(gl), fabs(gu));
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x * (HT / 64) + (threadIdx.x >> 6);
  if (k >= n) return;
  double lo = gl - 2.0 * DBL_EPSILON * tnorm * n - 1e-300;
  double hi = gu + 2.0 * DBL_EPSILON * tnorm * n + 1e-300;
  const double pivmin = DBL_MIN * fmax(1.0, emax);
  int b0 = 0, b1 = n;
  for (int i = k - lane;; i -= 64) {  // 64 rows at a time, the nearest in lane 0
    const unsigned long long m = __ballot(i <= 0 || se2[i - 1] == 0.0);
    if (m != 0ull) {
      b0 = max(0, __builtin_amdgcn_readlane(i, __ffsll((long long)m) - 1));
      break;
    }
  }
  for (int i = k + lane;; i += 64) {
    const unsigned long long m = __ballot(i >= n - 1 || se2[i] == 0.0);
    if (m != 0ull) {
      b1 = min(n, __builtin_amdgcn_readlane(i, __ffsll((long long)m) - 1) + 1);
      break;
    }
  }
  for (int round = 0; round < 40; ++round) {
    if (hi - lo <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi)) + 4.0 * pivmin) break;
    const double w = (hi - lo) / 65.0;
    const double x = lo + w * (lane + 1);
    // (a call of its own for all of T: from row b0 on the loop takes twice as long)
    const int cnt = b1 - b0 == n ? sturm(sd, se2, n, x, pivmin) : sturm(sd + b0, se2 + b0, b1 - b0, x, pivmin);
    const unsigned long long m = __ballot(cnt > k - b0);
    const double xs = x;
    if (m == 0ull) {
      lo = __shfl(xs, 63, 64);
    } else {
      const int q = __ffsll((long long)m) - 1;
      const double nh = __shfl(xs, q, 64);
      const double nl = (q > 0) ? __shfl(xs, q - 1 < 0 ? 0 : q - 1, 64) : lo;
      hi = nh;
      lo = nl;
    }
  }
  if (lane == 0) {
    theta[k] = 0.5 * (lo + hi);
    block[k] = make_int2(b0, b1);
  }
}

__device__ __forceinline__ uint64_t hmix(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Inverse iteration, thread j <-> eigenvalue j; Zt comes in with the start
// vectors.  Work arrays are laid out [k * n + j] so that a wave's accesses are
// contiguous.  Output Zt[i*n + j].
// LU of T - lam I with partial pivoting: row k of U holds the pivot's reciprocal
// (array U), Vv on column k + 1 and, where rows k and k + 1 were swapped, e_{k+1}
// on column k + 2; Lm is the multiplier; the swaps are bits in the LDS.
// Every pass is one serial chain per thread, so what counts is the chain's length
// (one reciprocal a step in the LU, one or two multiply-adds in the sweeps) and
// that no load is waited for: a pass loads its next IB steps before it works on
// these.  n = 948: 880 us with divisions in the chains and each IB steps' loads
// waited for (and five work arrays, start vectors formed here),
// now 510 us.
__global__ __launch_bounds__(64) void k_tri_invit(const double* dg, const double* eg, int n,
                                                  const double* raw, const int2* block, double* theta,
                                                  double* U, double* Vv, double* Lm, double* Zt,
                                                  const double* tnorm_dev) {
  constexpr int IB = 16;
  const double tnorm = *tnorm_dev;
  extern __shared__ double sm[];
  double* d = sm;                        // n + IB + 1 entries each, zeros behind T
  double* e = sm + n + IB + 1;
  unsigned short* swaps = (unsigned short*)(e + n + IB + 1);  // IB steps a word: [step / IB][thread]
  for (int i = threadIdx.x; i < n + IB + 1; i += 64) {
    d[i] = i < n ? dg[i] : 0.0;
    e[i] = i < n - 1 ? eg[i] : 0.0;
  }
  __syncthreads();
  const int j = blockIdx.x * 64 + threadIdx.x;
  if (j >= n) return;
  swaps += threadIdx.x;
  const double lam = raw[j];
  // The start vector is zero outside its block, and so is the result: another block's
  // rows would outweigh this one's where they come closer to the eigenvalue (a row
  // of zeros to 1e-71, its own block to a rounding error of its norm).
  const int b0 = block[j].x, b1 = block[j].y;
  int col = j;  // the eigenvalue's place among all, by value and then by row
  if (b0 > 0 || b1 < n) {
    const auto key = [](double x) { return x == x ? x : DBL_MAX * 2.0; };
    const double mine = key(lam);
    col = 0;
    for (int i = 0; i < n; ++i) {
      const double other = key(raw[i]);
      col += other < mine || (other == mine && i < j);
    }
  }
  theta[col] = lam;
  const double tiny = fmax(0x1p-300 * tnorm, 0x1p-960);  // stands for a smaller pivot
  // entry k of thread j's column of a work array, and of its vector
  auto at = [&](double* A, int k) -> double& { return A[(int64_t)k * n + j]; };
  auto zt = [&](int k) -> double& { return Zt[(int64_t)k * n + col]; };
  for (int k = 0; k < b0; ++k) zt(k) = 0.0;
  for (int k = b1; k < n; ++k) zt(k) = 0.0;
  const int nb = (n + IB - 1) / IB;  // blocks of IB steps
  // working row k: (al, be) on columns (k, k+1); the last step is its pivot alone
  double al = d[0] - lam, be = e[0];
  for (int blk = 0; blk < nb; ++blk) {
    const int k0 = blk * IB;
    unsigned bits = 0;
    double dv[IB], ev[IB + 1];
#pragma unroll
    for (int q = 0; q < IB; ++q) {
      dv[q] = d[k0 + q + 1] - lam;
      ev[q] = e[k0 + q];
    }
    ev[IB] = e[k0 + IB];
#pragma unroll
    for (int q = 0; q < IB; ++q) {
      const int k = k0 + q;
      const double ck = ev[q], an = dv[q], bn = ev[q + 1];
      const bool sw = fabs(al) < fabs(ck);  // pivot on the next original row (ck, an, bn)
      double piv = sw ? ck : al;
      if (fabs(piv) < tiny) piv = copysign(tiny, piv);
      const double rp = recip(piv), l = (sw ? al : ck) * rp;
      if (k < n) {
        at(U, k) = rp;
        at(Vv, k) = sw ? an : be;
        at(Lm, k) = l;
      }
      bits |= (unsigned)sw << q;
      const double x = sw ? be : an, y = sw ? an : be;
      al = fma(-l, y, x);
      be = sw ? -l * bn : bn;
    }
    swaps[64 * blk] = (unsigned short)bits;
  }
  // Two sweeps of inverse iteration.  The growth of the first sweep is removed
  // by a power-of-two factor folded into the second sweep's loads (exact, no
  // extra pass); the second sweep's backward pass also accumulates the sum of
  // squares, so one final pass normalises.
  struct Fwd {
    double l[IB], a[IB];
  };
  struct Bwd {
    double y[IB], v[IB], u[IB];
  };
  double sc = 1.0, ssq = 0.0, mx = 0.0;
  for (int it = 0; it < 2; ++it) {
    // forward: apply the row swaps and multipliers; c is the current y_k
    auto load_f = [&](Fwd& f, int blk) {
#pragma unroll
      for (int q = 0; q < IB; ++q) {
        const int k = min(blk * IB + q, n - 1);
        f.l[q] = at(Lm, k);
        f.a[q] = zt(min(k + 1, n - 1));
      }
    };
    double c = zt(0) * sc;
    auto pass_f = [&](const Fwd& f, int blk) {
      const unsigned bits = swaps[64 * blk];
#pragma unroll
      for (int q = 0; q < IB; ++q) {
        const int k = blk * IB + q;
        const double a = f.a[q] * sc;
        const bool sw = (bits >> q) & 1;
        if (k < n - 1) {
          zt(k) = sw ? a : c;
          c = fma(-f.l[q], sw ? a : c, sw ? c : a);
        }
      }
    };
    Fwd f0, f1;
    load_f(f0, 0);
    for (int blk = 0; blk < nb; blk += 2) {
      load_f(f1, blk + 1);
      __builtin_amdgcn_sched_barrier(0);
      pass_f(f0, blk);
      __builtin_amdgcn_sched_barrier(0);
      load_f(f0, blk + 2);
      __builtin_amdgcn_sched_barrier(0);
      if (blk + 1 < nb) pass_f(f1, blk + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    zt(n - 1) = c;
    // backward: U x = y with U upper triangular, bandwidth 3
    double x1 = 0.0, x2 = 0.0;
    mx = 0.0;
    ssq = 0.0;
    auto load_b = [&](Bwd& f, int blk) {
#pragma unroll
      for (int q = 0; q < IB; ++q) {
        const int k = min(max(blk * IB + q, 0), n - 1);
        f.y[q] = zt(k);
        f.v[q] = at(Vv, k);
        f.u[q] = at(U, k);
      }
    };
    auto pass_b = [&](const Bwd& f, int blk) {
      const unsigned bits = swaps[64 * blk];
#pragma unroll
      for (int q = IB - 1; q >= 0; --q) {
        const int k = blk * IB + q;
        if (k < n) {
          const double w = (bits >> q) & 1 ? e[k + 1] : 0.0;
          const double x = fma(-f.v[q], x1, fma(-w, x2, f.y[q])) * f.u[q];
          zt(k) = x;
          x2 = x1;
          x1 = x;
          mx = fmax(mx, fabs(x));
          ssq = fma(x, x, ssq);
        }
      }
    };
    Bwd b0, b1;
    load_b(b0, nb - 1);
    for (int blk = nb - 1; blk >= 0; blk -= 2) {
      load_b(b1, blk - 1);
      __builtin_amdgcn_sched_barrier(0);
      pass_b(b0, blk);
      __builtin_amdgcn_sched_barrier(0);
      load_b(b0, blk - 2);
      __builtin_amdgcn_sched_barrier(0);
      if (blk - 1 >= 0) pass_b(b1, blk - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    int ex = 0;
    (void)frexp(mx, &ex);
    sc = (mx > 0.0 && isfinite(mx)) ? ldexp(1.0, -ex) : 1.0;
  }
  // normalise: from the sum of squares when it is finite, else after scaling
  // by the power of two (a second pass, only for extreme growth)
  constexpr int NB = 32;
  double inv;
  if (ssq > 0.0 && isfinite(ssq)) {
    inv = 1.0 / sqrt(ssq);
  } else {
    double nrm = 0.0;
    for (int k0 = 0; k0 < n; k0 += NB) {
      double zv[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (k0 + q < n) zv[q] = zt(k0 + q);
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (k0 + q < n) nrm += (zv[q] * sc) * (zv[q] * sc);
    }
    inv = (nrm > 0.0 && isfinite(nrm)) ? sc / sqrt(nrm) : 0.0;
  }
  for (int k0 = 0; k0 < n; k0 += NB) {
    double zv[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (k0 + q < n) zv[q] = zt(k0 + q);
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (k0 + q < n) zt(k0 + q) = zv[q] * inv;
  }
}

// Modified Gram-Schmidt inside clusters of (numerically) equal eigenvalues:
// work-group b handles the cluster that starts at index b (if any).
__global__ __launch_bounds__(HT) void k_tri_cluster_mgs(const double* theta, int n, double* Zt,
                                                        const double* tnorm_dev) {
  const double ctol = 1e3 * DBL_EPSILON * fmax(*tnorm_dev, 1e-300);
  __shared__ double sh[4];
  const int b = blockIdx.x;
  if (b >= n) return;
  const bool start = (b == 0 || theta[b] - theta[b - 1] > ctol);
  if (!start || b + 1 >= n || theta[b + 1] - theta[b] > ctol) return;
  int end = b + 1;
  while (end + 1 < n && theta[end + 1] - theta[end] <= ctol) ++end;
  for (int pass = 0; pass < 2; ++pass)
    for (int m = b; m <= end; ++m) {
      for (int q = b; q < m; ++q) {
        double s = 0.0;
        for (int i = threadIdx.x; i < n; i += HT) s += Zt[(int64_t)i * n + q] * Zt[(int64_t)i * n + m];
        s = bsum(s, sh);
        for (int i = threadIdx.x; i < n; i += HT) Zt[(int64_t)i * n + m] -= s * Zt[(int64_t)i * n + q];
        __syncthreads();
      }
      double s = 0.0;
      for (int i = threadIdx.x; i < n; i += HT) {
        const double v = Zt[(int64_t)i * n + m];
        s += v * v;
      }
      s = bsum(s, sh);
      const double inv = (s > 0.0) ? 1.0 / sqrt(s) : 0.0;
      for (int i = threadIdx.x; i < n; i += HT) Zt[(int64_t)i * n + m] *= inv;
      __syncthreads();
    }
}

// Zc(i, j) = Zt[i*n + j] as complex, 32 x 32 tiles through LDS
__global__ __launch_bounds__(256) void k_zt_to_complex(const double* Zt, int n, zd* Z, int64_t ldz) {
  __shared__ double t[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int i0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
  for (int r = ty; r < 32; r += 8) {
    const int i = i0 + r, j = j0 + tx;
    t[r][tx] = (i < n && j < n) ? Zt[(int64_t)i * n + j] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int j = j0 + r, i = i0 + tx;
    if (i < n && j < n) Z[i + (int64_t)j * ldz] = make_double2(t[tx][r], 0.0);
  }
}

// Group 0: the norm of T, and its couplings without those that T is as well without:
//  - up to 16 rounding errors of the larger of the two entries beside them, and not
//    above what moves the smaller one by as many of its own.  Parts of T that differ
//    in size by the rounding error or more (a matrix of low rank) are blocks of their
//    own then: an eigenvalue that is zero but for rounding would, by inverse
//    iteration in both, give the smaller part's vector a second time;
//  - below the square of the rounding error of T (a vector's entries on both sides of
//    one could differ by more than the range of numbers), or whose square is none.
// The others: the start vectors of the inverse iteration
__global__ __launch_bounds__(HT) void k_tri_start(const double* d, const double* e, int n, double* out,
                                                  double* ec, double* Zt) {
  if (blockIdx.x > 0) {
    for (int64_t k = (int64_t)(blockIdx.x - 1) * HT + threadIdx.x; k < (int64_t)n * n;
         k += (int64_t)(gridDim.x - 1) * HT) {
      const uint64_t i = k / n, j = k % n;
      const uint64_t r = hmix((j << 32) ^ i ^ 0x5DEECE66Dull);
      Zt[k] = ((double)(r >> 11) * (1.0 / 9007199254740992.0)) - 0.5;
    }
    return;
  }
  __shared__ double sh[4];
  double m = 0.0;
  for (int i = threadIdx.x; i < n; i += HT)
    m = fmax(m, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + (i < n - 1 ? fabs(e[i]) : 0.0));
  m = bmax(m, sh);
  if (threadIdx.x == 0) out[0] = m;
  for (int i = threadIdx.x; i < n - 1; i += HT) {
    const double x = fabs(e[i]), a = fabs(d[i]), b = fabs(d[i + 1]), eps = 16.0 * DBL_EPSILON;
    const bool none = (x <= eps * fmax(a, b) && x * x <= eps * a * b) || x < 0x1p-106 * m || x * x == 0.0;
    ec[i] = none ? 0.0 : e[i];
  }
}
}  // namespace

// work-groups of the tridiagonalisation: one column per wave as far as the
// order allows, and at most HT, since the next step's block reduction reads
// one work-group partial per thread (measured at n = 948: 12.4 ms per
// eigensolve with 256 groups, 13.2 with 192, 17.6 with 64)
inline int trd_groups(int64_t n) { return (int)(n - 1 < HT ? (n > 1 ? n - 1 : 1) : HT); }

size_t tridiag_eig_work_bytes(int64_t n) {
  // U, Vv, Lm and four vectors, or the tridiagonalisation's exchange
  return std::max(5 * ws_round(sizeof(double) * n * n), 3 * ws_round(sizeof(double) * n * n) +
                                                            3 * ws_round(sizeof(double) * n)) +
         ws_round(sizeof(double) * 8);
}

gevp_status tridiag_eig(gevp_ctx* c, int64_t n64, const double* d, const double* e, double* theta,
                        double* Zt, void* work) {
  if (n64 <= 0) return GEVP_OK;
  const int n = (int)n64;
  char* w = (char*)work;
  auto take = [&](size_t bytes) {
    void* p = w;
    w += ws_round(bytes);
    return p;
  };
  double* U = (double*)take(sizeof(double) * n * n);
  double* Vv = (double*)take(sizeof(double) * n * n);
  double* Lm = (double*)take(sizeof(double) * n * n);
  double* ec = (double*)take(sizeof(double) * n);
  double* raw = (double*)take(sizeof(double) * n);  // eigenvalues by block and their blocks
  int2* block = (int2*)take(sizeof(int2) * n);
  double* tn = (double*)take(sizeof(double) * 8);
  hipLaunchKernelGGL(k_tri_start, dim3(1 + (unsigned)std::min<int64_t>(((int64_t)n * n + HT - 1) / HT, 512)),
                     dim3(HT), 0, c->stream, d, e, n, tn, ec, Zt);
  GEVP_HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(k_tri_bisect, dim3((n + 3) / 4), dim3(HT), sizeof(double) * 2 * n, c->stream,
                     d, ec, n, raw, block);
  GEVP_HIP_TRY(hipGetLastError());
  const size_t shi = sizeof(double) * 2 * (n + 17) + 2 * 64 * (size_t)((n + 15) / 16);
  hipLaunchKernelGGL(k_tri_invit, dim3((n + 63) / 64), dim3(64), shi, c->stream,
                     d, ec, n, raw, block, theta, U, Vv, Lm, Zt, tn);
  GEVP_HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(k_tri_cluster_mgs, dim3(n), dim3(HT), 0, c->stream, theta, n, Zt, tn);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

// Back-transformation Z <- Q Z, Q = G_0 G_1 ... G_{k-1} = I - V T V^H with the
// k = n - 1 reflectors G_i = I - tau_i v_i v_i^H as the columns of V.  For the
// forward accumulation (T_ii = tau_i, T(0:i-1, i) = -tau_i T(0:i-1, 0:i-1)
// V(:, 0:i-1)^H v_i) the inverse of T is diag(1/tau) + striu(V^H V) (the UT
// transform), so with L = T^{-H} = diag(conj(1/tau)) + stril(V^H V):
//   S = V^H Z,   S <- L^{-H} S (= T S),   Z <- Z - V S,
// a Gram product, a triangular solve and two products on the FP64 matrix
// cores.  A reflector with tau = 0 is the identity: its column of V is
// cleared and its diagonal entry of L set to 1, which leaves it out.
__global__ __launch_bounds__(256) void k_ut_clear(int n, int k, zd* V, int64_t ldv, const zd* tau) {
  const int i = blockIdx.x;
  if (i >= k) return;
  const zd t = tau[i];
  if (t.x != 0.0 || t.y != 0.0) return;
  for (int r = threadIdx.x; r < n; r += 256) V[r + (int64_t)i * ldv] = make_double2(0.0, 0.0);
}

__global__ __launch_bounds__(256) void k_ut_diag(int k, zd* L, int64_t ldl, const zd* tau) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= k) return;
  const zd t = tau[i];
  const double dd = t.x * t.x + t.y * t.y;
  // conj(1 / t) = t / |t|^2
  L[i + (int64_t)i * ldl] = (dd == 0.0) ? make_double2(1.0, 0.0) : make_double2(t.x / dd, t.y / dd);
}

size_t heev_work_bytes(int64_t n) {
  const int G = trd_groups(n);
  size_t b = 0;
  b += ws_round(sizeof(zd) * n * n);          // V (reflectors)
  b += ws_round(sizeof(zd) * n);              // tau
  b += 2 * ws_round(sizeof(double) * n);      // d, e
  b += ws_round(sizeof(zd) * 2 * n);          // pb
  b += ws_round(sizeof(zd) * 2 * G);          // pp
  b += ws_round(sizeof(double) * n * n);      // Zt
  b += tridiag_eig_work_bytes(n);
  b += 2 * ws_round(sizeof(zd) * n * n);     // L = T^{-H}, S
  b += ws_round(sizeof(zd) * n * 64);         // inverses of L's diagonal blocks
  return b;
}

// One launch per reflector, where the single launch may not run or gave up: the
// kernel boundary is the grid-wide barrier (a cooperative single launch with
// explicit barriers measured slower, because each barrier must write back and
// invalidate the XCD caches).  Issued one by one, the launches cost the host
// about 4.4 us each at n = 948, more than the later, shorter steps take on the
// GPU; so the sequence is captured once per
// argument set into a graph and replayed (the first call also pays the
// capture).  Any failure of the graph calls falls back to direct launches.
namespace {
constexpr size_t MAX_GRAPHS = 8;

gevp_status hetrd_direct(gevp_ctx* c, hipStream_t st, const TrdArgs& a, int G, size_t sh3) {
  for (int s = 0; s <= a.n - 1; ++s) {
    hipLaunchKernelGGL(k_hetrd_step, dim3(G), dim3(HT), sh3, st, a, s);
    GEVP_HIP_TRY(hipGetLastError());
  }
  return GEVP_OK;
}

gevp_status hetrd_launches(gevp_ctx* c, const TrdArgs& a, int G, size_t sh3) {
  const std::vector<int64_t> key = {a.n, G, (int64_t)(uintptr_t)a.H, a.ldh, (int64_t)(uintptr_t)a.V,
                                    a.ldv, (int64_t)(uintptr_t)a.tau, (int64_t)(uintptr_t)a.d,
                                    (int64_t)(uintptr_t)a.e, (int64_t)(uintptr_t)a.pb,
                                    (int64_t)(uintptr_t)a.pp, (int64_t)sh3};
  for (gevp_ctx::GraphEntry& g : c->graphs)
    if (g.key == key) {
      if (hipGraphLaunch(g.exec, c->stream) == hipSuccess) return GEVP_OK;
      (void)hipGetLastError();
      return hetrd_direct(c, c->stream, a, G, sh3);
    }
  if (!c->cap_stream && hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking) != hipSuccess) {
    c->cap_stream = nullptr;
    (void)hipGetLastError();
    return hetrd_direct(c, c->stream, a, G, sh3);
  }
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  bool ok = hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed) == hipSuccess;
  if (ok) {
    const gevp_status st = hetrd_direct(c, c->cap_stream, a, G, sh3);
    ok = (hipStreamEndCapture(c->cap_stream, &graph) == hipSuccess) && st == GEVP_OK && graph;
  }
  if (ok) ok = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) == hipSuccess;
  if (graph) (void)hipGraphDestroy(graph);
  if (!ok) {
    (void)hipGetLastError();
    if (gevp_log_enabled()) fprintf(stderr, "[gevp] tridiagonalisation graph unavailable: direct launches\n");
    return hetrd_direct(c, c->stream, a, G, sh3);
  }
  if (c->graphs.size() >= MAX_GRAPHS) {  // the oldest may still run on the stream
    GEVP_HIP_TRY(hipStreamSynchronize(c->stream));
    (void)hipGraphExecDestroy(c->graphs.front().exec);
    c->graphs.erase(c->graphs.begin());
  }
  c->graphs.push_back({key, exec});
  GEVP_HIP_TRY(hipGraphLaunch(exec, c->stream));
  return GEVP_OK;
}
}  // namespace

namespace {
// The tridiagonalisation in one launch; *done = false when it may not run or gave
// up, H being unchanged.  A handle whose launch gave up once (its stream may be
// confined to some of the compute units) does not try again.
gevp_status hetrd_all(gevp_ctx* c, const TrdArgs& a, TrdExchange x, bool* done) {
  *done = false;
  if (!resident_allowed(c)) return GEVP_OK;
  const int n = a.n;
  auto* f = n <= 256    ? k_hetrd_all<256, 1>
            : n <= 512  ? k_hetrd_all<512, 1>
            : n <= 1024 ? k_hetrd_all<512, 2>
            : n <= 1536 ? k_hetrd_all<512, 3>
                        : k_hetrd_all<512, 4>;
  const int threads = n <= 256 ? 256 : 512, groups = (n + TRD_COLS - 1) / TRD_COLS;
  if (!resident_fits(c, f, threads, groups)) return GEVP_OK;
  x.ld = (n + 15) / 16 * 16;
  const int64_t words = (int64_t)n * 4 * x.ld;
  if (c->defer_err) {
    x.err = c->defer_err;
    GEVP_TRY(fill_holes(c, x.x, words, nullptr));
    hipLaunchKernelGGL(f, dim3((unsigned)groups), dim3((unsigned)threads), 0, c->stream, a, x);
    GEVP_HIP_TRY(hipGetLastError());
    GEVP_HIP_TRY(hipEventRecord(c->defer_done, c->stream));
    *done = true;
    return GEVP_OK;
  }
  // (eight problems of n = 1500 to 3000 at a time took 90 ms with a launch per
  // reflector, 76 ms with shares of the device)
  GEVP_TRY(fill_holes(c, x.x, words, x.err));
  LaunchTurn turn(c, groups);
  hipLaunchKernelGGL(f, dim3((unsigned)groups), dim3((unsigned)threads), 0, c->stream, a, x);
  const hipError_t launched = hipGetLastError();
  int err = 1;
  GEVP_HIP_TRY(hipMemcpyAsync(&err, x.err, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  GEVP_HIP_TRY(hipStreamSynchronize(c->stream));
  GEVP_HIP_TRY(launched);
  *done = err == 0;
  if (err) {
    if (gevp_log_enabled()) fprintf(stderr, "[gevp] the single-launch tridiagonalisation gave up (n %d)\n", n);
    c->shared_gpu = true;
  }
  return GEVP_OK;
}
}  // namespace

gevp_status heev_small(gevp_ctx* c, int64_t n64, zd* H, int64_t ldh, double* theta, zd* Z,
                       int64_t ldz, void* work) {
  if (n64 <= 0) return GEVP_OK;
  // the reflector step keeps at most QMAX rows per thread and three n-vectors in LDS
  if (n64 > (int64_t)QMAX * HT) return GEVP_ERR_INVALID;
  const int n = (int)n64;
  const int G = trd_groups(n);
  char* w = (char*)work;
  auto take = [&](size_t bytes) {
    void* p = w;
    w += ws_round(bytes);
    return p;
  };
  TrdArgs a;
  a.n = n;
  a.H = H;
  a.ldh = ldh;
  a.V = (zd*)take(sizeof(zd) * n * n);
  a.ldv = n;
  a.tau = (zd*)take(sizeof(zd) * n);
  a.d = (double*)take(sizeof(double) * n);
  a.e = (double*)take(sizeof(double) * n);
  a.pb = (zd*)take(sizeof(zd) * 2 * n);
  a.pp = (zd*)take(sizeof(zd) * 2 * G);
  a.G = G;
  double* Zt = (double*)take(sizeof(double) * n * n);
  void* tw = take(tridiag_eig_work_bytes(n));
  zd* Lut = (zd*)take(sizeof(zd) * n * n);
  zd* Sut = (zd*)take(sizeof(zd) * n * n);
  zd* Dut = (zd*)take(sizeof(zd) * n * 64);

  const size_t shv = sizeof(zd) * (size_t)n;
  const size_t sh3 = 3 * shv;  // v_s, w_{s-1}, v_{s-1}
  static const bool attr = [&]() {
    (void)hipFuncSetAttribute((const void*)k_hetrd_step, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)(3 * sizeof(zd) * 2048));
    return true;
  }();
  (void)attr;
  // Many work-groups in one launch where they can be resident together; one
  // work-group where the exchange through memory costs more than it spreads (the
  // whole eigensolver at n = 32, 64, 116: 0.25, 0.47, 0.94 ms with one, 0.28,
  // 0.45, 0.76 with many); a launch per reflector where that one gave up.  The
  // exchange lies in the tridiagonal solver's workspace, not in use yet (40 n^2 bytes
  // against 32 n (n + 15): enough from n = 60).
  bool done = false;
  if (n > TRD1_MAX && n <= TRDM_MAX && !c->shared_gpu) {
    TrdExchange x{(unsigned long long*)tw, 0, (int*)a.pb, exchange_spins(c)};
    GEVP_TRY(hetrd_all(c, a, x, &done));
  }
  if (n <= TRD1_MAX) {
    hipLaunchKernelGGL(k_hetrd_one, dim3(1), dim3(1024), 0, c->stream, a);
    GEVP_HIP_TRY(hipGetLastError());
    done = true;
  }
  if (!done) {
    GEVP_HIP_TRY(hipMemsetAsync(a.tau, 0, sizeof(zd) * n, c->stream));
    GEVP_TRY(hetrd_launches(c, a, G, sh3));
  }
  GEVP_TRY(tridiag_eig(c, n, a.d, a.e, theta, Zt, tw));
  const unsigned tb = (unsigned)((n + 31) / 32);
  hipLaunchKernelGGL(k_zt_to_complex, dim3(tb, tb), dim3(256), 0, c->stream, Zt, n, Z, ldz);
  GEVP_HIP_TRY(hipGetLastError());
  if (n > 1) {
    const int k = n - 1;
    hipLaunchKernelGGL(k_ut_clear, dim3((unsigned)k), dim3(256), 0, c->stream, n, k, a.V, a.ldv, a.tau);
    GEVP_HIP_TRY(hipGetLastError());
    // FP64 products: short reflectors and eigenvectors of T that decay along it have
    // entries that residues never hold well enough (all four products of 1300 <= n <=
    // 2048 were done again: 24.4 ms a call at 2048, 22.7 with these alone)
    const Fp64Products fp64(c);
    GEVP_TRY(launch_zgemm(c, 1, 0, k, k, n, 1.0, a.V, a.ldv, a.V, a.ldv, 0.0, nullptr, 0, 0.0, nullptr,
                          0, nullptr, Lut, k, nullptr, 1));  // lower triangle of V^H V
    hipLaunchKernelGGL(k_ut_diag, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, c->stream, k, Lut, k,
                       a.tau);
    GEVP_HIP_TRY(hipGetLastError());
    GEVP_TRY(diag_block_inverses(c, k, Lut, k, Dut, k));
    // (V^H is upper triangular: reflector s begins at row s + 1)
    GEVP_TRY(launch_zgemm(c, 1, 0, k, n, n, 1.0, a.V, a.ldv, Z, ldz, 0.0, nullptr, 0, 0.0, nullptr, 0,
                          nullptr, Sut, k, nullptr, 0, 1));
    GEVP_TRY(trsm_left_lower_c(c, k, n, Lut, k, Dut, k, Sut, k, 0));
    GEVP_TRY(launch_zgemm(c, 0, 0, n, n, k, -1.0, a.V, a.ldv, Sut, k, 1.0, Z, ldz, 0.0, nullptr, 0,
                          nullptr, Z, ldz));
  }
  return GEVP_OK;
}
