// Complex128 GEMM in residue arithmetic on the INT8 matrix cores of gfx950
// (v_mfma_i32_16x16x64_i8), for products large enough to amortise the
// conversions.
//
//   D = alpha op(A) op(B) + beta Cm + gamma diag(gcol) E
//
// The method is the Chinese-remainder form of error-free matrix
// multiplication by integer slices (Ozaki, Ogita, Oishi, Rump 2012; the
// modular form: Ozaki, Uchino, Imamura 2025), here for complex matrices:
//
//  1. Row i of op(A) is scaled by a power of two so that its 2-norm lies in
//     [2^57, 2^58) and rounded to integers, column j of op(B) likewise.  By
//     Cauchy-Schwarz every entry of the integer product is below 2^116 in
//     modulus, so it is determined by its residues modulo M > 2^117.6.
//  2. M is a product of 16 pairwise coprime moduli p <= 241 whose prime
//     factors are all 1 mod 4.  -1 then has a square root J mod p and
//     a + ib -> (a + Jb, a - Jb) is a ring isomorphism Z_p[i] -> Z_p x Z_p:
//     a complex product mod p costs TWO real products of residues (against
//     three in Gauss's form), 32 INT8 products in all, each exact in its
//     INT32 accumulators.
//  3. The integer product is rebuilt from its 32 residues by the Chinese
//     remainder theorem in exact FP64 arithmetic (weights cut in three pieces
//     of at most 40 bits), scaled back, and goes through the epilogue.
//
// The only rounding errors are those of step 1 (relative to a row's or a
// column's norm, at most 2^-58 per entry) and of the last few FP64
// operations; the summation itself is exact.  Rows, columns whose norm is
// not finite, or too large or small to be squared, raise a flag on the
// device: the reconstruction then writes nothing and the FP64 kernels
// (zgemm.hip), launched behind it, do the product; they return at once when
// the flag is down.
//
// A row norm says little about a row's small entries, which matter where the
// other operand's entries for the same k are large.  So op(A) op(B) is first
// balanced as (op(A) T)(T^-1 op(B)), T diagonal with powers of two (exact)
// that bring each row of op(B) below 1 (each column of op(A) when op(A) is
// converted ahead, for several products); a slice that is zero in the operand
// looked at is left out of the other one, where it contributes nothing.
//
// Balancing serves gradings along k that all rows share, no others.  So every
// entry of the product is checked.  Each rounding of step 1 being uniform, an entry
// is off by sqrt((|a|^2 + |b|^2) / 6), root mean square, in the integers' unit, a and
// b its row and column; the FP64 kernels' error was measured at 2^-53.9 / sqrt(parts)
// of the entry's sum of sizes S = sum_k |op(A)(i, k)| |op(B)(k, j)| for random
// operands of any k, parts being the parts they cut k in (more where the terms have
// one sign: 2^-51.1 to 2^-52.9 S, here 2^-54.4 S).  Where the former is not
// the smaller, the flag is raised and the FP64 kernels do the product.  S is bounded
// from below by an INT8 product of sizes: each entry's over its row's root mean
// square, rounded down and cut at 127.  A coarse one with k eight times shorter
// comes first and mostly suffices; a tile of the result where it does not takes the
// one of all sizes, as long as a residue product.
// In time: 8192 x 948 x 8192 2.74 ms without the check, 2.81 with it, 3001 x 768 x
// 768 0.181 and 0.185.
//
// Planes: residues of 16 rows and 64 consecutive k are stored as one
// 1 KB MFMA fragment (lane l: row l % 16, sixteen k), so that global loads,
// LDS transfers and fragment reads are all linear.  The order of k inside a
// fragment is free as long as both operands agree: lane group g holds
// k = 4 q + g, q = 0..15, which keeps the conversion's loads of both storage
// orders in runs of at least 64 bytes.
#include <cmath>

#include "common.h"

typedef int i4 __attribute__((ext_vector_type(4)));

template <int V>
struct ic {
  static constexpr int value = V;
};

namespace {
constexpr int NMOD = 16, NCH = 2 * NMOD;  // moduli, residue channels
constexpr int NPL = NCH + 1;              // planes of an operand: the residues, then the sizes
constexpr int COARSE = 8;                 // sizes summed up in one of the coarse plane behind them
constexpr int FR = 16, FK = 64;           // rows and k of a fragment
constexpr int TM = 256;                   // largest output tile of a work-group (rows and columns)
constexpr int SCALE_EXP = 58;             // row and column norms are scaled below 2^58
constexpr float SIZE_UNIT = 48.f;         // size of a root-mean-square entry of a row of norm 2^58
// least sum of sizes of an entry over sqrt(|a|^2 + |b|^2), in units of K and of the
// norms' bound, against FP64 kernels in one part: 2^53.9 / 2^58 / sqrt(6)
constexpr float MIN_SIZES = SIZE_UNIT * SIZE_UNIT * 0.0238f;

typedef unsigned __int128 u128;

struct ModTable {
  int p[NMOD];
  unsigned dlo[NMOD], dhi[NMOD];    // 256^0..3 and 256^4..7 mod p as signed bytes
  unsigned jlo[NMOD], jhi[NMOD];    // J 256^i mod p
  double wre[NMOD][3], wim[NMOD][3];  // CRT weights of u+ + u- and u+ - u-, cut at 2^40 and 2^80
  double M[3], invM;                // M likewise, and 2^80 / M
};

constexpr int mod_list[NMOD] = {241, 233, 229, 221, 205, 197, 193, 181,
                                173, 157, 149, 137, 113, 109, 101, 97};

constexpr int inv_mod(int a, int p) {
  for (int x = 1; x < p; ++x)
    if ((int64_t)a * x % p == 1) return x;
  return 0;
}
constexpr int sqrt_m1(int p) {
  for (int x = 1; x < p; ++x)
    if (x * x % p == p - 1) return x;
  return 0;
}
constexpr unsigned sym_byte(int r, int p) {  // residue as a signed byte
  return (unsigned)(unsigned char)(r > p / 2 ? r - p : r);
}
constexpr ModTable make_table() {
  ModTable t{};
  u128 M = 1;
  for (int i = 0; i < NMOD; ++i) M *= (u128)mod_list[i];
  const u128 mask = ((u128)1 << 40) - 1;
  for (int i = 0; i < NMOD; ++i) {
    const int p = mod_list[i], J = sqrt_m1(p);
    t.p[i] = p;
    int pw = 1;
    for (int d = 0; d < 8; ++d) {
      const unsigned b = sym_byte(pw, p), jb = sym_byte(pw * J % p, p);
      if (d < 4) {
        t.dlo[i] |= b << (8 * d);
        t.jlo[i] |= jb << (8 * d);
      } else {
        t.dhi[i] |= b << (8 * (d - 4));
        t.jhi[i] |= jb << (8 * (d - 4));
      }
      pw = pw * 256 % p;
    }
    // re = (u+ + u-) / 2, im = (u+ - u-) / (2 J); weight = (M/p) [(M/p)^-1 / 2 or / 2J]_p
    const u128 Mp = M / (u128)p;
    const int ip = inv_mod((int)(Mp % (u128)p), p);
    const int yre = ip * inv_mod(2, p) % p, yim = ip * inv_mod(2 * J % p, p) % p;
    const u128 wr = Mp * (u128)yre, wi = Mp * (u128)yim;
    for (int c = 0; c < 3; ++c) {
      const u128 a = wr >> (40 * c), b = wi >> (40 * c);
      t.wre[i][c] = (double)(uint64_t)(c < 2 ? (a & mask) : a);
      t.wim[i][c] = (double)(uint64_t)(c < 2 ? (b & mask) : b);
    }
  }
  t.M[0] = (double)(uint64_t)(M & mask);
  t.M[1] = (double)(uint64_t)((M >> 40) & mask);
  t.M[2] = (double)(uint64_t)(M >> 80);
  t.invM = 1.0 / ((t.M[0] / 1099511627776.0 + t.M[1]) / 1099511627776.0 + t.M[2]);
  return t;
}
__constant__ ModTable c_tab = make_table();

// One operand as stored: element (r, k) of the r-indexed matrix op(A) (or of
// op(B)^T) is src[r * rs + k * ks], conjugated if conj; rows >= r1 come from
// src2 (row r - r1); tri = 1: entries with k < r read as zero.
struct ModSrc {
  const zd* src;
  const zd* src2;
  int64_t ld;
  int rows, K, r1;
  int kfast;  // 1: k is the contiguous index
  int conj, tri;
};

// (no branch around the load: an entry outside reads element 0 instead, so that
// a loop's loads can all be issued before the first is used)
__device__ __forceinline__ zd mod_elem(const ModSrc& s, int r, int k) {
  const bool in = r < s.rows && k < s.K && !(s.tri && k < r);
  const bool lo = in && r >= s.r1;
  const int64_t rr = lo ? r - s.r1 : r;
  const int64_t off = in ? (s.kfast ? k + rr * s.ld : rr + k * s.ld) : 0;
  const zd v = (lo ? s.src2 : s.src)[off];
  return in ? v : make_double2(0.0, 0.0);
}

// The balancing scales, ks0[k] = 2^-x for the operand looked at here, ks1[k] =
// 2^x for the other one: the largest entry of its slice k is brought into
// [1/2, 1).  Every entry counts (a sample of a slice may see only small ones).
// Of a zero slice the other operand's entries count for nothing, however large.
// With several chunks of rows the maxima go to part[chunk][k] first.
constexpr int BAL_ROWS = 1024;  // rows of a chunk, k contiguous
__device__ __forceinline__ void balance_store(int k, double m, double* ks0, double* ks1) {
  int x = 0;
  if (m > 0.0 && m < 1e300) (void)frexp(m, &x);
  x = max(-250, min(250, x));
  ks0[k] = ldexp(1.0, -x);
  ks1[k] = m == 0.0 ? 0.0 : ldexp(1.0, x);  // (a NaN or an infinity still raises the flag)
}
__global__ __launch_bounds__(1024) void k_mod_balance(ModSrc s, double* ks0, double* ks1, double* part,
                                                      int chunks) {
  __shared__ double sh[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto mag = [&](int r, int k) {
    const zd v = mod_elem(s, r, k);
    return fmax(fabs(v.x), fabs(v.y));
  };
  double m = 0.0;
  if (s.kfast) {  // k contiguous: 64 k and a chunk of rows per work-group
    const int kb = blockIdx.x / chunks, c = blockIdx.x - kb * chunks;
    const int k = kb * 64 + lane, r1 = chunks == 1 ? s.rows : min(s.rows, (c + 1) * BAL_ROWS);
#pragma unroll 8
    for (int r = c * BAL_ROWS + wave; r < r1; r += 16) m = fmax(m, mag(r, k));
    sh[wave][lane] = m;
    __syncthreads();
    if (wave != 0 || k >= s.K) return;
#pragma unroll
    for (int q = 1; q < 16; ++q) m = fmax(m, sh[q][lane]);
    if (chunks > 1)
      part[(int64_t)c * s.K + k] = m;
    else
      balance_store(k, m, ks0, ks1);
  } else {  // rows contiguous: a wave per k
    const int k = blockIdx.x * 16 + wave;
    if (k >= s.K) return;
#pragma unroll 8
    for (int r = lane; r < s.rows; r += 64) m = fmax(m, mag(r, k));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    if (lane == 0) balance_store(k, m, ks0, ks1);
  }
}
__global__ __launch_bounds__(256) void k_mod_balance_finish(const double* part, int K, int chunks, double* ks0,
                                                            double* ks1) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= K) return;
  double m = 0.0;
  for (int c = 0; c < chunks; ++c) m = fmax(m, part[(int64_t)c * K + k]);
  balance_store(k, m, ks0, ks1);
}

// Row sums of squares in at most MAXC chunks of k (part[chunk][row]; -1 for a
// chunk without a nonzero entry that counts), each operand in the order its
// storage favours.
constexpr int MAXC = 16;
__device__ __forceinline__ void norm_kfast(const ModSrc& s, const double* ks, int blk, int nch, int clen,
                                           double* part) {
  // one wave per row and chunk
  const int64_t w = (int64_t)blk * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, c = (int)(w % nch);
  const int64_t r = w / nch;
  if (r >= s.rows) return;
  const int k1 = min(s.K, (c + 1) * clen);
  double ss = 0.0, nz = 0.0;
#pragma unroll 8
  for (int k = c * clen + lane; k < k1; k += 64) {
    zd v = mod_elem(s, (int)r, k);
    nz = ((v.x != 0.0 || v.y != 0.0) && ks[k] != 0.0) ? 1.0 : nz;
    v.x *= ks[k];
    v.y *= ks[k];
    ss += v.x * v.x + v.y * v.y;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ss += __shfl_xor(ss, o, 64);
    nz = fmax(nz, __shfl_xor(nz, o, 64));
  }
  if (lane == 0) part[(int64_t)c * s.rows + r] = (nz == 0.0 && ss == 0.0) ? -1.0 : ss;
}
__device__ __forceinline__ void norm_rfast(const ModSrc& s, const double* ks, int blk, int nch, int clen,
                                           double* part) {
  // 64 rows and one chunk per work-group
  __shared__ double sh[4][64];
  const int rb = blk / nch, c = blk % nch;
  const int r = rb * 64 + (threadIdx.x & 63), w = threadIdx.x >> 6;
  double ss = 0.0, nz = 0.0;
  if (r < s.rows) {
    const int k1 = min(s.K, (c + 1) * clen);
#pragma unroll 8
    for (int k = c * clen + w; k < k1; k += 4) {
      zd v = mod_elem(s, r, k);
      nz = ((v.x != 0.0 || v.y != 0.0) && ks[k] != 0.0) ? 1.0 : nz;
      v.x *= ks[k];
      v.y *= ks[k];
      ss += v.x * v.x + v.y * v.y;
    }
  }
  sh[w][threadIdx.x & 63] = (nz == 0.0 && ss == 0.0) ? -1.0 : ss;
  __syncthreads();
  if (w == 0 && r < s.rows) {
    double t = -1.0;
    for (int q = 0; q < 4; ++q) {
      const double v = sh[q][threadIdx.x];
      if (v != -1.0) t = (t == -1.0 ? 0.0 : t) + v;
    }
    part[(int64_t)c * s.rows + r] = t;
  }
}

struct ConvArgs {
  ModSrc s[2];             // op(A), op(B)^T
  int blk[2];              // work-groups of each (0: already converted)
  int nch[2], clen[2];
  const double* ks[2];     // balancing scale of each k
  double* part[2];
  int* ex[2];              // scale exponents, written by the conversion
  float* nr[2];            // scaled norms over 2^58: in [1/2, 1), 0 for a row of zeros
  unsigned char* planes[2];
  int rg[2], kb[2];        // fragments along rows and k
  int* flag;
};
__global__ __launch_bounds__(256) void k_mod_norms(ConvArgs p) {
  const int w = (int)blockIdx.x >= p.blk[0];
  const int b = blockIdx.x - (w ? p.blk[0] : 0);
  if (blockIdx.x == 0 && threadIdx.x < 2) p.flag[threadIdx.x] = 0;  // raised by the conversion and the check
  if (p.s[w].kfast)
    norm_kfast(p.s[w], p.ks[w], b, p.nch[w], p.clen[w], p.part[w]);
  else
    norm_rfast(p.s[w], p.ks[w], b, p.nch[w], p.clen[w], p.part[w]);
}

// v mod p in the low byte, nearest zero (|v| < 2^24, so v is exact in FP32 and
// the rounded quotient is off by at most p 2^-7 in the remainder).  Only the
// low byte of v - q p is needed, so q is read from the bits of a float whose
// unit is 1: its exponent adds a multiple of 2^22.
__device__ __forceinline__ unsigned low_residue(int v, float ip, int mod) {
  const float q = fmaf((float)v, ip, 12582912.0f);
  return (unsigned)(v - __mul24((int)__float_as_uint(q), mod));
}
// the low bytes of four words
__device__ __forceinline__ unsigned pack4(unsigned a, unsigned b, unsigned c, unsigned d) {
  const unsigned ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);
  const unsigned cd = __builtin_amdgcn_perm(d, c, 0x04000c0cu);
  return ab | cd;
}

// Conversion of one operand: each lane scales and rounds sixteen entries of
// one row to integers (eight signed digits of base 256 each for re and im)
// and writes their residues in every channel: a residue of a + Jb is a sum of
// sixteen digit products (v_dot4_i32_i8, below 2^18), reduced with one FP32
// multiply-round-subtract, which is exact at that size.  Bound by the bytes
// written (32 per complex entry) as much as by the about 550 vector
// instructions per entry.  The sizes (|entry| over its row's root mean square) go
// out as one plane more.
__device__ __forceinline__ void digits(double x, unsigned& lo, unsigned& hi) {
  const long long t = __double2ll_rn(x);
  const unsigned long long u = (unsigned long long)t + 0x0080808080808080ull;
  lo = (unsigned)u ^ 0x80808080u;
  hi = (unsigned)(u >> 32) ^ 0x00808080u;
}
__global__ __launch_bounds__(256, 4) void k_mod_split(ConvArgs p) {
  const int lane = threadIdx.x & 63;
  const int w = (int)blockIdx.x >= p.blk[0];
  const int64_t f = (int64_t)(blockIdx.x - (w ? p.blk[0] : 0)) * 4 + (threadIdx.x >> 6);
  const ModSrc& s = p.s[w];
  const int rg = p.rg[w], nkb = p.kb[w];
  if (f >= (int64_t)rg * nkb) return;
  int g, kb;
  if (s.kfast) {  // neighbouring waves on neighbouring k of the same rows
    g = (int)(f / nkb);
    kb = (int)(f - (int64_t)g * nkb);
  } else {
    kb = (int)(f / rg);
    g = (int)(f - (int64_t)kb * rg);
  }
  const int r = g * FR + (lane & 15), k0 = kb * FK + (lane >> 4);
  // the row's scale: 2^e times it has its norm in [2^57, 2^58).  A sum that is
  // not finite, or whose terms left the range of safe squares, raises the flag.
  double ss = 0.0;
  int any = 0;
  if (r < s.rows)
    for (int c = lane >> 4; c < p.nch[w]; c += 4) {
      const double v = p.part[w][(int64_t)c * s.rows + r];
      if (v != -1.0) {
        ss += v;
        any = 1;
      }
    }
  ss += __shfl_xor(ss, 16, 64);
  ss += __shfl_xor(ss, 32, 64);
  any |= __shfl_xor(any, 16, 64);
  any |= __shfl_xor(any, 32, 64);
  int e = 0;
  float nr = 0.f;
  if (any) {
    if (ss > 1e-250 && ss < 1e250) {
      int x = 0;
      nr = (float)frexp(sqrt(ss), &x);
      e = SCALE_EXP - x;
    } else {
      *p.flag = 1;
    }
  }
  if (kb == 0 && lane < 16 && r < s.rows) {
    p.ex[w][r] = e;
    p.nr[w][r] = nr;
  }
  const double sc = ldexp(1.0, e);
  const int64_t chs = (int64_t)rg * nkb * 1024;  // bytes per channel
  unsigned char* out = p.planes[w] + ((int64_t)g * nkb + kb) * 1024 + lane * 16;
  unsigned alo[16], ahi[16], blo[16], bhi[16];
  {
    const float unit = SIZE_UNIT * __builtin_amdgcn_sqrtf((float)s.K) * 0x1p-58f;
    unsigned size[4] = {0, 0, 0, 0}, sum[2] = {0, 0}, least[2] = {127, 127};
    zd v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = mod_elem(s, r, k0 + 4 * q);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      // (a factor past 2^1023 would need both scales at their limits)
      const double f = sc * (k0 + 4 * q < s.K ? p.ks[w][k0 + 4 * q] : 0.0);
      digits(v[q].x * f, alo[q], ahi[q]);
      digits((s.conj ? -v[q].y : v[q].y) * f, blo[q], bhi[q]);
      const float x = (float)(v[q].x * f), y = (float)(v[q].y * f);
      const unsigned z = (unsigned)fminf(unit * __builtin_amdgcn_sqrtf(x * x + y * y), 127.f);
      size[q >> 2] |= z << (8 * (q & 3));
      sum[q >> 3] += z;
      least[q >> 3] = min(least[q >> 3], z);
      if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
    // the coarse plane: eight of a lane's sizes in one, their mean on the left, their
    // least on the right (the sum of the eight products is at least eight times the
    // product of these)
    const unsigned c8 = w == 0 ? sum[0] / 8 | sum[1] / 8 << 8 : least[0] | least[1] << 8;
    const int nkc = (nkb + COARSE - 1) / COARSE;
    unsigned char* oc = p.planes[w] + NPL * chs + ((int64_t)g * nkc + kb / COARSE) * 1024 + lane * 16;
    *reinterpret_cast<unsigned short*>(oc + 2 * (kb % COARSE)) = (unsigned short)c8;
    if (kb == nkb - 1)  // zeros to the fragment's end
      for (int z = kb % COARSE + 1; z < COARSE; ++z) *reinterpret_cast<unsigned short*>(oc + 2 * z) = 0;
    *reinterpret_cast<uint4*>(out + (int64_t)NCH * chs) = make_uint4(size[0], size[1], size[2], size[3]);
  }
  for (int m = 0; m < NMOD; ++m) {
    const unsigned dlo = c_tab.dlo[m], dhi = c_tab.dhi[m], jlo = c_tab.jlo[m], jhi = c_tab.jhi[m];
    const int mod = c_tab.p[m];
    const float ip = 1.0f / (float)mod;
    unsigned up[4], um[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      unsigned zp[4], zm[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int z = 4 * w + q;
        int sa = __builtin_amdgcn_sdot4((int)ahi[z], (int)dhi, 0, false);
        sa = __builtin_amdgcn_sdot4((int)alo[z], (int)dlo, sa, false);
        int sb = __builtin_amdgcn_sdot4((int)bhi[z], (int)jhi, 0, false);
        sb = __builtin_amdgcn_sdot4((int)blo[z], (int)jlo, sb, false);
        zp[q] = low_residue(sa + sb, ip, mod);
        zm[q] = low_residue(sa - sb, ip, mod);
      }
      up[w] = pack4(zp[0], zp[1], zp[2], zp[3]);
      um[w] = pack4(zm[0], zm[1], zm[2], zm[3]);
    }
    *reinterpret_cast<uint4*>(out + (int64_t)(2 * m) * chs) = make_uint4(up[0], up[1], up[2], up[3]);
    *reinterpret_cast<uint4*>(out + (int64_t)(2 * m + 1) * chs) = make_uint4(um[0], um[1], um[2], um[3]);
  }
}

// The residue products: channel c of the result is the INT32 product of the
// operands' channel-c planes, reduced mod p to one byte.  Beside them the check's
// sums of sizes, which are compared and not kept.
//
// Eight waves (2 x 4) own a 32 MI x 64 NJ tile, each MI x NJ MFMA blocks.  The
// largest, 256 x 256 with 128 accumulators per wave and two waves per SIMD,
// moves the fewest bytes per product; 256 x 128 and 128 x 128 serve results
// that would leave compute units idle or be mostly padding (mod_tile).  K
// advances 64 per stage through four stages, filled by direct global -> LDS
// transfers three stages ahead.  Within a stage the fragments of the next few
// MFMAs are read from the LDS while the current ones run, so no wave waits
// for a whole stage of reads.
struct ModGemmArgs {
  const unsigned char* A;
  const unsigned char* B;
  unsigned* R;
  int rga, rgb, kb;      // fragments of A rows, B columns, k
  int tiles_m, tiles_n, tiles;
  int lower, tri;
  int rb, cb;            // 16 x 16 blocks of the result
  int total, checks;     // work-groups of the residue products, and of the check (a multiple of 8)
  int small;             // 1: the INT32 sums stay below 2^24
  // the check: norms of A's rows and B's columns, the least sum of sizes of an entry
  // over the root of the sum of their squares
  const float *nra, *nrb;
  int M, N;
  float least;
  // flag[0]: an operand could not be scaled, flag[1]: raised by the check here; of
  // an operand converted ahead the first alone
  int* flag;
  const int* flag2;
};

// The INT32 product of a tile: ga, gb the first fragments of A and B this wave
// transfers, fs bytes from one fragment row to the next, stages kb0 .. kb - 1.
// off: the transfers issued ahead are waited for and nothing is computed.
template <int MI, int NJ>
struct ModTile {
  static constexpr int TM = 32 * MI, TN = 64 * NJ;
  static constexpr int A_ST = (TM / FR) * 1024, ST = A_ST + (TN / FR) * 1024;
  static constexpr int TA = MI / 4, TB = NJ / 2;  // fragments of A and B a wave transfers per stage
};
template <int MI, int NJ>
__device__ __forceinline__ void mod_product(const unsigned char* ga, const unsigned char* gb, int64_t fs, int kb0,
                                            int kb, int off, unsigned char* s0, unsigned char* s1,
                                            unsigned char* s2, unsigned char* s3, i4 (&acc)[MI][NJ]) {
  typedef ModTile<MI, NJ> G;
  constexpr int A_ST = G::A_ST, TA = G::TA, TB = G::TB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave >> 2, wc = wave & 3;
  auto issue = [&](int kk, unsigned char* st) {
#pragma unroll
    for (int i = 0; i < TA; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(ga + i * fs + (int64_t)kk * 1024 + lane * 16),
                                       (__attribute__((address_space(3))) void*)(st + (wave * TA + i) * 1024),
                                       16, 0, 0);
#pragma unroll
    for (int i = 0; i < TB; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(gb + i * fs + (int64_t)kk * 1024 + lane * 16),
                                       (__attribute__((address_space(3))) void*)(st + A_ST + (wave * TB + i) * 1024),
                                       16, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = i4{0, 0, 0, 0};
  auto rd_a = [&](const unsigned char* st, int i) {
    return *(const i4*)(st + (wr * MI + i) * 1024 + lane * 16);
  };
  auto rd_b = [&](const unsigned char* st, int j) {
    return *(const i4*)(st + A_ST + (wc * NJ + j) * 1024 + lane * 16);
  };
  i4 b0[NJ], b1[NJ], a0[2], a1[2];  // B fragments of this and the next stage; two A fragments ahead
  // stages beyond the last are filled with the last one again, so that every
  // pass through the loop issues and waits alike and runs without branches
  const int n = kb - kb0, last = kb - 1;
  constexpr int T = TA + TB;  // transfers a stage
  issue(kb0, s0);
  issue(min(kb0 + 1, last), s1);
  issue(min(kb0 + 2, last), s2);
  if (off != 0) {
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), as at the end
    return;
  }
  __builtin_amdgcn_s_waitcnt(0x0f70 | (2 * T));  // vmcnt(2 T): stage 0 has landed
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int j = 0; j < NJ; ++j) b0[j] = rd_b(s0, j);
  a0[0] = rd_a(s0, 0);
  a0[1] = rd_a(s0, 1);
  // st holds stage u, st1 stage u + 1, st3 takes stage u + 3 (its last readers
  // finished before the barrier).  Phases of 2 NJ MFMAs, each first waiting for
  // the LDS reads of the phase before and then issuing the next ones: two A
  // fragments for the next phase, and B fragments for the next stage.  (The
  // waits are explicit since the compiler, seeing transfers to the LDS in
  // flight, would wait for the newest read.)  A bare barrier: __syncthreads()
  // would also drain the transfers.
  auto body = [&](i4(&b)[NJ], i4(&bn)[NJ], const unsigned char* st, const unsigned char* st1,
                  unsigned char* st3, int u) {
    __builtin_amdgcn_s_waitcnt(0x0f70 | T);  // vmcnt(T): stage u + 1 has landed
    __builtin_amdgcn_s_barrier();
    issue(min(kb0 + u + 3, last), st3);
    auto phase = [&](auto P, i4(&a)[2], i4(&an)[2]) {
      constexpr int q = decltype(P)::value, np = MI / 2;
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
      an[0] = q + 1 < np ? rd_a(st, 2 * q + 2) : rd_a(st1, 0);
      an[1] = q + 1 < np ? rd_a(st, 2 * q + 3) : rd_a(st1, 1);
#pragma unroll
      for (int j = q * NJ / np; j < (q + 1) * NJ / np; ++j) bn[j] = rd_b(st1, j);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[2 * q + i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[2 * q + i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    phase(ic<0>{}, a0, a1);
    phase(ic<1>{}, a1, a0);
    if constexpr (MI == 8) {
      phase(ic<2>{}, a0, a1);
      phase(ic<3>{}, a1, a0);
    }
  };
  int u = 0;
  for (; u + 4 <= n; u += 4) {
    body(b0, b1, s0, s1, s3, u);
    body(b1, b0, s1, s2, s0, u + 1);
    body(b0, b1, s2, s3, s1, u + 2);
    body(b1, b0, s3, s0, s2, u + 3);
  }
  if (u < n) body(b0, b1, s0, s1, s3, u);
  if (u + 1 < n) body(b1, b0, s1, s2, s0, u + 1);
  if (u + 2 < n) body(b0, b1, s2, s3, s1, u + 2);
  // nothing may be in flight to the LDS when the work-group ends
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
}

template <int MI, int NJ>
__global__ __launch_bounds__(512, 2) void k_mod_gemm(ModGemmArgs p) {
  typedef ModTile<MI, NJ> G;
  constexpr int TM = G::TM, TN = G::TN;
  __shared__ __attribute__((aligned(16))) unsigned char s0[G::ST], s1[G::ST], s2[G::ST], s3[G::ST];
  __shared__ int below;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: addresses in scalar registers
  // The check's tiles come first: they are the short ones (and spread over the XCDs
  // as they are).  Then XCD-aware order: eight consecutive work-groups go to the
  // eight XCDs; give each XCD a contiguous range
  const bool check = (int)blockIdx.x < p.checks;
  int t = blockIdx.x, ch = 0;
  if (!check) {
    const int per = (p.total + 7) >> 3, q = blockIdx.x - p.checks;
    const int L = (q & 7) * per + (q >> 3);
    if (L >= p.total) return;
    ch = L / p.tiles;
    t = L - ch * p.tiles;
  } else if (t >= p.tiles) {
    return;
  }
  // groups of eight row tiles, walked column by column: the tiles in flight
  // on an XCD share few row and column panels
  const int gsz = 8 * p.tiles_n, gi = t / gsz, gr = min(8, p.tiles_m - gi * 8);
  t -= gi * gsz;
  const int tn = t / gr, tm = gi * 8 + (t - tn * gr);
  const int row0 = tm * TM, col0 = tn * TN;
  if (p.lower && col0 > row0 + TM - 1) return;  // entirely above the diagonal
  const int kb0 = p.tri ? min(row0 / FK, p.kb - 1) : 0;  // (rows beyond K: one stage of zeros)
  const int wr = wave >> 2, wc = wave & 3;
  const int off = p.flag[0] | (p.flag2 ? *p.flag2 : 0);  // left to the FP64 kernels
  const int64_t fs = (int64_t)p.kb * 1024;
  const int64_t fra = row0 / FR + wave * G::TA, frb = col0 / FR + wave * G::TB;  // this wave's transfers
  i4 acc[MI][NJ];

  if (check) {
    // the sums of sizes, compared with the norms: those of the coarse planes where
    // they suffice for the tile, else those of the full ones
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
      const int kb = pass == 0 ? (p.kb + COARSE - 1) / COARSE : p.kb, planes = pass == 0 ? NPL : NCH;
      const int64_t fp = (int64_t)kb * 1024;
      mod_product<MI, NJ>(p.A + planes * p.rga * fs + fra * fp, p.B + planes * p.rgb * fs + frb * fp, fp,
                          pass == 0 ? kb0 / COARSE : kb0, kb, off, s0, s1, s2, s3, acc);
      if (off != 0) return;
      const float least = pass == 0 ? p.least * (1.f / COARSE) : p.least;
      // the comparison's addresses and norms belong here, not in registers across the product
      int wr = wave >> 2, wc = wave & 3;
      asm volatile("" : "+s"(wr), "+s"(wc));
      bool low = false;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int rb = row0 / FR + wr * MI + i;
        if (rb >= p.rb) continue;
        float na[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = rb * 16 + 4 * (lane >> 4) + r;
          na[r] = row < p.M ? p.nra[row] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int cb = col0 / FR + wc * NJ + j, col = cb * 16 + (lane & 15);
          if (cb >= p.cb || (p.lower && (cb >> 2) > (rb >> 2))) continue;
          const float nb = col < p.N ? p.nrb[col] : 0.f;
#pragma unroll
          for (int r = 0; r < 4; ++r)  // (a row or column of zeros needs no check)
            low |= na[r] * nb > 0.f &&
                   (float)acc[i][j][r] < least * __builtin_amdgcn_sqrtf(na[r] * na[r] + nb * nb);
        }
      }
      if (threadIdx.x == 0) below = 0;
      __syncthreads();
      if (low) below = 1;
      __syncthreads();
      const int again = below;
      __syncthreads();
      if (again == 0) return;
    }
    if (threadIdx.x == 0) p.flag[1] = 1;
    return;
  }
  mod_product<MI, NJ>(p.A + ((int64_t)ch * p.rga + fra) * fs, p.B + ((int64_t)ch * p.rgb + frb) * fs, fs, kb0, p.kb,
                      off, s0, s1, s2, s3, acc);
  if (off != 0) return;

  // residues of the INT32 sums, folded at 2^16 first where they may pass 2^24
  const int mod = c_tab.p[ch >> 1];
  const float ip = 1.0f / (float)mod;
  const int c16 = 65536 % mod > mod / 2 ? 65536 % mod - mod : 65536 % mod;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int rb = row0 / FR + wr * MI + i;
    if (rb >= p.rb) continue;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int cb = col0 / FR + wc * NJ + j;
      if (cb >= p.cb) continue;
      unsigned z[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int v = acc[i][j][r];
        if (!p.small) v = (v >> 16) * c16 + (v & 65535);
        z[r] = low_residue(v, ip, mod);
      }
      p.R[(((int64_t)ch * p.rb + rb) * p.cb + cb) * 64 + lane] = pack4(z[0], z[1], z[2], z[3]);
    }
  }
}

// Reconstruction and epilogue: one wave per 16 x 16 block of the result, four
// rows of one column per lane.  The weighted sums are exact (pieces of 40
// bits times 9-bit integers, sixteen terms), the multiple of M to take off
// comes from the top piece, and only the last additions round.
struct CrtArgs {
  const unsigned* R;
  const int *exa, *exb, *flag, *flag2;
  int M, N, rb, cb, lower;
  const zd* Cm;
  int64_t ldc;
  const zd* E;
  int64_t lde;
  const double* gcol;
  zd* D;
  int64_t ldd;
  double alpha, beta, gamma;
  const double* coef;
};
__global__ __launch_bounds__(256) void k_mod_crt(CrtArgs p) {
  if ((p.flag[0] | p.flag[1]) != 0 || (p.flag2 && *p.flag2 != 0)) return;  // the FP64 kernels take over
  const int lane = threadIdx.x & 63;
  const int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (blk >= (int64_t)p.rb * p.cb) return;
  const int cb = (int)(blk / p.rb), rb = (int)(blk - (int64_t)cb * p.rb);
  // a lower-triangle product writes the same 64 x 64 tiles as the FP64 kernels
  if (p.lower && (cb >> 2) > (rb >> 2)) return;
  unsigned res[NCH];
  const int64_t chs = (int64_t)p.rb * p.cb * 64;
  const unsigned* src = p.R + ((int64_t)rb * p.cb + cb) * 64 + lane;
#pragma unroll
  for (int c = 0; c < NCH; ++c) res[c] = src[c * chs];
  double alpha = p.alpha, beta = p.beta, gamma = p.gamma;
  if (p.coef) {
    alpha = p.coef[0];
    beta = p.coef[1];
    gamma = p.coef[2];
  }
  const int col = cb * 16 + (lane & 15), rowb = rb * 16 + 4 * (lane >> 4);
  if (col >= p.N) return;
  const bool useC = (p.Cm != nullptr) && (beta != 0.0);
  const bool useE = (p.E != nullptr) && (gamma != 0.0);
  const double g = useE ? gamma * (p.gcol ? p.gcol[col] : 1.0) : 0.0;
  const int eb = p.exb[col];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = rowb + r;
    double re[3] = {0, 0, 0}, im[3] = {0, 0, 0};
#pragma unroll
    for (int m = 0; m < NMOD; ++m) {
      const int up = (int)(res[2 * m] << (24 - 8 * r)) >> 24, um = (int)(res[2 * m + 1] << (24 - 8 * r)) >> 24;
      const double s = (double)(up + um), d = (double)(up - um);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        re[c] = fma(s, c_tab.wre[m][c], re[c]);
        im[c] = fma(d, c_tab.wim[m][c], im[c]);
      }
    }
    if (row >= p.M) continue;
    constexpr double T40 = 1099511627776.0;
    auto rebuild = [&](const double* v) {
      const double q = rint((v[2] + v[1] / T40) * c_tab.invM);
      const double h = fma(-q, c_tab.M[2], v[2]), md = fma(-q, c_tab.M[1], v[1]),
                   lo = fma(-q, c_tab.M[0], v[0]);
      return (h * T40 + md) * T40 + lo;
    };
    const int e = -(p.exa[row] + eb);
    double vr = alpha * ldexp(rebuild(re), e), vi = alpha * ldexp(rebuild(im), e);
    if (useC) {
      const zd cv = p.Cm[row + (int64_t)col * p.ldc];
      vr += beta * cv.x;
      vi += beta * cv.y;
    }
    if (useE) {
      const zd ev = p.E[row + (int64_t)col * p.lde];
      vr += g * ev.x;
      vi += g * ev.y;
    }
    p.D[row + (int64_t)col * p.ldd] = make_double2(vr, vi);
  }
}

inline int64_t up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }
// planes of a rows x k operand: rows padded to the largest tile (the padding is
// never written: it only has to be readable), k to a fragment (zeros)
inline int64_t plane_bytes(int64_t rows, int64_t k) {
  return up(rows, TM) * (up(k, FK) * NPL + up(k, FK * COARSE) / COARSE);
}
inline int chunks(int64_t k) { return (int)std::max<int64_t>(1, std::min<int64_t>(MAXC, k / 128)); }
inline size_t conv_bytes(int64_t rows, int64_t k) {
  return ws_round(plane_bytes(rows, k)) + ws_round(sizeof(int) * rows) + ws_round(sizeof(float) * rows) +
         ws_round(sizeof(double) * rows * chunks(k));
}

struct Carver {
  char* p;
  void* take(size_t b) {
    void* r = p;
    p += ws_round(b);
    return r;
  }
};

void set_operand(ConvArgs& c, int w, const ModSrc& s, Carver& m) {
  c.s[w] = s;
  c.nch[w] = chunks(s.K);
  c.clen[w] = (s.K + c.nch[w] - 1) / c.nch[w];
  c.rg[w] = (int)((s.rows + FR - 1) / FR);
  c.kb[w] = (int)(up(s.K, FK) / FK);
  c.planes[w] = (unsigned char*)m.take(plane_bytes(s.rows, s.K));
  c.ex[w] = (int*)m.take(sizeof(int) * s.rows);
  c.nr[w] = (float*)m.take(sizeof(float) * s.rows);
  c.part[w] = (double*)m.take(sizeof(double) * s.rows * c.nch[w]);
}

// balancing scales from operand w, for both; ks: balance_bytes(rows, K)
inline int balance_chunks(int64_t rows) { return (int)((rows + BAL_ROWS - 1) / BAL_ROWS); }
inline size_t balance_bytes(int64_t rows, int64_t k) {
  return ws_round(sizeof(double) * k * (2 + balance_chunks(rows)));
}
gevp_status balance(gevp_ctx* c, ConvArgs& p, int w, double* ks) {
  const ModSrc& s = p.s[w];
  p.ks[w] = ks;
  p.ks[1 - w] = ks + s.K;
  const int ch = s.kfast ? balance_chunks(s.rows) : 1;
  const int64_t blocks = s.kfast ? (int64_t)((s.K + 63) / 64) * ch : (s.K + 15) / 16;
  hipLaunchKernelGGL(k_mod_balance, dim3((unsigned)blocks), dim3(1024), 0, c->stream, s, ks, ks + s.K,
                     ks + 2 * s.K, ch);
  if (ch > 1)
    hipLaunchKernelGGL(k_mod_balance_finish, dim3((unsigned)((s.K + 255) / 256)), dim3(256), 0, c->stream,
                       ks + 2 * s.K, s.K, ch, ks, ks + s.K);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

// two launches: row norms, then the conversion, of the operands with on[w]
gevp_status convert(gevp_ctx* c, ConvArgs p, bool on0, bool on1) {
  const bool on[2] = {on0, on1};
  for (int w = 0; w < 2; ++w) {
    const int64_t units = p.s[w].kfast ? ((int64_t)p.s[w].rows * p.nch[w] + 3) / 4
                                       : ((int64_t)(p.s[w].rows + 63) / 64) * p.nch[w];
    p.blk[w] = on[w] ? (int)units : 0;
  }
  hipLaunchKernelGGL(k_mod_norms, dim3((unsigned)(p.blk[0] + p.blk[1])), dim3(256), 0, c->stream, p);
  for (int w = 0; w < 2; ++w) p.blk[w] = on[w] ? (int)(((int64_t)p.rg[w] * p.kb[w] + 3) / 4) : 0;
  hipLaunchKernelGGL(k_mod_split, dim3((unsigned)(p.blk[0] + p.blk[1])), dim3(256), 0, c->stream, p);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}

ModSrc left_src(int op, const zd* A, int64_t lda, const zd* A2, int64_t m, int64_t m1, int64_t k, int tri) {
  return ModSrc{A, A2, lda, (int)m, (int)k, (int)(A2 ? m1 : m), op ? 1 : 0, op ? 1 : 0, tri};
}
ModSrc right_src(int op, const zd* B, int64_t ldb, int64_t n, int64_t k) {
  return ModSrc{B, nullptr, ldb, (int)n, (int)k, (int)n, op ? 0 : 1, op ? 1 : 0, 0};
}

// Output tile by a count of rounds: one 256-row work-group per compute unit at
// a time (LDS), two 128 x 128 ones; the smaller tiles move more bytes per
// product (per-round costs relative to a 256 x 256 tile).
int mod_tile(int64_t m, int64_t n, int cus) {
  auto rounds = [&](int64_t tm, int64_t tn, int64_t slots) {
    const int64_t t = ((m + tm - 1) / tm) * ((n + tn - 1) / tn) * NCH;
    return (double)((t + slots - 1) / slots);
  };
  const double c0 = rounds(256, 256, cus), c1 = 0.58 * rounds(256, 128, cus),
               c2 = 0.65 * rounds(128, 128, 2 * cus);
  if (c0 <= c1 && c0 <= c2) return 0;
  return c1 <= c2 ? 1 : 2;
}

template <int MI, int NJ>
gevp_status launch_tiles(gevp_ctx* c, ModGemmArgs q, int64_t m, int64_t n) {
  q.tiles_m = (int)((m + 32 * MI - 1) / (32 * MI));
  q.tiles_n = (int)((n + 64 * NJ - 1) / (64 * NJ));
  q.tiles = q.tiles_m * q.tiles_n;
  q.total = q.tiles * NCH;
  q.checks = (q.tiles + 7) / 8 * 8;
  hipLaunchKernelGGL((k_mod_gemm<MI, NJ>), dim3((unsigned)(q.checks + (q.total + 7) / 8 * 8)), dim3(512), 0,
                     c->stream, q);
  GEVP_HIP_TRY(hipGetLastError());
  return GEVP_OK;
}
}  // namespace

// Scratch of one product: both operands' planes, exponents and partial norms,
// the residues of the result, the flag.
size_t mod_gemm_bytes(int64_t m, int64_t n, int64_t k) {
  return conv_bytes(m, k) + conv_bytes(n, k) + ws_round(up(m, 16) * up(n, 16) * NCH) +
         balance_bytes(n, k) + 256;
}

// The route by estimated times.  Residues: 45 us for six launches and their
// gaps, the conversions (64 bytes per entry: read twice, 33 written; 16 more
// for the balancing), the result (residues written and read, the result read
// and written), the INT8 products of whole 128-wide tiles; FP64: the rate of
// the operand form at sizes where the two meet.  Measured residues / FP64, in
// ms: NN 8192 x 8192 x 384 2.39 / 2.68, 4096 x 4096 x 384 0.71 / 0.68, 2048 x
// 2048 x 512 0.234 / 0.225, 4096 x 474 x 1024 0.211 / 0.221, 948^3 0.116 / 0.116
// (CN 0.127 / 0.147), 2048 x 237 x 2048 0.132 / 0.129, 512^3 0.069 / 0.036; 8192
// x 128 x 8192 1.42 / 0.86 (the conversion of a large matrix for few columns);
// 8192 x 948 x 8192 2.8 / 6.7, 4096^3 2.4 / 6.7.
bool mod_gemm_pays(int opA, int opB, int64_t m, int64_t n, int64_t k, int lower, int upperA, bool prepared) {
  if (k < 192 || k > 65536 || m < 64 || n < 64) return false;
  const double md = (double)m, nd = (double)n, kd = (double)k;
  const double mp = (double)up(m, 128), np = (double)up(n, 128), kp = (double)up(k, FK);
  const double out = lower ? 0.5 : 1.0, prod = lower || upperA ? 0.5 : 1.0;
  const double conv = kd * (prepared ? 64.0 * nd : 64.0 * md + 80.0 * nd) / 4.2e12;
  const double t_mod = 45e-6 + conv + out * 96.0 * md * nd / 3.9e12 + prod * 64.0 * mp * np * kp / 2.2e15;
  const double nn = md * nd < 2048.0 * 64 * 64 ? 66e12 : 72e12;  // few rounds of 64 x 64 tiles, or many
  const double rate = opA == 0 && opB == 0 ? nn : opB == 0 ? 50e12 : 57e12;
  return t_mod < 0.95 * prod * 8.0 * md * nd * kd / rate;
}

size_t mod_prepared_bytes(int64_t m, int64_t k) {
  return conv_bytes(m, k) + balance_bytes(m, k) + 256;
}

gevp_status mod_prepare(gevp_ctx* c, int64_t m, int64_t k, int opA, const zd* A, int64_t lda, void* buf,
                        ModPrepared* out) {
  Carver w{(char*)buf};
  ConvArgs p{};
  set_operand(p, 0, left_src(opA, A, lda, nullptr, m, m, k, 0), w);
  p.flag = (int*)w.take(256);
  double* ks = (double*)w.take(balance_bytes(m, k));
  GEVP_TRY(balance(c, p, 0, ks));
  out->ks = p.ks[1];
  out->planes = p.planes[0];
  out->ex = p.ex[0];
  out->nr = p.nr[0];
  out->flag = p.flag;
  out->m = m;
  out->k = k;
  return convert(c, p, true, false);
}

gevp_status launch_mod_gemm(gevp_ctx* c, const ModGemmCall& g, void* scratch, const int** flag1,
                            const int** flag2) {
  Carver w{(char*)scratch};
  const ModPrepared* pa = g.prepared;
  ConvArgs p{};
  set_operand(p, 1, right_src(g.opB, g.B, g.ldb, g.n, g.k), w);
  if (!pa) set_operand(p, 0, left_src(g.opA, g.A, g.lda, g.A2, g.m, g.m1, g.k, g.upperA), w);
  unsigned* R = (unsigned*)w.take(up(g.m, 16) * up(g.n, 16) * NCH);
  p.flag = (int*)w.take(256);
  if (pa)
    p.ks[1] = pa->ks;
  else
    GEVP_TRY(balance(c, p, 1, (double*)w.take(balance_bytes(g.n, g.k))));
  GEVP_TRY(convert(c, p, !pa, true));
  ModGemmArgs q{};
  q.A = pa ? (const unsigned char*)pa->planes : p.planes[0];
  q.B = p.planes[1];
  q.R = R;
  q.rga = (int)((g.m + FR - 1) / FR);
  q.rgb = p.rg[1];
  q.kb = p.kb[1];
  q.lower = g.lower;
  q.tri = g.upperA;
  q.rb = q.rga;
  q.cb = q.rgb;
  q.small = g.k <= 1024;  // 1024 * 120^2 < 2^24
  q.nra = pa ? pa->nr : p.nr[0];
  q.nrb = p.nr[1];
  q.M = (int)g.m;
  q.N = (int)g.n;
  q.least = MIN_SIZES * (float)g.k * std::sqrt((float)g.parts);
  q.flag = p.flag;
  q.flag2 = pa ? pa->flag : nullptr;
  switch (mod_tile(g.m, g.n, gevp_device_cus(c->device))) {
    case 0: GEVP_TRY((launch_tiles<8, 4>(c, q, g.m, g.n))); break;
    case 1: GEVP_TRY((launch_tiles<8, 2>(c, q, g.m, g.n))); break;
    default: GEVP_TRY((launch_tiles<4, 2>(c, q, g.m, g.n)));
  }
  CrtArgs r{};
  r.R = R;
  r.exa = pa ? pa->ex : p.ex[0];
  r.exb = p.ex[1];
  r.flag = p.flag;
  r.flag2 = pa ? pa->flag : nullptr;
  r.M = (int)g.m;
  r.N = (int)g.n;
  r.rb = q.rb;
  r.cb = q.cb;
  r.lower = g.lower;
  r.Cm = g.Cm;
  r.ldc = g.ldc;
  r.E = g.E;
  r.lde = g.lde;
  r.gcol = g.gcol;
  r.D = g.D;
  r.ldd = g.ldd;
  r.alpha = g.alpha;
  r.beta = g.beta;
  r.gamma = g.gamma;
  r.coef = g.coef;
  const int64_t blks = (int64_t)q.rb * q.cb;
  hipLaunchKernelGGL(k_mod_crt, dim3((unsigned)((blks + 3) / 4)), dim3(256), 0, c->stream, r);
  GEVP_HIP_TRY(hipGetLastError());
  *flag1 = r.flag;
  *flag2 = r.flag2;
  return GEVP_OK;
}
