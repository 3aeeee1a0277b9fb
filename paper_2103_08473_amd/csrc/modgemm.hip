// FP64 complex products on the INT8 matrix cores.
//
// The FP64 matrix rate of gfx950 (78.6 TFLOP/s) bounds the FP64 GETT, which already runs at
// 0.8 to 0.95 of it on large products.  The INT8 rate is about 64 times higher, so a large
// product is formed exactly on integers instead, in a residue number system:
//   * every operand row a_m is scaled by a power of two to the 2-norm range (2^(S-1), 2^S]
//     and rounded to integers (S = 55 or 58 bits, more than the 53 of a double);
//   * modulo a prime (or product of primes) p = 1 mod 4 there is j with j^2 = -1, and a
//     complex integer x + iy is held as the pair (x + jy, x - jy) mod p: in this form a
//     complex product is two real products (the quadratic residue number system of
//     Leung and of Jenkins and Krogmeier), so 15 or 16 moduli give 30 or 32 INT8 planes;
//   * per plane one INT8 GEMM with INT32 accumulation (exact: |sum| <= K (p/2)^2 < 2^31 for
//     K <= kMaxK), reduced mod p to one byte per output;
//   * the Chinese remainder theorem gives the exact integer product back: by the
//     Cauchy-Schwarz inequality |re|, |im| <= |a_m| |b_n| <= 2^(2S) < M / 2, M the product of
//     the moduli, so value / M is the fractional part of sum_i r_i w_i / p_i, summed as an
//     exact high part (multiples of 2^-42) and an FP64 remainder.
// The only rounding is that of the scaled operands to integers (relative to the row's norm)
// and of the result to FP64; sums over k are exact, so results do not depend on tiling.
// A row with a non-finite element gives NaN outputs.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "common.h"

namespace exacc {
namespace {

constexpr int kNP = 16;           // most moduli; see moduli_for
constexpr int kPlanes = 2 * kNP;
constexpr int kMaxK = 131072;     // K (p / 2)^2 < 2^31 with p <= 241
constexpr int kShortK = 1152;     // K (p / 2)^2 + 128 < 2^24
constexpr int kNaN = 0x40000000;  // exponent of a row that holds a non-finite element
constexpr int kZero = 4096;       // of a row of zeros: above that of any other finite row

typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i16v __attribute__((ext_vector_type(16)));
typedef double d2v __attribute__((ext_vector_type(2)));
typedef unsigned __int128 u128;

// Pairwise coprime products of primes = 1 mod 4 (so that -1 has a square root), largest first.
constexpr int kMods[16] = {241, 233, 229, 221, 205, 197, 193, 181, 173, 157, 149, 137, 113, 109, 101, 97};

struct ModTab {
  int np;  // moduli in use
  int S;   // operand bits: 2^(2 S) (1 + 2^-40) < M / 2
  int p[kNP];
  float pf[kNP], ipf[kNP];  // p, 1 / p
  int w[kNP][4];  // 256^d mod p (d = 0..7, one byte each), then j 256^d mod p
  double hr[kNP], lr[kNP], hi[kNP], li[kNP];  // CRT weights of re and im, high and low parts
  double mhi, mlo;                            // M
};

constexpr int inv_mod(int a, int p) {
  for (int x = 1; x < p; ++x)
    if ((int)((int64_t)a * x % p) == 1) return x;
  return 0;
}

ModTab make_tab(int np) {
  ModTab t{};
  t.np = np;
  u128 M = 1;
  for (int i = 0; i < np; ++i) M *= (u128)kMods[i];
  u128 top = 1;
  for (t.S = 0; top * 4 < M / 2 - M / 64; ++t.S) top *= 4;  // 3% left for the rounding of operands
  for (int i = 0; i < np; ++i) {
    const int p = kMods[i];
    int j = 1;
    while ((j * j + 1) % p) ++j;
    if (2 * j > p) j = p - j;
    t.p[i] = p;
    t.pf[i] = (float)p;
    t.ipf[i] = 1.0f / (float)p;
    int w = 1;
    for (int d = 0; d < 8; ++d, w = w * 256 % p) {
      auto put = [&](int word, int x) {
        if (2 * x > p) x -= p;
        t.w[i][word] |= (int)((unsigned)(x & 255) << (8 * (d & 3)));
      };
      put(d / 4, w);
      put(2 + d / 4, w * j % p);
    }
    const int mi = inv_mod((int)((M / (u128)p) % (u128)p), p);
    // re = (u + v) / 2 and im = (u - v) / (2 j), times the CRT factor of p, in (-p/2, p/2)
    int cr = (int)((int64_t)mi * inv_mod(2, p) % p), ci = (int)((int64_t)cr * inv_mod(j, p) % p);
    if (2 * cr > p) cr -= p;
    if (2 * ci > p) ci -= p;
    auto parts = [&](int c, double& hpart, double& lpart) {
      const int64_t num = (int64_t)c << 42;
      const int64_t h = (num + (num < 0 ? -p / 2 : p / 2)) / p;
      hpart = (double)h * 0x1p-42;
      lpart = (double)(num - h * p) / (double)p * 0x1p-42;
    };
    parts(cr, t.hr[i], t.lr[i]);
    parts(ci, t.hi[i], t.li[i]);
  }
  t.mhi = (double)M;
  const u128 mh = (u128)t.mhi;
  t.mlo = mh > M ? -(double)(mh - M) : (double)(M - mh);
  return t;
}

// 15 moduli (S = 55) or 16 (S = 58).  The operands' rounding grows with sqrt(K) like the FP64
// GETT's sums do, and 15 moduli stay below those (relative rms error of re / im against
// 80-bit sums, FP64 GETT | 15 moduli: K 504 7.0e-16 / 1.2e-15 | 5.4e-16, 1131 6.4e-16 / 1.1e-15 |
// 7.2e-16, 4032 2.1e-15 / 3.8e-15 | 1.5e-15, 8000 1.7e-15 / 3.0e-15 | 1.5e-15) but where the
// FP64 GETT splits a long K into short chains (600 x 700 x 40000 1.7e-15 / 2.9e-15 | 5.9e-15):
// there 16 are taken (7.2e-16).
const ModTab& tab(int np) {
  static const ModTab t15 = make_tab(15), t16 = make_tab(16);
  return np == 15 ? t15 : t16;
}
int moduli_for(int64_t M, int64_t N, int64_t K) {
  const bool split = ((M + 63) / 64) * ((N + 63) / 64) < 1024;
  return K <= 8192 || !split ? 15 : 16;
}

__device__ __forceinline__ int64_t cmap(int x, int in, int64_t so, int64_t si) {
  const int q = x / in;
  return (int64_t)q * so + (int64_t)(x - q * in) * si;
}

// One operand as rows x K of complex FP64 values with composite row and k maps.
struct Src {
  const double* p;
  int row0, rows, K;  // rows [row0, rows) of the operand
  int r_in, k_in;
  int64_t r_so, r_si, k_so, k_si;
  int r_valid;  // if not 0: rows whose inner index is r_valid or more are padding (zero)
  int kfast;  // consecutive k are the nearer neighbours in memory
  int conj;
  // planes[row / 32][k / 64][z][(k / 32) % 2][lane][16]: lane l holds row l % 32 and
  // k 16 (l / 32) .. + 15 of its 32 x 32 block, the fragment order of the 32x32x32 INT8 MFMA;
  // zero past rows and K.  All planes of 32 rows x 64 k are together, so that splitting writes
  // whole 64 KiB runs (a plane-major order: 2.3 TB/s at 12363^2, this one: see mod_split_kernel)
  signed char* planes;
  int* exps;        // power of two each row was scaled by
  int rb, kb;       // 32-row and 32-k blocks (kb even)
};

// Scale exponents: per row the largest |component| and the sum of squares (fixed order).
// kfast: tpr threads per row; else 32 rows x 32 k phases per workgroup.  Bound by reading
// the operand once.
__global__ __launch_bounds__(1024) void mod_norm_kernel(Src a, int blocks_a, Src b, int tpr_a, int tpr_b, int S) {
  const bool first = (int)blockIdx.x < blocks_a;
  const Src s = first ? a : b;
  const int blk = first ? blockIdx.x : blockIdx.x - blocks_a;
  const int tid = threadIdx.x;
  __shared__ double ssum[1024], smax[1024];
  int row, k0, kstep, stride, width;
  if (s.kfast) {
    const int tpr = first ? tpr_a : tpr_b;
    row = s.row0 + blk * (1024 / tpr) + tid / tpr;
    k0 = tid % tpr;
    kstep = width = tpr;
    stride = 1;
  } else {
    row = s.row0 + blk * 32 + (tid & 31);
    k0 = tid >> 5;
    kstep = width = 32;
    stride = 32;
  }
  double sum = 0.0, mx = 0.0;
  if (row < s.rows && (s.r_valid == 0 || row % s.r_in < s.r_valid)) {
    const double* p = s.p + 2 * cmap(row, s.r_in, s.r_so, s.r_si);
    if (s.k_in == s.K) {
#pragma unroll 4
      for (int k = k0; k < s.K; k += kstep) {
        const d2v x = *reinterpret_cast<const d2v*>(p + 2 * (int64_t)k * s.k_si);
        sum += x.x * x.x + x.y * x.y;
        mx = fmax(mx, fmax(fabs(x.x), fabs(x.y)));
      }
    } else {
#pragma unroll 4
      for (int k = k0; k < s.K; k += kstep) {
        const d2v x = *reinterpret_cast<const d2v*>(p + 2 * cmap(k, s.k_in, s.k_so, s.k_si));
        sum += x.x * x.x + x.y * x.y;
        mx = fmax(mx, fmax(fabs(x.x), fabs(x.y)));
      }
    }
  }
  ssum[tid] = sum;
  smax[tid] = mx;
  __syncthreads();
  for (int w = width / 2; w > 0; w >>= 1) {
    if (k0 < w) {
      ssum[tid] += ssum[tid + w * stride];
      smax[tid] = fmax(smax[tid], smax[tid + w * stride]);
    }
    __syncthreads();
  }
  if (k0 == 0 && row < s.rows) {
    sum = ssum[tid];
    mx = smax[tid];
    int e = kZero;
    if (sum != sum || mx > 1.7976931348623157e308) {
      e = kNaN;
    } else if (mx > 0.0) {
      int ex;
      if (sum > 1e-280 && sum < 1e300) {  // norm < 2^(ex / 2)
        (void)frexp(sum, &ex);
        ex = (ex + 1) >> 1;
      } else {  // squares out of range: norm <= max sqrt(2 K)
        (void)frexp(mx, &ex);
        ex += (33 - __clz(2 * s.K)) >> 1;
      }
      e = S - ex;
    }
    s.exps[row] = e;
  }
}

// Residue planes of 32 rows x 64 k per workgroup: the scaled, rounded values are staged in
// LDS as 8 balanced base-256 digits (re, im), then each wave forms every second modulus of one
// 32 x 32 block, 16 k per lane: x mod p is a dot product of the digits with 256^d mod p (two
// 4-byte dot instructions) and one rounding step, 16 instructions per element and modulus
// against 16 bytes read and 4 written.
__global__ __launch_bounds__(256) void mod_split_kernel(Src a, int blocks_a, Src b, ModTab t) {
  const bool first = (int)blockIdx.x < blocks_a;
  const Src s = first ? a : b;
  const int blk = first ? blockIdx.x : blockIdx.x - blocks_a;
  const int kg = s.kb / 2;
  const int rblk = blk / kg, kgrp = blk - rblk * kg;
  const int tid = threadIdx.x;
  __shared__ i4v sv[32][65];
  // all loads first (rows and k past the end are clamped and zeroed below)
  d2v xs[8];
  int es[8];
  const int r0 = s.kfast ? tid >> 6 : tid & 31, kk0 = s.kfast ? tid & 63 : tid >> 5;
  const int rstep = s.kfast ? 4 : 0, kstep = s.kfast ? 0 : 8;
  const int rowb = s.row0 + rblk * 32;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    int row = min(rowb + r0 + rstep * q, s.rows - 1);
    if (s.r_valid) {
      const int in = row % s.r_in;
      row -= max(0, in - s.r_valid + 1);
    }
    const int k = min(kgrp * 64 + kk0 + kstep * q, s.K - 1);
    const int64_t ro = s.r_in < s.rows ? cmap(row, s.r_in, s.r_so, s.r_si) : row * s.r_si;
    const int64_t ko = s.k_in < s.K ? cmap(k, s.k_in, s.k_so, s.k_si) : k * s.k_si;
    es[q] = s.exps[row];
    xs[q] = *reinterpret_cast<const d2v*>(s.p + 2 * (ro + ko));
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int r = r0 + rstep * q, kk = kk0 + kstep * q;
    d2v x = {0.0, 0.0};
    const bool pad = s.r_valid && (rowb + r) % s.r_in >= s.r_valid;
    if (rowb + r < s.rows && kgrp * 64 + kk < s.K && es[q] != kNaN && !pad) {
      x.x = rint(ldexp(xs[q].x, es[q]));
      x.y = rint(ldexp(s.conj ? -xs[q].y : xs[q].y, es[q]));
    }
    // digits: the bytes of x + 0x80..80, each less 128 (flipping the top bit does that)
    constexpr uint64_t kBias = 0x8080808080808080ull;
    const uint64_t re = ((uint64_t)(int64_t)x.x + kBias) ^ kBias, im = ((uint64_t)(int64_t)x.y + kBias) ^ kBias;
    sv[r][kk] = i4v{(int)re, (int)(re >> 32), (int)im, (int)(im >> 32)};
  }
  __syncthreads();
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kblk = w & 1, half = w >> 1;
  i4v x[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) x[q] = sv[lane & 31][kblk * 32 + (lane >> 5) * 16 + q];
  signed char* out = s.planes + (int64_t)blk * (kPlanes * 2048) + kblk * 1024 + lane * 16;
  for (int i = half; i < t.np; i += 2) {
    const float pf = t.pf[i], ipf = t.ipf[i], off = -128.0f * ipf;
    const int w0 = t.w[i][0], w1 = t.w[i][1], j0 = t.w[i][2], j1 = t.w[i][3];
    i4v u, v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      unsigned ub = 0, vb = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const i4v y = x[4 * q + r];
        // below 8 128 120 each in magnitude, so the sums are exact in FP32; 128 makes the
        // rounded residues unsigned bytes
        const int re = __builtin_amdgcn_sdot4(y.y, w1, __builtin_amdgcn_sdot4(y.x, w0, 128, false), false);
        const int im = __builtin_amdgcn_sdot4(y.w, j1, __builtin_amdgcn_sdot4(y.z, j0, 0, false), false);
        const float tu = (float)(re + im), tv = (float)(re - im);
        const float ru = fmaf(-rintf(fmaf(tu, ipf, off)), pf, tu);
        const float rv = fmaf(-rintf(fmaf(tv, ipf, off)), pf, tv);
        ub = __builtin_amdgcn_cvt_pk_u8_f32(ru, r, ub);
        vb = __builtin_amdgcn_cvt_pk_u8_f32(rv, r, vb);
      }
      u[q] = (int)(ub ^ 0x80808080u);
      v[q] = (int)(vb ^ 0x80808080u);
    }
    *reinterpret_cast<i4v*>(out + (2 * i) * 2048) = u;
    *reinterpret_cast<i4v*>(out + (2 * i + 1) * 2048) = v;
  }
}

// Workgroup order: each XCD (own L2) takes a contiguous run of logical ids, which walk
// groups of 4 tiles along m by all of n.
__device__ __forceinline__ void tile_of(int id, int n, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int per = (n + 7) / 8, tall = n % 8 == 0 ? 8 : n % 8;
  const int x = id % 8, l = id / 8;
  const int t = x < tall ? x * per + l : tall * per + (x - tall) * (per - 1) + l;
  const int gsz = 4 * tiles_n, g = t / gsz, gm = min(4, tiles_m - g * 4), r = t - g * gsz;
  tm = g * 4 + r % gm;
  tn = r / gm;
}

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;

struct PlaneGemm {
  const signed char *A, *B;
  signed char* C;              // [mblk][nblk][z][lane][q][r]: row 8 q + 4 (lane / 32) + r, column lane % 32
  int mb, nb, kb;              // kb even
  int a_in, a_outer;           // A block of m-block x: (x / a_in) * a_outer + x % a_in
  int b_in, b_outer;           // likewise B
  int tiles_m, tiles_n;
  int planes;                  // 2 np of the kPlanes that the layouts have room for
  int p[kNP];
  // SEG kernels: k in three segments of kb / 3 blocks, segment q of product y of a batch at
  // 16-byte units a_seg[q] + y a_bat[q] of A (B likewise), C of product y c_bat bytes further
  int batch;
  int64_t a_seg[3], b_seg[3], a_bat[3], b_bat[3], c_bat;
};

// C[z] = A[z] B[z]^T mod p: WM x WN waves of TM x TN 32 x 32 blocks, stages of 64 k in three
// LDS buffers filled by direct global-to-LDS loads, two stages ahead.  Operands lie in
// fragment order, so a block is one contiguous 1 KiB copy and every LDS read is
// conflict-free.  The grid is what the chip holds; a workgroup walks tiles grid apart and
// loads the next tile's first stages before it reduces and stores this one's outputs.
// Bound by the power the INT8 matrix cores draw: 4032^3 x 32 planes 2380 TOP/s, the same
// launch on zeros and ones about 3000; one tile per workgroup 2250 there and 1426 instead of
// 1895 at 1268 x 25000 x 951, where filling the pipeline is a larger part.
template <int WM, int WN, int TM, int TN, int OCC, bool LONG, bool SEG>
__global__ __launch_bounds__(64 * WM * WN, OCC) void mod_gemm_kernel(PlaneGemm g) {
  constexpr int KB = 2, S = 3;
  constexpr int T = 64 * WM * WN, RA = WM * TM, RB = WN * TN;
  constexpr int NA = RA * KB * 64 / T, NB = RB * KB * 64 / T;
  static_assert(NA * T == RA * KB * 64 && NB * T == RB * KB * 64, "whole copies per thread");
  __shared__ i4v sm[S][(RA + RB) * KB * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w % WM, wn = w / WM;
  // a batch's products are further tiles along n, so that what they share of A is read together
  const int tiles_n = SEG ? g.tiles_n * g.batch : g.tiles_n;
  const int tiles = g.tiles_m * tiles_n, total = tiles * g.planes;
  const int nk = g.kb / KB, nseg = SEG ? nk / 3 : nk;
  const int64_t rs = (int64_t)nseg * kPlanes * 128;  // 16-byte units per row block
  const i4v* pa[NA];
  const i4v* pb[NB];
  int m0, n0, z, bat = 0;
  int64_t sa[3] = {0, 0, 0}, sb[3] = {0, 0, 0};
  // blocks past mb (nb) are clamped: they feed only outputs that are not stored
  auto start = [&](int job) {
    z = job / tiles;
    int tm, tn;
    tile_of(job - z * tiles, tiles, g.tiles_m, tiles_n, tm, tn);
    if (SEG) {
      bat = tn / g.tiles_n;
      tn -= bat * g.tiles_n;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        sa[q] = g.a_seg[q] + bat * g.a_bat[q];
        sb[q] = g.b_seg[q] + bat * g.b_bat[q];
      }
    }
    m0 = tm * RA;
    n0 = tn * RB;
    const i4v* A = reinterpret_cast<const i4v*>(g.A + z * 2048);
    const i4v* B = reinterpret_cast<const i4v*>(g.B + z * 2048);
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int e = tid + T * q, m = min(m0 + e / (KB * 64), g.mb - 1), o = m / g.a_in;
      pa[q] = A + ((int64_t)o * g.a_outer + (m - o * g.a_in)) * rs + e % (KB * 64);
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int e = tid + T * q, n = min(n0 + e / (KB * 64), g.nb - 1), o = n / g.b_in;
      pb[q] = B + ((int64_t)o * g.b_outer + (n - o * g.b_in)) * rs + e % (KB * 64);
    }
  };
  auto load = [&](int kt, int buf) {
    int64_t ka = (int64_t)kt * (kPlanes * 128), kb = ka;
    if (SEG) {
      const int sg = kt >= 2 * nseg ? 2 : kt >= nseg ? 1 : 0;
      ka -= (int64_t)sg * nseg * (kPlanes * 128);
      kb = ka + (sg == 2 ? sb[2] : sg == 1 ? sb[1] : sb[0]);
      ka += sg == 2 ? sa[2] : sg == 1 ? sa[1] : sa[0];
    }
#pragma unroll
    for (int q = 0; q < NA; ++q)
      __builtin_amdgcn_global_load_lds((global_void*)(pa[q] + ka), (lds_void*)&sm[buf][w * 64 + T * q], 16, 0, 0);
#pragma unroll
    for (int q = 0; q < NB; ++q)
      __builtin_amdgcn_global_load_lds((global_void*)(pb[q] + kb),
                                       (lds_void*)&sm[buf][RA * KB * 64 + w * 64 + T * q], 16, 0, 0);
  };
  int job = blockIdx.x;
  if (job >= total) return;
  start(job);
#pragma unroll
  for (int s = 0; s < S - 1; ++s) load(min(s, nk - 1), s);
  constexpr int kBias = LONG ? 0 : 128;  // see the reduction below
  int cur = 0;
  while (true) {
    const int cm0 = m0, cn0 = n0, cz = z, cbat = bat, next = job + (int)gridDim.x;
    i16v acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = kBias;
    for (int kt = 0; kt < nk; ++kt) {
      // this wave's loads of stage kt have landed when at most those of the next S - 2 stages
      // are outstanding (stores only make the wait longer); behind the barrier so have all
      // waves', and all have read stage kt - 1, whose buffer is loaded next
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NA + NB) * (S - 2)) : "memory");
      const i4v* sa = &sm[cur][wm * TM * KB * 64 + lane];
      const i4v* sb = &sm[cur][RA * KB * 64 + wn * TN * KB * 64 + lane];
      i4v a[KB][TM], b[KB][TN];
#pragma unroll
      for (int s = 0; s < KB; ++s) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a[s][i] = sa[(i * KB + s) * 64];
#pragma unroll
        for (int j = 0; j < TN; ++j) b[s][j] = sb[(j * KB + s) * 64];
      }
      // past the last tile the last stage is loaded again, into a buffer that is not read any
      // more, so that the count of loads in flight is the same in every step
      int kn = kt + S - 1;
      if (kn >= nk) {
        if (next < total) {
          kn -= nk;
          if (kn == 0) start(next);
          kn = min(kn, nk - 1);
        } else {
          kn = nk - 1;
        }
      }
      load(kn, cur == 0 ? S - 1 : cur - 1);
#pragma unroll
      for (int s = 0; s < KB; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[s][i], b[s][j], acc[i][j], 0, 0, 0);
      cur = cur + 1 == S ? 0 : cur + 1;
    }
    // Residues in [-p/2, p/2], kept 128 higher as unsigned bytes.  Up to kShortK the sums are
    // exact in FP32 and one rounded quotient suffices; beyond, a first step on the integers
    // (quotients below 2^23, off by at most 2) brings them there.
    const int p = g.p[cz >> 1];
    const float pf = (float)p, ip = 1.0f / pf, off = -128.0f * ip;
    i4v* C = reinterpret_cast<i4v*>(g.C + (SEG ? cbat * g.c_bat : 0) + cz * 1024);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int bm = cm0 + wm * TM + i, bn = cn0 + wn * TN + j;
        if (bm >= g.mb || bn >= g.nb) continue;
        i4v o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          unsigned pk = 0;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            int x = acc[i][j][4 * q + r];
            if (LONG) x = 128 + x - __mul24((int)rintf((float)x * ip), p);
            const float y = (float)x;
            pk = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(-rintf(fmaf(y, ip, off)), pf, y), r, pk);
          }
          o[q] = (int)(pk ^ 0x80808080u);
        }
        C[((int64_t)bm * g.nb + bn) * (kPlanes * 64) + lane] = o;
      }
    job = next;
    if (job >= total) break;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the repeated loads, before LDS is given back
}

// (re, im) of the four outputs in one dword of every plane, as the integer product over M.
struct Frac4 {
  double re[4], im[4];
};
__device__ __forceinline__ Frac4 crt4(const int* c, const ModTab& t) {
  double hr[4] = {0, 0, 0, 0}, lr[4] = {0, 0, 0, 0}, hi[4] = {0, 0, 0, 0}, li[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < kNP; ++i) {
    if (i >= 15 && i >= t.np) break;
    const int u = c[(2 * i) * 256], v = c[(2 * i + 1) * 256];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ur = (int)((unsigned)u << (24 - 8 * r)) >> 24, vr = (int)((unsigned)v << (24 - 8 * r)) >> 24;
      const double a = (double)(ur + vr), b = (double)(ur - vr);
      hr[r] = fma(a, t.hr[i], hr[r]);  // exact: multiples of 2^-42 below 2^11
      lr[r] = fma(a, t.lr[i], lr[r]);
      hi[r] = fma(b, t.hi[i], hi[r]);
      li[r] = fma(b, t.li[i], li[r]);
    }
  }
  Frac4 f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double x = (hr[r] - rint(hr[r])) + lr[r], y = (hi[r] - rint(hi[r])) + li[r];
    // the fractional part can straddle +-1/2 only above the Cauchy-Schwarz bound
    f.re[r] = fma(x, t.mhi, x * t.mlo);
    f.im[r] = fma(y, t.mhi, y * t.mlo);
  }
  return f;
}

// C(m, n) = alpha * product (+ C) for m0 <= m < m0 + 32 mb, n likewise; one dword (4 rows of
// one column) per lane.  Grid y: products of a batch, cp_bat dwords and c_bat elements apart.
// Bound by reading 2 kNP bytes and writing 16 per output.
__global__ __launch_bounds__(256) void mod_crt_kernel(const int* Cp, int mb, int nb, int m0, int n0,
                                                      const int* ea, const int* eb, Gett<double> g, int64_t cp_bat,
                                                      int64_t c_bat, ModTab t) {
  Cp += blockIdx.y * cp_bat;
  g.C += 2 * (int64_t)blockIdx.y * c_bat;
  const int64_t tot = (int64_t)mb * nb * 4;
  const int lane = threadIdx.x & 63;
  for (int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); u < tot; u += (int64_t)gridDim.x * 4) {
    // dword 64 q + lane of the tile: column and first of four rows
    const int q = (int)(u & 3), col = 16 * (q & 1) + (lane >> 2), row = 8 * (lane & 3) + 4 * (q >> 1);
    const int64_t tile = u >> 2;
    const int bm = (int)(tile / nb), bn = (int)(tile - (int64_t)bm * nb);
    const int n = n0 + 32 * bn + col, mr = m0 + 32 * bm + row;
    const Frac4 f = crt4(Cp + tile * (kPlanes * 256) + q * 64 + lane, t);
    if (n >= g.N) continue;
    const int en = eb[n];
    const int64_t co = cmap(n, g.n_in, g.c_no, g.c_ni);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mr + r;
      if (m >= g.M) continue;
      const int em = ea[m];
      const bool bad = em == kNaN || en == kNaN;
      const double xr = bad ? __builtin_nan("") : ldexp(f.re[r], -(em + en));
      const double xi = bad ? __builtin_nan("") : ldexp(f.im[r], -(em + en));
      d2v* c = reinterpret_cast<d2v*>(g.C + 2 * (co + cmap(m, g.m_in, g.c_mo, g.c_mi)));
      d2v y = {g.alpha_re * xr - g.alpha_im * xi, g.alpha_re * xi + g.alpha_im * xr};
      if (g.accumulate) y += *c;
      *c = y;
    }
  }
}

// W[(a, b)][(c < d)] = T[a][c][b][d] - T[a][d][b][c] for the pairs of 32-blocks p <= q of c and d
// (grid x), b (y) and a (z) of one product of the residues of rows (a, c) and (b, d); T is
// reconstructed as in mod_crt_kernel, one half transposed through LDS, and never stored:
// 64 bytes read and 16 written per pair, against 96 for a stored T and a pass over it.
struct LadderTiles {
  const int* C;
  const int* exps;  // of row (a, c): a 32 vb + c
  int v, vb, wvb, blk0;  // blocks of c: blk0 .. vb - 1, wvb of them
  int a0;                // pairs c < d from a0 on, packed
  int a_first, b_first, nbn;
  int64_t row0;          // packed pair index of W's first row
  double* W;
  int64_t ldw;
};
__global__ __launch_bounds__(256) void mod_ladder_antisym_kernel(LadderTiles g, ModTab t) {
  const int a = g.a_first + blockIdx.z, b = g.b_first + blockIdx.y;
  if (b <= a) return;
  int p = 0, q = blockIdx.x;
  while (q >= g.wvb - p) q -= g.wvb - p++;
  q += p;
  __shared__ d2v sy[32][33];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = 16 * (w & 1) + (lane >> 2), row = 8 * (lane & 3) + 4 * (w >> 1);
  const int64_t ld = (int64_t)g.nbn * g.wvb;
  const int bp = 32 * (g.blk0 + p), bq = 32 * (g.blk0 + q);
  auto value = [&](int rb, int cb, d2v* y) {  // T[a][32 rb + row + r][b][32 cb + col]
    const int64_t tile =
        ((int64_t)blockIdx.z * g.wvb + rb) * ld + (int64_t)blockIdx.y * g.wvb + cb;
    const Frac4 f = crt4(g.C + tile * (kPlanes * 256) + w * 64 + lane, t);
    const int r0 = 32 * (g.blk0 + rb) + row, c0 = 32 * (g.blk0 + cb) + col;
    const int en = c0 < g.v ? g.exps[b * 32 * g.vb + c0] : 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int em = r0 + r < g.v ? g.exps[a * 32 * g.vb + r0 + r] : 0;
      const bool bad = em == kNaN || en == kNaN;
      y[r].x = bad ? __builtin_nan("") : ldexp(f.re[r], -(em + en));
      y[r].y = bad ? __builtin_nan("") : ldexp(f.im[r], -(em + en));
    }
  };
  d2v x[4], y[4];
  value(p, q, x);
  if (p == q) {
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = x[r];
  } else {
    value(q, p, y);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) sy[col][row + r] = y[r];
  __syncthreads();
  const int d = bq + col, wv = g.v - g.a0;
  const int64_t xrow = (int64_t)a * g.v - (int64_t)a * (a + 1) / 2 + b - a - 1 - g.row0;
  double* out = g.W + 2 * xrow * g.ldw;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = bp + row + r;
    if (c < g.a0 || c >= d || d >= g.v) continue;
    const int cc = c - g.a0;
    const int64_t pos = (int64_t)cc * wv - (int64_t)cc * (cc + 1) / 2 + d - c - 1;
    *reinterpret_cast<d2v*>(out + 2 * pos) = x[r] - sy[row + r][col];
  }
}

// Rows whose products are summed get one scale: exps[g n + r], g < groups, becomes the least
// of them less 1, room for three rows in one Cauchy-Schwarz bound (sqrt(3) < 2).  One thread
// per r; nothing beside what it prepares (groups n dwords).
__global__ __launch_bounds__(256) void mod_joint_exps_kernel(int* exps, int groups, int n) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= n) return;
  int e = kZero;
  bool bad = false;
#pragma unroll 8
  for (int g = 0; g < groups; ++g) {
    const int x = exps[(int64_t)g * n + r];
    bad |= x == kNaN;
    e = min(e, x);
  }
  e = bad ? kNaN : e - 1;
  for (int g = 0; g < groups; ++g) exps[(int64_t)g * n + r] = e;
}

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

int tpr_of(const Src& s) { return s.K >= 4096 ? 256 : 64; }
int norm_blocks(const Src& s) {
  return cdiv(std::min(s.rows - s.row0, 32 * s.rb), s.kfast ? 1024 / tpr_of(s) : 32);
}

// Scale and split one or two operands (b may have rows == 0).
void split_scaled(const Src& a, const Src& b, const ModTab& t, hipStream_t s) {
  const int sa = a.rb * (a.kb / 2), sb = b.rows ? b.rb * (b.kb / 2) : 0;
  hipLaunchKernelGGL(mod_split_kernel, dim3(sa + sb), dim3(256), 0, s, a, sa, b, t);
  HIPCHECK(hipGetLastError());
}
void split(const Src& a, const Src& b, const ModTab& t, hipStream_t s) {
  const int na = norm_blocks(a), nb = b.rows ? norm_blocks(b) : 0;
  hipLaunchKernelGGL(mod_norm_kernel, dim3(na + nb), dim3(1024), 0, s, a, na, b, tpr_of(a), tpr_of(b), t.S);
  HIPCHECK(hipGetLastError());
  split_scaled(a, b, t, s);
}

// RES: workgroups one CU holds (of 160 KiB LDS).  256 CUs.
template <int WM, int WN, int TM, int TN, int OCC, int RES, bool SEG = false>
void launch_planes(PlaneGemm g, hipStream_t s) {
  g.tiles_m = cdiv(g.mb, WM * TM);
  g.tiles_n = cdiv(g.nb, WN * TN);
  const int64_t jobs = (int64_t)g.tiles_m * g.tiles_n * g.planes * (SEG ? g.batch : 1);
  if (jobs > 0x7fffffffLL) raise(-1, "contraction too large for one launch");
  const dim3 grid((unsigned)std::min<int64_t>(jobs, 256 * RES)), block(64 * WM * WN);
  if (32 * g.kb <= kShortK)
    hipLaunchKernelGGL((mod_gemm_kernel<WM, WN, TM, TN, OCC, false, SEG>), grid, block, 0, s, g);
  else
    hipLaunchKernelGGL((mod_gemm_kernel<WM, WN, TM, TN, OCC, true, SEG>), grid, block, 0, s, g);
  HIPCHECK(hipGetLastError());
}

// Tile choice: the padded block count of each tile shape over its measured rate (TOP/s at
// full tiles, see mod_gemm_kernel), in whole rounds of the workgroups the chip holds.
void gemm_planes(PlaneGemm g, hipStream_t s) {
  if (g.kb < 4) raise(-1, "residue product: K too short for its pipeline");  // two stages at least
  for (int i = 0; i < kNP; ++i) g.p[i] = kMods[i];
  auto cost = [&](int ra, int rb, int resident, double rate) {
    const int64_t wgs = (int64_t)cdiv(g.mb, ra) * cdiv(g.nb, rb) * g.planes;
    const double rounds = wgs >= 8 * resident ? (double)wgs / resident : (double)((wgs + resident - 1) / resident);
    return rounds * resident * ra * rb / rate;
  };
  const double c0 = cost(8, 8, 256, 2200), c1 = cost(4, 8, 512, 1900), c2 = cost(8, 4, 512, 1940),
               c3 = cost(4, 4, 768, 1720);
  const double best = std::min(std::min(c0, c1), std::min(c2, c3));
  if (best == c0)
    launch_planes<2, 4, 4, 2, 1, 1>(g, s);
  else if (best == c1)
    launch_planes<2, 2, 2, 4, 2, 2>(g, s);
  else if (best == c2)
    launch_planes<2, 2, 4, 2, 2, 2>(g, s);
  else
    launch_planes<2, 2, 2, 2, 3, 3>(g, s);
}

thread_local char* t_ws = nullptr;
thread_local size_t t_ws_bytes = 0;

inline size_t up256(size_t b) { return (b + 255) / 256 * 256; }
inline int kblocks(int K) { return 2 * cdiv(K, 64); }

}  // namespace

// Estimated times (us).  FP64 GETT: 64 x 64 tiles at 62 TFLOP/s (55 to 72 reached).  Here: four
// launches, splitting 15 ps per element, reconstruction 15 ps per output, the plane products at
// 1.7 POP/s on 32 x 32 blocks.  Measured at the line (us, FP64 GETT / this): 900^3 138 / 107,
// 400 x 19800 x 600 687 / 540, 4032 x 576 x 504 176 / 155, 190 x 9730 x 9730 2266 / 2215; under
// it 640^3 59 / 66, 28224 x 168 x 504 391 / 440, 1131 x 1131 x 259 67 / 82.
bool mod_gemm_pays(int64_t M, int64_t N, int64_t K) {
  if (M < 128 || N < 128 || K < 128) return false;
  auto up = [](int64_t x, int64_t m) { return (double)((x + m - 1) / m * m); };
  const double t64 = 8.0 * up(M, 64) * up(N, 64) * (double)K / 62e6;
  const double tm = 25.0 + (double)(M + N) * K * 15e-6 + (double)M * N * 15e-6 +
                    2.0 * kPlanes * up(M, 32) * up(N, 32) * up(K, 64) / 1.7e9;
  return tm < 0.95 * t64;
}

int64_t mod_plane_bytes(int64_t rows, int64_t K) {
  return kPlanes * ((rows + 31) / 32) * ((K + 63) / 64) * 2048;
}
int64_t mod_out_bytes(int64_t M, int64_t N) { return kPlanes * ((M + 31) / 32) * ((N + 31) / 32) * 1024; }

void set_mod_workspace(void* p, size_t bytes) {
  t_ws = static_cast<char*>(p);
  t_ws_bytes = p ? bytes : 0;
}

bool mod_gemm(const Gett<double>& g0, hipStream_t s) {
  Gett<double> g = g0;
  if (!t_ws || g.K < 1 || !mod_gemm_pays(g.M, g.N, g.K)) return false;
  if (g.nbatch > 1) {
    for (int q = 0; q < g0.nbatch; ++q) {
      Gett<double> h = g0;
      h.nbatch = 1;
      h.A = g0.A + 2 * (int64_t)q * g0.a_b;
      h.B = g0.B + 2 * (int64_t)q * g0.b_b;
      h.C = g0.C + 2 * (int64_t)q * g0.c_b;
      if (!mod_gemm(h, s)) {  // the first refuses or none does: sizes and workspace are the same
        if (q > 0) raise(-1, "residue products of one batch took different routes");
        return false;
      }
    }
    return true;
  }
  // columns of C (n) are the nearer neighbours in memory
  if (g.c_ni != 1 && g.c_mi == 1) {
    std::swap(g.A, g.B);
    std::swap(g.M, g.N);
    std::swap(g.m_in, g.n_in);
    std::swap(g.a_mo, g.b_no);
    std::swap(g.a_mi, g.b_ni);
    std::swap(g.a_ko, g.b_ko);
    std::swap(g.a_ki, g.b_ki);
    std::swap(g.c_mo, g.c_no);
    std::swap(g.c_mi, g.c_ni);
    std::swap(g.conj_a, g.conj_b);
  }
  const int mb = cdiv(g.M, 32), nb = cdiv(g.N, 32);
  const int kc_max = std::min(g.K, kMaxK);
  const size_t rbytes = (size_t)kPlanes * kblocks(kc_max) * 1024, tbytes = (size_t)kPlanes * 1024;
  const size_t ebytes = up256((size_t)g.M * 4) + up256((size_t)g.N * 4);
  // A and B blocks resident at a time (ma, nbr) and C blocks per product (mc x nc): C is kept
  // to what the last-level cache holds, since the reconstruction reads it right away
  constexpr size_t kC = (size_t)512 << 20;
  if (ebytes + 64 * tbytes > t_ws_bytes) return false;
  const size_t room = t_ws_bytes - ebytes;
  size_t cbytes = std::min(std::min(kC, room / 4), (size_t)mb * nb * tbytes);
  if (cbytes < (size_t)std::min(mb, 8) * std::min(nb, 8) * tbytes) return false;
  const size_t rows_room = (room - cbytes) / rbytes;  // row blocks of A and B together
  int ma = mb, nr = nb;
  if ((size_t)mb + nb > rows_room) {
    if (std::min(mb, nb) * 2 <= (int64_t)rows_room) {  // the smaller operand whole
      if (mb <= nb)
        nr = (int)(rows_room - mb);
      else
        ma = (int)(rows_room - nb);
    } else {
      ma = nr = (int)(rows_room / 2);
    }
    if (ma < std::min(mb, 16) || nr < std::min(nb, 16)) return false;
    if (ma < mb) ma = ma / 8 * 8;
    if (nr < nb) nr = nr / 8 * 8;
  }
  const int cb = (int)(cbytes / tbytes);  // C blocks
  int mc = std::min(ma, std::max(8, cb / std::min(nr, 64) / 8 * 8));
  int nc = std::min(nr, std::max(1, cb / mc));
  if (nc < nr && nc >= 8) nc = nc / 8 * 8;
  char* w = t_ws;
  int* ea = reinterpret_cast<int*>(w);
  int* eb = reinterpret_cast<int*>(w + up256((size_t)g.M * 4));
  w += ebytes;
  signed char* Cp = reinterpret_cast<signed char*>(w);
  signed char* Ap = Cp + cbytes / 1024 * 1024;
  signed char* Bp = Ap + (size_t)ma * rbytes;
  if (g.K > kMaxK && g.k_in != g.K) return false;  // a k slice needs a shifted base
  auto src = [&](bool is_a, signed char* planes, int blk0, int rb, int k0, int kc) {
    Src x{};
    x.p = (is_a ? g.A : g.B) + 2 * (int64_t)k0 * (is_a ? g.a_ki : g.b_ki);
    x.row0 = 32 * blk0;
    x.rows = is_a ? g.M : g.N;
    x.K = kc;
    x.r_in = is_a ? g.m_in : g.n_in;
    x.k_in = g.k_in == g.K ? kc : g.k_in;
    x.r_so = is_a ? g.a_mo : g.b_no;
    x.r_si = is_a ? g.a_mi : g.b_ni;
    x.k_so = is_a ? g.a_ko : g.b_ko;
    x.k_si = is_a ? g.a_ki : g.b_ki;
    x.kfast = x.k_si == 1 || x.r_si != 1;
    x.conj = is_a ? g.conj_a : g.conj_b;
    x.planes = planes;
    x.rb = rb;
    x.kb = kblocks(kc);
    x.exps = is_a ? ea : eb;
    return x;
  };
  const ModTab& t = tab(moduli_for(g.M, g.N, g.K));
  // a product of an operand with itself (the same element map) needs its residues once
  const bool same = g.A == g.B && g.M == g.N && g.m_in == g.n_in && g.a_mo == g.b_no && g.a_mi == g.b_ni &&
                    g.a_ko == g.b_ko && g.a_ki == g.b_ki && g.conj_a == g.conj_b && ma == mb && nr == nb;
  for (int k0 = 0; k0 < g.K; k0 += kMaxK) {
    const int kc = std::min(g.K - k0, kMaxK);
    Gett<double> h = g;
    if (k0 > 0) h.accumulate = 1;
    for (int m0 = 0; m0 < mb; m0 += ma) {
      const int am = std::min(ma, mb - m0);
      for (int n0 = 0; n0 < nb; n0 += nr) {
        const int bn = std::min(nr, nb - n0);
        const bool do_a = n0 == 0, do_b = m0 == 0 || nr < nb;
        const Src a = src(true, Ap, m0, am, k0, kc), b = src(false, Bp, n0, bn, k0, kc);
        if (do_a)
          split(a, do_b && !same ? b : Src{}, t, s);
        else
          split(b, Src{}, t, s);
        for (int m1 = 0; m1 < am; m1 += mc)
          for (int n1 = 0; n1 < bn; n1 += nc) {
            PlaneGemm pg{};
            pg.mb = std::min(mc, am - m1);
            pg.nb = std::min(nc, bn - n1);
            pg.kb = a.kb;
            pg.planes = 2 * t.np;
            pg.A = Ap + (int64_t)m1 * (a.kb / 2) * kPlanes * 2048;
            pg.B = (same ? Ap : Bp) + (int64_t)n1 * (b.kb / 2) * kPlanes * 2048;
            pg.C = Cp;
            pg.a_in = pg.a_outer = pg.mb;
            pg.b_in = pg.b_outer = pg.nb;
            gemm_planes(pg, s);
            const int64_t units = (int64_t)pg.mb * pg.nb;
            hipLaunchKernelGGL(mod_crt_kernel, dim3((unsigned)std::min<int64_t>(units, 65535)), dim3(256), 0, s,
                               reinterpret_cast<const int*>(Cp), pg.mb, pg.nb, 32 * (m0 + m1),
                               32 * (n0 + n1), ea, same ? ea : eb, h, (int64_t)0, (int64_t)0, t);
            HIPCHECK(hipGetLastError());
          }
      }
    }
  }
  return true;
}

// ---------------------------------------------------------------- particle ladder
ModLadder::ModLadder(const double* F, int64_t row_stride, int v, int X, hipStream_t s) {
  const int vb = cdiv(v, 32), kb = kblocks(X);
  const size_t eb = up256((size_t)v * vb * 32 * 4), pb = (size_t)mod_plane_bytes((int64_t)v * vb * 32, X);
  const size_t least = (size_t)vb * vb * std::min(v, 8) * kPlanes * 1024;  // tiles of one a and 8 b
  if (!t_ws || v <= kModLadderNvir || X < kModLadderNaux || (int64_t)v * vb * 32 > 0x7fffffffLL ||
      eb + pb + least > t_ws_bytes)
    return;
  v_ = v;
  X_ = X;
  exps_ = reinterpret_cast<int*>(t_ws);
  planes_ = reinterpret_cast<signed char*>(t_ws + eb);
  held_ = eb + pb;
  Src a{};
  a.p = F;
  a.rows = v * vb * 32;
  a.K = X;
  a.r_in = vb * 32;
  a.r_valid = v;
  a.k_in = X;
  a.r_so = row_stride;
  a.r_si = X;
  a.k_so = a.k_si = 1;
  a.kfast = 1;
  a.planes = planes_;
  a.exps = exps_;
  a.rb = v * vb;
  a.kb = kb;
  split(a, Src{}, tab(15), s);  // K = naux: below the line of moduli_for, or no split
  t_ws += held_;  // the rest serves this ladder's tiles and, in turn, other products
  t_ws_bytes -= held_;
}

ModLadder::~ModLadder() {
  t_ws -= held_;
  t_ws_bytes += held_;
}

void ModLadder::rows(int a_lo, int a_hi, int a0, int64_t row0, double* W, int64_t ldw, hipStream_t s) const {
  const int v = v_, vb = cdiv(v, 32), blk0 = a0 / 32, wvb = vb - blk0;
  const int64_t run = (int64_t)(kblocks(X_) / 2) * kPlanes * 2048;  // bytes per row block
  // several rows a per product: 24 blocks or more along m keep the tile padding small
  const int ga_max = wvb >= 16 ? 2 : wvb >= 6 ? 4 : 8;
  constexpr size_t kC = (size_t)512 << 20;
  const int64_t cblocks = (int64_t)(std::min(kC, t_ws_bytes) / (kPlanes * 1024));
  for (int a = a_lo; a < a_hi; a += ga_max) {
    int ga = std::min(ga_max, a_hi - a);
    while (ga > 1 && (int64_t)ga * wvb * wvb > cblocks) --ga;
    for (int a1 = a; a1 < std::min(a + ga_max, a_hi); a1 += ga) {
      const int g1 = std::min(ga, std::min(a + ga_max, a_hi) - a1);
      const int nbmax = (int)std::min<int64_t>(v, std::max<int64_t>(1, cblocks / ((int64_t)g1 * wvb * wvb)));
      for (int b = a1 + 1; b < v; b += nbmax) {
        const int nbn = std::min(nbmax, v - b);
        PlaneGemm pg{};
        pg.A = planes_ + ((int64_t)a1 * vb + blk0) * run;
        pg.B = planes_ + ((int64_t)b * vb + blk0) * run;
        pg.C = reinterpret_cast<signed char*>(t_ws);
        pg.mb = g1 * wvb;
        pg.nb = nbn * wvb;
        pg.kb = kblocks(X_);
        pg.planes = 2 * 15;
        pg.a_in = pg.b_in = wvb;
        pg.a_outer = pg.b_outer = vb;
        gemm_planes(pg, s);
        LadderTiles lt{reinterpret_cast<const int*>(t_ws), exps_, v, vb, wvb, blk0, a0, a1, b, nbn, row0, W, ldw};
        hipLaunchKernelGGL(mod_ladder_antisym_kernel, dim3(wvb * (wvb + 1) / 2, nbn, g1), dim3(256), 0, s, lt, tab(15));
        HIPCHECK(hipGetLastError());
      }
    }
  }
}

// ---------------------------------------------------------------- triples
// nvir 126 per triple: FP64 products 49 us; here 20 (1.2 POP/s: 6 stages of K per tile, 70 MB
// of planes and residues moved) and 11.5 for the reconstruction.  Tiles of 8 x 4 blocks, two
// workgroups per CU, which load 1.2 times the operand bytes, took 22.9, of 4 x 4 blocks 28;
// with the products of a batch one after the other instead of side by side along n, the planes
// of V_j and V_k are read from memory for each, 1.7 more.
// Per triple the FP64 tiles take TFP us at 62 TFLOP/s (K = nvir in three passes over the
// output), the residues their plane products and one reconstruction (the estimates of
// mod_gemm_pays; splitting is amortised over nocc^2 / 6 triples per operand).
bool ModTriples::pays(int o, int v) {
  if (o < 3 || v < 32) return false;
  auto up = [](double x, double m) { return std::ceil(x / m) * m; };
  if ((int64_t)o * ((int64_t)v * v + 32) > 0x3fffffffLL || (int64_t)o * o * (v + 32) > 0x3fffffffLL) return false;
  const double P = 0.5 * v * (v - 1.0), n = o * (o - 1.0) * (o - 2.0) / 6.0;
  const double t64 = 3 * 8.0 * up(P, 64) * up(v, 64) * v / 62e6;
  const double tm = P * v * 15e-6 + 2.0 * kPlanes * up(P, 32) * up(v, 32) * 3 * up(v, 64) / 1.7e9;
  const double once = 50.0 + ((double)o * P * v + (double)o * o * v * v) * 15e-6;
  return tm + once / n < 0.9 * t64;
}

size_t ModTriples::bytes(int o, int v, int ni) {
  const int64_t P = (int64_t)v * (v - 1) / 2;
  const size_t mb = (size_t)cdiv(P, 32), nb = (size_t)cdiv(v, 32), rows = 32 * (o * mb + (size_t)o * o * nb);
  return up256(rows * 4) + (size_t)mod_plane_bytes(rows, v) + (size_t)ni * mb * nb * kPlanes * 1024;
}

ModTriples::ModTriples(void* ws, const double* V, const double* T2, int o, int v, int ni, hipStream_t s)
    : o_(o), v_(v), ni_(ni) {
  const int64_t P = (int64_t)v * (v - 1) / 2;
  mb_ = cdiv(P, 32);
  nb_ = cdiv(v, 32);
  const int kb = kblocks(v);
  ea_ = static_cast<int*>(ws);
  eb_ = ea_ + (size_t)32 * o * mb_;
  pa_ = static_cast<signed char*>(ws) + up256((size_t)32 * ((size_t)o * mb_ + (size_t)o * o * nb_) * 4);
  pb_ = pa_ + mod_plane_bytes(32LL * o * mb_, v);
  out_ = pb_ + mod_plane_bytes(32LL * o * o * nb_, v);
  Src a{};
  a.p = V;
  a.rows = 32 * o * mb_;
  a.K = a.k_in = v;
  a.r_in = 32 * mb_;
  a.r_valid = (int)P;
  a.r_so = P * v;
  a.r_si = v;
  a.k_so = a.k_si = 1;
  a.kfast = 1;
  a.planes = pa_;
  a.exps = ea_;
  a.rb = o * mb_;
  a.kb = kb;
  Src b = a;
  b.p = T2;
  b.rows = 32 * o * o * nb_;
  b.r_in = 32 * nb_;
  b.r_valid = v;
  b.r_so = (int64_t)v * v;
  b.planes = pb_;
  b.exps = eb_;
  b.rb = o * o * nb_;
  const ModTab& t = tab(15);  // K = 3 nvir: short chains in the FP64 products too
  const int na = norm_blocks(a), nbk = norm_blocks(b);
  hipLaunchKernelGGL(mod_norm_kernel, dim3(na + nbk), dim3(1024), 0, s, a, na, b, tpr_of(a), tpr_of(b), t.S);
  HIPCHECK(hipGetLastError());
  hipLaunchKernelGGL(mod_joint_exps_kernel, dim3(cdiv(32LL * mb_, 256)), dim3(256), 0, s, ea_, o, 32 * mb_);
  HIPCHECK(hipGetLastError());
  hipLaunchKernelGGL(mod_joint_exps_kernel, dim3(cdiv(32LL * nb_, 256)), dim3(256), 0, s, eb_, o * o, 32 * nb_);
  HIPCHECK(hipGetLastError());
  split_scaled(a, b, t, s);
}

void ModTriples::rows(int i0, int ni, int j, int k, double* We, hipStream_t s) const {
  const int64_t P = (int64_t)v_ * (v_ - 1) / 2;
  const int64_t seg = (int64_t)kblocks(v_) / 2 * kPlanes * 128;  // 16-byte units per row block
  const int64_t ta = mb_ * seg, tb = nb_ * seg;                  // per tile and per pair
  const int64_t cb = (int64_t)mb_ * nb_ * kPlanes * 1024;
  for (int y = 0; y < ni; y += ni_) {
    const int i = i0 + y, n = std::min(ni_, ni - y);
    PlaneGemm g{};
    g.A = pa_;
    g.B = pb_;
    g.C = out_;
    g.mb = g.a_in = g.a_outer = mb_;
    g.nb = g.b_in = g.b_outer = nb_;
    g.kb = 3 * kblocks(v_);
    g.planes = 2 * 15;
    for (int q = 0; q < kNP; ++q) g.p[q] = kMods[q];
    g.batch = n;
    const int64_t at[3] = {i, j, k}, bt[3] = {(int64_t)j * o_ + k, (int64_t)k * o_ + i, (int64_t)i * o_ + j};
    const int abat[3] = {1, 0, 0}, bbat[3] = {0, 1, o_};
    for (int q = 0; q < 3; ++q) {
      g.a_seg[q] = at[q] * ta;
      g.b_seg[q] = bt[q] * tb;
      g.a_bat[q] = abat[q] * ta;
      g.b_bat[q] = bbat[q] * tb;
    }
    g.c_bat = cb;
    if (nb_ <= 4)
      launch_planes<4, 2, 4, 2, 1, 1, true>(g, s);
    else
      launch_planes<2, 4, 4, 2, 1, 1, true>(g, s);
    Gett<double> c{};
    c.M = c.m_in = (int)P;
    c.N = c.n_in = v_;
    c.c_mi = v_;
    c.c_ni = 1;
    c.alpha_re = -1.0;
    c.C = We + 2 * y * P * v_;
    hipLaunchKernelGGL(mod_crt_kernel, dim3((unsigned)std::min<int64_t>((int64_t)mb_ * nb_, 65535), n), dim3(256), 0, s,
                       reinterpret_cast<const int*>(out_), mb_, nb_, 0, 0, ea_, eb_, c, cb / 4, P * v_, tab(15));
    HIPCHECK(hipGetLastError());
  }
}

}  // namespace exacc
