// FP64 complex products on the INT8 matrix cores.
//
// The FP64 matrix rate of gfx950 (78.6 TFLOP/s) bounds the FP64 GETT, which already runs at
// 0.8 to 0.95 of it on large products.  The INT8 rate is about 64 times higher, so a large
// product is formed exactly on integers instead, in a residue number system:
//   * every operand row a_m is scaled by a power of two to the 2-norm range (2^(S-1), 2^S]
//     and rounded to integers (S = 58 or 61 bits, more than the 53 of a double);
//   * modulo a prime (or product of primes) p = 1 mod 4 there is j with j^2 = -1, and a
//     complex integer x + iy is held as the pair (x + jy, x - jy) mod p: in this form a
//     complex product is two real products (the quadratic residue number system of
//     Leung and of Jenkins and Krogmeier), so 16 or 17 moduli give 32 or 34 INT8 planes;
//   * per plane one INT8 GEMM with INT32 accumulation (exact: |sum| <= K (p/2)^2 < 2^31 for
//     K <= kMaxK), reduced mod p to one byte per output;
//   * the Chinese remainder theorem gives the exact integer product back: by the
//     Cauchy-Schwarz inequality |re|, |im| <= |a_m| |b_n| <= 2^(2S) < M / 2, M the product of
//     the moduli, so value / M is the fractional part of sum_i r_i w_i / p_i, summed as an
//     exact high part (multiples of 2^-42) and an FP64 remainder.
// The only rounding is that of the scaled operands to integers (relative to the row's norm)
// and of the result to FP64; sums over k are exact, so results do not depend on tiling.
//
// That rounding is relative to |a_m| |b_n|, an FP64 sum's to sum_k |a_mk| |b_nk|, which is far
// smaller where the entries of a row differ in size and the large ones of a_m meet the small
// ones of b_n.  So each product is tested before it is formed: one further INT8 plane holds the
// rows' magnitudes in units of 1/32 of the row's rms, rounded down and cut at 127, and its product
// bounds sum_k |a_mk| |b_nk| from below for every output.  The largest ratio F of |a_m| |b_n| to that
// bound picks 16 moduli (F <= kFlat), 17 (F <= 8 kFlat) or the FP64 kernel, which is launched
// behind every residue product and returns at once unless it is wanted: no host decision, so
// a recorded graph decides anew on each replay.  Rows that are not finite, or whose squares leave
// the range of a double, take the FP64 kernel too.
// rms error over sum |a||b| in units of 2^-53, K 1131, the sums in the FP64 kernel's form against
// 58 and 61 bits (80-bit reference): Gaussian entries, F 1.7, 0.28 (re) | 0.023, 0.011; scales
// along k opposed by 1 decade, F 4.0, 0.28 | 0.049, 0.012; lognormal sizes, F 10, 0.70 | 0.071,
// 0.030; scales opposed by 2 decades, F 29, 0.27 | 0.24, 0.033; by 4, F 64000, 0.26 | 12, 1.5.
// An FP64 sum split over K in eight has a third of these errors, which is where kFlat lies.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "common.h"

namespace exacc {

constexpr int kNP = 17;           // most moduli

// Which moduli a launch takes: 0, 1 (see Tabs), or 2, none at all; read from the device where
// the product's test has left it, or known.
struct Level {
  const int* flag;
  int known;
};
struct PlaneGemm {
  const signed char *A, *B;
  signed char* C;              // [mblk][nblk][z][lane][q][r]: row 8 q + 4 (lane / 32) + r, column lane % 32
  int mb, nb, kb;              // kb even
  int a_in, a_outer;           // A block of m-block x: (x / a_in) * a_outer + x % a_in
  int b_in, b_outer;           // likewise B
  int tiles_m, tiles_n;
  Level lv;                    // 2 (16 + level) of the kPlanes that the layouts have room for
  int p[kNP];
  // TEST kernels: one plane, of magnitudes; rows' and columns' flatness and where the level goes
  const float *fa, *fb;
  float flat;                  // kFlat, less where a product's rounding is more
  int* out;
  // SEG kernels: k in three segments of kb / 3 blocks, segment q of product y of a batch at
  // 16-byte units a_seg[q] + y a_bat[q] of A (B likewise), C of product y c_bat bytes further
  int batch;
  int64_t a_seg[3], b_seg[3], a_bat[3], b_bat[3], c_bat;
};

namespace {

constexpr int kPlanes = 2 * kNP;
constexpr int kMaxK = 131072;     // K (p / 2)^2 < 2^31 with p <= 241
constexpr int kShortK = 1152;     // K (p / 2)^2 + 128 < 2^24
constexpr int kZero = 4096;       // exponent of a row of zeros: above that of any other
constexpr double kUnit = 32.0;    // units of a magnitude in its row's rms
constexpr float kFlat = 6.0f;     // largest F (see the top) that 16 moduli are taken for

typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i16v __attribute__((ext_vector_type(16)));
typedef double d2v __attribute__((ext_vector_type(2)));
typedef unsigned __int128 u128;

// Pairwise coprime products of primes = 1 mod 4 (so that -1 has a square root), largest first.
constexpr int kMods[kNP] = {241, 233, 229, 221, 205, 197, 193, 181, 173, 157, 149, 137, 113, 109, 101, 97, 89};

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

// Both choices of moduli: t[0] 16 of them (S = 58), t[1] 17 (S = 61).  Scale exponents are
// those of t[1]; t[0] takes kShift less.
struct Tabs {
  ModTab t[2];
};
constexpr int kShift = 3;
const Tabs& tabs() {
  static const Tabs t = [] {
    Tabs x{{make_tab(16), make_tab(17)}};
    if (x.t[1].S - x.t[0].S != kShift) raise(-3, "residue tables");
    return x;
  }();
  return t;
}

__device__ __forceinline__ int level_of(const Level& l) { return l.flag ? *l.flag : l.known; }

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
  // whole 68 KiB runs (a plane-major order: 2.3 TB/s at 12363^2, this one: see mod_split_kernel)
  signed char* planes;
  int* exps;        // power of two each row was scaled by (of t[1], see Tabs)
  // magnitudes, max(|re|, |im|) in units of the row's rms / kUnit, rounded down and at most 127, in
  // the order of the planes without z, and per row its norm in that unit: 0 for a row of zeros,
  // infinite for a row that residues are not for
  signed char* mags;
  float* flat;
  double* norm;     // if not null: per row its norm (0 where it is not in range)
  int rb, kb;       // 32-row and 32-k blocks (kb even)
};

// Scale exponents, magnitudes and flatness of all rows of an operand, padding included: per row
// the largest |component| and the sum of squares (fixed order), then the magnitudes, of which each
// thread has kept its first kKeep entries' (the upper words, below the entries themselves); a
// longer row is read again.  kfast: tpr threads per row; else 1024 / tpr rows of a
// workgroup side by side, 32, or 8 where 32 would give too few workgroups.
// what: 1 the scales, 2 the magnitudes (with the norms of an earlier launch where 1 is left
// out), 3 both.  Bound by reading the operand.
__global__ __launch_bounds__(1024) void mod_norm_kernel(Src a, int blocks_a, Src b, int tpr_a, int tpr_b, int S,
                                                        int what, int* flag) {
  const bool first = (int)blockIdx.x < blocks_a;
  const Src s = first ? a : b;
  const int blk = first ? blockIdx.x : blockIdx.x - blocks_a;
  const int tid = threadIdx.x;
  __shared__ double ssum[1024], smax[1024];
  if (flag && blockIdx.x == 0 && tid == 0) *flag = 0;
  const int width = first ? tpr_a : tpr_b, rows = 1024 / width;
  const int row = blk * rows + (s.kfast ? tid / width : tid % rows);
  const int k0 = s.kfast ? tid % width : tid / rows, stride = s.kfast ? 1 : rows;
  const bool has = row < s.rows && (s.r_valid == 0 || row % s.r_in < s.r_valid);
  const bool plain = s.k_in == s.K;
  const double* p = has ? s.p + 2 * cmap(row, s.r_in, s.r_so, s.r_si) : nullptr;
  auto at = [&](int k) {
    return *reinterpret_cast<const d2v*>(p + 2 * (plain ? (int64_t)k * s.k_si : cmap(k, s.k_in, s.k_so, s.k_si)));
  };
  constexpr int kKeep = 32, kG = 8;
  unsigned keep[kKeep] = {};
  double sum = 0.0, mx = 0.0, norm = 0.0;
  if (what & 1) {
    if (has) {
#pragma unroll
      for (int j = 0; j < kKeep; j += kG) {
        if (j * width >= s.K) break;
        d2v x[kG];
#pragma unroll
        for (int i = 0; i < kG; ++i) x[i] = at(min(k0 + (j + i) * width, s.K - 1));
#pragma unroll
        for (int i = 0; i < kG; ++i) {
          if (k0 + (j + i) * width >= s.K) x[i] = d2v{0.0, 0.0};
          const double m = fmax(fabs(x[i].x), fabs(x[i].y));
          sum += x[i].x * x[i].x + x[i].y * x[i].y;
          mx = fmax(mx, m);
          keep[j + i] = (unsigned)__double2hiint(m);
        }
      }
#pragma unroll 4
      for (int k = k0 + kKeep * width; k < s.K; k += width) {
        const d2v x = at(k);
        sum += x.x * x.x + x.y * x.y;
        mx = fmax(mx, fmax(fabs(x.x), fabs(x.y)));
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
    sum = ssum[tid - k0 * stride];
    mx = smax[tid - k0 * stride];
    // (a sum that is not finite fails the second comparison)
    const bool ok = sum > 1e-280 && sum < 1e300;
    if (k0 == 0 && row < 32 * s.rb) {
      int ex = 0;
      if (ok) {
        (void)frexp(sum, &ex);  // norm < 2^(ex / 2)
        ex = (ex + 1) >> 1;
      }
      s.exps[row] = ok ? S - ex : kZero;
      const bool zero = sum == 0.0 && mx == 0.0;
      s.flat[row] = zero ? 0.0f : ok ? (float)(kUnit * sqrt((double)s.K)) : __builtin_huge_valf();
      if (s.norm) s.norm[row] = ok ? sqrt(sum) : 0.0;
    }
    if (ok) norm = sqrt(sum);
  } else if (row < s.rows) {
    norm = s.norm[row];
  }
  if (!(what & 2) || row >= 32 * s.rb) return;
  const double inv = norm > 0.0 ? kUnit * sqrt((double)s.K) / norm : 0.0;
  signed char* out = s.mags + (int64_t)(row >> 5) * (s.kb / 2) * 2048 + (row & 31) * 16;
  auto put = [&](int k, double m) {
    out[(int64_t)(k >> 6) * 2048 + ((k >> 5) & 1) * 1024 + ((k >> 4) & 1) * 512 + (k & 15)] =
        (signed char)(int)fmin(m * inv, 127.0);
  };
  if (what & 1) {
#pragma unroll
    for (int j = 0; j < kKeep; ++j) {
      const int k = k0 + j * width;
      if (j * width >= 32 * s.kb) break;
      if (k < 32 * s.kb) put(k, __hiloint2double((int)keep[j], 0));
    }
  }
#pragma unroll 4
  for (int k = k0 + (what & 1 ? kKeep * width : 0); k < 32 * s.kb; k += width) {
    double m = 0.0;
    if (has && k < s.K && inv > 0.0) {
      const d2v x = at(k);
      m = fmax(fabs(x.x), fabs(x.y));
    }
    put(k, m);
  }
}

// Residue planes of 32 rows x 64 k per workgroup: the scaled, rounded values are staged in
// LDS as 8 balanced base-256 digits (re, im), then each wave forms every second modulus of one
// 32 x 32 block, 16 k per lane: x mod p is a dot product of the digits with 256^d mod p (two
// 4-byte dot instructions) and one rounding step, 16 instructions per element and modulus
// against 16 bytes read and 4 written.
__global__ __launch_bounds__(256) void mod_split_kernel(Src a, int blocks_a, Src b, Level lv, Tabs tt) {
  const int level = level_of(lv);
  if (level > 1) return;
  const ModTab& t = tt.t[level];
  const int shift = level ? 0 : kShift;
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
    if (rowb + r < s.rows && kgrp * 64 + kk < s.K && !pad) {
      x.x = rint(ldexp(xs[q].x, es[q] - shift));
      x.y = rint(ldexp(s.conj ? -xs[q].y : xs[q].y, es[q] - shift));
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


// C[z] = A[z] B[z]^T mod p: WM x WN waves of TM x TN 32 x 32 blocks, stages of 64 k in three
// LDS buffers filled by direct global-to-LDS loads, two stages ahead.  Operands lie in
// fragment order, so a block is one contiguous 1 KiB copy and every LDS read is
// conflict-free.  The grid is what the chip holds; a workgroup walks tiles grid apart and
// loads the next tile's first stages before it reduces and stores this one's outputs.
// Bound by the power the INT8 matrix cores draw: 4032^3 x 32 planes 2380 TOP/s, the same
// launch on zeros and ones about 3000; one tile per workgroup 2250 there and 1426 instead of
// 1895 at 1268 x 25000 x 951, where filling the pipeline is a larger part.
// TEST: the product of the magnitudes, which is not stored: the outputs' largest
// fa fb / sum gives the level (see the top).
template <int WM, int WN, int TM, int TN, int OCC, bool LONG, bool SEG, bool TEST>
__global__ __launch_bounds__(64 * WM * WN, OCC) void mod_gemm_kernel(PlaneGemm g) {
  constexpr int KB = 2, S = 3;
  constexpr int kStage = TEST ? 128 : kPlanes * 128;  // 16-byte units of a stage of one row block
  const int level = TEST ? 0 : level_of(g.lv);
  if (!TEST && level > 1) return;
  const int planes = TEST ? 1 : 2 * (16 + level);
  constexpr int T = 64 * WM * WN, RA = WM * TM, RB = WN * TN;
  constexpr int NA = RA * KB * 64 / T, NB = RB * KB * 64 / T;
  static_assert(NA * T == RA * KB * 64 && NB * T == RB * KB * 64, "whole copies per thread");
  __shared__ i4v sm[S][(RA + RB) * KB * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w % WM, wn = w / WM;
  // a batch's products are further tiles along n, so that what they share of A is read together
  const int tiles_n = SEG ? g.tiles_n * g.batch : g.tiles_n;
  const int tiles = g.tiles_m * tiles_n, total = tiles * planes;
  const int nk = g.kb / KB, nseg = SEG ? nk / 3 : nk;
  const int64_t rs = (int64_t)nseg * kStage;  // 16-byte units per row block
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
    int64_t ka = (int64_t)kt * kStage, kb = ka;
    if (SEG) {
      const int sg = kt >= 2 * nseg ? 2 : kt >= nseg ? 1 : 0;
      ka -= (int64_t)sg * nseg * kStage;
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
  constexpr int kBias = LONG || TEST ? 0 : 128;  // see the reduction below
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
    if constexpr (TEST) {
      int worst = 0;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int bm = cm0 + wm * TM + i, bn = cn0 + wn * TN + j;
          if (bm >= g.mb || bn >= g.nb) continue;
          const float fb = g.fb[32 * bn + (lane & 31)];
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float x = g.fa[32 * bm + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] * fb;
            const float y = g.flat * (float)acc[i][j][r];
            worst = max(worst, y >= x ? 0 : 8.0f * y >= x ? 1 : 2);  // 2 where x is no number
          }
        }
      const bool any2 = __ballot(worst == 2) != 0, any1 = __ballot(worst == 1) != 0;
      if (lane == 0 && (any1 || any2)) atomicMax(g.out, any2 ? 2 : 1);
      job = next;
      if (job >= total) break;
      continue;
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
    if (i >= 16 && i >= t.np) break;
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
                                                      int64_t c_bat, Level lv, Tabs tt) {
  const int level = level_of(lv);
  if (level > 1) return;
  const ModTab& t = tt.t[level];
  const int shift = level ? 0 : 2 * kShift;
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
    const int en = eb[n] - shift;
    const int64_t co = cmap(n, g.n_in, g.c_no, g.c_ni);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mr + r;
      if (m >= g.M) continue;
      const int em = ea[m];
      const double xr = ldexp(f.re[r], -(em + en)), xi = ldexp(f.im[r], -(em + en));
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
__global__ __launch_bounds__(256) void mod_ladder_antisym_kernel(LadderTiles g, int level, Tabs tt) {
  const ModTab& t = tt.t[level];
  const int shift = level ? 0 : 2 * kShift;
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
    const int en = c0 < g.v ? g.exps[b * 32 * g.vb + c0] - shift : 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int em = r0 + r < g.v ? g.exps[a * 32 * g.vb + r0 + r] : 0;
      y[r].x = ldexp(f.re[r], -(em + en));
      y[r].y = ldexp(f.im[r], -(em + en));
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
// of them less 1, room for three rows in one Cauchy-Schwarz bound (sqrt(3) < 2); the norm
// becomes the group's largest, and so does the flatness.  One thread per r; nothing beside what it prepares (groups n rows).
__global__ __launch_bounds__(256) void mod_joint_exps_kernel(int* exps, double* norm, float* flat, int groups, int n) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= n) return;
  int e = kZero;
  double top = 0.0;
  float f = 0.0f;
#pragma unroll 8
  for (int g = 0; g < groups; ++g) {
    const int64_t q = (int64_t)g * n + r;
    e = min(e, exps[q]);
    top = fmax(top, norm[q]);
    f = fmaxf(f, flat[q]);
  }
  for (int g = 0; g < groups; ++g) {
    const int64_t q = (int64_t)g * n + r;
    exps[q] = e - 1;
    norm[q] = top;
    flat[q] = f;
  }
}

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Threads per row of mod_norm_kernel: as many as keep a whole row, up to 32768 entries.
int tpr_of(const Src& s) { return s.kfast ? (s.K <= 2048 ? 64 : s.K <= 8192 ? 256 : 1024) : s.rb < 256 ? 128 : 32; }
int norm_blocks(const Src& s) { return cdiv(32 * s.rb, 1024 / tpr_of(s)); }

// Residue planes of one or two operands (b may have rows == 0).
void split(const Src& a, const Src& b, Level lv, hipStream_t s) {
  const int sa = a.rb * (a.kb / 2), sb = b.rows ? b.rb * (b.kb / 2) : 0;
  hipLaunchKernelGGL(mod_split_kernel, dim3(sa + sb), dim3(256), 0, s, a, sa, b, lv, tabs());
  HIPCHECK(hipGetLastError());
}
// Their scales (what & 1) and magnitudes (what & 2); flag: set to 0 (may be null).
void norms(const Src& a, const Src& b, int what, int* flag, hipStream_t s) {
  const int na = norm_blocks(a), nb = b.rows ? norm_blocks(b) : 0;
  hipLaunchKernelGGL(mod_norm_kernel, dim3(na + nb), dim3(1024), 0, s, a, na, b, tpr_of(a), tpr_of(b), tabs().t[1].S,
                     what, flag);
  HIPCHECK(hipGetLastError());
}

// RES: workgroups one CU holds (of 160 KiB LDS).  256 CUs.
template <int WM, int WN, int TM, int TN, int OCC, int RES, bool SEG = false, bool TEST = false>
void launch_planes(PlaneGemm g, hipStream_t s) {
  // the grid is laid out for 17 moduli or one plane of magnitudes; fewer leave workgroups without a tile
  const int planes = TEST ? 1 : kPlanes;
  g.tiles_m = cdiv(g.mb, WM * TM);
  g.tiles_n = cdiv(g.nb, WN * TN);
  const int64_t jobs = (int64_t)g.tiles_m * g.tiles_n * planes * (SEG ? g.batch : 1);
  if (jobs > 0x7fffffffLL) raise(-1, "contraction too large for one launch");
  const dim3 grid((unsigned)std::min<int64_t>(jobs, 256 * RES)), block(64 * WM * WN);
  if constexpr (TEST)
    hipLaunchKernelGGL((mod_gemm_kernel<WM, WN, TM, TN, OCC, true, SEG, true>), grid, block, 0, s, g);
  else if (32 * g.kb <= kShortK)
    hipLaunchKernelGGL((mod_gemm_kernel<WM, WN, TM, TN, OCC, false, SEG, false>), grid, block, 0, s, g);
  else
    hipLaunchKernelGGL((mod_gemm_kernel<WM, WN, TM, TN, OCC, true, SEG, false>), grid, block, 0, s, g);
  HIPCHECK(hipGetLastError());
}

// Tile choice: the padded block count of each tile shape over its measured rate (TOP/s at
// full tiles, see mod_gemm_kernel), in whole rounds of the workgroups the chip holds.
struct Tile {
  int pick;     // 0: 8 x 8 blocks, 1: 4 x 8, 2: 8 x 4, 3: 4 x 4
  double cost;  // padded blocks / (TOP/s)
};
Tile tile_for(int mb, int nb, int planes) {
  static const struct {
    int ra, rb, resident;
    double rate;
  } c[4] = {{8, 8, 256, 2200}, {4, 8, 512, 1900}, {8, 4, 512, 1940}, {4, 4, 768, 1720}};
  Tile best{0, 1e300};
  for (int q = 0; q < 4; ++q) {
    const int64_t wgs = (int64_t)cdiv(mb, c[q].ra) * cdiv(nb, c[q].rb) * planes, r = c[q].resident;
    const double rounds = wgs >= 8 * r ? (double)wgs / r : (double)((wgs + r - 1) / r);
    const double cost = rounds * r * c[q].ra * c[q].rb / c[q].rate;
    if (cost < best.cost) best = {q, cost};
  }
  return best;
}
template <bool TEST = false>
void gemm_planes(PlaneGemm g, hipStream_t s) {
  if (g.kb < 4) raise(-1, "residue product: K too short for its pipeline");  // two stages at least
  for (int i = 0; i < kNP; ++i) g.p[i] = kMods[i];
  switch (tile_for(g.mb, g.nb, TEST ? 1 : kPlanes - 2).pick) {  // 16 moduli as a rule
    case 0: return launch_planes<2, 4, 4, 2, 1, 1, false, TEST>(g, s);
    case 1: return launch_planes<2, 2, 2, 4, 2, 2, false, TEST>(g, s);
    case 2: return launch_planes<2, 2, 4, 2, 2, 2, false, TEST>(g, s);
    default: return launch_planes<2, 2, 2, 2, 3, 3, false, TEST>(g, s);
  }
}

thread_local char* t_ws = nullptr;
thread_local size_t t_ws_bytes = 0;

inline size_t up256(size_t b) { return (b + 255) / 256 * 256; }
inline int kblocks(int K) { return 2 * cdiv(K, 64); }

}  // namespace

// Estimated times (us).  FP64 GETT: 64 x 64 tiles at 58 TFLOP/s (43 to 67 reached).  Here: seven
// launches, two of them the FP64 kernel's that return; scales, magnitudes and splitting 18 ps per
// element; reconstruction 15 ps per output; the plane products as tile_for has them; the test
// 0.36 per stage of a tile alone on its CU, or the whole at 1.7 POP/s.  Measured (us, FP64 GETT /
// this): 900^3 135 / 103, 1131^3 213 / 146, 400 x 19800 x 600 696 / 643, 700 x 900 x 5000 461 / 351,
// 600 x 700 x 40000 2056 / 1813; under the line 640^3 57 / 65, 28224 x 168 x 504 396 / 508,
// 1131 x 1131 x 259 64 / 80, 190 x 9730 x 9730 2129 / 2355, 400 x 400 x 19600 579 / 613.  Operands
// that fail the test cost the FP64 GETT and the test: 1131^3 257, 1200 x 1200 x 4096 776 / 838.
bool mod_gemm_pays(int64_t M, int64_t N, int64_t K) {
  if (M < 128 || N < 128 || K < 128 || M > 0x7fffffffLL || N > 0x7fffffffLL) return false;
  auto up = [](int64_t x, int64_t m) { return (double)((x + m - 1) / m * m); };
  const double t64 = 8.0 * up(M, 64) * up(N, 64) * (double)K / 58e6;
  const double test = std::max(0.36 * up(K, 64) / 64, 2.0 * up(M, 32) * up(N, 32) * up(K, 64) / 1.7e9);
  const double tm = 30.0 + (double)(M + N) * K * (K > kMaxK ? 23e-6 : 18e-6) + (double)M * N * 15e-6 +
                    tile_for(cdiv(M, 32), cdiv(N, 32), kPlanes - 2).cost * 2048e-6 * up(K, 64) + test;
  return tm < 0.95 * t64;
}

static int64_t plane_bytes(int64_t rows, int64_t K) {
  return kPlanes * ((rows + 31) / 32) * ((K + 63) / 64) * 2048;
}
static int64_t mag_bytes(int64_t rows, int64_t K) { return ((rows + 31) / 32) * ((K + 63) / 64) * 2048; }
int64_t mod_operand_bytes(int64_t rows, int64_t K) {
  return plane_bytes(rows, K) + mag_bytes(rows, K) + ((rows + 31) / 32) * 256;
}
int64_t mod_out_bytes(int64_t M, int64_t N) { return kPlanes * ((M + 31) / 32) * ((N + 31) / 32) * 1024; }

void set_mod_workspace(void* p, size_t bytes) {
  t_ws = static_cast<char*>(p);
  t_ws_bytes = p ? bytes : 0;
}

bool mod_gemm_wanted(const Gett<double>& g) { return t_ws && g.K >= 1 && mod_gemm_pays(g.M, g.N, g.K); }

const int* mod_gemm(const Gett<double>& g0, hipStream_t s) {
  Gett<double> g = g0;
  if (!mod_gemm_wanted(g) || g.nbatch != 1) return nullptr;
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
  // K in near-equal slices of whole 64-k groups, so that no slice is short
  const int nsl = cdiv(g.K, kMaxK), ks = nsl == 1 ? g.K : 64 * cdiv(cdiv(g.K, nsl), 64);
  if (nsl > 1 && g.k_in != g.K) return nullptr;  // a k slice needs a shifted base
  const size_t rbytes = (size_t)kPlanes * kblocks(ks) * 1024, tbytes = (size_t)kPlanes * 1024;
  // ahead of the planes: the level, scale exponents and flatness of every row, magnitudes
  const size_t ra = up256((size_t)mb * 128), rb = up256((size_t)nb * 128);
  const size_t ebytes = 256 + 2 * (ra + rb) + (size_t)mag_bytes(g.M, ks) + (size_t)mag_bytes(g.N, ks);
  // A and B blocks resident at a time (ma, nbr) and C blocks per product (mc x nc): C is kept
  // to what the last-level cache holds, since the reconstruction reads it right away
  constexpr size_t kC = (size_t)512 << 20;
  if (ebytes + 64 * tbytes > t_ws_bytes) return nullptr;
  const size_t room = t_ws_bytes - ebytes;
  size_t cbytes = std::min(std::min(kC, room / 4), (size_t)mb * nb * tbytes);
  if (cbytes < (size_t)std::min(mb, 8) * std::min(nb, 8) * tbytes) return nullptr;
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
    if (ma < std::min(mb, 16) || nr < std::min(nb, 16)) return nullptr;
    if (ma < mb) ma = ma / 8 * 8;
    if (nr < nb) nr = nr / 8 * 8;
  }
  const int cb = (int)(cbytes / tbytes);  // C blocks
  int mc = ma, nc = nr;
  if ((int64_t)ma * nr > cb) {
    mc = std::min(ma, std::max(8, cb / std::min(nr, 64) / 8 * 8));
    nc = std::min(nr, std::max(1, cb / mc));
    if (nc < nr && nc >= 8) nc = nc / 8 * 8;
  }
  char* w = t_ws;
  auto take = [&](size_t bytes) {
    char* p = w;
    w += bytes;
    return p;
  };
  int* const flag = reinterpret_cast<int*>(take(256));
  int* const ea = reinterpret_cast<int*>(take(ra));
  int* const eb = reinterpret_cast<int*>(take(rb));
  float* const fa = reinterpret_cast<float*>(take(ra));
  float* const fb = reinterpret_cast<float*>(take(rb));
  signed char* const ga = reinterpret_cast<signed char*>(take((size_t)mag_bytes(g.M, ks)));
  signed char* const gb = reinterpret_cast<signed char*>(take((size_t)mag_bytes(g.N, ks)));
  signed char* Cp = reinterpret_cast<signed char*>(w);
  signed char* Ap = Cp + cbytes / 1024 * 1024;
  signed char* Bp = Ap + (size_t)ma * rbytes;
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
    x.flat = is_a ? fa : fb;
    x.mags = is_a ? ga : gb;
    return x;
  };
  // a product of an operand with itself (the same element map) needs its residues once
  const bool same = g.A == g.B && g.M == g.N && g.m_in == g.n_in && g.a_mo == g.b_no && g.a_mi == g.b_ni &&
                    g.a_ko == g.b_ko && g.a_ki == g.b_ki && g.conj_a == g.conj_b && ma == mb && nr == nb;
  // scales and magnitudes of the slice from k0 on
  auto scale = [&](int k0, int kc, int* level) {
    norms(src(true, nullptr, 0, mb, k0, kc), same ? Src{} : src(false, nullptr, 0, nb, k0, kc), 3, level, s);
  };
  // the level of the whole product comes first: C may be accumulated into
  for (int k0 = 0; k0 < g.K; k0 += ks) {
    const int kc = std::min(g.K - k0, ks);
    scale(k0, kc, k0 == 0 ? flag : nullptr);
    PlaneGemm pg{};
    pg.A = ga;
    pg.B = same ? ga : gb;
    pg.mb = pg.a_in = pg.a_outer = mb;
    pg.nb = pg.b_in = pg.b_outer = nb;
    pg.kb = kblocks(kc);
    pg.fa = fa;
    pg.fb = same ? fa : fb;
    pg.flat = kFlat;
    pg.out = flag;
    gemm_planes<true>(pg, s);
  }
  const Level lv{flag, 0};
  for (int k0 = 0; k0 < g.K; k0 += ks) {
    const int kc = std::min(g.K - k0, ks);
    if (nsl > 1) scale(k0, kc, nullptr);
    Gett<double> h = g;
    if (k0 > 0) h.accumulate = 1;
    for (int m0 = 0; m0 < mb; m0 += ma) {
      const int am = std::min(ma, mb - m0);
      for (int n0 = 0; n0 < nb; n0 += nr) {
        const int bn = std::min(nr, nb - n0);
        const bool do_a = n0 == 0, do_b = m0 == 0 || nr < nb;
        const Src a = src(true, Ap, m0, am, k0, kc), b = src(false, Bp, n0, bn, k0, kc);
        if (do_a)
          split(a, do_b && !same ? b : Src{}, lv, s);
        else
          split(b, Src{}, lv, s);
        for (int m1 = 0; m1 < am; m1 += mc)
          for (int n1 = 0; n1 < bn; n1 += nc) {
            PlaneGemm pg{};
            pg.mb = std::min(mc, am - m1);
            pg.nb = std::min(nc, bn - n1);
            pg.kb = a.kb;
            pg.lv = lv;
            pg.A = Ap + (int64_t)m1 * (a.kb / 2) * kPlanes * 2048;
            pg.B = (same ? Ap : Bp) + (int64_t)n1 * (b.kb / 2) * kPlanes * 2048;
            pg.C = Cp;
            pg.a_in = pg.a_outer = pg.mb;
            pg.b_in = pg.b_outer = pg.nb;
            gemm_planes(pg, s);
            const int64_t units = (int64_t)pg.mb * pg.nb;
            hipLaunchKernelGGL(mod_crt_kernel, dim3((unsigned)std::min<int64_t>(units, 65535)), dim3(256), 0, s,
                               reinterpret_cast<const int*>(Cp), pg.mb, pg.nb, 32 * (m0 + m1),
                               32 * (n0 + n1), ea, same ? ea : eb, h, (int64_t)0, (int64_t)0, lv, tabs());
            HIPCHECK(hipGetLastError());
          }
      }
    }
  }
  return flag;
}

// ---------------------------------------------------------------- particle ladder
// Rows (a, c) of the factors as one operand, each a padded to whole blocks.
static Src ladder_rows(const double* F, int64_t row_stride, int v, int X) {
  const int vb = cdiv(v, 32);
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
  a.rb = v * vb;
  a.kb = kblocks(X);
  return a;
}
static bool ladder_wanted(int v, int X) {
  return t_ws && v > kModLadderNvir && X >= kModLadderNaux && (int64_t)v * cdiv(v, 32) * 32 <= 0x7fffffffLL;
}

int ModLadder::level(const double* F, int64_t row_stride, int v, int X, hipStream_t s) {
  if (!ladder_wanted(v, X)) return 2;
  Src a = ladder_rows(F, row_stride, v, X);
  const size_t rows = up256((size_t)a.rows * 4), mags = (size_t)mag_bytes(a.rows, X);
  if (256 + 2 * rows + mags > t_ws_bytes) return 2;
  int* flag = reinterpret_cast<int*>(t_ws);
  a.exps = reinterpret_cast<int*>(t_ws + 256);
  a.flat = reinterpret_cast<float*>(t_ws + 256 + rows);
  a.mags = reinterpret_cast<signed char*>(t_ws + 256 + 2 * rows);
  norms(a, Src{}, 3, flag, s);
  // the pairs of rows once each, up to the blocks of an eighth of them
  const int step = std::max(64, 8 * cdiv(a.rb, 64));
  for (int b0 = 0; b0 < a.rb; b0 += step) {
    PlaneGemm g{};
    g.A = g.B = a.mags + (int64_t)b0 * (a.kb / 2) * 2048;
    g.mb = g.a_in = g.a_outer = std::min(step, a.rb - b0);
    g.nb = g.b_in = g.b_outer = a.rb - b0;
    g.kb = a.kb;
    g.fa = g.fb = a.flat + 32 * b0;
    g.flat = kFlat;
    g.out = flag;
    gemm_planes<true>(g, s);
  }
  int lv = 2;
  HIPCHECK(hipMemcpyAsync(&lv, flag, sizeof lv, hipMemcpyDeviceToHost, s));
  HIPCHECK(hipStreamSynchronize(s));
  return lv;
}

ModLadder::ModLadder(const double* F, int64_t row_stride, int v, int X, int level, hipStream_t s) : level_(level) {
  const int vb = cdiv(v, 32);
  const size_t eb = up256((size_t)v * vb * 32 * 4), pb = (size_t)plane_bytes((int64_t)v * vb * 32, X);
  const size_t least = (size_t)vb * vb * std::min(v, 8) * kPlanes * 1024;  // tiles of one a and 8 b
  if (level < 0 || level > 1 || !ladder_wanted(v, X) || 2 * eb + pb + least > t_ws_bytes) return;
  v_ = v;
  X_ = X;
  Src a = ladder_rows(F, row_stride, v, X);
  a.exps = exps_ = reinterpret_cast<int*>(t_ws);
  a.flat = reinterpret_cast<float*>(t_ws + eb);
  a.planes = planes_ = reinterpret_cast<signed char*>(t_ws + 2 * eb);
  held_ = 2 * eb + pb;
  norms(a, Src{}, 1, nullptr, s);
  split(a, Src{}, Level{nullptr, level_}, s);
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
        pg.lv = Level{nullptr, level_};
        pg.a_in = pg.b_in = wvb;
        pg.a_outer = pg.b_outer = vb;
        gemm_planes(pg, s);
        LadderTiles lt{reinterpret_cast<const int*>(t_ws), exps_, v, vb, wvb, blk0, a0, a1, b, nbn, row0, W, ldw};
        hipLaunchKernelGGL(mod_ladder_antisym_kernel, dim3(wvb * (wvb + 1) / 2, nbn, g1), dim3(256), 0, s, lt, level_,
                           tabs());
        HIPCHECK(hipGetLastError());
      }
    }
  }
}

// ---------------------------------------------------------------- triples
// nvir 126 per triple: FP64 products 49 us; here 22 (1.2 POP/s: 6 stages of K per tile, 70 MB
// of planes and residues moved), 10.6 for the reconstruction and 3 for the test.  Tiles of 8 x 4
// blocks, two workgroups per CU, which load 1.2 times the operand bytes, took 2.9 more, of 4 x 4
// blocks 8; with the products of a batch one after the other instead of side by side along n, the planes
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
  const double tm = P * v * 15e-6 + 2.0 * (kPlanes - 1) * up(P, 32) * up(v, 32) * 3 * up(v, 64) / 1.7e9;
  const double once = 50.0 + ((double)o * P * v + (double)o * o * v * v) * 15e-6;
  return tm + once / n < 0.9 * t64;
}

size_t ModTriples::bytes(int o, int v, int ni) {
  const int64_t P = (int64_t)v * (v - 1) / 2;
  const size_t mb = (size_t)cdiv(P, 32), nb = (size_t)cdiv(v, 32), rows = 32 * (o * mb + (size_t)o * o * nb);
  // per row norm, flatness and scale
  return 256 + rows * 16 + (size_t)mag_bytes(rows, v) + (size_t)plane_bytes(rows, v) +
         (size_t)ni * mb * nb * kPlanes * 1024;
}

ModTriples::ModTriples(void* ws, const double* V, const double* T2, int o, int v, int ni, hipStream_t s)
    : o_(o), v_(v), ni_(ni) {
  const int64_t P = (int64_t)v * (v - 1) / 2;
  mb_ = cdiv(P, 32);
  nb_ = cdiv(v, 32);
  const int kb = kblocks(v);
  const int64_t rows_a = 32LL * o * mb_, rows_b = 32LL * o * o * nb_, rows = rows_a + rows_b;
  char* w = static_cast<char*>(ws);
  int* flag = reinterpret_cast<int*>(w);
  double* norm = reinterpret_cast<double*>(w + 256);
  float* flat = reinterpret_cast<float*>(norm + rows);
  ea_ = reinterpret_cast<int*>(flat + rows);
  eb_ = ea_ + rows_a;
  signed char* mags = reinterpret_cast<signed char*>(ea_ + rows);
  pa_ = mags + mag_bytes(rows, v);
  pb_ = pa_ + plane_bytes(rows_a, v);
  out_ = pb_ + plane_bytes(rows_b, v);
  Src a{};
  a.p = V;
  a.rows = (int)rows_a;
  a.K = a.k_in = v;
  a.r_in = 32 * mb_;
  a.r_valid = (int)P;
  a.r_so = P * v;
  a.r_si = v;
  a.k_so = a.k_si = 1;
  a.kfast = 1;
  a.planes = pa_;
  a.mags = mags;
  a.exps = ea_;
  a.norm = norm;
  a.flat = flat;
  a.rb = o * mb_;
  a.kb = kb;
  Src b = a;
  b.p = T2;
  b.rows = (int)rows_b;
  b.r_in = 32 * nb_;
  b.r_valid = v;
  b.r_so = (int64_t)v * v;
  b.planes = pb_;
  b.mags = mags + mag_bytes(rows_a, v);
  b.exps = eb_;
  b.norm = norm + rows_a;
  b.flat = flat + rows_a;
  b.rb = o * o * nb_;
  norms(a, b, 1, flag, s);
  hipLaunchKernelGGL(mod_joint_exps_kernel, dim3(cdiv(32LL * mb_, 256)), dim3(256), 0, s, ea_, a.norm, a.flat, o,
                     32 * mb_);
  HIPCHECK(hipGetLastError());
  hipLaunchKernelGGL(mod_joint_exps_kernel, dim3(cdiv(32LL * nb_, 256)), dim3(256), 0, s, eb_, b.norm, b.flat, o * o,
                     32 * nb_);
  HIPCHECK(hipGetLastError());
  norms(a, b, 2, nullptr, s);
  // the level, from all triples: the scales are the largest of any i and any pair, so a triple
  // whose own integrals or amplitudes are far smaller takes the FP64 products with all others
  for (int k = 2; k < o; ++k)
    for (int j = 1; j < k; ++j) {
      PlaneGemm g = segments(0, j, k, 128);
      g.A = a.mags;
      g.B = b.mags;
      g.batch = j;
      g.fa = a.flat;
      g.fb = b.flat;
      // one bit less and three sums: 2 sqrt(3) times the rounding of one product
      g.flat = kFlat / 3.5f;
      g.out = flag;
      if (nb_ <= 4)
        launch_planes<4, 2, 4, 2, 1, 1, true, true>(g, s);
      else
        launch_planes<2, 4, 4, 2, 1, 1, true, true>(g, s);
    }
  HIPCHECK(hipMemcpyAsync(&level_, flag, sizeof level_, hipMemcpyDeviceToHost, s));
  HIPCHECK(hipStreamSynchronize(s));
  if (level_ <= 1) split(a, b, Level{nullptr, level_}, s);
}

// The products of (i, j, k) and of the i after it; unit: 16-byte units of 64 k of one row block.
PlaneGemm ModTriples::segments(int i, int j, int k, int64_t unit) const {
  const int64_t seg = (int64_t)kblocks(v_) / 2 * unit;  // per row block
  const int64_t ta = mb_ * seg, tb = nb_ * seg;          // per tile and per pair
  PlaneGemm g{};
  g.mb = g.a_in = g.a_outer = mb_;
  g.nb = g.b_in = g.b_outer = nb_;
  g.kb = 3 * kblocks(v_);
  for (int q = 0; q < kNP; ++q) g.p[q] = kMods[q];
  const int64_t at[3] = {i, j, k}, bt[3] = {(int64_t)j * o_ + k, (int64_t)k * o_ + i, (int64_t)i * o_ + j};
  const int abat[3] = {1, 0, 0}, bbat[3] = {0, 1, o_};
  for (int q = 0; q < 3; ++q) {
    g.a_seg[q] = at[q] * ta;
    g.b_seg[q] = bt[q] * tb;
    g.a_bat[q] = abat[q] * ta;
    g.b_bat[q] = bbat[q] * tb;
  }
  return g;
}

void ModTriples::rows(int i0, int ni, int j, int k, double* We, hipStream_t s) const {
  const int64_t P = (int64_t)v_ * (v_ - 1) / 2;
  const int64_t cb = (int64_t)mb_ * nb_ * kPlanes * 1024;
  const Level lv{nullptr, level_};
  for (int y = 0; y < ni; y += ni_) {
    const int n = std::min(ni_, ni - y);
    PlaneGemm g = segments(i0 + y, j, k, kPlanes * 128);
    g.A = pa_;
    g.B = pb_;
    g.C = out_;
    g.lv = lv;
    g.batch = n;
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
                       reinterpret_cast<const int*>(out_), mb_, nb_, 0, 0, ea_, eb_, c, cb / 4, P * v_, lv,
                       tabs());
    HIPCHECK(hipGetLastError());
  }
}

}  // namespace exacc
