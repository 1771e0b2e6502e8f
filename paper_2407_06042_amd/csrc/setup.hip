// Instance setup: Gram matrix, matched filter, preconditioner and packing.
//
// One workgroup per instance, float64 arithmetic, bound by latency (waits for H, the pivots of the inverse, barriers;
// launch_setup chooses how many instances share a CU against that).  Computes in the complex
// form (the real-equivalent matrices of eq. sys_model are expanded only when
// packing):
//   G = H^H H, z = H^H y, ||y||^2                      (gradient of eq. grad: grad f = -(2/sigma^2)(Gx - z))
//   M = (G + gamma I)^-1 by blocked Gauss-Jordan        (preconditioner of the Remark after Algorithm 1;
//                                                         G + gamma I is Hermitian positive definite, so no pivoting)
//   A = M G = I - gamma M,  b = M z                     (so that M grad f = -(2/sigma^2)(A x - b))
// and writes, scaled to the index units of the sampler (see common.hpp),
//   energy matrix  EG = 2 s^2 log2(e)/(tau sigma^2) * R(G),  ez = 2 s log2(e)/(tau sigma^2) * R(z)
//   proposal matrix P = alpha/(2 tau sigma^2) * R(A),       pb = alpha/(2 tau sigma^2 s) * R(b)
// where R(.) is the Re/Im-interleaved real-equivalent.  The MFMA path also
// stores two per-antenna features of the learned proposal's network, in index
// units (level step 2 s): af_{2m} = log2(sigma^2 M_mm / (8 s^2)) / 8 (variance
// of the damped LS estimate) and af_{2m+1} = log2(sigma^2 / (8 s^2 G_mm)) / 8
// (variance of one axis given the others).  On the MFMA path each
// matrix is scaled by a power of two and split into fp16 (or bf16) terms laid
// out as 16x16x32 MFMA A-operand fragments; on the float64 path it is stored
// as a dense row-major array.
#include <type_traits>

#include "common.hpp"

namespace dmala {

struct cd { double re, im; };
__device__ __forceinline__ cd cadd(cd a, cd b) { return {a.re + b.re, a.im + b.im}; }

__device__ __forceinline__ double realeq_vec(const cd* v, int n) { return (n & 1) ? v[n >> 1].im : v[n >> 1].re; }

// Hermitian matrices (G, M) are held as the 16 x 16 tiles (i, j), i <= j, of their nb x nb tile grid, tile rows of 16
// entries with entry c of row r at r ^ c: the 16 lanes that read one row, one column, or the rows of a column of an
// accumulator reach different LDS banks.
__host__ __device__ constexpr int tile_count(int nb) { return nb * (nb + 1) / 2; }
__device__ __forceinline__ int tile_index(int nb, int i, int j) { return i * (2 * nb - i - 1) / 2 + j; }

// Entry (r, c) of tile (i, j) of X, any i and j.  SUB: of I - g X instead.
template <bool SUB>
__device__ __forceinline__ cd tile_entry(const cd* X, int nb, double g, int i, int j, int r, int c) {
  cd e;
  if (i <= j) {
    e = X[tile_index(nb, i, j) * 256 + 16 * r + (r ^ c)];
  } else {
    e = X[tile_index(nb, j, i) * 256 + 16 * c + (r ^ c)];
    e.im = -e.im;
  }
  if constexpr (SUB) e = {fma(-g, e.re, i == j && r == c ? 1.0 : 0.0), -g * e.im};
  return e;
}
template <bool SUB>
__device__ __forceinline__ cd mat_entry(const cd* X, int nb, double g, int m, int m2) {
  return tile_entry<SUB>(X, nb, g, m >> 4, m2 >> 4, m & 15, m2 & 15);
}

// Value of v in lane `lane` of the wavefront (lane uniform).
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Value of v in lane P of each group of 16 lanes (row_newbcast).
template <int P>
__device__ __forceinline__ double bcast16(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + P, 0xf, 0xf, false);
}
// The 16 lanes of group G (of four), copied to every group.
template <int G>
__device__ __forceinline__ unsigned group16(unsigned v) {
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  const unsigned x = h[G >> 1];
  const auto q = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return q[G & 1];
}
template <int G>
__device__ __forceinline__ double group16(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = group16<G>((unsigned)u), hi = group16<G>((unsigned)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

typedef double d4 __attribute__((ext_vector_type(4)));

// In-place Gauss-Jordan inverse of a Hermitian positive definite 16 x 16 tile in one wavefront's registers, in the
// accumulator layout (lane l, element j: row l / 16 + 4 j, column l % 16), pivots 0 .. lim - 1 (the rest is the identity).
// Pivots are real.  Step p: column p by a lane broadcast, row p by two swaps between the lane groups, no LDS.
template <int P>
__device__ __forceinline__ void invert_step(double (&re)[4], double (&im)[4], int lane) {
  constexpr int J = P >> 2, G = P & 3;
  const double piv = readlane_f64(re[J], 16 * G + P);
  // reciprocal by Newton steps from the hardware's estimate
  double inv = __builtin_amdgcn_rcp(piv);
  inv = fma(fma(-piv, inv, 1.0), inv, inv);
  inv = fma(fma(-piv, inv, 1.0), inv, inv);
  const bool pc = (lane & 15) == P, pr = (lane >> 4) == G;
  double rr = group16<G>(re[J]), ri = group16<G>(im[J]);
  rr = pc ? inv : rr * inv;
  ri = pc ? 0.0 : ri * inv;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double cr = bcast16<P>(re[j]), ci = bcast16<P>(im[j]);
    const double br = pc ? 0.0 : re[j], bi = pc ? 0.0 : im[j];
    const double nr = fma(-cr, rr, fma(ci, ri, br)), ni = fma(-cr, ri, fma(-ci, rr, bi));
    re[j] = j == J && pr ? rr : nr;
    im[j] = j == J && pr ? ri : ni;
  }
}
template <int P>
__device__ __forceinline__ void invert_from(double (&re)[4], double (&im)[4], int lane, int lim) {
  if constexpr (P < 16) {
    if (P < lim) {
      invert_step<P>(re, im, lane);
      invert_from<P + 1>(re, im, lane, lim);
    }
  }
}

enum { kSigma2, kStep, kGamma, kCE, kCz, kCP, kCb, kYY, kNonfinite, kConsts };   // constants kept in LDS
constexpr int kRedSlots = 16;   // one per wavefront of a workgroup of up to 1024 threads

// Sum (or maximum) of v over the workgroup, returned to every thread: a butterfly within each
// wavefront, then one pass over the per-wave partials in a fixed order (two barriers).
__device__ double block_reduce(double v, double* red, bool is_max) {
  const int tid = threadIdx.x, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double u = __shfl_xor(v, o, 64);
    v = is_max ? fmax(v, u) : v + u;
  }
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  double r = red[0];
  for (int w = 1; w < nw; ++w) r = is_max ? fmax(r, red[w]) : r + red[w];
  __syncthreads();
  return r;
}

// double -> float in hardware, kept as a separate step: the compiler would otherwise
// fold the two conversions to half (or bfloat16) into one emulated in software.
__device__ __forceinline__ float via_float(double v) {
  float f = (float)v;
  asm volatile("" : "+v"(f));
  return f;
}

// Pack c * R(Y) (N x N, zero-padded to Npad) into MFMA fragments, Y = X or (SUB) I - g X.
// npass = 3 (fp16 lo, mid, hi), 2 (fp16 lo, hi) or 1 (fp16 or bf16 when bf16 != 0);
// the terms are stored in accumulation order, small terms first.
// Fragment (pass p, row tile rt, K block kb) lane l element j holds entry
// (16 rt + l%16, 16 (2 kb + j/4) + 4 (l/16) + j%4): the K order matches the
// dimensions each lane owns in the accumulator layout, so the sampler builds
// the B operand from its own registers.
// With cx != 0 the complex planes are packed instead (the sampler's complex-plane layouts): pass p,
// plane pl (real, imaginary), antenna tile at (16 rows), K block kb of 32 antennas; lane l element j
// holds plane(Y)[16 at + l%16][16 (2 kb + j/4) + 4 (l/16) + j%4] -- the same K permutation over
// antennas that the real-equivalent packing applies to real dimensions.
// The form (NPASS terms, bf16, complex planes) is a compile-time choice and the function is inlined,
// so that the element loop has no branches and X keeps its address space (LDS reads, not flat loads).
template <int NPASS, bool BF16, bool CX, bool SUB>
__device__ __forceinline__ float pack_fragments(const cd* X, int tid, int nb, double g, double c, int nt, int RT, int KB,
                                                unsigned char* dst) {
  constexpr bool cx = CX;
  // Y is Hermitian positive semidefinite (G, and A = I - gamma M, whose eigenvalues lie in [0, 1)),
  // so |Re y_ij|, |Im y_ij| <= |y_ij| <= sqrt(y_ii y_jj) <= max_i y_ii: the largest entry is the
  // largest diagonal one.  Every wavefront reads the diagonal and reduces it for itself (no barrier).
  double mx = 0.0;
  for (int i = tid & 63; i < nt; i += 64) mx = fmax(mx, fabs(mat_entry<SUB>(X, nb, g, i, i).re));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  mx *= fabs(c);
  int ex = 0;
  if (mx > 0.0) frexp(mx, &ex);
  const int e2 = 14 - ex;  // scaled max in [2^13, 2^14)
  const double sc = ldexp(c, e2);
  const int AT = RT / 2, KBX = RT / 4;
  const size_t pass_stride = cx ? (size_t)2 * AT * KBX * 1024 : (size_t)RT * KB * 1024;
  // a wavefront packs one fragment at a time (cx: both planes of it), so that the tile is uniform
  const int nfrag = cx ? AT * KBX : RT * KB;
  const int l = tid & 63, lr = l & 15, lg = l >> 4;
  for (int t = __builtin_amdgcn_readfirstlane(tid >> 6); t < nfrag; t += blockDim.x >> 6) {
    const int kb = cx ? t % KBX : t % KB, rt = cx ? t / KBX : t / KB;
    union Frag { _Float16 h[8]; __bf16 b[8]; uint4 u; };
    Frag f[cx ? 2 : 1][NPASS];
    auto put = [&](Frag (&o)[NPASS], int j, double v) {
      if constexpr (BF16) {
        o[0].b[j] = (__bf16)via_float(v);
      } else {
        const _Float16 hi = (_Float16)via_float(v);
        const double r1 = v - (double)hi;
        const _Float16 mid = (_Float16)via_float(r1);
        const double r2 = r1 - (double)mid;
        o[NPASS - 1].h[j] = hi;
        if constexpr (NPASS > 1) o[NPASS - 2].h[j] = mid;
        if constexpr (NPASS > 2) o[0].h[j] = (_Float16)via_float(r2);
      }
    };
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int ct = 2 * kb + q;   // tile column (cx), or half of one
      if constexpr (cx) {
        const int n = 16 * rt + lr;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int n2 = 16 * ct + 4 * lg + j;
          cd e = {0.0, 0.0};
          if (rt < nb && ct < nb) e = tile_entry<SUB>(X, nb, g, rt, ct, lr, 4 * lg + j);
          const bool ok = n < nt && n2 < nt;
          put(f[0], 4 * q + j, ok ? sc * e.re : 0.0);
          put(f[1], 4 * q + j, ok ? sc * e.im : 0.0);
        }
      } else {
        const int m = 8 * rt + (lr >> 1);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int m2 = 8 * ct + 2 * lg + j;
          cd e = {0.0, 0.0};
          if ((rt >> 1) < nb && (ct >> 1) < nb) e = tile_entry<SUB>(X, nb, g, rt >> 1, ct >> 1, m & 15, m2 & 15);
          const bool ok = m < nt && m2 < nt;
          const double vr = ok ? sc * e.re : 0.0, vi = ok ? sc * e.im : 0.0;
          // real-equivalent rows (Re, Im): [re -im; im re]
          put(f[0], 4 * q + 2 * j, (lr & 1) ? vi : vr);
          put(f[0], 4 * q + 2 * j + 1, (lr & 1) ? vr : -vi);
        }
      }
    }
#pragma unroll
    for (int pl = 0; pl < (cx ? 2 : 1); ++pl) {
      // cx: plane, antenna tile, K block
      unsigned char* o = dst + (size_t)(cx ? pl * nfrag + t : t) * 1024 + l * 16;
#pragma unroll
      for (int ps = 0; ps < NPASS; ++ps) *(uint4*)(o + ps * pass_stride) = f[pl][ps].u;
    }
  }
  return (float)ldexp(1.0, -e2);
}

// Dense row-major double copy of c * R(Y), zero-padded to Npad x Npad.
template <bool SUB>
__device__ void pack_dense(const cd* X, int nb, double g, double c, int N, int Npad, double* dst) {
  for (int e = threadIdx.x; e < Npad * Npad; e += blockDim.x) {
    const int n = e / Npad, n2 = e % Npad, p = n & 1, p2 = n2 & 1;
    double v = 0.0;
    if (n < N && n2 < N) {
      const cd x = mat_entry<SUB>(X, nb, g, n >> 1, n2 >> 1);
      v = c * (p == p2 ? x.re : (p == 0 ? -x.im : x.im));
    }
    dst[e] = v;
  }
}

// Sum of eight partials that P consecutive lanes hold, SP each (partial i + p P in lane i): pairs of distance 4,
// then 2, then 1, whatever P (additions commute bit for bit).
template <int P, int SP>
__device__ __forceinline__ cd sum8(const cd (&v)[SP]) {
  cd s = v[0];
  if constexpr (SP == 2) s = cadd(s, v[1]);
#pragma unroll
  for (int o = P >> 1; o > 0; o >>= 1) {
    s.re += __shfl_xor(s.re, o, 64);
    s.im += __shfl_xor(s.im, o, 64);
  }
  return s;
}

// LDS: a region for the matrix's tiles, the staged chunk of H (before them) and the panels of the Gauss-Jordan sweep
// (between the two packings), then z and b, then kRedSlots partials of block_reduce and
// the instance's constants.
__host__ __device__ constexpr int setup_chunk(int rmax) { return rmax <= 32 ? 16 : 32; }
inline size_t setup_lds_bytes(int nt, int rmax) {
  const int nb = (nt + 15) / 16;
  size_t region = (size_t)tile_count(nb) * 4096;
  const size_t stage = ((size_t)setup_chunk(rmax) * (nt + 1) + 16) * sizeof(cd), panels = nb > 1 ? (3 * (size_t)(nb - 1) + 1) * 4096 : 0;
  region = stage > region ? stage : region;
  region = panels > region ? panels : region;
  return region + 2 * (size_t)nt * sizeof(cd) + (kRedSlots + kConsts) * sizeof(double);
}

// RMAX: largest number of antennas.
template <typename TIn, int BS, int RMAX>
__device__ __forceinline__ void setup_body(const SetupArgs& a, const int b) {
  int tid = threadIdx.x;
  // (opaque: a persistent launch's loop would keep every lane offset below in registers from item to item)
  asm volatile("" : "+v"(tid));
  const int nt = a.nt, nr = a.nr, N = a.N, Npad = a.Npad;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = (nt + 15) >> 4;
  const InstDesc dsc = inst_desc(a.desc, b, nt, nr, a.Q * a.Q, 1);
  const TIn* Hg = (const TIn*)a.H + 2 * dsc.h_off;
  const TIn* y = (const TIn*)a.y + 2 * dsc.y_off;
  extern __shared__ double smem_setup[];
  cd* W = (cd*)smem_setup;
  cd* z;
  {
    constexpr int kIC = setup_chunk(RMAX);
    int region = tile_count(nb) * 256;
    const int stage = kIC * (nt + 1) + 16, panels = nb > 1 ? (3 * (nb - 1) + 1) * 256 : 0;
    region = stage > region ? stage : region;
    region = panels > region ? panels : region;
    z = W + region;
  }
  cd* bv = z + nt;
  double* red = (double*)(bv + nt);   // kRedSlots partials of block_reduce
  double* cst = red + kRedSlots;      // the instance's constants (kept here, not in 24 registers through every phase)
  unsigned char* blk = a.ws_inst + (size_t)b * a.inst_stride;

  const int Q = a.Q, M = Q * Q;
  // G = H^H H and z = H^H y.  H is staged in LDS in chunks of receive antennas,
  // transposed with a padded row whose last entry holds y (Ht[i][m], Ht[i][nt] = y_i).
  // G on the matrix cores: with X = Re + i Im of the staged H^T (nt x nr),
  //   Re G = Re Re^T + Im Im^T,   Im G = Re Im^T - Im Re^T,
  // four float64 16x16x4 MFMAs per 16 x 16 tile and 4 receive antennas; each wave accumulates the tiles (i <= j)
  // assigned to it in registers across the chunks; they stay there for the inverse.  Rows past nt - 1 read whatever
  // follows in the staged rows: they only reach tile rows and columns past nt - 1, which are replaced.  z on the vector
  // ALUs, as 8 partial sums over every eighth receive antenna, added in pairs of distance 4, 2, 1: P = BS / RMAX
  // consecutive threads share an antenna m and take SP = 8 / P of them each, so that the sums and their
  // order are the same for every workgroup size (as for b = M z below), and an instance's packed block is the same bytes
  // in any launch and in a plan.
  constexpr int NW = BS / 64;
  constexpr int kNT = (RMAX + 15) / 16;                         // tile rows at nt = RMAX
  constexpr int kTPW = (kNT * (kNT + 1) / 2 + NW - 1) / NW;     // tiles per wave
  constexpr int P = BS / RMAX;
  constexpr int SP = 8 / P;
  static_assert(P * SP == 8 && SP <= 2, "eight partial sums, the threads of an antenna in one wavefront");
  const int ntiles = tile_count(nb);
  int m0[kTPW], m1[kTPW];
  d4 gre[kTPW], gim[kTPW];
  double nonfinite = 0.0;
  double yy = 0.0;
  {
    constexpr int kIC = setup_chunk(RMAX);
    const int ld = nt + 1;
    cd* Ht = W;   // kIC x ld, then 16 spare entries; the tiles are written after the last read
#pragma unroll
    for (int q = 0; q < kTPW; ++q) {
      int t = wv + q * NW, tr = 0;
      if (t >= ntiles) t = 0;
      while (t >= nb - tr) { t -= nb - tr; ++tr; }
      m0[q] = tr;
      m1[q] = tr + t;
      gre[q] = d4{0.0, 0.0, 0.0, 0.0};
      gim[q] = d4{0.0, 0.0, 0.0, 0.0};
    }
    const int zm = tid / P, zp = tid % P;
    cd zacc[SP];
#pragma unroll
    for (int p = 0; p < SP; ++p) zacc[p] = {0.0, 0.0};
    // The chunk of receive antennas i0 .. i0 + kIC - 1 is loaded into registers (every load
    // issued before the first is waited for), then stored to LDS; the next chunk's loads are
    // issued before this chunk's products, so that they overlap.  Element e of a chunk:
    // receive antenna i0 + e % kIC, column e / kIC (column nt: y).
    constexpr int kSt = (kIC * (RMAX + 1) + BS - 1) / BS;
    TIn hv[kSt][2];
    auto load_chunk = [&](int i0) {
      const int ic = nr - i0 < kIC ? nr - i0 : kIC;
#pragma unroll
      for (int k = 0; k < kSt; ++k) {
        const int e = tid + k * BS, mm = e / kIC, ii = e % kIC;
        if (mm <= nt && ii < ic) {
          const TIn* src = mm < nt ? Hg + 2 * ((size_t)mm * nr + i0 + ii) : y + 2 * (i0 + ii);
          hv[k][0] = src[0];
          hv[k][1] = src[1];
        }
      }
    };
    load_chunk(0);
    // (the constants while the first loads are on their way)
    if (tid == 0) {
      const double sigma2 = a.sigma2 ? (double)((const TIn*)a.sigma2)[dsc.orig] : a.sigma2_val;
      const double s = sqrt(3.0 / (2.0 * (M - 1))), tau = a.tau, alpha = a.alpha_mult * sigma2;
      cst[kSigma2] = sigma2;
      cst[kStep] = s;
      cst[kGamma] = a.gamma_mult * sigma2 / (2.0 * s * s);
      cst[kCE] = 2.0 * s * s * kLog2e / (tau * sigma2);
      cst[kCz] = 2.0 * s * kLog2e / (tau * sigma2);
      cst[kCP] = alpha / (2.0 * tau * sigma2);
      cst[kCb] = alpha / (2.0 * tau * sigma2 * s);
    }
    for (int i0 = 0; i0 < nr; i0 += kIC) {
      const int ic = nr - i0 < kIC ? nr - i0 : kIC;
#pragma unroll
      for (int k = 0; k < kSt; ++k) {
        const int e = tid + k * BS, mm = e / kIC, ii = e % kIC;
        // (receive antennas past the last, up to the MFMA's four: zero)
        if (mm <= nt && ii < ((ic + 3) & ~3)) Ht[ii * ld + mm] = ii < ic ? cd{(double)hv[k][0], (double)hv[k][1]} : cd{0.0, 0.0};
      }
      __syncthreads();
      if (i0 + kIC < nr) load_chunk(i0 + kIC);
      // |y|^2 from the staged y
      if (tid < ic) {
        const cd yv = Ht[tid * ld + nt];
        yy = fma(yv.re, yv.re, fma(yv.im, yv.im, yy));
      }
#pragma unroll
      for (int q = 0; q < kTPW; ++q) {
        if (wv + q * NW < ntiles) {
          const cd* pa = Ht + (lane >> 4) * ld + 16 * m0[q] + (lane & 15);
          const cd* pb = Ht + (lane >> 4) * ld + 16 * m1[q] + (lane & 15);
#pragma unroll 4
          for (int kk = 0; kk < ic; kk += 4) {
            const cd va = pa[kk * ld], vb = pb[kk * ld];
            gre[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(va.re, vb.re, gre[q], 0, 0, 0);
            gim[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(va.re, vb.im, gim[q], 0, 0, 0);
            gre[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(va.im, vb.im, gre[q], 0, 0, 0);
            gim[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(-va.im, vb.re, gim[q], 0, 0, 0);
          }
        }
      }
      if (zm < nt) {
        for (int i8 = zp; i8 < ic; i8 += 8) {
#pragma unroll
          for (int p = 0; p < SP; ++p) {
            const int ii = i8 + p * P;
            if (ii < ic) {
              const cd h = Ht[ii * ld + zm], yv = Ht[ii * ld + nt];
              zacc[p].re = fma(h.re, yv.re, fma(h.im, yv.im, zacc[p].re));
              zacc[p].im = fma(h.re, yv.im, fma(-h.im, yv.re, zacc[p].im));
            }
          }
        }
      }
      __syncthreads();
    }
    const cd zs = sum8<P, SP>(zacc);
    if (zm < nt && zp == 0) {
      z[zm] = zs;
      if (!isfinite(zs.re) || !isfinite(zs.im)) nonfinite = 1.0;
    }
    // lane l, register j of a tile's accumulator: row l / 16 + 4 j, column l % 16
    const double gamma = cst[kGamma];
#pragma unroll
    for (int q = 0; q < kTPW; ++q) {
      if (wv + q * NW < ntiles) {
        const int c = lane & 15, col = 16 * m1[q] + c;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = (lane >> 4) + 4 * j, row = 16 * m0[q] + r;
          const bool in = row < nt && col < nt;
          const double re = in ? gre[q][j] : 0.0, im = in ? gim[q][j] : 0.0;
          W[(wv + q * NW) * 256 + 16 * r + (r ^ c)] = {re, im};
          if (!isfinite(re) || !isfinite(im)) nonfinite = 1.0;
          // from here on G + gamma I, continued by the identity
          gre[q][j] = re + (row == col ? (in ? gamma : 1.0) : 0.0);
          gim[q][j] = im;
        }
      }
    }
  }
  __syncthreads();
  yy = block_reduce(yy, red, false);
  {
    const double sigma2 = cst[kSigma2];
    if (!isfinite(yy) || !(sigma2 > 0.0) || !isfinite(sigma2)) nonfinite = 1.0;
  }
  nonfinite = block_reduce(nonfinite, red, true);
  if (tid == 0) { cst[kYY] = yy; cst[kNonfinite] = nonfinite; }

  const int npP = p_passes(a.pm);
  unsigned char* frag = blk + kParamBytes;
  // bytes of one split term of a packed matrix (real-equivalent, or complex planes: half of it)
  const size_t pass_bytes = a.cx ? (size_t)a.RT * a.RT / 4 * 1024 : (size_t)a.RT * a.KB * 1024;
  float scaleE = 1.0f, scaleP = 1.0f;

  // energy matrix and vector
  {
  const double cE = cst[kCE], cz = cst[kCz];
  if (a.fp64) {
    double* EGd = (double*)(blk + kParamBytes) + (size_t)Npad * Npad;
    pack_dense<false>(W, nb, 0.0, cE, N, Npad, EGd);
    double* ezd = (double*)(blk + kParamBytes) + 2 * (size_t)Npad * Npad + Npad;
    for (int n = tid; n < Npad; n += blockDim.x) ezd[n] = n < N ? cz * realeq_vec(z, n) : 0.0;
  } else {
    unsigned char* fe = frag + (size_t)npP * pass_bytes;
    scaleE = a.cx ? pack_fragments<kEPasses, false, true, false>(W, tid, nb, 0.0, cE, nt, a.RT, a.KB, fe)
                  : pack_fragments<kEPasses, false, false, false>(W, tid, nb, 0.0, cE, nt, a.RT, a.KB, fe);
    float* ezf = (float*)(frag + (size_t)(npP + kEPasses) * pass_bytes) + Npad;
    for (int n = tid; n < Npad; n += blockDim.x) ezf[n] = n < N ? (float)(cz * realeq_vec(z, n)) : 0.0f;
    float* afv = ezf + Npad;
    for (int n = tid; n < Npad; n += blockDim.x) {
      const int m = n >> 1;
      const double s = cst[kStep], sigma2 = cst[kSigma2];
      afv[n] = (n < N && (n & 1)) ? (float)(log2(sigma2 / (8.0 * s * s * mat_entry<false>(W, nb, 0.0, m, m).re)) / 8.0) : 0.0f;
    }
  }
  }
  __syncthreads();

  if (!a.naive) {
    // M = (G + gamma I)^-1 by Gauss-Jordan over 16 x 16 blocks.  The tiles (i <= j) stay in the accumulators of their
    // waves; the matrix of a step is Hermitian up to the sign of the tiles between a block that has been a pivot and
    // one that has not.  Step k:
    //   C_j = tile (k, j) of every other block j to LDS; the pivot tile's wave inverts it, D;
    //   R_j = D C_j;
    //   tile (i, j) -= W_ik R_j with W_ik = C_i^H, or -C_i^H if i has been a pivot; tile (k, j) = R_j;
    //   tile (j, k) = R_j^H; tile (k, k) = D.
    // A stored tile serves both MFMA operands as it lies: entry (l / 16 + 4 s, l % 16) is lane l's operand B of K step s,
    // and, conjugated, its operand A of the Hermitian transpose.  C alternates between two buffers, so that two
    // barriers order a step, and the next pivot's wave starts its inverse while others still update.
    // Bound by the serial pivots of each block's inverse (about 600 clocks each, no barrier).  Against one or two pivots per
    // barrier with the matrix in vector registers, clocks of an instance alone on its CU: 32 antennas 31k -> 25k, 64
    // 89k -> 60k, 128 405k -> 183k, with half of the matrix products and 44 KiB of LDS instead of 75 at 64.
    cd* panC = W;
    cd* panR = W + 2 * (nb - 1) * 256;
    cd* panD = panR + (nb - 1) * 256;
    const int lg = lane >> 4, lc = lane & 15;
#pragma unroll 1
    for (int k = 0; k < nb; ++k) {
      cd* C = panC + (k & 1) * (nb - 1) * 256;
      auto slot = [&](int j) { return (j - (j > k ? 1 : 0)) * 256; };
      double dr[4], di[4];
      bool mine = false;
#pragma unroll
      for (int q = 0; q < kTPW; ++q) {
        if (wv + q * NW >= ntiles) continue;
        if (m0[q] == k && m1[q] == k) {
          mine = true;
#pragma unroll
          for (int j = 0; j < 4; ++j) { dr[j] = gre[q][j]; di[j] = gim[q][j]; }
        } else if (m0[q] == k) {
          cd* o = C + slot(m1[q]);
#pragma unroll
          for (int j = 0; j < 4; ++j) { const int r = lg + 4 * j; o[16 * r + (r ^ lc)] = {gre[q][j], gim[q][j]}; }
        } else if (m1[q] == k) {
          cd* o = C + slot(m0[q]);
#pragma unroll
          for (int j = 0; j < 4; ++j) { const int r = lg + 4 * j; o[16 * lc + (r ^ lc)] = {-gre[q][j], gim[q][j]}; }
        }
      }
      if (mine) {
        invert_from<0>(dr, di, lane, nt - 16 * k);
        if (nb > 1) {
#pragma unroll
          for (int j = 0; j < 4; ++j) { const int r = lg + 4 * j; panD[16 * r + (r ^ lc)] = {dr[j], di[j]}; }
        }
#pragma unroll
        for (int q = 0; q < kTPW; ++q)
          if (m0[q] == k && m1[q] == k && wv + q * NW < ntiles) {
#pragma unroll
            for (int j = 0; j < 4; ++j) { gre[q][j] = dr[j]; gim[q][j] = di[j]; }
          }
      }
      if (nb == 1) break;
      __syncthreads();
      for (int u = wv; u < 2 * (nb - 1); u += NW) {
        // real (even u) or imaginary part of a panel tile
        const cd* c = C + (u >> 1) * 256;
        const bool ip = u & 1;
        d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = lg + 4 * j, e = 16 * r + (r ^ lc);
          const cd d = panD[e], x = c[e];
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(d.re, ip ? x.im : x.re, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ip ? -d.im : d.im, ip ? x.re : x.im, acc, 0, 0, 0);
        }
        double* o = (double*)(panR + (u >> 1) * 256) + (ip ? 1 : 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) { const int r = lg + 4 * j; o[2 * (16 * r + (r ^ lc))] = acc[j]; }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kTPW; ++q) {
        if (wv + q * NW >= ntiles || (m0[q] == k && m1[q] == k)) continue;
        if (m0[q] != k && m1[q] != k) {
          const cd* c = C + slot(m0[q]);
          const cd* x = panR + slot(m1[q]);
          const double sg = m0[q] < k ? 1.0 : -1.0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int r = lg + 4 * j, e = 16 * r + (r ^ lc);
            const double cr = sg * c[e].re, ci = sg * c[e].im;
            const cd v = x[e];
            gre[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(cr, v.re, gre[q], 0, 0, 0);
            gim[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(cr, v.im, gim[q], 0, 0, 0);
            gre[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(ci, v.im, gre[q], 0, 0, 0);
            gim[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ci, v.re, gim[q], 0, 0, 0);
          }
        } else if (m0[q] == k) {
          const cd* x = panR + slot(m1[q]);
#pragma unroll
          for (int j = 0; j < 4; ++j) { const int r = lg + 4 * j; const cd v = x[16 * r + (r ^ lc)]; gre[q][j] = v.re; gim[q][j] = v.im; }
        } else {
          const cd* x = panR + slot(m0[q]);
#pragma unroll
          for (int j = 0; j < 4; ++j) { const int r = lg + 4 * j; const cd v = x[16 * lc + (r ^ lc)]; gre[q][j] = v.re; gim[q][j] = -v.im; }
        }
      }
    }
    __syncthreads();   // (the panels are read)
#pragma unroll
    for (int q = 0; q < kTPW; ++q)
      if (wv + q * NW < ntiles) {
#pragma unroll
        for (int j = 0; j < 4; ++j) { const int r = lg + 4 * j; W[(wv + q * NW) * 256 + 16 * r + (r ^ lc)] = {gre[q][j], gim[q][j]}; }
      }
    __syncthreads();
    // b = M z (eight partial sums, as z's) and the preconditioned variance feature from M's diagonal
    float* afv = (float*)(frag + (size_t)(npP + kEPasses) * pass_bytes) + 2 * Npad;
    {
      const int m = tid / P, q = tid % P;
      if (m < nt) {
        cd bp[SP];
#pragma unroll
        for (int p = 0; p < SP; ++p) bp[p] = {0.0, 0.0};
        for (int j8 = q; j8 < nt; j8 += 8) {
#pragma unroll
          for (int p = 0; p < SP; ++p) {
            const int j = j8 + p * P;
            if (j < nt) {
              const cd e = mat_entry<false>(W, nb, 0.0, m, j), v = z[j];
              bp[p].re = fma(e.re, v.re, fma(-e.im, v.im, bp[p].re));
              bp[p].im = fma(e.re, v.im, fma(e.im, v.re, bp[p].im));
            }
          }
        }
        const cd bs = sum8<P, SP>(bp);
        if (q == 0) {
          bv[m] = bs;
          const double s = cst[kStep], sigma2 = cst[kSigma2];
          if (!a.fp64) afv[2 * m] = (float)(log2(sigma2 * mat_entry<false>(W, nb, 0.0, m, m).re / (8.0 * s * s)) / 8.0);
        }
      }
    }
    __syncthreads();
    const double gamma = cst[kGamma], cP = cst[kCP], cb = cst[kCb];
    if (a.fp64) {
      pack_dense<true>(W, nb, gamma, cP, N, Npad, (double*)(blk + kParamBytes));
      double* pbd = (double*)(blk + kParamBytes) + 2 * (size_t)Npad * Npad;
      for (int n = tid; n < Npad; n += blockDim.x) pbd[n] = n < N ? cb * realeq_vec(bv, n) : 0.0;
    } else {
      auto packP = [&](auto CXC) {
        constexpr bool C = decltype(CXC)::value;
        if (a.pm == PM_BF16X1) return pack_fragments<1, true, C, true>(W, tid, nb, gamma, cP, nt, a.RT, a.KB, frag);
        if (npP == 2) return pack_fragments<2, false, C, true>(W, tid, nb, gamma, cP, nt, a.RT, a.KB, frag);
        return pack_fragments<1, false, C, true>(W, tid, nb, gamma, cP, nt, a.RT, a.KB, frag);
      };
      scaleP = a.cx ? packP(std::true_type{}) : packP(std::false_type{});
      float* pbf = (float*)(frag + (size_t)(npP + kEPasses) * pass_bytes);
      for (int n = tid; n < Npad; n += blockDim.x) pbf[n] = n < N ? (float)(cb * realeq_vec(bv, n)) : 0.0f;
    }
  } else if (a.fp64) {
    double* Pd = (double*)(blk + kParamBytes);
    for (int e = tid; e < Npad * Npad; e += blockDim.x) Pd[e] = 0.0;
    double* pbd = Pd + 2 * (size_t)Npad * Npad;
    for (int n = tid; n < Npad; n += blockDim.x) pbd[n] = 0.0;
  }

  if (tid == 0) {
    InstParams ip;
    const double sigma2 = cst[kSigma2], s = cst[kStep], tau = a.tau, alpha = a.alpha_mult * sigma2;
    const double beta = a.naive ? 1.0 : a.beta_mult * s * s / sigma2;
    ip.yy = cst[kYY];
    ip.eunit = tau * sigma2 / kLog2e;
    ip.kL = kLog2e * 2.0 * s * s / (alpha * beta);
    ip.rho = alpha / (4.0 * s * s * kLog2e);
    ip.sigma2 = sigma2;
    ip.s = s;
    ip.tau = tau;
    ip.scaleP = scaleP;
    ip.scaleE = scaleE;
    ip.nonfinite = cst[kNonfinite] > 0.0 ? 1 : 0;
    ip.pad_[0] = ip.pad_[1] = ip.pad_[2] = 0;
    *(InstParams*)blk = ip;
    if (a.status) a.status[dsc.orig] = ip.nonfinite ? kStatusNonfinite : 0;
  }
}

// Direct launch (PERS false): instance blockIdx.x.  Persistent launch: items from the list, each
// with its class's arguments.
template <typename TIn, int BS, int RMAX, bool PERS = false>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(PERS ? 2 : (BS == 256 && RMAX > 32 ? 3 : 4))))
void setup_kernel(SetupArgs a, Persist p) {
  if constexpr (!PERS) {
    setup_body<TIn, BS, RMAX>(a, blockIdx.x);
  } else {
    extern __shared__ double smem_setup[];
    for (;;) {
      const int it = persist_take(p, (unsigned char*)smem_setup);
      if (it >= p.n_items) break;
      const WorkItem w = p.items[it];
      SetupArgs ca = ((const SetupArgs*)p.cls)[__builtin_amdgcn_readfirstlane(w.cls)];
      // the sizes in scalar registers (loaded through a pointer they take vector registers)
      ca.nt = __builtin_amdgcn_readfirstlane(ca.nt);
      ca.nr = __builtin_amdgcn_readfirstlane(ca.nr);
      ca.Q = __builtin_amdgcn_readfirstlane(ca.Q);
      ca.N = __builtin_amdgcn_readfirstlane(ca.N);
      ca.Npad = __builtin_amdgcn_readfirstlane(ca.Npad);
      ca.RT = __builtin_amdgcn_readfirstlane(ca.RT);
      ca.KB = __builtin_amdgcn_readfirstlane(ca.KB);
      ca.fp64 = __builtin_amdgcn_readfirstlane(ca.fp64);
      ca.pm = __builtin_amdgcn_readfirstlane(ca.pm);
      ca.naive = __builtin_amdgcn_readfirstlane(ca.naive);
      ca.cx = __builtin_amdgcn_readfirstlane(ca.cx);
      setup_body<TIn, BS, RMAX>(ca, __builtin_amdgcn_readfirstlane(w.inst));
    }
    persist_done(p);
  }
}

template <int BS, int RMAX, bool PERS = false>
hipError_t launch_setup_bs(const SetupArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  if (a.nt > RMAX) return hipErrorInvalidValue;
  const size_t lds = setup_lds_bytes(a.nt, RMAX);
  void (*k)(SetupArgs, Persist);
  k = a.fp64 ? setup_kernel<double, BS, RMAX, PERS> : setup_kernel<float, BS, RMAX, PERS>;
  if (cfg) {
    cfg->k = (const void*)k;
    cfg->threads = BS;
    cfg->lds = lds;
    cfg->gx = a.n_inst;
    cfg->gy = 1;
    return hipSuccess;
  }
  // a persistent launch keeps one more aligned word after the body's LDS (the item broadcast)
  const size_t lds_run = p ? ((p->lds_off + 4 + 15) & ~(size_t)15) : lds;
  if (lds_run > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_run);
    if (e != hipSuccess) return e;
  }
  if (p) hipLaunchKernelGGL(k, dim3(gn), dim3(BS), lds_run, s, a, *p);
  else hipLaunchKernelGGL(k, dim3(a.n_inst), dim3(BS), lds, s, a, Persist{});
  return hipGetLastError();
}

// Threads per workgroup.  One instance is a chain of latencies (loads, pivots, barriers), so a launch of more instances
// than the larger workgroups hold at once takes smaller ones, more of them per CU, and the others the larger ones,
// which end sooner.  us, larger / smaller workgroups: 8x8, 8192 instances 73 / 52, 1000 of 4x4 16.2 / 17.8; 32x32, 4096
// instances 142 / 110; 64x64, 2048 instances 275 / 240, one 48 / 57.
// Persistent launches keep their arguments in registers beside the body's and share the GPU with other classes: two
// sizes, of at most 512 threads, so that nothing spills.
hipError_t launch_setup(const SetupArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  if (p || cfg) {
    if (a.nt <= 32) return launch_setup_bs<128, 32, true>(a, s, p, gn, cfg);
    if (a.nt <= 64) return launch_setup_bs<256, 64, true>(a, s, p, gn, cfg);
    return launch_setup_bs<512, 128, true>(a, s, p, gn, cfg);
  }
  if (a.nt <= 16 && a.n_inst > 1024) return launch_setup_bs<64, 16>(a, s, p, gn, cfg);
  if (a.nt <= 32) return a.n_inst > 1024 ? launch_setup_bs<128, 32>(a, s, p, gn, cfg) : launch_setup_bs<256, 32>(a, s, p, gn, cfg);
  if (a.nt <= 64) return a.n_inst > 512 ? launch_setup_bs<256, 64>(a, s, p, gn, cfg) : launch_setup_bs<512, 64>(a, s, p, gn, cfg);
  return launch_setup_bs<1024, 128>(a, s, p, gn, cfg);
}

}  // namespace dmala
