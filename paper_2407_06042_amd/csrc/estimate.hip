// Estimators on the final samples (Algorithm 2, steps after sampling).
//
// One workgroup per instance.  For every chain's final state x^[s] (the sample
// list of Section IV-A) the kernel recomputes the residual r = y - H x from the
// inputs, E = ||r||^2, f = -E/sigma^2 and c = H^H r.  Moving coordinate n of a
// sample from level k_n to level k (e = k - k_n, real step d = 2 s e) changes f by
//     delta(e) = (2 d c_n - d^2 ||h_m||^2) / sigma^2 = e (a_n - a2_m e),
//     a_n = 4 s c_n / sigma^2,  a2_m = 4 s^2 ||h_m||^2 / sigma^2,
// which gives, per bit (eq. llr_is in the log-sum-exp form of eq. llr_simple,
// F(a) = log(1 + e^a) evaluated exactly)
//     L = LSE_s[((tau-1)/tau) F+ - F(-g)] - LSE_s[((tau-1)/tau) F- - F(g)],  g = (F+ - F-)/tau,
// and per antenna and point a = (kI, kQ) the symbol-level IS estimate
//     p(a) propto sum_s pi_a(a | x^[s]_-m) exp(((tau-1)/tau) f(x^[s]_{m<-a}))
//          = sum_s exp(((tau-1)/tau) f_s + delta_I(kI) + delta_Q(kQ) - lse_I - lse_Q),
// lse_{I,Q} = log sum_k exp(delta_{I,Q}(k)/tau): the I/Q parts separate because
// the real-equivalent columns of one antenna are orthogonal.  The hard decision
// is the chain whose tracked best state has the smallest recomputed energy.
//
// Chains are processed in chunks staged in LDS; every output keeps a running
// log-sum-exp in registers across chunks.  A thread owns (antenna, kI) and the
// Q points (kI, 0..Q-1), so the inner loop has Q independent accumulators.
#include "common.hpp"

namespace dmala {

__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
__device__ __forceinline__ float fex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float flg2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ double fex2(double x) { return exp2(x); }
__device__ __forceinline__ double flg2(double x) { return log2(x); }
__device__ __forceinline__ float flog(float x) { return __builtin_amdgcn_logf(x) * 0.6931471805599453f; }
__device__ __forceinline__ double fexp(double x) { return exp(x); }
__device__ __forceinline__ double flog(double x) { return log(x); }

template <typename R>
struct OnlineLse {
  R mx, sum;
  __device__ OnlineLse() : mx(-INFINITY), sum(R(0)) {}
  __device__ __forceinline__ void add(R v) {  // branch-free: both lanes of a divergent update cost the same
    const R m2 = fmax(v, mx);
    sum = sum * fexp(mx - m2) + fexp(v - m2);
    mx = m2;
  }
  __device__ R value() const { return mx + flog(sum); }
};

constexpr int kLlrPerThread = 4;  // bits per instance <= 128 antennas x 8 bits = 4 x 256 threads

// Exchanges inside groups of Q consecutive lanes (Q <= 16, so a group never straddles a 32-lane
// half) by ds_swizzle in its bit mode: lane j reads lane ((j & and) | or) ^ xor of its half, an
// immediate pattern, so no lane-address registers are needed.
template <int PAT> __device__ __forceinline__ float swz(float x) {
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), PAT));
}
template <int PAT> __device__ __forceinline__ double swz(double x) {
  const long long u = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_ds_swizzle((int)u, PAT), hi = __builtin_amdgcn_ds_swizzle((int)(u >> 32), PAT);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// x of every member of the lane's group, in member order
template <int Q, int K = 0, typename R> __device__ __forceinline__ void group_gather(R x, R (&out)[Q]) {
  out[K] = swz<(0x1F & ~(Q - 1)) | (K << 5)>(x);
  if constexpr (K + 1 < Q) group_gather<Q, K + 1>(x, out);
}
// the largest x of the group (a butterfly)
template <int Q, int O = 1, typename R> __device__ __forceinline__ R group_max(R x) {
  if constexpr (O < Q) return group_max<Q, 2 * O>(fmax(x, swz<0x1F | (O << 10)>(x)));
  else return x;
}

// Per (chain, antenna) values staged in LDS.
template <typename R>
struct CM {
  R aI, aQ, base;  // base = ((tau-1)/tau) f_s - lse_I - lse_Q
  int kI, kQ;
};

// The float64 path (at most 32 antennas, 256 threads).
template <int Q, bool SH>
__device__ __forceinline__ void estimate_d(const EstArgs& a, const int b) {
  using R = double;
  constexpr int M = Q * Q;
  constexpr int NB = Q == 2 ? 1 : (Q == 4 ? 2 : (Q == 8 ? 3 : 4));
  const int tid = threadIdx.x, nth = blockDim.x;
  const int nt = a.nt, nr = a.nr, C = a.C, Npad = a.Npad, N = a.N, CH = a.chunk;
  const InstDesc dsc = inst_desc(a.desc, b, nt, nr, M, C);
  const R* Hg = (const R*)a.H + 2 * dsc.h_off;
  const R* y = (const R*)a.y + 2 * dsc.y_off;
  const InstParams ip = *(const InstParams*)(a.ws_inst + (size_t)b * a.inst_stride);
  if (ip.nonfinite) {
    // a flagged instance (see the setup kernel): no samples to estimate from; symbols -1,
    // every other output NaN (the whole workgroup leaves here)
    const float nan = __builtin_nanf("");
    for (int m = tid; m < nt; m += nth)
      if (a.symbols) a.symbols[dsc.sym_off + m] = -1;
    for (int e = tid; e < nt * M; e += nth) {
      if (a.marginals) a.marginals[dsc.marg_off + e] = nan;
      if (a.marginals_mc) a.marginals_mc[dsc.marg_off + e] = nan;
    }
    for (int e = tid; e < nt * 2 * NB; e += nth)
      if (a.llrs) a.llrs[dsc.llr_off + e] = nan;
    if (a.best_energy && tid == 0) a.best_energy[dsc.orig] = nan;
    return;
  }
  const R s = (R)ip.s, tau = (R)ip.tau;
  const R inv_s2 = R(1) / (R)ip.sigma2, inv_tau = R(1) / tau;
  const R cw = (tau - R(1)) * inv_tau;
  const StateOff so = state_offsets(a.Cpad, Npad);
  const unsigned char* st = a.ws_state + (size_t)b * a.state_stride;
  const int8_t* K = (const int8_t*)(st + so.k);
  const int8_t* Kb = (const int8_t*)(st + so.kbest);

  extern __shared__ __attribute__((aligned(16))) unsigned char esm[];
  CM<R>* cm = (CM<R>*)esm;                           // CH x nt
  const int lrs = 2 * nr + 2;                        // residual row stride (one pad entry: chain-strided reads
                                                     // of one column hit distinct banks)
  R* rs = (R*)(cm + (size_t)CH * nt);                // CH x nr complex residuals of the final states
  R* rb2 = rs + (size_t)CH * lrs;                    // CH x nr |residual|^2 of the best states
  R* fs = rb2 + (size_t)CH * nr;                     // CH
  R* ebs = fs + CH;                                  // CH
  R* a2 = ebs + CH;                                  // nt
  R* ys = a2 + nt;                                   // nr complex: y + s (Q-1) sum_m h_m
  int8_t* Ks = (int8_t*)(ys + 2 * nr);               // CH x N
  int8_t* Kbs = Ks + (size_t)CH * N;                 // CH x N
  __shared__ R best_e;
  __shared__ int best_c;
  __shared__ unsigned char dupf[1024];   // list LLRs: chain repeats an earlier chain's final state
  // H is read many times per element: stage it in LDS when it fits, transposed
  // with a padded row (Ht[i][m], leading dimension nt + 1) so that both the
  // row-wise (residual) and the column-wise (H^H r) sweeps are conflict-free.
  const int ldh = nt + 1;
  // (an offset from the LDS array itself: a round trip through an integer address
  // would leave a generic pointer, and flat loads, for every read of H)
  const size_t ht_off = ((size_t)((const unsigned char*)(Kbs + (size_t)CH * N) - esm) + 15) & ~(size_t)15;
  R* Ht = (R*)(esm + ht_off);
  if constexpr (SH) {
    for (int e = tid; e < nt * nr; e += nth) {
      const int m = e / nr, i = e % nr;
      Ht[2 * (i * ldh + m)] = Hg[2 * (size_t)e];
      Ht[2 * (i * ldh + m) + 1] = Hg[2 * (size_t)e + 1];
    }
    __syncthreads();
  }
  auto hre = [&](int m, int i) -> R { if constexpr (SH) return Ht[2 * (i * ldh + m)]; else return Hg[2 * ((size_t)m * nr + i)]; };
  auto him = [&](int m, int i) -> R { if constexpr (SH) return Ht[2 * (i * ldh + m) + 1]; else return Hg[2 * ((size_t)m * nr + i) + 1]; };

  // With the symbol x_m = s ((2 kI - Q + 1) + j (2 kQ - Q + 1)) of level indices k the
  // residual is r = y - H x = y' - 2 s H k, k_m = kI + j kQ, y' = y + s (Q - 1) (1 + j)
  // sum_m h_m: the level indices enter the products directly.
  for (int i = tid; i < nr; i += nth) {
    R sr = 0, si = 0;
    for (int m = 0; m < nt; ++m) { sr += hre(m, i) - him(m, i); si += hre(m, i) + him(m, i); }
    ys[2 * i] = y[2 * i] + s * R(Q - 1) * sr;
    ys[2 * i + 1] = y[2 * i + 1] + s * R(Q - 1) * si;
  }
  for (int m = tid; m < nt; m += nth) {
    R g = 0;
    for (int i = 0; i < nr; ++i) {
      const R hr = hre(m, i), hi = him(m, i);
      g += hr * hr + hi * hi;
    }
    a2[m] = R(4) * s * s * g * inv_s2;
  }
  if (tid == 0) { best_e = R(INFINITY); best_c = 0; }
  const int mode = a.llr_mode;
  if (mode == 1 && a.llrs) {
    // the list holds distinct samples: flag every chain whose first N levels equal an earlier chain's
    const int nw = (N + 3) >> 2;
    for (int c = tid; c < C; c += nth) {
      const uint32_t* kc = (const uint32_t*)(K + (size_t)c * Npad);
      bool dup = false;
      for (int c2 = 0; c2 < c && !dup; ++c2) {
        const uint32_t* k2 = (const uint32_t*)(K + (size_t)c2 * Npad);
        bool same = true;
        for (int w = 0; w < nw; ++w) {
          const int valid = N - 4 * w;
          const uint32_t msk = valid >= 4 ? 0xFFFFFFFFu : ((1u << (8 * valid)) - 1u);
          same = same && ((kc[w] ^ k2[w]) & msk) == 0u;
        }
        dup = same;
      }
      dupf[c] = dup ? 1 : 0;
    }
  }

  // ownership: marginal rows (m, kI), in blocks of one row per thread, and bits (m, ax, bit)
  const int n_rows = nt * Q, n_llr = nt * 2 * NB;
  const int n_rb = (n_rows + nth - 1) / nth;
  const bool single_chunk = CH >= C;
  const bool want_mc = a.marginals_mc != nullptr;
  OnlineLse<R> lnum[kLlrPerThread], lden[kLlrPerThread];
  int cplus[kLlrPerThread];
#pragma unroll
  for (int q = 0; q < kLlrPerThread; ++q) cplus[q] = 0;

  for (int rb = 0; rb < n_rb; ++rb) {
    const int row = rb * nth + tid;
    // row sums sum_c 2^(v_c(kQ) - Mx) (log2 units) with one running maximum Mx for the
    // row: a point more than 2^-126 below the row's largest term underflows to zero,
    // as it would in the normalised marginal anyway
    R Mx = R(-INFINITY), sums[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) sums[j] = R(0);
    int cnt[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) cnt[j] = 0;

    for (int c0 = 0; c0 < C; c0 += CH) {
      const int ch = C - c0 < CH ? C - c0 : CH;
      if (!single_chunk || rb == 0) {
        __syncthreads();
        for (int it = tid; it < ch * N; it += nth) {
          const int c = it / N, n = it % N;
          Ks[it] = K[(size_t)(c0 + c) * Npad + n];
          Kbs[it] = Kb[(size_t)(c0 + c) * Npad + n];
        }
        __syncthreads();
        // residuals of the final and of the best states
        for (int it = tid; it < ch * nr; it += nth) {
          const int c = it / nr, i = it % nr;
          const uint16_t* kf = (const uint16_t*)(Ks + c * N);   // (k_I, k_Q) of antenna m, as bytes
          const uint16_t* kb = (const uint16_t*)(Kbs + c * N);
          R re = 0, im = 0, bre = 0, bim = 0;
          for (int m = 0; m < nt; ++m) {
            const R hr = hre(m, i), hi = him(m, i);
            const uint32_t f = kf[m], g = kb[m];
            const R xr = R(f & 0xFFu), xi = R(f >> 8), br = R(g & 0xFFu), bi = R(g >> 8);
            re += hr * xr - hi * xi;
            im += hr * xi + hi * xr;
            bre += hr * br - hi * bi;
            bim += hr * bi + hi * br;
          }
          const R s2 = R(2) * s;
          re = ys[2 * i] - s2 * re;
          im = ys[2 * i + 1] - s2 * im;
          bre = ys[2 * i] - s2 * bre;
          bim = ys[2 * i + 1] - s2 * bim;
          rs[c * lrs + 2 * i] = re;
          rs[c * lrs + 2 * i + 1] = im;
          rb2[it] = bre * bre + bim * bim;
        }
        __syncthreads();
        for (int c = tid; c < ch; c += nth) {
          R e = 0, eb = 0;
          for (int i = 0; i < nr; ++i) {
            e += rs[c * lrs + 2 * i] * rs[c * lrs + 2 * i] + rs[c * lrs + 2 * i + 1] * rs[c * lrs + 2 * i + 1];
            eb += rb2[c * nr + i];
          }
          fs[c] = -e * inv_s2;
          ebs[c] = eb;
        }
        __syncthreads();
        // per (chain, antenna): H^H r, the per-axis log normalisers, the base term.  With H
        // in LDS consecutive lanes take consecutive antennas (conflict-free columns of Ht);
        // with H in global memory they take consecutive chains, so that the lanes of one
        // antenna share each cache line of its column
        for (int it = tid; it < ch * nt; it += nth) {
          const int c = SH ? it / nt : it % ch, m = SH ? it % nt : it / ch;
          CM<R> v;
          {
            R re = 0, im = 0;
            for (int i = 0; i < nr; ++i) {
              const R hr = hre(m, i), hi = him(m, i);
              const R rr = rs[c * lrs + 2 * i], ri = rs[c * lrs + 2 * i + 1];
              re += hr * rr + hi * ri;
              im += hr * ri - hi * rr;
            }
            v.aI = R(4) * s * re * inv_s2;
            v.aQ = R(4) * s * im * inv_s2;
          }
          v.kI = Ks[c * N + 2 * m];
          v.kQ = Ks[c * N + 2 * m + 1];
          {
            const R q2 = a2[m];
            OnlineLse<R> li, lq;
#pragma unroll
            for (int k = 0; k < Q; ++k) {
              const R eI = R(k - v.kI), eQ = R(k - v.kQ);
              li.add(eI * (v.aI - q2 * eI) * inv_tau);
              lq.add(eQ * (v.aQ - q2 * eQ) * inv_tau);
            }
            v.base = cw * fs[c] - li.value() - lq.value();
          }
          cm[c * nt + m] = v;
        }
        if (tid == 0 && rb == 0) {
          for (int c = 0; c < ch; ++c)
            if (ebs[c] < best_e) { best_e = ebs[c]; best_c = c0 + c; }
        }
        __syncthreads();
      }

      // symbol marginals and the plain Monte Carlo histogram: row (m, kI).  For chain c the row's
      // terms are b0 + B(kQ), the kI part b0 plus a kQ part B shared by the Q rows of antenna m,
      // which sit in Q consecutive lanes: lane kI of the group forms B(kQ = kI) and its
      // exponential relative to the largest B once, and the group exchanges those Q values by
      // shuffles, so that a row takes three exponentials per chain instead of Q + 1.  The level
      // offsets are differences of small integers, exact in floating point.
      if (row < n_rows) {
        const int m = row / Q, kIt = row % Q;
        const R q2 = a2[m];
        const R l2e = R(1.4426950408889634), q2l = q2 * l2e;
        for (int c = 0; c < ch; ++c) {
          const CM<R> v = cm[c * nt + m];
          const R eI = R(kIt) - R(v.kI), eQ = R(kIt) - R(v.kQ);
          const R b0 = (v.base + eI * (v.aI - q2 * eI)) * l2e;
          const R bq = eQ * (v.aQ * l2e - q2l * eQ);       // B(kQ = kIt)
          const R bmax = group_max<Q>(bq);
          R eqs[Q];
          group_gather<Q>(fex2(bq - bmax), eqs);
          const R lm = b0 + bmax;                          // the row's largest term for chain c
          const R Mn = fmax(lm, Mx);
          const R sc = fex2(Mx - Mn), w = fex2(lm - Mn);
#pragma unroll
          for (int kQt = 0; kQt < Q; ++kQt) sums[kQt] = sums[kQt] * sc + w * eqs[kQt];
          Mx = Mn;
          if (want_mc) {
#pragma unroll
            for (int kQt = 0; kQt < Q; ++kQt) cnt[kQt] += (v.kI == kIt && v.kQ == kQt) ? 1 : 0;
          }
        }
      }
      // bit LLRs: item (m, ax, bit)
      if (rb == 0) {
#pragma unroll
        for (int q = 0; q < kLlrPerThread; ++q) {
          const int it = tid + q * nth;
          if (it < n_llr) {
            const int m = it / (2 * NB), ax = (it / NB) % 2, bit = it % NB;
            const int mask = 1 << (NB - 1 - bit);
            const R q2 = a2[m];
            // one loop per form (the form is uniform: no branch inside the chain loop)
            if (mode == 0) {
              for (int c = 0; c < ch; ++c) {
                const CM<R> v = cm[c * nt + m];
                const int k = ax ? v.kQ : v.kI;
                const R av = ax ? v.aQ : v.aI;
                // the level with this Gray bit cleared (ep) or set (em), as an offset from k: changing
                // Gray bit j of k flips the binary bits j..0, and one of the two is k itself
                const bool gb = ((k ^ (k >> 1)) & mask) != 0;
                const R d = R((k ^ (2 * mask - 1)) - k);
                const R ep = gb ? d : R(0), em = gb ? R(0) : d;
                const R Fp = fs[c] + ep * (av - q2 * ep);
                const R Fm = fs[c] + em * (av - q2 * em);
                const R gm = (Fp - Fm) * inv_tau;
                // F(gm) and F(-gm), F(a) = log(1 + e^a), share log(1 + e^-|gm|) and differ by
                // max(gm, 0) vs max(-gm, 0)
                const R l1 = flog(R(1) + fexp(-fabs(gm)));
                lnum[q].add(cw * Fp - ((gm < R(0) ? -gm : R(0)) + l1));
                lden[q].add(cw * Fm - ((gm > R(0) ? gm : R(0)) + l1));
              }
            } else if (mode == 1) {
              for (int c = 0; c < ch; ++c) {
                const CM<R> v = cm[c * nt + m];
                const int k = ax ? v.kQ : v.kI;
                const bool plus = ((k ^ (k >> 1)) & mask) == 0;   // label bit 0 <-> b = +1
                if (!dupf[c0 + c]) {
                  if (plus) lnum[q].add(fs[c]);
                  else lden[q].add(fs[c]);
                }
              }
            } else {
              for (int c = 0; c < ch; ++c) {
                const CM<R> v = cm[c * nt + m];
                const int k = ax ? v.kQ : v.kI;
                cplus[q] += (((k ^ (k >> 1)) & mask) == 0) ? 1 : 0;
              }
            }
          }
        }
      }
    }
    // normalise over the M points of antenna m: its Q rows sit in Q consecutive
    // lanes of one wavefront, so the log-sum-exp is a Q-lane butterfly
    {
      R lv[Q];
      R mx = R(-INFINITY);
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        lv[j] = (Mx + flg2(sums[j])) * R(0.6931471805599453);
        mx = lv[j] > mx ? lv[j] : mx;
      }
#pragma unroll
      for (int off = 1; off < Q; off <<= 1) { const R o = __shfl_xor(mx, off); mx = o > mx ? o : mx; }
      R sm = R(0);
#pragma unroll
      for (int j = 0; j < Q; ++j) sm += fexp(lv[j] - mx);
#pragma unroll
      for (int off = 1; off < Q; off <<= 1) sm += __shfl_xor(sm, off);
      if (row < n_rows) {
        const int m = row / Q, kIt = row % Q;
        const R inv = R(1) / sm;
        if (a.marginals) {
#pragma unroll
          for (int j = 0; j < Q; ++j) a.marginals[dsc.marg_off + (size_t)m * M + kIt * Q + j] = (float)(fexp(lv[j] - mx) * inv);
        }
        if (want_mc) {
#pragma unroll
          for (int j = 0; j < Q; ++j) a.marginals_mc[dsc.marg_off + (size_t)m * M + kIt * Q + j] = (float)cnt[j] / (float)C;
        }
      }
    }
  }

  if (a.llrs) {
#pragma unroll
    for (int q = 0; q < kLlrPerThread; ++q) {
      const int it = tid + q * nth;
      if (it < n_llr) {
        R v;
        const R clip = (R)a.llr_clip;
        if (mode == 0) {
          v = lnum[q].value() - lden[q].value();
        } else if (mode == 1) {
          const bool hp = lnum[q].mx > R(-INFINITY), hm = lden[q].mx > R(-INFINITY);
          v = !hp ? -clip : (!hm ? clip : lnum[q].value() - lden[q].value());
          v = v > clip ? clip : (v < -clip ? -clip : v);
        } else {
          const int cm_ = C - cplus[q];
          v = cm_ == 0 ? clip : (cplus[q] == 0 ? -clip : flog(R(cplus[q])) - flog(R(cm_)));
          v = v > clip ? clip : (v < -clip ? -clip : v);
        }
        a.llrs[dsc.llr_off + it] = (float)v;
      }
    }
  }
  // hard decision: smallest recomputed energy among the chains' best states (best_c and
  // best_e were last written before a barrier inside the chunk loop)
  {
    const int bc = best_c;
    if (a.best_energy && tid == 0) a.best_energy[dsc.orig] = (float)best_e;
    if (a.symbols)
      for (int m = tid; m < nt; m += nth)
        a.symbols[dsc.sym_off + m] = Kb[(size_t)bc * Npad + 2 * m] * Q + Kb[(size_t)bc * Npad + 2 * m + 1];
  }
}


// A sum of exponentials 2^(u (v - mx)) with its running maximum mx, values v in log2 units (u = 1) or natural ones
// (u = log2(e)): one exponential per value (of the distance to the maximum) instead of one for the old sum and
// one for the value.
// The maximum starts at the lowest finite number: a value of -inf (a chain whose f overflows) then adds
// nothing wherever it stands, where from -inf the distance would be NaN; sum is 0 as long as nothing was added.
constexpr float kLowest = -3.402823466e38f;
struct Lse2 {
  float mx = kLowest, sum = 0.f;
  __device__ __forceinline__ void add(float v, float u) {
    const float d = v - mx, e = fex2(-u * fabsf(d));
    sum = d > 0.f ? __builtin_fmaf(sum, e, 1.f) : sum + e;
    mx = fmaxf(v, mx);
  }
  // merge another sum (either may be empty)
  __device__ __forceinline__ void merge(float omx, float osum, float u) {
    const float m2 = fmaxf(mx, omx);
    sum = sum * fex2(u * (mx - m2)) + osum * fex2(u * (omx - m2));
    mx = m2;
  }
  __device__ __forceinline__ float value(float u) const {
    return u == 1.f ? (mx + flg2(sum)) * 0.6931471805599453f : mx + flg2(sum) * 0.6931471805599453f;
  }
};

// Threads that share a row's (or a bit's) C chains: the largest power of two that keeps them within the given threads,
// at most 8 and one chain each.
__host__ __device__ inline int est_groups(int items, int threads, int C) {
  int g = 1;
  while (2 * g * items <= threads && g < 8 && 2 * g <= C) g *= 2;
  return g;
}

// LDS of the float path (bytes): per-(chain, antenna) values -- the residuals before them, the bits' merges after --,
// energies, per-antenna constants, y', level bytes (rows padded to 16), H.
struct EstLds {
  size_t fs, a2, ys, ks, ht, end;
};
__host__ __device__ inline EstLds est_lds(int nt, int nr, int Q, int N, int chunk, int gm, int gl, bool h_lds) {
  const int NB = Q == 2 ? 1 : (Q == 4 ? 2 : (Q == 8 ? 3 : 4)), NS = (N + 15) & ~15;
  size_t r0 = (size_t)16 * chunk * nt;
  const size_t res = (size_t)4 * chunk * (3 * (size_t)nr + 2);
  const size_t mm = (size_t)4 * (2 * Q + 1) * nt * Q * (gm - 1), ml = (size_t)4 * 5 * nt * 2 * NB * (gl - 1);
  r0 = res > r0 ? res : r0;
  r0 = mm > r0 ? mm : r0;
  r0 = ml > r0 ? ml : r0;
  EstLds o;
  o.fs = (r0 + 15) & ~(size_t)15;
  o.a2 = o.fs + (size_t)8 * chunk;
  o.ys = o.a2 + (size_t)4 * nt;
  o.ks = (o.ys + (size_t)8 * nr + 15) & ~(size_t)15;
  o.ht = o.ks + (size_t)2 * chunk * NS;
  o.end = o.ht + (h_lds ? (size_t)8 * (nt + 1) * nr : 0);
  return o;
}

// The float path.  Phases per chunk of chains (one chunk where LDS holds them all): levels staged in LDS;
// residuals and energies of the final and best states; per (chain, antenna) the axis coefficients and log
// normalisers; the marginal rows and the bits.
// |f| reaches 1e5 at high SNR, where one rounding of a quantity of that size moves a marginal by 1e-2: the sums
// behind f and the marginals keep one order whatever the number of threads (y', the column norms and the energies
// run sequentially in one thread each, with their loads ahead of the sums; residuals in the form a.res names).
// Residuals r = y' - 2 s H k from the level indices, y' = y + s (Q - 1) (1 + j) sum_m h_m:
//   res 0: one thread per (receive antenna, chain);
//   res 1: on the float32 matrix cores (v_mfma_f32_16x16x4f32, [Re r; Im r] = y' - 2 s [Hr -Hi; Hi Hr] k over the real
//          dimensions n).  A wave takes a tile of 16 receive antennas x 16 chains of the final or of the best states;
//          lane l holds A[l % 16][4 s + l / 16], so that whether it multiplies a real or an imaginary column
//          (n odd) is fixed per lane, and one 16-byte read of its chain's levels serves four K steps;
//   res 2: the same with the two halves of the K steps summed apart and added.
// H^H r of the final states comes from the sampler's energy gradient.
// Bound by issue (per 64x64 64-QAM problem of 64 chains about 16k clocks of float32 MFMA, 15k in the rows, 12k in the
// bits, 8k in the normalisers).  Two-pass normalisers, byte-wise levels, one row per thread whatever the shape and
// branches inside the bits' chain loop took (us, full batches): 8x8 64-QAM 72 -> 68, 32x32 326 -> 263,
// 64x64 947 -> 752, 128x128 256-QAM 414 -> 210.
// RPT: marginal rows per thread (256-QAM beyond 64 antennas has twice as many rows as threads; two rows' sums do not fit
// the registers beside the rest, so that the other shapes have kernels of their own: 2000 problems of 40x40, 32 chains,
// 338 us with two rows' registers, 309 in the former kernel).
template <int Q, bool SH, int BS, int RPT>
__device__ __forceinline__ void estimate_f(const EstArgs& a, const int b) {
  using R = float;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  constexpr int M = Q * Q, NW = BS / 64;
  constexpr int NB = Q == 2 ? 1 : (Q == 4 ? 2 : (Q == 8 ? 3 : 4));
  constexpr float kL2e = 1.4426950408889634f;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = a.nt, nr = a.nr, C = a.C, Npad = a.Npad, N = a.N, CH = a.chunk;
  const InstDesc dsc = inst_desc(a.desc, b, nt, nr, M, C);
  const float* Hg = (const float*)a.H + 2 * dsc.h_off;
  const float* y = (const float*)a.y + 2 * dsc.y_off;
  const InstParams ip = *(const InstParams*)(a.ws_inst + (size_t)b * a.inst_stride);
  if (ip.nonfinite) {
    // a flagged instance (see the setup kernel): no samples to estimate from; symbols -1,
    // every other output NaN (the whole workgroup leaves here)
    const float nan = __builtin_nanf("");
    for (int m = tid; m < nt; m += BS)
      if (a.symbols) a.symbols[dsc.sym_off + m] = -1;
    for (int e = tid; e < nt * M; e += BS) {
      if (a.marginals) a.marginals[dsc.marg_off + e] = nan;
      if (a.marginals_mc) a.marginals_mc[dsc.marg_off + e] = nan;
    }
    for (int e = tid; e < nt * 2 * NB; e += BS)
      if (a.llrs) a.llrs[dsc.llr_off + e] = nan;
    if (a.best_energy && tid == 0) a.best_energy[dsc.orig] = nan;
    return;
  }
  const R s = (R)ip.s, tau = (R)ip.tau;
  const R inv_s2 = R(1) / (R)ip.sigma2, inv_tau = R(1) / tau;
  const R cw = (tau - R(1)) * inv_tau;
  const R kA = R(-2) * tau * R(0.69314718055994530942);
  const StateOff so = state_offsets(a.Cpad, Npad);
  const unsigned char* st = a.ws_state + (size_t)b * a.state_stride;
  const unsigned char* K = st + so.k;
  const unsigned char* Kb = st + so.kbest;

  extern __shared__ __attribute__((aligned(16))) unsigned char esm[];
  const EstLds lo = est_lds(nt, nr, Q, N, CH, a.gm, a.gl, SH);
  const int NS = (N + 15) & ~15;                 // level row stride (a multiple of 16, at most Npad)
  const int ldh = nt + 1;                        // H transposed with a padded row: row- and column-wise reads
  const int lrs = 2 * nr + 2;                    // residual row stride
  f32x4* cm = (f32x4*)esm;                       // [chain][antenna]: a_I, a_Q, base, packed levels
  R* rs = (R*)esm;                               // CH x nr complex residuals of the final states
  R* rb2 = rs + (size_t)CH * lrs;                // CH x nr |residual|^2 of the best states
  R* fs = (R*)(esm + lo.fs);                     // f of the final states, then the best states' energies
  R* ebs = fs + CH;
  R* a2 = (R*)(esm + lo.a2);                     // 4 s^2 |h_m|^2 / sigma^2
  R* ys = (R*)(esm + lo.ys);                     // y'
  unsigned char* Ks = esm + lo.ks;               // CH x NS
  unsigned char* Kbs = Ks + (size_t)CH * NS;     // CH x NS
  f32x2* Ht = (f32x2*)(esm + lo.ht);
  __shared__ R best_e;
  __shared__ int best_c;
  __shared__ unsigned char dupf[1024];   // list LLRs: chain repeats an earlier chain's final state

  // level rows as 16-byte pieces, np of them a row; the first chunk's ahead of everything else
  auto stage = [&](int c0, int ch) {
    const int np = NS >> 4, tot = ch * np;
    for (int e = tid; e < 2 * tot; e += BS) {
      const int e1 = e < tot ? e : e - tot, c = e1 / np, w = e1 - c * np;
      const unsigned char* src = (e < tot ? K : Kb) + (size_t)(c0 + c) * Npad + 16 * w;
      *(uint4*)((e < tot ? Ks : Kbs) + c * NS + 16 * w) = *(const uint4*)src;
    }
  };
  stage(0, C < CH ? C : CH);
  if constexpr (SH) {
    int m = tid / nr, i = tid % nr;
    const int dm = BS / nr, di = BS % nr;
    for (int e = tid; e < nt * nr; e += BS) {
      Ht[i * ldh + m] = f32x2{Hg[2 * (size_t)e], Hg[2 * (size_t)e + 1]};
      m += dm;
      i += di;
      if (i >= nr) { i -= nr; ++m; }
    }
    __syncthreads();
  }
  auto hcol = [&](int m, int i) -> f32x2 {
    if constexpr (SH) return Ht[i * ldh + m];
    else return f32x2{Hg[2 * ((size_t)m * nr + i)], Hg[2 * ((size_t)m * nr + i) + 1]};
  };
  // y' from the first threads, the column norms from the last ones
  for (int i = tid; i < nr; i += BS) {
    R sr = 0, si = 0;
#pragma unroll 8
    for (int m = 0; m < nt; ++m) { const f32x2 v = hcol(m, i); sr += v.x - v.y; si += v.x + v.y; }
    ys[2 * i] = y[2 * i] + s * R(Q - 1) * sr;
    ys[2 * i + 1] = y[2 * i + 1] + s * R(Q - 1) * si;
  }
  for (int m = BS - 1 - tid; m < nt; m += BS) {
    R g = 0;
#pragma unroll 8
    for (int i = 0; i < nr; ++i) {
      const f32x2 v = hcol(m, i);
      const R hr = v.x, hi = v.y;
      g += hr * hr + hi * hi;
    }
    a2[m] = R(4) * s * s * g * inv_s2;
  }
  if (tid == 0) { best_e = R(INFINITY); best_c = 0; }
  const int mode = a.llr_mode;
  if (mode == 1 && a.llrs) {
    // the list holds distinct samples: flag every chain whose first N levels equal an earlier chain's
    const int nw = (N + 3) >> 2;
    for (int c = tid; c < C; c += BS) {
      const uint32_t* kc = (const uint32_t*)(K + (size_t)c * Npad);
      bool dup = false;
      for (int c2 = 0; c2 < c && !dup; ++c2) {
        const uint32_t* k2 = (const uint32_t*)(K + (size_t)c2 * Npad);
        bool same = true;
        for (int w = 0; w < nw; ++w) {
          const int valid = N - 4 * w;
          const uint32_t msk = valid >= 4 ? 0xFFFFFFFFu : ((1u << (8 * valid)) - 1u);
          same = same && ((kc[w] ^ k2[w]) & msk) == 0u;
        }
        dup = same;
      }
      dupf[c] = dup ? 1 : 0;
    }
  }

  // Ownership: RPT marginal rows (m, kI) and a bit (m, axis, bit) per thread, or per GM (GL) threads with every
  // GM-th (GL-th) chain each (merged at the end).  The host takes enough threads for the rows, no shape has more bits
  // than threads, and the groups follow from the shape alone, so that the results do not depend on the launch's size.
  const int n_rows = nt * Q, n_llr = nt * 2 * NB;
  const int GM = a.gm, GL = a.gl, LM = BS / GM, LP = BS / GL;   // (powers of two)
  const int gm = tid / LM, it_row = tid - gm * LM, gl = tid / LP, it_llr = tid - gl * LP;
  const bool want_mc = a.marginals_mc != nullptr;
  Lse2 lnum, lden;
  const R lu = mode == 1 ? kL2e : R(1);   // their units
  int cplus = 0;
  // row sums sum_c 2^(v_c(kQ) - Mx) (log2 units) with one running maximum Mx for the row: a point more than 2^-126
  // below the row's largest term underflows to zero, as it would in the normalised marginal anyway
  // (from kLowest, as the bits')
  R Mx[RPT], sums[RPT][Q];
  uint32_t cnt[RPT][Q / 2];   // histogram: levels 2 w, 2 w + 1 in the halves of word w (at most 1024 chains)
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    Mx[r] = kLowest;
#pragma unroll
    for (int j = 0; j < Q; ++j) { sums[r][j] = R(0); cnt[r][j >> 1] = 0u; }
  }
  auto count = [&](int r, int j) { return (int)((cnt[r][j >> 1] >> (16 * (j & 1))) & 0xFFFFu); };

  for (int c0 = 0; c0 < C; c0 += CH) {
    const int ch = C - c0 < CH ? C - c0 : CH;
    if (c0) {
      __syncthreads();   // (the chunk before is read)
      stage(c0, ch);
    }
    __syncthreads();
    const R s2 = R(2) * s;
    if (a.res == 0) {
      // a thread takes rows i and i + h2 of a chain: its levels are read (16 bytes: eight antennas) and converted once
      // for both
      const int h2 = (nr + 1) >> 1;
      int c = tid / h2, i = tid - c * h2;
      const int dc = BS / h2, di = BS - dc * h2;
      for (int it = tid; it < ch * h2; it += BS) {
        const unsigned char* kf = Ks + c * NS;   // (k_I, k_Q) of antenna m in bytes 2 m, 2 m + 1
        const unsigned char* kb = Kbs + c * NS;
        const int i1 = i + h2 < nr ? i + h2 : i;
        R re[2] = {0, 0}, im[2] = {0, 0}, bre[2] = {0, 0}, bim[2] = {0, 0};
        auto term = [&](int m, uint32_t f, uint32_t g) {
          const R xr = R(f & 0xFFu), xi = R((f >> 8) & 0xFFu), br = R(g & 0xFFu), bi = R((g >> 8) & 0xFFu);
          const f32x2 v[2] = {hcol(m, i), hcol(m, i1)};
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const R hr = v[q].x, hi = v[q].y;
            re[q] += hr * xr - hi * xi;
            im[q] += hr * xi + hi * xr;
            bre[q] += hr * br - hi * bi;
            bim[q] += hr * bi + hi * br;
          }
        };
        int m = 0;
        for (; m + 8 <= nt; m += 8) {
          const uint4 f4 = *(const uint4*)(kf + 2 * m), g4 = *(const uint4*)(kb + 2 * m);
          const uint32_t f[4] = {f4.x, f4.y, f4.z, f4.w}, g[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
          for (int q = 0; q < 8; ++q) term(m + q, f[q >> 1] >> (16 * (q & 1)), g[q >> 1] >> (16 * (q & 1)));
        }
        for (; m < nt; ++m) term(m, *(const uint16_t*)(kf + 2 * m), *(const uint16_t*)(kb + 2 * m));
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int iq = i + q * h2;
          if (iq < nr) {
            const R rr = ys[2 * iq] - s2 * re[q], ri = ys[2 * iq + 1] - s2 * im[q];
            const R br = ys[2 * iq] - s2 * bre[q], bi = ys[2 * iq + 1] - s2 * bim[q];
            rs[c * lrs + 2 * iq] = rr;
            rs[c * lrs + 2 * iq + 1] = ri;
            rb2[c * nr + iq] = br * br + bi * bi;
          }
        }
        c += dc;
        i += di;
        if (i >= h2) { i -= h2; ++c; }
      }
    } else {
      const int nct = (ch + 15) >> 4, nrt = (nr + 15) >> 4, ksteps = (N + 3) >> 2;
      const int half = a.res == 2 ? ((ksteps + 1) / 2 + 1) / 2 * 2 : 1 << 30;
      const int h = lane >> 4;
      const bool odd = h & 1;
      for (int u = wv; u < 2 * nct * nrt; u += NW) {
        const int state = u & 1, rt = (u >> 1) % nrt, ct = (u >> 1) / nrt;
        const int c = 16 * ct + (lane & 15), cc = c < ch ? c : ch - 1;
        const unsigned char* kr = (state ? Kbs : Ks) + cc * NS;
        const int ia = 16 * rt + (lane & 15), iac = ia < nr ? ia : nr - 1;
        f32x4 re = {0.f, 0.f, 0.f, 0.f}, im = re, re1 = re, im1 = re;
        for (int st0 = 0; st0 < ksteps; st0 += 4) {
          // (the last piece may run past N, inside the padded row; the columns there are masked)
          const uint4 kw = *(const uint4*)(kr + 4 * st0);
          const uint32_t w4[4] = {kw.x, kw.y, kw.z, kw.w};
          f32x2 hv[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int m = 2 * (st0 + q) + (h >> 1);
            hv[q] = hcol(m < nt ? m : nt - 1, iac);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (st0 + q == half) { re1 = re; im1 = im; re = f32x4{0.f, 0.f, 0.f, 0.f}; im = re; }
            const bool ok = 2 * (st0 + q) + (h >> 1) < nt && ia < nr;
            const float hr = ok ? hv[q].x : 0.f, hi = ok ? hv[q].y : 0.f;
            const float k = (float)((w4[q] >> (8 * h)) & 255u);
            re = __builtin_amdgcn_mfma_f32_16x16x4f32(odd ? -hi : hr, k, re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f32_16x16x4f32(odd ? hr : hi, k, im, 0, 0, 0);
          }
        }
        if (half < ksteps) { re = re1 + re; im = im1 + im; }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int i = 16 * rt + 4 * h + j;
          if (i < nr && c < ch) {
            const R rr = ys[2 * i] - s2 * re[j], ri = ys[2 * i + 1] - s2 * im[j];
            if (state) {
              rb2[c * nr + i] = rr * rr + ri * ri;
            } else {
              rs[c * lrs + 2 * i] = rr;
              rs[c * lrs + 2 * i + 1] = ri;
            }
          }
        }
      }
    }
    __syncthreads();
    // energies: the final states' from the first threads, the best states' from the last ones
    for (int c = tid; c < ch; c += BS) {
      R e = 0;
#pragma unroll 16
      for (int i = 0; i < nr; ++i)
        e += rs[c * lrs + 2 * i] * rs[c * lrs + 2 * i] + rs[c * lrs + 2 * i + 1] * rs[c * lrs + 2 * i + 1];
      fs[c] = -e * inv_s2;
    }
    for (int c = BS - 1 - tid; c < ch; c += BS) {
      R eb = 0;
#pragma unroll 16
      for (int i = 0; i < nr; ++i) eb += rb2[c * nr + i];
      ebs[c] = eb;
    }
    __syncthreads();
    // Per (chain, antenna): a_n = 4 s (H^H r)_n / sigma^2 = -2 tau ln(2) g from the sampler's energy gradient at the
    // final state, g = -2 s log2(e) H^H r / (tau sigma^2); the per-axis log normalisers over the Q levels, accumulated
    // in log2 units; the base term.  (The residuals are done with: cm takes their place.)
    {
      int c = tid / nt, m = tid - c * nt;
      const int dc = BS / nt, dm = BS - dc * nt;
      const float* eg = (const float*)(st + so.eg) + (size_t)c0 * Npad;
      for (int it = tid; it < ch * nt; it += BS) {
        const R aI = kA * eg[(size_t)c * Npad + 2 * m], aQ = kA * eg[(size_t)c * Npad + 2 * m + 1];
        const uint32_t kk = *(const uint16_t*)(Ks + c * NS + 2 * m);
        const R sc = inv_tau * R(1.4426950408889634);
        const R q2s = a2[m] * sc, aIs = aI * sc, aQs = aQ * sc;
        const R kIf = (R)(kk & 255u), kQf = (R)(kk >> 8);
        R mi = R(-INFINITY), mq = R(-INFINITY), si = R(0), sq = R(0);
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          const R eI = R(k) - kIf, eQ = R(k) - kQf;
          const R ti = eI * (aIs - q2s * eI), tq = eQ * (aQs - q2s * eQ);
          // one exponential per level: of the distance to the running maximum
          const R di = ti - mi, dq = tq - mq, xi = fex2(-fabsf(di)), xq = fex2(-fabsf(dq));
          si = di > R(0) ? si * xi + R(1) : si + xi;
          sq = dq > R(0) ? sq * xq + R(1) : sq + xq;
          mi = fmaxf(mi, ti);
          mq = fmaxf(mq, tq);
        }
        const R base = cw * fs[c] - (mi + flg2(si) + mq + flg2(sq)) * R(0.6931471805599453);
        cm[c * nt + m] = f32x4{aI, aQ, base, __uint_as_float(kk)};
        c += dc;
        m += dm;
        if (m >= nt) { m -= nt; ++c; }
      }
    }
    if (wv == NW - 1) {
      // the best state: smallest energy, then lowest chain
      R be = R(INFINITY);
      int bc = 0x7FFFFFFF;
      for (int c = lane; c < ch; c += 64)
        if (ebs[c] < be) { be = ebs[c]; bc = c; }
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const R oe = __shfl_xor(be, o);
        const int oc = __shfl_xor(bc, o);
        if (oe < be || (oe == be && oc < bc)) { be = oe; bc = oc; }
      }
      if (lane == 0 && be < best_e) { best_e = be; best_c = c0 + bc; }
    }
    __syncthreads();

    // Symbol marginals and the plain Monte Carlo histogram.  For chain c the row's terms are b0 + B(kQ), the kI
    // part b0 plus a kQ part B shared by the Q rows of antenna m, which sit in Q consecutive lanes: lane kI of the
    // group forms the exponential of B(kQ = kI) relative to the largest B, and the group exchanges those Q
    // values, so that a row takes two exponentials per chain.
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const int row = it_row + r * BS;
      if (row < n_rows) {
        const int m = row / Q;
        const R kt = (R)(row & (Q - 1));
        const R q2 = a2[m];
        const R l2e = R(1.4426950408889634), q2l = q2 * l2e;
        for (int c = (gm - c0) & (GM - 1); c < ch; c += GM) {
          const f32x4 v = cm[c * nt + m];
          const uint32_t kk = __float_as_uint(v.w);
          const R kI = (R)(kk & 255u), kQ = (R)((kk >> 8) & 255u);
          const R eI = kt - kI, eQ = kt - kQ;
          const R b0 = (v.z + eI * (v.x - q2 * eI)) * l2e;
          const R bq = eQ * (v.y * l2e - q2l * eQ);       // B(kQ = kt)
          const R bmax = group_max<Q>(bq);
          R eqs[Q];
          group_gather<Q>(fex2(bq - bmax), eqs);
          const R lm = b0 + bmax;                          // the row's largest term for chain c
          const R d = lm - Mx[r], e = fex2(-fabsf(d));
          const bool up = d > R(0);
          const R sc = up ? e : R(1), w = up ? R(1) : e;
#pragma unroll
          for (int j = 0; j < Q; ++j) sums[r][j] = sums[r][j] * sc + w * eqs[j];
          Mx[r] = fmaxf(lm, Mx[r]);
        }
        // (a loop of its own: the counts would take the sums' registers)
        if (want_mc) {
          for (int c = (gm - c0) & (GM - 1); c < ch; c += GM) {
            const uint32_t kk = __float_as_uint(cm[c * nt + m].w), kQ = kk >> 8;
            const uint32_t hit = (kk & 255u) == (uint32_t)(row & (Q - 1)) ? 1u << (16 * (kQ & 1u)) : 0u;
#pragma unroll
            for (int w = 0; w < Q / 2; ++w) cnt[r][w] += (kQ >> 1) == (uint32_t)w ? hit : 0u;
          }
        }
      }
    }
    // Bit LLRs.  f stays in natural units up to its one product with (tau - 1) / tau log2(e): scaled to log2 units by
    // itself it would be rounded once more (|f| reaches 1e5, where a rounding moves an LLR by 1e-2), and
    // overflow from 2.4e38 on.
    if (a.llrs && it_llr < n_llr) {
      const int m = it_llr / (2 * NB), rem = it_llr - m * 2 * NB, ax = rem >= NB ? 1 : 0, bit = rem - ax * NB;
      const int mask = 1 << (NB - 1 - bit);
      const R q2 = a2[m], cwl = cw * kL2e, itl = inv_tau * kL2e;
      // one loop per form (the form is uniform: no branch inside the chain loop)
      if (mode == 0) {
        for (int c = (gl - c0) & (GL - 1); c < ch; c += GL) {
          const f32x4 v = cm[c * nt + m];
          const uint32_t kk = __float_as_uint(v.w);
          const int k = ax ? (int)(kk >> 8) : (int)(kk & 255u);
          const R av = ax ? v.y : v.x;
          // the other value of this Gray bit: changing bit j of the label flips the binary bits j..0
          const bool gb = ((k ^ (k >> 1)) & mask) != 0;
          const R d = (R)((k ^ (2 * mask - 1)) - k);
          const R f0 = fs[c], dl = d * (av - q2 * d);   // F of the sample, and the move's change
          // g = (F+ - F-) / tau; F(a) = log(1 + e^a): F(g) and F(-g) share log(1 + e^-|g|) (log2 units)
          const R g = (gb ? dl : -dl) * itl;
          const R l1 = flg2(R(1) + fex2(-fabsf(g)));
          const R f1 = f0 + dl, Fp = gb ? f1 : f0, Fm = gb ? f0 : f1;
          lnum.add(__builtin_fmaf(cwl, Fp, -(fmaxf(-g, R(0)) + l1)), R(1));
          lden.add(__builtin_fmaf(cwl, Fm, -(fmaxf(g, R(0)) + l1)), R(1));
        }
      } else {
        for (int c = (gl - c0) & (GL - 1); c < ch; c += GL) {
          const uint32_t kk = __float_as_uint(cm[c * nt + m].w);
          const int k = ax ? (int)(kk >> 8) : (int)(kk & 255u);
          const bool plus = ((k ^ (k >> 1)) & mask) == 0;   // label bit 0 <-> b = +1
          if (mode == 2) {
            cplus += plus ? 1 : 0;
          } else if (!dupf[c0 + c]) {
            if (plus) lnum.add(fs[c], kL2e);
            else lden.add(fs[c], kL2e);
          }
        }
      }
    }
  }
  // merge the threads' shares of a bit's and of a row's chains (through LDS, groups in order)
  if (GL > 1) {
    R* o = (R*)esm;
    __syncthreads();
    if (gl > 0 && it_llr < n_llr) {
      R* q = o + (size_t)(gl - 1) * 5 * n_llr + it_llr;
      q[0] = lnum.mx; q[n_llr] = lnum.sum; q[2 * n_llr] = lden.mx; q[3 * n_llr] = lden.sum;
      q[4 * n_llr] = (R)cplus;
    }
    __syncthreads();
    if (gl == 0 && it_llr < n_llr) {
      for (int g = 1; g < GL; ++g) {
        const R* q = o + (size_t)(g - 1) * 5 * n_llr + it_llr;
        lnum.merge(q[0], q[n_llr], lu);
        lden.merge(q[2 * n_llr], q[3 * n_llr], lu);
        cplus += (int)q[4 * n_llr];
      }
    }
  }
  if (GM > 1) {
    // (only shapes with one row per thread)
    R* o = (R*)esm;
    __syncthreads();
    if (gm > 0 && it_row < n_rows) {
      R* q = o + (size_t)(gm - 1) * (2 * Q + 1) * n_rows + it_row;
      q[0] = Mx[0];
#pragma unroll
      for (int j = 0; j < Q; ++j) { q[(1 + j) * n_rows] = sums[0][j]; q[(1 + Q + j) * n_rows] = (R)count(0, j); }
    }
    __syncthreads();
    if (gm == 0 && it_row < n_rows) {
      for (int g = 1; g < GM; ++g) {
        const R* q = o + (size_t)(g - 1) * (2 * Q + 1) * n_rows + it_row;
        const R om = q[0], nm = fmaxf(om, Mx[0]);
        const R sa = fex2(Mx[0] - nm), sb = fex2(om - nm);
        Mx[0] = nm;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          sums[0][j] = sums[0][j] * sa + q[(1 + j) * n_rows] * sb;
          cnt[0][j >> 1] += (uint32_t)q[(1 + Q + j) * n_rows] << (16 * (j & 1));
        }
      }
    }
  }
  // normalise over the M points of antenna m: its Q rows sit in Q consecutive
  // lanes of one wavefront, so the log-sum-exp is a Q-lane butterfly
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    if (r && r * BS >= n_rows) break;   // (no thread has a second row)
    const int row = it_row + r * BS;
    R lv[Q];
    R mx = R(-INFINITY);
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      lv[j] = (Mx[r] + flg2(sums[r][j])) * R(0.6931471805599453);
      mx = lv[j] > mx ? lv[j] : mx;
    }
#pragma unroll
    for (int off = 1; off < Q; off <<= 1) { const R o = __shfl_xor(mx, off); mx = o > mx ? o : mx; }
    R sm = R(0);
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      lv[j] = fexp(lv[j] - mx);
      sm += lv[j];
    }
#pragma unroll
    for (int off = 1; off < Q; off <<= 1) sm += __shfl_xor(sm, off);
    if (gm == 0 && row < n_rows) {
      const R inv = R(1) / sm;
      const size_t o = dsc.marg_off + (size_t)row * Q;
      auto store = [&](float* dst, auto&& val) {
        if (Q >= 4 && ((uintptr_t)dst & 15) == 0) {
#pragma unroll
          for (int j = 0; j + 3 < Q; j += 4) *(f32x4*)(dst + j) = f32x4{val(j), val(j + 1), val(j + 2), val(j + 3)};
        } else {
#pragma unroll
          for (int j = 0; j < Q; ++j) dst[j] = val(j);
        }
      };
      if (a.marginals) store(a.marginals + o, [&](int j) { return lv[j] * inv; });
      if (want_mc) store(a.marginals_mc + o, [&](int j) { return (float)count(r, j) / (float)C; });
    }
  }
  if (a.llrs && gl == 0 && it_llr < n_llr) {
    R v;
    const R clip = a.llr_clip;
    if (mode == 0) {
      v = lnum.value(lu) - lden.value(lu);
    } else if (mode == 1) {
      const bool hp = lnum.mx > kLowest, hm = lden.mx > kLowest;
      v = !hp ? -clip : (!hm ? clip : lnum.value(lu) - lden.value(lu));
      v = v > clip ? clip : (v < -clip ? -clip : v);
    } else {
      const int cm_ = C - cplus;
      v = cm_ == 0 ? clip : (cplus == 0 ? -clip : flog(R(cplus)) - flog(R(cm_)));
      v = v > clip ? clip : (v < -clip ? -clip : v);
    }
    a.llrs[dsc.llr_off + it_llr] = v;
  }
  // hard decision (best_c and best_e were last written before a barrier inside the chunk loop)
  {
    const int bc = best_c;
    if (a.best_energy && tid == 0) a.best_energy[dsc.orig] = best_e;
    if (a.symbols)
      for (int m = tid; m < nt; m += BS)
        a.symbols[dsc.sym_off + m] = Kb[(size_t)bc * Npad + 2 * m] * Q + Kb[(size_t)bc * Npad + 2 * m + 1];
  }
}

// One instance by the path of the input type.
template <typename R, int Q, bool SH, int BS, int RPT>
__device__ __forceinline__ void estimate_one(const EstArgs& a, const int b) {
  if constexpr (sizeof(R) == 8) estimate_d<Q, SH>(a, b);
  else estimate_f<Q, SH, BS, RPT>(a, b);
}

// Direct launch (PERS false): instance blockIdx.x.  Persistent launch: items from the list, each
// with its class's arguments.
template <typename R, int Q, bool SH, int BS, bool PERS = false, int RPT = 1>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 1 : (BS == 256 && Q <= 8 && !PERS ? 5 : 4))))
void estimate_kernel(EstArgs a, Persist p) {
  if constexpr (!PERS) {
    estimate_one<R, Q, SH, BS, RPT>(a, blockIdx.x);
  } else {
    extern __shared__ __attribute__((aligned(16))) unsigned char esm[];
    for (;;) {
      const int it = persist_take(p, esm);
      if (it >= p.n_items) break;
      const WorkItem w = p.items[it];
      const EstArgs ca = ((const EstArgs*)p.cls)[__builtin_amdgcn_readfirstlane(w.cls)];
      estimate_one<R, Q, SH, BS, RPT>(ca, __builtin_amdgcn_readfirstlane(w.inst));
    }
    persist_done(p);
  }
}

// LDS of the float64 path without H.
static size_t estimate_lds_bytes(int nt, int nr, int N, int chunk) {
  return 32 * (size_t)chunk * nt + 8 * (3 * (size_t)chunk * nr + 4 * (size_t)chunk + nt + 2 * (size_t)nr) + 2 * (size_t)chunk * N + 16;
}

// H is staged in LDS when it fits 64 KiB (transposed, padded rows).
static bool estimate_h_in_lds(int nt, int nr, bool fp64) {
  return 2 * (size_t)(nt + 1) * nr * (fp64 ? 8 : 4) <= 65536;
}

// Threads per workgroup: one (antenna, kI) row each, in 256, 512 or 1024 threads; 1024 whenever H is
// read from global memory.  Launches of at most one workgroup per CU take 1024 threads where the phases of C chains are
// work enough for them (us for 256 problems, 1024 threads / the shape's own: 32x32 64-QAM 64 chains 48 / 54, 24x24 16-QAM 32
// chains 20.7 / 21.3, 32x32 256-QAM 64 chains 51 / 53; below, more waves only wait for one another: 16x16 16-QAM 64 chains
// 23.0 / 20.6, 8x8 256-QAM 16 chains 17.5 / 15.6, 4x4 16-QAM 16 chains 14.4 / 12.3).  The float64 path (nt <= 32) keeps 256.
static int estimate_threads(int nt, int nr, int Q, int C, bool fp64, int n_inst) {
  if (fp64) return 256;
  if (!estimate_h_in_lds(nt, nr, false) || nt * Q > 512) return 1024;
  if (n_inst <= 256 && (size_t)nt * nt * nr * C >= 360000) return 1024;
  return nt * Q > 256 ? 512 : 256;
}

// Threads that share a row's (a bit's) chains, of those that a large launch gives the shape.
static void estimate_groups(int nt, int nr, int Q, int C, int* gm, int* gl) {
  const int NB = Q == 2 ? 1 : (Q == 4 ? 2 : (Q == 8 ? 3 : 4)), th = estimate_threads(nt, nr, Q, C, false, 1 << 30);
  *gm = est_groups(nt * Q, th < 512 ? th : 512, C);
  *gl = est_groups(nt * 2 * NB, th, C);
}

static size_t estimate_lds(int nt, int nr, int Q, int N, int C, int chunk, bool fp64) {
  const bool sh = estimate_h_in_lds(nt, nr, fp64);
  if (fp64) return estimate_lds_bytes(nt, nr, N, chunk) + (sh ? 2 * (size_t)(nt + 1) * nr * 8 + 16 : 0);
  int gm, gl;
  estimate_groups(nt, nr, Q, C, &gm, &gl);
  return est_lds(nt, nr, Q, N, chunk, gm, gl, sh).end;
}

// LDS of a workgroup beside what est_lds counts: the static arrays, in a persistent launch the item word.
constexpr size_t kEstStatic = 1024 + 16 + 16;

// Chains per chunk: all of them where they fit 128 KiB of LDS (96 KiB with 256 or 512 threads, whose
// workgroups share a CU); a smaller chunk, of at least 16 chains, where that lets more workgroups share a CU.
// 512-thread workgroups run two per CU within 80 KiB (with the static arrays; one of 81 KiB took, us for 4096
// instances, 861 instead of 563 for 48x48 64-QAM and 64 chains, 1060 instead of 786 for 67x67 16-QAM).  256-thread ones run
// four or five per CU within 32 KiB: those of the last KiB, four, are still faster so than with half the chunk or with
// the next larger one that a limit for five would give them (34x34 4-QAM, 64 chains: 230 against 248; 45x45: 352 against
// 433).
static int estimate_chunk(int nt, int nr, int Q, int N, int C, bool fp64, int threads) {
  const size_t most = (!fp64 && threads == 1024 ? 128 : 96) * 1024;   // (float64: beside H)
  int ch = C;
  while (ch > 1 && (fp64 ? estimate_lds_bytes(nt, nr, N, ch) : estimate_lds(nt, nr, Q, N, C, ch, false)) > most)
    ch = (ch + 1) / 2;
  if (!fp64 && threads <= 512) {
    const size_t budget = threads == 256 ? 32 * 1024 : 80 * 1024 - kEstStatic;
    int c2 = ch;
    while (c2 > 16 && estimate_lds(nt, nr, Q, N, C, c2, false) > budget) c2 = (c2 + 1) / 2;
    if (estimate_lds(nt, nr, Q, N, C, c2, false) <= budget) ch = c2;
  }
  return ch;
}

template <typename R, int Q, int BS>
static hipError_t launch_eb(const EstArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  const bool sh = estimate_h_in_lds(a.nt, a.nr, sizeof(R) == 8);
  const size_t lds = estimate_lds(a.nt, a.nr, Q, a.N, a.C, a.chunk, sizeof(R) == 8);
  void (*k)(EstArgs, Persist);
  // (the smaller workgroups only run with H in LDS)
  constexpr bool kGlob = BS == 1024 || sizeof(R) == 8;
  if (!sh && !kGlob) return hipErrorInvalidConfiguration;
  auto pick = [&](auto rows) {
    constexpr int RPT = decltype(rows)::value;
    if (p || cfg) k = sh ? estimate_kernel<R, Q, true, BS, true, RPT> : estimate_kernel<R, Q, !kGlob, BS, true, RPT>;
    else k = sh ? estimate_kernel<R, Q, true, BS, false, RPT> : estimate_kernel<R, Q, !kGlob, BS, false, RPT>;
  };
  constexpr bool kTwo = sizeof(R) == 4 && Q == 16 && BS == 1024;   // (64 antennas and fewer: a row per thread)
  if (kTwo && a.nt * Q > BS) pick(std::integral_constant<int, kTwo ? 2 : 1>{});
  else pick(std::integral_constant<int, 1>{});
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

template <typename R, int Q>
static hipError_t launch_e(const EstArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  if constexpr (sizeof(R) == 8) {
    return launch_eb<R, Q, 256>(a, s, p, gn, cfg);
  } else {
    const int bs = a.threads;
    return bs == 256 ? launch_eb<R, Q, 256>(a, s, p, gn, cfg)
                     : (bs == 512 ? launch_eb<R, Q, 512>(a, s, p, gn, cfg) : launch_eb<R, Q, 1024>(a, s, p, gn, cfg));
  }
}

template <typename R>
static hipError_t launch_r(const EstArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  switch (a.Q) {
    case 2: return launch_e<R, 2>(a, s, p, gn, cfg);
    case 4: return launch_e<R, 4>(a, s, p, gn, cfg);
    case 8: return launch_e<R, 8>(a, s, p, gn, cfg);
    case 16: return launch_e<R, 16>(a, s, p, gn, cfg);
  }
  return hipErrorInvalidValue;
}

// The order of the residual sums of a shape with C chains (EstArgs::res), whatever the launch's size: one
// thread per sum for the shapes of at most 256 marginal rows, matrix cores for the others, their K steps in two halves
// where the chains that fit 96 KiB of LDS with 20 bytes per (chain, antenna) make at most 8 tiles for a workgroup's 16
// waves.  (Any one order would do; changing a shape's moves its marginals by up to 1e-2 where |f| is 1e5.)
static int estimate_res(int nt, int nr, int Q, int C, bool fp64) {
  const int bs = estimate_threads(nt, nr, Q, C, fp64, 1 << 30);
  if (fp64 || bs == 256) return 0;
  if (bs == 512) return 1;
  int ch = C;
  while (ch > 1 && 20 * (size_t)ch * nt + 4 * (3 * (size_t)ch * nr + 4 * (size_t)ch + nt + 2 * (size_t)nr) + 4 * (size_t)ch * nt + 16 > 96 * 1024)
    ch = (ch + 1) / 2;
  const int units = ((nr + 15) / 16) * ((ch + 15) / 16);
  return 2 * units <= 16 && (size_t)units * 4096 <= (size_t)ch * nt * 20 ? 2 : 1;
}

void estimate_shape(EstArgs* ea, int nt, int nr, int M, int N, int C, bool fp64, int n_inst) {
  const int Q = M <= 4 ? 2 : (M <= 16 ? 4 : (M <= 64 ? 8 : 16));
  ea->threads = estimate_threads(nt, nr, Q, C, fp64, n_inst);
  ea->res = estimate_res(nt, nr, Q, C, fp64);
  ea->chunk = estimate_chunk(nt, nr, Q, N, C, fp64, ea->threads);
  estimate_groups(nt, nr, Q, C, &ea->gm, &ea->gl);
}

hipError_t launch_estimate(const EstArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  return a.fp64 ? launch_r<double>(a, s, p, gn, cfg) : launch_r<float>(a, s, p, gn, cfg);
}

}  // namespace dmala
