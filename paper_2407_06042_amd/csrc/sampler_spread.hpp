// The chain kernel for launches that leave SIMDs idle: a 16-chain block spread over more waves.
//
// sampler_impl.hpp gives a wave 16 (or 8) dimensions of every chain per lane, which keeps the most
// work per instruction when the chip is full; with few chain blocks a transition then takes one
// wave's serial issue time (about 3.5 us at 64 dimensions) while most SIMDs have nothing to do.  Here
// a wave owns four dimensions of every chain per lane, so that a block runs on four times (layout 0:
// twice) the waves, in one workgroup.
//
// The results are bit for bit those of the base layout (RTW row tiles per wave, WD waves):
// the contraction keeps its products and their order, every per-dimension value is computed by the
// same functions, and the sums over a base wave's dimensions -- fused multiply-adds per lane in a fixed
// order (add_square) -- are taken in the same sequence: the factors go through LDS, and each of the four chains of
// sums (forward and reverse proposal, energy, log normaliser) is run by one wave of the block.  Three
// barriers per transition: proposed levels, factors, sums.
//
// What the few registers per wave leave room for: the packed matrices stay in registers (no LDS or
// L2 stream), and the draw's cumulative weights are kept until a chain of the block accepts (most
// transitions of a settled chain are rejected, and then only the random words change).
#pragma once
#include "sampler_impl.hpp"

namespace dmala {

// v summed over the chain's four lanes, as bfly4 does ((v0 + v1) + (v2 + v3) in every lane), by
// exchanges of 16- and 32-lane rows instead of LDS permutes.
__device__ __forceinline__ float rows4(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// LDS of a workgroup: the proposed levels (MFMA B operands), the factors of the sums (6 values per
// dimension), the sums, the accept uniforms, the random words shared by the waves of an antenna tile,
// the window table.
constexpr int kSpreadTerms = 6;
constexpr size_t spread_lds(int rt, int wd, bool cx, int win) {
  return (size_t)(rt / 2) * 1024 + (size_t)kSpreadTerms * rt * 1024 + (size_t)wd * 4 * 256 + 256 +
         (cx ? (size_t)rt * 512 : 0) + (win > 0 ? kCtabBytes : 0);
}

// One wave per four dimensions of a lane: real-equivalent layouts (CX false), row tile `wave`, dimensions
// 16 wave + 4 h + d; complex planes, antenna tile at = wave / 2 and its real (wave even) or imaginary
// parts, dimensions 32 at + 8 h + 2 d + wave % 2, so that a wave multiplies for its own outputs only.
template <int RTW, int WD, int Q, int PM, int WIN, bool CX>
__device__ __forceinline__ void spread_body(const SamplerArgs& a, const int inst, const int cblock) {
  static_assert(PM != PM_NAIVE && (!CX || RTW == 4), "preconditioned float chains; complex planes: two antenna tiles per slice");
  constexpr int RT = RTW * WD, D = 4;
  constexpr int KB = CX ? RT / 4 : RT / 2;               // K blocks (32 antennas, or 32 dimensions)
  constexpr int NPP = p_passes(PM), NP = NPP + kEPasses, QM1 = Q - 1;
  constexpr int W = WIN > 0 ? WIN : Q - 1;
  constexpr int NC = WIN > 0 ? 2 * W : Q - 1;            // partial sums a draw compares against
  constexpr int AT = RT / 2;
  constexpr size_t PASS = CX ? (size_t)RT * RT / 4 * 1024 : (size_t)RT * KB * 1024;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int N = a.N, Npad = a.Npad;
  const unsigned char* blk = a.ws_inst + (size_t)inst * a.inst_stride;
  const uint32_t rid = a.desc ? (uint32_t)a.desc[inst].orig : (uint32_t)inst;
  const uint32_t rctr = rid + a.ctr_base;
  const size_t fs_base = a.desc ? (size_t)a.desc[inst].fs_off : (size_t)inst * a.C * N;
  const int lane = threadIdx.x & 63, cl = lane & 15, h = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wd = wave / RTW, ws = wave % RTW;            // slice (a base wave's dimensions), wave of the slice
  const int at = wave >> 1, part = wave & 1;             // complex planes: antenna tile, real or imaginary
  const int chain = cblock * 16 + cl;
  const bool live = chain < a.C;

  if (((const InstParams*)blk)->nonfinite) {
    // a flagged instance: the optional per-chain outputs as zeros
    if (live && h == 0 && wave == 0) {
      const size_t trow = (size_t)rid * a.C + chain;
      if (a.accept_count) a.accept_count[trow] = 0;
      if (a.final_state)
        for (int n = 0; n < N; ++n) a.final_state[fs_base + (size_t)chain * N + n] = 0;
      if (a.trace_accept)
        for (int w = 0; w < a.trace_words; ++w) a.trace_accept[trow * a.trace_words + w] = 0u;
      if (a.trace_hash)
        for (int t = 0; t < a.T; ++t) a.trace_hash[trow * a.T + t] = 0u;
      if (a.train_rows) {
        const int Nt = N >> 1;
        const int64_t sym0 = a.desc ? a.desc[inst].sym_off : (int64_t)inst * Nt;
        float* row = a.train_rows + ((size_t)sym0 * a.C + (size_t)chain * Nt) * kTrainRow;
        for (int i = 0; i < Nt * kTrainRow; ++i) row[i] = 0.f;
      }
    }
    return;
  }

  unsigned char* xbuf = smem;                                            // RT / 2 KiB
  f32x4* term = (f32x4*)(xbuf + (size_t)(RT / 2) * 1024);                // [factor][wave][lane]
  float* res = (float*)(term + (size_t)kSpreadTerms * RT * 64);          // [slice][sum][lane]
  float* lub = res + WD * 4 * 64;                                        // [lane]
  uint2* wbuf = (uint2*)(lub + 64);                                      // complex planes: [wave][lane]
  float* ctab_p = (float*)(wbuf + (CX ? RT * 64 : 0));
  auto put = [&](int f, const float (&v)[D]) { term[(f * RT + wave) * 64 + lane] = f32x4{v[0], v[1], v[2], v[3]}; };
  // factor f of the slice's dimensions, in the order of a base lane's dimensions
  auto get = [&](int f, float (&v)[4 * RTW]) {
    const f32x4* src = term + (f * RT + wd * RTW) * 64 + lane;
#pragma unroll
    for (int g = 0; g < RTW; ++g) {
      const f32x4 x = src[g * 64];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[CX ? (g >> 1) * 8 + 2 * i + (g & 1) : 4 * g + i] = x[i];
    }
  };

  const InstParams ip = *(const InstParams*)blk;
  WinCoef wc;
  wc.tab = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)ctab_p;
  wc.dmax = fmaxf(0.5f, 12.5f / (float)ip.kL);
  if constexpr (WIN > 0) ctab_fill<Q>(ctab_p, (float)ip.kL);
  // (constants of the transition loop in vector registers: an operation with a scalar operand issues at
  // half the rate, 4.3 instead of 2.6 cycles with two waves per SIMD)
  float kL = (float)ip.kL, sP = ip.scaleP, sE = ip.scaleE, kB = 0x1p100f;
  asm volatile("" : "+v"(kL), "+v"(sP), "+v"(sE), "+v"(kB));
  const float* pbv = (const float*)(blk + kParamBytes + (size_t)NP * PASS);
  const float* ezv = pbv + Npad;
  const float* afv = ezv + Npad;
  const int dim0 = CX ? 32 * at + 8 * h + part : 16 * wave + 4 * h;
  auto dim_of = [&](int d) { return dim0 + (CX ? 2 * d : d); };

  // the wave's matrix fragments, in registers for every transition: both planes of its antenna tile, or
  // its row tile
  constexpr int NF = CX ? 2 : 1;
  half8 fr[NP][NF][KB];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const size_t o = CX ? (size_t)((p * 2 + f) * AT + at) * KB + kb : (size_t)(p * RT + wave) * KB + kb;
        fr[p][f][kb] = *(const half8*)(blk + kParamBytes + o * 1024 + lane * 16);
      }
  float pb[D], ez[D];
  bool valid[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    pb[d] = pbv[dim_of(d)];
    ez[d] = ezv[dim_of(d)];
    valid[d] = dim_of(d) < N;
  }

  // Random words.  A wave generates one block of the stream; with complex planes block 2 at + part holds
  // (Re, Im) of antennas 2 part, 2 part + 1 of the lane's four, and the tile's two waves exchange halves.
  const uint32_t key0 = a.key0, key1 = a.key1;
  uint32_t w[4], wown[2], lubits;
  struct Rounds { uint32_t c[4], k0, k1; };
  auto words_begin = [&](int tt) {
    return Rounds{{(uint32_t)(CX ? (32 * at + 8 * h + 4 * part) >> 2 : dim0 >> 2), (uint32_t)tt, (uint32_t)chain, rctr}, key0, key1};
  };
  auto words_round = [&](Rounds& s) {
    philox4x32_round<true>(s.c, s.k0, s.k1);
    s.k0 += 0x9E3779B9u;
    s.k1 += 0xBB67AE85u;
  };
  auto words_end = [&](const Rounds& s) {
    const uint32_t* c = s.c;
    lubits = low_bytes24(c[0], c[1], c[2]);   // the accept uniform, in wave 0's lanes h = 0
    if constexpr (CX) {
      wown[0] = part ? c[1] : c[0];
      wown[1] = part ? c[3] : c[2];
      wbuf[wave * 64 + lane] = part ? make_uint2(c[0], c[2]) : make_uint2(c[1], c[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = c[i];
    }
  };
  auto words = [&](int tt) {
    Rounds s = words_begin(tt);
#pragma unroll
    for (int r = 0; r < 10; ++r) words_round(s);
    words_end(s);
  };
  auto take_words = [&]() {   // after the barrier that follows words()
    if constexpr (CX) {
      const uint2 o = wbuf[(wave ^ 1) * 64 + lane];
      w[0] = part ? o.x : wown[0];
      w[1] = part ? o.y : wown[1];
      w[2] = part ? wown[0] : o.x;
      w[3] = part ? wown[1] : o.y;
    }
  };

  // proposed levels into the B operands, and (after a barrier) the contraction, with the products
  // in the base layout's order
  auto put_levels = [&](const float (&k)[D]) {
    const int o = CX ? (part * KB + (at >> 1)) * 1024 + lane * 16 + (at & 1) * 8 : (wave >> 1) * 1024 + lane * 16 + (wave & 1) * 8;
    *(uint2*)(xbuf + o) = make_uint2(lv_pair<QM1>(k[0], k[1]), lv_pair<QM1>(k[2], k[3]));
  };
  auto mma = [&](bool energy, half8 m, half8 x, bf16x8 b, f32x4 c) {
    if constexpr (PM == PM_BF16X1) {
      if (!energy) {
        bf16x8 mb;
        __builtin_memcpy(&mb, &m, 16);
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(mb, b, c, 0, 0, 0);
      }
    }
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(m, x, c, 0, 0, 0);
  };
  auto to_bf = [](half8 x) {
    bf16x8 b;
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = (__bf16)(float)x[j];
    return b;
  };
  // (between(i) runs after the i-th pair of products: independent work that fills their latency)
  auto grad_at = [&](const float (&k)[D], float (&mu)[D], float (&eg)[D], auto&& between) {
    // complex planes: Re = re x_re + im (-x_im), Im = im x_re + re x_im, the first and second operand
    // of each product pair in (m0, x0), (m1, x1)
    half8 x0[KB], x1[CX ? KB : 1];
    bf16x8 b0[KB], b1[CX ? KB : 1];
    const uint32_t sgn = part ? 0u : 0x80008000u;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      x0[kb] = *(const half8*)(xbuf + kb * 1024 + lane * 16);
      if constexpr (PM == PM_BF16X1) b0[kb] = to_bf(x0[kb]);
      if constexpr (CX) {
        uint4 u = *(const uint4*)(xbuf + (KB + kb) * 1024 + lane * 16);
        u.x ^= sgn; u.y ^= sgn; u.z ^= sgn; u.w ^= sgn;   // exact: the levels are never zero
        __builtin_memcpy(&x1[kb], &u, 16);
        if constexpr (PM == PM_BF16X1) b1[kb] = to_bf(x1[kb]);
      }
    }
    f32x4 e = {0.f, 0.f, 0.f, 0.f}, q = e;
    // product i of a matrix: pass i / (KB NF), K block, plane
    auto step = [&](int i, bool en, f32x4 c) {
      const int p = i / (KB * NF), kb = (i / NF) % KB, f = i % NF;
      return f == 0 ? mma(en, fr[en ? NPP + p : p][0][kb], x0[kb], b0[kb], c)
                    : mma(en, fr[en ? NPP + p : p][NF - 1][kb], x1[CX ? kb : 0], b1[CX ? kb : 0], c);
    };
#pragma unroll
    for (int i = 0; i < kEPasses * KB * NF; ++i) {
      e = step(i, true, e);
      if (i < NPP * KB * NF) q = step(i, false, q);
      between(i);
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
      eg[d] = e[d] * sE - ez[d];
      mu[d] = k[d] - (q[d] * sP - pb[d]);
    }
  };
  if constexpr (CX) {
    // the imaginary wave multiplies (im, x_re) first: its planes in that order
    if (part) {
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const half8 t = fr[p][0][kb];
          fr[p][0][kb] = fr[p][1][kb];
          fr[p][1][kb] = t;
        }
    }
  }

  // Proposal weights at centre mu: the draw's partial sums cum and total Z (ascending levels) and mode jf,
  // as window_weights and draw_level form them; the reverse normaliser's weight sum Zr and mode offset b, as
  // norm_parts does.
  struct Prop { float cum[D][NC], Z[D], jf[D]; };
  auto weights_at = [&](const float (&mu)[D], Prop& o, float (&Zr)[D], float (&b)[D]) {
    float F[D], G[D], cu[D][W], cd[D][W];
    if constexpr (WIN > 0) {
      // every dimension's table reads in flight before the first is used
#pragma unroll
      for (int d = 0; d < D; ++d) window_coefs<Q, W, true>(mu[d], kL, wc, F[d], G[d], cu[d], cd[d], o.jf[d], b[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if constexpr (WIN > 0) {
        const float zu = __builtin_fmaf(F[d], __builtin_fmaf(F[d], __builtin_fmaf(F[d], cu[d][2], cu[d][1]), cu[d][0]), 1.0f);
        Zr[d] = __builtin_fmaf(G[d], __builtin_fmaf(G[d], __builtin_fmaf(G[d], cd[d][2], cd[d][1]), cd[d][0]), zu);
        const float F2 = F[d] * F[d], G2 = G[d] * G[d];
        float s = cd[d][2] * (G2 * G[d]);
        o.cum[d][0] = s;
        s += cd[d][1] * G2; o.cum[d][1] = s;
        s += cd[d][0] * G[d]; o.cum[d][2] = s;
        s += 1.0f; o.cum[d][3] = s;
        s += cu[d][0] * F[d]; o.cum[d][4] = s;
        s += cu[d][1] * F2; o.cum[d][5] = s;
        s += cu[d][2] * (F2 * F[d]);
        o.Z[d] = s;
      } else {
        float e[Q], b2;
        level_weights<Q>(mu[d], kL, e, b2);
        o.jf[d] = mode_of<Q>(mu[d]);
        b[d] = o.jf[d] - mu[d];
        float s = e[0];
#pragma unroll
        for (int j = 1; j < Q; ++j) {
          o.cum[d][j - 1] = s;
          s += e[j];
        }
        o.Z[d] = s;
        Zr[d] = s;
      }
    }
  };

  words(0);
  __syncthreads();
  take_words();
  float kc[D], mu[D], eg[D];
#pragma unroll
  for (int d = 0; d < D; ++d) kc[d] = float((int)(((uint64_t)(w[d] >> 8) * Q) >> 24));
  put_levels(kc);
  __syncthreads();
  grad_at(kc, mu, eg, [](int) {});
  // initial energy and log normaliser sums, one value per dimension through the factors
  float lz[D], et[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    lz[d] = log2_norm<Q, WIN, W, (WIN > 0)>(mu[d], kL, wc);
    et[d] = valid[d] ? (2 * kc[d] - QM1) * (eg[d] - ez[d]) : 0.f;
  }
  put(0, et);
  put(1, lz);
  words(1);
  __syncthreads();
  take_words();
  if (ws < 2) {
    float v[4 * RTW], s = 0.f;
    get(ws, v);
#pragma unroll
    for (int i = 0; i < 4 * RTW; ++i) s += v[i];
    res[(wd * 4 + ws) * 64 + lane] = s;
  }
  __syncthreads();
  float lzs[WD], ep = 0;
#pragma unroll
  for (int sl = 0; sl < WD; ++sl) {
    const float e = rows4(res[sl * 4 * 64 + lane]);
    ep = sl ? ep + e : e;
    lzs[sl] = res[(sl * 4 + 1) * 64 + lane];
  }
  __syncthreads();
  const float eunit = (float)ip.eunit;
  float E = (float)ip.yy + 0.5f * eunit * ep;
  float Ebest = E;
  auto pack = [&]() { return (uint32_t)kc[0] | ((uint32_t)kc[1] << 8) | ((uint32_t)kc[2] << 16) | ((uint32_t)kc[3] << 24); };
  uint32_t kbest = pack();
  int nacc = 0;
  uint32_t abits = 0;
  const size_t trow = (size_t)rid * a.C + (live ? chain : 0);

  Prop cur;
  {
    float z_[D], b_[D];
    weights_at(mu, cur, z_, b_);
  }
  // The three barriers of a transition order the shared arrays, each with one between its last read and its next
  // write as well as between its write and its reads:
  //   xbuf: written before the first, read between first and second;
  //   term: factor 0 written before the first, 1 to 5 between first and second, read between second and third;
  //   wbuf: written between first and second, read between second and third;
  //   lub: written between first and second, read after the third (and so before the next first);
  //   res: written between second and third, read after the third.
  for (int t = 1; t <= a.T; ++t) {
    // draw x' (inverse CDF; the arithmetic of draw_level)
    float kp[D], t0[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if constexpr (WIN > 0) {
        const float tB = u23f_x2p100(w[d]) * cur.Z[d];
        float in[2 * W];
#pragma unroll
        for (int i = 0; i < 2 * W; ++i) in[i] = __builtin_amdgcn_fmed3f(0.0f, 1.0f, __builtin_fmaf(cur.cum[d][i], kB, -tB));
        static_assert(W == 3, "six partial sums");
        // (small integers: exact in any order)
        const float above = ((in[0] + in[1]) + (in[2] + in[3])) + (in[4] + in[5]);
        kp[d] = __builtin_amdgcn_fmed3f((cur.jf[d] + float(W)) - above, 0.0f, float(Q - 1));
      } else {
        const float target = u23f(w[d]) * cur.Z[d];
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < Q - 1; ++j) cnt += (cur.cum[d][j] <= target) ? 1 : 0;
        kp[d] = float(cnt);
      }
    }
    // (all four drawn before the padding masks: otherwise every mask becomes a branch around its draw)
    asm volatile("" : "+v"(kp[0]), "+v"(kp[1]), "+v"(kp[2]), "+v"(kp[3]));
#pragma unroll
    for (int d = 0; d < D; ++d) {
      kp[d] = valid[d] ? kp[d] : kc[d];
      t0[d] = kp[d] - mu[d];
    }
    put_levels(kp);
    put(0, t0);
    const float lu0 = lg2((float)lubits * 5.9604644775390625e-08f);   // (wave 0's)
    __syncthreads();
    // (not earlier: a late wave still reads the last transition's until it reaches the barrier above)
    if (wave == 0) lub[lane] = h == 0 ? lu0 : 0.f;
    float mup[D], egp[D];
    // The next transition's random words.  With one wave per SIMD (64 dimensions) their rounds are pinned
    // between the products, whose latency they fill (139 against 142 us per 100 transitions); with two
    // the waves fill each other's gaps and the pinning costs (218 against 207 us at 128 dimensions).
    constexpr bool kPin = CX && KB == 1;
    Rounds rd = words_begin(t + 1);
    if constexpr (kPin) {
      constexpr int kPairs = kEPasses * KB * NF;
      grad_at(kp, mup, egp, [&](int i) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 10 * i / kPairs; r < 10 * (i + 1) / kPairs; ++r) words_round(rd);
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {
      asm volatile("" : "+v"(rd.c[0]));   // keeps the rounds on this side of the barrier
#pragma unroll
      for (int r = 0; r < 10; ++r) words_round(rd);
      grad_at(kp, mup, egp, [](int) {});
    }
    words_end(rd);
    Prop nxt;
    {
      float tr[D], df[D], sg[D], Zr[D], bs[D];
      weights_at(mup, nxt, Zr, bs);
#pragma unroll
      for (int d = 0; d < D; ++d) {
        tr[d] = kc[d] - mup[d];
        df[d] = kp[d] - kc[d];
        sg[d] = eg[d] + egp[d];
      }
      put(1, tr);
      put(2, df);
      put(3, sg);
      put(4, Zr);
      put(5, bs);
    }
    __syncthreads();
    take_words();
    // the sums over the slice's dimensions, each in the base layout's sequence, by one of its waves
#pragma unroll
    for (int k = 0; k < 4 / RTW; ++k) {
      const int task = ws + k * RTW;
      float v[4 * RTW], u[4 * RTW], r;
      auto squares = [&](auto paired) {
        get(task, v);
        float first = 0.f;
        r = 0.f;
#pragma unroll
        for (int i = 0; i < 4 * RTW; ++i) add_square<decltype(paired)::value>(i, v[i], first, r);
      };
      if (task == 0 && !forward_paired(RTW, WD)) {
        squares(std::false_type{});
      } else if (task < 2) {
        squares(std::true_type{});
      } else if (task == 2) {
        get(2, v);
        get(3, u);
        r = 0.f;
#pragma unroll
        for (int i = 0; i < 4 * RTW; ++i) r = __builtin_fmaf(-v[i], u[i], r);
      } else {
        get(4, v);
        get(5, u);
        float z = 1.f, s = 0.f, u0 = 0.f;
#pragma unroll
        for (int i = 0; i < 4 * RTW; ++i) { z *= v[i]; add_square<true>(i, u[i], u0, s); }
        r = __builtin_fmaf(-s, kL, lg2(z));
      }
      res[(wd * 4 + task) * 64 + lane] = r;
    }
    __syncthreads();
    // MH test, as every wave of the block sees it
    float S = 0, T2 = 0, lzn[WD];
    const float lu = lub[lane];
#pragma unroll
    for (int sl = 0; sl < WD; ++sl) {
      const float* r = res + sl * 4 * 64 + lane;
      lzn[sl] = r[192];
      float s = __builtin_fmaf(r[0], kL, lzs[sl]) - __builtin_fmaf(r[64], kL, lzn[sl]);
      s = r[128] + s;
      if (sl == 0) s -= lu;
      s = rows4(s);
      const float t2 = rows4(r[128]);
      S = sl ? S + s : s;
      T2 = sl ? T2 + t2 : t2;
    }
    const bool acc = S > 0.f;
    // Accepted chains take over the proposal's values: moves under the lanes' mask, skipped when every
    // chain rejects (an empty asm keeps the branch: as selects on vcc they measured 17 cycles each)
    if (acc) {
      asm volatile("");
#pragma unroll
      for (int d = 0; d < D; ++d) {
        kc[d] = kp[d];
        mu[d] = mup[d];
        eg[d] = egp[d];
        cur.Z[d] = nxt.Z[d];
        cur.jf[d] = nxt.jf[d];
#pragma unroll
        for (int i = 0; i < NC; ++i) cur.cum[d][i] = nxt.cum[d][i];
      }
#pragma unroll
      for (int sl = 0; sl < WD; ++sl) lzs[sl] = lzn[sl];
      E = E - T2 * eunit;
      nacc += 1;
      if (E < Ebest) {
        asm volatile("");
        Ebest = E;
        kbest = pack();
      }
    }
    if (a.trace_accept) {
      abits |= (acc ? 1u : 0u) << ((t - 1) & 31);
      if (((t & 31) == 0 || t == a.T) && live && h == 0 && wave == 0)
        a.trace_accept[trow * a.trace_words + ((t - 1) >> 5)] = abits;
      if ((t & 31) == 0) abits = 0;
    }
    if (a.trace_hash) {
      uint32_t hs = 0;
#pragma unroll
      for (int d = 0; d < D; ++d) hs += valid[d] ? ((uint32_t)kc[d] + 1u) * hash_mult(dim_of(d)) : 0u;
      hs += __shfl_xor(hs, 16);
      hs += __shfl_xor(hs, 32);
      uint32_t* hb = (uint32_t*)(term + RT * 64);   // factor 1: read by now, next written after a barrier
      if (h == 0) hb[wave * 16 + cl] = hs;
      __syncthreads();
      if (wave == 0 && h == 0 && live) {
        uint32_t s = 0;
        for (int i = 0; i < RT; ++i) s += hb[i * 16 + cl];
        a.trace_hash[trow * a.T + (t - 1)] = s;
      }
    }
  }

  if (a.train_rows) {
    // training rows at the final state (as the base kernel's): a row needs both parts of an antenna
    put(2, kc);
    put(3, mu);
    __syncthreads();
    const int Nt = N >> 1;
    const int64_t sym0 = a.desc ? a.desc[inst].sym_off : (int64_t)inst * Nt;
    constexpr float kCq = 0.5f * (Q - 1), kIhq = 2.0f / Q;
    if (live && (!CX || part == 0)) {
      const f32x4 kx = term[(2 * RT + (CX ? wave + 1 : wave)) * 64 + lane], mx = term[(3 * RT + (CX ? wave + 1 : wave)) * 64 + lane];
#pragma unroll
      for (int i = 0; i < (CX ? 4 : 2); ++i) {
        const int ant = CX ? 16 * at + 4 * h + i : (dim0 >> 1) + i;
        const float mr = CX ? mu[i] : mu[2 * i], mi = CX ? mx[i] : mu[2 * i + 1];
        const float kr = CX ? kc[i] : kc[2 * i], ki = CX ? kx[i] : kc[2 * i + 1];
        if (ant < Nt) {
          float* row = a.train_rows + ((size_t)sym0 * a.C + (size_t)chain * Nt + ant) * kTrainRow;
          row[0] = (mr - kCq) * kIhq;
          row[1] = (mi - kCq) * kIhq;
          row[2] = (kr - kCq) * kIhq;
          row[3] = (ki - kCq) * kIhq;
          row[4] = afv[2 * ant];
          row[5] = afv[2 * ant + 1];
          row[6] = 0.25f * (Q == 2 ? 1.f : Q == 4 ? 2.f : Q == 8 ? 3.f : 4.f);
          row[7] = mr;
          row[8] = mi;
          row[9] = kL / float(kLog2e);
          row[10] = (float)Q;
          row[11] = 0.f;
        }
      }
    }
  }
  if (!live) return;
  const StateOff so = state_offsets(a.Cpad, Npad);
  unsigned char* st = a.ws_state + (size_t)inst * a.state_stride;
  float* egs = (float*)(st + so.eg) + (size_t)chain * Npad;
  int8_t* ks = (int8_t*)(st + so.k) + (size_t)chain * Npad;
  int8_t* kb = (int8_t*)(st + so.kbest) + (size_t)chain * Npad;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const int n = dim_of(d);
    egs[n] = valid[d] ? eg[d] : 0.0f;
    ks[n] = (int8_t)(int)kc[d];
    kb[n] = (int8_t)(kbest >> (8 * d));
    if (a.final_state && valid[d]) a.final_state[fs_base + (size_t)chain * N + n] = (int8_t)(int)kc[d];
  }
  if (h == 0 && wave == 0) {
    ((double*)(st + so.ebest))[chain] = (double)Ebest;
    ((int32_t*)(st + so.nacc))[chain] = nacc;
    if (a.accept_count) a.accept_count[(size_t)rid * a.C + chain] = nacc;
  }
}

template <int RTW, int WD, int Q, int PM, int WIN, bool CX, bool PERS>
__global__ __launch_bounds__(64 * RTW * WD) void spread_kernel(SamplerArgs a, Persist p) {
  if constexpr (!PERS) {
    spread_body<RTW, WD, Q, PM, WIN, CX>(a, blockIdx.x, blockIdx.y);
  } else {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    for (;;) {
      const int it = persist_take(p, smem);
      if (it >= p.n_items) break;
      const WorkItem w = p.items[it];
      const SamplerArgs ca = ((const SamplerArgs*)p.cls)[__builtin_amdgcn_readfirstlane(w.cls)];
      spread_body<RTW, WD, Q, PM, WIN, CX>(ca, __builtin_amdgcn_readfirstlane(w.inst),
                                               __builtin_amdgcn_readfirstlane(w.cg));
    }
    persist_done(p);
  }
}

template <int RTW, int WD, int Q, int PM, int WIN, bool CX>
hipError_t launch_spread_t(const Shape& sh, const SamplerArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  const size_t lds = (spread_lds(RTW * WD, WD, CX, WIN) + 15) & ~(size_t)15;
  constexpr int threads = 64 * RTW * WD;
  void (*k)(SamplerArgs, Persist) = (p || cfg) ? spread_kernel<RTW, WD, Q, PM, WIN, CX, true>
                                               : spread_kernel<RTW, WD, Q, PM, WIN, CX, false>;
  const dim3 grid(a.n_inst, sh.Cpad / 16);
  if (cfg) {
    cfg->k = (const void*)k;
    cfg->threads = threads;
    cfg->lds = lds;
    cfg->gx = (int)grid.x;
    cfg->gy = (int)grid.y;
    return hipSuccess;
  }
  const size_t lds_run = p ? ((p->lds_off + 4 + 15) & ~(size_t)15) : lds;
  if (lds_run > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_run);
    if (e != hipSuccess) return e;
  }
  if (p) hipLaunchKernelGGL(k, dim3(gn), dim3(threads), lds_run, s, a, *p);
  else hipLaunchKernelGGL(k, grid, dim3(threads), lds, s, a, Persist{});
  return hipGetLastError();
}

template <int RTW, int WD, int PM, bool CX>
hipError_t launch_spread_q(const Shape& sh, const SamplerArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  const bool win = sh.win == 3;
  switch (sh.Q) {
    case 2: return launch_spread_t<RTW, WD, 2, PM, 0, CX>(sh, a, s, p, gn, cfg);
    case 4: return launch_spread_t<RTW, WD, 4, PM, 0, CX>(sh, a, s, p, gn, cfg);
    case 8: return win ? launch_spread_t<RTW, WD, 8, PM, 3, CX>(sh, a, s, p, gn, cfg)
                       : launch_spread_t<RTW, WD, 8, PM, 0, CX>(sh, a, s, p, gn, cfg);
    case 16: return win ? launch_spread_t<RTW, WD, 16, PM, 3, CX>(sh, a, s, p, gn, cfg)
                        : launch_spread_t<RTW, WD, 16, PM, 0, CX>(sh, a, s, p, gn, cfg);
  }
  return hipErrorInvalidValue;
}

// The spread form of the base layouts 0 (32 dimensions), 9 (64) and 7 (128).
template <int PM>
hipError_t launch_spread_pm(const Shape& sh, const SamplerArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  switch (sh.cfg) {
    case 0: return launch_spread_q<2, 1, PM, false>(sh, a, s, p, gn, cfg);
    case 9: return launch_spread_q<4, 1, PM, true>(sh, a, s, p, gn, cfg);
    case 7: return launch_spread_q<4, 2, PM, true>(sh, a, s, p, gn, cfg);
  }
  return hipErrorInvalidValue;
}

}  // namespace dmala
