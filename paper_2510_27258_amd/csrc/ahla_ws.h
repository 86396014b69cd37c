// Wave-specialised AHLA walk for d = 128 on 64-token tiles and its two-pass
// plan.  Included by ahla.hip only.
//
// Per tile (rows = the tile's tokens; P0, m0, E0, n0 the carry before it):
//   A = L (.) Q K^T,  R = A V + Q P0,  s = A 1 + Q m0,
//   P0 += K^T V,  m0 += K^T 1                                  (P side)
//   O = A R + Q E0,  den = A s + Q n0,  E0 += K^T R,  n0 += K^T s   (E side)
// The P side of tile c + 1 does not depend on the E side of tile c, which
// needs only A, R and s of tile c.  So waves 0-3 hold P0 (wave w: columns
// 32w .. 32w + 31, all 128 rows) and run the P side one tile ahead, while
// waves 4-7 hold E0 the same way and run the E side; each SIMD has one wave of
// each with independent work.  They meet at three barriers a tile:
//   phase 1: A_{c+1}, Q P0;             Q E0, the rows' denominators
//   phase 2: A V, the P0 advance;       A R, the E0 and n0 advances
//   phase 3: R_{c+1} and s_{c+1} stored; O_c stored; the next tiles staged.
// Q, K and A are double-buffered (the E side reads them one tile later); the
// output goes through the E side's A tile, dead after phase 2, a row tile at a
// time.  Numerics as k_ahla_walk.
//
// Two-pass plan (ws_plan): the first launch walks segment 0's output beside
// summary walks of segments 1 .. P-2 from a zero state, which also form K^T Q
// and write no output; k_ws_bracket and k_seg_prefix make the true carries;
// the second launch walks the outputs of segments 1 .. P-1, each row final
// (divided) when written.  Against one walk from the P prefix (a moments
// launch before it, a fix-up over every row after it), at one wave a SIMD
// with both state columns, 64 heads of 8000 tokens: 431 -> 329 us, on another box 428 -> 313 (walk 316,
// fix-up 92, moments 73 against first launch 135, outputs 178, brackets 17, sums 7).
#pragma once
#include "ws_common.h"

namespace hla {
namespace {

struct CfgAW {
  static constexpr int C = 64, D = 128, DV = 128;
  static constexpr int NT = 512;                                 // 8 waves
  static constexpr int ldQ = D + kPad, ldK = D + kPad;
  static constexpr int ldV = DV + 16;                            // read through the transpose unit only
  static constexpr int ldA = C + kPad, ldR = C + kPad;
  static constexpr int sQ = C * ldQ, sK = C * ldK, sA = 2 * C * ldA;   // one buffer (A: hi, then lo)
  static constexpr int oQ = 0, oK = oQ + 2 * sQ, oV = oK + 2 * sK, oA = oV + C * ldV;
  static constexpr int oRh = oA + 2 * sA, oRl = oRh + DV * ldR;  // R^T[column][token]
  static constexpr int n16 = oRl + DV * ldR;
  static constexpr int f_m = 0, f_n = D, f_s = 2 * D, f_rs = f_s + C, f_inv = f_rs + 96;
  static constexpr int nf32 = f_inv + C;
  static constexpr size_t bytes = (size_t)n16 * 2 + (size_t)nf32 * 4;
  static constexpr int PF = C * D / 8 / NT;                      // 16-byte pieces per thread per operand
  static_assert(PF * NT * 8 == C * D && (n16 * 2) % 16 == 0, "staging split");
  static_assert(4 * 32 * 32 * 4 <= sA * 2, "output staging fits an A buffer");
  static_assert(bytes <= 160 * 1024, "LDS budget");
};

// One segment's walk over tiles [c_begin, c_begin + nt) of head bh.  p_in: P0
// then m0 at the start (null: zero); e_in: E0 then n0 (null: zero; unused by
// SUMMARY); rec: this segment's record (null: none), which receives the ending
// P, m, E, n in its C, m, G and h slots (m and n: zero unless normalized), and
// with SUMMARY K^T Q in its S slot.
template <bool SUMMARY>
__device__ __forceinline__ void walk_aw(uint16_t* lds, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                        const uint16_t* __restrict__ v, float* __restrict__ out,
                                        const float* __restrict__ p_in, const float* __restrict__ e_in,
                                        float* __restrict__ rec, int bh, int n, int c_begin, int nt, int normalized,
                                        float eps) {
  using G = CfgAW;
  constexpr int C = G::C, D = G::D, DV = G::DV, NT = G::NT;
  uint16_t* Vs = lds + G::oV;
  uint16_t* Rh = lds + G::oRh;
  uint16_t* Rl = lds + G::oRl;
  float* fl = reinterpret_cast<float*>(lds + G::n16);
  float* m0 = fl + G::f_m;        // P side: m before its tile
  float* n0 = fl + G::f_n;        // E side: n before its tile
  float* sv = fl + G::f_s;        // s of the E side's tile
  float* rs = fl + G::f_rs;       // row sums of A: key tile 0 over 64 queries, key tile 1 over queries 32 ..
  float* inv = fl + G::f_inv;     // 1 / (den_t + eps)

  const int tid = threadIdx.x, l = tid & 63, lr = l & 31, lg = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool pside = w < 4;
  const int cw = w & 3;           // this wave's state column tile

  f32x16 st[4];                   // rows 32i .. 32i + 31 of column tile cw of P0 or E0
  {
    const float* src = pside ? p_in : (SUMMARY ? nullptr : e_in);
    if (src) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) st[i][e] = src[(size_t)(32 * i + acc_row(e, lg)) * DV + cw * 32 + lr];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) st[i] = zero16();
    }
  }
  f32x16 qk[SUMMARY ? 4 : 1];     // SUMMARY, E side: column tile cw of K^T Q
#pragma unroll
  for (int i = 0; i < (SUMMARY ? 4 : 1); ++i) qk[i] = zero16();
  if (tid < D) {
    m0[tid] = p_in ? p_in[D * DV + tid] : 0.f;
    n0[tid] = !SUMMARY && e_in ? e_in[D * DV + tid] : 0.f;
  }

  const rsrc_t rq = make_rsrc(q + (size_t)bh * n * D, (uint32_t)n * D * 2);
  const rsrc_t rk = make_rsrc(k + (size_t)bh * n * D, (uint32_t)n * D * 2);
  const rsrc_t rv = make_rsrc(v + (size_t)bh * n * DV, (uint32_t)n * DV * 2);
  // staging registers: consecutive lanes take consecutive 16-byte pieces of a token row
  uint4 pq[G::PF], pk[G::PF], pv[G::PF];
  auto fetch = [&](int c) {
#pragma unroll
    for (int i = 0; i < G::PF; ++i) {
      const int e = tid + NT * i;
      const uint32_t off = (((uint32_t)c * C + e / (D / 8)) * D + (e % (D / 8)) * 8) * 2;
      pq[i] = buf_load16(rq, off);
      pk[i] = buf_load16(rk, off);
      pv[i] = buf_load16(rv, off);
    }
  };
  auto stage = [&](int b) {
#pragma unroll
    for (int i = 0; i < G::PF; ++i) {
      const int e = tid + NT * i, t = e / (D / 8), a = (e % (D / 8)) * 8;
      *reinterpret_cast<uint4*>(lds + G::oQ + b * G::sQ + t * G::ldQ + a) = pq[i];
      *reinterpret_cast<uint4*>(lds + G::oK + b * G::sK + t * G::ldK + a) = pk[i];
      *reinterpret_cast<uint4*>(Vs + t * G::ldV + a) = pv[i];
    }
  };
  // Tile t + 2 is loaded at the end of phase 1 of step t and staged in its
  // phase 3: the E side is done with Q and K of tile t (whose buffers it
  // takes), the P side with V of tile t + 1.
  auto prefetch = [&](int t) {
    if (t + 2 < nt) fetch(c_begin + t + 2);
  };
  auto restage = [&](int t) {
    if (t + 2 < nt) stage(t & 1);
  };

  fetch(c_begin);
  stage(0);
  __syncthreads();

  // The two sides run separate loops with the same three barriers per step.
  if (pside) {
    for (int t = -1; t < nt; ++t) {
      const bool hasX = t + 1 < nt;  // P side on tile t + 1
      const int b = (t + 1) & 1;
      const uint16_t* Qx = lds + G::oQ + b * G::sQ;
      const uint16_t* Kx = lds + G::oK + b * G::sK;
      uint16_t* Ah = lds + G::oA + b * G::sA;
      uint16_t* Al = Ah + C * G::ldA;
      // the lane index made opaque once per step: offsets are formed here and
      // every access adds a constant, none hoisted out of the loop
      int ln = tid & 63;
      asm volatile("" : "+v"(ln));
      const int lr = ln & 31, lg = ln >> 5, u = ln + 64 * w;
      f32x16 acc[2];
      // phase 1: A^T tile (keys it, queries jt) = K Q^T, it <= jt; R = Q P0
      if (hasX && cw < 3) {
        const int it = cw == 2 ? 1 : 0, jt = cw == 0 ? 0 : 1;
        f32x16 a = zero16();
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
          a = mfma(frag<true>(Kx, G::ldK, it * 32, s * 16, ln), frag<true>(Qx, G::ldQ, jt * 32, s * 16, ln), a);
        read_ahead<6, 8, 16>();
        if (it == jt)
#pragma unroll
          for (int e = 0; e < 16; ++e)   // keep key <= query
            if (acc_row(e, lg) > lr) a[e] = 0.f;
        if (normalized) {
          float ps = 0.f;
#pragma unroll
          for (int e = 0; e < 16; ++e) ps += a[e];
          ps += __shfl_xor(ps, 32);
          if (lg == 0) rs[(it ? 64 : jt * 32) + lr] = ps;
        }
        store_T<true>(a, Ah, Al, G::ldA, it * 32, jt * 32, ln);
      }
      if (hasX) {
        acc[0] = zero16();
        acc[1] = zero16();
#pragma unroll
        for (int j = 0; j < D / 16; ++j) {
          bf16x8 ph, pl;
          frag_from_acc(st[j >> 1], j & 1, ph, pl);
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) {
            const bf16x8 aQ = frag_acc_order<true>(Qx, G::ldQ, rt * 32, j * 16, ln);
            acc[rt] = mfma(aQ, ph, acc[rt]);
            acc[rt] = mfma(aQ, pl, acc[rt]);
          }
        }
        read_ahead<6, 32, 16>();
      }
      prefetch(t);
      lds_barrier();
      // phase 2: R += A V, P0 += K^T V; q . m0 and the m0 increments
      float sd = 0.f, minc = 0.f;
      if (hasX) {
        bf16x8 bV[C / 16];
#pragma unroll
        for (int s = 0; s < C / 16; ++s) {
          bV[s] = frag_tr<true>(Vs, G::ldV, cw * 32, s * 16, ln);
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
            if (s < 2 || rt == 1) {    // keys past the query tile: A is zero
              acc[rt] = mfma(frag<true>(Ah, G::ldA, rt * 32, s * 16, ln), bV[s], acc[rt]);
              acc[rt] = mfma(frag<true>(Al, G::ldA, rt * 32, s * 16, ln), bV[s], acc[rt]);
            }
        }
#pragma unroll
        for (int s = 0; s < C / 16; ++s)
#pragma unroll
          for (int i = 0; i < 4; ++i) st[i] = mfma(frag_tr<true>(Kx, G::ldK, i * 32, s * 16, ln), bV[s], st[i]);
        read_ahead<16, 28, 52>();
        if (normalized) {            // four lanes per token, 32 dimensions each
          const int tok = u >> 2, p0 = (u & 3) * 32;
          const uint16_t* row = Qx + tok * G::ldQ + p0;
#pragma unroll
          for (int a = 0; a < 32; a += 8) {
            const uint4 x = *reinterpret_cast<const uint4*>(row + a);
            const float4 e0 = *reinterpret_cast<const float4*>(m0 + p0 + a);
            const float4 e1 = *reinterpret_cast<const float4*>(m0 + p0 + a + 4);
            sd += __uint_as_float(x.x << 16) * e0.x + __uint_as_float(x.x & 0xffff0000u) * e0.y;
            sd += __uint_as_float(x.y << 16) * e0.z + __uint_as_float(x.y & 0xffff0000u) * e0.w;
            sd += __uint_as_float(x.z << 16) * e1.x + __uint_as_float(x.z & 0xffff0000u) * e1.y;
            sd += __uint_as_float(x.w << 16) * e1.z + __uint_as_float(x.w & 0xffff0000u) * e1.w;
          }
          sd += __shfl_xor(sd, 1);
          sd += __shfl_xor(sd, 2);
        }
        if (normalized) {            // two lanes per dimension, 32 tokens each
          const uint16_t* colp = Kx + (u & 1) * 32 * G::ldK + (u >> 1);
#pragma unroll 8
          for (int j = 0; j < 32; ++j) minc += bf16_to_f(colp[j * G::ldK]);
          minc += __shfl_xor(minc, 1);
        }
      }
      lds_barrier();
      // phase 3: R^T and s of tile t + 1 for the E side, and m0 after it
      if (hasX) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) store_T<true>(acc[rt], Rh, Rl, G::ldR, rt * 32, cw * 32, ln);
        if (normalized && (u & 3) == 0) {
          const int tok = u >> 2;
          sv[tok] = sd + rs[tok] + (tok >= 32 ? rs[32 + tok] : 0.f);
        }
        if (normalized && (u & 1) == 0) m0[u >> 1] += minc;
      }
      restage(t);
      lds_barrier();
    }
  } else {
    const rsrc_t ro = make_rsrc(SUMMARY ? nullptr : out + (size_t)bh * n * DV, SUMMARY ? 0u : (uint32_t)n * DV * 4);
    for (int t = -1; t < nt; ++t) {
      const bool hasY = t >= 0;      // E side on tile t
      const int b = t & 1;
      const uint16_t* Qy = lds + G::oQ + b * G::sQ;
      const uint16_t* Ky = lds + G::oK + b * G::sK;
      const uint16_t* Ah = lds + G::oA + b * G::sA;
      const uint16_t* Al = Ah + C * G::ldA;
      int ln = tid & 63;
      asm volatile("" : "+v"(ln));
      const int lr = ln & 31, lg = ln >> 5, u = ln + 64 * (w - 4);
      f32x16 acc[2];
      // phase 1: O = Q E0 and the rows' 1 / (A s + q . n0 + eps); SUMMARY: K^T Q
      if (SUMMARY && hasY) {
#pragma unroll
        for (int s = 0; s < C / 16; ++s) {
          const bf16x8 bQ = frag_tr<true>(Qy, G::ldQ, cw * 32, s * 16, ln);
#pragma unroll
          for (int i = 0; i < 4; ++i) qk[i] = mfma(frag_tr<true>(Ky, G::ldK, i * 32, s * 16, ln), bQ, qk[i]);
        }
      }
      if (!SUMMARY && hasY) {
        acc[0] = zero16();
        acc[1] = zero16();
#pragma unroll
        for (int j = 0; j < D / 16; ++j) {
          bf16x8 eh, el;
          frag_from_acc(st[j >> 1], j & 1, eh, el);
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) {
            const bf16x8 aQ = frag_acc_order<true>(Qy, G::ldQ, rt * 32, j * 16, ln);
            acc[rt] = mfma(aQ, eh, acc[rt]);
            acc[rt] = mfma(aQ, el, acc[rt]);
          }
        }
        read_ahead<6, 32, 16>();
        if (normalized) {            // four lanes per token: 32 dimensions of q . n0, 16 keys of A s each
          const int tok = u >> 2, p = u & 3;
          float sd = 0.f;
          const uint16_t* row = Qy + tok * G::ldQ + p * 32;
#pragma unroll
          for (int a = 0; a < 32; a += 8) {
            const uint4 x = *reinterpret_cast<const uint4*>(row + a);
            const uint32_t xx[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              sd += __uint_as_float(xx[j] << 16) * n0[p * 32 + a + 2 * j];
              sd += __uint_as_float(xx[j] & 0xffff0000u) * n0[p * 32 + a + 2 * j + 1];
            }
          }
          if (p < 2 || tok >= 32) {   // key tile 1 is not stored for queries below 32
            const uint16_t* ah = Ah + tok * G::ldA + p * 16;
            const uint16_t* al = Al + tok * G::ldA + p * 16;
#pragma unroll
            for (int a = 0; a < 16; a += 8) {
              const uint4 xh = *reinterpret_cast<const uint4*>(ah + a);
              const uint4 xl = *reinterpret_cast<const uint4*>(al + a);
              const uint32_t uh[4] = {xh.x, xh.y, xh.z, xh.w}, ul[4] = {xl.x, xl.y, xl.z, xl.w};
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const float* s2 = sv + p * 16 + a + 2 * j;
                sd += (__uint_as_float(uh[j] << 16) + __uint_as_float(ul[j] << 16)) * s2[0];
                sd += (__uint_as_float(uh[j] & 0xffff0000u) + __uint_as_float(ul[j] & 0xffff0000u)) * s2[1];
              }
            }
          }
          sd += __shfl_xor(sd, 1);
          sd += __shfl_xor(sd, 2);
          if (p == 0) inv[tok] = 1.f / (sd + eps);
        }
      }
      prefetch(t);
      lds_barrier();
      // phase 2: O += A R (A and R split: hi hi, hi lo, lo hi), E0 += K^T R, n0 += K^T s
      if (hasY) {
#pragma unroll
        for (int s = 0; s < C / 16; ++s) {
          const bf16x8 brh = frag<true>(Rh, G::ldR, cw * 32, s * 16, ln);
          const bf16x8 brl = frag<true>(Rl, G::ldR, cw * 32, s * 16, ln);
          if (!SUMMARY)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
              if (s < 2 || rt == 1) {
                const bf16x8 ah = frag<true>(Ah, G::ldA, rt * 32, s * 16, ln);
                const bf16x8 al = frag<true>(Al, G::ldA, rt * 32, s * 16, ln);
                acc[rt] = mfma(ah, brh, acc[rt]);
                acc[rt] = mfma(ah, brl, acc[rt]);
                acc[rt] = mfma(al, brh, acc[rt]);
              }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const bf16x8 aK = frag_tr<true>(Ky, G::ldK, i * 32, s * 16, ln);
            st[i] = mfma(aK, brh, st[i]);
            st[i] = mfma(aK, brl, st[i]);
          }
        }
        if constexpr (SUMMARY) read_ahead<12, 32, 40>();
        else read_ahead<12, 50, 52>();
        if (normalized) {            // two lanes per dimension, 32 tokens each
          float ninc = 0.f;
          const uint16_t* colp = Ky + (u & 1) * 32 * G::ldK + (u >> 1);
#pragma unroll 8
          for (int j = 0; j < 32; ++j) ninc += bf16_to_f(colp[j * G::ldK]) * sv[(u & 1) * 32 + j];
          ninc += __shfl_xor(ninc, 1);
          if ((u & 1) == 0) n0[u >> 1] += ninc;
        }
      }
      lds_barrier();
      // phase 3: the next tile staged first, so that waiting for its loads
      // never waits for the output stores (one in-order counter covers both);
      // then the output rows, staged a row tile at a time through this wave's
      // slot of the dead A tile so that every lane stores 16 bytes
      restage(t);
      if (!SUMMARY && hasY) {
        const uint32_t t0 = (uint32_t)(c_begin + t) * C;
        float* ob = reinterpret_cast<float*>(lds + G::oA + b * G::sA) + cw * 1024;   // [32][32] fp32
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) {
            const int r0 = 8 * qd + 4 * lg;
            const float4 sc = normalized ? *reinterpret_cast<const float4*>(inv + rt * 32 + r0) : make_float4(1.f, 1.f, 1.f, 1.f);
            ob[(r0 + 0) * 32 + lr] = acc[rt][4 * qd + 0] * sc.x;
            ob[(r0 + 1) * 32 + lr] = acc[rt][4 * qd + 1] * sc.y;
            ob[(r0 + 2) * 32 + lr] = acc[rt][4 * qd + 2] * sc.z;
            ob[(r0 + 3) * 32 + lr] = acc[rt][4 * qd + 3] * sc.w;
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {       // rows past n fall outside the buffer and are dropped
            const int row = 8 * j + (ln >> 3), c4 = (ln & 7) * 4;
            buf_store16(ro, ((t0 + rt * 32 + row) * DV + cw * 32 + c4) * 4,
                        *reinterpret_cast<const float4*>(ob + row * 32 + c4));
          }
        }
      }
      lds_barrier();
    }
  }
  if (rec) {
    int col = cw * 32 + lr;
    asm volatile("" : "+v"(col));
    float* dst = rec + (pside ? off_C(D, DV) : off_G(D, DV));
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) dst[(size_t)(32 * i + acc_row(e, lg)) * DV + col] = st[i][e];
    if (SUMMARY && !pside) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) rec[(size_t)(32 * i + acc_row(e, lg)) * D + col] = qk[i][e];
    }
    if (tid < D) {
      rec[off_m(D, DV) + tid] = m0[tid];
      rec[off_h(D, DV) + tid] = n0[tid];
    }
  }
}

// First launch, grid (P - 1, BH): segment 0's output walk and the summary
// walks of segments 1 .. P-2, each writing its record.
__global__ __launch_bounds__(CfgAW::NT, 1) void k_ahla_ws_first(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    float* __restrict__ out, float* __restrict__ rec, int n, int c0, int cps, int nseg, int normalized, float eps) {
  extern __shared__ __align__(16) uint16_t lds[];
  int seg, bh;
  seg_head(seg, bh);
  int cb, nt;
  ws_range(seg, c0, cps, (n + CfgAW::C - 1) / CfgAW::C, cb, nt);
  float* r = rec + ((size_t)bh * (nseg + 1) + seg) * state_floats(CfgAW::D, CfgAW::DV);
  if (seg == 0)
    walk_aw<false>(lds, q, k, v, out, nullptr, nullptr, r, bh, n, cb, nt, normalized, eps);
  else
    walk_aw<true>(lds, q, k, v, nullptr, nullptr, nullptr, r, bh, n, cb, nt, normalized, 0.f);
}

// Output walks of segments seg0, seg0 + 1, .. from their carries: ppre
// [BH][nseg][D DV | D] the prefixes of P and m, carry likewise of E and n
// (both null for a single segment).
__global__ __launch_bounds__(CfgAW::NT, 1) void k_ahla_ws_out(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    float* __restrict__ out, const float* __restrict__ ppre, const float* __restrict__ carry, int n, int c0, int cps,
    int nseg, int seg0, int normalized, float eps) {
  extern __shared__ __align__(16) uint16_t lds[];
  int seg, bh;
  seg_head(seg, bh);
  seg += seg0;
  int cb, nt;
  ws_range(seg, c0, cps, (n + CfgAW::C - 1) / CfgAW::C, cb, nt);
  const size_t at = ((size_t)bh * nseg + seg) * (CfgAW::D * CfgAW::DV + CfgAW::D);
  walk_aw<false>(lds, q, k, v, out, ppre ? ppre + at : nullptr, carry ? carry + at : nullptr, nullptr, bh, n, cb, nt,
                 normalized, eps);
}

}  // namespace
}  // namespace hla
