// The two-pass plan of the d = 128 walks (second order and AHLA): its
// segments, and the launch between the two passes that forms the prefixes and
// the segment brackets.  Included by the .hip files only.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "fused_tiles.h"

namespace hla {
namespace {

constexpr int kWsTile = 64;   // tokens a tile

// Tile range of segment seg: segment 0 holds tiles [0, c0), segment s >= 1
// tiles [c0 + (s - 1) cps, c0 + s cps), cut at M.
__device__ __forceinline__ void ws_range(int seg, int c0, int cps, int M, int& c_begin, int& nt) {
  c_begin = seg == 0 ? 0 : c0 + (seg - 1) * cps;
  nt = min(M, seg == 0 ? c0 : c_begin + cps) - c_begin;
}

// Instruction order for one block of LDS-fed products: PRE LDS reads first,
// then the NM MFMAs with the remaining NR - PRE reads spread evenly between
// them, so each wave keeps several fragment reads in flight instead of
// waiting on the read that feeds the very next MFMA (mask 0x100: LDS reads,
// 0x008: MFMAs).  It only orders; data dependences still hold.
template <int PRE, int NM, int NR, int I = 0>
__device__ __forceinline__ void read_ahead() {
  if constexpr (I == 0) __builtin_amdgcn_sched_group_barrier(0x100, PRE, 0);
  if constexpr (I < NM) {
    constexpr int c = ((I + 1) * (NR - PRE)) / NM - (I * (NR - PRE)) / NM;
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if constexpr (c > 0) __builtin_amdgcn_sched_group_barrier(0x100, c, 0);
    read_ahead<PRE, NM, NR, I + 1>();
  }
}

// Per-tile time of the summary walk over that of the output walk (both at
// one workgroup per CU, d = dv = 128: about 3.9 and 6.6 us per tile).
constexpr double kWsSummaryRatio = 0.65;

// Segments of the two-pass plan: with Q = 256 / BH walks per head in each
// launch (one workgroup per CU), segments 1 .. P-1 get x tiles each (the
// last the rest) and segment 0 about r x, r the ratio above, so that segment
// 0's output walk and the summary walks beside it end together.  With fewer
// than two later segments the plan is a single output walk per head.
inline void ws_plan(int BH, int n, int* P, int* cps, int* c0) {
  const int M = (n + kWsTile - 1) / kWsTile;
  int Q = 256 / BH;
  if (const char* e = getenv("HLA_FUSED_SEGMENTS")) Q = atoi(e) - 1;
  double r = kWsSummaryRatio;
  if (const char* e = getenv("HLA_WS_RATIO")) r = atof(e);
  if (Q >= 2 && M >= 3 && r > 0.0) {
    int x = (int)ceil(M / (Q + r));
    const int l0 = std::max(1, (int)lround(r * x));
    if (l0 < M) {
      const int rest = M - l0;
      if ((rest + x - 1) / x > Q) x = (rest + Q - 1) / Q;
      const int p1 = (rest + x - 1) / x;
      if (p1 >= 2) {
        *P = 1 + p1;
        *cps = x;
        *c0 = l0;
        return;
      }
    }
  }
  *P = 1;
  *cps = M;
  *c0 = M;
}

// Segments per head up to which the bracket launch sums the prefixes itself;
// above it k_seg_prefix writes them first.  A bracket workgroup reads every
// earlier record, P^2 / 2 of them a head in chains of P / 2 loads: 45 us with
// 61 segments (4 heads of 30 000 tokens) against 10 us for the launch and 17 us
// for the brackets after it.  At 9 segments (32 heads, two prefills of about
// 4000 tokens) the extra launch costs 2 % (333 against 326 us), and so it does
// at 5 (64 heads of 16 384: 658 against 650 us).
constexpr int kBracketSumMax = 12;

// The prefixes and the brackets of the two-pass plan (Eq. semidirect in the
// Phi form).  For segment s = 1 .. nseg-1: S_{<s}, the sum of the S
// slots of records 0 .. s-1 (record 0 holds the ending state of segment 0's
// output walk, records 1 .. nseg-2 the summaries), into spre[s] for the
// output walks.  For s <= nseg-2, whose record holds its S, C, m, Phi, eta
// from a zero start, also b_s = (Phi_s + S_{<s} C_s, eta_s + S_{<s} m_s),
// written in place of (Phi_s, eta_s); record 0 already holds b_0.
// AH (AHLA): records hold K^T Q in the S slot, P = K^T V and m^K in C | m, E and
// n in G | h; the prefixes are those of (P, m^K) ([D DV | D] in spre[s]) and
// the bracket is (E_s + (K^T Q)_s P_{<s}, n_s + (K^T Q)_s m_{<s}) (Eq.
// AHLA-semidirect).
// grid (nseg - 1, BH), 1024 threads, one workgroup per (segment, head), a
// head's workgroups on one XCD.  S_{<s} and C_s are split into three bf16
// pieces (24 bits: the fp32 values) in LDS, one half of the contraction at a
// time, and wave w forms the 32 x 32 tile (w / 4, w % 4) of S_{<s} C_s from
// the six products of at least 2^-16 with fp32 accumulation: the bracket is
// what the later segments' carries are summed from, and with two pieces
// (three products) it was the larger part of their error (prefill of 8000
// tokens on 32 heads, outputs 4.3-4.7e-6 from the 64-bit result, now 2.9e-6).  The
// loads bound it: 1 MB a workgroup at 8 segments.
template <int D, int DV, bool AH = false>
__global__ __launch_bounds__(1024) void k_ws_bracket(float* __restrict__ rec, float* __restrict__ spre, int nseg,
                                                     int summed) {
  constexpr int KH = D / 2, ldS = KH + kPad, ldC = DV + 16, NT = 1024;   // ldC: C is read through the transpose unit
  static_assert(D == 128 && DV == 128, "16 waves of 32 x 32 output tiles");
  __shared__ __align__(16) uint16_t Sp[3][D * ldS], Cp[3][KH * ldC];
  __shared__ float mv[D], ep[D];
  int s, bh;
  seg_head(s, bh);
  s += 1;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, lr = l & 31, lg = l >> 5;
  const int r0 = 32 * (w >> 2), c0 = 32 * (w & 3);
  const size_t F = state_floats(D, DV);
  float* r = rec + ((size_t)bh * (nseg + 1) + s) * F;
  constexpr int NS4 = D * D / 4 / NT;
  // the segment's own C (AH: K^T Q) and Phi first (the last segment's record
  // is not read: it has no bracket)
  const bool own = s < nseg - 1;
  float4 sx[NS4], cx[NS4];     // the left and the right operand
  float4* mine = AH ? sx : cx;
  float4* pre = AH ? cx : sx;
  constexpr size_t oPre = AH ? (size_t)D * D : 0, oMine = AH ? 0 : (size_t)D * D;   // S at 0, C at D D
  f32x16 acc;        // b_s: element e is row r0 + acc_row(e, lg), column c0 + lr
  float eta = 0.f, m = 0.f;
  if (own) {
#pragma unroll
    for (int i = 0; i < NS4; ++i) mine[i] = reinterpret_cast<const float4*>(r + oMine)[tid + NT * i];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = r[off_G(D, DV) + (size_t)(r0 + acc_row(e, lg)) * DV + c0 + lr];
    if (tid < D) {
      eta = r[off_h(D, DV) + tid];
      if (!AH) m = r[off_m(D, DV) + tid];
    }
  }
  // the prefix: already in spre (summed), or the earlier records' S (AH: C)
  // slots, two records' loads in flight at a time
#pragma unroll
  for (int i = 0; i < NS4; ++i) pre[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  const float* r0s = rec + (size_t)bh * (nseg + 1) * F + oPre;
  for (int j0 = 0; j0 < (summed ? 0 : s); j0 += 2) {
    float4 u[2][NS4];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < NS4; ++i)
        u[j][i] = j0 + j < s ? reinterpret_cast<const float4*>(r0s + (size_t)(j0 + j) * F)[tid + NT * i]
                             : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < NS4; ++i) {
        pre[i].x += u[j][i].x; pre[i].y += u[j][i].y; pre[i].z += u[j][i].z; pre[i].w += u[j][i].w;
      }
  }
  float* sp = spre + ((size_t)bh * nseg + s) * (AH ? D * DV + D : D * D);
  if (summed) {
    if (!own) return;
#pragma unroll
    for (int i = 0; i < NS4; ++i) pre[i] = reinterpret_cast<const float4*>(sp)[tid + NT * i];
    if (AH && tid < D) m = sp[D * DV + tid];
  } else {
#pragma unroll
    for (int i = 0; i < NS4; ++i) reinterpret_cast<float4*>(sp)[tid + NT * i] = pre[i];
    if (AH && tid < D) {
#pragma unroll 4
      for (int j = 0; j < s; ++j) m += r0s[(size_t)j * F + D * DV + tid];
      sp[D * DV + tid] = m;
    }
  }
  if (!own) return;
  if (tid < D) mv[tid] = m;
  auto put = [](uint16_t* p0, uint16_t* p1, uint16_t* p2, const float4& x) {
    uint32_t h0, h1, m0, m1, l0, l1;
    split3(x.x, x.y, h0, m0, l0);
    split3(x.z, x.w, h1, m1, l1);
    *reinterpret_cast<uint2*>(p0) = make_uint2(h0, h1);
    *reinterpret_cast<uint2*>(p1) = make_uint2(m0, m1);
    *reinterpret_cast<uint2*>(p2) = make_uint2(l0, l1);
  };
  const int row = tid / (D / 4), col = 4 * (tid % (D / 4));   // of piece 0; piece i is 32 rows further down
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h) __syncthreads();
#pragma unroll
    for (int i = 0; i < NS4; ++i)
      if (col / KH == h) {
        const int o = (row + 32 * i) * ldS + col - KH * h;
        put(Sp[0] + o, Sp[1] + o, Sp[2] + o, sx[i]);
      }
#pragma unroll
    for (int i = 0; i < NS4 / 2; ++i) {
      const int o = (row + 32 * i) * ldC + col;
      put(Cp[0] + o, Cp[1] + o, Cp[2] + o, cx[i + NS4 / 2 * h]);
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KH / 16; ++ks) {
      bf16x8 a[3], b[3];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        a[j] = frag(Sp[j], ldS, r0, 16 * ks);
        b[j] = frag_tr(Cp[j], ldC, c0, 16 * ks);
      }
      acc = mfma(a[0], b[0], acc);
      acc = mfma(a[0], b[1], acc);
      acc = mfma(a[1], b[0], acc);
      acc = mfma(a[0], b[2], acc);
      acc = mfma(a[1], b[1], acc);
      acc = mfma(a[2], b[0], acc);
    }
  }
  // the left operand times m from the registers: 32 lanes hold a row
#pragma unroll
  for (int i = 0; i < NS4; ++i) {
    float x = sx[i].x * mv[col] + sx[i].y * mv[col + 1] + sx[i].z * mv[col + 2] + sx[i].w * mv[col + 3];
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) x += __shfl_xor(x, o);
    if (col == 0) ep[row + 32 * i] = x;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) r[off_G(D, DV) + (size_t)(r0 + acc_row(e, lg)) * DV + c0 + lr] = acc[e];
  __syncthreads();
  if (tid < D) r[off_h(D, DV) + tid] = eta + ep[tid];
}

}  // namespace
}  // namespace hla
