// The two-pass plan of the d = 128 walks (second order and AHLA): its
// segments, and the launch between the two passes that forms the prefixes and
// the segment brackets.  Included by the .hip files only.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "fused_tiles.h"
#include "profile.h"

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

// Per-tile time of the summary walk over that of the output walk, both at one
// workgroup per CU: second order about 3.9 and 6.6 us per tile, of which 0.65
// measured best (0.5 to 1 were tried); AHLA (us at 0.55 / 0.65 / 0.75 / 0.85) 64 heads of
// 8000 tokens 317 / 311 / 311 / 310, of 3000 144 / 144 / 138 / 142, 100 of 4000
// 257 / 250 / 241 / 253, 16 of 8000 123 / 121 / 120 / 120.
constexpr double kWsSummaryRatio = 0.65, kAhlaSummaryRatio = 0.75;

// Segments of the two-pass plan: with Q = 256 / BH walks per head in each
// launch (one workgroup per CU), segments 1 .. P-1 get x tiles each (the
// last the rest) and segment 0 about r x, r the ratio above, so that segment
// 0's output walk and the summary walks beside it end together.  With fewer
// than two later segments the plan is a single output walk per head.
inline void ws_plan(int BH, int n, double r, int* P, int* cps, int* c0) {
  const int M = (n + kWsTile - 1) / kWsTile;
  int Q = 256 / BH;
  if (const char* e = getenv("HLA_FUSED_SEGMENTS")) Q = atoi(e) - 1;
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
// earlier record, P^2 / 2 of them a head in chains of P / 4 rounds, against one
// more launch.  With itself / with the launch, us a forward: 13 segments (20
// heads of 4000 tokens) 90.7 / 93.2, 17 (16 heads of 4000) 83.3 / 84.6 (AHLA, 16
// heads of 6000, 104.0 / 106.7), 22 (12 heads of 6000) 99.3 / 90.4, 33 (8 heads of
// 6000) 82.4 / 78.6, 52 (5 heads of 6000) 86.4 / 68.1.
constexpr int kBracketSumMax = 17;
// (segment, head) pairs up to which two workgroups share a bracket: 14 pairs (2
// heads of 500 tokens) 34.7 -> 30.9 us a forward, 60 (4 heads of 1000) 43.8 ->
// 41.1, 124 (4 heads of 2000) 47.5 -> 46.1.  With more than half of the chip's
// CUs at work two only add reads: 156 pairs (4 heads of 2500) 50.4 -> 51.3, 240
// (24 heads of 4000) 100.6 -> 106.1.
constexpr int kBracketSplitMax = 128;

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
// grid (HALVES (nseg - 1), BH), 1024 / HALVES threads: HALVES workgroups a
// (segment, head), each one part of the prefix (rows of S_{<s}; AH: columns of
// P_{<s}) and of the bracket, a head's workgroups on one XCD.  S_{<s} and C_s are
// split into three bf16 pieces (24 bits: the fp32 values) in LDS, 32 steps of
// the contraction at a time, and each wave forms one 32 x 32 tile of S_{<s} C_s
// from the six products of at least 2^-16 with fp32 accumulation: the bracket
// is what the later segments' carries are summed from, and with two pieces
// (three products) it was the larger part of their error (prefill of 8000
// tokens on 32 heads, outputs 4.3-4.7e-6 from the 64-bit result, now 2.9e-6).
// The third piece costs about 1 us a forward where all CUs are at work (with
// two pieces / now: 32 heads of 4000 tokens 114.2 / 115.8 us, 16 of 2000 66.8 /
// 67.5, 64 of 1000 77.0 / 78.4).  Slabs of 64, or 8 waves of two tiles each, are
// no faster.
template <int D, int DV, bool AH, int HALVES>
__global__ __launch_bounds__(1024 / HALVES, 4) void k_ws_bracket(float* __restrict__ rec, float* __restrict__ spre,
                                                                 int nseg, int summed) {
  static_assert(D == 128 && DV == 128, "16 waves of 32 x 32 tiles a bracket");
  constexpr int KH = 32, NT = 1024 / HALVES, NK = D / KH;             // slabs of the contraction
  constexpr int RL = AH ? D : D / HALVES, CR = AH ? DV / HALVES : DV;    // rows of the left, columns of the right operand
  constexpr int LQ = KH / 4, RQ = CR / 4;                                // float4 a row of their slabs
  constexpr int LS = NT / LQ, RS = NT / RQ, NL = RL / LS, NR = KH / RS;  // rows at a time; float4 a thread and slab
  constexpr int ldS = KH + kPad, ldC = CR + 16;                          // ldC: read through the transpose unit
  constexpr int NP = NK * (AH ? NR : NL), NO = NK * (AH ? NL : NR);      // float4 a thread: prefix part, own operand
  __shared__ __align__(16) uint16_t Sp[3][RL * ldS], Cp[3][KH * ldC];
  __shared__ float mv[D], ep[D];
  int s, bh;
  seg_head(s, bh);
  const int half = s % HALVES;
  s = 1 + s / HALVES;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, lr = l & 31, lg = l >> 5;
  const int r0 = 32 * (w / (CR / 32)), c0 = 32 * (w % (CR / 32));
  const size_t F = state_floats(D, DV);
  float* r = rec + ((size_t)bh * (nseg + 1) + s) * F;
  // piece i of a thread: NL of a slab of the left operand (KH of its columns), NR
  // of a slab of the right one (KH of its rows), so that every lane has its
  // share of each slab
  const int lrow = tid / LQ, lcol = (tid % LQ) * 4, rrow = tid / RQ, rcol = (tid % RQ) * 4;
  auto at_left = [&](int i) { return (lrow + LS * (i % NL) + (AH ? 0 : RL * half)) * D + KH * (i / NL) + lcol; };
  auto at_right = [&](int i) { return (rrow + RS * i) * DV + rcol + (AH ? CR * half : 0); };
  auto at_pre = [&](int i) { return AH ? at_right(i) : at_left(i); };
  auto at_own = [&](int i) { return AH ? at_left(i) : at_right(i); };
  constexpr size_t oPre = AH ? (size_t)D * D : 0, oOwn = AH ? 0 : (size_t)D * D;   // S at 0, C at D D
  // the segment's own operand first (the last segment's record is not read: it has no bracket)
  const bool own = s < nseg - 1;
  float4 ox[NO], px[NP];
  if (own) {
#pragma unroll
    for (int i = 0; i < NO; ++i) ox[i] = *reinterpret_cast<const float4*>(r + oOwn + at_own(i));
  }
  // the prefix: already in spre (summed), or the earlier records' S (AH: C)
  // slots, four records' loads in flight at a time
  float m = !AH && own && tid < D ? r[off_m(D, DV) + tid] : 0.f;
  float* sp = spre + ((size_t)bh * nseg + s) * (AH ? D * DV + D : D * D);
  if (summed) {
    if (!own) return;
#pragma unroll
    for (int i = 0; i < NP; ++i) px[i] = *reinterpret_cast<const float4*>(sp + at_pre(i));
    if (AH && tid < D) m = sp[D * DV + tid];
  } else {
    const float* r0s = rec + (size_t)bh * (nseg + 1) * F + oPre;
#pragma unroll
    for (int i = 0; i < NP; ++i) px[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j0 = 0; j0 < s; j0 += 4) {
      float4 u[4][NP];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < NP; ++i)
          u[j][i] = j0 + j < s ? *reinterpret_cast<const float4*>(r0s + (size_t)(j0 + j) * F + at_pre(i))
                               : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          px[i].x += u[j][i].x; px[i].y += u[j][i].y; px[i].z += u[j][i].z; px[i].w += u[j][i].w;
        }
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) *reinterpret_cast<float4*>(sp + at_pre(i)) = px[i];
    if (AH && tid < D) {
#pragma unroll 4
      for (int j = 0; j < s; ++j) m += r0s[(size_t)j * F + D * DV + tid];
      if (half == 0) sp[D * DV + tid] = m;
    }
  }
  if (!own) return;
  float* out = r + off_G(D, DV) + (AH ? CR * half : RL * half * DV);
  f32x16 acc;        // the bracket: element e is row r0 + acc_row(e, lg), column c0 + lr
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = out[(size_t)(r0 + acc_row(e, lg)) * DV + c0 + lr];
  // eta (AH: n) of this part's rows (AH: all rows, by part 0)
  const int er = (AH ? 0 : RL * half) + tid;
  const bool eown = tid < RL && (!AH || half == 0);
  const float eta = eown ? r[off_h(D, DV) + er] : 0.f;
  if (tid < D) mv[tid] = m;
  auto put = [](uint16_t* p0, uint16_t* p1, uint16_t* p2, const float4& x) {
    uint32_t h0, h1, m0, m1, l0, l1;
    split3(x.x, x.y, h0, m0, l0);
    split3(x.z, x.w, h1, m1, l1);
    *reinterpret_cast<uint2*>(p0) = make_uint2(h0, h1);
    *reinterpret_cast<uint2*>(p1) = make_uint2(m0, m1);
    *reinterpret_cast<uint2*>(p2) = make_uint2(l0, l1);
  };
#pragma unroll
  for (int h = 0; h < NK; ++h) {
    if (h) __syncthreads();
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int o = (lrow + LS * i) * ldS + lcol;
      put(Sp[0] + o, Sp[1] + o, Sp[2] + o, AH ? ox[NL * h + i] : px[NL * h + i]);
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int o = (rrow + RS * i) * ldC + rcol;
      put(Cp[0] + o, Cp[1] + o, Cp[2] + o, AH ? px[NR * h + i] : ox[NR * h + i]);
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
  // the left operand times m from the registers: LQ lanes hold a row
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    float x = 0.f;
#pragma unroll
    for (int h = 0; h < NK; ++h) {
      const float4 v = AH ? ox[NL * h + i] : px[NL * h + i];
      const float* y = mv + KH * h + lcol;
      x += v.x * y[0] + v.y * y[1] + v.z * y[2] + v.w * y[3];
    }
#pragma unroll
    for (int o = 1; o < LQ; o <<= 1) x += __shfl_xor(x, o);
    if (lcol == 0) ep[lrow + LS * i] = x;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) out[(size_t)(r0 + acc_row(e, lg)) * DV + c0 + lr] = acc[e];
  __syncthreads();
  if (eown) r[off_h(D, DV) + er] = eta + ep[tid];
}
template <int D, int DV, bool AH>
hipError_t ws_bracket(float* rec, float* spre, int nseg, int BH, int summed, hipStream_t s) {
  if (BH * (nseg - 1) <= kBracketSplitMax)
    HLA_LAUNCH((k_ws_bracket<D, DV, AH, 2>), dim3(2 * (nseg - 1), BH), dim3(512), 0, s, rec, spre, nseg, summed);
  else
    HLA_LAUNCH((k_ws_bracket<D, DV, AH, 1>), dim3(nseg - 1, BH), dim3(1024), 0, s, rec, spre, nseg, summed);
  return hipGetLastError();
}

}  // namespace
}  // namespace hla
