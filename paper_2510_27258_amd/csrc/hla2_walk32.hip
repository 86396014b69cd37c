// Segment walk of the second-order forward in fp32 and fp64 arithmetic, masked
// or unmasked, d = dv, fp32 or bf16 inputs, no decay and no states (the
// chunked kernels of hla2_chunk.hip and hla2_scan.hip take the rest).
//
// A head's 32-token tiles are cut into P segments; a workgroup walks one
// segment with the running state in its accumulators, so no state crosses
// memory between tiles.  Per tile, with the carry S0 and X0 before it:
//   W = L (.) Q K^T,  R = W K + Q S0           (row t: r_t = S_t q_t)
//   masked    T = L (.) Q R^T,  O = T V + Q X0,  X0 += R^T V   (X = Phi = S C - G,
//             o_t = q_t^T Phi_t with Phi_t = sum_{j<=t} r_j v_j^T, Thm. 1)
//   unmasked  T = L (.) R Q^T,  O = T V + R X0,  X0 += Q^T V   (X = C)
//   S0 += K^T K;  den: the row sums of T plus q . y0 (masked, y = eta += R^T 1)
//   or r . y0 (unmasked, y = m += Q^T 1).
// Launches: k_gmoments sums S (unmasked: and C, m) over each segment; the
// walks start from the sums of the segments before them.  Unmasked rows are
// then final.  Masked walks start from X = y = 0 and leave their segment's
// (X, y), whose running sums over the segments are the missing carries (the
// Phi form of Eq. (semidirect): Phi_{A(+)B} = Phi_A + Phi_B + S_A C_B, and the
// walk from the true S prefix forms the bracket Phi_B + S_A C_B); k_gfix adds
// q_t^T X and divides.  Up to kSelfSum segments a head the walk and the fix-up
// sum the records themselves, above it k_gprefix writes the running sums.
//
// Arithmetic as the readout of hla2_chunk.hip: Q S0, Q K^T, W K, the T products
// and the carry product on fp64 MFMA with fp32 operands widened exactly and R
// in fp64, T V and the state sums on fp32 MFMA.  Each tile's part of S0, X0 and
// y is formed from zero and added to the running state once, so a state sees
// one rounding at its own size a tile (accumulated into the running state
// itself, four tokens an MFMA, one segment of 4096 tokens was 2-6 times
// further off; at d = 128 that is 2 % of the time, 237.5 -> 242.5 us for fp32
// 4x12x1290).  Distance from the 64-bit result, the chunked kernels' (one
// rounding a 64-token chunk) and this: 3.3e-7 and 1.5e-7 at d = 64, n = 4096
// in 22 segments; with one segment a head, masked, d = 128, n = 4096 3.3e-7 and
// 2.3e-7, n = 16384 5.7e-7 and 3.9e-7 (X needs no difference of two products
// S C and G).  Unmasked, C is the same sum in both: in one segment of 4096
// tokens 2.6e-7 and 2.7e-7, of 16384 3.9e-7 and 4.8e-7, so unmasked segments
// are bounded (kMaxTiles): 2.0e-7 and 2.9e-7.  Up to 64 tokens, one chunk,
// 0.7-1.0e-7 and 0.8-1.2e-7: one fp32 rounding of the state more.
//
// Against a summary, a scan and a readout a 64-token chunk (one fp32 state of
// d^2 + 2 d^2 + 2 d floats a chunk written, read, written and read again): fp32
// 2x16x4096, d = 64, 455 -> 163 us (walk 104, fix-up 32, moments 15, running
// sums 2 x 7); bf16 unmasked 1x16x4001, d = 128, 675 -> 163 us (walk 131,
// moments 25, sums 12); fp32 1x2x256, d = 32, 35 -> 19 us.
// The largest part of the walk is fp64 MFMA: 2 d^2 products a token in the
// carry terms and 3 x 24 d in the triangles, at the part's 71 TFLOP/s 47 of the
// 104 us at d = 64 above (3.4 GFLOP) and 76 of the 131 at d = 128 (5.4 GFLOP).
// For the rest all waves wait at the tile's barriers.  Tiles of 32 tokens keep
// the triangles short and the LDS at 72 KB for d = 128, 39 KB for 64.
//
// Layout: D / 16 waves; wave w holds column tile w of S0 and X0, all rows, as
// 16 x 16 accumulator tiles.  Element i of lane (g, n) is row 4 g + i, so with
// the contraction index of step (kt, i) taken as 16 kt + 4 g + i a state tile
// is its own B operand, and an A operand's four steps are one 16-byte read.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "common.h"
#include "fused_tiles.h"
#include "mfma16.h"
#include "profile.h"
#include "walk32.h"

namespace hla {
namespace {

constexpr int kTile = 32;
constexpr int kSelfSum = 8;
// Tiles of the longest unmasked segment (2048 tokens), whatever the head count.
// Where this cuts a head, it is cut into enough segments for four rounds of
// the chip at least, so that a last round which is partly empty costs little:
// fp32 1x160x4096, d = 128, one segment 2118 us, two 2741, seven 2008.
constexpr int kMaxTiles = 64;

template <int D>
struct GW {
  static constexpr int NT = 4 * D, NW = D / 16, ldq = D + 4, ldr = D + 2, ldw = kTile + 4;
  static constexpr int LPR = NT / kTile;                 // lanes per token row, 8 dimensions each
  // Q, V [32][ldq] fp32; K [32][ldq] fp32 in the space of R [32][ldr] fp64;
  // W, then T [32][ldw]; y [D]; the rows' denominators [32]
  static constexpr int oQ = 0, oV = oQ + kTile * ldq, oR = oV + kTile * ldq, oW = oR + 2 * kTile * ldr;
  static constexpr int oy = oW + kTile * ldw, oden = oy + D, nf = oden + kTile;
  static constexpr size_t bytes = sizeof(float) * nf;
  static constexpr size_t F = (size_t)2 * D * D + D;      // a record: S | X | y
  static_assert(oR % 4 == 0 && oW % 4 == 0 && bytes <= 80 * 1024, "LDS layout");
  // walks a CU, by their registers (178 to 200 at d = 128, 130 to 168 at 64).  Forcing
  // 128 registers and 2 and 4 walks a CU spilled: 210 for 163 us unmasked at
  // d = 128, 182 for 163 us in fp32 at d = 64.
  static constexpr int kBlocks = D == 128 ? 1 : D == 64 ? 3 : 6;
};

// Four consecutive values: as loaded, and widened (exact).
template <typename T>
struct Four;
template <>
struct Four<float> {
  using raw = float4;
  static __device__ __forceinline__ float4 wide(const raw& x) { return x; }
};
template <>
struct Four<uint16_t> {
  using raw = uint2;
  static __device__ __forceinline__ float4 wide(const raw& x) {
    return make_float4(__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xffff0000u), __uint_as_float(x.y << 16),
                       __uint_as_float(x.y & 0xffff0000u));
  }
};

// A 32 x D tile of [n][D] in registers: two pieces of four values a thread, zero past n.
template <typename T, int D>
struct Tile {
  using raw = typename Four<T>::raw;
  raw p[2];
  __device__ __forceinline__ void fetch(const T* src, int t0, int n) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = threadIdx.x + 4 * D * i, t = t0 + e / (D / 4), a = (e % (D / 4)) * 4;
      p[i] = t < n ? *reinterpret_cast<const raw*>(src + (size_t)t * D + a) : raw{};
    }
  }
  __device__ __forceinline__ void store(float* dst) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = threadIdx.x + 4 * D * i;
      *reinterpret_cast<float4*>(dst + (e / (D / 4)) * GW<D>::ldq + (e % (D / 4)) * 4) = Four<T>::wide(p[i]);
    }
  }
};

// The column tile of a [D][D] part of the records, summed over records [lo, hi)
// (stride F floats), into accumulator tiles.
template <int D>
__device__ __forceinline__ void load_state(f32x4c* st, const float* part, size_t stride, int lo, int hi, int col, int g) {
  constexpr int NW = D / 16;
#pragma unroll
  for (int rt = 0; rt < NW; ++rt) st[rt] = f32x4c{0.f, 0.f, 0.f, 0.f};
  for (int s = lo; s < hi; ++s) {
    const float* x = part + (size_t)s * stride;
    float u[NW][4];
#pragma unroll
    for (int rt = 0; rt < NW; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) u[rt][i] = x[(size_t)(16 * rt + 4 * g + i) * D + col];
#pragma unroll
    for (int rt = 0; rt < NW; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) st[rt][i] += u[rt][i];
  }
}
template <int D>
__device__ __forceinline__ void store_state(const f32x4c* st, float* part, int col, int g) {
#pragma unroll
  for (int rt = 0; rt < D / 16; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[(size_t)(16 * rt + 4 * g + i) * D + col] = st[rt][i];
}

// The eight tokens 16 kt + 4 g + i of column c of a [32][ldq] fp32 tile in LDS.
template <int D>
__device__ __forceinline__ void column8(float* x, const float* Y, int c, int g) {
#pragma unroll
  for (int j = 0; j < 8; ++j) x[j] = Y[(16 * (j >> 2) + 4 * g + (j & 3)) * GW<D>::ldq + c];
}
// Eight values that are bf16 exactly, as an operand of v_mfma_f32_16x16x32_bf16.
__device__ __forceinline__ bf16x8 pack8(const float* x) {
  uint32_t u[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    u[j] = (__float_as_uint(x[2 * j]) >> 16) | (__float_as_uint(x[2 * j + 1]) & 0xffff0000u);
  return __builtin_bit_cast(bf16x8, make_uint4(u[0], u[1], u[2], u[3]));
}

// st += Y^T Z over the tile's 32 tokens, Y [32][ldq] in LDS, z the wave's
// column of Z (column8).  Y and Z are inputs: when those are bf16 the
// products are exact on either unit and the sums fp32, so one bf16 MFMA takes
// the place of eight fp32 ones.
template <typename T, int D>
__device__ __forceinline__ void add_outer(f32x4c* st, const float* Y, const float* z, int nn, int g) {
  constexpr int NW = D / 16;
#pragma unroll
  for (int rt = 0; rt < NW; ++rt) {
    float x[8];
    column8<D>(x, Y, 16 * rt + nn, g);
    f32x4c t = {0.f, 0.f, 0.f, 0.f};
    if constexpr (sizeof(T) == 2) {
      t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pack8(x), pack8(z), t, 0, 0, 0);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) t = mfma4(x[j], z[j], t);
    }
    st[rt] += t;
  }
}

// rec[bh][seg] <- S = K^T K of the segment's tiles, with CM also X = Q^T V, y = Q^T 1.
template <typename T, int D, bool CM>
__global__ __launch_bounds__(4 * D) void k_gmoments(const T* __restrict__ q, const T* __restrict__ k,
                                                    const T* __restrict__ v, float* __restrict__ rec, int n, int cps,
                                                    int nseg) {
  using G = GW<D>;
  __shared__ __align__(16) float Ks[kTile * G::ldq], Qs[CM ? kTile * G::ldq : 4], Vs[CM ? kTile * G::ldq : 4];
  const int seg = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x;
  const int nn = tid & 15, g = (tid >> 4) & 3, col = (tid >> 6) * 16 + nn;
  const int M = (n + kTile - 1) / kTile, c0 = seg * cps, c1 = min(M, c0 + cps);
  q += (size_t)bh * n * D;
  k += (size_t)bh * n * D;
  v += (size_t)bh * n * D;
  f32x4c S[G::NW], X[CM ? G::NW : 1];
#pragma unroll
  for (int rt = 0; rt < G::NW; ++rt) S[rt] = f32x4c{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int rt = 0; rt < (CM ? G::NW : 1); ++rt) X[rt] = f32x4c{0.f, 0.f, 0.f, 0.f};
  float y = 0.f;      // four lanes a dimension, eight tokens each
  Tile<T, D> pk, pq, pv;
  auto fetch = [&](int c) {
    pk.fetch(k, c * kTile, n);
    if (CM) {
      pq.fetch(q, c * kTile, n);
      pv.fetch(v, c * kTile, n);
    }
  };
  fetch(c0);
  for (int c = c0; c < c1; ++c) {
    pk.store(Ks);
    if (CM) {
      pq.store(Qs);
      pv.store(Vs);
    }
    lds_barrier();
    if (c + 1 < c1) fetch(c + 1);
    float z[8];
    column8<D>(z, Ks, col, g);
    add_outer<T, D>(S, Ks, z, nn, g);
    if (CM) {
      column8<D>(z, Vs, col, g);
      add_outer<T, D>(X, Qs, z, nn, g);
      float yt = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) yt += Qs[((tid & 3) * 8 + j) * G::ldq + (tid >> 2)];
      y += yt;
    }
    lds_barrier();
  }
  float* r = rec + ((size_t)bh * nseg + seg) * G::F;
  store_state<D>(S, r, col, g);
  if (CM) {
    store_state<D>(X, r + D * D, col, g);
    y += __shfl_xor(y, 1);
    y += __shfl_xor(y, 2);
    if ((tid & 3) == 0) r[2 * D * D + (tid >> 2)] = y;
  }
}

// pre[bh][s][off .. off + len): the sum of that part of the records before
// segment s, sixteen records' loads in flight.  grid (ceil(len / 256), BH).
__global__ __launch_bounds__(256) void k_gprefix(const float* __restrict__ rec, float* __restrict__ pre, size_t F,
                                                 size_t off, size_t len, int nseg) {
  const size_t p = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= len) return;
  const float* src = rec + (size_t)blockIdx.y * nseg * F + off + p;
  float* dst = pre + (size_t)blockIdx.y * nseg * F + off + p;
  float x = 0.f;
  for (int s = 0; s < nseg; s += 16) {
    float u[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) u[j] = src[(size_t)min(s + j, nseg - 1) * F];
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (s + j < nseg) {
        dst[(size_t)(s + j) * F] = x;
        x += u[j];
      }
  }
}

// One segment's walk, grid (nseg, BH).  pre: the running sums (null: sum the
// records before this segment here).  den: the rows' denominators without the
// carry (masked with several segments: k_gfix divides) or den_out (final).
template <typename T, int D, bool MASKED>
__global__ __launch_bounds__(4 * D, D == 128 ? 2 : 3) void k_gwalk(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, float* __restrict__ out,
    float* __restrict__ den, float* __restrict__ rec, const float* __restrict__ pre, int n, int cps, int nseg,
    int normalized, float eps) {
  using G = GW<D>;
  constexpr int NW = G::NW, ldq = G::ldq, ldr = G::ldr, ldw = G::ldw;
  extern __shared__ __align__(16) float smem32[];
  float* Qs = smem32 + G::oQ;
  float* Vs = smem32 + G::oV;
  float* Ks = smem32 + G::oR;
  double* R = reinterpret_cast<double*>(smem32 + G::oR);
  float* W = smem32 + G::oW;
  float* ys = smem32 + G::oy;
  float* dn = smem32 + G::oden;
  int seg, bh;
  seg_head(seg, bh);
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nn = tid & 15, g = (tid >> 4) & 3, col = w * 16 + nn;
  const int M = (n + kTile - 1) / kTile, c0 = seg * cps, c1 = min(M, c0 + cps);
  const bool divide = normalized && (!MASKED || nseg == 1);
  q += (size_t)bh * n * D;
  k += (size_t)bh * n * D;
  v += (size_t)bh * n * D;
  out += (size_t)bh * n * D;
  if (den) den += (size_t)bh * n;
  Tile<T, D> pq, pk, pv;
  auto fetch = [&](int c) {
    pq.fetch(q, c * kTile, n);
    pk.fetch(k, c * kTile, n);
    pv.fetch(v, c * kTile, n);
  };
  fetch(c0);
  // the carry: the records before this segment
  const float* src = (pre ? pre : rec) + (size_t)bh * nseg * G::F;
  const int lo = pre ? seg : 0, hi = pre ? seg + 1 : seg;
  f32x4c S[NW], X[NW];
  load_state<D>(S, src, G::F, lo, hi, col, g);
  load_state<D>(X, src + D * D, G::F, lo, MASKED ? lo : hi, col, g);
  if (tid < D) {
    float y = 0.f;
    if (!MASKED)
      for (int s = lo; s < hi; ++s) y += src[(size_t)s * G::F + 2 * D * D + tid];
    ys[tid] = y;
  }
  // the three tiles on or below the diagonal: rows m0, columns n0
  auto tri = [&](int tile, int& m0, int& n0) {
    m0 = tile == 0 ? 0 : 16;
    n0 = tile == 2 ? 16 : 0;
  };
  const f64x4c zd = {0.0, 0.0, 0.0, 0.0};

  for (int c = c0; c < c1; ++c) {
    // the lane index made opaque once per tile: LDS offsets are formed here
    // and none is hoisted out of the loop, where they would fill the registers
    int ln = tid & 63;
    asm volatile("" : "+v"(ln));
    const int nn = ln & 15, g = ln >> 4, col = w * 16 + nn, pr = mfma_pr(nn);
    pq.store(Qs);
    pk.store(Ks);
    pv.store(Vs);
    lds_barrier();
    if (c + 1 < c1) fetch(c + 1);
    auto put_tri = [&](const f64x4c& acc, int m0, int n0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = m0 + 4 * g + i, j = n0 + nn;
        W[t * ldw + j] = j <= t ? (float)acc[i] : 0.f;
      }
    };

    // W, and the carry products Q S0 and (masked) Q X0
    for (int tile = w; tile < 3; tile += NW) {
      int m0, n0;
      tri(tile, m0, n0);
      f64x4c acc = zd;
#pragma unroll
      for (int kt = 0; kt < NW; ++kt) {
        const float4 a = *reinterpret_cast<const float4*>(Qs + (m0 + pr) * ldq + 16 * kt + 4 * g);
        const float4 b = *reinterpret_cast<const float4*>(Ks + (n0 + nn) * ldq + 16 * kt + 4 * g);
        acc = mfma4((double)a.x, (double)b.x, acc);
        acc = mfma4((double)a.y, (double)b.y, acc);
        acc = mfma4((double)a.z, (double)b.z, acc);
        acc = mfma4((double)a.w, (double)b.w, acc);
      }
      put_tri(acc, m0, n0);
    }
    f64x4c r[2] = {zd, zd}, o[2] = {zd, zd};
#pragma unroll
    for (int kt = 0; kt < NW; ++kt) {
      float4 a4[2];
#pragma unroll
      for (int m = 0; m < 2; ++m)
        a4[m] = *reinterpret_cast<const float4*>(Qs + (16 * m + pr) * ldq + 16 * kt + 4 * g);
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const double a[4] = {(double)a4[m].x, (double)a4[m].y, (double)a4[m].z, (double)a4[m].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          r[m] = mfma4(a[i], (double)S[kt][i], r[m]);
          if (MASKED) o[m] = mfma4(a[i], (double)X[kt][i], o[m]);
        }
      }
    }
    lds_barrier();

    // R += W K (W is zero past the diagonal); S0 += K^T K
    float kb[8];
    column8<D>(kb, Ks, col, g);
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const float* b = kb + 4 * kt;
#pragma unroll
      for (int m = kt; m < 2; ++m) {
        const float4 a = *reinterpret_cast<const float4*>(W + (16 * m + pr) * ldw + 16 * kt + 4 * g);
        r[m] = mfma4((double)a.x, (double)b[0], r[m]);
        r[m] = mfma4((double)a.y, (double)b[1], r[m]);
        r[m] = mfma4((double)a.z, (double)b[2], r[m]);
        r[m] = mfma4((double)a.w, (double)b[3], r[m]);
      }
    }
    if (c + 1 < c1) add_outer<T, D>(S, Ks, kb, nn, g);
    lds_barrier();                     // K is dead: R takes its space
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) R[(16 * m + 4 * g + i) * ldr + col] = r[m][i];
    lds_barrier();

    // T, unmasked R X0, the denominators' carry part, and the advance of X0 and y
    for (int tile = w; tile < 3; tile += NW) {
      int m0, n0;
      tri(tile, m0, n0);
      const int rq = MASKED ? m0 + pr : n0 + nn, rr = MASKED ? n0 + nn : m0 + pr;
      f64x4c acc = zd;
#pragma unroll
      for (int kt = 0; kt < NW; ++kt) {
        const float4 a = *reinterpret_cast<const float4*>(Qs + rq * ldq + 16 * kt + 4 * g);
        const double2 b0 = *reinterpret_cast<const double2*>(R + rr * ldr + 16 * kt + 4 * g);
        const double2 b1 = *reinterpret_cast<const double2*>(R + rr * ldr + 16 * kt + 4 * g + 2);
        const double x[4] = {(double)a.x, (double)a.y, (double)a.z, (double)a.w}, y[4] = {b0.x, b0.y, b1.x, b1.y};
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = MASKED ? mfma4(x[i], y[i], acc) : mfma4(y[i], x[i], acc);
      }
      put_tri(acc, m0, n0);
    }
    if (!MASKED) {
#pragma unroll
      for (int kt = 0; kt < NW; ++kt)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const double2 b0 = *reinterpret_cast<const double2*>(R + (16 * m + pr) * ldr + 16 * kt + 4 * g);
          const double2 b1 = *reinterpret_cast<const double2*>(R + (16 * m + pr) * ldr + 16 * kt + 4 * g + 2);
          o[m] = mfma4(b0.x, (double)X[kt][0], o[m]);
          o[m] = mfma4(b0.y, (double)X[kt][1], o[m]);
          o[m] = mfma4(b1.x, (double)X[kt][2], o[m]);
          o[m] = mfma4(b1.y, (double)X[kt][3], o[m]);
        }
    }
    const int trow = tid / G::LPR, part = tid % G::LPR;
    double sd = 0.0;
    float yinc = 0.f;
    if (normalized) {
#pragma unroll
      for (int a = 0; a < 8; ++a)
        sd += (MASKED ? (double)Qs[trow * ldq + part * 8 + a] : R[trow * ldr + part * 8 + a]) * (double)ys[part * 8 + a];
      double yd = 0.0;                 // four lanes a dimension, eight tokens each
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int t = (tid & 3) * 8 + j;
        yd += MASKED ? R[t * ldr + (tid >> 2)] : (double)Qs[t * ldq + (tid >> 2)];
      }
      yd += __shfl_xor(yd, 1);
      yd += __shfl_xor(yd, 2);
      yinc = (float)yd;
    }
    float vb[8];
    column8<D>(vb, Vs, col, g);
    if constexpr (MASKED) {
      constexpr int GR = D == 128 ? 4 : 1;   // row tiles side by side: fp32 1x300x2048 2285 -> 2246 us; none at d = 64
#pragma unroll
      for (int r0 = 0; r0 < NW; r0 += GR) {
        f32x4c x[GR];
#pragma unroll
        for (int r = 0; r < GR; ++r) x[r] = f32x4c{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int r = 0; r < GR; ++r)
            x[r] = mfma4((float)R[(16 * (j >> 2) + 4 * g + (j & 3)) * ldr + 16 * (r0 + r) + nn], vb[j], x[r]);
#pragma unroll
        for (int r = 0; r < GR; ++r) X[r0 + r] += x[r];
      }
    } else {
      add_outer<T, D>(X, Qs, vb, nn, g);
    }
    lds_barrier();

    // O = carry + T V, and the rows' denominators
    if (normalized) {
      float s = 0.f;
      for (int j = part; j <= trow; j += G::LPR) s += W[trow * ldw + j];
#pragma unroll
      for (int x = 1; x < G::LPR; x <<= 1) {
        s += __shfl_xor(s, x);
        sd += __shfl_xor(sd, x);
      }
      s += (float)sd;
      if (part == 0) {
        dn[trow] = s;
        if (den && c * kTile + trow < n) den[c * kTile + trow] = s;
      }
      if ((tid & 3) == 0) ys[tid >> 2] += yinc;
      if (divide) lds_barrier();
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      f32x4c acc;
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = (float)o[m][i];
#pragma unroll
      for (int kt = 0; kt <= m; ++kt) {
        const float4 a = *reinterpret_cast<const float4*>(W + (16 * m + nn) * ldw + 16 * kt + 4 * g);
        acc = mfma4(a.x, vb[4 * kt + 0], acc);
        acc = mfma4(a.y, vb[4 * kt + 1], acc);
        acc = mfma4(a.z, vb[4 * kt + 2], acc);
        acc = mfma4(a.w, vb[4 * kt + 3], acc);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tl = 16 * m + 4 * g + i, t = c * kTile + tl;
        if (t < n) out[(size_t)t * D + col] = divide ? acc[i] / (dn[tl] + eps) : acc[i];
      }
    }
    lds_barrier();                     // the next tile rewrites every LDS tile
  }
  if (MASKED && nseg > 1) {            // the segment's bracket
    float* r = rec + ((size_t)bh * nseg + seg) * G::F + D * D;
    store_state<D>(X, r, col, g);
    if (tid < D) r[D * D + tid] = ys[tid];
  }
}

// out_t += q_t^T X with X the brackets of the segments before t's, and the
// division when normalised; grid (nseg sub, BH), tpw tiles of one segment a
// workgroup.  Segment 0 has nothing to add.
template <typename T, int D>
__global__ __launch_bounds__(4 * D) void k_gfix(const T* __restrict__ q, float* __restrict__ out,
                                                const float* __restrict__ den, float* __restrict__ den_out,
                                                const float* __restrict__ rec, const float* __restrict__ pre, int n,
                                                int cps, int nseg, int sub, int tpw, int normalized, float eps) {
  using G = GW<D>;
  constexpr int NW = G::NW, ldq = G::ldq;
  __shared__ __align__(16) float Qs[kTile * G::ldq];
  __shared__ float ys[D], inv[kTile];
  int seg, bh;
  seg_head(seg, bh);
  const int part0 = seg % sub * tpw;
  seg /= sub;
  const int tid = threadIdx.x, nn = tid & 15, g = (tid >> 4) & 3, col = (tid >> 6) * 16 + nn, pr = mfma_pr(nn);
  const int M = (n + kTile - 1) / kTile, c0 = seg * cps + part0, c1 = min(M, min(c0 + tpw, (seg + 1) * cps));
  if (c0 >= c1 || (seg == 0 && !normalized)) return;
  q += (size_t)bh * n * D;
  out += (size_t)bh * n * D;
  Tile<T, D> pq;
  pq.fetch(q, c0 * kTile, n);
  const float* src = (pre ? pre : rec) + (size_t)bh * nseg * G::F + D * D;
  const int lo = pre ? seg : 0, hi = pre ? seg + 1 : seg;
  f32x4c X[NW];
  load_state<D>(X, src, G::F, lo, hi, col, g);
  if (tid < D) {
    float y = 0.f;
    for (int s = lo; s < hi; ++s) y += src[(size_t)s * G::F + D * D + tid];
    ys[tid] = y;
  }
  for (int c = c0; c < c1; ++c) {
    float prev[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = c * kTile + 16 * m + 4 * g + i;
        prev[m][i] = t < n ? out[(size_t)t * D + col] : 0.f;
      }
    pq.store(Qs);
    lds_barrier();
    if (c + 1 < c1) pq.fetch(q, (c + 1) * kTile, n);
    if (normalized) {
      const int trow = tid / G::LPR, part = tid % G::LPR, t = c * kTile + trow;
      double sd = 0.0;
#pragma unroll
      for (int a = 0; a < 8; ++a) sd += (double)Qs[trow * ldq + part * 8 + a] * (double)ys[part * 8 + a];
#pragma unroll
      for (int x = 1; x < G::LPR; x <<= 1) sd += __shfl_xor(sd, x);
      if (part == 0 && t < n) {
        const float s = den[(size_t)bh * n + t] + (float)sd;
        inv[trow] = s + eps;
        if (den_out) den_out[(size_t)bh * n + t] = s;
      }
    }
    f64x4c o[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int kt = 0; kt < NW; ++kt)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const float4 a = *reinterpret_cast<const float4*>(Qs + (16 * m + pr) * ldq + 16 * kt + 4 * g);
        o[m] = mfma4((double)a.x, (double)X[kt][0], o[m]);
        o[m] = mfma4((double)a.y, (double)X[kt][1], o[m]);
        o[m] = mfma4((double)a.z, (double)X[kt][2], o[m]);
        o[m] = mfma4((double)a.w, (double)X[kt][3], o[m]);
      }
    lds_barrier();                     // the denominators; Q is rewritten by the next tile
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tl = 16 * m + 4 * g + i, t = c * kTile + tl;
        const float x = prev[m][i] + (float)o[m][i];
        if (t < n) out[(size_t)t * D + col] = normalized ? x / inv[tl] : x;
      }
    if (normalized) lds_barrier();     // inv is rewritten by the next tile
  }
}

// Floats of workspace at P segments a head: the records, their running sums
// when there are more than kSelfSum, and the walks' denominators.
size_t ws_floats(int BH, int n, int d, int P, int masked, int normalized) {
  const size_t F = (size_t)2 * d * d + d, r = P > 1 ? (size_t)BH * P * F : 0;
  return (P > kSelfSum ? 2 : 1) * r + (masked && normalized && P > 1 ? (size_t)BH * n : 0);
}

template <typename T, int D>
hipError_t run(const Fwd& f, float* ws, size_t ws_bytes, hipStream_t s) {
  using G = GW<D>;
  const int M = (f.n + kTile - 1) / kTile, BH = f.BH, n = f.n;
  // enough segments to fill the chip, as many as the workspace holds
  int P = 256 * G::kBlocks / BH;
  if (!f.masked && M > kMaxTiles * std::max(P, 1))
    P = std::max((M + kMaxTiles - 1) / kMaxTiles, (4 * 256 * G::kBlocks + BH - 1) / BH);
  if (const char* e = getenv("HLA_FUSED_SEGMENTS")) P = atoi(e);
  P = P < 1 ? 1 : P > M ? M : P;
  while (P > 1 && 4 * ws_floats(BH, n, D, P, f.masked, f.normalized) > ws_bytes) --P;
  const int cps = (M + P - 1) / P;
  P = (M + cps - 1) / cps;
  float* rec = ws;
  float* pre = P > kSelfSum ? rec + (size_t)BH * P * G::F : nullptr;
  float* den = rec + (size_t)(P > kSelfSum ? 2 : 1) * BH * P * G::F;
  const T* q = static_cast<const T*>(f.q);
  const T* k = static_cast<const T*>(f.k);
  const T* v = static_cast<const T*>(f.v);
  hipError_t e;
  auto prefix = [&](size_t off, size_t len) {
    HLA_LAUNCH(k_gprefix, dim3((unsigned)((len + 255) / 256), BH), dim3(256), 0, s, rec, pre, G::F, off, len, P);
    return hipGetLastError();
  };
  if (P > 1) {
    prof_start("moments32", s);
    if (f.masked)
      HLA_LAUNCH((k_gmoments<T, D, false>), dim3(P, BH), dim3(G::NT), 0, s, q, k, v, rec, n, cps, P);
    else
      HLA_LAUNCH((k_gmoments<T, D, true>), dim3(P, BH), dim3(G::NT), 0, s, q, k, v, rec, n, cps, P);
    prof_stop(s);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (pre && (e = HLA_PROF("prefix32", s, prefix(0, f.masked ? (size_t)D * D : G::F))) != hipSuccess) return e;
  }
  const bool later = f.masked && P > 1;
  float* dp = later ? (f.normalized ? den : nullptr) : f.den_out;
  const void* fn = f.masked ? (const void*)k_gwalk<T, D, true> : (const void*)k_gwalk<T, D, false>;
  if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::bytes)) != hipSuccess) return e;
  float* out = f.out;
  const float* cpre = pre;
  int ni = n, ci = cps, pi = P, no = f.normalized;
  float eps = f.eps;
  void* args[] = {&q, &k, &v, &out, &dp, &rec, &cpre, &ni, &ci, &pi, &no, &eps};
  prof_start("walk32", s);
  e = prof_launch(fn, dim3(P, BH), dim3(G::NT), args, G::bytes, s);
  prof_stop(s);
  if (e != hipSuccess || (e = hipGetLastError()) != hipSuccess) return e;
  if (later) {
    if (pre && (e = HLA_PROF("prefix32", s, prefix((size_t)D * D, (size_t)D * D + D))) != hipSuccess) return e;
    prof_start("fix32", s);
    const int tpw = D <= 32 ? 1 : 2, sub = (cps + tpw - 1) / tpw;
    HLA_LAUNCH((k_gfix<T, D>), dim3(P * sub, BH), dim3(G::NT), 0, s, q, f.out, den, f.den_out, rec, pre, n, cps, P,
               sub, tpw, f.normalized, f.eps);
    prof_stop(s);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
hipError_t run_d(const Fwd& f, float* ws, size_t ws_bytes, hipStream_t s) {
  switch (f.d) {
    case 16: return run<T, 16>(f, ws, ws_bytes, s);
    case 32: return run<T, 32>(f, ws, ws_bytes, s);
    case 64: return run<T, 64>(f, ws, ws_bytes, s);
    case 128: return run<T, 128>(f, ws, ws_bytes, s);
  }
  return hipErrorNotSupported;
}

}  // namespace

bool walk32_supported(const Fwd& f) { return f.d == f.dv && f.gamma == 1.f && f.out; }

hipError_t launch_walk32(const Fwd& f, void* ws, size_t ws_bytes, hipStream_t s) {
  if (!walk32_supported(f)) return hipErrorNotSupported;
  float* w = static_cast<float*>(ws);
  return f.dtype == 1 ? run_d<uint16_t>(f, w, ws_bytes, s) : run_d<float>(f, w, ws_bytes, s);
}

}  // namespace hla
