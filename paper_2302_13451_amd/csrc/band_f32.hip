// Band attention in float32 arithmetic on the matrix cores
// (v_mfma_f32_16x16x4_f32), any window: the float32 SA and LLSA forward, and
// the backward of SA, two-branch LLSA and the paper's LLSA for float32 tensors
// and for the bfloat16 windows that no staged kernel takes.
//
// One wave owns 16 rows (queries, or keys in the backward's key role), one row
// per lane column of the MFMA's N dimension, and sweeps the rows its window
// reads in blocks of 16 that start exactly at the window's first row. Operands
// go from memory straight into the operand registers, in two patterns:
//   * rows (products that contract over the head dim): lane (g, col) loads
//     row col's pieces g. Which feature a contraction step takes does not
//     matter as long as both operands agree, so a lane's 16-byte load serves
//     several steps;
//   * transposed rows (products that contract over frames): lane (g, col)
//     loads features F col .. F col + F - 1 (F = D / 16) of row 4g + i for step
//     i. A score tile comes out as rows 4g + i of column col, which is the
//     weight operand of step i: weights never leave their registers.
// Both patterns read whole rows per instruction, the four waves of a workgroup
// own neighbouring rows and meet in the L1, and a block's loads are issued
// before the products of the block before it finish, so no LDS and no barrier
// is needed. What bounds it: the float32 MFMA rate (157 TFLOP/s: a 16 x 16
// block and 64 features is 512 cycles of one SIMD per product) against the
// rows' way through the L1; HBM only sees each row about once.
//
// A matrix product multiplies the rows outside a row's window by a zero
// weight, and 0 * inf is NaN: a wave that ends with a value that is not finite
// recomputes its rows one by one over their own windows only (rows_slow), so
// that an infinity or NaN reaches exactly the rows whose window holds it.
#include "device_common.h"
#include "kernels.h"
#include "sa.h"

namespace sa {
namespace {

constexpr int kThreads = 256;
constexpr int kRowsPerWave = 16;
constexpr int kTileRows = 64;          // rows of a workgroup (four waves)
constexpr int kMaxGrid = 1 << 20;      // workgroups per launch; more items loop
constexpr int kMaxOut = SA_LLSA_PAPER_MAX_LA + 1;  // outputs and branches of one backward call

__device__ __forceinline__ float lo_bf(uint32_t x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float hi_bf(uint32_t x) { return __uint_as_float(x & 0xffff0000u); }

// Row pattern: this lane's D / 4 features of a row, in contraction-step order.
template <int D>
__device__ __forceinline__ void row_frag(const float* row, int g, float* x) {
#pragma unroll
  for (int j = 0; j < D / 16; ++j) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(row + 16 * j + 4 * g);
#pragma unroll
    for (int s = 0; s < 4; ++s) x[4 * j + s] = v[s];
  }
}
template <int D>
__device__ __forceinline__ void row_frag(const uint16_t* row, int g, float* x) {
#pragma unroll
  for (int j = 0; j < D / 32; ++j) {
    const u32x4 v = ld16(row + 32 * j + 8 * g);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      x[8 * j + 2 * s] = lo_bf(v[s]);
      x[8 * j + 2 * s + 1] = hi_bf(v[s]);
    }
  }
}

// Features F col .. F col + F - 1 of a row (F = D / 16: 2 or 4).
template <int D>
__device__ __forceinline__ void feat_frag(const float* row, int col, float* x) {
  if constexpr (D == 64) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(row + 4 * col);
    x[0] = v[0]; x[1] = v[1]; x[2] = v[2]; x[3] = v[3];
  } else {
    const f32x2 v = *reinterpret_cast<const f32x2*>(row + 2 * col);
    x[0] = v[0]; x[1] = v[1];
  }
}
template <int D>
__device__ __forceinline__ void feat_frag(const uint16_t* row, int col, float* x) {
  if constexpr (D == 64) {
    const u32x2 v = *reinterpret_cast<const u32x2*>(row + 4 * col);
    x[0] = lo_bf(v[0]); x[1] = hi_bf(v[0]); x[2] = lo_bf(v[1]); x[3] = hi_bf(v[1]);
  } else {
    const uint32_t v = *reinterpret_cast<const uint32_t*>(row + 2 * col);
    x[0] = lo_bf(v); x[1] = hi_bf(v);
  }
}
__device__ __forceinline__ void store_feat(float* p, const float* x, int n) {
  if (n == 4) *reinterpret_cast<f32x4*>(p) = f32x4{x[0], x[1], x[2], x[3]};
  else *reinterpret_cast<f32x2*>(p) = f32x2{x[0], x[1]};
}
__device__ __forceinline__ void store_feat(uint16_t* p, const float* x, int n) {
  if (n == 4) st8(p, u32x2{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])});
  else *reinterpret_cast<uint32_t*>(p) = pack_bf16x2(x[0], x[1]);
}

// A . B over the head dim: 16 rows against the wave's 16 own rows. Two chains,
// so that a product does not wait for the one before it.
template <int N>
__device__ __forceinline__ f32x4 row_product(const float* a, const float* b) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
  for (int n = 0; n < N; n += 2) {
    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[n], b[n], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[n + 1], b[n + 1], s1, 0, 0, 0);
  }
  return s0 + s1;
}

// acc[f] += X^T W over 16 frames: x[i] this lane's features of frame 4g + i,
// w[i] the weights of that frame.
template <int F>
__device__ __forceinline__ void col_product(const float (*x)[F], const float* w, f32x4* acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int f = 0; f < F; ++f) acc[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][f], w[i], acc[f], 0, 0, 0);
}

template <int F>
__device__ __forceinline__ bool all_finite(const f32x4* acc) {
  float z = 0.f;
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) z = __builtin_fmaf(acc[f][r], 0.f, z);  // NaN for an infinity or NaN
  return z == 0.f;
}

// Stores row col's features, held as acc[f][r] = feature F (4g + r) + f,
// times mul (zero rows when !valid). The lanes of a row first trade values
// (the swaps exchange a lane bit with a register index), so that every store
// instruction writes 64 contiguous bytes (32 of bfloat16) of 16 rows.
template <int D, typename E>
__device__ __forceinline__ void store_own_row(E* row, const f32x4* acc, float mul, bool valid, bool write, int g) {
  constexpr int F = D / 16;
  float x[4][F];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int f = 0; f < F; ++f) x[r][f] = valid ? acc[f][r] * mul : 0.f;
  auto swap32 = [](float& p, float& q) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    p = __uint_as_float(r[0]);
    q = __uint_as_float(r[1]);
  };
  auto swap16 = [](float& p, float& q) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    p = __uint_as_float(r[0]);
    q = __uint_as_float(r[1]);
  };
  if constexpr (D == 64) {
    // 4 x 4 transpose of the groups and the register rows: register row r then
    // holds features 16 r + 4 g ..
#pragma unroll
    for (int f = 0; f < F; ++f) {
      swap32(x[0][f], x[2][f]);
      swap32(x[1][f], x[3][f]);
      swap16(x[0][f], x[1][f]);
      swap16(x[2][f], x[3][f]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (write) store_feat(row + 16 * r + 4 * g, x[r], 4);
  } else {
    // features 8g + 2r + f: four of them (r = 0, 1 and r = 2, 3) make a piece;
    // after exchanging the upper lane bit with the piece index, piece n of lane
    // (b5, b4) is features 16 n + 8 b4 + 4 b5 ..
    float p[2][4] = {{x[0][0], x[0][1], x[1][0], x[1][1]}, {x[2][0], x[2][1], x[3][0], x[3][1]}};
#pragma unroll
    for (int j = 0; j < 4; ++j) swap32(p[0][j], p[1][j]);
#pragma unroll
    for (int n = 0; n < 2; ++n)
      if (write) store_feat(row + 16 * n + 8 * (g & 1) + 4 * (g >> 1), p[n], 4);
  }
}

// The frames one of a wave's columns sees, as a start and a width: frame x is
// inside iff unsigned(x - start) <= width; an empty range never matches.
struct Span {
  int start;
  unsigned width;
  __device__ __forceinline__ Span(bool valid, int lo, int hi) {
    const bool any = valid && hi >= lo;
    start = any ? lo : 1 << 30;
    width = any ? static_cast<unsigned>(hi - lo) : 0u;
  }
  __device__ __forceinline__ bool has(int x) const { return static_cast<unsigned>(x - start) <= width; }
};

// Zeros rows r0 .. r1 - 1 of a slice (one wave).
template <int D, typename E>
__device__ __forceinline__ void zero_rows(E* dst, int fs, int r0, int r1, int lane) {
  constexpr int CPR = D * sizeof(E) / 16, EPC = 16 / sizeof(E);
  for (int e = lane; e < (r1 - r0) * CPR; e += 64) st16(dst + (r0 + e / CPR) * fs + EPC * (e % CPR), kZero16);
}

// ---------------------------------------------------------------------------
// Forward: up to two outputs, each over one or two window segments.
struct FwdDev {
  BandJob job[2];
  int njobs, B, T, H, ntiles, items;
  const int32_t* lengths;
  float scale_log2;  // log2(e) / sqrt(d)
};

// The wave's rows one by one, lanes 16 i .. 16 i + 15 row r0 + 4 it + i: an
// online softmax over the row's own window.
template <int D>
__device__ void fwd_rows_slow(const FwdDev& a, const BandJob& job, size_t slice, int fs, int r0, int len,
                              float* lse, int lane) {
  constexpr int F = D / 16;
  const int col = lane & 15, g = lane >> 4;
  for (int it = 0; it < 4; ++it) {
    const int t = r0 + 4 * it + g;
    if (t >= len) continue;
    float q[F], acc[F];
    feat_frag<D>(static_cast<const float*>(job.q) + slice + t * fs, col, q);
#pragma unroll
    for (int f = 0; f < F; ++f) acc[f] = 0.f;
    float m = kNegInf, l = 0.f;
    for (int si = 0; si < job.nseg; ++si) {
      const BandSegment& sg = job.seg[si];
      const int lo = max(0, t + sg.lo_off), hi = min(len - 1, t + sg.hi_off);
      for (int key = lo; key <= hi; ++key) {
        float x[F], s = 0.f;
        feat_frag<D>(static_cast<const float*>(sg.k) + slice + key * fs, col, x);
#pragma unroll
        for (int f = 0; f < F; ++f) s += q[f] * x[f];
        s = group_sum<16>(s) * a.scale_log2;
        const float mn = fmaxf(m, s), alpha = fast_exp2(m - mn), p = fast_exp2(s - mn);
        m = mn;
        l = l * alpha + p;
        feat_frag<D>(static_cast<const float*>(sg.v) + slice + key * fs, col, x);
#pragma unroll
        for (int f = 0; f < F; ++f) acc[f] = acc[f] * alpha + p * x[f];
      }
    }
    const float inv = 1.f / l;
#pragma unroll
    for (int f = 0; f < F; ++f) acc[f] *= inv;
    store_feat(static_cast<float*>(job.out) + slice + t * fs + F * col, acc, F);
    if (lse && col == 0) lse[t] = (m + log2f(l)) * kLn2;
  }
}

// One wave, 16 queries; the window in steps of 32 keys with an online softmax.
template <int D>
__global__ __launch_bounds__(kThreads) void band_fwd_f32_kernel(FwdDev a) {
  constexpr int N = D / 4, F = D / 16;
  const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int T = a.T, H = a.H, fs = H * D;
  const float c2 = a.scale_log2;
  for (int bid = blockIdx.x; bid < a.items; bid += gridDim.x) {
    int bh, item;
    if (!xcd_slice_item(bid, a.B * H, a.njobs * a.ntiles, bh, item)) continue;
    const int tile = a.njobs > 1 ? item >> 1 : item;
    const BandJob& job = a.job[a.njobs > 1 ? item & 1 : 0];
    const int b = bh / H, h = bh - b * H;
    const int len = clamp_len_uniform(a.lengths, b, T);
    const int r0 = tile * kTileRows + kRowsPerWave * w;
    if (r0 >= T) continue;
    const size_t slice = row_index(b, 0, h, T, H, D);
    float* out = static_cast<float*>(job.out) + slice;
    float* lse = job.lse ? job.lse + (static_cast<size_t>(b) * H + h) * T : nullptr;
    const int t = r0 + col;
    if (r0 >= len) {
      zero_rows<D>(out, fs, r0, min(r0 + kRowsPerWave, T), lane);
      if (lse && g == 0 && t < T) lse[t] = kNegInf;
      continue;
    }
    const bool valid = t < len;
    const int wmax = min(r0 + kRowsPerWave - 1, len - 1);
    float q[N];
    row_frag<D>(static_cast<const float*>(job.q) + slice + min(t, len - 1) * fs, g, q);
    float m = kNegInf, lsum = 0.f;
    f32x4 acc[F];
#pragma unroll
    for (int f = 0; f < F; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int si = 0; si < job.nseg; ++si) {
      const BandSegment& sg = job.seg[si];
      const float* kp = static_cast<const float*>(sg.k) + slice;
      const float* vp = static_cast<const float*>(sg.v) + slice;
      const int wlo = max(0, r0 + sg.lo_off), whi = min(len - 1, wmax + sg.hi_off);
      if (wlo > whi) continue;
      const Span win(valid, max(0, t + sg.lo_off), min(len - 1, t + sg.hi_off));
      const int last = len - 1;
      float k[2][N];
      auto load_keys = [&](int kb) {
#pragma unroll
        for (int u = 0; u < 2; ++u) row_frag<D>(kp + min(kb + 16 * u + col, last) * fs, g, k[u]);
      };
      load_keys(wlo);
      for (int kb = wlo; kb <= whi; kb += 32) {
        float v[2][4][F];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) feat_frag<D>(vp + min(kb + 16 * u + 4 * g + i, last) * fs, col, v[u][i]);
        float z[2][4], zmax = kNegInf;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x4 s = row_product<N>(k[u], q);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            z[u][i] = win.has(kb + 16 * u + 4 * g + i) ? s[i] : kNegInf;
            zmax = fmaxf(zmax, z[u][i]);
          }
        }
        if (kb + 32 <= whi) load_keys(kb + 32);  // in flight behind the softmax and the PV product
        const float mn = fmaxf(m, max_over_column(zmax) * c2);
        const float ms = mn == kNegInf ? 0.f : mn;  // no key of the row so far
        const float alpha = fast_exp2(m - ms);
        m = mn;
        lsum *= alpha;
#pragma unroll
        for (int f = 0; f < F; ++f) acc[f] *= alpha;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            z[u][i] = fast_exp2(__builtin_fmaf(z[u][i], c2, -ms));
            lsum += z[u][i];
          }
          col_product<F>(v[u], z[u], acc);
        }
      }
    }
    if (__any(valid && !all_finite<F>(acc))) {
      fwd_rows_slow<D>(a, job, slice, fs, r0, len, lse, lane);
      if (wmax < r0 + kRowsPerWave - 1) zero_rows<D>(out, fs, wmax + 1, min(r0 + kRowsPerWave, T), lane);
      if (lse && g == 0 && !valid && t < T) lse[t] = kNegInf;
      continue;
    }
    lsum = sum_over_column(lsum);
    store_own_row<D>(out + static_cast<ptrdiff_t>(t) * fs, acc, valid ? 1.f / lsum : 0.f, valid, t < T, g);
    if (lse && g == 0 && t < T) lse[t] = valid ? (m + log2f(lsum)) * kLn2 : kNegInf;
  }
}

// ---------------------------------------------------------------------------
// Backward, in the general channel form (Eq. 7-13 per output row; the paper's
// Eq. 16 prints only the value part of the LLSA gradient). Channels
// c = 0 .. La, each held by a branch (tensor); output o computes channel c_o
// with the query of branch qb_o. Query t of output o reads the frames tau in
// [t + c_o - La - Lb, t + c_o] (clipped to the sequence), frame tau from the
// branch whose interval [elo, ehi] holds e = t + c_o - tau, so that output o
// reads from branch i the band t + c_o - ehi_i .. t + c_o - elo_i. SA is one
// output and one branch. With P the attention weights of a row,
// dP_tau = dout . v_tau, D = dout . out and dS = P (dP - D):
//   dq[qb_o]_t  += (1/sqrt d) sum_tau dS_(t,tau) k[i]_tau
//   dk[i]_tau   += (1/sqrt d) sum over the (o, t) that read tau from i of dS_(t,tau) q[qb_o]_t
//   dv[i]_tau   += sum over the same (o, t) of P_(t,tau) dout[o]_t
// A query role per (output, 16 frames) gathers dq over its bands, a key role
// per (branch, 16 frames) gathers dk and dv over the outputs' queries that
// read it. Each output's query branch is distinct, so every gradient row has
// one writer: no atomics, no workspace, deterministic.
struct BwdDev {
  const void *q, *k, *v, *out, *dout;
  const float* lse;
  void *dq, *dk, *dv;
  int B, T, H, ntiles, items;
  int nout, nbranch;
  int c[kMaxOut];    // channel of output o
  int qb[kMaxOut];   // branch of output o's query
  int elo[kMaxOut];  // e-interval of branch i (empty: elo > ehi)
  int ehi[kMaxOut];
  size_t bstride;  // elements of one branch (or output) tensor
  size_t lstride;  // floats of one output's lse
  const int32_t* lengths;
  float scale, scale_log2;
};

template <typename E, int D>
__device__ __forceinline__ float feat_dot(const float* x, const E* row, int col) {
  constexpr int F = D / 16;
  float y[F], s = 0.f;
  feat_frag<D>(row, col, y);
#pragma unroll
  for (int f = 0; f < F; ++f) s += x[f] * y[f];
  return group_sum<16>(s);
}

// The wave's gradient rows one by one (as fwd_rows_slow): the query role of
// output x, or the key role of branch x.
template <typename E, int D>
__device__ void bwd_rows_slow(const BwdDev& a, bool key_role, int x, int b, int h, int r0, int len, int lane) {
  constexpr int F = D / 16;
  const int col = lane & 15, g = lane >> 4;
  const int T = a.T, fs = a.H * D;
  const size_t slice = row_index(b, 0, h, T, a.H, D);
  const E *q = static_cast<const E*>(a.q) + slice, *k = static_cast<const E*>(a.k) + slice;
  const E *v = static_cast<const E*>(a.v) + slice, *o = static_cast<const E*>(a.out) + slice;
  const E* dout = static_cast<const E*>(a.dout) + slice;
  const float* lse = a.lse + (static_cast<size_t>(b) * a.H + h) * T;
  for (int it = 0; it < 4; ++it) {
    const int t = r0 + 4 * it + g;
    if (t >= len) continue;
    float acc0[F], acc1[F], x0[F], x1[F], y[F];
#pragma unroll
    for (int f = 0; f < F; ++f) acc0[f] = acc1[f] = 0.f;
    if (!key_role) {
      const size_t qo = a.qb[x] * a.bstride, oo = x * a.bstride;
      feat_frag<D>(q + qo + t * fs, col, x0);
      feat_frag<D>(dout + oo + t * fs, col, x1);
      const float dn = feat_dot<E, D>(x1, o + oo + t * fs, col);
      const float lse2 = lse[x * a.lstride + t] * kLog2e;
      for (int i = 0; i < a.nbranch; ++i) {
        const size_t ko = i * a.bstride;
        const int lo = max(0, t + a.c[x] - a.ehi[i]), hi = min(len - 1, t + a.c[x] - a.elo[i]);
        for (int tau = lo; tau <= hi; ++tau) {
          const float p = fast_exp2(feat_dot<E, D>(x0, k + ko + tau * fs, col) * a.scale_log2 - lse2);
          const float ds = p * (feat_dot<E, D>(x1, v + ko + tau * fs, col) - dn);
          feat_frag<D>(k + ko + tau * fs, col, y);
#pragma unroll
          for (int f = 0; f < F; ++f) acc0[f] += ds * y[f];
        }
      }
#pragma unroll
      for (int f = 0; f < F; ++f) acc0[f] *= a.scale;
      store_feat(static_cast<E*>(a.dq) + slice + qo + t * fs + F * col, acc0, F);
      continue;
    }
    const size_t ko = x * a.bstride;
    feat_frag<D>(k + ko + t * fs, col, x0);
    feat_frag<D>(v + ko + t * fs, col, x1);
    for (int oi = 0; oi < a.nout; ++oi) {
      const size_t qo = a.qb[oi] * a.bstride, oo = oi * a.bstride;
      const int lo = max(0, t - a.c[oi] + a.elo[x]), hi = min(len - 1, t - a.c[oi] + a.ehi[x]);
      for (int n = lo; n <= hi; ++n) {
        float dr[F];
        feat_frag<D>(dout + oo + n * fs, col, dr);
        feat_frag<D>(q + qo + n * fs, col, y);
        const float dn = feat_dot<E, D>(dr, o + oo + n * fs, col);
        float s = 0.f, dp = 0.f;
#pragma unroll
        for (int f = 0; f < F; ++f) {
          s += x0[f] * y[f];
          dp += x1[f] * dr[f];
        }
        const float p = fast_exp2(group_sum<16>(s) * a.scale_log2 - lse[oi * a.lstride + n] * kLog2e);
        const float ds = p * (group_sum<16>(dp) - dn);
#pragma unroll
        for (int f = 0; f < F; ++f) {
          acc0[f] += ds * y[f];
          acc1[f] += p * dr[f];
        }
      }
    }
#pragma unroll
    for (int f = 0; f < F; ++f) acc0[f] *= a.scale;
    store_feat(static_cast<E*>(a.dk) + slice + ko + t * fs + F * col, acc0, F);
    store_feat(static_cast<E*>(a.dv) + slice + ko + t * fs + F * col, acc1, F);
  }
}

template <typename E, int D>
__global__ __launch_bounds__(kThreads) void band_bwd_f32_kernel(BwdDev a) {
  constexpr int N = D / 4, F = D / 16;
  const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int T = a.T, H = a.H, fs = H * D;
  const int nroles = a.nbranch + a.nout;
  const float c2 = a.scale_log2;
  for (int bid = blockIdx.x; bid < a.items; bid += gridDim.x) {
    // items of a slice: the key roles and query roles of tile 0, of tile 1, ...
    int bh, item;
    if (!xcd_slice_item(bid, a.B * H, nroles * a.ntiles, bh, item)) continue;
    const int tile = item / nroles, role = item - tile * nroles;
    const bool key_role = role < a.nbranch;
    const int x = key_role ? role : role - a.nbranch;  // branch or output
    const int b = bh / H, h = bh - b * H;
    const int len = clamp_len_uniform(a.lengths, b, T);
    const int r0 = tile * kTileRows + kRowsPerWave * w;
    if (r0 >= T) continue;
    const size_t slice = row_index(b, 0, h, T, H, D);
    const int r1 = min(r0 + kRowsPerWave, T);
    E* const d0 = static_cast<E*>(key_role ? a.dk : a.dq) + slice + (key_role ? x : a.qb[x]) * a.bstride;
    E* const d1 = static_cast<E*>(a.dv) + slice + x * a.bstride;  // key role only
    if (r0 >= len) {
      zero_rows<D>(d0, fs, r0, r1, lane);
      if (key_role) zero_rows<D>(d1, fs, r0, r1, lane);
      continue;
    }
    const E *q = static_cast<const E*>(a.q) + slice, *k = static_cast<const E*>(a.k) + slice;
    const E *v = static_cast<const E*>(a.v) + slice, *o = static_cast<const E*>(a.out) + slice;
    const E* dout = static_cast<const E*>(a.dout) + slice;
    const float* lse = a.lse + (static_cast<size_t>(b) * H + h) * T;
    const int me = r0 + col, last = len - 1;
    const bool valid = me < len;
    const int wmax = min(r0 + kRowsPerWave - 1, last);
    const int own = min(me, last) * fs;
    f32x4 acc0[F], acc1[F];
#pragma unroll
    for (int f = 0; f < F; ++f) acc0[f] = acc1[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (key_role) {
      float kf[N], vf[N];
      row_frag<D>(k + x * a.bstride + own, g, kf);
      row_frag<D>(v + x * a.bstride + own, g, vf);
      for (int oi = 0; oi < a.nout; ++oi) {
        const int lo = a.c[oi] - a.ehi[x], hi = a.c[oi] - a.elo[x];
        const int wlo = max(0, r0 - hi), whi = min(last, wmax - lo);
        if (lo > hi || wlo > whi) continue;
        const Span see(valid, max(0, me - hi), min(last, me - lo));  // queries that see this lane's key
        const E *qp = q + a.qb[oi] * a.bstride, *dp = dout + oi * a.bstride, *op = o + oi * a.bstride;
        const float* lp = lse + oi * a.lstride;
        for (int qb = wlo; qb <= whi; qb += 16) {
          float qr[N], dr[N], orow[N], qt[4][F], dt[4][F], l2[4];
          const int rr = min(qb + col, last) * fs;
          row_frag<D>(qp + rr, g, qr);
          row_frag<D>(dp + rr, g, dr);
          row_frag<D>(op + rr, g, orow);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int n = min(qb + 4 * g + i, last);
            l2[i] = lp[n];
            feat_frag<D>(dp + n * fs, col, dt[i]);
            feat_frag<D>(qp + n * fs, col, qt[i]);
          }
          const f32x4 s = row_product<N>(qr, kf), dpv = row_product<N>(dr, vf);
          // D of query col in every lane of the column, then of the queries
          // 4g + i whose scores this lane holds
          float dn = 0.f;
#pragma unroll
          for (int n = 0; n < N; ++n) dn += dr[n] * orow[n];
          dn = sum_over_column(dn);
          float p[4], ds[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float di =
                __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (4 * g + i), __float_as_int(dn)));
            const bool in = see.has(qb + 4 * g + i);
            const float pw = fast_exp2(__builtin_fmaf(s[i], c2, -l2[i] * kLog2e));
            p[i] = in ? pw : 0.f;
            ds[i] = in ? pw * (dpv[i] - di) : 0.f;
          }
          col_product<F>(dt, p, acc1);
          col_product<F>(qt, ds, acc0);
        }
      }
    } else {
      const size_t oo = x * a.bstride;
      float qf[N], df[N], dn = 0.f;
      row_frag<D>(q + a.qb[x] * a.bstride + own, g, qf);
      row_frag<D>(dout + oo + own, g, df);
      {
        float of[N];
        row_frag<D>(o + oo + own, g, of);
#pragma unroll
        for (int n = 0; n < N; ++n) dn += df[n] * of[n];
        dn = sum_over_column(dn);
      }
      const float l2 = lse[x * a.lstride + min(me, last)] * kLog2e;
      for (int i = 0; i < a.nbranch; ++i) {
        const int lo = a.c[x] - a.ehi[i], hi = a.c[x] - a.elo[i];
        const int wlo = max(0, r0 + lo), whi = min(last, wmax + hi);
        if (lo > hi || wlo > whi) continue;
        const Span win(valid, max(0, me + lo), min(last, me + hi));
        const E *kp = k + i * a.bstride, *vp = v + i * a.bstride;
        for (int kb = wlo; kb <= whi; kb += 16) {
          float kr[N], vr[N], kt[4][F];
          const int rr = min(kb + col, last) * fs;
          row_frag<D>(kp + rr, g, kr);
          row_frag<D>(vp + rr, g, vr);
#pragma unroll
          for (int u = 0; u < 4; ++u) feat_frag<D>(kp + min(kb + 4 * g + u, last) * fs, col, kt[u]);
          const f32x4 s = row_product<N>(kr, qf), dpv = row_product<N>(vr, df);
          float ds[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float pw = fast_exp2(__builtin_fmaf(s[u], c2, -l2));
            ds[u] = win.has(kb + 4 * g + u) ? pw * (dpv[u] - dn) : 0.f;
          }
          col_product<F>(kt, ds, acc0);
        }
      }
    }
    if (__any(valid && !(all_finite<F>(acc0) && all_finite<F>(acc1)))) {
      bwd_rows_slow<E, D>(a, key_role, x, b, h, r0, len, lane);
      if (len < r1) {
        zero_rows<D>(d0, fs, len, r1, lane);
        if (key_role) zero_rows<D>(d1, fs, len, r1, lane);
      }
      continue;
    }
    store_own_row<D>(d0 + static_cast<ptrdiff_t>(me) * fs, acc0, a.scale, valid, me < T, g);
    if (key_role) store_own_row<D>(d1 + static_cast<ptrdiff_t>(me) * fs, acc1, 1.f, valid, me < T, g);
  }
}

template <typename E>
hipError_t launch_bwd(BwdDev& a, int d, hipStream_t stream) {
  a.ntiles = (a.T + kTileRows - 1) / kTileRows;
  a.items = xcd_slice_grid(a.B * a.H, (a.nbranch + a.nout) * a.ntiles);
  a.scale = 1.f / sqrtf(static_cast<float>(d));
  a.scale_log2 = kLog2e * a.scale;
  const dim3 grid(a.items < kMaxGrid ? a.items : kMaxGrid), block(kThreads);
  if (d == 64)
    hipLaunchKernelGGL((band_bwd_f32_kernel<E, 64>), grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((band_bwd_f32_kernel<E, 32>), grid, block, 0, stream, a);
  return hipGetLastError();
}

template <typename Args>
BwdDev common(const Args& x) {
  BwdDev a{};
  a.q = x.q;
  a.k = x.k;
  a.v = x.v;
  a.out = x.out;
  a.dout = x.dout;
  a.lse = x.lse;
  a.dq = x.dq;
  a.dk = x.dk;
  a.dv = x.dv;
  a.B = x.B;
  a.T = x.T;
  a.H = x.H;
  a.lengths = x.lengths;
  a.bstride = static_cast<size_t>(x.B) * x.T * x.H * x.d;
  a.lstride = static_cast<size_t>(x.B) * x.H * x.T;
  return a;
}

hipError_t launch_bwd_typed(BwdDev& a, int d, ElemType et, hipStream_t stream) {
  return et == kBF16 ? launch_bwd<uint16_t>(a, d, stream) : launch_bwd<float>(a, d, stream);
}

}  // namespace

hipError_t launch_band_forward_f32(const BandForwardArgs& x, hipStream_t stream) {
  FwdDev a{};
  a.job[0] = x.job[0];
  a.job[1] = x.job[x.njobs > 1 ? 1 : 0];
  a.njobs = x.njobs;
  a.B = x.B;
  a.T = x.T;
  a.H = x.H;
  a.ntiles = (x.T + kTileRows - 1) / kTileRows;
  a.items = xcd_slice_grid(x.B * x.H, x.njobs * a.ntiles);
  a.lengths = x.lengths;
  a.scale_log2 = kLog2e / sqrtf(static_cast<float>(x.d));
  const dim3 grid(a.items < kMaxGrid ? a.items : kMaxGrid), block(kThreads);
  if (x.d == 64)
    hipLaunchKernelGGL(band_fwd_f32_kernel<64>, grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL(band_fwd_f32_kernel<32>, grid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_sa_backward_f32(const SaBackwardArgs& x, hipStream_t stream) {
  BwdDev a = common(x);
  a.nout = a.nbranch = 1;
  a.c[0] = x.La;
  a.ehi[0] = x.La + x.Lb;
  return launch_bwd<float>(a, x.d, stream);
}

hipError_t launch_llsa_backward_general(const LlsaBackwardArgs& x, ElemType et, hipStream_t stream) {
  BwdDev a = common(x);
  // branch 0 (causal) holds channels 0 .. La-1, branch 1 (look-ahead) channel La;
  // output 0 is channel 0 with branch 0's query, output 1 channel La with branch 1's
  a.nout = 2;
  a.nbranch = 2;
  a.c[1] = x.La;
  a.qb[1] = 1;
  a.ehi[0] = x.La - 1;  // empty when La = 0
  a.elo[1] = x.La;
  a.ehi[1] = x.La + x.Lb;
  return launch_bwd_typed(a, x.d, et, stream);
}

hipError_t launch_llsa_paper_backward_general(const LlsaPaperBwdArgs& x, ElemType et, hipStream_t stream) {
  BwdDev a = common(x);
  // every channel a branch of its own, computed with its own query
  a.nout = x.La + 1;
  a.nbranch = x.La + 1;
  for (int c = 0; c <= x.La; ++c) {
    a.c[c] = c;
    a.qb[c] = c;
    a.elo[c] = c;
    a.ehi[c] = c < x.La ? c : x.La + x.Lb;
  }
  return launch_bwd_typed(a, x.d, et, stream);
}

}  // namespace sa
