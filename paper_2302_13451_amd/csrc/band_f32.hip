// Band attention in float32 arithmetic on the matrix cores
// (v_mfma_f32_16x16x4_f32), any window: the float32 SA and LLSA forward, and
// the float32 backward of SA, two-branch LLSA and the paper's LLSA.
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
// The four waves of a workgroup own neighbouring rows and meet in the L1; a
// block's row loads are issued once the score products of the block before it
// have taken their operands, its transposed rows before its score products, so
// neither LDS nor a barrier is needed.
//
// What bounds it (B = 8, T = 500, H = 12, d = 64, Lb = 32, La = 8, ragged):
// backward 54 us, of which the float32 matrix instructions are 14 us (512 cycles
// of one SIMD per product of a 16 x 16 block and 64 features) and the traffic 14
// us at the device copy's rate; the rest is the latency of a wave's four to five
// blocks at two waves per SIMD. One thread per row on the vector ALUs took 441
// us, loads in the order of use 57 us, and rows staged through LDS by a
// workgroup 61 us. Forward 16 us (177 us), at the same shape.
//
// A matrix product multiplies the rows outside a row's window by a zero
// weight, and 0 * inf is NaN: a wave that ends with a value that is not finite
// recomputes its rows one by one over their own windows only (rows_slow), so
// that an infinity or NaN reaches exactly the rows whose window holds it.
#include "device_common.h"
#include "channel_bwd.h"
#include "kernels.h"
#include "rows16.h"

namespace sa {
namespace {

constexpr int kThreads = 256;
constexpr int kTileRows = 64;  // rows of a workgroup (four waves)

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
    float acc[F];
    FeatFrag<float, D> q, x;
    q.load(static_cast<const float*>(job.q) + slice + t * fs, col);
#pragma unroll
    for (int f = 0; f < F; ++f) acc[f] = 0.f;
    float m = kNegInf, l = 0.f;
    for (int si = 0; si < job.nseg; ++si) {
      const BandSegment& sg = job.seg[si];
      const int lo = max(0, t + sg.lo_off), hi = min(len - 1, t + sg.hi_off);
      for (int key = lo; key <= hi; ++key) {
        float s = 0.f;
        x.load(static_cast<const float*>(sg.k) + slice + key * fs, col);
#pragma unroll
        for (int f = 0; f < F; ++f) s += q[f] * x[f];
        s = group_sum<16>(s) * a.scale_log2;
        const float mn = fmaxf(m, s), alpha = fast_exp2(m - mn), p = fast_exp2(s - mn);
        m = mn;
        l = l * alpha + p;
        x.load(static_cast<const float*>(sg.v) + slice + key * fs, col);
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
  constexpr int F = D / 16;
  const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int T = a.T, H = a.H, fs = H * D;
  const float c2 = a.scale_log2;
  const BlockRows<D> rows(fs, col, g);
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
    RowFrag<float, D> q;
    q.load(static_cast<const float*>(job.q) + slice + min(t, len - 1) * fs, g);
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
      RowFrag<float, D> k[2];
      auto load_keys = [&](int kb) {
#pragma unroll
        for (int u = 0; u < 2; ++u) k[u].load(kp + rows.row(kb + 16 * u, last), g);
      };
      load_keys(wlo);
      for (int kb = wlo; kb <= whi; kb += 32) {
        FeatFrag<float, D> v[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) v[u][i].load(vp + rows.frame(kb + 16 * u, i, last), col);
        float z[2][4], zmax = kNegInf;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x4 s = row_product(k[u], q);
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
          col_product(v[u], z[u], acc);
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
// Backward (the channel form of channel_bwd.h): a query role per (output, 16
// frames) gathers dq over its bands, a key role per (branch, 16 frames) gathers
// dk and dv over the outputs' queries that read it. Every gradient row has one
// writer: no atomics, no workspace, deterministic.
template <int D>
__global__ __launch_bounds__(kThreads) void band_bwd_f32_kernel(BwdDev a) {
  typedef float E;
  constexpr int N = D / 4, F = D / 16;
  const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int T = a.T, H = a.H, fs = H * D;
  const BlockRows<D> rows(fs, col, g);
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
      RowFrag<E, D> kf, vf;
      kf.load(k + x * a.bstride + own, g);
      vf.load(v + x * a.bstride + own, g);
      // the own rows are in before the loops: a wait for them inside would also
      // wait for the loads issued there
      __builtin_amdgcn_s_waitcnt(0x0f70);
      for (int oi = 0; oi < a.nout; ++oi) {
        const int lo = a.c[oi] - a.ehi[x], hi = a.c[oi] - a.elo[x];
        const int wlo = max(0, r0 - hi), whi = min(last, wmax - lo);
        if (lo > hi || wlo > whi) continue;
        const Span see(valid, max(0, me - hi), min(last, me - lo));  // queries that see this lane's key
        const E *qp = q + a.qb[oi] * a.bstride, *dp = dout + oi * a.bstride, *op = o + oi * a.bstride;
        const float* lp = lse + oi * a.lstride;
        // a block's rows are loaded while the dk and dv products of the block
        // before run, its transposed rows while its score products run
        RowFrag<E, D> qr, dr, orow;
        float lv;
        auto load_rows = [&](int qb) {
          const size_t rr = rows.row(qb, last);
          qr.load(qp + rr, g);
          dr.load(dp + rr, g);
          orow.load(op + rr, g);
          lv = lp[min(qb + col, last)];
        };
        load_rows(wlo);
        for (int qb = wlo; qb <= whi; qb += 16) {
          FeatFrag<E, D> qt[4], dt[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const size_t rt = rows.frame(qb, i, last);
            dt[i].load(dp + rt, col);
            qt[i].load(qp + rt, col);
          }
          const f32x4 s = row_product(qr, kf), dpv = row_product(dr, vf);
          // D and lse of query col in every lane of the column, then of the
          // queries 4g + i whose scores this lane holds
          float dn = 0.f;
#pragma unroll
          for (int n = 0; n < N; ++n) dn += dr[n] * orow[n];
          dn = sum_over_column(dn);
          const float l2 = lv * kLog2e;
          if (qb + 16 <= whi) load_rows(qb + 16);
          float p[4], ds[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int src = 4 * (4 * g + i);
            const float di = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(dn)));
            const float li = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(l2)));
            const bool in = see.has(qb + 4 * g + i);
            const float pw = fast_exp2(__builtin_fmaf(s[i], c2, -li));
            p[i] = in ? pw : 0.f;
            ds[i] = in ? pw * (dpv[i] - di) : 0.f;
          }
          col_product(dt, p, acc1);
          col_product(qt, ds, acc0);
        }
      }
    } else {
      const size_t oo = x * a.bstride;
      RowFrag<E, D> qf, df;
      float dn = 0.f;
      qf.load(q + a.qb[x] * a.bstride + own, g);
      df.load(dout + oo + own, g);
      {
        RowFrag<E, D> of;
        of.load(o + oo + own, g);
#pragma unroll
        for (int n = 0; n < N; ++n) dn += df[n] * of[n];
        dn = sum_over_column(dn);
      }
      const float l2 = lse[x * a.lstride + min(me, last)] * kLog2e;
      __builtin_amdgcn_s_waitcnt(0x0f70);
      for (int i = 0; i < a.nbranch; ++i) {
        const int lo = a.c[x] - a.ehi[i], hi = a.c[x] - a.elo[i];
        const int wlo = max(0, r0 + lo), whi = min(last, wmax + hi);
        if (lo > hi || wlo > whi) continue;
        const Span win(valid, max(0, me + lo), min(last, me + hi));
        const E *kp = k + i * a.bstride, *vp = v + i * a.bstride;
        RowFrag<E, D> kr, vr;
        auto load_rows = [&](int kb) {
          const size_t rr = rows.row(kb, last);
          kr.load(kp + rr, g);
          vr.load(vp + rr, g);
        };
        load_rows(wlo);
        for (int kb = wlo; kb <= whi; kb += 16) {
          FeatFrag<E, D> kt[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) kt[u].load(kp + rows.frame(kb, u, last), col);
          const f32x4 s = row_product(kr, qf), dpv = row_product(vr, df);
          if (kb + 16 <= whi) load_rows(kb + 16);
          float ds[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float pw = fast_exp2(__builtin_fmaf(s[u], c2, -l2));
            ds[u] = win.has(kb + 4 * g + u) ? pw * (dpv[u] - dn) : 0.f;
          }
          col_product(kt, ds, acc0);
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

hipError_t launch_bwd(BwdDev a, int d, hipStream_t stream) {
  set_items(a, d, kTileRows);
  const dim3 grid(a.items < kMaxGrid ? a.items : kMaxGrid), block(kThreads);
  if (d == 64)
    hipLaunchKernelGGL(band_bwd_f32_kernel<64>, grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL(band_bwd_f32_kernel<32>, grid, block, 0, stream, a);
  return hipGetLastError();
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
  return launch_bwd(sa_args(x), x.d, stream);
}

hipError_t launch_llsa_backward_f32(const LlsaBackwardArgs& x, hipStream_t stream) {
  return launch_bwd(llsa_args(x), x.d, stream);
}

hipError_t launch_llsa_paper_backward_f32(const LlsaPaperBwdArgs& x, hipStream_t stream) {
  return launch_bwd(paper_args(x), x.d, stream);
}

}  // namespace sa
