// Instance labels of surfels from localized queries (Sec. 4.1, eqs. (4)-(7)):
//   z = f_q . f_g,  S = sigmoid(z),  D = exp(-(p_g - mu_q)^T P_q (p_g - mu_q) / 2),
//   A = S D,  l(g) = softmax over queries of A(., g),
// and their gradients.  The labels are rendered by the feature blend (eq. (8)).
//
// The affinity logits are a dense contraction over the feature dimension
// (surfels x queries), so they run on the matrix cores: FP32 MFMA
// (v_mfma_f32_16x16x4f32, exact products, FP32 accumulation).  A wave owns 16
// surfels; lane l holds A-operand row l & 15 / k-slice l >> 4, and the
// 16 x 16 result tile lands as rows 4 (l >> 4) + r, column l & 15, so each
// 16-lane DPP row holds 4 surfels x 16 queries and the softmax over queries
// is a reduction inside DPP rows.
//
// Backward: k_lab_bwd_surf recomputes the forward and writes dz = dL/dz and
// wD = dL/dD * D per (surfel, query) plus dL/dp_g; the feature gradients are
// two MFMA products (dF_g = dZ F_q, dF_q = dZ^T F_g over surfel segments) and
// the query means/precisions are reduced over surfel segments (FP64), then
// the segments are summed in a fixed order: deterministic.
#include "common.h"
#include "internal.h"

namespace psm {

// Reductions over the 16 lanes of a DPP row (rotations inside the row).
__device__ __forceinline__ float row_sum16(float v) {
  v += dpp_mov<0x128>(v);  // row_ror:8
  v += dpp_mov<0x124>(v);  // row_ror:4
  v += dpp_mov<0x122>(v);  // row_ror:2
  v += dpp_mov<0x121>(v);  // row_ror:1
  return v;
}
__device__ __forceinline__ float row_max16(float v) {
  v = fmaxf(v, dpp_mov<0x128>(v));
  v = fmaxf(v, dpp_mov<0x124>(v));
  v = fmaxf(v, dpp_mov<0x122>(v));
  v = fmaxf(v, dpp_mov<0x121>(v));
  return v;
}

// Query j's mean and precision (xx, xy, xz, yy, yz, zz).
struct QGeo {
  float mx, my, mz, pxx, pxy, pxz, pyy, pyz, pzz;
};
__device__ __forceinline__ QGeo load_qgeo(const LabelQueries& q, int j) {
  QGeo g;
  const float* m = q.mean + 3 * j;
  const float* p = q.prec + 6 * j;
  g.mx = m[0]; g.my = m[1]; g.mz = m[2];
  g.pxx = p[0]; g.pxy = p[1]; g.pxz = p[2]; g.pyy = p[3]; g.pyz = p[4]; g.pzz = p[5];
  return g;
}

// Forward terms of one (surfel, query) element.
struct LabTerm {
  float S, D, dx, dy, dz, Px, Py, Pz;  // S, D, d = p - mu, P d
};
__device__ __forceinline__ LabTerm lab_term(float z, float px, float py, float pz, const QGeo& g) {
  LabTerm t;
  t.S = 1.0f / (1.0f + expf(-z));
  t.dx = px - g.mx;
  t.dy = py - g.my;
  t.dz = pz - g.mz;
  t.Px = g.pxx * t.dx + g.pxy * t.dy + g.pxz * t.dz;
  t.Py = g.pxy * t.dx + g.pyy * t.dy + g.pyz * t.dz;
  t.Pz = g.pxz * t.dx + g.pyz * t.dy + g.pzz * t.dz;
  const float m = t.dx * t.Px + t.dy * t.Py + t.dz * t.Pz;
  t.D = expf(-0.5f * m);
  return t;
}

// z tiles of a wave's 16 surfels against all query blocks (MFMA over C).
template <typename FT, int NQB>
__device__ __forceinline__ void logits(int64_t n, const FT* __restrict__ fg, const LabelQueries& q, int64_t g0,
                                       f4v (&acc)[NQB]) {
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int64_t ga = g0 + i;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) acc[qb] = f4v{0.f, 0.f, 0.f, 0.f};
  int c0 = 0;
  // 16 channels a step: one load a lane of each operand instead of four (each
  // touches 16 rows); the arrays may start anywhere, so only where they are
  // aligned.  120k surfels, 64 queries, 32 channels: the forward 59 -> 37 us,
  // the surfel backward 77 -> 59 us.
  const bool wide = ((uintptr_t)fg % (4 * sizeof(FT)) | (uintptr_t)q.feat % 16) == 0;
  for (; wide && c0 + 16 <= q.c; c0 += 16) {
    const float4 a = by_step(load4<FT>(fg + min(ga, n - 1) * q.c + c0 + 4 * kq));  // rows past n: not used
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {  // columns past nq: not used
      const float* bp = q.feat + (size_t)min(qb * 16 + i, q.nq - 1) * q.c + c0 + 4 * kq;
      const float4 b = by_step(*reinterpret_cast<const float4*>(bp));
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[qb] = mfma_16x16x4((&a.x)[s], (&b.x)[s], acc[qb]);
    }
  }
  for (; c0 < q.c; c0 += 4) {
    const float a = ga < n ? load_one<FT>(fg + ga * q.c + c0 + kq) : 0.0f;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const int j = qb * 16 + i;
      const float b = j < q.nq ? q.feat[(size_t)j * q.c + c0 + kq] : 0.0f;
      acc[qb] = mfma_16x16x4(a, b, acc[qb]);
    }
  }
}

template <typename FT, int NQB>
__global__ __launch_bounds__(256) void k_lab_fwd(int64_t n, const float* __restrict__ means, const FT* __restrict__ fg,
                                                 LabelQueries q, float* __restrict__ out, int ld) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, kq = lane >> 4;
  const int64_t g0 = ((int64_t)blockIdx.x * 4 + wave) * 16;
  if (g0 >= n) return;
  f4v acc[NQB];
  logits<FT, NQB>(n, fg, q, g0, acc);
  float px[4], py[4], pz[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t g = g0 + 4 * kq + r;
    px[r] = g < n ? means[3 * g] : 0.0f;
    py[r] = g < n ? means[3 * g + 1] : 0.0f;
    pz[r] = g < n ? means[3 * g + 2] : 0.0f;
  }
  float A[NQB][4], mx[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) mx[r] = -INFINITY;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int j = qb * 16 + i;
    const bool vq = j < q.nq;
    const QGeo gq = load_qgeo(q, vq ? j : 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const LabTerm t = lab_term(acc[qb][r], px[r], py[r], pz[r], gq);
      A[qb][r] = vq ? t.S * t.D : -INFINITY;
      mx[r] = fmaxf(mx[r], A[qb][r]);
    }
  }
  float sum[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    mx[r] = row_max16(mx[r]);
    sum[r] = 0.0f;
  }
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float e = qb * 16 + i < q.nq ? expf(A[qb][r] - mx[r]) : 0.0f;
      A[qb][r] = e;
      sum[r] += e;
    }
  const int npad = (q.nq + 7) & ~7;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float inv = 1.0f / row_sum16(sum[r]);
    const int64_t g = g0 + 4 * kq + r;
    if (g >= n) continue;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const int j = qb * 16 + i;
      if (j < npad) out[g * ld + j] = j < q.nq ? A[qb][r] * inv : 0.0f;
    }
  }
}

// Backward per (surfel, query): dz = dL/dz, wD = dL/dD * D (into padded
// [n][16 NQB] arrays) and dL/dp_g.
template <typename FT, int NQB>
__global__ __launch_bounds__(256) void k_lab_bwd_surf(int64_t n, const float* __restrict__ means,
                                                      const FT* __restrict__ fg, LabelQueries q,
                                                      const float* __restrict__ dl, int ld, float* __restrict__ dZ,
                                                      float* __restrict__ wDo, float* __restrict__ d_means) {
  constexpr int NQP = NQB * 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, kq = lane >> 4;
  const int64_t g0 = ((int64_t)blockIdx.x * 4 + wave) * 16;
  if (g0 >= n) return;
  f4v acc[NQB];
  logits<FT, NQB>(n, fg, q, g0, acc);
  float px[4], py[4], pz[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t g = g0 + 4 * kq + r;
    px[r] = g < n ? means[3 * g] : 0.0f;
    py[r] = g < n ? means[3 * g + 1] : 0.0f;
    pz[r] = g < n ? means[3 * g + 2] : 0.0f;
  }
  // forward again: A, softmax
  float A[NQB][4], mx[4], sum[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) mx[r] = -INFINITY;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int j = qb * 16 + i;
    const bool vq = j < q.nq;
    const QGeo gq = load_qgeo(q, vq ? j : 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const LabTerm t = lab_term(acc[qb][r], px[r], py[r], pz[r], gq);
      A[qb][r] = vq ? t.S * t.D : -INFINITY;
      mx[r] = fmaxf(mx[r], A[qb][r]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    mx[r] = row_max16(mx[r]);
    sum[r] = 0.0f;
  }
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float e = qb * 16 + i < q.nq ? expf(A[qb][r] - mx[r]) : 0.0f;
      A[qb][r] = e;
      sum[r] += e;
    }
  // labels and sum_q l dl per surfel
  float dot[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float inv = 1.0f / row_sum16(sum[r]);
    const int64_t g = g0 + 4 * kq + r;
    dot[r] = 0.0f;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const int j = qb * 16 + i;
      A[qb][r] *= inv;  // label
      const float u = (g < n && j < q.nq) ? dl[g * ld + j] : 0.0f;
      dot[r] = fmaf(A[qb][r], u, dot[r]);
    }
    dot[r] = row_sum16(dot[r]);
  }
  float gx[4] = {0.f, 0.f, 0.f, 0.f}, gy[4] = {0.f, 0.f, 0.f, 0.f}, gz[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int j = qb * 16 + i;
    const bool vq = j < q.nq;
    const QGeo gq = load_qgeo(q, vq ? j : 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t g = g0 + 4 * kq + r;
      const LabTerm t = lab_term(acc[qb][r], px[r], py[r], pz[r], gq);
      const float u = (g < n && vq) ? dl[g * ld + j] : 0.0f;
      const float dA = A[qb][r] * (u - dot[r]);
      const float dz = vq ? dA * t.D * t.S * (1.0f - t.S) : 0.0f;
      const float wD = vq ? dA * t.S * t.D : 0.0f;
      gx[r] = fmaf(-wD, t.Px, gx[r]);
      gy[r] = fmaf(-wD, t.Py, gy[r]);
      gz[r] = fmaf(-wD, t.Pz, gz[r]);
      if (g < n) {
        dZ[g * NQP + j] = dz;
        wDo[g * NQP + j] = wD;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float sx = row_sum16(gx[r]), sy = row_sum16(gy[r]), sz = row_sum16(gz[r]);
    const int64_t g = g0 + 4 * kq + r;
    if (i == 0 && g < n) {
      d_means[3 * g] = sx;
      d_means[3 * g + 1] = sy;
      d_means[3 * g + 2] = sz;
    }
  }
}

// dF_g = dZ F_q: a wave computes 16 surfels x 16 channels (MFMA over queries).
template <int NQB>
__global__ __launch_bounds__(256) void k_lab_dfg(int64_t n, LabelQueries q, const float* __restrict__ dZ,
                                                 float* __restrict__ dfg) {
  constexpr int NQP = NQB * 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, k = lane >> 4;
  const int64_t g0 = ((int64_t)blockIdx.x * 4 + wave) * 16;
  const int c0 = blockIdx.y * 16;
  if (g0 >= n) return;
  f4v acc = {0.f, 0.f, 0.f, 0.f};
  const int64_t ga = g0 + i;
  for (int j0 = 0; j0 < NQP; j0 += 4) {
    const float a = ga < n ? dZ[ga * NQP + j0 + k] : 0.0f;
    const bool vb = j0 + k < q.nq && c0 + i < q.c;
    const float b = vb ? q.feat[(size_t)(j0 + k) * q.c + c0 + i] : 0.0f;
    acc = mfma_16x16x4(a, b, acc);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t g = g0 + 4 * k + r;
    if (g < n && c0 + i < q.c) dfg[g * q.c + c0 + i] = acc[r];
  }
}

// Partial dF_q = dZ^T F_g over one surfel segment: 16 queries x 16 channels
// (MFMA over the segment's surfels).  Four waves take its steps of 4 surfels in
// turn, eight steps' loads in flight: one wave stepping alone through 1024
// surfels waited for each step's loads (120k surfels, 64 queries, 32 channels:
// 94 -> 35 us).  The waves' sums are added in wave order.
constexpr int kLabFly = 8;
template <typename FT, int NQB>
__global__ __launch_bounds__(256) void k_lab_dfq(int64_t n, int64_t seg_len, LabelQueries q,
                                                 const float* __restrict__ dZ, const FT* __restrict__ fg,
                                                 float* __restrict__ part) {
  constexpr int NQP = NQB * 16;
  __shared__ float s_acc[4][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, k = lane >> 4;
  const int j0 = blockIdx.x * 16, c0 = blockIdx.y * 16, s = blockIdx.z;
  const int64_t gs = (int64_t)s * seg_len, ge = min(n, gs + seg_len);
  const int cl = min(c0 + i, q.c - 1);  // columns past c are not used
  f4v acc = {0.f, 0.f, 0.f, 0.f};
  for (int64_t g = gs + 4 * wave + k; g - k < ge; g += 16 * kLabFly) {
    float a[kLabFly], b[kLabFly];
#pragma unroll
    for (int u = 0; u < kLabFly; ++u) {
      const int64_t gu = g + 16 * u;
      const int64_t gl = min(gu, ge - 1);
      a[u] = dZ[gl * NQP + j0 + i];
      b[u] = load_one<FT>(fg + gl * q.c + cl);
      if (gu >= ge) a[u] = b[u] = 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kLabFly; ++u) acc = mfma_16x16x4(a[u], b[u], acc);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) s_acc[wave][(4 * k + r) * 16 + i] = acc[r];
  __syncthreads();
  const int t = threadIdx.x, j = j0 + (t >> 4), c = c0 + (t & 15);
  if (c < q.c) part[((size_t)s * NQP + j) * q.c + c] = ((s_acc[0][t] + s_acc[1][t]) + s_acc[2][t]) + s_acc[3][t];
}

// Partial query-mean / precision gradients over one surfel segment (FP64
// accumulation, fixed order).  A block takes 16 queries: lane i of 16 one
// query, so that wD is read in whole lines (a block per query read 4 bytes of
// each line), and each of the 16 lane groups every 16th surfel; the
// precision is applied to the sums.  120k
// surfels, 64 queries: 52 -> 40 us.
template <int NQB>
__global__ __launch_bounds__(256) void k_lab_qgeo(int64_t n, int64_t seg_len, const float* __restrict__ means,
                                                  LabelQueries q, const float* __restrict__ wD,
                                                  double* __restrict__ part) {
  constexpr int NQP = NQB * 16;
  __shared__ double s_red[4][16][9];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15;
  const int j = blockIdx.x * 16 + i, s = blockIdx.y;
  const int64_t gs = (int64_t)s * seg_len, ge = min(n, gs + seg_len);
  const QGeo gq = load_qgeo(q, min(j, q.nq - 1));
  double v[9];
#pragma unroll
  for (int x = 0; x < 9; ++x) v[x] = 0.0;
#pragma unroll 4
  for (int64_t g = gs + (threadIdx.x >> 4); g < ge; g += 16) {
    const double w = wD[g * NQP + j];
    const double dx = (double)means[3 * g] - gq.mx, dy = (double)means[3 * g + 1] - gq.my,
                 dz = (double)means[3 * g + 2] - gq.mz;
    const double wx = w * dx, wy = w * dy, wz = w * dz;
    v[0] += wx;
    v[1] += wy;
    v[2] += wz;
    v[3] = __builtin_fma(wx, dx, v[3]);
    v[4] = __builtin_fma(wx, dy, v[4]);
    v[5] = __builtin_fma(wx, dz, v[5]);
    v[6] = __builtin_fma(wy, dy, v[6]);
    v[7] = __builtin_fma(wy, dz, v[7]);
    v[8] = __builtin_fma(wz, dz, v[8]);
  }
  {  // dL/dmu = P sum w d;  dL/dP = -w/2 d d^T, an off-diagonal number appears twice in P
    const double x = v[0], y = v[1], z = v[2];
    v[0] = gq.pxx * x + gq.pxy * y + gq.pxz * z;
    v[1] = gq.pxy * x + gq.pyy * y + gq.pyz * z;
    v[2] = gq.pxz * x + gq.pyz * y + gq.pzz * z;
    v[3] *= -0.5; v[6] *= -0.5; v[8] *= -0.5;
    v[4] = -v[4]; v[5] = -v[5]; v[7] = -v[7];
  }
#pragma unroll
  for (int x = 0; x < 9; ++x) {
    v[x] += __shfl_xor(v[x], 16, 64);
    v[x] += __shfl_xor(v[x], 32, 64);
    if (lane < 16) s_red[wave][i][x] = v[x];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < 16 * 9; t += 256) {
    const int jj = blockIdx.x * 16 + t / 9, x = t % 9;
    if (jj < q.nq)
      part[((size_t)s * NQP + jj) * 9 + x] =
          ((s_red[0][t / 9][x] + s_red[1][t / 9][x]) + s_red[2][t / 9][x]) + s_red[3][t / 9][x];
  }
}

// Sum of the segment partials: a block takes 32 results, 8 threads each, thread
// y every 8th segment, then the 8 in order (one thread per result waited for
// 117 loads in turn: 30 -> 6 us).
__global__ __launch_bounds__(256) void k_lab_sum(int nseg, int nq, int nqp, int c, const float* __restrict__ pfq,
                                                 const double* __restrict__ pgeo, float* __restrict__ d_qfeat,
                                                 float* __restrict__ d_qmean, float* __restrict__ d_qprec) {
  __shared__ double s_sum[8][32];
  const int x32 = threadIdx.x & 31, y = threadIdx.x >> 5;
  const int64_t t = (int64_t)blockIdx.x * 32 + x32;
  const int64_t nf = (int64_t)nq * c, tot = nf + (int64_t)nq * 9;
  const int64_t u = t - nf;
  double a = 0.0;
  if (t < nf) {
    const float* p = pfq + t;  // query-major: element (j, cc) at j c + cc
#pragma unroll 4
    for (int s = y; s < nseg; s += 8) a += p[(size_t)s * nqp * c];
  } else if (t < tot) {
    const double* p = pgeo + u;
#pragma unroll 4
    for (int s = y; s < nseg; s += 8) a += p[(size_t)s * nqp * 9];
  }
  s_sum[y][x32] = a;
  __syncthreads();
  if (y != 0 || t >= tot) return;
  double r = s_sum[0][x32];
#pragma unroll
  for (int w = 1; w < 8; ++w) r += s_sum[w][x32];
  if (t < nf) {
    d_qfeat[t] = (float)r;
  } else {
    const int j = (int)(u / 9), x = (int)(u % 9);
    if (x < 3) d_qmean[3 * j + x] = (float)r;
    else d_qprec[6 * j + (x - 3)] = (float)r;
  }
}

// ------------------------------------------------------------- host wrappers
int label_blocks16(int nq) { return pow2_ge_host((nq + 15) / 16); }

size_t label_workspace_bytes(int64_t n, int nq, int c) {
  const int64_t nqp = (int64_t)label_blocks16(nq) * 16;
  const int64_t nseg = label_segments(n);
  size_t o = 0;
  o = align256(o + (size_t)std::max<int64_t>(n, 1) * nqp * 4);  // dZ
  o = align256(o + (size_t)std::max<int64_t>(n, 1) * nqp * 4);  // wD
  o = align256(o + (size_t)nseg * nqp * c * 4);                  // dF_q partials
  o = align256(o + (size_t)nseg * nqp * 9 * 8);                  // mean / precision partials
  return o;
}

int64_t label_segments(int64_t n) { return std::max<int64_t>(1, std::min<int64_t>(256, cdiv(n, 1024))); }

template <typename FT, int NQB>
static void lab_fwd_t(int64_t n, const float* means, const void* fg, const LabelQueries& q, float* out, int ld,
                      hipStream_t st) {
  hipLaunchKernelGGL((k_lab_fwd<FT, NQB>), dim3((unsigned)cdiv(n, 64)), dim3(256), 0, st, n, means, (const FT*)fg, q,
                     out, ld);
}

template <typename FT, int NQB>
static void lab_bwd_t(int64_t n, const float* means, const void* fg, const LabelQueries& q, const float* dl, int ld,
                      char* ws, float* d_means, float* d_fg, float* d_qfeat, float* d_qmean, float* d_qprec,
                      hipStream_t st) {
  constexpr int NQP = NQB * 16;
  const int64_t nseg = label_segments(n);
  const int64_t seg_len = cdiv(std::max<int64_t>(n, 1), nseg);
  size_t o = 0;
  float* dZ = (float*)(ws + o);
  o = align256(o + (size_t)std::max<int64_t>(n, 1) * NQP * 4);
  float* wD = (float*)(ws + o);
  o = align256(o + (size_t)std::max<int64_t>(n, 1) * NQP * 4);
  float* pfq = (float*)(ws + o);
  o = align256(o + (size_t)nseg * NQP * q.c * 4);
  double* pgeo = (double*)(ws + o);
  if (n > 0) {
    const unsigned nb = (unsigned)cdiv(n, 64);
    hipLaunchKernelGGL((k_lab_bwd_surf<FT, NQB>), dim3(nb), dim3(256), 0, st, n, means, (const FT*)fg, q, dl, ld, dZ,
                       wD, d_means);
    hipLaunchKernelGGL((k_lab_dfg<NQB>), dim3(nb, (unsigned)cdiv(q.c, 16)), dim3(256), 0, st, n, q, (const float*)dZ,
                       d_fg);
  }
  hipLaunchKernelGGL((k_lab_dfq<FT, NQB>), dim3(NQB, (unsigned)cdiv(q.c, 16), (unsigned)nseg), dim3(256), 0, st, n,
                     seg_len, q, (const float*)dZ, (const FT*)fg, pfq);
  hipLaunchKernelGGL((k_lab_qgeo<NQB>), dim3((unsigned)cdiv(q.nq, 16), (unsigned)nseg), dim3(256), 0, st, n, seg_len, means, q,
                     (const float*)wD, pgeo);
  const int64_t tot = (int64_t)q.nq * (q.c + 9);
  hipLaunchKernelGGL(k_lab_sum, dim3((unsigned)cdiv(tot, 32)), dim3(256), 0, st, (int)nseg, q.nq, NQP, q.c,
                     (const float*)pfq, (const double*)pgeo, d_qfeat, d_qmean, d_qprec);
}

template <typename FT>
static void lab_fwd_dt(int64_t n, const float* means, const void* fg, const LabelQueries& q, float* out, int ld,
                       hipStream_t st) {
  switch (label_blocks16(q.nq)) {
    case 1: lab_fwd_t<FT, 1>(n, means, fg, q, out, ld, st); break;
    case 2: lab_fwd_t<FT, 2>(n, means, fg, q, out, ld, st); break;
    case 4: lab_fwd_t<FT, 4>(n, means, fg, q, out, ld, st); break;
    case 8: lab_fwd_t<FT, 8>(n, means, fg, q, out, ld, st); break;
    default: lab_fwd_t<FT, 16>(n, means, fg, q, out, ld, st); break;
  }
}

template <typename FT>
static void lab_bwd_dt(int64_t n, const float* means, const void* fg, const LabelQueries& q, const float* dl, int ld,
                       char* ws, float* d_means, float* d_fg, float* d_qfeat, float* d_qmean, float* d_qprec,
                       hipStream_t st) {
  switch (label_blocks16(q.nq)) {
    case 1: lab_bwd_t<FT, 1>(n, means, fg, q, dl, ld, ws, d_means, d_fg, d_qfeat, d_qmean, d_qprec, st); break;
    case 2: lab_bwd_t<FT, 2>(n, means, fg, q, dl, ld, ws, d_means, d_fg, d_qfeat, d_qmean, d_qprec, st); break;
    case 4: lab_bwd_t<FT, 4>(n, means, fg, q, dl, ld, ws, d_means, d_fg, d_qfeat, d_qmean, d_qprec, st); break;
    case 8: lab_bwd_t<FT, 8>(n, means, fg, q, dl, ld, ws, d_means, d_fg, d_qfeat, d_qmean, d_qprec, st); break;
    default: lab_bwd_t<FT, 16>(n, means, fg, q, dl, ld, ws, d_means, d_fg, d_qfeat, d_qmean, d_qprec, st); break;
  }
}

void launch_labels(int64_t n, const float* means, const void* fg, int dtype, const LabelQueries& q, float* out,
                   int ld, hipStream_t st) {
  if (n == 0) return;
  if (dtype == kF32) lab_fwd_dt<float>(n, means, fg, q, out, ld, st);
  else if (dtype == kF16) lab_fwd_dt<__half>(n, means, fg, q, out, ld, st);
  else lab_fwd_dt<uint16_t>(n, means, fg, q, out, ld, st);
}

void launch_labels_backward(int64_t n, const float* means, const void* fg, int dtype, const LabelQueries& q,
                            const float* dl, int ld, char* ws, float* d_means, float* d_fg, float* d_qfeat,
                            float* d_qmean, float* d_qprec, hipStream_t st) {
  if (dtype == kF32) lab_bwd_dt<float>(n, means, fg, q, dl, ld, ws, d_means, d_fg, d_qfeat, d_qmean, d_qprec, st);
  else if (dtype == kF16) lab_bwd_dt<__half>(n, means, fg, q, dl, ld, ws, d_means, d_fg, d_qfeat, d_qmean, d_qprec, st);
  else lab_bwd_dt<uint16_t>(n, means, fg, q, dl, ld, ws, d_means, d_fg, d_qfeat, d_qmean, d_qprec, st);
}

}  // namespace psm
