// SOGMM geometric loss of surfels (Sec. 3.2 eq. (3), Sec. 4.2 eq. (13) and
// the anisotropy term):
//   component k of the plane prior: weight pi_k, mean mu_k, covariance
//     Sigma_k, reference normal n_k = eigenvector of Sigma_k's smallest
//     eigenvalue;
//   surfel i takes the component of largest posterior pi_k N(mu_i; mu_k,
//     Sigma_k): the smallest score (x - mu_k)^T Sigma_k^-1 (x - mu_k) +
//     ln det Sigma_k - 2 ln pi_k, evaluated in FP32 in a prescribed order
//     (ties to the lower index);
//   L_geo = sum_i |(mu_i - mu_k) . n_k| + lambda_n (1 - |n_i . n_k|),
//   L_iso = sum_i (s_i1 - s_i2)^2,
// and the gradients with the assignment held fixed.
//
// k_gmm_prep: thread per component (FP64): precision by the adjugate, the
//   score constant, the reference normal by cyclic Jacobi sweeps; an FP32
//   record of 16 floats, and the component's share of the bound's operands.
// k_geo_loss: the minimum over the components, without scoring most of them.
//   A lower bound of every score comes from the matrix cores; only components
//   whose bound does not exceed the best exact score are scored, in the
//   prescribed order, so the assignment is bit for bit the full scan's.
//   Bound (y = x - c0, m = mu - c0, c0 = the mean of the components'; eigenpairs
//   l1 >= l2 >= l3, v1..v3 of the precision): the score is at least
//     a |y - m|^2 + b1 (v1.(y-m))^2 + b2 (v2.(y-m))^2 + c - margins,
//   a = l3, b_i = l_i - l3: one product linear in (y, |y|^2, 1) and two in
//   (y, 1).  Each is a 32-long bf16 MFMA row: y, |y|^2 and the coefficients
//   split into three bf16 parts, all cross terms down to 2^-24 kept.
//   Margins, all folded into the coefficients: the products' error, taken as
//   kEps = 2^-17 of the sum of |terms| (32 FP32 additions and the dropped
//   terms stay under 2^-17.5); a squared product loses at most
//   (1 + 1/kTheta) of its squared error beyond a share kTheta; and the FP32
//   score's own rounding, under 2^-19 l1 |x - mu|^2 + 2^-20 |c|.
//   A component out of the ranges that this assumes gets a bound below every
//   score, a surfel out of them the full scan.
//   One plain scan of 512 components is 27 vector instructions for 64 pairs;
//   the bound is 3.25 and 3 MFMA for 256.
//   1M surfels, 512 components: 345 us the scan, 129 us this (prep 17 and 10,
//   the sums 16 and 4).  The loop is bound by issue (64 vector and 12 matrix
//   instructions a tile of 1024 pairs), about half of the time; the rest is
//   the split, the exact scores and the FP64 loss terms, once a surfel.
// k_geo_sum: the blocks' FP64 sums, in a fixed order.
#include "common.h"
#include "internal.h"

namespace psm {

constexpr int kGmmRec = 16;     // floats per component record
constexpr int kGmmTile = 16;    // components per MFMA tile
constexpr int kGmmTileBytes = 3 * 64 * 16;  // its three operands, 16 bytes a lane
constexpr int kGmmChunk = 16;   // tiles staged per chunk (48 KB)
constexpr int kGeoThreads = 512;
constexpr double kEps = 1.0 / 131072, kTheta = 1.0 / 256;
constexpr float kGmmFar = 1e30f;   // bound of a component that cannot win
constexpr float kGmmSpan = 1e9f;   // largest coordinate that the margins cover

typedef __bf16 Bf8 __attribute__((ext_vector_type(8)));
typedef float F4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned bf16_bits(float v) {  // finite v, to nearest even
  const unsigned b = __float_as_uint(v);
  return (b + 0x7fffu + ((b >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ float bf16_value(unsigned h) { return __uint_as_float(h << 16); }

// v in three bf16 parts; what is left is under 2^-25 |v|
struct Split {
  unsigned h, m, l;
};
__device__ __forceinline__ Split split3(double v) {
  Split s;
  s.h = bf16_bits((float)v);
  v -= (double)bf16_value(s.h);
  s.m = bf16_bits((float)v);
  v -= (double)bf16_value(s.m);
  s.l = bf16_bits((float)v);
  return s;
}
__device__ __forceinline__ Split split3(float v) {  // the differences are exact
  Split s;
  s.h = bf16_bits(v);
  v -= bf16_value(s.h);
  s.m = bf16_bits(v);
  v -= bf16_value(s.m);
  s.l = bf16_bits(v);
  return s;
}

// One component's row of an operand: coefficients u of (y, |y|^2), constant c.
// The 32 products, eight to a group of 16 lanes, against the surfel's
// [yh yh] [ym ym] [yh yl] [1 1 1 0 ym].
__device__ __forceinline__ void store_row(uint4* op, int row, const double u[4], double c) {
  Split s[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i] = split3(u[i]);
  const Split k = split3(c);
  const uint2 H = {s[0].h | s[1].h << 16, s[2].h | s[3].h << 16};
  const uint2 M = {s[0].m | s[1].m << 16, s[2].m | s[3].m << 16};
  const uint2 L = {s[0].l | s[1].l << 16, s[2].l | s[3].l << 16};
  op[row] = uint4{H.x, H.y, M.x, M.y};
  op[16 + row] = uint4{H.x, H.y, M.x, M.y};
  op[32 + row] = uint4{L.x, L.y, H.x, H.y};
  op[48 + row] = uint4{k.h | k.m << 16, k.l, L.x, L.y};
}

// Origin of the bound's coordinates: the mean of up to 512 of the component
// means, the same in every block; the margins grow with the distance to it.
__device__ __forceinline__ void bound_origin(int k, const float* __restrict__ mean, float c[3]) {
  float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  const int step = (k + 511) / 512;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int j = step * (64 * i + (int)threadIdx.x);
    const float* m = mean + 3 * (size_t)min(j, k - 1);
    const float x = m[0], y = m[1], z = m[2];
    const bool in = j < k && fabsf(x) <= kGmmSpan && fabsf(y) <= kGmmSpan && fabsf(z) <= kGmmSpan;
    s[0] += in ? x : 0.0f;
    s[1] += in ? y : 0.0f;
    s[2] += in ? z : 0.0f;
    s[3] += in ? 1.0f : 0.0f;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s[i] += __shfl_xor(s[i], o, 64);
  for (int i = 0; i < 3; ++i) c[i] = s[i] / fmaxf(s[3], 1.0f);
}

// record: mean (3), precision xx xy xz yy yz zz (6), constant (1), normal (3),
// the bound's origin (3)
__global__ __launch_bounds__(64) void k_gmm_prep(int k, const float* __restrict__ mean, const float* __restrict__ cov,
                           const float* __restrict__ weight, float* __restrict__ rec, uint4* __restrict__ ops) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  float org[3];
  bound_origin(k, mean, org);
  uint4* op = ops + (size_t)(j / kGmmTile) * (kGmmTileBytes / 16);
  const int row = j % kGmmTile;
  const double zero[4] = {0.0, 0.0, 0.0, 0.0};
  if (j >= k) {
    if (j < (k + kGmmTile - 1) / kGmmTile * kGmmTile) {  // rest of the last tile
      store_row(op, row, zero, kGmmFar);
      store_row(op + 64, row, zero, 0.0);
      store_row(op + 128, row, zero, 0.0);
    }
    return;
  }
  double a[3][3];
  const float* c = cov + 6 * (size_t)j;
  a[0][0] = c[0]; a[0][1] = a[1][0] = c[1]; a[0][2] = a[2][0] = c[2];
  a[1][1] = c[3]; a[1][2] = a[2][1] = c[4]; a[2][2] = c[5];
  // precision = adjugate / det
  const double A00 = a[1][1] * a[2][2] - a[1][2] * a[2][1];
  const double A01 = a[0][2] * a[2][1] - a[0][1] * a[2][2];
  const double A02 = a[0][1] * a[1][2] - a[0][2] * a[1][1];
  const double A11 = a[0][0] * a[2][2] - a[0][2] * a[2][0];
  const double A12 = a[0][2] * a[1][0] - a[0][0] * a[1][2];
  const double A22 = a[0][0] * a[1][1] - a[0][1] * a[1][0];
  const double det = a[0][0] * A00 + a[0][1] * (a[1][2] * a[2][0] - a[1][0] * a[2][2]) + a[0][2] * (a[1][0] * a[2][1] - a[1][1] * a[2][0]);
  const double id = 1.0 / det;
  float* r = rec + (size_t)kGmmRec * j;
  r[0] = mean[3 * (size_t)j];
  r[1] = mean[3 * (size_t)j + 1];
  r[2] = mean[3 * (size_t)j + 2];
  r[3] = (float)(A00 * id);
  r[4] = (float)(A01 * id);
  r[5] = (float)(A02 * id);
  r[6] = (float)(A11 * id);
  r[7] = (float)(A12 * id);
  r[8] = (float)(A22 * id);
  r[9] = (float)(log(det) - 2.0 * log((double)weight[j]));
  // cyclic Jacobi: a -> V^T a V diagonal; the column of V at the smallest
  // diagonal entry is the reference normal
  double V[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
  // an entry below the last bit of both its diagonal entries is zero; a
  // sweep without rotations ends it (4 or 5 of them)
  bool turned = true;
  for (int sweep = 0; sweep < 12 && turned; ++sweep) {
    turned = false;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = p + 1; q < 3; ++q) {
        const double apq = a[p][q];
        if (apq == 0.0) continue;
        if (fabs(apq) <= 1e-17 * fmin(fabs(a[p][p]), fabs(a[q][q]))) {
          a[p][q] = a[q][p] = 0.0;
          continue;
        }
        turned = true;
        const double theta = (a[q][q] - a[p][p]) / (2.0 * apq);
        const double t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
        const double cs = 1.0 / sqrt(t * t + 1.0), sn = t * cs;
        for (int m = 0; m < 3; ++m) {  // columns p, q of a
          const double amp = a[m][p], amq = a[m][q];
          a[m][p] = cs * amp - sn * amq;
          a[m][q] = sn * amp + cs * amq;
        }
        for (int m = 0; m < 3; ++m) {  // rows p, q of a
          const double apm = a[p][m], aqm = a[q][m];
          a[p][m] = cs * apm - sn * aqm;
          a[q][m] = sn * apm + cs * aqm;
        }
        for (int m = 0; m < 3; ++m) {
          const double vmp = V[m][p], vmq = V[m][q];
          V[m][p] = cs * vmp - sn * vmq;
          V[m][q] = sn * vmp + cs * vmq;
        }
      }
  }
  const double g0 = a[0][0], g1 = a[1][1], g2 = a[2][2];
  int im = 0;
  if (g1 < g0) im = 1;
  if (g2 < (im ? g1 : g0)) im = 2;
  const int ia = im == 0 ? 1 : 0, ib = im == 2 ? 1 : 2;  // the other two
  const int iw = (ib == 2 ? g2 : g1) > (ia == 1 ? g1 : g0) ? ib : ia, ic = ia + ib - iw;
  // constant indices only: V and a stay in registers
  double e1 = 0.0, e2 = 0.0, e3 = 0.0, v1[3] = {}, v2[3] = {};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (q == im) e1 = a[q][q];
    if (q == ic) e2 = a[q][q];
    if (q == iw) e3 = a[q][q];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      if (q == im) v1[m] = V[m][q];
      if (q == ic) v2[m] = V[m][q];
    }
  }
  r[10] = (float)v1[0];
  r[11] = (float)v1[1];
  r[12] = (float)v1[2];
  r[13] = org[0];
  r[14] = org[1];
  r[15] = org[2];

  // the bound's rows
  const double cst = (double)r[9];
  double m[3], mm = 0.0;
  bool safe = true;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const float mq = mean[3 * (size_t)j + q];
    safe = safe && fabsf(mq) <= kGmmSpan;
    m[q] = (double)mq - (double)org[q];
    mm += m[q] * m[q];
  }
  // the adjugate's FP64 rounding stays within the margins for e3^2 <= 1e12 e1 e2
  safe = safe && e1 >= 1e-16 && e3 <= 1e16 && e3 * e3 <= 1e12 * e1 * e2 && fabs(cst) <= 1e9;
  double u[4] = {}, w1[4] = {}, w2[4] = {}, cu = -(double)kGmmFar, c1 = 0.0, c2 = 0.0;
  if (!(cst < INFINITY)) cu = kGmmFar;  // score +inf or NaN: never taken
  if (safe) {
    const double l1 = 1.0 / e1, l2 = 1.0 / e2, l3 = 1.0 / e3;
    const double delta = l1 * (1.0 / 524288);
    const double b1 = fmax(l1 - l3, 0.0) * (1.0 - 2.0 * kTheta), b2 = fmax(l2 - l3, 0.0) * (1.0 - 2.0 * kTheta);
    const double aa = l3 * (1.0 - 2.0 * kTheta) - delta;
    const double my = 520.0 * kEps * kEps * (b1 + b2) + 4.0 * kEps * (l3 + delta);
    const double s1 = sqrt(b1), s2 = sqrt(b2);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      u[q] = -2.0 * aa * m[q];
      w1[q] = s1 * v1[q];
      w2[q] = s2 * v2[q];
      c1 -= w1[q] * m[q];
      c2 -= w2[q] * m[q];
    }
    u[3] = aa - my;
    cu = (aa - my) * mm + cst - 4.0 * kEps * fabs(cst) - 1e-20;
  }
  store_row(op, row, u, cu);
  store_row(op + 64, row, w1, c1);
  store_row(op + 128, row, w2, c2);
}

__device__ __forceinline__ double block_sum_f64(double v, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = red[0];
#pragma unroll
  for (int w = 1; w < kGeoThreads / 64; ++w) t += red[w];
  __syncthreads();
  return t;
}

// the score in the prescribed order
__device__ __forceinline__ float score(float x0, float x1, float x2, const float4& r0, const float4& r1,
                                       float r8, float r9) {
  const float d0 = x0 - r0.x, d1 = x1 - r0.y, d2 = x2 - r0.z;
  const float t0 = (r0.w * d0 + r1.x * d1) + r1.y * d2;
  const float t1 = (r1.x * d0 + r1.z * d1) + r1.w * d2;
  const float t2 = (r1.y * d0 + r1.w * d1) + r8 * d2;
  return ((d0 * t0 + d1 * t1) + d2 * t2) + r9;
}

// strict: of equal scores the lowest index stays; +inf and NaN never win
__device__ __forceinline__ void keep_lower(float s, int j, float& bs, int& bi) {
  const bool up = (s < bs) | ((s == bs) & (s < INFINITY) & (j < bi));
  bs = up ? s : bs;
  bi = up ? j : bi;
}

// Where bounds tell little (components much thinner than their distance from
// the origin times 2^-17, or surfels so many deviations away that the share
// kTheta of their scores exceeds the components' differences), a wave is
// better off scoring every component, a lane per surfel.  Seen twice: after an
// eighth of the components, by more than kGmmMany undecided lanes of its first
// kGmmProbe tiles (from 256 components on: below, the bounds cost less than
// the look); and by the number of lane groups left to score in the end, a scan
// of one being about 30 instructions per 256 components and 200 for its
// exchange, against 27 per component.  The whole call on 1M surfels, a fifth to
// a third of them off the planes, as plain scan / with bounds and scans of lane
// groups only / this, us: 60 m of planes, 512 components of 0.5 mm 352 / 410 /
// 340, 2000 of 2 mm 1134 / 2572 / 1234; a 100 m street 512 of 2 mm 354 / 417 /
// 325, of 0.5 mm 348 / 612 / 389, 2000 of 2 mm 1138 / 4267 / 1227; 3 cm (what
// bounds are for) 364 / 136 / 142.
constexpr int kGmmProbe = 2, kGmmMany = 4;
__device__ __forceinline__ int plain_scans(int k) { return (int)(27ll * k / (30 * ((k + 255) / 256) + 200)); }

// A wave takes 64 surfels in four column tiles: lane (g, c) of tile t sees
// surfel 16 t + c against components 4 g .. 4 g + 3 of each component tile.
// Per such quad the smallest bound is kept with the quad's number in its low
// bits (`low` accounts for them), the smallest two per lane.
__global__ __launch_bounds__(kGeoThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_geo_loss(
    int64_t n, const float* __restrict__ means, const float* __restrict__ scales, const float* __restrict__ quats,
    int k, const float* __restrict__ rec, const uint4* __restrict__ ops, float lambda_n, int32_t* __restrict__ assign,
    float* __restrict__ d_means, float* __restrict__ d_scales, float* __restrict__ d_quats,
    double* __restrict__ part) {
  __shared__ uint4 s_op[kGmmChunk * kGmmTileBytes / 16];
  __shared__ double s_red[kGeoThreads / 64];
  constexpr float kNone = 3e38f;
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool ok = i < n;
  const int tiles = (k + kGmmTile - 1) / kGmmTile;
  const int nbits = 32 - __clz(4 * tiles - 1);
  const unsigned idmask = (1u << nbits) - 1u, keep = ~idmask;
  const float slack = ldexpf(1.0f, nbits - 22);

  // each lane splits its own surfel; the tiles' columns are exchanged
  const float* xm = means + 3 * min(i, n - 1);
  const float x0 = n > 0 ? xm[0] : 0.f, x1 = n > 0 ? xm[1] : 0.f, x2 = n > 0 ? xm[2] : 0.f;
  bool wild;  // a surfel that the margins do not cover
  Bf8 pt[4];
  {
    float y0 = x0 - rec[13], y1 = x1 - rec[14], y2 = x2 - rec[15];
    wild = !(fabsf(y0) <= kGmmSpan && fabsf(y1) <= kGmmSpan && fabsf(y2) <= kGmmSpan);
    if (wild) y0 = y1 = y2 = 0.0f;
    const Split s0 = split3(y0), s1 = split3(y1), s2 = split3(y2), s3 = split3((y0 * y0 + y1 * y1) + y2 * y2);
    const unsigned h0 = s0.h | s1.h << 16, h1 = s2.h | s3.h << 16, m0 = s0.m | s1.m << 16, m1 = s2.m | s3.m << 16,
                   l0 = s0.l | s1.l << 16, l1 = s2.l | s3.l << 16;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int from = 16 * t + (lane & 15);
      const unsigned H0 = __shfl(h0, from, 64), H1 = __shfl(h1, from, 64), M0 = __shfl(m0, from, 64),
                     M1 = __shfl(m1, from, 64), L0 = __shfl(l0, from, 64), L1 = __shfl(l1, from, 64);
      pt[t] = __builtin_bit_cast(Bf8, uint4{g == 1 ? M0 : (g == 3 ? 0x3f803f80u : H0),
                                            g == 1 ? M1 : (g == 3 ? 0x3f80u : H1),
                                            g == 0 ? H0 : (g == 2 ? L0 : M0), g == 0 ? H1 : (g == 2 ? L1 : M1)});
    }
  }
  float v1[4], v2[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) v1[t] = v2[t] = kNone;
  // whether the wave scores every component instead
  bool plain = 4 * __popcll(__ballot(wild)) > plain_scans(k);
  const auto contended = [&]() {
    int c = 0;
#pragma unroll
    for (int t = 0; t < kGmmProbe; ++t) {
      const int from = 16 * t + (lane & 15);
      float vm = fminf(v1[t], __shfl_xor(v1[t], 16, 64));
      vm = fminf(vm, __shfl_xor(vm, 32, 64));
      const float4* r = (const float4*)(rec + (size_t)kGmmRec * min((int)(__float_as_uint(vm) & idmask) * 4 + g, k - 1));
      const float4 a0 = r[0], a1 = r[1], a2 = r[2];
      float s = score(__shfl(x0, from, 64), __shfl(x1, from, 64), __shfl(x2, from, 64), a0, a1, a2.x, a2.y);
      s = fminf(s, __shfl_xor(s, 16, 64));
      s = fminf(s, __shfl_xor(s, 32, 64));
      c += __popcll(__ballot(!(v2[t] - fabsf(v2[t]) * slack > s)));
    }
    return c > kGmmMany;
  };
  const int probe = tiles >= 16 ? tiles / 8 : -1;
  for (int k0 = 0; k0 < tiles; k0 += kGmmChunk) {
    const int nt = min(kGmmChunk, tiles - k0);
    if (k0 == 0) __syncthreads();
    else if (__syncthreads_and(plain)) break;
    for (int t = threadIdx.x; t < nt * (kGmmTileBytes / 16); t += kGeoThreads)
      s_op[t] = ops[(size_t)k0 * (kGmmTileBytes / 16) + t];
    __syncthreads();
    for (int j = 0; j < nt && !plain; ++j) {
      if (k0 + j == probe) plain = contended();
      const uint4* o = s_op + j * (kGmmTileBytes / 16) + lane;
      const Bf8 U = __builtin_bit_cast(Bf8, o[0]), A = __builtin_bit_cast(Bf8, o[64]),
                B = __builtin_bit_cast(Bf8, o[128]);
      const unsigned id = 4 * (k0 + j) + g;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const F4 zero = {0.f, 0.f, 0.f, 0.f};
        const F4 lq = __builtin_amdgcn_mfma_f32_16x16x32_bf16(U, pt[t], zero, 0, 0, 0);
        const F4 h1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, pt[t], zero, 0, 0, 0);
        const F4 h2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B, pt[t], zero, 0, 0, 0);
        float b[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) b[r] = __builtin_fmaf(h1[r], h1[r], __builtin_fmaf(h2[r], h2[r], lq[r]));
        const float low4 = fminf(fminf(fminf(b[0], b[1]), b[2]), b[3]);
        const float v = __uint_as_float((__float_as_uint(low4) & keep) | id);
        v2[t] = __builtin_amdgcn_fmed3f(v1[t], v2[t], v);
        v1[t] = __builtin_amdgcn_fmed3f(v1[t], v, -kNone);  // the lower
      }
    }
  }
  float ms = INFINITY;
  int mi = 0x7fffffff;  // this lane's surfel (tile g, column lane & 15)
  if (!plain) [&]() {
    // exact scores: per surfel the quad of the smallest bound, a component a
    // lane, while a lane's smallest bound does not exceed the best score
    float bs[4], ball[4], x[4][3];
    int bi[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      bs[t] = ball[t] = INFINITY;
      bi[t] = 0x7fffffff;
      const int from = 16 * t + (lane & 15);
      x[t][0] = __shfl(x0, from, 64);
      x[t][1] = __shfl(x1, from, 64);
      x[t][2] = __shfl(x2, from, 64);
      if (__shfl((int)wild, from, 64)) {
        v1[t] = kNone;
        v2[t] = -kNone;
      }
    }
#pragma unroll 1
    for (int it = 0; it < 4; ++it) {  // a lane group is taken once
      bool act[4], any = false;
      int cand[4];
      float4 ra[4], rb[4];
      float2 rc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float vm = fminf(v1[t], __shfl_xor(v1[t], 16, 64));
        vm = fminf(vm, __shfl_xor(vm, 32, 64));
        act[t] = vm < 2e38f && !(vm - fabsf(vm) * slack > ball[t]);
        any = any || act[t];
        cand[t] = act[t] ? (int)(__float_as_uint(vm) & idmask) * 4 + g : k;
        v1[t] = (act[t] & (v1[t] == vm)) ? kNone : v1[t];
      }
      if (!__any(any)) break;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float4* r = (const float4*)(rec + (size_t)kGmmRec * min(cand[t], k - 1));
        ra[t] = r[0];
        rb[t] = r[1];
        rc[t] = *(const float2*)(r + 2);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float s = score(x[t][0], x[t][1], x[t][2], ra[t], rb[t], rc[t].x, rc[t].y);
        keep_lower(cand[t] < k ? s : INFINITY, cand[t], bs[t], bi[t]);
        ball[t] = fminf(bs[t], __shfl_xor(bs[t], 16, 64));
        ball[t] = fminf(ball[t], __shfl_xor(ball[t], 32, 64));
      }
    }
    // a lane whose second bound is not above the best score: its quads are
    // scored by the whole wave
    uint64_t todos[4];
    int scans = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      todos[t] = __ballot(!(v2[t] - fabsf(v2[t]) * slack > ball[t]));
      scans += __popcll(todos[t]);
    }
    if (scans > plain_scans(k)) {
      plain = true;
      return;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      uint64_t todo = todos[t];
      while (todo) {
        const int from = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1;
        const float y0 = __shfl(x[t][0], from, 64), y1 = __shfl(x[t][1], from, 64), y2 = __shfl(x[t][2], from, 64);
        float ws = INFINITY;
        int wi = 0x7fffffff;
        for (int j = 16 * (lane >> 2) + 4 * (from >> 4) + (lane & 3); j < k; j += 256) {
          const float4* r = (const float4*)(rec + (size_t)kGmmRec * j);
          const float4 a0 = r[0], a1 = r[1], a2 = r[2];
          keep_lower(score(y0, y1, y2, a0, a1, a2.x, a2.y), j, ws, wi);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          const float os = __shfl_xor(ws, o, 64);
          const int oi = __shfl_xor(wi, o, 64);
          keep_lower(os, oi, ws, wi);
        }
        keep_lower(lane == from ? ws : INFINITY, wi, bs[t], bi[t]);
      }
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float os = __shfl_xor(bs[t], o, 64);
        const int oi = __shfl_xor(bi[t], o, 64);
        keep_lower(os, oi, bs[t], bi[t]);
      }
      if (t == g) {
        ms = bs[t];
        mi = bi[t];
      }
    }
  }();
  if (plain) {
    // records two ahead, through the scalar cache (the last one again past the
    // end, which cannot win: strict, of equal scores the lowest index stays)
    struct Rec {
      float4 a, b;
      float2 c;
    };
    const auto at = [&](int j) {
      const float4* r = (const float4*)(rec + (size_t)kGmmRec * min(j, k - 1));
      return Rec{r[0], r[1], *(const float2*)(r + 2)};
    };
    Rec r0 = at(0), r1 = at(1);
#pragma unroll 2
    for (int j = 0; j < k; j += 2) {
      const Rec n0 = at(j + 2), n1 = at(j + 3);
      const float s0 = score(x0, x1, x2, r0.a, r0.b, r0.c.x, r0.c.y);
      const bool up0 = s0 < ms;
      ms = up0 ? s0 : ms;
      mi = up0 ? j : mi;
      const float s1 = score(x0, x1, x2, r1.a, r1.b, r1.c.x, r1.c.y);
      const bool up1 = s1 < ms;
      ms = up1 ? s1 : ms;
      mi = up1 ? j + 1 : mi;
      r0 = n0;
      r1 = n1;
    }
  }
  const int bk = ms < INFINITY ? mi : 0;
  double geo = 0.0, iso = 0.0;
  if (ok) {
    // loss terms and gradients in FP64 (the projection onto the unit
    // quaternion's tangent space cancels most of its input)
    const float* r = rec + (size_t)kGmmRec * bk;
    const double nk0 = r[10], nk1 = r[11], nk2 = r[12];
    const double delta = ((x0 - (double)r[0]) * nk0 + (x1 - (double)r[1]) * nk1) + (x2 - (double)r[2]) * nk2;
    // surfel normal: third column of the rotation of the normalised quaternion
    const double q0 = quats[4 * i], q1 = quats[4 * i + 1], q2 = quats[4 * i + 2], q3 = quats[4 * i + 3];
    const double qq = ((q0 * q0 + q1 * q1) + q2 * q2) + q3 * q3;
    const double rq = qq > 0.0 ? 1.0 / sqrt(qq) : 0.0;
    const double w = q0 * rq, x = q1 * rq, y = q2 * rq, z = q3 * rq;
    const double n0 = 2.0 * (x * z + w * y), n1 = 2.0 * (y * z - w * x), n2 = 1.0 - 2.0 * (x * x + y * y);
    const double dot = (n0 * nk0 + n1 * nk1) + n2 * nk2;
    const double s0 = scales[2 * i], s1 = scales[2 * i + 1];
    geo = fabs(delta) + (double)lambda_n * (1.0 - fabs(dot));
    iso = (s0 - s1) * (s0 - s1);
    const double sd = delta > 0.0 ? 1.0 : (delta < 0.0 ? -1.0 : 0.0);
    d_means[3 * i] = (float)(sd * nk0);
    d_means[3 * i + 1] = (float)(sd * nk1);
    d_means[3 * i + 2] = (float)(sd * nk2);
    d_scales[2 * i] = (float)(2.0 * (s0 - s1));
    d_scales[2 * i + 1] = (float)(-2.0 * (s0 - s1));
    // dL/dn = -lambda_n sign(dot) n_k, through n(w, x, y, z) and q / |q|
    const double sg = dot > 0.0 ? 1.0 : (dot < 0.0 ? -1.0 : 0.0);
    const double g0 = -lambda_n * sg * nk0, g1 = -lambda_n * sg * nk1, g2 = -lambda_n * sg * nk2;
    const double gw = 2.0 * y * g0 - 2.0 * x * g1;
    const double gx = 2.0 * z * g0 - 2.0 * w * g1 - 4.0 * x * g2;
    const double gy = 2.0 * w * g0 + 2.0 * z * g1 - 4.0 * y * g2;
    const double gz = 2.0 * x * g0 + 2.0 * y * g1;
    const double pr = ((gw * w + gx * x) + gy * y) + gz * z;
    d_quats[4 * i] = (float)((gw - w * pr) * rq);
    d_quats[4 * i + 1] = (float)((gx - x * pr) * rq);
    d_quats[4 * i + 2] = (float)((gy - y * pr) * rq);
    d_quats[4 * i + 3] = (float)((gz - z * pr) * rq);
    if (assign) assign[i] = bk;
  }
  const double bg = block_sum_f64(geo, s_red);
  const double bo = block_sum_f64(iso, s_red);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = bg;
    part[2 * blockIdx.x + 1] = bo;
  }
}

// One block: the blocks' sums, thread-strided in block order, then a fixed
// tree (one wave took 16 us for 3907 blocks, all of it waiting for loads).
__global__ __launch_bounds__(kGeoThreads) void k_geo_sum(int64_t nb, const double* __restrict__ part,
                                                         double* __restrict__ out) {
  __shared__ double s_red[kGeoThreads / 64];
  double g = 0.0, s = 0.0;
  for (int64_t b = threadIdx.x; b < nb; b += kGeoThreads) {
    g += part[2 * b];
    s += part[2 * b + 1];
  }
  g = block_sum_f64(g, s_red);
  s = block_sum_f64(s, s_red);
  if (threadIdx.x == 0) {
    out[0] = g;
    out[1] = s;
  }
}

// workspace: records, the bound's operands, the blocks' sums
static size_t rec_bytes(int k) { return ((size_t)k * kGmmRec * 4 + 255) & ~(size_t)255; }
static size_t op_bytes(int k) { return (size_t)cdiv(k, kGmmTile) * kGmmTileBytes; }

size_t geometry_workspace_bytes(int64_t n, int k) {
  const int64_t nb = cdiv(std::max<int64_t>(n, 1), kGeoThreads);
  return rec_bytes(k) + op_bytes(k) + (size_t)nb * 16;
}

void launch_geometry_loss(const GeometryArgs& a, char* ws, hipStream_t st) {
  const int64_t nb = cdiv(std::max<int64_t>(a.n, 1), kGeoThreads);
  float* rec = (float*)ws;
  uint4* ops = (uint4*)(ws + rec_bytes(a.k));
  double* part = (double*)(ws + rec_bytes(a.k) + op_bytes(a.k));
  hipLaunchKernelGGL(k_gmm_prep, dim3((unsigned)cdiv(a.k, 64)), dim3(64), 0, st, a.k, a.gmean, a.gcov, a.gweight,
                     rec, ops);
  hipLaunchKernelGGL(k_geo_loss, dim3((unsigned)nb), dim3(kGeoThreads), 0, st, a.n, a.means, a.scales, a.quats, a.k,
                     (const float*)rec, (const uint4*)ops, a.lambda_n, a.assign, a.d_means, a.d_scales, a.d_quats,
                     part);
  hipLaunchKernelGGL(k_geo_sum, dim3(1), dim3(kGeoThreads), 0, st, nb, (const double*)part, a.losses);
}

}  // namespace psm
