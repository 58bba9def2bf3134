// Key stage of the rasterizer (Sec. 5, Precise Tile Intersection):
//   preprocess  -- per surfel: rotation, camera space, culling, the projected
//                  cutoff ellipse, its footprint count, the walk record;
//   count scan  -- exclusive prefix of the counts in depth order;
//   emission    -- (tile id, surfel id) pairs, written in depth order;
//   tile ranges -- [start, end) of every tile in the tile-sorted pair list.
//
// Every floating-point decision here (cull, depth key, footprint) follows one
// prescribed sequence of IEEE FP32 operations: this translation unit is built
// with -ffp-contract=off and correctly rounded division and square root.
#include "common.h"
#include "internal.h"

#pragma clang fp contract(off)

namespace psm {

using Cam = CamArgs;

// Projected cutoff ellipse of a visible surfel; with the low-pass filter also
// the projected centre and the filter disk's radius^2 (rf2 = 0: no filter).
struct Foot {
  float ecx, ecy, S01, S11, ex, ey, gam;
  float kk;  // chord factor |c detA|; half-size of the isotropic square in its mode
  float xc, yc, rf2;
};

// Quantities of the prescribed FP32 key stage for one surfel.
struct Key {
  int cull;
  int flip;
  float mc2, p, q, xc, yc, A00, A01, A10, A11, dA;
  float nc[3];
  Foot f;
};

// Opacity-aware footprint radius^2 (an exact work reduction): a pixel is
// skipped when alpha = o exp(-rho/2) < 1/255 (Sec. 3.1), i.e. when
// rho > 2 ln(255 o), so a surfel's footprint only needs rho <= min(9,
// 2 ln(255 o)).  The bound gets a 2^-10 absolute and relative margin (the
// per-pixel FP32 alpha is within a few ulp of exact) and is rounded up to a
// multiple of 2^-12 in FP64, which is exact in FP32, so correctly rounded
// and faithful FP64 logarithms give the same value.
__device__ __forceinline__ float opacity_foot2(float o) {
  const double L = 2.0 * log(255.0 * (double)o);
  const double r = ceil((L + 0x1p-10) * (1.0 + 0x1p-10) * 4096.0) * (1.0 / 4096.0);
  return (float)fmin((double)kFoot2, fmax(r, 1.0 / 4096.0));
}

// Radius^2 beyond which alpha < 1/255 for the walks' sub-tile culling: the
// same bound with a plain FP32 logarithm and a margin of 2^-8 (absolute) and
// 2^-9 (relative), far above its rounding.
__device__ __forceinline__ float cull_foot2(float o) {
  return fmaxf(2.0f * __logf(255.0f * o) * (1.0f + 0x1p-9f) + 0x1p-8f, 0x1p-12f);
}

// foot2: footprint radius^2 (kFoot2, or the opacity-aware bound).  The cull
// decisions always use kFoot2, so both footprints keep the same visible set.
// lowpass: the footprint also takes the low-pass filter's disk.
__device__ __forceinline__ Key key_stage(const float* mu, const float* sc, const float* qq, const Cam& k, float foot2,
                                      int mode, int lowpass) {
  Key r;
  r.cull = 0;
  r.flip = 0;
  const float nq = ((qq[0] * qq[0] + qq[1] * qq[1]) + qq[2] * qq[2]) + qq[3] * qq[3];
  if (!(nq > 0.0f)) { r.cull = 1; return r; }
  const float rn = 1.0f / sqrtf(nq);
  const float w = qq[0] * rn, x = qq[1] * rn, y = qq[2] * rn, z = qq[3] * rn;
  const float xx = x * x, yy = y * y, zz = z * z;
  const float xy = x * y, xz = x * z, yz = y * z;
  const float wx = w * x, wy = w * y, wz = w * z;
  const float tu0 = 1.0f - 2.0f * (yy + zz), tu1 = 2.0f * (xy + wz), tu2 = 2.0f * (xz - wy);
  const float tv0 = 2.0f * (xy - wz), tv1 = 1.0f - 2.0f * (xx + zz), tv2 = 2.0f * (yz + wx);
  const float nn0 = 2.0f * (xz + wy), nn1 = 2.0f * (yz - wx), nn2 = 1.0f - 2.0f * (xx + yy);
  float mc[3], a[3], b[3], rnv[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float R0 = k.R[3 * i], R1 = k.R[3 * i + 1], R2 = k.R[3 * i + 2];
    mc[i] = ((R0 * mu[0] + R1 * mu[1]) + R2 * mu[2]) + k.t[i];
    const float ra = (R0 * tu0 + R1 * tu1) + R2 * tu2;
    const float rb = (R0 * tv0 + R1 * tv1) + R2 * tv2;
    rnv[i] = (R0 * nn0 + R1 * nn1) + R2 * nn2;
    a[i] = sc[0] * ra;
    b[i] = sc[1] * rb;
  }
  const float dn = (rnv[0] * mc[0] + rnv[1] * mc[1]) + rnv[2] * mc[2];
  r.flip = dn > 0.0f ? 1 : 0;
#pragma unroll
  for (int i = 0; i < 3; ++i) r.nc[i] = r.flip ? -rnv[i] : rnv[i];
  if (!(mc[2] > k.near_plane)) { r.cull = 2; return r; }
  const float zmin = mc[2] - kCut * sqrtf(a[2] * a[2] + b[2] * b[2]);
  if (!(zmin > k.near_plane)) { r.cull = 3; return r; }
  const float iz = 1.0f / mc[2];
  const float p = a[2] * iz, q = b[2] * iz;
  const float g2 = p * p + q * q;
  const float gam = 1.0f - kFoot2 * g2;
  if (!(gam > 0.0f)) { r.cull = 3; return r; }
  const float mx = mc[0] * iz, my = mc[1] * iz;
  const float xc = k.fx * mx + k.cx, yc = k.fy * my + k.cy;
  const float A00 = k.fx * ((a[0] - mx * a[2]) * iz);
  const float A01 = k.fx * ((b[0] - mx * b[2]) * iz);
  const float A10 = k.fy * ((a[1] - my * a[2]) * iz);
  const float A11 = k.fy * ((b[1] - my * b[2]) * iz);
  const float dA = A00 * A11 - A01 * A10;
  if (!(fabsf(dA) > 0.0f)) { r.cull = 4; return r; }
  float cc = kFoot2 / gam;
  const float w0 = A00 * p + A01 * q, w1 = A10 * p + A11 * q;
  float S00 = cc * ((A00 * A00 + A01 * A01) + cc * (w0 * w0));
  float S01 = cc * ((A00 * A10 + A01 * A11) + cc * (w0 * w1));
  float S11 = cc * ((A10 * A10 + A11 * A11) + cc * (w1 * w1));
  if (!(S00 > 0.0f && S11 > 0.0f && S00 < 1e24f && S11 < 1e24f)) { r.cull = 4; return r; }
  float gf = gam;
  if (foot2 != kFoot2) {  // the same ellipse formulas at the smaller radius
    gf = 1.0f - foot2 * g2;
    cc = foot2 / gf;
    S00 = cc * ((A00 * A00 + A01 * A01) + cc * (w0 * w0));
    S01 = cc * ((A00 * A10 + A01 * A11) + cc * (w0 * w1));
    S11 = cc * ((A10 * A10 + A11 * A11) + cc * (w1 * w1));
  }
  r.mc2 = mc[2]; r.p = p; r.q = q; r.xc = xc; r.yc = yc;
  r.A00 = A00; r.A01 = A01; r.A10 = A10; r.A11 = A11; r.dA = dA;
  r.f.ecx = xc - cc * w0;
  r.f.ecy = yc - cc * w1;
  r.f.S01 = S01; r.f.S11 = S11;
  r.f.ex = sqrtf(S00);
  r.f.ey = sqrtf(S11);
  r.f.gam = gf;
  r.f.kk = fabsf(cc * dA);
  r.f.xc = xc;
  r.f.yc = yc;
  r.f.rf2 = lowpass ? 0.5f * foot2 + kLpPad : 0.0f;
  if (mode == kSphere) {
    const float hs = 0.5f * (S00 + S11);
    const float hd = 0.5f * (S00 - S11);
    const float lmax = hs + sqrtf(hd * hd + S01 * S01);
    r.f.kk = fmaxf(sqrtf(lmax), fmaxf(r.f.ex, r.f.ey));
  }
  return r;
}

// Culling record (CullRec) of a visible surfel from the walk record's FP64
// quantities: the hit test is FP64, and in FP32 the camera-space position alone
// is off by fx 2^-24 (|R mu| + |t|) / z pixels, more than any fixed slack once
// the world's origin is some hundred metres from the camera.  Here only the
// last steps are FP32, with relative errors near 2^-22 of the extents.  lp:
// the low-pass filter, whose record is a box and keeps the key stage's
// centre and rf2 (the emission's footprint).  A surfel that the FP64 values put
// across the camera plane has no ellipse: infinite slack, never culled.  1M
// surfels: preprocess 78 us, as with the FP32 record.
__device__ __forceinline__ CullRec cull_record(double A00, double A01, double A10, double A11, double p, double q,
                                               double xc, double yc, float cull2, int lp, const Foot& f) {
  CullRec c;
  const double gd = 1.0 - (double)cull2 * (p * p + q * q);
  const float gc = (float)gd, a00 = (float)A00, a01 = (float)A01, a10 = (float)A10, a11 = (float)A11;
  const float w0 = (float)(A00 * p + A01 * q), w1 = (float)(A10 * p + A11 * q);
  const float c2 = cull2 * __builtin_amdgcn_rcpf(gc);
  const float T00 = c2 * ((a00 * a00 + a01 * a01) + c2 * (w0 * w0));
  const float T01 = c2 * ((a00 * a10 + a01 * a11) + c2 * (w0 * w1));
  const float T11 = c2 * ((a10 * a10 + a11 * a11) + c2 * (w1 * w1));
  const float ex = __builtin_amdgcn_sqrtf(T00), ey = __builtin_amdgcn_sqrtf(T11);
  const double cx = xc - (double)(c2 * w0), cy = yc - (double)(c2 * w1);
  if (lp) {
    const float rf = sqrtf(f.rf2);
    const double x0 = fmin(cx - (double)ex, xc - (double)rf), x1 = fmax(cx + (double)ex, xc + (double)rf);
    const double y0 = fmin(cy - (double)ey, yc - (double)rf), y1 = fmax(cy + (double)ey, yc + (double)rf);
    c.e0 = make_float4((float)(0.5 * (x0 + x1)), (float)(0.5 * (y0 + y1)), (float)(0.5 * (x1 - x0)),
                       (float)(0.5 * (y1 - y0)));
    c.e1 = make_float4(f.xc, f.yc, f.rf2, 0.0f);
  } else {
    const float it = __builtin_amdgcn_rcpf(T11);
    c.e0 = make_float4((float)cx, (float)cy, ex, ey);
    c.e1 = make_float4(T01 * __builtin_amdgcn_rcpf(ex), T01 * it,
                       fabsf(c2 * (float)(A00 * A11 - A01 * A10)) * it * __builtin_amdgcn_rsqf(gc), 0.0f);
  }
  c.e1.w = 0x1p-6f + 0x1p-16f * (c.e0.z + c.e0.w) + 0x1p-20f * (fabsf(c.e0.x) + fabsf(c.e0.y));
  if (!(gd > 0.0)) {
    c.e0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    c.e1.w = INFINITY;
  }
  return c;
}

// Walk record of a visible surfel (not part of any decision): the centred,
// depth-normalised homography's A^-1, e = (p, q) A^-1 and the projected centre,
// evaluated and kept in FP64 (the per-pixel solve is FP64 as well).  cull2:
// radius^2 of the walks' culling ellipse.
__device__ __forceinline__ void walk_record(const float* mu_f, const float* sc, const float* qf, float o,
                                         const float* rgb, const float* nc, const Foot& f, float cull2, int lp,
                                         const Cam& k, WalkRec* out) {
  const double q0 = qf[0], q1 = qf[1], q2 = qf[2], q3 = qf[3];
  const double rn = 1.0 / sqrt(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
  const double w = q0 * rn, x = q1 * rn, y = q2 * rn, z = q3 * rn;
  const double tu[3] = {1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y + w * z), 2.0 * (x * z - w * y)};
  const double tv[3] = {2.0 * (x * y - w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z + w * x)};
  double mc[3], a[3], b[3];
  for (int i = 0; i < 3; ++i) {
    const double R0 = k.R[3 * i], R1 = k.R[3 * i + 1], R2 = k.R[3 * i + 2];
    mc[i] = R0 * mu_f[0] + R1 * mu_f[1] + R2 * mu_f[2] + (double)k.t[i];
    a[i] = sc[0] * (R0 * tu[0] + R1 * tu[1] + R2 * tu[2]);
    b[i] = sc[1] * (R0 * tv[0] + R1 * tv[1] + R2 * tv[2]);
  }
  const double iz = 1.0 / mc[2];
  const double p = a[2] * iz, q = b[2] * iz, mx = mc[0] * iz, my = mc[1] * iz;
  const double xc = (double)k.fx * mx + (double)k.cx, yc = (double)k.fy * my + (double)k.cy;
  const double A00 = k.fx * (a[0] - mx * a[2]) * iz, A01 = k.fx * (b[0] - mx * b[2]) * iz;
  const double A10 = k.fy * (a[1] - my * a[2]) * iz, A11 = k.fy * (b[1] - my * b[2]) * iz;
  const double idA = 1.0 / (A00 * A11 - A01 * A10);
  const double i00 = A11 * idA, i01 = -A01 * idA, i10 = -A10 * idA, i11 = A00 * idA;
  const double e0 = p * i00 + q * i10, e1 = p * i01 + q * i11;
  WalkRec r;
  r.d0 = make_double2(i00, i01);
  r.d1 = make_double2(i10, i11);
  r.d2 = make_double2(e0, e1);
  r.d3 = make_double2(xc, yc);
  r.f0 = make_float4((float)mc[2], o, rgb[0], rgb[1]);
  r.f1 = make_float4(rgb[2], nc[0], nc[1], nc[2]);
  r.c = cull_record(A00, A01, A10, A11, p, q, xc, yc, cull2, lp, f);
  *out = r;
}

// Tiles whose pixel-centre hull [t*T + 0.5, min(t*T + T - 0.5, npix - 0.5)]
// meets [lo, hi] along one axis (T = the tile's size along it).
__device__ __forceinline__ bool tile_span(float lo, float hi, int npix, int T, int nt, int& t0, int& t1) {
  if (!(hi >= 0.5f) || !(lo <= (float)npix - 0.5f)) return false;
  float f0 = ceilf((lo - ((float)T - 0.5f)) / (float)T);
  float f1 = floorf((hi - 0.5f) / (float)T);
  f0 = fmaxf(f0, 0.0f);
  f1 = fminf(f1, (float)(nt - 1));
  if (!(f0 <= f1)) return false;
  t0 = (int)f0;
  t1 = (int)f1;
  return true;
}

// Tile box of the footprint of mode `mode`; false if it meets no tile.  With
// the low-pass filter the footprint is the union with the filter's disk: the
// disk's box joins every mode's box.
struct TileBox {
  int x0, x1, y0, y1;
};
__device__ __forceinline__ bool foot_box(const Foot& f, int mode, int W, int H, int tw, int th, int ntx, int nty,
                                         TileBox& box) {
  const bool lp = f.rf2 > 0.0f;
  const float rf = lp ? sqrtf(f.rf2) : 0.0f;
  float bx0, bx1, by0, by1;
  if (mode == kSphere) {
    const float rr = f.kk;
    bx0 = f.ecx - rr;
    bx1 = f.ecx + rr;
    by0 = f.ecy - rr;
    by1 = f.ecy + rr;
  } else {
    bx0 = f.ecx - f.ex;
    bx1 = f.ecx + f.ex;
    by0 = f.ecy - f.ey;
    by1 = f.ecy + f.ey;
  }
  if (lp) {
    bx0 = fminf(bx0, f.xc - rf);
    bx1 = fmaxf(bx1, f.xc + rf);
    by0 = fminf(by0, f.yc - rf);
    by1 = fmaxf(by1, f.yc + rf);
  }
  return tile_span(bx0, bx1, W, tw, ntx, box.x0, box.x1) && tile_span(by0, by1, H, th, nty, box.y0, box.y1);
}

// Tiles [x0, x1] of tile row ty of the footprint.  The exact mode takes the
// x-extent of the ellipse inside the row's band (with the filter, the hull of
// the ellipse's and the disk's).
__device__ __forceinline__ bool foot_row(const Foot& f, int mode, int W, int H, int tw, int th, int ntx,
                                         const TileBox& box, int ty, int& x0, int& x1) {
  x0 = box.x0;
  x1 = box.x1;
  if (mode != kEllipse) return true;
  const bool lp = f.rf2 > 0.0f;
  const float yr = f.S01 / f.ex;
  const float rlo = (float)(ty * th) + 0.5f;
  const float rhi = fminf((float)(ty * th) + ((float)th - 0.5f), (float)H - 0.5f);
  const float ylo = rlo - f.ecy;
  const float yhi = rhi - f.ecy;
  const float lo = fmaxf(ylo, -f.ey), hi = fminf(yhi, f.ey);
  bool have = false;
  float xl = 0.0f, xr = 0.0f;
  if (lo <= hi) {
    const float dR = fminf(fmaxf(yr, lo), hi);
    const float dL = fminf(fmaxf(-yr, lo), hi);
    const float hR = sqrtf(fmaxf(0.0f, (f.S11 - dR * dR) / f.gam)) * f.kk;
    const float hL = sqrtf(fmaxf(0.0f, (f.S11 - dL * dL) / f.gam)) * f.kk;
    const float xR = (f.S01 * dR + hR) / f.S11;
    const float xL = (f.S01 * dL - hL) / f.S11;
    xl = f.ecx + xL;
    xr = f.ecx + xR;
    have = true;
  }
  if (lp) {  // the disk's widest chord within the band
    const float dlo = rlo - f.yc, dhi = rhi - f.yc;
    const float dy = fminf(fmaxf(0.0f, dlo), dhi);
    const float h2 = f.rf2 - dy * dy;
    if (h2 >= 0.0f) {
      const float h = sqrtf(h2);
      const float dl = f.xc - h, dr = f.xc + h;
      xl = have ? fminf(xl, dl) : dl;
      xr = have ? fmaxf(xr, dr) : dr;
      have = true;
    }
  }
  if (!have || !tile_span(xl, xr, W, tw, ntx, x0, x1)) return false;
  x0 = max(x0, box.x0);
  x1 = min(x1, box.x1);
  return x0 <= x1;
}

// A surfel near the camera covers up to thousands of tiles.  Footprints of
// more tile rows (counting) or tiles (emission) than these are taken by the
// whole wave, a lane per row, and not by their own lane while 63 wait.  Below
// the bounds a lane's own loop is shorter than the wave's common steps.
// Emission of 1M street surfels 515 -> 61 us, of a 400k room 197 -> 101 us;
// preprocess 125 -> 72 us and 64 -> 59 us.
constexpr int kTallRows = 6;
constexpr int kWidePairs = 16;

__device__ __forceinline__ float lane_f(float v, int lane) { return __uint_as_float(lane_value(__float_as_uint(v), lane)); }
__device__ __forceinline__ Foot lane_foot(const Foot& f, int l) {
  return Foot{lane_f(f.ecx, l), lane_f(f.ecy, l), lane_f(f.S01, l), lane_f(f.S11, l), lane_f(f.ex, l), lane_f(f.ey, l),
              lane_f(f.gam, l), lane_f(f.kk, l), lane_f(f.xc, l), lane_f(f.yc, l), lane_f(f.rf2, l)};
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t v, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = i; j < count; j += stride) p[j] = v;
}

// Status words and empty tile ranges, before a forward.
__global__ __launch_bounds__(256) void k_init_forward(uint32_t* __restrict__ st, uint32_t n, uint32_t tiles,
                                                      uint64_t total, uint32_t cap, uint2* __restrict__ ranges) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < kStWords) st[i] = init_word(i, n, tiles, total, cap);
  if (i < tiles) ranges[i] = make_uint2(0u, 0u);
}

// Thread per virtual surfel v = b * N + i (surfel i seen by camera b).
__global__ __launch_bounds__(256) void k_preprocess(
    int64_t nv, const float* __restrict__ means, const float* __restrict__ scales,
    const float* __restrict__ quats, const float* __restrict__ opacity, const float* __restrict__ rgb,
    CamTable ct, int mode, int opacity_foot, int lowpass, WalkRec* __restrict__ rec, float4* __restrict__ fp,
    uint32_t* __restrict__ key, uint32_t* __restrict__ ids, uint32_t* __restrict__ count,
    int32_t* __restrict__ cull) {
  __shared__ Cam s_cam[kMaxCams];  // cameras by constant index (no private copy of the table)
#pragma unroll
  for (int b = 0; b < kMaxCams; ++b)
    if (threadIdx.x == b && b < ct.n) s_cam[b] = ct.cam[b];
  __syncthreads();
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = v < nv;  // every lane stays for the tall footprints
  const int b = valid ? camera_of(ct, v) : 0;
  const int64_t i = valid ? v - (int64_t)b * ct.nsurf : 0;
  const Cam& cam = s_cam[b];
  Key kk;
  kk.cull = 1;
  TileBox box{0, -1, 0, -1};
  uint32_t c = 0;
  bool listed = false;
  if (valid) {
    const float foot2 = opacity_foot ? opacity_foot2(opacity[i]) : kFoot2;
    kk = key_stage(means + 3 * i, scales + 2 * i, quats + 4 * i, cam, foot2, mode, lowpass);
    ids[v] = (uint32_t)v;
    cull[v] = kk.cull | (kk.flip << 8);  // bit 8: normal flipped toward the camera
    key[v] = kk.cull != 0 ? 0xFFFFFFFFu : __float_as_uint(kk.mc2);
    if (kk.cull == 0) {
      fp[2 * v] = make_float4(kk.f.ecx, kk.f.ecy, kk.f.ex, kk.f.ey);
      fp[2 * v + 1] = make_float4(kk.f.S01, kk.f.S11, kk.f.gam, kk.f.kk);
      const float cull2 = lowpass ? foot2 : fminf(foot2, cull_foot2(opacity[i]));
      walk_record(means + 3 * i, scales + 2 * i, quats + 4 * i, opacity[i], rgb + 3 * i, kk.nc, kk.f, cull2, lowpass,
                  cam, rec + v);
      listed = foot_box(kk.f, mode, cam.W, cam.H, ct.tw, ct.th, ct.ntx[b], ct.nty[b], box);
    }
  }
  // pairs: boxes need no row test; short ellipses by their lane, tall ones by the wave
  const bool rows = listed && mode == kEllipse;
  const bool tall = rows && box.y1 - box.y0 >= kTallRows;
  if (listed && !rows) c = (uint32_t)(box.y1 - box.y0 + 1) * (uint32_t)(box.x1 - box.x0 + 1);
  if (rows && !tall) {
    for (int ty = box.y0; ty <= box.y1; ++ty) {
      int x0, x1;
      if (foot_row(kk.f, mode, cam.W, cam.H, ct.tw, ct.th, ct.ntx[b], box, ty, x0, x1)) c += (uint32_t)(x1 - x0 + 1);
    }
  }
  const int lane = threadIdx.x & 63;
  for (uint64_t m = __ballot(tall); m; m &= m - 1) {
    const int o = __builtin_ctzll(m);
    const Foot f = lane_foot(kk.f, o);
    const int bo = (int)lane_value((uint32_t)b, o);
    const TileBox bx{(int)lane_value((uint32_t)box.x0, o), (int)lane_value((uint32_t)box.x1, o),
                     (int)lane_value((uint32_t)box.y0, o), (int)lane_value((uint32_t)box.y1, o)};
    int sum = 0;
    for (int ty = bx.y0 + lane; ty <= bx.y1; ty += 64) {
      int x0, x1;
      if (foot_row(f, mode, s_cam[bo].W, s_cam[bo].H, ct.tw, ct.th, ct.ntx[bo], bx, ty, x0, x1)) sum += x1 - x0 + 1;
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) sum += __shfl_xor(sum, w, 64);
    if (lane == o) c = (uint32_t)sum;
  }
  if (valid) count[v] = c;
}

// Cull codes of all virtual surfels into the status words (stats read-back):
// counting them in k_preprocess cost it 9 ns per block and code on one shared
// line, 113 of its us for 1M surfels against the rest of its work.
__global__ __launch_bounds__(256) void k_count_culls(int64_t nv, const int32_t* __restrict__ cull,
                                                     uint32_t* __restrict__ status) {
  __shared__ uint32_t s_cnt[5];
  if (threadIdx.x < 5) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < nv; v += (int64_t)gridDim.x * 256)
    atomicAdd(&s_cnt[min(cull[v] & 0xFF, 4)], 1u);
  __syncthreads();
  if (threadIdx.x < 5 && s_cnt[threadIdx.x]) atomicAdd(&status[kStCull + threadIdx.x], s_cnt[threadIdx.x]);
  if (threadIdx.x == 0 && s_cnt[0]) atomicAdd(&status[kStVisible], s_cnt[0]);
}

// ---- exclusive scan of the pair counts, gathered in depth order ------------
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(int64_t n, const uint32_t* __restrict__ order,
                                                             const uint32_t* __restrict__ count,
                                                             uint64_t* __restrict__ bsum) {
  __shared__ uint64_t s[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  uint64_t acc = 0;
#pragma unroll 4
  for (int j = 0; j < kScanItems; ++j) {
    const int64_t r = base + (int64_t)j * kScanThreads + threadIdx.x;
    if (r < n) acc += count[order[r]];
  }
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int o = kScanThreads / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[blockIdx.x] = s[0];
}

// One block: exclusive scan of the block sums, total -> status.
__global__ __launch_bounds__(1024) void k_scan_top(int64_t nb, uint64_t* __restrict__ bsum, int64_t cap,
                                                   uint32_t* __restrict__ status) {
  __shared__ uint64_t s[1024];
  const int t = threadIdx.x;
  const int64_t per = cdiv(nb, 1024);
  const int64_t b0 = t * per, b1 = min<int64_t>(nb, b0 + per);
  uint64_t acc = 0;
  for (int64_t b = b0; b < b1; ++b) acc += bsum[b];
  s[t] = acc;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    uint64_t v = t >= o ? s[t - o] : 0;
    __syncthreads();
    s[t] += v;
    __syncthreads();
  }
  uint64_t run = s[t] - acc;
  for (int64_t b = b0; b < b1; ++b) {
    const uint64_t v = bsum[b];
    bsum[b] = run;
    run += v;
  }
  if (t == 1023) {
    write_pair_total(status, s[1023], (uint64_t)cap);
  }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_down(int64_t n, const uint32_t* __restrict__ order,
                                                           const uint32_t* __restrict__ count,
                                                           const uint64_t* __restrict__ bsum,
                                                           uint32_t* __restrict__ offs) {
  __shared__ uint64_t s[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  uint64_t acc = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    const int64_t r = base + j;
    v[j] = r < n ? count[order[r]] : 0u;
    acc += v[j];
  }
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 1; o < kScanThreads; o <<= 1) {
    uint64_t x = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
    __syncthreads();
    s[threadIdx.x] += x;
    __syncthreads();
  }
  uint64_t run = bsum[blockIdx.x] + s[threadIdx.x] - acc;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    const int64_t r = base + j;
    if (r < n) offs[r] = (uint32_t)run;
    run += v[j];
  }
}

// ---- pair emission in depth order --------------------------------------------
// Thread per depth rank r: the pairs of virtual surfel v = order[r] go to
// [offs[r], offs[r] + count[v]), tile rows in order; vbase[v] = offs[r].  More
// than kWidePairs pairs are emitted by the whole wave.
__global__ __launch_bounds__(256) void k_emit(int64_t nv, const uint32_t* __restrict__ order,
                                              const uint32_t* __restrict__ count,
                                              const uint32_t* __restrict__ offs, const float4* __restrict__ fp,
                                              const WalkRec* __restrict__ rec, int lowpass, CamTable ct, int mode, int64_t cap, uint32_t* __restrict__ vbase,
                                              uint32_t* __restrict__ ptile, uint32_t* __restrict__ eid,
                                              uint32_t* __restrict__ sid_emit) {
  __shared__ int s_pre[4][64], s_x0[4][64];
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t v = 0, cnt = 0, off = 0;
  if (r < nv) {
    v = order[r];
    off = offs[r];
    vbase[v] = off;
    cnt = count[v];
  }
  const bool wide = cnt > (uint32_t)kWidePairs;
  Foot f{};
  const int b = cnt ? camera_of(ct, v) : 0;
  if (cnt) {
    const float4 f0 = fp[2 * (size_t)v], f1 = fp[2 * (size_t)v + 1];
    float4 f2 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (lowpass) f2 = rec[v].c.e1;
    f = Foot{f0.x, f0.y, f1.x, f1.y, f0.z, f0.w, f1.z, f1.w, f2.x, f2.y, f2.z};
  }
  const auto put = [&](int64_t o, uint32_t tile, uint32_t id) {
    if (o < cap) {
      ptile[o] = tile;
      eid[o] = (uint32_t)o;
      sid_emit[o] = id;
    }
  };
  TileBox box{0, -1, 0, -1};
  if (cnt && foot_box(f, mode, ct.cam[b].W, ct.cam[b].H, ct.tw, ct.th, ct.ntx[b], ct.nty[b], box) && !wide) {
    int64_t o = off;
    for (int ty = box.y0; ty <= box.y1; ++ty) {
      int x0, x1;
      if (!foot_row(f, mode, ct.cam[b].W, ct.cam[b].H, ct.tw, ct.th, ct.ntx[b], box, ty, x0, x1)) continue;
      for (int tx = x0; tx <= x1; ++tx, ++o) put(o, (uint32_t)(ct.tile0[b] + ty * ct.ntx[b] + tx), v);
    }
  }
  // wide footprints: a lane per tile row, then the rows' tiles as one flat
  // sequence, a lane per tile (coalesced writes)
  for (uint64_t m = __ballot(wide); m; m &= m - 1) {
    const int l = __builtin_ctzll(m);
    const Foot g = lane_foot(f, l);
    const int bo = (int)lane_value((uint32_t)b, l);
    const uint32_t vo = lane_value(v, l);
    const TileBox bx{(int)lane_value((uint32_t)box.x0, l), (int)lane_value((uint32_t)box.x1, l),
                     (int)lane_value((uint32_t)box.y0, l), (int)lane_value((uint32_t)box.y1, l)};
    const int ntx = ct.ntx[bo], t0 = ct.tile0[bo];
    int64_t o = lane_value(off, l);
    for (int yb = bx.y0; yb <= bx.y1; yb += 64) {
      const int ty = yb + lane;
      int x0 = 0, x1 = -1;
      if (ty > bx.y1 || !foot_row(g, mode, ct.cam[bo].W, ct.cam[bo].H, ct.tw, ct.th, ntx, bx, ty, x0, x1)) x1 = x0 - 1;
      const int w = x1 - x0 + 1;
      int xs = w;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(xs, d, 64);
        if (lane >= d) xs += y;
      }
      const int total = __shfl(xs, 63, 64);
      wave_lds_sync();
      s_pre[wave][lane] = xs - w;
      s_x0[wave][lane] = x0;
      wave_lds_sync();
      for (int t = lane; t < total; t += 64) {
        int row = 0;  // the last row that starts at or before t
#pragma unroll
        for (int step = 32; step > 0; step >>= 1)
          if (s_pre[wave][row + step] <= t) row += step;
        put(o + t, (uint32_t)(t0 + (yb + row) * ntx + s_x0[wave][row] + (t - s_pre[wave][row])), vo);
      }
      o += total;
    }
  }
}

// Per-surfel key-stage results in surfel order (inspection / tests).
__global__ __launch_bounds__(256) void k_export_keys(int64_t n, const int32_t* __restrict__ cull,
                                                     const uint32_t* __restrict__ skey,
                                                     const uint32_t* __restrict__ sid,
                                                     const uint32_t* __restrict__ count, int32_t* __restrict__ o_cull,
                                                     uint32_t* __restrict__ o_depth, int32_t* __restrict__ o_count) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  if (o_cull) o_cull[r] = cull[r] & 0xFF;
  if (o_count) o_count[r] = (int32_t)count[r];
  if (o_depth) {
    const uint32_t i = sid[r];  // depth-sorted rank r holds surfel i
    o_depth[i] = cull[i] & 0xFF ? 0u : skey[r];
  }
}

// After the tile sort: surfel id of each sorted pair and the tile ranges.  The
// sorted values keep each pair's emission index, where the backward writes the
// pair's partial sums.
__global__ __launch_bounds__(256) void k_finalize_pairs(const uint32_t* __restrict__ ptile,
                                                        const uint32_t* __restrict__ eid,
                                                        const uint32_t* __restrict__ sid_emit,
                                                        const uint32_t* __restrict__ status, uint32_t* __restrict__ pid,
                                                        uint2* __restrict__ ranges, uint64_t* __restrict__ stat,
                                                        uint32_t slots) {
  const uint32_t P = status[kStP];
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < slots) {  // slots <= 256: the first block clears the walk's counters
#pragma unroll
    for (int i = 0; i < 3; ++i) stat[j * kStatLine + i] = 0ull;
  }
  if (j >= P) return;
  pid[j] = sid_emit[eid[j]];
  const uint32_t t = ptile[j];
  if (j == 0 || ptile[j - 1] != t) ranges[t].x = j;
  if (j == P - 1 || ptile[j + 1] != t) ranges[t].y = j + 1;
}

// Tile order, longest lists first: tiles binned by length (four bins per power
// of two, one block, a set of counters per wave so that equal lengths meet in one
// wave only), the bins taken in descending order.  The order within a bin does
// not matter: it only decides when a tile starts, never a result.
constexpr int kOrderBins = 132;
__device__ __forceinline__ int length_bin(uint32_t len) {
  if (len < 4) return (int)len;
  const int e = 31 - __clz(len);
  return 4 * (e - 1) + (int)((len >> (e - 2)) & 3u);
}
__global__ __launch_bounds__(1024) void k_tile_order(int tiles, const uint2* __restrict__ ranges,
                                                     uint32_t* __restrict__ order) {
  __shared__ uint32_t s_off[16][kOrderBins + 1];
  __shared__ uint32_t s_wave[16];
  const int tid = threadIdx.x, wave = tid >> 6;
  for (int i = tid; i < 16 * (kOrderBins + 1); i += 1024) (&s_off[0][0])[i] = 0u;
  __syncthreads();
  constexpr int kItems = 8;  // lengths loaded together
  for (int pass = 0; pass < 2; ++pass) {
    for (int t0 = 0; t0 < tiles; t0 += 1024 * kItems) {
      uint32_t len[kItems];
#pragma unroll
      for (int j = 0; j < kItems; ++j) {
        const int t = t0 + j * 1024 + tid;
        const uint2 r = t < tiles ? ranges[t] : make_uint2(0u, 0u);
        len[j] = r.y - r.x;
      }
#pragma unroll
      for (int j = 0; j < kItems; ++j) {
        const int t = t0 + j * 1024 + tid;
        if (t >= tiles) continue;
        const uint32_t at = atomicAdd(&s_off[wave][length_bin(len[j])], 1u);
        if (pass == 1) order[at] = (uint32_t)t;
      }
    }
    __syncthreads();
    if (pass == 1) break;
    // bins descending, then waves: first position of each (wave, bin); thread
    // t has bin kOrderBins - 1 - t
    const int bin = kOrderBins - 1 - tid;
    uint32_t c[16], tot = 0;
    if (bin >= 0) {
#pragma unroll
      for (int w = 0; w < 16; ++w) c[w] = s_off[w][bin];
#pragma unroll
      for (int w = 0; w < 16; ++w) tot += c[w];
    }
    uint32_t x = tot;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if ((tid & 63) >= o) x += y;
    }
    if ((tid & 63) == 63) s_wave[wave] = x;
    __syncthreads();
    if (bin >= 0) {
      uint32_t run = x - tot;
      for (int w = 0; w < wave; ++w) run += s_wave[w];
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        s_off[w][bin] = run;
        run += c[w];
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------- host wrappers
void launch_fill_u32(void* p, uint32_t v, int64_t count, hipStream_t st) {
  if (count <= 0) return;
  const int64_t blocks = std::min<int64_t>(cdiv(count, 256), 4096);
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, (uint32_t*)p, v, count);
}

void launch_init_forward(const Layout& L, char* ws, hipStream_t st) {
  const int64_t items = std::max<int64_t>(L.tiles, kStWords);
  hipLaunchKernelGGL(k_init_forward, dim3((unsigned)cdiv(items, 256)), dim3(256), 0, st, (uint32_t*)(ws + L.status),
                     (uint32_t)L.n, (uint32_t)L.tiles, (uint64_t)L.total, (uint32_t)L.cap, (uint2*)(ws + L.ranges));
}

void launch_preprocess(const SurfelArgs& s, const CamTable& ct, int mode, bool opacity_foot, bool lowpass,
                       const Layout& L, char* ws, hipStream_t st) {
  if (L.n == 0) return;
  hipLaunchKernelGGL(k_preprocess, dim3((unsigned)cdiv(L.n, 256)), dim3(256), 0, st, L.n, s.means, s.scales,
                     s.quats, s.opacity, s.rgb, ct, mode, opacity_foot ? 1 : 0, lowpass ? 1 : 0, (WalkRec*)(ws + L.rec),
                     (float4*)(ws + L.fp),
                     (uint32_t*)(ws + L.key0), (uint32_t*)(ws + L.id0), (uint32_t*)(ws + L.count),
                     (int32_t*)(ws + L.cull));
}

void launch_count_culls(const Layout& L, char* ws, hipStream_t st) {
  uint32_t* status = (uint32_t*)(ws + L.status);
  static_assert(kStCull == kStVisible + 1, "the visible count and the cull codes are cleared together");
  launch_fill_u32(status + kStVisible, 0u, 6, st);
  if (L.n == 0) return;
  hipLaunchKernelGGL(k_count_culls, dim3((unsigned)std::min<int64_t>(256, cdiv(L.n, 256))), dim3(256), 0, st, L.n,
                     (const int32_t*)(ws + L.cull), status);
}

void launch_scan_counts(const Layout& L, char* ws, hipStream_t st) {
  const int64_t nb = std::max<int64_t>(cdiv(L.n, kScanTile), 1);
  const uint32_t* order = (const uint32_t*)(ws + L.id0);
  const uint32_t* count = (const uint32_t*)(ws + L.count);
  uint64_t* bsum = (uint64_t*)(ws + L.bsum);
  hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kScanThreads), 0, st, L.n, order, count, bsum);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, st, nb, bsum, L.cap, (uint32_t*)(ws + L.status));
  hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kScanThreads), 0, st, L.n, order, count,
                     (const uint64_t*)bsum, (uint32_t*)(ws + L.offs));
}

void launch_emit(const CamTable& ct, int mode, bool lowpass, const Layout& L, char* ws, hipStream_t st) {
  if (L.n == 0) return;
  hipLaunchKernelGGL(k_emit, dim3((unsigned)cdiv(L.n, 256)), dim3(256), 0, st, L.n,
                     (const uint32_t*)(ws + L.id0), (const uint32_t*)(ws + L.count),
                     (const uint32_t*)(ws + L.offs), (const float4*)(ws + L.fp), (const WalkRec*)(ws + L.rec), lowpass ? 1 : 0,
                     ct, mode, L.cap,
                     (uint32_t*)(ws + L.vbase), (uint32_t*)(ws + L.ptile0), (uint32_t*)(ws + L.eid0),
                     (uint32_t*)(ws + L.sid_emit));
}

void launch_export_keys(const Layout& L, char* ws, int32_t* cull, uint32_t* depth, int32_t* count, hipStream_t st) {
  if (L.n == 0 || (!cull && !depth && !count)) return;
  hipLaunchKernelGGL(k_export_keys, dim3((unsigned)cdiv(L.n, 256)), dim3(256), 0, st, L.n,
                     (const int32_t*)(ws + L.cull), (const uint32_t*)(ws + L.key0), (const uint32_t*)(ws + L.id0),
                     (const uint32_t*)(ws + L.count), cull, depth, count);
}

void launch_ranges(const Layout& L, char* ws, hipStream_t st) {
  const int slots = stat_slots(L);
  if (L.cap == 0) {
    launch_fill_u32(ws + L.hist, 0u, (int64_t)slots * kStatLine * 2, st);
    return;
  }
  hipLaunchKernelGGL(k_finalize_pairs, dim3((unsigned)cdiv(L.cap, 256)), dim3(256), 0, st,
                     (const uint32_t*)(ws + L.ptile0), (const uint32_t*)(ws + L.eid0),
                     (const uint32_t*)(ws + L.sid_emit), (const uint32_t*)(ws + L.status), (uint32_t*)(ws + L.pid),
                     (uint2*)(ws + L.ranges), (uint64_t*)(ws + L.hist), (uint32_t)slots);
}

void launch_tile_order(const Layout& L, char* ws, hipStream_t st) {
  if (L.tiles == 0) return;
  hipLaunchKernelGGL(k_tile_order, dim3(1), dim3(1024), 0, st, (int)L.tiles, (const uint2*)(ws + L.ranges),
                     (uint32_t*)(ws + L.torder0));
}

}  // namespace psm
