// Shared definitions of the gfx950 rasterizer: constants, workspace layout,
// the per-surfel walk record and the per-pixel ray/surfel evaluation used by
// both the forward and the backward walk (so both take identical decisions).
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace psm {

// ----------------------------------------------------------------- constants
// Cutoff r = 3 in tangent units ("3 sigma", Sec. 5), applied per pixel.
constexpr float kCut = 3.0f;
// Footprint radius^2 = 9 (1 + 2^-10): a superset of the FP32 per-pixel test.
constexpr float kFoot2 = 9.0087890625f;
// Low-pass filter disk in the footprint: radius^2 = foot2 / 2 + 1/16 about the
// FP32 projected centre (the pad covers that centre's rounding).
constexpr float kLpPad = 0.0625f;
// Thresholds the paper leaves to the 3DGS conventions.
constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kAlphaMax = 0.99f;
constexpr float kTMin = 1e-4f;

// A tile has kTilePix = 256 pixels, one per thread of a 4-wave block: tw x th
// pixels with tw in {8, 16, 32, 64} (a launch choice, 16 x 16 by default).
// Wave w owns a sub-tile of 8 x 8 pixels (16 x 4 in a 64 x 4 tile), the
// sub-tiles row-major in the tile and the pixels row-major in the sub-tile: a
// compact sub-tile meets fewer of the tile's surfels than 16 x 4 rows do.  (The
// backward walk's waves own rows: the order of its sums is fixed.)
constexpr int kTilePix = 256;
constexpr int kTileDefault = 16;
constexpr int kMaxK = 32;

enum : int { kSphere = 0, kAabb = 1, kEllipse = 2 };
enum : int { kFull = 0, kTopK = 1 };
enum : int { kF32 = 0, kF16 = 1, kBF16 = 2 };

// Status words kept in the workspace (uint32 each).
enum : int {
  kStP = 0,        // pairs emitted (min(required, capacity))
  kStOverflow = 1, // 1 if required > capacity
  kStN = 2,        // number of virtual surfels
  kStVisible = 3,  // written by the stats read-back
  kStCull = 4,     // 4 .. 8: cull codes 0..4, written by the stats read-back
  kStTiles = 9,    // number of tiles (length of the tile work order)
  kStReqLo = 10,   // required pairs, 64-bit
  kStReqHi = 11,
  // walk counters, 64-bit, written by the stats read-back from the walk's slots
  kStWalked = 12,  // pixel x list-entry evaluations of the forward walk
  kStBlended = 14, // blended (pixel, surfel) pairs
  kStWide = 20,    // tiles the Top-K blend left to its windowed pass
  kStSigCap = 21,  // layout the forward ran with: pair capacity, tiles, total bytes (64-bit)
  kStSigTiles = 22,
  kStBwdEntries = 24,  // sum over pixels of n_last (list entries the backward walk must evaluate)
  kStSigLo = 26,
  kStSigHi = 27,
  kStUnique = 28,  // 64-bit, written by the stats read-back: distinct selected virtual surfels
  kStSelected = 30,  // 64-bit, written by the stats read-back: (pixel, slot) selections
  kStSelPairs = 32,  // 64-bit, written by the stats read-back: (tile, surfel) pairs with a selection
  kStHeavy = 34,     // backward: surfels with more than kHeavyRows flagged rows (length of their list)
  kStWords = 36
};
// Words updated by 64-bit atomics must be 8-byte aligned (a misaligned atomic
// is a memory violation); the status block itself starts the workspace.
static_assert(kStReqLo % 2 == 0 && kStWalked % 2 == 0 && kStBlended % 2 == 0 && kStBwdEntries % 2 == 0 &&
                  kStUnique % 2 == 0 && kStSelected % 2 == 0 && kStSelPairs % 2 == 0 && kStSigLo % 2 == 0,
              "64-bit status words sit at even word indices");
// Radix sort tiling.
// Surfels with more flagged feature-gradient rows than this (over all
// cameras) have them summed by a block of their own rather than a lane group.
constexpr int kHeavyRows = 64;

constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;
// Count-scan tiling.
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ----------------------------------------------------------------- cameras
constexpr int kMaxCams = 8;

struct CamArgs {
  float R[9], t[3], fx, fy, cx, cy, near_plane;
  int W, H;
};

// The cameras of one call, passed to kernels by value.  Surfel i seen by
// camera b is the virtual surfel v = b * N + i; camera b's tiles are the
// global tiles [tile0[b], tile0[b + 1]) and its images start at pixel
// pix0[b] of the concatenated output maps.
struct CamTable {
  int n;
  int64_t nsurf;
  int tw, th, tsh;  // tile width and height in pixels (tw * th = 256), log2(tw)
  int ssh;          // log2 of the sub-tile width
  CamArgs cam[kMaxCams];
  int ntx[kMaxCams], nty[kMaxCams];
  int tile0[kMaxCams + 1];
  int64_t pix0[kMaxCams + 1];
};

// Tile-local column and row of pixel p (0..255) of a tile.
__host__ __device__ inline int tile_lx(const CamTable& ct, int p) {
  return (p & ((1 << ct.ssh) - 1)) + (((p >> 6) & ((1 << (ct.tsh - ct.ssh)) - 1)) << ct.ssh);
}
__host__ __device__ inline int tile_ly(const CamTable& ct, int p) {
  return ((p & 63) >> ct.ssh) + (((p >> 6) >> (ct.tsh - ct.ssh)) << (6 - ct.ssh));
}

// The same the other way: the index of the tile-local pixel (lx, ly).
__host__ __device__ inline int tile_index(const CamTable& ct, int lx, int ly) {
  const int sx = lx >> ct.ssh, sy = ly >> (6 - ct.ssh);
  return 64 * (sx + (sy << (ct.tsh - ct.ssh))) + (lx & ((1 << ct.ssh) - 1)) +
         ((ly & ((64 >> ct.ssh) - 1)) << ct.ssh);
}

// Where global tile g lies: its camera, tile coordinates and image.
struct TileLoc {
  int b, tx, ty, W, H;
  int64_t pix0;  // first pixel of the camera's images
  int64_t v0;    // first virtual surfel of the camera
};

// Camera of virtual surfel v (no 64-bit division).
__host__ __device__ inline int camera_of(const CamTable& ct, int64_t v) {
  int b = 0;
#pragma unroll
  for (int k = 1; k < kMaxCams; ++k) b += (k < ct.n && v >= (int64_t)k * ct.nsurf) ? 1 : 0;
  return b;
}

__host__ __device__ inline TileLoc locate(const CamTable& ct, int g) {
  int b = 0;
#pragma unroll
  for (int k = 1; k < kMaxCams; ++k) b += (k < ct.n && g >= ct.tile0[k]) ? 1 : 0;
  const int lt = g - ct.tile0[b];
  TileLoc t;
  t.b = b;
  t.tx = lt % ct.ntx[b];
  t.ty = lt / ct.ntx[b];
  t.W = ct.cam[b].W;
  t.H = ct.cam[b].H;
  t.pix0 = ct.pix0[b];
  t.v0 = (int64_t)b * ct.nsurf;
  return t;
}

// ---------------------------------------------------------- workspace layout
struct Layout {
  int64_t n, nreal, cap, tiles, spix;  // n = virtual surfels; spix = tiles * 256 (tile-major pixels)
  int k, c, ncam;
  size_t rec, fp, key0, key1, id0, id1, vbase, count, offs, cull, ptile0, ptile1, eid0, eid1, sid_emit, pid, ranges,
      torder0, wide, nlast, tfinal, selpos, selw, seldot, gflag, fflag, gpart, fpart, hist, bsum, ubits, heavy, hbits,
      status, total;
};

inline Layout make_layout(const CamTable& ct, int k, int c, int64_t cap) {
  Layout L{};
  L.nreal = ct.nsurf;
  L.ncam = ct.n;
  L.n = ct.nsurf * ct.n;
  L.cap = cap;
  L.k = k;
  L.c = c;
  L.tiles = ct.tile0[ct.n];
  L.spix = L.tiles * kTilePix;
  const int64_t n1 = L.n > 0 ? L.n : 1, cap1 = cap > 0 ? cap : 1, t1 = L.tiles > 0 ? L.tiles : 1;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = align256(o + bytes); return at; };
  L.status = take(kStWords * 4);  // first, so a read-back can check the layout before any other access
  L.rec = take(n1 * 128);         // walk record and the walks' culling record
  L.fp = take(n1 * 32);           // footprint of the tile lists, 8 floats
  L.key0 = take(n1 * 4);          // depth keys (sort ping-pong)
  L.key1 = take(n1 * 4);
  L.id0 = take(n1 * 4);           // virtual surfel ids (sort ping-pong)
  L.id1 = take(n1 * 4);
  L.vbase = take(n1 * 4);         // first emitted pair of each virtual surfel
  L.count = take(n1 * 4);         // pairs per virtual surfel
  L.offs = take((n1 + 1) * 4);    // exclusive scan of counts in depth order
  L.cull = take(n1 * 4);
  L.ptile0 = take(cap1 * 4);      // pair tile ids (sort keys, ping-pong)
  L.ptile1 = take(cap1 * 4);
  L.eid0 = take(cap1 * 4);        // pair emission index (sort values, ping-pong)
  L.eid1 = take(cap1 * 4);
  L.sid_emit = take(cap1 * 4);    // virtual surfel id of each emitted pair
  L.pid = take(cap1 * 4);         // virtual surfel id of each sorted pair
  L.ranges = take(t1 * 8);        // [start, end) per tile
  L.torder0 = take(t1 * 4);       // tile work order, longest lists first
  L.wide = take(t1 * 4);          // tiles of the Top-K blend's windowed pass
  L.nlast = take(L.spix * 4);
  L.tfinal = take(L.spix * 4);
  L.selpos = take(L.spix * (size_t)k * 4);
  L.selw = take(L.spix * (size_t)k * 4);
  L.seldot = take(L.spix * (size_t)k * 4);
  // backward partial sums per (tile, surfel) pair, at the pair's emission index
  L.gflag = take(cap1);
  L.fflag = take(cap1);
  L.gpart = take(cap1 * 64);      // 16 floats: geometric and colour terms
  L.fpart = take(cap1 * (size_t)(c > 0 ? c : 1) * 4);  // feature gradient rows
  int64_t big = n1 > cap1 ? n1 : cap1;
  big = big > t1 ? big : t1;
  const int64_t nb = cdiv(big, kSortTile);
  L.hist = take((256 * nb + 256) * 4);
  L.bsum = take((cdiv(n1, kScanTile) + 1) * 8);
  L.ubits = take(cdiv(n1, 32) * 4);  // one bit per virtual surfel: selected somewhere (stats read-back)
  // surfels with more than kHeavyRows flagged rows: the rows are pairs, whose
  // ranges are disjoint inside the capacity, so at most cap / (kHeavyRows + 1)
  L.heavy = take((cap1 / (kHeavyRows + 1) + 1) * 4);
  // in the backward, a bit per surfel: its pairs are summed by a block of its
  // own.  In the depth sort's second buffer, which nothing reads after the sort
  // (not with the read-back's bits: it may run beside a backward)
  L.hbits = L.key1;
  L.total = o;
  return L;
}

// Walk counters: every wave of the forward walk adds its three sums (entries
// walked, contributors, entries up to the last contributor) to one of
// stat_slots 128-byte lines, and the stats read-back adds up the lines.  One
// shared line took 9 ns per addition whatever the walk did: 0.88 of 0.90 ms
// for the 98k additions of a 1080p frame.  The lines are the sort's histogram
// area, which is free once the pairs are sorted (16 lines at least).
constexpr int kStatLine = 16;  // 64-bit words per line
__host__ __device__ inline int stat_slots(const Layout& L) {
  const int64_t lines = (int64_t)((L.bsum - L.hist) / (8 * kStatLine));
  return lines >= 256 ? 256 : (lines >= 64 ? 64 : 16);
}

// Initial value of status word i of a forward.
__device__ inline uint32_t init_word(uint32_t i, uint32_t n, uint32_t tiles, uint64_t total, uint32_t cap) {
  uint32_t v = 0u;
  v = i == kStN ? n : v;
  v = i == kStTiles ? tiles : v;
  v = i == kStSigLo ? (uint32_t)total : v;
  v = i == kStSigHi ? (uint32_t)(total >> 32) : v;
  v = i == kStSigCap ? cap : v;
  v = i == kStSigTiles ? tiles : v;
  return v;
}

// The pairs the frame needs: required (64-bit), emitted, overflow.
__device__ inline void write_pair_total(uint32_t* status, uint64_t total, uint64_t cap) {
  status[kStReqLo] = (uint32_t)total;
  status[kStReqHi] = (uint32_t)(total >> 32);
  status[kStP] = (uint32_t)(total < cap ? total : cap);
  status[kStOverflow] = total > cap ? 1u : 0u;
}

// ------------------------------------------------------------ walk record
// Sub-tile culling of the walks: a wave skips a surfel no pixel centre of its
// pixels can blend.  Per surfel the key stage keeps the ellipse of
// rho <= min(9, 2 ln(255 o)) (beyond it alpha < 1/255), widened like the
// footprint, as centre (ecx, ecy), half-extents (ex, ey), the y offset of the
// rightmost point yr, the slope of the chord midpoints and the half-chord
// factor, so its x-extent over the rows [y0, y1] of the wave is two
// clamps and two square roots.  One lane tests one list entry, so a test
// costs each pixel 1/64 of that.  The ellipse comes from the same FP64
// projection as the walk record, so it is the hit test's own; the slack
// covers the rounding of the record to FP32 and the FP32 test (relative 2^-16
// of the extents: a thin ellipse's chord is a difference of terms of the size
// of its extents).  With the low-pass filter the record is the box of the
// ellipse and the filter's disk.
struct CullRec {
  float4 e0;  // ecx, ecy, ex, ey
  float4 e1;  // yr, slope, half-chord factor, slack (low-pass: xc, yc, rf2, slack)
};

// Walk record per surfel, computed in FP64 from the FP32 inputs:
//   d0 = (Ai00, Ai01), d1 = (Ai10, Ai11)   FP64: inverse of A, the centred,
//                                          depth-normalised homography [[A,0],[p q 1]]
//   d2 = (e0, e1)                          FP64: e = (p, q) A^-1
//   d3 = (xc, yc)                          FP64: projected surfel centre
//   f0 = (mz, o, r, g), f1 = (b, n0, n1, n2)  FP32
// For a pixel offset d = (x - xc, y - yc):  u' = A^-1 d, w' = 1 - e.d,
// (u, v) = u'/w', intersection depth z = mz / w'.
//
// The solve is FP64: for a surfel seen at a grazing angle A is ill-conditioned
// and an FP32 evaluation of u' loses eps * cond(A) relative accuracy (1e-4 in
// rho at cond(A) ~ 100), far beyond the 1e-5 image tolerance; FP32 pixel
// coordinates near 10^3 would also carry 6e-5 px of rounding.

// It shares its 128-byte line with the culling record, which a wave reads a
// chunk of entries ahead: the line is then in the XCD's L2 when the entry's
// turn comes and its scalar load is one entry ahead.  (Apart, a record's first
// read by an XCD came from beyond L2, some 2000 cycles, the walks' largest
// wait.)
struct __align__(128) WalkRec {
  double2 d0, d1, d2, d3;
  float4 f0, f1;
  CullRec c;
};
static_assert(sizeof(WalkRec) == 128, "a record is a cache line");

// The record as the per-pixel evaluation takes it.
struct LRec {
  double a00, a01, a10, a11, e0, e1, xc, yc;
  float mz, o, r, g, b, n0, n1, n2;
};

// Walk record by a wave-uniform surfel id through the scalar cache: 24 words
// in scalar registers, which the per-pixel arithmetic takes as operands, so an
// entry costs no LDS traffic and no vector registers.  (The records are
// written by an earlier kernel: nothing in a walk writes them.)
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
struct SRec {
  u32x16 a;
  u32x8 b;
  __device__ __forceinline__ LRec get() const {
    LRec s;
    auto d = [](uint32_t lo, uint32_t hi) { return __hiloint2double((int)hi, (int)lo); };
    s.a00 = d(a[0], a[1]); s.a01 = d(a[2], a[3]); s.a10 = d(a[4], a[5]); s.a11 = d(a[6], a[7]);
    s.e0 = d(a[8], a[9]); s.e1 = d(a[10], a[11]); s.xc = d(a[12], a[13]); s.yc = d(a[14], a[15]);
    s.mz = __uint_as_float(b[0]); s.o = __uint_as_float(b[1]); s.r = __uint_as_float(b[2]); s.g = __uint_as_float(b[3]);
    s.b = __uint_as_float(b[4]); s.n0 = __uint_as_float(b[5]); s.n1 = __uint_as_float(b[6]); s.n2 = __uint_as_float(b[7]);
    return s;
  }
};
__device__ __forceinline__ SRec load_rec(const WalkRec* rec, uint32_t id) {
  const uint64_t p = (uint64_t)rec + (uint64_t)id * sizeof(WalkRec);
  SRec r;
  r.a = *(const __attribute__((address_space(4))) u32x16*)p;
  r.b = *(const __attribute__((address_space(4))) u32x8*)(p + 64);
  return r;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// LDS staging of a batch of records (structure of arrays, so a batch is
// written with consecutive addresses and read by broadcast).
template <int B>
struct Staged {
  double2 a0[B], a1[B], e[B], o[B];
  float4 f0[B], f1[B];

  __device__ __forceinline__ void put(int slot, const WalkRec& r) {
    a0[slot] = r.d0;
    a1[slot] = r.d1;
    e[slot] = r.d2;
    o[slot] = r.d3;
    f0[slot] = r.f0;
    f1[slot] = r.f1;
  }
  __device__ __forceinline__ LRec get(int k) const {
    LRec s;
    const double2 x0 = a0[k], x1 = a1[k], x2 = e[k], x3 = o[k];
    const float4 y0 = f0[k], y1 = f1[k];
    s.a00 = x0.x; s.a01 = x0.y; s.a10 = x1.x; s.a11 = x1.y;
    s.e0 = x2.x; s.e1 = x2.y; s.xc = x3.x; s.yc = x3.y;
    s.mz = y0.x; s.o = y0.y; s.r = y0.z; s.g = y0.w;
    s.b = y1.x; s.n0 = y1.y; s.n1 = y1.z; s.n2 = y1.w;
    return s;
  }
};

// Per-pixel evaluation of one surfel (Sec. 3.1): the intersection (u, v) of
// the pixel ray with the surfel plane, rho = u^2 + v^2, hit iff rho <= 9,
// alpha = min(0.99, o exp(-rho/2)).  Returns true for a contributor
// (hit and alpha >= 1/255).  The hit decision is taken in FP64; rho, alpha
// and the values handed on are FP32.
//
// LP: the optional screen-space low-pass filter (the 2DGS variant),
// rho = min(u^2 + v^2, 2 |d|^2) with d the pixel's offset from the projected
// centre; the term is chosen in FP64, ties to the ray-splat term.  Where the
// filter term is taken (filt), u = v = 0 and iw = 1, so the depth mz * iw is
// the centre's depth.
struct PixEval {
  float dx, dy, u, v, iw, G, alpha;
  bool clamped, filt;
};

// Evaluated without branches: a wave reaches it with entries that meet its
// pixels, of which nearly every one has a pixel that hits.  A pixel that
// has stopped passes x = NaN, which fails the hit test.  EARLY: leave at the
// hit test, for a walk that takes every entry of the tile (most have no pixel
// of the wave).
template <bool LP = false, bool EARLY = false>
__device__ __forceinline__ bool eval_pixel(const LRec& s, double x, double y, PixEval& e) {
  const double dx = x - s.xc, dy = y - s.yc;
  const double u1 = fma(s.a00, dx, s.a01 * dy);
  const double v1 = fma(s.a10, dx, s.a11 * dy);
  const double w1 = 1.0 - fma(s.e0, dx, s.e1 * dy);
  const double num = fma(u1, u1, v1 * v1), w2 = w1 * w1;
  bool hit = (w1 > 0.0) & (num <= 9.0 * w2);
  if (EARLY && !LP && !hit) return false;
  e.filt = false;
  e.dx = (float)dx;
  e.dy = (float)dy;
  e.iw = __builtin_amdgcn_rcpf((float)w1);
  e.u = (float)u1 * e.iw;
  e.v = (float)v1 * e.iw;
  float rho = fmaf(e.u, e.u, e.v * e.v);
  if constexpr (LP) {
    const double rf = 2.0 * fma(dx, dx, dy * dy);
    const bool splat = (w1 > 0.0) & (num <= rf * w2);
    hit = splat ? num <= 9.0 * w2 : rf <= 9.0;
    if (EARLY && !hit) return false;
    e.filt = !splat;
    e.iw = splat ? e.iw : 1.0f;
    e.u = splat ? e.u : 0.0f;
    e.v = splat ? e.v : 0.0f;
    rho = splat ? rho : 2.0f * fmaf(e.dx, e.dx, e.dy * e.dy);
  }
  e.G = __builtin_amdgcn_exp2f(rho * -0.72134752044448170f);  // exp(-rho/2)
  const float oG = s.o * e.G;
  e.clamped = oG > kAlphaMax;
  e.alpha = e.clamped ? kAlphaMax : oG;
  return hit & (e.alpha >= kAlphaMin);
}

template <bool LP>
__device__ __forceinline__ bool rect_meets(const CullRec& c, float x0, float x1, float y0, float y1) {
  const float sl = c.e1.w, ey = c.e0.w;
  const float lo = fmaxf((y0 - c.e0.y) - sl, -ey), hi = fminf((y1 - c.e0.y) + sl, ey);
  float xl, xr;
  if constexpr (LP) {
    xl = c.e0.x - c.e0.z;
    xr = c.e0.x + c.e0.z;
  } else {
    const float dr = fminf(fmaxf(c.e1.x, lo), hi), dl = fminf(fmaxf(-c.e1.x, lo), hi);
    const float s2 = ey * ey;
    xr = c.e0.x + (c.e1.y * dr + c.e1.z * __builtin_amdgcn_sqrtf(fmaxf(0.0f, s2 - dr * dr)));
    xl = c.e0.x + (c.e1.y * dl - c.e1.z * __builtin_amdgcn_sqrtf(fmaxf(0.0f, s2 - dl * dl)));
  }
  return !(lo > hi) && !(xr + sl < x0) && !(xl - sl > x1);
}

// Pixel centres of a wave's sub-tile (pixels past the image included).
struct SubRect {
  float x0, x1, y0, y1;
};
__device__ __forceinline__ SubRect sub_rect(const CamTable& ct, const TileLoc& tl, int wave) {
  SubRect r;
  r.x0 = (float)(tl.tx * ct.tw + tile_lx(ct, 64 * wave)) + 0.5f;
  r.y0 = (float)(tl.ty * ct.th + tile_ly(ct, 64 * wave)) + 0.5f;
  r.x1 = r.x0 + (float)((1 << ct.ssh) - 1);
  r.y1 = r.y0 + (float)((64 >> ct.ssh) - 1);
  return r;
}

// Tile index of a block: consecutive block ids are dispatched round-robin
// over the 8 XCDs, so give each XCD a contiguous run of tiles (neighbouring
// tiles share surfels, and each XCD has its own L2).
__device__ inline int xcd_tile(int bid, int tiles) {
  const int per = (tiles + 7) >> 3;
  return (bid & 7) * per + (bid >> 3);
}
inline int xcd_grid(int64_t tiles) { return (int)(((tiles + 7) >> 3) << 3); }

// Tile scheduling of the per-tile kernels, one block per tile.  order == null:
// neighbouring tiles on one XCD.  Otherwise block i takes tile order[i], the
// tiles of the longest lists first: blocks are dispatched in index order as
// others finish, so long tiles start early and short ones fill the gaps, with
// no queue and no loop over tiles in the kernel (a resident grid taking tiles
// from an atomic queue kept its arguments live across that loop: 80 spilled
// scalar registers in the forward walk, and two barriers per tile).
struct TileOrder {
  const uint32_t* order;
  int tiles;
};

template <class F>
__device__ __forceinline__ void with_tile(const TileOrder& q, F&& body) {
  const int b = (int)blockIdx.x;
  const int tile = q.order ? b : xcd_tile(b, q.tiles);
  if (tile < q.tiles) body(q.order ? (int)q.order[tile] : tile);
}

// ------------------------------------------------------------ wave helpers
// Cross-lane exchanges without LDS: v_permlane32_swap / v_permlane16_swap
// (gfx950) exchange halves of the wave / of 32-lane halves between two
// registers, DPP row operations pair lanes inside a 16-lane row.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
constexpr int kDppRowRor8 = 0x128;      // lane l <- lane l ^ 8 within a row
constexpr int kDppRowRor4 = 0x124;      // lane l <- lane l - 4 within a row

// x + x(lane ^ 32) (first) and y + y(lane ^ 32) (second), for the lanes whose
// bit 5 selects x (lanes 0-31) or y (lanes 32-63).
__device__ __forceinline__ float swap32_add(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_add(float x, float y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS ordering between the lanes of one wave (no block barrier involved).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Four lane groups hold four channels each (group k: channels 4 k ..); after
// this, component s of every group k is channel 4 s + k: four matrix steps of
// four channels in order, from one 16-byte load a lane.  (The order matters:
// the geometric chain of surfels seen edge-on amplifies a dot's rounding.)
__device__ __forceinline__ float4 by_step(float4 v) {
  const auto u = [](float x) { return __float_as_uint(x); };
  const auto a = __builtin_amdgcn_permlane32_swap(u(v.x), u(v.z), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(u(v.y), u(v.w), false, false);
  const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  return make_float4(__uint_as_float(c[0]), __uint_as_float(c[1]), __uint_as_float(d[0]), __uint_as_float(d[1]));
}

// FP32 matrix-core product on a 16 x 16 tile, k = 4 (v_mfma_f32_16x16x4f32):
// lane l supplies A[l & 15][l >> 4] and B[l >> 4][l & 15] and holds
// D[4 (l >> 4) + r][l & 15] in component r.  Products are exact and summed in
// FP32 in a fixed order, so a sequence of these is deterministic.
typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4v mfma_16x16x4(float a, float b, f4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ------------------------------------------------ feature loads (to float)
// Storage types: float, __half, and uint16_t holding bf16 bits.
template <typename FT>
__device__ __forceinline__ float load_one(const FT* p);
template <>
__device__ __forceinline__ float load_one<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float load_one<__half>(const __half* p) { return __half2float(*p); }
template <>
__device__ __forceinline__ float load_one<uint16_t>(const uint16_t* p) {
  return __uint_as_float(((uint32_t)*p) << 16);
}

// Four consecutive feature channels as float.
template <typename FT>
__device__ __forceinline__ float4 load4(const FT* p);
template <>
__device__ __forceinline__ float4 load4<float>(const float* p) {
  return *reinterpret_cast<const float4*>(p);
}
template <>
__device__ __forceinline__ float4 load4<__half>(const __half* p) {
  const uint2 x = *reinterpret_cast<const uint2*>(p);
  return make_float4(__half2float(__ushort_as_half((unsigned short)(x.x & 0xFFFF))),
                     __half2float(__ushort_as_half((unsigned short)(x.x >> 16))),
                     __half2float(__ushort_as_half((unsigned short)(x.y & 0xFFFF))),
                     __half2float(__ushort_as_half((unsigned short)(x.y >> 16))));
}
template <>
__device__ __forceinline__ float4 load4<uint16_t>(const uint16_t* p) {
  const uint2 x = *reinterpret_cast<const uint2*>(p);
  return make_float4(__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xFFFF0000u), __uint_as_float(x.y << 16),
                     __uint_as_float(x.y & 0xFFFF0000u));
}

// The feature rows a render blends: channels [0, ca) from a (storage type FT,
// row stride ca) and channels [ca, ca + cb) from b (FP32, row stride cb; the
// second source is optional: cb = 0).  Both widths are multiples of 8, so a
// group of 4 channels starting at a multiple of 4 lies in one source.
template <typename FT>
struct FeatSrc {
  const FT* a;
  const float* b;
  int ca, cb;
  __device__ __forceinline__ float4 load4(size_t row, int c) const {
    return c < ca ? psm::load4<FT>(a + row * ca + c) : psm::load4<float>(b + row * cb + (c - ca));
  }
  __device__ __forceinline__ float load1(size_t row, int c) const {
    return c < ca ? load_one<FT>(a + row * ca + c) : b[row * cb + (c - ca)];
  }
};

}  // namespace psm
