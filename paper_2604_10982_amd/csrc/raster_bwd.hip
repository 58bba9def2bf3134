// Backward of the renderer: gradients of L = <upstream, outputs> with respect
// to every surfel parameter.  The selection (eq. (18)), the contributor set,
// the stop point and the alpha clamp are held fixed.
//
// Deterministic and free of floating-point atomics: every (tile, surfel) pair
// owns a slot for its partial sums at the index where the key stage emitted
// it, so a surfel's pairs are contiguous and a per-surfel pass adds them in
// a fixed order (emission order).
//
// k_feat_bwd_topk: per tile, for every (pixel, selected surfel): the dot
//   product of the pixel's feature gradient with the surfel's feature row
//   (needed by the alpha adjoint); and, per distinct selected surfel of the
//   tile, the row sum_p w_p g_F(p) over the pixels that selected it, in pixel
//   order.
// k_walk_bwd: per tile, back to front from each pixel's last contributor,
//   recovering T_i = T_{i+1} / (1 - alpha_i).  Per surfel the per-pixel terms
//   are summed over the wave by small matrix products, then over the 4 waves
//   through LDS, and written as the pair's 16 partial sums.  In dense-blend mode each batch also forms
//   the feature dot products and feature-gradient rows tile-wide.
// k_reduce_geo / k_reduce_feat (and their _heavy forms for surfels with many
//   pairs): per surfel, sum of its pairs' partials, then
//   the chain rule to mu, s, q (FP64, as the forward's walk record).
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "select.h"

namespace psm {

constexpr int kBB = 32;          // surfels per backward batch

// ------------------------------------------------------------ Top-K feature
// Per tile, the distinct selected surfels of the tile (a few dozen: each is
// chosen by about a hundred of the 256 pixels for K = 16) get slots in list
// order, 48 per chunk.  With G = the pixels' feature gradients (256 x C),
// F = the slots' feature rows and W = the selection weights (pixel x slot,
// zero where the pixel did not select the slot), the adjoint needs
//   dots = G F^T  at the selected (pixel, slot) entries   (alpha adjoint)
//   rows = W^T G                                           (feature gradient)
// and the weight matrix of a tile is dense enough (about half its entries)
// that both run as dense FP32 matrix-core products.
//
// Eight waves, 32 pixels each: a wave's dots and weight operands then take 48
// registers for 48 slots, and four waves fit on a SIMD (with four waves of 64
// pixels and 64 slots it was two, and half of the time no wave had an
// instruction ready; 64 slots for eight waves spill inside the passes: 945
// against 832 us, and 32 slots read G more often).
// Both operands of the dots come straight from memory, 4 channels a lane, and
// are put in step order by lane swaps; G goes through the wave's own LDS slab only to be read with pixels
// along the contraction.  So a pass of 16 channels has one block barrier,
// before the sum of the waves' partial rows (in wave order; two buffers).  Weights and dots
// cross between a pixel's selections and the matrix layout through the same
// slab, 16 slots at a time.  Every sum has a fixed order.
// 1080p, K = 16: 1M plane surfels, C = 128: 1065 -> 826 us; 1M street surfels,
// C = 256 (bf16): 1680 -> 1293 us.  Of the 826: 330 the slots and operands of
// the tiles with one pass, the matrix products about 300, waiting for G 80.
constexpr int kFbSlots = 48;                  // slots per chunk: 3 blocks of 16
constexpr int kFbThreads = 512;
constexpr int kFbWaves = kFbThreads / 64;
constexpr int kFbPix = kTilePix / kFbWaves;   // pixels per wave
constexpr int kFbPass = 16;                   // channels per pass
constexpr int kFbPart = kFbWaves * kFbSlots * kFbPass;  // partial rows of a pass
// Slab strides in floats: rows of G 4 apart are 16 banks apart (one step's
// four pixels); a slot's 32 pixels at 37, so that 16 slots spread over the banks.
constexpr int kFbGS = 20, kFbWS = 37;
static_assert(kFbPix == 32 && 16 * kFbWS + kFbPix <= kFbPix * kFbGS, "slab");

// Keeps what is derived from v from being formed before this point (and held
// in registers through the products).
__device__ __forceinline__ uint32_t formed_here(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// SPLIT: features in two arrays.
template <typename FT, int KMAX, bool SPLIT>
__global__ __launch_bounds__(kFbThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_feat_bwd_topk(
    const uint32_t* __restrict__ pid, const uint32_t* __restrict__ eid, const uint2* __restrict__ ranges,
    const int32_t* __restrict__ selpos, const float* __restrict__ selw, const FeatSrc<FT> feat,
    const float* __restrict__ gfeat, int C, int K, CamTable ct, TileOrder tq, float* __restrict__ seldot,
    float* __restrict__ fpart, uint8_t* __restrict__ fflag, int renorm) {
  constexpr int QH = KMAX / 2;  // selections per lane: a pixel's are shared by lanes l and l + 32
  __shared__ SelShared S;
  __shared__ __align__(16) float s_slab[kFbWaves][kFbPix * kFbGS];
  __shared__ uint32_t s_fe[kFbSlots];  // emitted pair index per slot
  extern __shared__ float s_part[];    // the waves' partial rows of a pass, two passes

  with_tile(tq, [&](const int tile) {
  const TileLoc tl = locate(ct, tile);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4, pl = lane & 31;
  const uint32_t start = ranges[tile].x;
  const int q0 = (lane >> 5) * QH;
  // the tile's selections: uniform bases, this lane's first at sel0
  const size_t tbase = (size_t)tile * K * kTilePix;
  const int32_t* const spos = selpos + tbase;
  const float* const sw = selw + tbase;
  float* const sdot = seldot + tbase;
  const uint32_t sel0 = (uint32_t)(q0 * kTilePix + wave * kFbPix + pl);
  float* const slab = s_slab[wave];

  // the selection positions are re-read where needed (an L2 hit) rather
  // than held in registers through the products
  // in range also for q0 + j >= K
  auto sel_at = [&](int j) { return formed_here(sel0) + (uint32_t)(min(j, K - 1 - q0) * kTilePix); };
  auto load_pos = [&](int (&pos)[QH]) {
#pragma unroll
    for (int j = 0; j < QH; ++j) pos[j] = spos[sel_at(j)];
#pragma unroll
    for (int j = 0; j < QH; ++j) pos[j] = q0 + j < K ? pos[j] : -1;
  };
  // list positions are below the tile's list length, which bounds the
  // windows (no block-wide maximum of the selections needed)
  const int lastpos = (int)(ranges[tile].y - start) - 1;
  int Uw0 = 0;
  float rw = 1.0f;  // renormalised Top-K: 1 / (sum of the pixel's selected weights)
  {
    int pos[QH];
    load_pos(pos);
#pragma unroll
    for (int j = 0; j < QH; ++j)  // unselected entries report dot 0
      if (q0 + j < K && pos[j] < 0) sdot[sel0 + j * kTilePix] = 0.0f;
    if (renorm) {
      float wsum = 0.0f;
#pragma unroll
      for (int j = 0; j < QH; ++j) {
        const float x = sw[sel_at(j)];
        wsum += pos[j] >= 0 ? x : 0.0f;
      }
      wsum += __shfl_xor(wsum, 32, 64);
      rw = wsum > 0.0f ? 1.0f / wsum : 0.0f;
    }
    if (lastpos >= 0) Uw0 = build_window<QH, kFbThreads>(S, pos, QH, 0, window_words(lastpos, 0));
  }
  // the two pixels whose gradients this lane loads
  uint32_t gpix[2];  // ~0: outside the image
#pragma unroll
  for (int pb = 0; pb < 2; ++pb) {
    const int p = wave * kFbPix + 16 * pb + li;
    const int px = tl.tx * ct.tw + tile_lx(ct, p), py = tl.ty * ct.th + tile_ly(ct, p);
    gpix[pb] = px < tl.W && py < tl.H ? (uint32_t)(tl.pix0 + (int64_t)py * tl.W + px) : ~0u;
  }
  for (int w0 = 0; w0 <= lastpos; w0 += kWinPos) {
    const int nw = window_words(lastpos, w0);
    int Uw = Uw0;
    if (w0 > 0) {
      int pos[QH];
      load_pos(pos);
      Uw = build_window<QH, kFbThreads>(S, pos, QH, w0, nw);
    }
    for (int c0 = 0; c0 < Uw; c0 += kFbSlots) {
      const int ns = min(kFbSlots, Uw - c0), nb = (ns + 15) >> 4;
      uint32_t sl[QH / 4];  // slot of each selection, a byte each: 255 = not in this chunk
#pragma unroll
      for (int j = 0; j < QH / 4; ++j) sl[j] = 0u;
      {
        int pos[QH];
        load_pos(pos);
#pragma unroll
        for (int j = 0; j < QH; ++j) {
          const int x = slot_of(S, pos[j], w0, nw) - c0;
          const bool in = x >= 0 && x < ns;
          sl[j / 4] |= (in ? (uint32_t)x : 255u) << (8 * (j % 4));
          if (in) S.lpos[x] = (uint32_t)pos[j];  // same value from every selecting pixel
        }
      }
      __syncthreads();
      if (tid < ns) {
        const uint32_t j = start + S.lpos[tid];
        s_fe[tid] = eid[j];
        S.fid[tid] = (uint32_t)(pid[j] - tl.v0);
      }
      __syncthreads();

      auto chunk = [&](auto nb_c) {
        constexpr int NB = decltype(nb_c)::value;
        // operands of a pass: 4 channels of the lane's two pixels and of its
        // slot of each block (slots past the last read a valid row: their
        // column of the dots is not used, their weights are 0)
        uint32_t fr[NB];
#pragma unroll
        for (int sb = 0; sb < NB; ++sb) fr[sb] = S.fid[min(16 * sb + li, ns - 1)];
        float4 g[2], f[NB];
        auto load_g = [&](int cc) {
          const int c = cc + 4 * lk;
#pragma unroll
          for (int pb = 0; pb < 2; ++pb) {
            const uint32_t pix = formed_here(gpix[pb]);
            g[pb] = c < C && pix != ~0u ? *reinterpret_cast<const float4*>(gfeat + (size_t)pix * C + c)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
          }
        };
        auto load_f = [&](int cc) {
          const int c = cc + 4 * lk;
#pragma unroll
          for (int sb = 0; sb < NB; ++sb)
            f[sb] = c >= C ? make_float4(0.f, 0.f, 0.f, 0.f)
                    : SPLIT ? feat.load4(formed_here(fr[sb]), c)
                            : load4<FT>(feat.a + (size_t)formed_here(fr[sb]) * C + c);
        };
        load_g(0);
        load_f(0);
        // weights: W[p][s] at lane (s = li, lk) of step ks, pixel of the step
        // and lane group (ks & 3) + 4 lk + 16 (ks >> 2)
        float wa[NB][8];
        {
          float wq[QH];
#pragma unroll
          for (int j = 0; j < QH; ++j)
            wq[j] = sw[sel_at(j)];
#pragma unroll
          for (int sb = 0; sb < NB; ++sb) {
            const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
            reinterpret_cast<float4*>(slab)[lane] = z;
            reinterpret_cast<float4*>(slab)[64 + lane] = z;
            if (lane < 32) reinterpret_cast<float4*>(slab)[128 + lane] = z;
            wave_lds_sync();
#pragma unroll
            for (int j = 0; j < QH; ++j) {
              const uint32_t x = (sl[j / 4] >> (8 * (j % 4))) & 255u;
              slab[((x >> 4) == sb ? x & 15u : 16u) * kFbWS + pl] = wq[j];  // row 16: not read
            }
            wave_lds_sync();
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) wa[sb][ks] = slab[li * kFbWS + (ks & 3) + 4 * lk + 16 * (ks >> 2)];
            wave_lds_sync();
          }
        }
        f4v dacc[2][NB];
#pragma unroll
        for (int pb = 0; pb < 2; ++pb)
#pragma unroll
          for (int sb = 0; sb < NB; ++sb) dacc[pb][sb] = f4v{0.f, 0.f, 0.f, 0.f};
        for (int cc = 0; cc < C; cc += kFbPass) {
          float* const part = s_part + (cc / kFbPass & 1) * kFbPart;
#pragma unroll
          for (int pb = 0; pb < 2; ++pb) {
            if (renorm) {  // the rows and dots see g / W
              const float r = __shfl(rw, 16 * pb + li, 64);
              g[pb] = make_float4(g[pb].x * r, g[pb].y * r, g[pb].z * r, g[pb].w * r);
            }
            *reinterpret_cast<float4*>(slab + (16 * pb + li) * kFbGS + 4 * lk) = g[pb];
          }
          wave_lds_sync();
          float gb[8];
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) gb[ks] = slab[((ks & 3) + 4 * lk + 16 * (ks >> 2)) * kFbGS + li];
          // dots: D[p][s] += G[p][c] F[s][c], 4 channels per step
#pragma unroll
          for (int pb = 0; pb < 2; ++pb) g[pb] = by_step(g[pb]);
#pragma unroll
          for (int sb = 0; sb < NB; ++sb) f[sb] = by_step(f[sb]);
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int sb = 0; sb < NB; ++sb)
#pragma unroll
              for (int pb = 0; pb < 2; ++pb)
                dacc[pb][sb] = mfma_16x16x4((&g[pb].x)[ks], (&f[sb].x)[ks], dacc[pb][sb]);
          if (cc + kFbPass < C) load_g(cc + kFbPass);
          // rows: R[s][c] += W[p][s] G[p][c] over this wave's pixels
#pragma unroll
          for (int sb = 0; sb < NB; ++sb) {
            f4v r = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) r = mfma_16x16x4(wa[sb][ks], gb[ks], r);
            // slot 16 sb + 4 lk + i at row 16 sb + 4 i + lk: the lane groups 16 banks apart
#pragma unroll
            for (int i = 0; i < 4; ++i) part[(wave * kFbSlots + 16 * sb + 4 * i + lk) * kFbPass + li] = r[i];
          }
          if (cc + kFbPass < C) load_f(cc + kFbPass);
          __syncthreads();
          {
            const int s = tid >> 3, c = 2 * (tid & 7);
            if (s < ns && cc + c < C) {
              const float* r = part + ((s & ~15) + 4 * (s & 3) + ((s >> 2) & 3)) * kFbPass + c;
              float2 v = *reinterpret_cast<const float2*>(r);
#pragma unroll
              for (int w = 1; w < kFbWaves; ++w) {
                const float2 x = *reinterpret_cast<const float2*>(r + w * kFbSlots * kFbPass);
                v.x += x.x;
                v.y += x.y;
              }
              *reinterpret_cast<float2*>(fpart + (size_t)s_fe[s] * C + cc + c) = v;
            }
          }
        }
        // dots of the selected entries, 16 slots at a time
        uint32_t sd[QH / 4];
#pragma unroll
        for (int j = 0; j < QH / 4; ++j) sd[j] = formed_here(sl[j]);
        float dq[QH] = {};
#pragma unroll
        for (int sb = 0; sb < NB; ++sb) {
          wave_lds_sync();
#pragma unroll
          for (int pb = 0; pb < 2; ++pb)
#pragma unroll
            for (int r = 0; r < 4; ++r) slab[li * kFbWS + 16 * pb + 4 * lk + r] = dacc[pb][sb][r];
          wave_lds_sync();
#pragma unroll
          for (int j = 0; j < QH; ++j) {
            const uint32_t x = (sd[j / 4] >> (8 * (j % 4))) & 255u;
            const float d = slab[(x & 15u) * kFbWS + pl];
            dq[j] = (x >> 4) == sb ? d : dq[j];
          }
        }
#pragma unroll
        for (int j = 0; j < QH; ++j)
          if (((sd[j / 4] >> (8 * (j % 4))) & 255u) != 255u) sdot[sel_at(j)] = dq[j];
        wave_lds_sync();
      };
      switch (nb) {
        case 1: chunk(std::integral_constant<int, 1>{}); break;
        case 2: chunk(std::integral_constant<int, 2>{}); break;
        default: chunk(std::integral_constant<int, 3>{}); break;
      }
      if (tid < ns) fflag[s_fe[tid]] = 1;
      __syncthreads();
    }
  }
  // renormalised Top-K: d/dw_q of F = sum w f / W is g.(f_q - F) / W, i.e.
  // dot'_q - sum_j (w_j / W) dot'_j with dot' = (g / W) . f
  if (renorm) {
    float cshift = 0.0f;
#pragma unroll
    for (int j = 0; j < QH; ++j)
      if (q0 + j < K) {
        const uint32_t at = sel0 + j * kTilePix;
        cshift = fmaf(spos[at] >= 0 ? sw[at] : 0.0f, sdot[at], cshift);  // this lane's own store
      }
    cshift += __shfl_xor(cshift, 32, 64);
    cshift *= rw;
#pragma unroll
    for (int j = 0; j < QH; ++j)
      if (q0 + j < K) sdot[sel0 + j * kTilePix] -= cshift;
  }
  });
}

// ------------------------------------------------------------- walk backward
// A wave owns 64 consecutive pixels of the tile in row-major order (16 x 4 in a
// 16 x 16 tile), a lane one of them.
//
// The per-surfel sums of a wave's pixels as small matrix products.  Every
// term is one of a few per-pixel factors times a column of the pixel: w times
// the upstream gradients (dC, dn_c), dL/du', dL/dv', dL/dw' times (1, dx, dy)
// with (dx, dy) the pixel's offset from the surfel's centre, and two plain
// sums.  The wave puts the factors of its contributing entries (and their
// offsets) in its LDS
// slice and multiplies them by the columns on v_mfma_f32_4x4x1 (16 blocks,
// block b holding four pixels, one per step); for four entries
// together the 16 blocks are then added across lanes.  Rows of the first
// product are an entry's four geometric factors (the offset columns are the
// entry's own; formed every second entry, so that LDS holds two entries'),
// rows of the others the four entries.  Forming 17 products per pixel and
// reducing them over the wave took 65 vector instructions per entry of the 142
// the walk issued (it is bound by their issue): 1M plane surfels at 1080p,
// K = 16, 1180 -> 1050 us; 150k dense 2245 -> 1840.
//
// The order of the geometric sums is part of the result: of a surfel seen
// edge-on the chain rule takes differences of these FP32 sums, which amplifies
// their last bit by the ellipse's aspect (quaternion elements by up to a few
// 1e-3), so another order gives other gradients, no nearer to the exact ones.
// (Sums against A^-1 d instead of d would not cancel: the quaternions of a 3k
// fit are then 1.8e-7 instead of 5.8e-6 from their 64-bit values, in the same
// time, but other values than these.)  The order is a tree over the wave's 64 pixels: pixels i and i ^ 32, then ^ 16,
// ^ 8, ^ 7, ^ 2 and ^ 1, every product rounded; the waves follow in order.  So
// step st of a block takes pixel 16 st + c, each step's product is kept apart, and block b has the
// column c for which the cross-lane adds (blocks ^ 8, ^ 4, ^ 2, ^ 1) are the
// tree's last four levels.  (Waves of 8 x 8 pixels meet a tenth fewer entries
// but have no such tree: 1045 us.)
constexpr int kGeoFac = 6;   // du', dv', dw', dop; dx, dy
// Sums per entry and wave, at 4 r + j: row r = 0, 1, 2: (du', dv', dw') times
// (1, dx, dy); column 3 of these rows: dn_1, dn_2, dz; row 3: dC, dn_0; then
// dop (and, low-pass, the filter term's centre gradient).
constexpr int kSums = 20;

// Place of the wave's pixel i among the 16 blocks of four pixels.
__device__ __forceinline__ int block_slot(int i) {
  const int c = i & 7;
  return 4 * ((i & 8) | (c < 4 ? c : 11 - c)) + (i >> 4);
}

__device__ __forceinline__ f4v mfma_4x4x1(float a, float b, f4v c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// DM (dense mode only): the batch's feature contractions on the matrix cores
// (true) or in vector FMAs (false); a launch choice, whichever is faster for
// the workload (the autotuner times both).
template <int MODE, typename FT, bool LP, bool DM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MODE == kTopK ? (LP ? 3 : 4) : 1))) void k_walk_bwd(
    const WalkRec* __restrict__ rec, const uint32_t* __restrict__ pid, const uint32_t* __restrict__ eid,
    const uint2* __restrict__ ranges, CamTable ct, TileOrder tq, int K, const uint32_t* __restrict__ nlast,
    const float* __restrict__ tfinal,
    const int32_t* __restrict__ selpos, const float* __restrict__ seldot, const float* __restrict__ g_rgb,
    const float* __restrict__ g_depth, const float* __restrict__ g_normal, const float* __restrict__ g_alpha,
    const float* __restrict__ g_feat, const FeatSrc<FT> feat, int C, float* __restrict__ gpart,
    uint8_t* __restrict__ gflag, float* __restrict__ fpart, uint8_t* __restrict__ fflag) {
#pragma clang fp contract(fast)
  // (products and sums written in this kernel may fuse into FMAs: its outputs
  // are gradients, which no decision depends on; the hit test, alpha and the
  // weights come from eval_pixel, written outside this scope and evaluated
  // exactly as in the forward)
  constexpr int NC = LP ? 4 : 2;  // w, dz (low-pass: and the filter term's centre gradient)
  __shared__ __align__(16) float s_geo[4][2][kGeoFac][64];  // [wave][entry of the pair][factor][pixel]
  __shared__ __align__(16) float s_col[4][NC][4][64];       // [wave][factor][entry of the group][pixel]
  __shared__ __align__(16) float s_part[4][kBB][kSums];
  __shared__ uint32_t s_has[4];
  __shared__ int s_lmax;
  // dense-blend mode only: the batch's feature dots, replaced by its weights
  // (rows padded to 260 floats: the matrix-core operand reads of 16 entries x
  // 4 pixels fall in distinct banks)
  constexpr int kOmS = kTilePix + 4;
  __shared__ float s_fc[MODE == kFull && !DM ? kBB : 1][64];  // vector form: the batch's feature chunk
  __shared__ __align__(16) float s_om[MODE == kFull ? kBB : 1][kOmS];
  __shared__ uint32_t s_id[MODE == kFull ? kBB : 1];
  // Top-K mode: every pixel's selected list positions ([K][256], 16 bits: a
  // tile whose pixels reach further takes them from memory), read back to
  // front by the pixel's own lane; the feature dots stay in global memory,
  // each loaded when the previous one is used.  (With K = 16 a block then
  // takes 39 KB of LDS and four share a CU; at three the walk is 15% slower.)
  extern __shared__ uint16_t s_sel[];

  with_tile(tq, [&](const int tile) {
  const TileLoc tl = locate(ct, tile);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tx = tl.tx, ty = tl.ty, W = tl.W, H = tl.H;
  const int lx = tid & (ct.tw - 1), ly = tid >> ct.tsh, at = tile_index(ct, lx, ly);
  const int px = tx * ct.tw + lx, py = ty * ct.th + ly;
  const bool inside = px < W && py < H;
  const double X = (double)px + 0.5, Y = (double)py + 0.5;
  SubRect sr;  // pixel centres of the wave's rows (pixels past the image included)
  sr.x0 = (float)(tx * ct.tw) + 0.5f;
  sr.x1 = sr.x0 + (float)(ct.tw - 1);
  sr.y0 = (float)(ty * ct.th + wave * (64 >> ct.tsh)) + 0.5f;
  sr.y1 = sr.y0 + (float)((64 >> ct.tsh) - 1);
  const uint32_t start = ranges[tile].x;
  const int sp = tile * kTilePix + at;
  const int my_last = (int)nlast[sp];
  float T = tfinal[sp];
  const int64_t pix = tl.pix0 + (int64_t)py * W + px;
  float gC0 = 0.f, gC1 = 0.f, gC2 = 0.f, gD = 0.f, gN0 = 0.f, gN1 = 0.f, gN2 = 0.f, gA = 0.f;
  if (inside) {
    if (g_rgb) { gC0 = g_rgb[3 * pix]; gC1 = g_rgb[3 * pix + 1]; gC2 = g_rgb[3 * pix + 2]; }
    if (g_depth) gD = g_depth[pix];
    if (g_normal) { gN0 = g_normal[3 * pix]; gN1 = g_normal[3 * pix + 1]; gN2 = g_normal[3 * pix + 2]; }
    if (g_alpha) gA = g_alpha[pix];
  }
  const float gAT = gA * T;
  // the columns, a step per pixel of the block: (dC, dn_0); (dn_1, dn_2, -, -);
  // and unit column 2 for the plain sum
  const int col = lane & 3, slot = block_slot(lane);
  f4v bc, bn;
  {
    float* f = &s_geo[wave][0][0][0];
    f[slot] = gC0;
    f[64 + slot] = gC1;
    f[128 + slot] = gC2;
    f[192 + slot] = gN0;
    wave_lds_sync();
    bc = *reinterpret_cast<const f4v*>(f + 64 * col + (lane & ~3));
    wave_lds_sync();
    f[slot] = gN1;
    f[64 + slot] = gN2;
    f[128 + slot] = 0.0f;
    wave_lds_sync();
    bn = *reinterpret_cast<const f4v*>(f + 64 * min(col, 2) + (lane & ~3));
    wave_lds_sync();
  }
  const float unit2 = col == 2 ? 1.0f : 0.0f;
  // Top-K: walk the saved selection from its back end.  kq: the last selection
  // before the current batch, at position cursel; kp: the next one whose dot is
  // used (held in nextdot)
  int kp = -1, kq = -1, cursel = -1;
  float nextdot = 0.0f;
  const size_t tbase = (size_t)tile * K * kTilePix;
  uint16_t* s_sp = s_sel;
  const float* g_sd = seldot + tbase + at;  // this pixel's dots, read one ahead of their use
  if (MODE == kTopK) {
    for (int q = 0; q < K; ++q) {
      const int sq = selpos[tbase + (size_t)q * kTilePix + at];
      s_sp[q * kTilePix + tid] = (uint16_t)sq;
      if (sq >= 0) {
        kp = q;
        cursel = sq;
      }
    }
    kq = kp;
    if (kp >= 0) nextdot = g_sd[(size_t)kp * kTilePix];
  }

  // the wave starts at its own last contributor: the entries past it change
  // nothing of its pixels
  int wmax = my_last;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) wmax = max(wmax, __shfl_xor(wmax, o, 64));
  wmax = __builtin_amdgcn_readfirstlane(wmax);
  if (tid == 0) s_lmax = 0;
  __syncthreads();
  if (lane == 0) atomicMax(&s_lmax, wmax);
  __syncthreads();
  const int Lmax = __builtin_amdgcn_readfirstlane(s_lmax);  // block-uniform: a scalar loop bound
  float suffix = 0.0f;

  // the batch's ids and culling records, a lane per entry (the upper half of
  // the wave repeats the lower); records are read one batch ahead, ids two
  const int el = lane & (kBB - 1);
  const auto id_at = [&](int h) {
    const int l = max(0, h - kBB);
    return h > 0 ? pid[start + min(l + el, h - 1)] : 0u;
  };
  uint32_t id1 = id_at(Lmax), id2 = id_at(Lmax - kBB);
  CullRec nc = rec[id1].c;
  for (int hi = Lmax; hi > 0; hi -= kBB) {
    const int lo = max(0, hi - kBB), nb = hi - lo;
    const uint32_t id = id1;
    const bool meets = rect_meets<LP>(nc, sr.x0, sr.x1, sr.y0, sr.y1);
    id1 = id2;
    id2 = id_at(hi - 2 * kBB);
    nc = rec[id1].c;
    // entries of the batch that meet this wave's pixels and lie before its
    // last contributor
    const int ktop = min(nb, wmax - lo);
    uint32_t mask = ktop > 0 ? (uint32_t)__ballot(meets) & (0xFFFFFFFFu >> (kBB - ktop)) : 0u;

    // dense mode: phi[k] = g_F(p) . f_k for the batch, left in s_om
    if constexpr (MODE == kFull) {
      if (wave == 0 && lane < nb) s_id[lane] = id;
      __syncthreads();
    }
    if constexpr (MODE == kFull && !DM) {
      // vector form: feature chunks of 64 channels staged in LDS, each pixel
      // its 32 dots (LDS reads by broadcast)
      float phi[kBB];
#pragma unroll
      for (int k = 0; k < kBB; ++k) phi[k] = 0.0f;
      if (g_feat) {
        const float* grow = g_feat + pix * C;
        const bool has_gf = inside;
        for (int c0 = 0; c0 < C; c0 += 64) {
          for (int e = tid; e < nb * 64; e += 256) {
            const int k = e >> 6, c = e & 63;
            s_fc[k][c] = (c0 + c < C) ? feat.load1(s_id[k] - tl.v0, c0 + c) : 0.0f;
          }
          __syncthreads();
          if (has_gf) {
            const int cn = min(64, C - c0);
            for (int c = 0; c < cn; c += 4) {
              const float4 g = *reinterpret_cast<const float4*>(grow + c0 + c);
#pragma unroll
              for (int k = 0; k < kBB; ++k)
                phi[k] = fmaf(g.x, s_fc[k][c], fmaf(g.y, s_fc[k][c + 1], fmaf(g.z, s_fc[k][c + 2], fmaf(g.w, s_fc[k][c + 3], phi[k]))));
            }
          }
          __syncthreads();
        }
      }
#pragma unroll
      for (int k = 0; k < kBB; ++k) s_om[k][tid] = phi[k];
    }
    if constexpr (MODE == kFull && DM) {
      // the product PHI = G F^T on the matrix cores: wave w takes its 4 pixel
      // blocks of 16 x the 2 entry blocks of 16, k = 4 channels per step (lane
      // (li, lk) loads channels 4 lk .. 4 lk + 3 of a 16-channel group as one
      // vector, component i feeding step i)
      const int li = lane & 15, lk = lane >> 4;
      int fr[2];  // feature row of the lane's entry of each block, -1 past the batch
#pragma unroll
      for (int eb = 0; eb < 2; ++eb) {
        const int e = 16 * eb + li;
        fr[eb] = e < nb ? (int)(s_id[e] - tl.v0) : -1;
      }
      for (int pb = 0; pb < 4; ++pb) {
        const int q = 64 * wave + 16 * pb + li;  // pixel of lane li
        const int qx = tx * ct.tw + (q & (ct.tw - 1)), qy = ty * ct.th + (q >> ct.tsh);
        const float* gq = g_feat && qx < W && qy < H ? g_feat + (tl.pix0 + (int64_t)qy * W + qx) * C : nullptr;
        f4v acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        // 128 channels at a time: every operand of the segment is loaded
        // before its products, so the loads are in flight together
        for (int cs = 0; g_feat && cs < C; cs += 128) {
          float4 a[8], b[2][8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int c = cs + 16 * j + 4 * lk;  // C % 4 == 0: a group of 4 is whole or absent
            a[j] = gq && c < C ? *reinterpret_cast<const float4*>(gq + c) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int eb = 0; eb < 2; ++eb)
              b[eb][j] = fr[eb] >= 0 && c < C ? feat.load4(fr[eb], c) : make_float4(0.f, 0.f, 0.f, 0.f);
          }
#pragma unroll
          for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int eb = 0; eb < 2; ++eb) {
              acc[eb] = mfma_16x16x4(a[j].x, b[eb][j].x, acc[eb]);
              acc[eb] = mfma_16x16x4(a[j].y, b[eb][j].y, acc[eb]);
              acc[eb] = mfma_16x16x4(a[j].z, b[eb][j].z, acc[eb]);
              acc[eb] = mfma_16x16x4(a[j].w, b[eb][j].w, acc[eb]);
            }
        }
#pragma unroll
        for (int eb = 0; eb < 2; ++eb)
          *reinterpret_cast<f4v*>(&s_om[16 * eb + li][64 * wave + 16 * pb + 4 * lk]) = acc[eb];
      }
      wave_lds_sync();  // a wave reads back its own pixels only
    }
    if constexpr (MODE == kFull) {
      // entries the wave does not evaluate have zero weight
      for (uint32_t m = ~mask & (0xFFFFFFFFu >> (kBB - nb)); m; m &= m - 1) s_om[__builtin_ctz(m)][tid] = 0.0f;
    }

    // the pixel's selections in the batch as bits, so that the entry loop
    // reads nothing from LDS for them: such a read is waited for together
    // with the next record's scalar load, whose latency it would expose
    uint32_t selbits = 0u;
    if (MODE == kTopK) {
      while (__any(cursel >= lo)) {
        const bool in = cursel >= lo;
        selbits |= in ? 1u << (cursel - lo) : 0u;
        kq -= in ? 1 : 0;
        const int q = max(kq, 0) * kTilePix;
        const int sq = Lmax <= 0xFFFF ? (int)s_sp[q + tid] : selpos[tbase + q + at];
        cursel = kq >= 0 ? sq : -1;
      }
    }
    // what the combination below needs of the pair and its record
    const int ce = (tid >> 2) & (kBB - 1), cq = tid & 3;
    const bool comb = wave < 2 && ce < nb;
    const uint32_t cid = (uint32_t)__shfl((int)id, ce, 64);
    float ca0 = 0.f, ca1 = 0.f, ca2 = 0.f, ca3 = 0.f, ca4 = 0.f, ca5 = 0.f;
    uint32_t cslot = 0u;
    if (comb) cslot = eid[start + lo + ce];

    uint32_t has = 0u;    // entries with a contributor in this wave
    uint32_t group = 0u;  // the open group's entries, 8 bits each
    int ng = 0;
    // geometric products of the open pair (entries 2 h, 2 h + 1 of the group),
    // the first two levels of the tree added:
    // entry i's row r, column j of block b in register r of lane 4 b + j
    f4v dg[4];
    const auto pair = [&](auto hc) {
      constexpr int h = decltype(hc)::value;
      wave_lds_sync();
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f4v f = *reinterpret_cast<const f4v*>(&s_geo[wave][i][lane & 3][lane & ~3]);
        // column 0 is 1, columns 1 and 2 are dx and dy, column 3 is not used
        const f4v xy = *reinterpret_cast<const f4v*>(&s_geo[wave][i][4 + (col >> 1)][lane & ~3]);
        f4v d[4];
#pragma unroll
        for (int st = 0; st < 4; ++st)
          d[st] = mfma_4x4x1(f[st], col == 0 ? 1.0f : xy[st], f4v{0.f, 0.f, 0.f, 0.f});
        dg[2 * h + i] = (d[0] + d[2]) + (d[1] + d[3]);
      }
      wave_lds_sync();
    };
    // the group's other products (entry i's column j in register i), then the
    // 16 blocks added across lanes, which leaves entry i's sums in lane group i
    const auto flush = [&]() {
      f4v dc = {0.f, 0.f, 0.f, 0.f}, dn = dc, dl = dc;
      wave_lds_sync();
      const auto fac = [&](int f) { return *reinterpret_cast<const f4v*>(&s_col[wave][f][lane & 3][lane & ~3]); };
      const f4v fw = fac(0), fz = fac(1);
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        dc = mfma_4x4x1(fw[st], bc[st], dc);
        dn = mfma_4x4x1(fw[st], bn[st], dn);
      }
#pragma unroll
      for (int st = 0; st < 4; ++st) dn = mfma_4x4x1(fz[st], unit2, dn);
      if constexpr (LP) {
        const f4v fx = fac(NC - 2), fy = fac(NC - 1);
#pragma unroll
        for (int st = 0; st < 4; ++st) {
          dl = mfma_4x4x1(fx[st], col == 1 ? 1.0f : 0.0f, dl);
          dl = mfma_4x4x1(fy[st], col == 2 ? 1.0f : 0.0f, dl);
        }
      }
      wave_lds_sync();
      float* dst = &s_part[wave][(group >> (8 * (lane >> 4))) & (kBB - 1)][0];
      const bool put = (lane & 12) == 0 && (lane >> 4) < ng;
      // x0..x3: the four entries' values; lane group i (16 lanes) gets entry i's
      const auto sum4 = [&](float x0, float x1, float x2, float x3) {
        float v = swap16_add(swap32_add(x0, x2), swap32_add(x1, x3));
        v += dpp_mov<kDppRowRor8>(v);
        v += dpp_mov<kDppRowRor4>(v);
        return v;
      };
      const float t0 = sum4(dg[0][0], dg[1][0], dg[2][0], dg[3][0]), t1 = sum4(dg[0][1], dg[1][1], dg[2][1], dg[3][1]);
      const float t2 = sum4(dg[0][2], dg[1][2], dg[2][2], dg[3][2]), t3 = sum4(dg[0][3], dg[1][3], dg[2][3], dg[3][3]);
      const float tc = sum4(dc[0], dc[1], dc[2], dc[3]), tn = sum4(dn[0], dn[1], dn[2], dn[3]);
      float tl = 0.0f;
      if constexpr (LP) tl = sum4(dl[0], dl[1], dl[2], dl[3]);
      if (put) {
        if (col < 3) {
          dst[col] = t0;
          dst[4 + col] = t1;
          dst[8 + col] = t2;
          dst[4 * col + 3] = tn;
        }
        dst[12 + col] = tc;
        if constexpr (LP) dst[16 + col] = col == 0 ? t3 : tl;
        else if (col == 0) dst[16] = t3;
      }
      group = 0u;
      ng = 0;
    };

    if (mask) {
      int k = 31 - __builtin_clz(mask);
      SRec next = load_rec(rec, lane_value(id, k));
      do {
        const int pos = lo + k, ke = k;
        const LRec s = next.get();
        mask &= ~(1u << k);
        if (mask) {
          k = 31 - __builtin_clz(mask);
          next = load_rec(rec, lane_value(id, k));
        }
        // the pixel's factors, all zero where it does not take part
        float w = 0.0f, du1 = 0.0f, dv1 = 0.0f, dw1 = 0.0f, dzi = 0.0f, dop = 0.0f, ex = 0.0f, ey = 0.0f;
        float gcx = 0.0f, gcy = 0.0f;  // low-pass term: direct gradient of the projected centre
        PixEval e;
        const bool contrib = eval_pixel<LP>(s, X, Y, e) & (pos < my_last);
        const bool takes = contrib & ((selbits & (1u << ke)) != 0u);
        if (contrib) {
          // 1 / (1 - alpha) once for both quotients: alpha <= 0.99, so the
          // reciprocal's relative error (about 1 ulp) stays that small
          const float r1m = __builtin_amdgcn_rcpf(1.0f - e.alpha);
          const float Tb = T * r1m;
          w = e.alpha * Tb;
          const float u = e.u, vv = e.v, z = s.mz * e.iw;
          float eF = 0.0f;
          if (MODE == kTopK) eF = takes ? nextdot : 0.0f;
          else eF = s_om[ke][tid];
          const float ei = gC0 * s.r + gC1 * s.g + gC2 * s.b + gD * z + gN0 * s.n0 + gN1 * s.n1 + gN2 * s.n2 + eF;
          const float da = Tb * ei - (suffix - gAT) * r1m;
          suffix = fmaf(w, ei, suffix);
          T = Tb;
          dop = e.clamped ? 0.0f : da * e.G;
          const float drho = e.clamped ? 0.0f : -0.5f * da * e.alpha;
          const float dz = w * gD;
          if (LP && e.filt) {
            // rho = 2 |d|^2 with d = pixel - centre, depth = centre depth
            gcx = -4.0f * drho * e.dx;
            gcy = -4.0f * drho * e.dy;
            dzi = dz;
          } else {
            const float du = 2.0f * u * drho, dv = 2.0f * vv * drho;
            du1 = du * e.iw;
            dv1 = dv * e.iw;
            dw1 = -(du * u + dv * vv + dz * z) * e.iw;
            dzi = dz * e.iw;
            ex = e.dx;
            ey = e.dy;
          }
        }
        if constexpr (MODE == kFull) s_om[ke][tid] = w;
        if (MODE == kTopK && __any(takes)) {
          // the next selection's dot, read by every lane, so that the load in
          // flight is waited for where it is used and not at once (as the
          // lanes that keep theirs would have it)
          kp -= takes ? 1 : 0;
          nextdot = g_sd[max(kp, 0) * kTilePix];
        }
        if (__any(contrib)) {
          float* f = &s_geo[wave][ng & 1][0][slot];
          f[0] = du1;
          f[64] = dv1;
          f[128] = dw1;
          f[192] = dop;
          f[256] = ex;
          f[320] = ey;
          float* fc = &s_col[wave][0][ng][slot];
          fc[0] = w;
          fc[256] = dzi;
          if constexpr (LP) {
            fc[512] = gcx;
            fc[768] = gcy;
          }
          has |= 1u << ke;
          group |= (uint32_t)ke << (8 * ng);
          ++ng;
          if (ng == 2) pair(std::integral_constant<int, 0>{});
          if (ng == 4) {
            pair(std::integral_constant<int, 1>{});
            flush();
          }
        }
      } while (mask);
      if (ng) {
        if (ng == 1) pair(std::integral_constant<int, 0>{});
        if (ng == 3) pair(std::integral_constant<int, 1>{});
        flush();
      }
    }
    if (lane == 0) s_has[wave] = has;

    // combine the 4 waves, four threads per entry, each one float4 of the
    // pair's 16 accumulators
    if (comb && cq == 1) {
      const WalkRec& rr = rec[cid];
      ca0 = (float)rr.d0.x; ca1 = (float)rr.d0.y;
      ca2 = (float)rr.d1.x; ca3 = (float)rr.d1.y;
      ca4 = (float)rr.d2.x; ca5 = (float)rr.d2.y;
    }
    __syncthreads();
    if (comb) {
      bool any = false;
      // the rows a thread needs: 0, 1 (and 2 for the second); 2, 3, 4; 0, 1, 3
      f4v A = {0.f, 0.f, 0.f, 0.f}, B = A, C4 = A, E = A;
      const int ra = cq == 2 ? 8 : 0, rb = cq == 2 ? 16 : 4, rc = cq < 2 ? 8 : 12;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (!((s_has[w] >> ce) & 1u)) continue;
        any = true;
        const float* x = s_part[w][ce];
        A += *reinterpret_cast<const f4v*>(x + ra);
        B += *reinterpret_cast<const f4v*>(x + rb);
        C4 += *reinterpret_cast<const f4v*>(x + rc);
        if constexpr (LP) E += *reinterpret_cast<const f4v*>(x + 16);
      }
      if (any) {
        const size_t slot = cslot;
        float4* g = reinterpret_cast<float4*>(gpart + slot * 16);
        // u' = A^-1 d, w' = 1 - e.d with d = pixel - centre; d depends on the
        // centre with slope -1
        if (cq == 0) {
          g[0] = make_float4(A[1], A[2], B[1], B[2]);
          gflag[slot] = 1;
        } else if (cq == 1) {
          float gxc = -(ca0 * A[0] + ca2 * B[0] - ca4 * C4[0]);
          float gyc = -(ca1 * A[0] + ca3 * B[0] - ca5 * C4[0]);
          if constexpr (LP) {
            gxc += E[1];
            gyc += E[2];
          }
          g[1] = make_float4(-C4[1], -C4[2], gxc, gyc);
        } else if (cq == 2) {
          g[2] = make_float4(A[3], B[0], C4[0], C4[1]);
        } else {
          g[3] = make_float4(C4[2], C4[3], A[3], B[3]);
        }
      }
    }
    __syncthreads();

    // dense mode: dL/df_k = sum_p w_k(p) g_F(p) for the batch, the product
    // R = W^T G on the matrix cores: units (entry block of 16, channel block
    // of 16) dealt to the waves, each a sum over the 256 pixels in 64 steps
    // of 4 (pixels 16 y + 4 u + lk of tile row y), written at the pair's
    // emission index
    if constexpr (MODE == kFull && !DM) {
      // vector form: wave w takes 8 surfels of the batch, lane = channel, the
      // 256 pixels 8 at a time (8 independent upstream loads in flight;
      // pixels outside the image have zero weight and read as zero)
      if (g_feat) {
        constexpr int PER = kBB / 4;
        // the tile's pixels inside the image: wl columns, hl rows; pixel
        // offsets from the tile's first one are below 2^29 (W, C and the tile
        // height are bounded)
        const int wl = min(ct.tw, W - tx * ct.tw), hl = min(ct.th, H - ty * ct.th), wc = W * C;
        for (int c0 = 0; c0 < C; c0 += 64) {
          const int c = c0 + lane;
          float acc[PER];
#pragma unroll
          for (int j = 0; j < PER; ++j) acc[j] = 0.0f;
          if (c < C) {
            const float* gt = g_feat + (tl.pix0 + (int64_t)(ty * ct.th) * W + tx * ct.tw) * C + c;
            for (int p0 = 0; p0 < kTilePix; p0 += 8) {
              float g[8];
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                const int p = p0 + u, lx = p & (ct.tw - 1), ly = p >> ct.tsh;
                g[u] = lx < wl && ly < hl ? gt[ly * wc + lx * C] : 0.0f;
              }
#pragma unroll
              for (int j = 0; j < PER; ++j) {
                const float4 w0 = *reinterpret_cast<const float4*>(&s_om[wave * PER + j][p0]);
                const float4 w1 = *reinterpret_cast<const float4*>(&s_om[wave * PER + j][p0 + 4]);
                float a = acc[j];
                a = fmaf(w0.x, g[0], a);
                a = fmaf(w0.y, g[1], a);
                a = fmaf(w0.z, g[2], a);
                a = fmaf(w0.w, g[3], a);
                a = fmaf(w1.x, g[4], a);
                a = fmaf(w1.y, g[5], a);
                a = fmaf(w1.z, g[6], a);
                a = fmaf(w1.w, g[7], a);
                acc[j] = a;
              }
            }
#pragma unroll
            for (int j = 0; j < PER; ++j) {
              const int k = wave * PER + j;
              if (k < nb) {
                const size_t slot = eid[start + lo + k];
                fpart[slot * C + c] = acc[j];
                if (c == 0) fflag[slot] = 1;
              }
            }
          }
        }
      }
    }
    if constexpr (MODE == kFull && DM) {
      if (g_feat) {
        const int li = lane & 15, lk = lane >> 4;
        const int ncb = (C + 15) >> 4;
        // the tile's pixels inside the image: wl columns, hl rows
        const int wl = min(ct.tw, W - tx * ct.tw), hl = min(ct.th, H - ty * ct.th);
        for (int unit = wave; unit < 2 * ncb; unit += 4) {
          const int eb = unit & 1, cb = unit >> 1;
          const int c = 16 * cb + li;
          f4v racc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
          const float* wrow = s_om[16 * eb + li];
          // G of the lane's first pixel (tile column lk, row 0); step t covers
          // pixels 4 t + lk (four neighbours of a row), whose offsets
          // from it are the same for all lanes and below 2^29 (W, C and the
          // tile height are bounded)
          const float* gt = g_feat + (tl.pix0 + (int64_t)(ty * ct.th) * W + tx * ct.tw + lk) * C + c;
          // 128 pixels (32 steps) at a time: their 32 G values are loaded
          // together, so enough of them are in flight to cover the memory
          // latency
          for (int t0 = 0; t0 < kTilePix / 4; t0 += 32) {
            // the shape values go through an empty asm statement so that the
            // step offsets and bounds are formed here and not kept live
            // across units (64 of them would not fit in the registers)
            int wc = W * C, cs = C, sh = ct.tsh, wlim = wl - lk, hlim = hl;
            asm volatile("" : "+s"(wc), "+s"(cs), "+s"(sh), "+v"(wlim), "+s"(hlim));
            float b[32];
#pragma unroll
            for (int t = 0; t < 32; ++t) {
              const int q4 = 4 * (t0 + t), lx = q4 & ((1 << sh) - 1), ly = q4 >> sh;
              b[t] = lx < wlim && ly < hlim && c < C ? gt[ly * wc + lx * cs] : 0.0f;
            }
#pragma unroll
            for (int t = 0; t < 32; ++t) racc[t & 1] = mfma_16x16x4(wrow[4 * (t0 + t) + lk], b[t], racc[t & 1]);
          }
          const f4v rs = racc[0] + racc[1];
          if (c < C) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int k = 16 * eb + 4 * lk + r;
              if (k < nb) {
                const size_t slot = eid[start + lo + k];
                fpart[slot * C + c] = rs[r];
                if (c == 0) fflag[slot] = 1;
              }
            }
          }
        }
      }
    }
  }
  });
}

// ------------------------------------------------------- per-surfel reduction

// Chain rule of one camera's view of a surfel: from the 16 pair sums G (dL/d
// of A^-1 (4), e (2), projected centre (2), centre depth, o, c (3), n_c (3))
// to the surfel parameters.  The walk record was evaluated in FP64 from the
// FP32 inputs; its chain rule is evaluated the same way.
struct SurfelGrad {
  double mu[3], su, sv, q[4], o, rgb[3];
};

__device__ __forceinline__ void chain_rule(const double (&G)[16], const CamArgs& k, bool flip, const double (&mu)[3],
                                           double su, double sv, const double (&qn)[4], const double (&Rq)[3][3],
                                           SurfelGrad& acc) {
  const double w = qn[0], x = qn[1], y = qn[2], z = qn[3];
  double mc[3], ra[3], rb[3], a[3], b[3];
  for (int r = 0; r < 3; ++r) {
    const float* Rr = k.R + 3 * r;
    mc[r] = Rr[0] * mu[0] + Rr[1] * mu[1] + Rr[2] * mu[2] + (double)k.t[r];
    ra[r] = Rr[0] * Rq[0][0] + Rr[1] * Rq[1][0] + Rr[2] * Rq[2][0];
    rb[r] = Rr[0] * Rq[0][1] + Rr[1] * Rq[1][1] + Rr[2] * Rq[2][1];
    a[r] = su * ra[r];
    b[r] = sv * rb[r];
  }
  const double sgn = flip ? -1.0 : 1.0;  // orientation chosen by the key stage
  const double fx = k.fx, fy = k.fy;
  const double iz = 1.0 / mc[2];
  const double p = a[2] * iz, q = b[2] * iz;
  const double mx = mc[0] * iz, my = mc[1] * iz;
  const double B00 = fx * (a[0] - mx * a[2]), B01 = fx * (b[0] - mx * b[2]);
  const double B10 = fy * (a[1] - my * a[2]), B11 = fy * (b[1] - my * b[2]);
  const double A00 = B00 * iz, A01 = B01 * iz, A10 = B10 * iz, A11 = B11 * iz;
  const double idA = 1.0 / (A00 * A11 - A01 * A10);
  const double Ai[2][2] = {{A11 * idA, -A01 * idA}, {-A10 * idA, A00 * idA}};
  const double dAi[2][2] = {{G[0], G[1]}, {G[2], G[3]}};
  const double de[2] = {G[4], G[5]};
  const double dxc = G[6], dyc = G[7], dmz = G[8];
  const double gv[2] = {p, q};
  // e = g^T A^-1
  double dAt[2][2];
  for (int r = 0; r < 2; ++r)
    for (int c = 0; c < 2; ++c) dAt[r][c] = dAi[r][c] + gv[r] * de[c];
  const double dp = de[0] * Ai[0][0] + de[1] * Ai[0][1];
  const double dq = de[0] * Ai[1][0] + de[1] * Ai[1][1];
  // A^-1: dA = -A^-T dAt A^-T
  double M1[2][2], dA[2][2];
  for (int r = 0; r < 2; ++r)
    for (int c = 0; c < 2; ++c) M1[r][c] = dAt[r][0] * Ai[c][0] + dAt[r][1] * Ai[c][1];
  for (int r = 0; r < 2; ++r)
    for (int c = 0; c < 2; ++c) dA[r][c] = -(Ai[0][r] * M1[0][c] + Ai[1][r] * M1[1][c]);
  // A = diag(fx, fy) [a_xy - m a_z | b_xy - m b_z] / z,  p = a_z / z, q = b_z / z
  double d_a[3], d_b[3], d_mc[3];
  d_a[0] = fx * iz * dA[0][0];
  d_b[0] = fx * iz * dA[0][1];
  d_a[1] = fy * iz * dA[1][0];
  d_b[1] = fy * iz * dA[1][1];
  d_a[2] = -(fx * mx * dA[0][0] + fy * my * dA[1][0]) * iz + iz * dp;
  d_b[2] = -(fx * mx * dA[0][1] + fy * my * dA[1][1]) * iz + iz * dq;
  const double d_mx = -fx * iz * (a[2] * dA[0][0] + b[2] * dA[0][1]) + fx * dxc;
  const double d_my = -fy * iz * (a[2] * dA[1][0] + b[2] * dA[1][1]) + fy * dyc;
  const double d_iz = dA[0][0] * B00 + dA[0][1] * B01 + dA[1][0] * B10 + dA[1][1] * B11 + dp * a[2] + dq * b[2] +
                      d_mx * mc[0] + d_my * mc[1];
  d_mc[0] = d_mx * iz;
  d_mc[1] = d_my * iz;
  d_mc[2] = -d_iz * iz * iz + dmz;
  const double dn[3] = {sgn * G[13], sgn * G[14], sgn * G[15]};
  // back through the world -> camera rotation
  double dtu[3], dtv[3], dnn[3];
  for (int c = 0; c < 3; ++c) {
    const double R0 = k.R[c], R1 = k.R[3 + c], R2 = k.R[6 + c];
    dtu[c] = su * (R0 * d_a[0] + R1 * d_a[1] + R2 * d_a[2]);
    dtv[c] = sv * (R0 * d_b[0] + R1 * d_b[1] + R2 * d_b[2]);
    dnn[c] = R0 * dn[0] + R1 * dn[1] + R2 * dn[2];
    acc.mu[c] += R0 * d_mc[0] + R1 * d_mc[1] + R2 * d_mc[2];
  }
  acc.su += d_a[0] * ra[0] + d_a[1] * ra[1] + d_a[2] * ra[2];
  acc.sv += d_b[0] * rb[0] + d_b[1] * rb[1] + d_b[2] * rb[2];
  // Rq columns are t_u, t_v, n;  Gm[r][c] = dL/dRq[r][c]
  const double Gm[3][3] = {{dtu[0], dtv[0], dnn[0]}, {dtu[1], dtv[1], dnn[1]}, {dtu[2], dtv[2], dnn[2]}};
  acc.q[0] += 2. * (-z * Gm[0][1] + y * Gm[0][2] + z * Gm[1][0] - x * Gm[1][2] - y * Gm[2][0] + x * Gm[2][1]);
  acc.q[1] += 2. * (y * Gm[0][1] + z * Gm[0][2] + y * Gm[1][0] - 2. * x * Gm[1][1] - w * Gm[1][2] + z * Gm[2][0] +
                    w * Gm[2][1] - 2. * x * Gm[2][2]);
  acc.q[2] += 2. * (-2. * y * Gm[0][0] + x * Gm[0][1] + w * Gm[0][2] + x * Gm[1][0] + z * Gm[1][2] - w * Gm[2][0] +
                    z * Gm[2][1] - 2. * y * Gm[2][2]);
  acc.q[3] += 2. * (-2. * z * Gm[0][0] - w * Gm[0][1] + x * Gm[0][2] + w * Gm[1][0] - 2. * z * Gm[1][1] +
                    y * Gm[1][2] + x * Gm[2][0] + y * Gm[2][1]);
  acc.o += G[9];
  acc.rgb[0] += G[10];
  acc.rgb[1] += G[11];
  acc.rgb[2] += G[12];
}

// The surfel parameters the chain rule takes.
struct SurfelParams {
  double mu[3], su, sv, rn, qn[4], Rq[3][3];
};
__device__ __forceinline__ void load_params(SurfelParams& P, int64_t i, const float* __restrict__ means,
                                            const float* __restrict__ scales, const float* __restrict__ quats) {
  P.mu[0] = means[3 * i]; P.mu[1] = means[3 * i + 1]; P.mu[2] = means[3 * i + 2];
  P.su = scales[2 * i]; P.sv = scales[2 * i + 1];
  const double q0 = quats[4 * i], q1 = quats[4 * i + 1], q2 = quats[4 * i + 2], q3 = quats[4 * i + 3];
  const double qq = q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3;
  P.rn = qq > 0.0 ? 1.0 / sqrt(qq) : 0.0;
  P.qn[0] = q0 * P.rn; P.qn[1] = q1 * P.rn; P.qn[2] = q2 * P.rn; P.qn[3] = q3 * P.rn;
  const double w = P.qn[0], x = P.qn[1], y = P.qn[2], z = P.qn[3];
  P.Rq[0][0] = 1. - 2. * (y * y + z * z); P.Rq[0][1] = 2. * (x * y - w * z); P.Rq[0][2] = 2. * (x * z + w * y);
  P.Rq[1][0] = 2. * (x * y + w * z); P.Rq[1][1] = 1. - 2. * (x * x + z * z); P.Rq[1][2] = 2. * (y * z - w * x);
  P.Rq[2][0] = 2. * (x * z - w * y); P.Rq[2][1] = 2. * (y * z + w * x); P.Rq[2][2] = 1. - 2. * (x * x + y * y);
}
__device__ __forceinline__ void clear_grad(SurfelGrad& g) {
  for (int j = 0; j < 3; ++j) g.mu[j] = g.rgb[j] = 0.0;
  for (int j = 0; j < 4; ++j) g.q[j] = 0.0;
  g.su = g.sv = g.o = 0.0;
}
struct GeoGrads {
  float *means, *scales, *quats, *opacity, *rgb;
};
__device__ __forceinline__ void write_grad(const SurfelGrad& acc, const SurfelParams& P, int64_t i,
                                           const GeoGrads& d) {
  // unit quaternion: project out the radial component
  const double dot = P.qn[0] * acc.q[0] + P.qn[1] * acc.q[1] + P.qn[2] * acc.q[2] + P.qn[3] * acc.q[3];
  for (int j = 0; j < 4; ++j) d.quats[4 * i + j] = (float)((acc.q[j] - P.qn[j] * dot) * P.rn);
  for (int j = 0; j < 3; ++j) d.means[3 * i + j] = (float)acc.mu[j];
  d.scales[2 * i] = (float)acc.su;
  d.scales[2 * i + 1] = (float)acc.sv;
  d.opacity[i] = (float)acc.o;
  for (int j = 0; j < 3; ++j) d.rgb[3 * i + j] = (float)acc.rgb[j];
}

// Wave per 64 surfels: for each camera in order, the sum of a surfel's pairs'
// partials (its emitted range [vbase, vbase + count), in emission order), then
// that camera's chain rule (a lane per surfel); the cameras' contributions are
// added in camera order.  The wave's 64 ranges are read as one flat sequence:
// lane l loads pair t0 + l of it (coalesced) and the batch is staged in LDS;
// then a group of 16 lanes (lane = component) takes every fourth surfel of the
// batch and adds its pairs to the surfel's FP64 sums in LDS.  The sums are the
// same, term by term, as a per-surfel loop over its range, and a batch that
// holds a surfel's 64 pairs costs 64 steps of one read instead of 64 of 16.
// A surfel with more than kHeavyGeo flagged pairs of one camera (a near, large
// one: up to several thousand) would still hold its wave: it is marked in
// `heavy` (a bit per surfel) and left to k_reduce_geo_heavy.  The choice
// depends on its flagged pairs alone.
constexpr int kHeavyGeo = 64;
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_reduce_geo(
    int64_t n, CamTable ct, const uint32_t* __restrict__ vbase, const uint32_t* __restrict__ count, int64_t cap,
    const float* __restrict__ gpart, const uint8_t* __restrict__ gflag, const float* __restrict__ means,
    const float* __restrict__ scales, const float* __restrict__ quats, const int32_t* __restrict__ cull, GeoGrads d,
    uint64_t* __restrict__ heavy) {
  constexpr int kPS = 17;  // LDS row stride of a staged pair (16 partials)
  __shared__ float s_part[4][64 * kPS];
  constexpr int kSS = 65;  // row stride of the sums: a group's 16 components fall in distinct banks
  __shared__ double s_sum[4][16 * kSS];
  __shared__ uint32_t s_pre[4][64];
  __shared__ uint32_t s_vb[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = ((int64_t)blockIdx.x * 4 + wave) * 64 + lane;
  if (i - lane >= n) return;  // no block barriers below
  const bool valid = i < n;   // every lane stays: the wave shares the pair loads
  const int64_t ii = valid ? i : 0;
  const int grp = lane >> 4, comp = lane & 15;
  SurfelGrad acc;
  clear_grad(acc);
  float* part = s_part[wave];
  double* sums = s_sum[wave];
  bool is_heavy = false;
  // the next camera's pair range is loaded while this camera's is summed
  int32_t ncv = valid ? cull[i] : 1;
  uint32_t nvb = valid ? vbase[i] : 0u, nvc = valid ? count[i] : 0u;
#pragma unroll 1
  for (int b = 0; b < ct.n; ++b) {
    const int32_t cv = ncv;
    const uint32_t vb = nvb;
    const int64_t end = min((int64_t)vb + (int64_t)nvc, cap);
    if (b + 1 < ct.n && valid) {
      const int64_t v = (int64_t)(b + 1) * n + i;
      ncv = cull[v];
      nvb = vbase[v];
      nvc = count[v];
    }
    const bool live = valid && (cv & 0xFF) == 0;
    uint32_t cnt = live && end > (int64_t)vb ? (uint32_t)(end - (int64_t)vb) : 0u;
    // long ranges: count the flagged pairs, four flag bytes a lane
    for (uint64_t m = __ballot(cnt > (uint32_t)kHeavyGeo); m; m &= m - 1) {
      const int o = __builtin_ctzll(m);
      const uint32_t p0 = lane_value(vb, o), p1 = p0 + lane_value(cnt, o);
      int nf = 0;
      for (uint32_t w = (p0 >> 2) + (uint32_t)lane; w <= (p1 - 1) >> 2; w += 64) {
        uint32_t x = reinterpret_cast<const uint32_t*>(gflag)[w] & 0x01010101u;
        if (4 * w < p0) x &= 0xFFFFFFFFu << (8 * (p0 - 4 * w));
        if (4 * w + 4 > p1) x &= 0xFFFFFFFFu >> (8 * (4 * w + 4 - p1));
        nf += __popc(x);
      }
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) nf += __shfl_xor(nf, s, 64);
      if (nf > kHeavyGeo && lane == o) {
        is_heavy = true;
        cnt = 0u;
      }
    }
    // the wave's pairs as one flat sequence: surfel l owns [pre_l, pre_l + cnt_l)
    uint32_t xs = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = __shfl_up(xs, o, 64);
      if (lane >= o) xs += t;
    }
    const uint32_t pre = xs - cnt, total = __shfl(xs, 63, 64);
    s_pre[wave][lane] = pre;
    s_vb[wave][lane] = vb;
#pragma unroll
    for (int j = 0; j < 16; ++j) sums[j * kSS + lane] = 0.0;
    wave_lds_sync();
    for (uint32_t t0 = 0; t0 < total; t0 += 64) {
      // 64 consecutive pairs of the sequence, one per lane; unflagged pairs
      // stage zeros (adding +0 leaves a sum unchanged)
      const uint32_t t = t0 + (uint32_t)lane;
      float4 r[4];
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) r[qd] = make_float4(0.f, 0.f, 0.f, 0.f);
      int o = 0;  // owner: the last surfel whose range starts at or before t
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
        if (s_pre[wave][o + step] <= min(t, total - 1)) o += step;
      if (t < total) {
        const uint32_t pr = s_vb[wave][o] + (t - s_pre[wave][o]);
        if (gflag[pr]) {
          const float4* g = reinterpret_cast<const float4*>(gpart + (size_t)pr * 16);
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) r[qd] = g[qd];
        }
      }
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        part[lane * kPS + 4 * qd] = r[qd].x;
        part[lane * kPS + 4 * qd + 1] = r[qd].y;
        part[lane * kPS + 4 * qd + 2] = r[qd].z;
        part[lane * kPS + 4 * qd + 3] = r[qd].w;
      }
      wave_lds_sync();
      // each surfel's pairs of this batch in emission order
      const int s0 = __shfl(o, 0, 64), s1 = __shfl(o, 63, 64);
      for (int s = s0 + ((grp - s0) & 3); s <= s1; s += 4) {
        const uint32_t ps = s_pre[wave][s], pe = s < 63 ? s_pre[wave][s + 1] : total;
        const uint32_t lo = max(ps, t0), hi = min(pe, t0 + 64u);
        if (lo >= hi) continue;
        double g = sums[comp * kSS + s];
        for (uint32_t u = lo; u < hi; ++u) g += part[(u - t0) * kPS + comp];
        sums[comp * kSS + s] = g;
      }
      wave_lds_sync();
    }
    if (live) {
      double G[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) G[j] = sums[j * kSS + lane];
      SurfelParams P;
      load_params(P, ii, means, scales, quats);
      chain_rule(G, ct.cam[b], ((cv >> 8) & 1) != 0, P.mu, P.su, P.sv, P.qn, P.Rq, acc);
    }
    wave_lds_sync();
  }
  const uint64_t hm = __ballot(is_heavy);
  if (lane == 0) heavy[i >> 6] = hm;
  if (!valid || is_heavy) return;
  SurfelParams P;
  load_params(P, ii, means, scales, quats);
  write_grad(acc, P, i, d);
}

// Heavy surfels (bits of `heavy`), a block each: per camera the flagged slots
// are compacted in emission order (256 a step, block prefix count) into an LDS
// list; row lane r of 16 adds, in FP64 and rank order, the rows whose rank
// among the camera's flagged pairs is r mod 16 (lane = component), the 16
// partials are added in row-lane order, and one thread applies the chain rule.
// The partition depends only on the sequence of flagged pairs.
__global__ __launch_bounds__(256) void k_reduce_geo_heavy(
    int64_t n, CamTable ct, const uint32_t* __restrict__ vbase, const uint32_t* __restrict__ count, int64_t cap,
    const float* __restrict__ gpart, const uint8_t* __restrict__ gflag, const float* __restrict__ means,
    const float* __restrict__ scales, const float* __restrict__ quats, const int32_t* __restrict__ cull, GeoGrads d,
    const uint64_t* __restrict__ heavy) {
  constexpr int kList = 2048;
  __shared__ uint32_t s_slot[kList];
  __shared__ double s_row[16][16];
  __shared__ uint64_t s_bits[256];
  __shared__ uint32_t s_red[8];
  const int t = threadIdx.x, comp = t & 15, rl = t >> 4;
  const int64_t words = cdiv(n, 64);
  // this block's words: blockIdx.x, + gridDim.x, ... (read 256 at a time)
  for (int64_t w0 = blockIdx.x; w0 < words; w0 += 256 * (int64_t)gridDim.x) {
    __syncthreads();
    const int64_t wt = w0 + (int64_t)t * gridDim.x;
    s_bits[t] = wt < words ? heavy[wt] : 0ull;
    const int any = __syncthreads_or(s_bits[t] != 0ull);
    if (!any) continue;
    const int nq = (int)min((int64_t)256, cdiv(words - w0, gridDim.x));
    for (int q = 0; q < nq; ++q) {
      for (uint64_t m = s_bits[q]; m; m &= m - 1) {
        const int64_t i = (w0 + (int64_t)q * gridDim.x) * 64 + __builtin_ctzll(m);
        SurfelGrad acc;
        clear_grad(acc);
        SurfelParams P;
        if (t == 0) load_params(P, i, means, scales, quats);
        for (int b = 0; b < ct.n; ++b) {
          const int64_t v = (int64_t)b * n + i;
          const int32_t cv = cull[v];
          if ((cv & 0xFF) != 0) continue;
          const int64_t base = vbase[v], end = min(base + (int64_t)count[v], cap);
          double sum = 0.0;
          uint32_t nl = 0, rank0 = 0;  // listed slots, rank of the first (block-uniform)
          auto drain = [&]() {
            __syncthreads();
            for (uint32_t j = (rl - rank0) & 15u; j < nl; j += 64) {
              float x[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) x[u] = j + 16 * u < nl ? gpart[(size_t)s_slot[j + 16 * u] * 16 + comp] : 0.0f;
#pragma unroll
              for (int u = 0; u < 4; ++u) sum += x[u];
            }
            rank0 += nl;
            nl = 0;
            __syncthreads();
          };
          for (int64_t c0 = base; c0 < end; c0 += 256) {
            const bool f = c0 + t < end && gflag[c0 + t];
            uint32_t total;
            const uint32_t pre = block_scan_excl(f ? 1u : 0u, s_red, total);
            if (f) s_slot[nl + pre] = (uint32_t)(c0 + t);  // nl <= kList - 256 here
            nl += total;
            if (nl > (uint32_t)(kList - 256)) drain();
          }
          drain();
          s_row[rl][comp] = sum;
          __syncthreads();
          if (t == 0) {
            double G[16];
            for (int j = 0; j < 16; ++j) {
              G[j] = s_row[0][j];
              for (int r = 1; r < 16; ++r) G[j] += s_row[r][j];
            }
            chain_rule(G, ct.cam[b], ((cv >> 8) & 1) != 0, P.mu, P.su, P.sv, P.qn, P.Rq, acc);
          }
          __syncthreads();
        }
        if (t == 0) write_grad(acc, P, i, d);
      }
    }
  }
}

// Lane group per surfel: dL/df = sum over cameras (in order) of the sum of its
// pairs' rows (emission order), channels [0, ca) written to dfa (row stride
// ca), channels [ca, C) to dfb (row stride C - ca); either may be null.
// A surfel with more than kHeavyRows flagged rows is not summed here (its
// rows would follow one another, four per round trip, and hold the whole
// kernel): the group stops when its count passes the bound and puts the
// surfel on the heavy list for k_reduce_feat_heavy.  The choice depends only
// on the surfel's flagged rows, like each path's order of addition.
template <int NG>
__global__ __launch_bounds__(256) void k_reduce_feat(int64_t n, int ncam, const uint32_t* __restrict__ vbase,
                                                     const uint32_t* __restrict__ count, int64_t cap,
                                                     const float* __restrict__ fpart,
                                                     const uint8_t* __restrict__ fflag, int C, int lpp2,
                                                     float* __restrict__ dfa, float* __restrict__ dfb, int ca,
                                                     uint32_t* __restrict__ heavy, uint32_t* __restrict__ status) {
  // lpp2 lanes (a power of two) per surfel, each lane up to NG float4 channel
  // groups: a wave reduces 64 / lpp2 surfels at once
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lpp = C / 4;
  const int spw = 64 / lpp2;
  const int sub = lane / lpp2, cl = lane % lpp2;
  const int64_t i = ((int64_t)blockIdx.x * 4 + wave) * spw + sub;
  if (i >= n) return;
  constexpr int kMaxGroups = NG;  // channel groups of 4 per lane (the registers it needs)
  constexpr int kRowsInFlight = 4;
  uint32_t nf = 0;  // flagged rows met so far (the same in every lane of the group)
  float4 acc[kMaxGroups];
#pragma unroll
  for (int j = 0; j < kMaxGroups; ++j) acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  const int ng = (lpp + lpp2 - 1) / lpp2;  // channel groups of this lane
  const uint64_t gmask = lpp2 == 64 ? ~0ull : ((1ull << lpp2) - 1ull);
  uint32_t nvb = vbase[i], nvc = count[i];
#pragma unroll 1
  for (int b = 0; b < ncam; ++b) {
    const int64_t base = nvb;
    const int64_t end = min(base + (int64_t)nvc, cap);
    if (b + 1 < ncam) {
      const int64_t v = (int64_t)(b + 1) * n + i;
      nvb = vbase[v];
      nvc = count[v];
    }
    // a scan tests `steps` strides of lpp2 flags at once (up to 64 slots, one
    // 64-bit mask: bit t = slot s0 + t), so a surfel with many pairs and few
    // flagged rows waits for one flag load per 64 slots, not per lpp2; the
    // flagged rows in emission order, up to kRowsInFlight rows loaded before
    // they are added
    const int steps = lpp2 >= 8 ? 64 / lpp2 : 8;
    for (int64_t s0 = base; s0 < end; s0 += (int64_t)steps * lpp2) {
      bool fl[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int64_t sj = s0 + (int64_t)j * lpp2 + cl;
        fl[j] = j < steps && sj < end && fflag[sj];
      }
      uint64_t m = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j < steps) m |= ((__ballot(fl[j]) >> (sub * lpp2)) & gmask) << (j * lpp2);
      nf += (uint32_t)__popcll(m);
      if (nf > (uint32_t)kHeavyRows) {
        if (cl == 0) heavy[atomicAdd(status + kStHeavy, 1u)] = (uint32_t)i;
        return;
      }
      while (m) {
        int us[kRowsInFlight];
#pragma unroll
        for (int r = 0; r < kRowsInFlight; ++r) {
          us[r] = m ? __ffsll((unsigned long long)m) - 1 : -1;
          m &= m - 1ull;
        }
        float4 t[kRowsInFlight][kMaxGroups];
#pragma unroll
        for (int r = 0; r < kRowsInFlight; ++r) {
          const float* row = fpart + (size_t)(s0 + max(us[r], 0)) * C;
#pragma unroll
          for (int j = 0; j < kMaxGroups; ++j)
            t[r][j] = us[r] >= 0 && j < ng && cl + j * lpp2 < lpp
                          ? *reinterpret_cast<const float4*>(row + (cl + j * lpp2) * 4)
                          : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int r = 0; r < kRowsInFlight; ++r)
#pragma unroll
          for (int j = 0; j < kMaxGroups; ++j)
            if (us[r] >= 0) {
              acc[j].x += t[r][j].x; acc[j].y += t[r][j].y; acc[j].z += t[r][j].z; acc[j].w += t[r][j].w;
            }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kMaxGroups; ++j)
    if (j < ng && cl + j * lpp2 < lpp) {
      const int c = (cl + j * lpp2) * 4;  // ca % 4 == 0: the group lies in one output
      float* dst = c < ca ? (dfa ? dfa + (size_t)i * ca + c : nullptr)
                          : (dfb ? dfb + (size_t)i * (C - ca) + (c - ca) : nullptr);
      if (dst) *reinterpret_cast<float4*>(dst) = acc[j];
    }
}

// Block per heavy surfel (a fixed grid strides over the heavy list, whose
// length it reads on the device): CL channel lanes (float4 groups) x R =
// 1024 / CL row lanes.  The surfel's flagged slots are compacted in emission
// order (camera by camera, 1024 slots a step, block prefix count) into an LDS
// list; row lane r adds, in rank order, the rows whose rank among the
// surfel's flagged rows is r mod R, eight rows in flight, and the R partial
// rows are then added in row-lane order.  The partition depends only on the
// sequence of flagged rows: the result is deterministic, the same for every
// launch choice, and unchanged by pairs that carry no row.  The longest
// surfel's rows bound the kernel, so as many as registers allow are in flight:
// 1M street surfels, C = 256: 390 -> 167 us against 256 threads and four rows.
constexpr int kHvList = 2048, kHvThreads = 1024, kHvFly = 8;
__global__ __launch_bounds__(kHvThreads) void k_reduce_feat_heavy(int64_t n, int ncam, const uint32_t* __restrict__ vbase,
                                                           const uint32_t* __restrict__ count, int64_t cap,
                                                           const float* __restrict__ fpart,
                                                           const uint8_t* __restrict__ fflag, int C,
                                                           float* __restrict__ dfa, float* __restrict__ dfb, int ca,
                                                           const uint32_t* __restrict__ heavy,
                                                           const uint32_t* __restrict__ status) {
  __shared__ uint32_t s_slot[kHvList];
  __shared__ float4 s_acc[kHvThreads];
  __shared__ uint32_t s_red[kHvThreads / 64];
  const int t = threadIdx.x;
  const int G = C / 4, CL = min(G, 64), R = kHvThreads / CL;
  const int rl = t / CL, cl = t % CL;
  const uint32_t nh = status[kStHeavy];
  for (uint32_t h = blockIdx.x; h < nh; h += gridDim.x) {
    const int64_t i = heavy[h];
    for (int g0 = 0; g0 < G; g0 += CL) {
      const int g = g0 + cl;
      float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
      uint32_t nl = 0, rank0 = 0;  // listed slots, rank of the first (block-uniform)
      // the listed rows added by their row lanes; the list is then empty
      auto drain = [&]() {
        __syncthreads();
        if (rl < R && g < G) {
          for (uint32_t j = (uint32_t)((rl + R - (int)(rank0 % (uint32_t)R)) % R); j < nl; j += (uint32_t)(kHvFly * R)) {
            float4 x[kHvFly];
#pragma unroll
            for (int u = 0; u < kHvFly; ++u) {
              const uint32_t jj = j + (uint32_t)(u * R);
              x[u] = jj < nl ? *reinterpret_cast<const float4*>(fpart + (size_t)s_slot[jj] * C + 4 * g)
                             : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < kHvFly; ++u) {
              acc.x += x[u].x; acc.y += x[u].y; acc.z += x[u].z; acc.w += x[u].w;
            }
          }
        }
        rank0 += nl;
        nl = 0;
        __syncthreads();
      };
      for (int b = 0; b < ncam; ++b) {
        const int64_t v = (int64_t)b * n + i, base = vbase[v];
        const int64_t end = min(base + (int64_t)count[v], cap);
        for (int64_t c0 = base; c0 < end; c0 += kHvThreads) {
          const bool f = c0 + t < end && fflag[c0 + t];
          uint32_t total;
          const uint32_t pre = block_scan_excl<kHvThreads>(f ? 1u : 0u, s_red, total);
          if (f) s_slot[nl + pre] = (uint32_t)(c0 + t);  // nl <= kHvList - kHvThreads here
          nl += total;
          if (nl > (uint32_t)(kHvList - kHvThreads)) drain();
        }
      }
      drain();
      s_acc[t] = acc;
      __syncthreads();
      if (rl == 0 && g < G) {
        float4 sum = s_acc[cl];
        for (int r = 1; r < R; ++r) {
          const float4 y = s_acc[r * CL + cl];
          sum.x += y.x; sum.y += y.y; sum.z += y.z; sum.w += y.w;
        }
        const int c = 4 * g;  // ca % 4 == 0: the group lies in one output
        float* dst = c < ca ? (dfa ? dfa + (size_t)i * ca + c : nullptr)
                            : (dfb ? dfb + (size_t)i * (C - ca) + (c - ca) : nullptr);
        if (dst) *reinterpret_cast<float4*>(dst) = sum;
      }
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------- host wrappers
template <typename FT, int KMAX, bool SPLIT>
static void feat_bwd_launch(const SurfelArgs& s, const Layout& L, const CamTable& ct, const Tuning& tu,
                            const ImageGradArgs& g, bool renorm, char* ws, hipStream_t st) {
  hipLaunchKernelGGL((k_feat_bwd_topk<FT, KMAX, SPLIT>), dim3(xcd_grid(L.tiles)), dim3(kFbThreads),
                     2 * kFbPart * sizeof(float), st,
                     (const uint32_t*)(ws + L.pid), (const uint32_t*)(ws + L.eid0), (const uint2*)(ws + L.ranges),
                     (const int32_t*)(ws + L.selpos), (const float*)(ws + L.selw), feat_src<FT>(s), g.feat, s.c, L.k,
                     ct, tile_order(L, tu.sched_bwd, ws), (float*)(ws + L.seldot), (float*)(ws + L.fpart),
                     (uint8_t*)(ws + L.fflag), renorm ? 1 : 0);
}

template <typename FT, bool SPLIT>
static void feat_bwd_k(const SurfelArgs& s, const Layout& L, const CamTable& ct, const Tuning& tu,
                       const ImageGradArgs& g, bool rn, char* ws, hipStream_t st) {
  if (L.k <= 8) feat_bwd_launch<FT, 8, SPLIT>(s, L, ct, tu, g, rn, ws, st);
  else if (L.k <= 16) feat_bwd_launch<FT, 16, SPLIT>(s, L, ct, tu, g, rn, ws, st);
  else feat_bwd_launch<FT, 32, SPLIT>(s, L, ct, tu, g, rn, ws, st);
}

template <int MODE, typename FT, bool LP, bool DM>
static void walk_bwd_launch_d(const SurfelArgs& s, const Layout& L, const CamTable& ct, const Tuning& tu,
                              const ImageGradArgs& g, bool want_f, char* ws, hipStream_t st) {
  const size_t shm = MODE == kTopK ? (size_t)L.k * kTilePix * 2 : 0;  // selection positions
  hipLaunchKernelGGL((k_walk_bwd<MODE, FT, LP, DM>), dim3(xcd_grid(L.tiles)), dim3(256), shm,
                     st, (const WalkRec*)(ws + L.rec), (const uint32_t*)(ws + L.pid),
                     (const uint32_t*)(ws + L.eid0), (const uint2*)(ws + L.ranges), ct,
                     tile_order(L, tu.sched_bwd, ws), L.k,
                     (const uint32_t*)(ws + L.nlast), (const float*)(ws + L.tfinal), (const int32_t*)(ws + L.selpos),
                     (const float*)(ws + L.seldot), g.rgb, g.depth, g.normal, g.alpha, want_f ? g.feat : nullptr,
                     feat_src<FT>(s), s.c, (float*)(ws + L.gpart), (uint8_t*)(ws + L.gflag), (float*)(ws + L.fpart),
                     (uint8_t*)(ws + L.fflag));
}

// dense mode: the feature-backward pass width selects the contraction unit
// (16: vector FMAs, 32: matrix cores)
template <int MODE, typename FT, bool LP>
static void walk_bwd_launch_t(const SurfelArgs& s, const Layout& L, const CamTable& ct, const Tuning& tu,
                              const ImageGradArgs& g, bool want_f, char* ws, hipStream_t st) {
  if (MODE == kFull && tu.bwd_pass == 32) walk_bwd_launch_d<MODE, FT, LP, true>(s, L, ct, tu, g, want_f, ws, st);
  else walk_bwd_launch_d<MODE, FT, LP, false>(s, L, ct, tu, g, want_f, ws, st);
}

template <int MODE, typename FT>
static void walk_bwd_launch(const SurfelArgs& s, const Layout& L, const CamTable& ct, const Tuning& tu,
                            const ImageGradArgs& g, bool want_f, bool lp, char* ws, hipStream_t st) {
  (lp ? walk_bwd_launch_t<MODE, FT, true> : walk_bwd_launch_t<MODE, FT, false>)(s, L, ct, tu, g, want_f, ws, st);
}

template <typename FT>
static void backward_typed(const SurfelArgs& s, const CamTable& ct, int blend, const Tuning& tu, const Layout& L,
                           const ImageGradArgs& g, const GradArgs& gr, bool renorm, bool lp, char* ws,
                           hipStream_t st, const ProfHook& prof) {
  const bool want_f = g.feat != nullptr && s.c > 0;
  if (L.tiles > 0) {
    if (blend == kTopK) {
      prof.begin(kStageBwdFeature, st);
      if (want_f) {
        if (feat_src<FT>(s).cb > 0) feat_bwd_k<FT, true>(s, L, ct, tu, g, renorm, ws, st);
        else feat_bwd_k<FT, false>(s, L, ct, tu, g, renorm, ws, st);
      } else {
        launch_fill_u32(ws + L.seldot, 0u, L.spix * (int64_t)L.k, st);
      }
      prof.end(kStageBwdFeature, st);
      prof.begin(kStageBwdWalk, st);
      walk_bwd_launch<kTopK, FT>(s, L, ct, tu, g, want_f, lp, ws, st);
      prof.end(kStageBwdWalk, st);
    } else {
      prof.begin(kStageBwdWalk, st);
      walk_bwd_launch<kFull, FT>(s, L, ct, tu, g, want_f, lp, ws, st);
      prof.end(kStageBwdWalk, st);
    }
  }
  prof.begin(kStageBwdPreprocess, st);
  const uint32_t* vbase = (const uint32_t*)(ws + L.vbase);
  const uint32_t* count = (const uint32_t*)(ws + L.count);
  if (s.n > 0) {
    const GeoGrads gg{gr.means, gr.scales, gr.quats, gr.opacity, gr.rgb};
    uint64_t* hbits = (uint64_t*)(ws + L.hbits);  // a bit per surfel (the region holds a word per virtual surfel)
    hipLaunchKernelGGL(k_reduce_geo, dim3((unsigned)cdiv(s.n, 256)), dim3(256), 0, st, s.n, ct, vbase, count, L.cap,
                       (const float*)(ws + L.gpart), (const uint8_t*)(ws + L.gflag), s.means, s.scales, s.quats,
                       (const int32_t*)(ws + L.cull), gg, hbits);
    if (L.cap > kHeavyGeo) {
      const unsigned gh = (unsigned)std::min<int64_t>(cdiv(s.n, 64), 1024);
      hipLaunchKernelGGL(k_reduce_geo_heavy, dim3(gh), dim3(256), 0, st, s.n, ct, vbase, count, L.cap,
                         (const float*)(ws + L.gpart), (const uint8_t*)(ws + L.gflag), s.means, s.scales, s.quats,
                         (const int32_t*)(ws + L.cull), gg, (const uint64_t*)hbits);
    }
    if (s.c > 0 && (gr.feat || gr.feat_ext)) {
      // two channel groups per lane (at most 4 for C = 1024): more surfels,
      // and so more independent row loads, in flight per wave
      const int lpp = s.c / 4;
      const int lpp2 = std::min(64, pow2_ge_host((lpp + 1) / 2));
      const int per_block = 4 * (64 / lpp2);
      const int ng = (lpp + lpp2 - 1) / lpp2;  // 1 or 2 up to C = 512, else at most 4
      auto k = ng <= 2 ? k_reduce_feat<2> : k_reduce_feat<4>;
      uint32_t* status = (uint32_t*)(ws + L.status);
      uint32_t* heavy = (uint32_t*)(ws + L.heavy);
      launch_fill_u32(status + kStHeavy, 0u, 1, st);
      hipLaunchKernelGGL(k, dim3((unsigned)cdiv(s.n, per_block)), dim3(256), 0, st, s.n, ct.n, vbase,
                         count, L.cap, (const float*)(ws + L.fpart), (const uint8_t*)(ws + L.fflag), s.c, lpp2,
                         gr.feat, gr.feat_ext, s.ca, heavy, status);
      const unsigned gh = (unsigned)std::min<int64_t>(L.cap / (kHeavyRows + 1) + 1, 1024);
      hipLaunchKernelGGL(k_reduce_feat_heavy, dim3(gh), dim3(kHvThreads), 0, st, s.n, ct.n, vbase, count, L.cap,
                         (const float*)(ws + L.fpart), (const uint8_t*)(ws + L.fflag), s.c, gr.feat, gr.feat_ext, s.ca,
                         (const uint32_t*)heavy, (const uint32_t*)status);
    }
  }
  prof.end(kStageBwdPreprocess, st);
}

void launch_backward(const SurfelArgs& s, const CamTable& ct, int blend, const Tuning& tu, const Layout& L,
                     const ImageGradArgs& g, const GradArgs& grads, bool renorm, bool lowpass, char* ws,
                     hipStream_t st, const ProfHook& prof) {
  prof.begin(kStageFill, st);
  launch_fill_u32(ws + L.gflag, 0u, cdiv(std::max<int64_t>(L.cap, 1), 4), st);
  launch_fill_u32(ws + L.fflag, 0u, cdiv(std::max<int64_t>(L.cap, 1), 4), st);
  prof.end(kStageFill, st);
  if (s.dtype == kF32) backward_typed<float>(s, ct, blend, tu, L, g, grads, renorm, lowpass, ws, st, prof);
  else if (s.dtype == kF16) backward_typed<__half>(s, ct, blend, tu, L, g, grads, renorm, lowpass, ws, st, prof);
  else backward_typed<uint16_t>(s, ct, blend, tu, L, g, grads, renorm, lowpass, ws, st, prof);
}

}  // namespace psm
