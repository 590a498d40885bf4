// Forward render of a selected set (Sec. 3: EWA projection, SH colour, Eq. 1
// front-to-back compositing with Eq. 2's alpha), tiled 16x16.
//
//  k_project  one thread per selected node: camera transform, near-plane test,
//             covariance from (scale, rotation), EWA Jacobian, projected
//             covariance + 0.3 px^2, conic, square footprint, tile rectangle,
//             opacity, SH colour.  Writes a 64-byte Splat record, the depth key
//             and the tile count (0 for a splat that is not drawn).
//  k_drawn_scan  ranks of the drawn splats (selection order) and their first
//             instance.
//  k_dup      one (tile, splat) instance per covered tile, with its block mask,
//             and the tiles' instance counts.
//  k_tile_scan  the tiles' ranges of the instance list, and the tiles by
//             descending count.
//  k_bucket   the instances' (depth, index) keys into their tile's range.
//  k_tile_sort, k_tile_merge  each tile's keys in LDS: by FP32 depth bits, ties
//             by selection order.  The list is then in the order of the
//             64-bit key (tile << 32 | depth), ties by selection order.
//             No splat or instance passes through a global radix sort: a sort
//             by depth of the splats and one by tile of the instances took 18
//             launches (82 of a 512 x 512 view's 164 us; 288 us of a street
//             view with 0.95M drawn splats and 2.1M instances), the six
//             kernels from k_drawn_scan on take 28 and 162 us there.
//  k_blend_fwd  a wave per 8x8 quarter or per 4x4 block of a tile; k_blend is
//             its general form, one workgroup per tile with PX pixels per
//             lane, and the evaluation count.  A 4x4 block replays only the
//             splats whose alpha >= 1/255 ellipse reaches it (elsewhere the
//             result is known).
#include "lodgs_internal.h"
#include "lodgs_proj.h"

namespace lodgs {

// Projection of one node.  The per-splat chain runs in FP64 with a fixed
// operation order (scales from the FP32 exp, opacity as the FP32 sigmoid);
// its decisions (near plane, positive determinant, footprint radius, tile
// rectangle) are taken in FP64 and its outputs rounded to the FP32 record.
struct Proj {
  bool visible;
  float depth;
  Splat sp;
  int x0, x1, y0, y1;
};

__device__ __forceinline__ int tile_clamp(double v, int hi) {
  if (v < 0.0) return 0;
  if (v > (double)hi) return hi;
  return (int)v;
}

__device__ __forceinline__ Proj project_node(const SceneDev& S, const ViewConst& v, int32_t node) {
  Proj P;
  P.visible = false;
  P.x0 = P.x1 = P.y0 = P.y1 = 0;
  const int64_t n = node;
  // every parameter but the colour is requested up front, before the
  // near-plane test needs the mean
  const NodeGeom geo = load_geom(S.means, S.log_scales, S.quats, n);
  const float theta = S.opacity_logits[n];
  Proj64 G;
  const bool ok = proj_chain64(geo, v, G);
  P.depth = (float)G.c[2];
  if (!ok) return P;
  const double A = G.A, B = G.B, C = G.C, det = G.det;
  const double fx = v.fx, fy = v.fy, u = G.u, vv = G.v;
  const double mx = fx * u + (double)v.cx, my = fy * vv + (double)v.cy;
  const double mid = 0.5 * (A + C);
  const double disc = mid * mid - det;
  const double r = ceil(3.0 * __builtin_sqrt(mid + __builtin_sqrt(fmax(0.1, disc))));
  P.x0 = tile_clamp(floor((mx - r) * 0.0625), v.tiles_x);
  P.x1 = tile_clamp(floor((mx + r) * 0.0625) + 1.0, v.tiles_x);
  P.y0 = tile_clamp(floor((my - r) * 0.0625), v.tiles_y);
  P.y1 = tile_clamp(floor((my + r) * 0.0625) + 1.0, v.tiles_y);
  P.visible = P.x1 > P.x0 && P.y1 > P.y0;
  // principal axes of the projected covariance
  const double l1 = mid + __builtin_sqrt(fmax(0.0, disc));
  const double l2 = det / l1;
  double vx, vy;
  if (A >= C) {
    vx = l1 - C;
    vy = B;
  } else {
    vx = B;
    vy = l1 - A;
  }
  const double nn = __builtin_sqrt(vx * vx + vy * vy);
  double ce = 1.0, se = 0.0;
  if (nn > 0.0) {
    ce = vx / nn;
    se = vy / nn;
  }
  P.sp.mxh = (float)mx;
  P.sp.mxl = (float)(mx - (double)P.sp.mxh);
  P.sp.myh = (float)my;
  P.sp.myl = (float)(my - (double)P.sp.myh);
  P.sp.ce = (float)ce;
  P.sp.se = (float)se;
  P.sp.h1 = (float)(-0.5 / l1);
  P.sp.h2 = (float)(-0.5 / l2);
  P.sp.o = 1.0f / (1.0f + fexp(-theta));
  P.sp.rect_x = (uint32_t)P.x0 | ((uint32_t)P.x1 << 16);
  P.sp.rect_y = (uint32_t)P.y0 | ((uint32_t)P.y1 << 16);
  P.sp.pad0 = P.sp.pad1 = 0u;
  return P;
}

// SH colour for the view direction (mu - pos) / |mu - pos|; returns the
// unclamped value in raw[3] and, in J[3 c + a], the derivative of channel c
// with respect to component a of the unit direction (sum over the basis of
// coefficient times basis gradient), which the colour backward takes in place
// of the coefficients, and the unit direction and 1 / |mu - pos| it used.
template <int DEG>
__device__ __forceinline__ void sh_color(const SceneDev& S, const ViewConst& v, int64_t n, float* raw, float* J,
                                         float* dir, float& inv_len) {
  const float dx = S.means[3 * n] - v.pos[0], dy = S.means[3 * n + 1] - v.pos[1], dz = S.means[3 * n + 2] - v.pos[2];
  const float il = 1.0f / __builtin_sqrtf(dx * dx + dy * dy + dz * dz);
  dir[0] = dx * il;
  dir[1] = dy * il;
  dir[2] = dz * il;
  inv_len = il;
  float Y[16], dY[16][3];
  sh_basis(DEG, dir[0], dir[1], dir[2], Y);
  sh_basis_grad(DEG, dir[0], dir[1], dir[2], dY);
  constexpr int nb = (DEG + 1) * (DEG + 1), nc = 3 * nb;
  // the coefficient row, as float4s when its length allows (rows are 16-byte
  // aligned: the scene's array is, and a row is a multiple of 16 bytes)
  float c[nc];
  if (nc % 4 == 0) {
    const float4* c4 = reinterpret_cast<const float4*>(S.sh + (int64_t)nc * n);
#pragma unroll
    for (int q = 0; q < nc / 4; ++q) {
      const float4 x = c4[q];
      c[4 * q] = x.x;
      c[4 * q + 1] = x.y;
      c[4 * q + 2] = x.z;
      c[4 * q + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int f = 0; f < nc; ++f) c[f] = S.sh[(int64_t)nc * n + f];
  }
  float r = 0.5f, g = 0.5f, b = 0.5f;
#pragma unroll
  for (int q = 0; q < 9; ++q) J[q] = 0.0f;
#pragma unroll
  for (int k = 0; k < nb; ++k) {
    const float c0 = c[3 * k], c1 = c[3 * k + 1], c2 = c[3 * k + 2];
    r = __builtin_fmaf(c0, Y[k], r);
    g = __builtin_fmaf(c1, Y[k], g);
    b = __builtin_fmaf(c2, Y[k], b);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      J[a] = __builtin_fmaf(c0, dY[k][a], J[a]);
      J[3 + a] = __builtin_fmaf(c1, dY[k][a], J[3 + a]);
      J[6 + a] = __builtin_fmaf(c2, dY[k][a], J[6 + a]);
    }
  }
  raw[0] = r;
  raw[1] = g;
  raw[2] = b;
}

template <int DEG>
__global__ void __launch_bounds__(kBlock, 3) k_project(SceneDev S, const ViewConst* __restrict__ vp, const int32_t* idx,
                                                    const int32_t* d_count, int64_t cap, Splat* splats,
                                                    uint32_t* depth_key, uint32_t* tiles, ushort4* rect,
                                                    float* dcol, uint2* wave_sums,
                                                    unsigned long long* run_sums) {
  const ViewConst v = *vp;
  const int64_t n = clamp_count(d_count, cap);
  const int lane = threadIdx.x & 63;
  for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63); i0 < n;
       i0 += (int64_t)gridDim.x * blockDim.x) {  // wave-uniform
    const int64_t i = i0 + lane;
    uint32_t t = 0;
    Proj P;
    P.visible = false;
    const int32_t node = i < n ? idx[i] : 0;
    if (i < n) P = project_node(S, v, node);
    if (P.visible) {
      float raw[3], J[9], dir[3], il;
      sh_color<DEG>(S, v, node, raw, J, dir, il);
      P.sp.r = fmaxf(raw[0], 0.0f);
      P.sp.g = fmaxf(raw[1], 0.0f);
      P.sp.b = fmaxf(raw[2], 0.0f);
      const uint32_t clamp = (raw[0] < 0.0f ? 1u : 0u) | (raw[1] < 0.0f ? 2u : 0u) | (raw[2] < 0.0f ? 4u : 0u);
      // the colour backward's record: everything it needs but the gradients
      float4* rec = reinterpret_cast<float4*>(dcol + kColorRec * i);
      rec[0] = make_float4(J[0], J[1], J[2], J[3]);
      rec[1] = make_float4(J[4], J[5], J[6], J[7]);
      rec[2] = make_float4(J[8], dir[0], dir[1], dir[2]);
      rec[3] = make_float4(il, __uint_as_float(clamp), 0.0f, 0.0f);
      t = (uint32_t)((P.x1 - P.x0) * (P.y1 - P.y0));
      splats[i] = P.sp;
      depth_key[i] = __float_as_uint(P.depth);
      rect[i] = make_ushort4((unsigned short)P.x0, (unsigned short)P.x1, (unsigned short)P.y0, (unsigned short)P.y1);
    }
    if (i < n) tiles[i] = t;  // 0: not drawn
    const uint32_t drawn = (uint32_t)__popcll(__ballot(t != 0u));
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) t += __shfl_xor(t, d, 64);  // (a splat has at most 2^20 tiles)
    if (lane == 0) {
      if (n <= kDrawnWide) wave_sums[i0 >> 6] = make_uint2(t, drawn);
      else if (drawn != 0u) atomicAdd(&run_sums[i0 / kDrawnRun], (unsigned long long)drawn << 32 | t);
    }
  }
}

// Ranks of the drawn splats and their first instances in one launch: the scan
// of (drawn, tile count) over the selection, in order, written for each drawn
// position as its place in the list of drawn positions and the index of its
// first instance, and for each 64-instance chunk the rank of the splat that
// holds its first instance (k_dup's chunks).  A workgroup takes a tile of 2
// positions per thread and adds up the projection's sums of all positions
// before it itself, so none waits for another (look-back over tiles numbered
// by ticket: 6.2 us at 170K positions, 16 at 1.5M).  Above kDrawnWide they are
// sums of 2048 positions, which the projection's waves make with atomics (2 us
// of a small view's projection, so not below): 12.8 us for a street view with
// 0.95M drawn splats, where sums of 64 and 8 positions a thread took 16.2.
constexpr int kDrawnThreads = 1024;
constexpr int kDrawnItems = 2;
static_assert(kDrawnThreads * kDrawnItems == kDrawnRun, "a tile is a run");

__device__ __forceinline__ void drawn_tile(const uint32_t* __restrict__ tiles, const uint2* __restrict__ wave_sums,
                                           const unsigned long long* __restrict__ run_sums, int64_t n, int64_t tile,
                                           bool last, FrameCounters* ctr, uint32_t* list, uint32_t* off,
                                           uint32_t* chunk_first, int64_t chunks, uint32_t (*wt)[kDrawnThreads / 64]) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t i0 = (tile * kDrawnThreads + t) * kDrawnItems;
  uint32_t v[kDrawnItems];
  if (i0 + kDrawnItems <= n) {
    const uint2 a = *reinterpret_cast<const uint2*>(tiles + i0);
    v[0] = a.x; v[1] = a.y;
  } else {
#pragma unroll
    for (int k = 0; k < kDrawnItems; ++k) v[k] = i0 + k < n ? tiles[i0 + k] : 0u;
  }
  uint32_t bc = 0, bd = 0;  // this thread's part of the positions before the tile
  if (n <= kDrawnWide) {
#pragma unroll 4
    for (int64_t i = t; i < tile * (kDrawnRun / 64); i += kDrawnThreads) {
      const uint2 a = wave_sums[i];
      bc = add_sat(bc, a.x);
      bd += a.y;
    }
  } else {
#pragma unroll 4
    for (int64_t i = t; i < tile; i += kDrawnThreads) {
      const unsigned long long a = run_sums[i];
      bc = add_sat(bc, (uint32_t)a);
      bd += (uint32_t)(a >> 32);
    }
  }
  uint32_t c = 0, d = 0;
#pragma unroll
  for (int k = 0; k < kDrawnItems; ++k) {
    c += v[k];
    d += v[k] != 0u ? 1u : 0u;
  }
  uint32_t xc = c, xd = d;
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    const uint32_t yc = __shfl_up(xc, s, 64), yd = __shfl_up(xd, s, 64);
    if (lane >= s) {
      xc = add_sat(xc, yc);
      xd += yd;
    }
    bc = add_sat(bc, __shfl_xor(bc, s, 64));
    bd += __shfl_xor(bd, s, 64);
  }
  uint32_t oc = __shfl_up(xc, 1, 64), od = xd - d;  // of the wave's lanes before
  oc = lane == 0 ? 0u : oc;
  if (lane == 63) {
    wt[0][wv] = xd;
    wt[1][wv] = xc;
    wt[2][wv] = bd;
    wt[3][wv] = bc;
  }
  __syncthreads();
  uint32_t td = 0, tc = 0, pd = 0, pc = 0;
#pragma unroll
  for (int w = 0; w < kDrawnThreads / 64; ++w) {
    const uint32_t wd = wt[0][w], wc = wt[1][w];
    od += w < wv ? wd : 0u;
    oc = add_sat(oc, w < wv ? wc : 0u);
    td += wd;
    tc = add_sat(tc, wc);
    pd += wt[2][w];
    pc = add_sat(pc, wt[3][w]);
  }
  if (last && t == 0) {
    ctr->n_drawn = (int32_t)(pd + td);
    ctr->n_instances = (int32_t)add_sat(pc, tc);
  }
  od += pd;
  oc = add_sat(oc, pc);
#pragma unroll
  for (int k = 0; k < kDrawnItems; ++k) {
    const uint32_t end = add_sat(oc, v[k]);
    uint32_t ch = 0, ch_end = 0;  // the chunks that start in [oc, end)
    if (v[k] != 0u) {
      list[od] = (uint32_t)(i0 + k);
      off[od] = oc;
      if ((int64_t)oc < 64 * chunks) {
        ch = (oc + 63u) / 64u;
        ch_end = (uint32_t)min((int64_t)((end - 1u) / 64u) + 1, chunks);
        if (ch < ch_end) chunk_first[ch++] = od;
      }
    }
    // a splat of many chunks is noted by its whole wave
    for (uint64_t more = __ballot(ch < ch_end); more; more &= more - 1) {  // wave-uniform
      const int l = __builtin_ctzll(more);
      const uint32_t b = __shfl(ch, l, 64), e = __shfl(ch_end, l, 64), r = __shfl(od, l, 64);
      for (uint32_t q = b + lane; q < e; q += 64) chunk_first[q] = r;
    }
    od += v[k] != 0u ? 1u : 0u;
    oc = end;
  }
}

__global__ void __launch_bounds__(kDrawnThreads) k_drawn_scan(const uint32_t* __restrict__ tiles,
                                                              const uint2* __restrict__ wave_sums,
                                                              const unsigned long long* __restrict__ run_sums,
                                                              FrameCounters* ctr, uint32_t* list, uint32_t* off,
                                                              uint32_t* chunk_first, int64_t icap) {
  __shared__ uint32_t wt[4][kDrawnThreads / 64];
  const int64_t n = ctr->n_render, chunks = (icap + 63) / 64;
  const int64_t ntiles = (n + kDrawnRun - 1) / kDrawnRun;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {  // block-uniform
    drawn_tile(tiles, wave_sums, run_sums, n, tile, tile == ntiles - 1, ctr, list, off, chunk_first, chunks, wt);
    __syncthreads();
  }
}

// Instance emission, load-balanced over the instances: the instances (splat,
// tile) in selection order of their splats are cut into chunks of 64 and each
// wave takes a contiguous run of chunks.  The drawn splats whose instances
// meet a chunk (at most 64, as every drawn splat has one) start at the one
// k_drawn_scan noted for the wave's first chunk; one comparison per chunk
// gives the next.  Lane l loads the l-th of them (splat,
// rectangle, 64-byte record, depth key and the per-splat part of the block
// mask) into LDS; lane l then emits instance k0 + l, whose splat is the last
// one starting at or before it (a binary search over the chunk's splats in
// LDS).  An instance is its tile (row-major in the rectangle) and depth key,
// and the (splat, block mask) word: the 4x4 blocks of the tile that the
// splat's alpha >= 1/255 ellipse can reach (splat_block_mask).  The chunk
// holding a splat's first instance also lists the splat when it has more than
// kLongSegment instances.  The instance count is clamped to the capacity here
// (block 0 publishes the clamped count and flags an overflow); only instances
// below it are emitted.
//
// The tiles' counts: a workgroup counts its own instances per tile in LDS (16
// bits each) and adds its non-zero counts to tile_count; where the image has
// more than kLdsTiles tiles, or a workgroup more instances than 16 bits hold,
// every instance adds to tile_count itself (3.3M instances at 4096 x 2048, 32768
// tiles, and at 4112 x 2064, 33153: 68 and 104 us).
//
// One workgroup of 16 waves per CU, so the counters are cleared and added up
// 256 times a launch, not once for every few hundred instances (a 4K view's
// 64 KB of counters: 37 us against 160 with 2048 workgroups of four waves);
// four times as many workgroups where a workgroup's instances would outgrow 16
// bits.  Bound by the block masks' arithmetic: 48 us for 2.1M instances.
constexpr int kDupThreads = 1024;
constexpr int kDupWaves = kDupThreads / 64;
constexpr int kDupFew = 256, kDupGrid = 1024;
constexpr int kLdsTiles = 32768;
constexpr int64_t kDupMost = 0xFFFF / (64 * kDupWaves);  // chunks per wave that 16-bit counts hold

// What block_mask needs of a splat, staged per chunk.
struct alignas(16) DupSplat {
  float4 mean;    // x hi, lo, y hi, lo
  float4 shape;   // ce, se, h1, h2
  float4 bound;   // K, hx, hy, depth bits (K < 0: alpha < 1/255 everywhere)
};

__global__ void __launch_bounds__(kDupThreads) k_dup(FrameCounters* ctr, const uint32_t* __restrict__ list,
                                                const uint32_t* __restrict__ inst_off,
                                                const uint32_t* __restrict__ chunk_first, int32_t tiles_x,
                                                int32_t lds_tiles, int64_t cap, const uint32_t* __restrict__ depth_key,
                                                uint2* inst_key, uint2* inst_info, uint32_t* long_list,
                                                const Splat* __restrict__ splats, uint32_t* tile_count) {
  __shared__ DupSplat rec[kDupWaves][64];
  __shared__ uint4 own[kDupWaves][64];  // (splat, instance offset, rectangle width, x0 | y0 << 16)
  extern __shared__ uint32_t hist[];    // two 16-bit counts per word (lds_tiles > 0)
  const uint32_t total = (uint32_t)ctr->n_instances;  // the scan's 32-bit sum
  const int64_t n = (int64_t)total > cap ? cap : (int64_t)total;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctr->n_inst_clamped = (int32_t)n;
    if ((int64_t)total > cap) ctr->status = LODGS_E_CAPACITY;
  }
  const int64_t nd = ctr->n_drawn;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t nchunks = (n + 63) / 64, few = (int64_t)kDupFew * kDupWaves;
  const int64_t nw = nchunks <= few * kDupMost ? few : (int64_t)gridDim.x * kDupWaves;  // waves, at most
  const int64_t per = (nchunks + nw - 1) / nw;
  // few chunks: as many waves of each workgroup as spread them over 256 (the
  // waves of a workgroup take neighbouring runs, whose tiles overlap)
  const int64_t spread = (nchunks + kDupFew - 1) / kDupFew;
  const int waves = spread < kDupWaves ? (int)spread : kDupWaves;
  if ((int64_t)blockIdx.x * waves * per >= nchunks) return;  // block-uniform
  const bool in_lds = lds_tiles > 0 && per <= kDupMost;
  if (in_lds) {
    for (int w = threadIdx.x; w < (lds_tiles + 1) / 2; w += kDupThreads) hist[w] = 0u;
    __syncthreads();
  }
  const int64_t c0 = wv < waves ? ((int64_t)blockIdx.x * waves + wv) * per : nchunks;
  const int64_t c1 = c0 + per < nchunks ? c0 + per : nchunks;
  int64_t rf = c0 < c1 ? chunk_first[c0] : 0;  // the splat that holds the chunk's first instance
  for (int64_t c = c0; c < c1; ++c) {  // wave-uniform
    const int64_t k0 = 64 * c, k1 = k0 + 64 < n ? k0 + 64 : n;
    // the splats rf .. rf + cnt - 1 start before k1
    const int64_t r = rf + lane;
    const uint32_t off = r < nd ? inst_off[r] : 0xFFFFFFFFu;
    const bool in = r < nd && (int64_t)off < k1;  // a prefix of the lanes (lane 0 always)
    const int cnt = __popcll(__ballot(in));
    bool is_long = false;
    if (in) {
      const uint32_t i = list[r];
      const Splat sp = splats[i];  // the record holds the rectangle
      const uint32_t x0 = sp.rect_x & 0xFFFFu, y0 = sp.rect_y & 0xFFFFu;
      const uint32_t w = (sp.rect_x >> 16) - x0, h = (sp.rect_y >> 16) - y0;
      const MaskSetup ms = block_mask_setup(sp);
      DupSplat& ds = rec[wv][lane];
      ds.mean = make_float4(sp.mxh, sp.mxl, sp.myh, sp.myl);
      ds.shape = make_float4(sp.ce, sp.se, sp.h1, sp.h2);
      ds.bound = make_float4(ms.ok ? ms.K : -1.0f, ms.hx, ms.hy, __uint_as_float(depth_key[i]));
      own[wv][lane] = make_uint4(i, off, w, x0 | (y0 << 16));
      is_long = (int64_t)off >= k0 && w * h > kLongSegment;  // and its first instance is in this chunk
    }
    const uint64_t longs = __ballot(is_long);
    if (longs != 0ull) {  // wave-uniform: one atomic per chunk
      uint32_t at = 0;
      if (lane == 0) at = (uint32_t)atomicAdd(&ctr->n_long, __popcll(longs));
      at = __shfl(at, 0, 64);
      if (is_long) long_list[at + (uint32_t)__popcll(longs & lanemask_lt())] = (uint32_t)r;
    }
    __builtin_amdgcn_wave_barrier();
    const int64_t k = k0 + lane;
    if (k < k1) {
      int o = 0;  // the last of the chunk's splats starting at or before k
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
        if (o + step < cnt && (int64_t)own[wv][o + step].y <= k) o += step;
      const uint4 ow = own[wv][o];
      const uint32_t l = (uint32_t)(k - ow.y);
      const uint32_t ty = (ow.w >> 16) + l / ow.z, tx = (ow.w & 0xFFFFu) + l % ow.z;
      const uint32_t tile = ty * (uint32_t)tiles_x + tx;
      const float4 a = rec[wv][o].mean, b = rec[wv][o].shape, q = rec[wv][o].bound;
      Splat sp;
      sp.mxh = a.x; sp.mxl = a.y; sp.myh = a.z; sp.myl = a.w;
      sp.ce = b.x; sp.se = b.y; sp.h1 = b.z; sp.h2 = b.w;
      MaskSetup ms;
      ms.K = q.x; ms.hx = q.y; ms.hy = q.z;
      ms.mx = a.x + a.y; ms.my = a.z + a.w;
      ms.ok = q.x >= 0.0f;
      inst_key[k] = make_uint2(tile, __float_as_uint(q.w));
      inst_info[k] = make_uint2(ow.x, splat_block_mask(sp, ms, (int)tx, (int)ty));
      if (in_lds) atomicAdd(&hist[tile >> 1], (tile & 1u) ? 0x10000u : 1u);
      else atomicAdd(&tile_count[tile], 1u);
    }
    __builtin_amdgcn_wave_barrier();  // rec and own are rewritten by the next chunk
    // the next chunk's first splat: the last one starting at or before k1
    const int64_t rn = rf + cnt;
    const uint32_t offn = rn < nd ? inst_off[rn] : 0xFFFFFFFFu;
    rf = (int64_t)offn == k1 ? rn : rn - 1;
  }
  if (in_lds) {
    __syncthreads();
    for (int w = threadIdx.x; w < (lds_tiles + 1) / 2; w += kDupThreads) {
      const uint32_t x = hist[w];
      if (x & 0xFFFFu) atomicAdd(&tile_count[2 * w], x & 0xFFFFu);
      if (x >> 16) atomicAdd(&tile_count[2 * w + 1], x >> 16);
    }
  }
}

// From the tiles' instance counts: the exclusive scan gives every tile its
// range of the instance list (and the cursor k_bucket fills it from), the
// chunks of tiles with more than kSortSmall instances are listed, and the
// tiles are put in the blend kernels' workgroup order, by descending class of
// the count n (its bit length and the two bits below its leading one, so
// classes are a quarter octave wide), so the longest workgroups start early;
// results do not depend on the order of the tiles.
// Each of the C workgroups takes one chunk of at most kOrderChunk tiles (one
// workgroup for 8160 tiles was bound by its own instructions: 10.6 us) and
// reads the counts of all others too: their sum before it, and how many tiles
// of each class lie before and after it (kept by lane, so that no two lanes of
// an LDS operation meet).  An order of each chunk by itself, interleaved,
// was shorter to make (6 against 8 us), but where one part of the image is
// heavier its tiles started late: 132 against 102 us for the blend backward of
// a 1080p iteration, 151 against 138 of an aerial 1080p view (before its later
// changes).  What all workgroups read grows with the square of the image's
// tiles: 7 us at 1080p, 16 at 4K, 82 at 8192 x 8192 and 350 at 16384 x 16384,
// the largest image (531 and 2157 with the ranges and the order in two kernels).
// Within its chunk a tile takes its rank in its class
// from an LDS counter; the order within a chunk and class is whatever the LDS
// atomics give.  The lanes of a wave whose tiles share the first lane's class
// (empty tiles, mostly) count with one atomic: same-address LDS atomics run
// one after another.
constexpr int kOrderThreads = 1024;
constexpr int kOrderBatch = 2;  // consecutive tiles per thread
static_assert(kOrderChunk == kOrderThreads * kOrderBatch, "two tiles per thread");
// A tile of up to this many instances has its segments and sort chunks listed by
// its own thread (one thread for a tile of 1M: 152 us, its wave: 9).
constexpr uint32_t kOwnTile = 32768;

constexpr int kTileClasses = 128;
__device__ __forceinline__ int tile_class(uint32_t n) {
  const int bl = min(31, 32 - __clz((int)n));  // 0 for an empty tile
  const int sub = bl >= 3 ? (int)((n >> (bl - 3)) & 3u) : 0;
  return bl * 4 + sub;  // < kTileClasses
}
constexpr int kHeavyClass = 4 * kHeavyBits;  // class of kHeavyTile instances
// The class from which on tiles are blended by a wave per 4x4 block, in an image
// of n instances and `many` tiles of at least kHeavyTile (k_blend_fwd says why).
constexpr uint32_t kHeavyShare = 2048, kHeavyFew = 512;
__device__ __forceinline__ int heavy_class(uint32_t n, uint32_t many) {
  return many <= kHeavyFew ? kHeavyClass : max(kHeavyClass, tile_class(n / kHeavyShare));
}
constexpr int kWaveClass = 4 * 7;  // class of 64 to 79 instances: a tile below it holds fewer than 64
constexpr int kClassLanes = 32;  // copies of a class's counter

// The sum of x over the wave's lanes, in every lane.
__device__ __forceinline__ uint32_t wave_add(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, false);  // row_half_mirror
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xf, 0xf, false);  // row_mirror
  const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = a[0] + a[1];
  const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return b[0] + b[1];
}

// Instances that a workgroup of k_tile_sort sorts; a tile with more is sorted
// in chunks of that many, which k_tile_merge puts together.
constexpr int kSortSmall = 2048;
static_assert(kSortSmall == 2 * kSortChunkHalf, "the chunk list's length");

__global__ void __launch_bounds__(kOrderThreads) k_tile_scan(const uint32_t* __restrict__ count, int32_t ntiles,
                                                             FrameCounters* ctr, uint2* ranges, uint32_t* cursor,
                                                             uint4* order, uint4* seg_list, uint2* big_list) {
  __shared__ uint32_t cnt[kTileClasses], pre[kTileClasses], post[kTileClasses];
  __shared__ uint32_t others[kTileClasses][kClassLanes];  // the other chunks' tiles: low half before, high half after
  __shared__ uint32_t half[2];
  __shared__ uint32_t wt[kOrderThreads / 64], wb[kOrderThreads / 64];
  __shared__ uint32_t big, big_base;  // this chunk's large tiles' sort chunks
  __shared__ uint32_t seg, seg_base;  // and blend segments
  __shared__ uint32_t many;  // the image's tiles of at least kHeavyTile instances
  const int32_t per = tile_chunk(ntiles), lo = blockIdx.x * per;
  const int32_t n = min(per, ntiles - lo);
  const uint32_t n_inst = (uint32_t)ctr->n_inst_clamped;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int32_t k0 = t * kOrderBatch;
  uint32_t m[kOrderBatch], sum = 0, before = 0;
#pragma unroll
  for (int k = 0; k < kOrderBatch; ++k) m[k] = k0 + k < n ? count[lo + k0 + k] : 0u;
  if (t < kTileClasses) cnt[t] = pre[t] = post[t] = 0;
  if (t == 0) big = seg = 0;
  if (gridDim.x > 1) {  // block-uniform
    static_assert(kTileClasses * kClassLanes == 4 * kOrderThreads, "one 16-byte store per thread");
    reinterpret_cast<uint4*>(&others[0][0])[t] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    // (a counter's half stays below 2^16: an image has at most 2^20 tiles, and
    // a counter takes a 32nd of them)
#pragma unroll 8
    for (int32_t i = t; i < ntiles - n; i += kOrderThreads) {
      const bool first = i < lo;
      const uint32_t x = count[first ? i : i + n];
      before += first ? x : 0u;
      atomicAdd(&others[tile_class(x)][lane & (kClassLanes - 1)], first ? 1u : 0x10000u);
    }
    before = wave_add(before);
    __syncthreads();
    const uint4 q = reinterpret_cast<const uint4*>(&others[0][0])[t];  // a class: eight threads
    uint32_t p = (q.x & 0xFFFFu) + (q.y & 0xFFFFu) + (q.z & 0xFFFFu) + (q.w & 0xFFFFu);
    uint32_t r = (q.x >> 16) + (q.y >> 16) + (q.z >> 16) + (q.w >> 16);
#pragma unroll
    for (int d = 1; d < 8; d <<= 1) {
      p += __shfl_xor(p, d, 64);
      r += __shfl_xor(r, d, 64);
    }
    if ((t & 7) == 0) {
      pre[t >> 3] = p;
      post[t >> 3] = r;
    }
  }
#pragma unroll
  for (int k = 0; k < kOrderBatch; ++k) sum += m[k];
  uint32_t x = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) {
    wt[wv] = x;
    wb[wv] = before;
  }
  __syncthreads();
  uint32_t start = x - sum;
#pragma unroll
  for (int w = 0; w < kOrderThreads / 64; ++w) start += wb[w] + (w < wv ? wt[w] : 0u);
  uint32_t key[kOrderBatch];  // class << 16 | rank within the chunk's class (rank < kOrderChunk)
  uint32_t big_at[kOrderBatch] = {}, seg_at[kOrderBatch] = {}, first[kOrderBatch] = {};
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int k = 0; k < kOrderBatch; ++k) {
    key[k] = 0;
    const bool in = k0 + k < n;
    const int c = tile_class(m[k]);
    const int c0 = __builtin_amdgcn_readfirstlane(c);
    const uint64_t same = __ballot(in && c == c0);
    uint32_t base = 0;
    if (lane == 0 && same) base = atomicAdd(&cnt[c0], (uint32_t)__popcll(same));
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    if (in) {
      const int32_t tile = lo + k0 + k;
      ranges[tile] = make_uint2(start, start + m[k]);
      cursor[tile] = start;
      first[k] = start;
      start += m[k];
      key[k] = ((uint32_t)c << 16) | (c == c0 ? base + (uint32_t)__popcll(same & lt) : atomicAdd(&cnt[c], 1u));
      if (m[k] > (uint32_t)kSegment) seg_at[k] = atomicAdd(&seg, (m[k] + kSegment - 1) / kSegment);
      if (m[k] > (uint32_t)kSortSmall) big_at[k] = atomicAdd(&big, (m[k] + kSortSmall - 1) / kSortSmall);
    }
  }
  __syncthreads();
  if (t == kOrderThreads - 2 && seg != 0u) seg_base = (uint32_t)atomicAdd(&ctr->n_seg, (int)seg);
  if (t == kOrderThreads - 1 && big != 0u) big_base = (uint32_t)atomicAdd(&ctr->n_big, (int)big);
  // pre[c] becomes the place of the chunk's first tile of class c: all tiles of
  // the classes above c and the ones of class c before the chunk (waves 0 and
  // 1, whole waves)
  const int c = t;
  uint32_t incl = 0;
  if (c < kTileClasses) {
    incl = cnt[c] + pre[c] + post[c];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(incl, d, 64);
      if (lane >= d) incl += y;
    }
    if (lane == 63) half[wv] = incl;
  }
  __syncthreads();
  uint32_t above = 0;
  if (c < kTileClasses) {
    above = half[0] + half[1] - (incl + (wv == 1 ? half[0] : 0u));
    pre[c] += above;
    if (c == kHeavyClass - 1) many = above;
    if (blockIdx.x == 0 && c == kWaveClass - 1) ctr->n_mid = (int32_t)above;
  }
  __syncthreads();
  const int heavy = heavy_class(n_inst, many);
  if (blockIdx.x == 0 && c == heavy - 1) ctr->n_heavy = (int32_t)above;
#pragma unroll
  for (int k = 0; k < kOrderBatch; ++k) {
    const uint32_t tile = (uint32_t)(lo + k0 + k);
    const bool in = k0 + k < n;
    if (in) {
      order[pre[key[k] >> 16] + (key[k] & 0xFFFFu)] =
          make_uint4(tile, first[k], first[k] + m[k], (int)(key[k] >> 16) >= heavy ? 1u : 0u);
      if (m[k] > (uint32_t)kSegment && m[k] <= kOwnTile)
        for (uint32_t q = 0; q * kSegment < m[k]; ++q)
          seg_list[seg_base + seg_at[k] + q] =
              make_uint4(tile, first[k], first[k] + q * kSegment, first[k] + min(m[k], (q + 1) * kSegment));
      if (m[k] > (uint32_t)kSortSmall && m[k] <= kOwnTile)
        for (uint32_t q = 0; q * kSortSmall < m[k]; ++q)
          big_list[big_base + big_at[k] + q] = make_uint2(tile, q);
    }
    // a longer tile's lists are its wave's to write
    for (uint64_t more = __ballot(in && m[k] > kOwnTile); more; more &= more - 1) {  // wave-uniform
      const int l = __builtin_ctzll(more);
      const uint32_t tl = __shfl(tile, l, 64), f = __shfl(first[k], l, 64), len = __shfl(m[k], l, 64);
      const uint32_t seg_to = seg_base + __shfl(seg_at[k], l, 64), big_to = big_base + __shfl(big_at[k], l, 64);
      for (uint32_t q = lane; q * kSegment < len; q += 64)
        seg_list[seg_to + q] = make_uint4(tl, f, f + q * kSegment, f + min(len, (q + 1) * kSegment));
      for (uint32_t q = lane; q * kSortSmall < len; q += 64) big_list[big_to + q] = make_uint2(tl, q);
    }
  }
}

// The instances' sort keys (depth bits, emission index) into their tile's
// range, in any order (the keys are distinct, so the sort fixes it).  A
// workgroup counts its instances per tile in LDS, the first
// instance of each tile takes the tile's places with one atomic and hands
// them to the others; only the counters of tiles it meets are touched.  Bound
// by those atomics (27 G/s over the chip): 22 us for 2.1M instances.
// Images of more than kBucketLdsTiles tiles take a place per instance (3.3M
// instances at 32768 and at 33153 tiles: 33 and 96 us).
constexpr int kBucketThreads = 1024;
constexpr int kBucketItems = 8;   // at most, per thread
constexpr int kBucketGrid = 512;  // a CU takes two where the counters leave room
constexpr int kBucketLdsTiles = 32768;  // 128 KB of counters

__global__ void __launch_bounds__(kBucketThreads) k_bucket(const FrameCounters* ctr, const uint2* __restrict__ inst_key,
                                                           int32_t lds_tiles, uint32_t* cursor,
                                                           unsigned long long* __restrict__ bkey) {
  extern __shared__ uint32_t place[];
  const int64_t n = ctr->n_inst_clamped;
  // items per thread: enough to keep to one round of the grid, at most kBucketItems
  const int64_t want = (n + (int64_t)gridDim.x * kBucketThreads - 1) / ((int64_t)gridDim.x * kBucketThreads);
  const int items = (int)(want < 1 ? 1 : (want > kBucketItems ? kBucketItems : want));
  const int64_t tile_n = (int64_t)items * kBucketThreads;
  for (int64_t b0 = (int64_t)blockIdx.x * tile_n; b0 < n; b0 += (int64_t)gridDim.x * tile_n) {  // block-uniform
    uint2 w[kBucketItems];
    bool in[kBucketItems];
    uint32_t pos[kBucketItems];
#pragma unroll
    for (int u = 0; u < kBucketItems; ++u) {
      const int64_t k = b0 + u * kBucketThreads + threadIdx.x;
      in[u] = u < items && k < n;
      w[u] = in[u] ? inst_key[k] : make_uint2(0u, 0u);
      pos[u] = 0u;
    }
    if (lds_tiles > 0) {
#pragma unroll
      for (int u = 0; u < kBucketItems; ++u)
        if (in[u]) place[w[u].x] = 0u;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kBucketItems; ++u)
        if (in[u]) pos[u] = atomicAdd(&place[w[u].x], 1u);
      __syncthreads();
      // the first of a tile takes its places: alone to read the tile's count
      uint32_t base[kBucketItems];
#pragma unroll
      for (int u = 0; u < kBucketItems; ++u)
        if (in[u] && pos[u] == 0u) base[u] = atomicAdd(&cursor[w[u].x], place[w[u].x]);
#pragma unroll
      for (int u = 0; u < kBucketItems; ++u)
        if (in[u] && pos[u] == 0u) place[w[u].x] = base[u];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kBucketItems; ++u)
        if (in[u]) pos[u] += place[w[u].x];
      __syncthreads();
    } else {
#pragma unroll
      for (int u = 0; u < kBucketItems; ++u)
        if (in[u]) pos[u] = atomicAdd(&cursor[w[u].x], 1u);
    }
#pragma unroll
    for (int u = 0; u < kBucketItems; ++u) {
      const uint32_t k = (uint32_t)(b0 + u * kBucketThreads + threadIdx.x);
      if (in[u]) bkey[pos[u]] = ((unsigned long long)w[u].y << 32) | k;
    }
  }
}

// Ascending order of one key per lane over the wave: a bitonic network whose
// rounds start by comparing mirrored lanes (l ^ (2^k - 1)), so that every step
// keeps the smaller key in the lower lane.  Partners inside a 16-lane row come
// by DPP moves.
#define LODGS_DPP64(v, ctrl)                                                                             \
  (((unsigned long long)(uint32_t)__builtin_amdgcn_update_dpp(0, (int)((v) >> 32), ctrl, 0xf, 0xf, false) \
    << 32) |                                                                                              \
   (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(v), ctrl, 0xf, 0xf, false))

__device__ __forceinline__ unsigned long long keep(unsigned long long v, unsigned long long o, bool low) {
  return (v < o) == low ? v : o;
}

__device__ __forceinline__ unsigned long long wave_sort(unsigned long long v) {
  const int lane = threadIdx.x & 63;
  const bool b0 = (lane & 1) == 0, b1 = (lane & 2) == 0, b2 = (lane & 4) == 0, b3 = (lane & 8) == 0;
  const bool b4 = (lane & 16) == 0, b5 = (lane & 32) == 0;
  const auto x1 = [](unsigned long long a) { return LODGS_DPP64(a, 0xB1); };    // l ^ 1: quad_perm [1,0,3,2]
  const auto x2 = [](unsigned long long a) { return LODGS_DPP64(a, 0x4E); };    // l ^ 2: quad_perm [2,3,0,1]
  const auto x3 = [](unsigned long long a) { return LODGS_DPP64(a, 0x1B); };    // l ^ 3: quad_perm [3,2,1,0]
  const auto x7 = [](unsigned long long a) { return LODGS_DPP64(a, 0x141); };   // l ^ 7: row_half_mirror
  const auto x8 = [](unsigned long long a) { return LODGS_DPP64(a, 0x128); };   // l ^ 8: row_ror 8
  const auto x15 = [](unsigned long long a) { return LODGS_DPP64(a, 0x140); };  // l ^ 15: row_mirror
  const auto x4 = [&](unsigned long long a) { return x3(x7(a)); };              // l ^ 4
  v = keep(v, x1(v), b0);
  v = keep(v, x3(v), b1);
  v = keep(v, x1(v), b0);
  v = keep(v, x7(v), b2);
  v = keep(v, x2(v), b1);
  v = keep(v, x1(v), b0);
  v = keep(v, x15(v), b3);
  v = keep(v, x4(v), b2);
  v = keep(v, x2(v), b1);
  v = keep(v, x1(v), b0);
  v = keep(v, __shfl_xor(v, 31, 64), b4);
  v = keep(v, x8(v), b3);
  v = keep(v, x4(v), b2);
  v = keep(v, x2(v), b1);
  v = keep(v, x1(v), b0);
  v = keep(v, __shfl_xor(v, 63, 64), b5);
  v = keep(v, __shfl_xor(v, 16, 64), b4);
  v = keep(v, x8(v), b3);
  v = keep(v, x4(v), b2);
  v = keep(v, x2(v), b1);
  v = keep(v, x1(v), b0);
  return v;
}
#undef LODGS_DPP64

// Sorts in[0, m) (STAGED: keys[0, m) itself) into keys (LDS; 0 < m <= THREADS
// * ITEMS, itself a power of two; distinct keys below ~0) with the whole
// workgroup: runs of 64 in registers, then rounds that merge neighbouring runs,
// every key finding its place by a binary search of the other run (the searches
// of a thread's keys run side by side).  Places past m hold ~0, so that every
// run is whole.
template <int THREADS, int ITEMS, bool STAGED>
__device__ __forceinline__ void block_sort(const unsigned long long* in, unsigned long long* keys, int m) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int whole = 64;
  while (whole < m) whole *= 2;
  for (int r = wv; r * 64 < whole; r += THREADS / 64) {  // wave-uniform
    const int j = r * 64 + lane;
    keys[j] = r * 64 < m ? wave_sort(j < m ? (STAGED ? keys[j] : in[j]) : ~0ull) : ~0ull;
  }
  __syncthreads();
  for (int w = 64; w < m; w *= 2) {  // block-uniform
    unsigned long long v[ITEMS];
    int sib[ITEMS], at[ITEMS];
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
      const int j = e * THREADS + t;
      v[e] = keys[j];
      sib[e] = (j & ~(w - 1)) ^ w;
      at[e] = 0;
      if (j >= whole) sib[e] = 0;  // past the padded keys: searched for nothing
    }
    for (int s = w >> 1; s > 0; s >>= 1) {
#pragma unroll
      for (int e = 0; e < ITEMS; ++e) at[e] += keys[sib[e] + at[e] + s - 1] < v[e] ? s : 0;
    }
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) at[e] += keys[sib[e] + at[e]] < v[e] ? 1 : 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
      const int j = e * THREADS + t;
      if (j < m) keys[(j & ~(2 * w - 1)) + (j & (w - 1)) + at[e]] = v[e];
    }
    __syncthreads();
  }
}

// block_sort with as many keys per thread as m needs.
template <int THREADS, bool STAGED = false>
__device__ __forceinline__ void block_sort_small(const unsigned long long* in, unsigned long long* keys, int m) {
  static_assert(kSortSmall == 8 * THREADS, "eight keys per thread at most");
  if (m <= THREADS) block_sort<THREADS, 1, STAGED>(in, keys, m);
  else if (m <= 2 * THREADS) block_sort<THREADS, 2, STAGED>(in, keys, m);
  else if (m <= 4 * THREADS) block_sort<THREADS, 4, STAGED>(in, keys, m);
  else block_sort<THREADS, 8, STAGED>(in, keys, m);
}

// Sorts the tiles' keys: the listed chunks of large tiles (in place, for
// k_tile_merge), then the tiles by descending class, those of at least 64
// instances one workgroup each, the others four to a workgroup, each by one
// wave in registers.  A tile's instance words and emission indices are written
// in its sorted order.  A fixed grid takes the work in that order (largest
// first), so no workgroup is launched for nothing.  Bound by the 64-bit
// comparisons: 5.8 us for 40K instances in 1024 tiles, 41 us (and 27 us for
// k_tile_merge) for 2.1M in 8160 tiles, 1.3M of them in tiles above 2048.
constexpr int kSmallThreads = 256;
constexpr int kSmallItems = kSortSmall / kSmallThreads;
constexpr int kTileSortGrid = 1792;  // seven workgroups per CU: what the registers allow

__global__ void __launch_bounds__(kSmallThreads) k_tile_sort(const FrameCounters* ctr, const uint2* __restrict__ ranges,
                                                             const uint4* __restrict__ tile_order,
                                                             int32_t ntiles, const uint2* __restrict__ big_list,
                                                             unsigned long long* bkey,
                                                             const uint2* __restrict__ inst_info,
                                                             uint2* __restrict__ info_k, uint32_t* __restrict__ ival) {
  __shared__ unsigned long long keys[kSortSmall];
  const int t = threadIdx.x, lane = t & 63;
  const int nb = ctr->n_big;
  for (int li = blockIdx.x; li < nb; li += gridDim.x) {  // block-uniform
    const uint2 e = big_list[li];
    const uint2 rg = ranges[e.x];
    const uint32_t x = rg.x + e.y * kSortSmall;
    const int m = (int)min(rg.y - x, (uint32_t)kSortSmall);
    block_sort_small<kSmallThreads>(bkey + x, keys, m);
    for (int j = t; j < m; j += kSmallThreads) bkey[x + j] = keys[j];
    __syncthreads();
  }
  // the tile order: a workgroup for each tile of at least 64 instances, then
  // a wave for each other one; the first items go to the workgroups after
  // those that took the last chunks
  const int32_t nm = ctr->n_mid, items = nm + (ntiles - nm + 3) / 4;
  int32_t it = (int32_t)blockIdx.x - nb % (int32_t)gridDim.x;
  if (it < 0) it += (int32_t)gridDim.x;
  for (; it < items; it += (int32_t)gridDim.x) {  // block-uniform
    if (it >= nm) {  // four tiles of fewer than 64 instances
      const int32_t at = nm + 4 * (it - nm) + (t >> 6);
      if (at < ntiles) {  // wave-uniform
        const uint4 o = tile_order[at];
        const uint2 rg = make_uint2(o.y, o.z);
        const int m = (int)(rg.y - rg.x);
        if (m > 0) {
          const uint32_t k = (uint32_t)wave_sort(lane < m ? bkey[rg.x + lane] : ~0ull);
          if (lane < m) {
            ival[rg.x + lane] = k;
            info_k[rg.x + lane] = inst_info[k];
          }
        }
      }
      continue;
    }
    const uint4 o = tile_order[it];
    const uint2 rg = make_uint2(o.y, o.z);
    if (rg.y - rg.x > (uint32_t)kSortSmall) continue;  // listed in chunks
    const int m = (int)(rg.y - rg.x);
    block_sort_small<kSmallThreads>(bkey + rg.x, keys, m);
    for (int j = t; j < m; j += kSmallThreads) {
      const uint32_t k = (uint32_t)keys[j];
      ival[rg.x + j] = k;
      info_k[rg.x + j] = inst_info[k];
    }
    __syncthreads();
  }
}

// How many of keys[lo, hi) (ascending) are below v, and lo.
__device__ __forceinline__ int keys_below(const unsigned long long* __restrict__ keys, int lo, int hi,
                                          unsigned long long v) {
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (keys[mid] < v) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// LDS of a tile's split; thread t keeps what it knows of chunks t, t + 256, ...
// (where v's place lies, [lo, hi] as lo | hi << 16, and the last place tried).
struct SplitLds {
  uint32_t window[kSortSmall];
  uint16_t at[kSortSmall];
};

// A value with exactly `rank` of a tile's n keys below it, the whole workgroup
// halving [lo, hi): fewer are below lo, more below hi (the keys are distinct).
// The keys are sorted chunks of kSortSmall.  The windows hold from one split to
// a later one of the same tile; a tile of more chunks than they have room for
// is searched whole each time.
__device__ __forceinline__ unsigned long long split_keys(const unsigned long long* __restrict__ keys, uint32_t n,
                                                         uint32_t rank, unsigned long long lo, unsigned long long hi,
                                                         SplitLds& lds, uint32_t (*part)[kSmallThreads / 64]) {
  const uint32_t t = threadIdx.x, nc = (n + kSortSmall - 1) / kSortSmall;
  const bool kept = nc <= (uint32_t)kSortSmall;
  __syncthreads();  // `part` may still be read
  for (int turn = 0; turn < 64; ++turn) {  // block-uniform; 64 halvings end any range
    const unsigned long long v = lo + (hi - lo) / 2;
    uint32_t below = 0;
    for (uint32_t c = t; c < nc; c += kSmallThreads) {
      const uint32_t w = kept ? lds.window[c] : (uint32_t)min(n - c * kSortSmall, (uint32_t)kSortSmall) << 16;
      const int k = keys_below(keys + c * kSortSmall, (int)(w & 0xFFFFu), (int)(w >> 16), v);
      if (kept) lds.at[c] = (uint16_t)k;
      below += (uint32_t)k;
    }
    below = wave_add(below);
    if ((t & 63u) == 0u) part[turn & 1][t >> 6] = below;
    __syncthreads();
    below = 0;
#pragma unroll
    for (int w = 0; w < kSmallThreads / 64; ++w) below += part[turn & 1][w];
    if (kept) {
      for (uint32_t c = t; c < nc; c += kSmallThreads) {
        const uint32_t w = lds.window[c], k = lds.at[c];
        // (found: what lies above stays open for a split at a higher rank)
        lds.window[c] = below == rank ? k | min(n - c * kSortSmall, (uint32_t)kSortSmall) << 16
                                      : (below < rank ? (w & 0xFFFF0000u) | k : (w & 0xFFFFu) | k << 16);
      }
    }
    if (below == rank) return v;
    if (below < rank) lo = v;
    else hi = v;
  }
  return hi;
}

// A workgroup's share of a tile of many sorted chunks: the keys of ranks [kSortSmall
// w, kSortSmall (w + 1)), found by splitting the tile at both ends, gathered
// from all chunks and sorted.
__device__ __forceinline__ void merge_share(const unsigned long long* __restrict__ keys_in, uint32_t n, uint32_t w,
                                            unsigned long long* keys, uint32_t (*part)[kSmallThreads / 64]) {
  const uint32_t t = threadIdx.x, lane = t & 63u, nc = (n + kSortSmall - 1) / kSortSmall;
  static_assert(sizeof(SplitLds) <= sizeof(unsigned long long) * kSortSmall, "the windows lie where the keys will");
  SplitLds& lds = *reinterpret_cast<SplitLds*>(keys);
  unsigned long long least = ~0ull, most = 0ull;
  for (uint32_t c = t; c < nc; c += kSmallThreads) {
    const uint32_t len = min(n - c * kSortSmall, (uint32_t)kSortSmall);
    if (c < (uint32_t)kSortSmall) lds.window[c] = len << 16;
    least = min(least, keys_in[c * kSortSmall]);
    most = max(most, keys_in[c * kSortSmall + len - 1]);
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    least = min(least, __shfl_xor(least, d, 64));
    most = max(most, __shfl_xor(most, d, 64));
  }
  __shared__ unsigned long long ends[2][kSmallThreads / 64];
  if (lane == 0) {
    ends[0][t >> 6] = least;
    ends[1][t >> 6] = most;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSmallThreads / 64; ++k) {
    least = min(least, ends[0][k]);
    most = max(most, ends[1][k]);
  }
  unsigned long long from = 0ull, to = ~0ull;
  if (w > 0) from = split_keys(keys_in, n, kSortSmall * w, least, most + 1, lds, part);
  if (w + 1 < nc) to = split_keys(keys_in, n, kSortSmall * (w + 1), w > 0 ? from : least, most + 1, lds, part);
  __syncthreads();
  uint32_t base = 0;
  for (uint32_t c0 = 0; c0 < nc; c0 += kSmallThreads) {  // block-uniform
    const uint32_t c = c0 + t;
    uint32_t a = 0, len = 0;
    if (c < nc) {
      const unsigned long long* in = keys_in + c * kSortSmall;
      const int all = (int)min(n - c * kSortSmall, (uint32_t)kSortSmall);
      a = (uint32_t)keys_below(in, 0, all, from);
      len = (uint32_t)keys_below(in, (int)a, all, to) - a;
      a += c * kSortSmall;
    }
    uint32_t tot;
    const uint32_t at = base + block_exclusive_scan(len, part[0], &tot);
    base += tot;
    len = min(len, kSortSmall - min(at, (uint32_t)kSortSmall));  // (the shares hold no more)
    if (len <= 8u) {
      for (uint32_t q = 0; q < len; ++q) keys[at + q] = keys_in[a + q];
    }
    for (uint64_t more = __ballot(len > 8u); more; more &= more - 1) {  // wave-uniform
      const int l = __builtin_ctzll(more);
      const uint32_t from_l = __shfl(a, l, 64), at_l = __shfl(at, l, 64), len_l = __shfl(len, l, 64);
      for (uint32_t q = lane; q < len_l; q += 64) keys[at_l + q] = keys_in[from_l + q];
    }
  }
  __syncthreads();
  block_sort_small<kSmallThreads, true>(nullptr, keys, (int)min(base, (uint32_t)kSortSmall));
}

// Puts the sorted chunks of a large tile together, one workgroup per chunk.  In
// a tile of up to kMergeChunks chunks a key's place is its index in its chunk
// and, for every other chunk, the number of smaller keys there, found by a
// binary search of the chunk staged in LDS: all chunks of all large tiles work
// at once, but the work grows with the square of the chunks.  In a tile of more
// a workgroup takes a share of the places instead (merge_share), which reads
// every chunk at some tens of places only.  Sort and merge of one tile of 8, 16,
// 24, 64, 256 and 1024 chunks, us: all by counting 51 / 77 / 102 / 222 / 835 /
// 3866, all by shares 90 / 102 / 103 / 126 / 137 / 970.
constexpr uint32_t kMergeChunks = 24;
__global__ void __launch_bounds__(kSmallThreads) k_tile_merge(const FrameCounters* ctr, const uint2* __restrict__ ranges,
                                                              const uint2* __restrict__ big_list,
                                                              const unsigned long long* __restrict__ bkey,
                                                              const uint2* __restrict__ inst_info,
                                                              uint2* __restrict__ info_k, uint32_t* __restrict__ ival) {
  __shared__ unsigned long long keys[kSortSmall];
  __shared__ uint32_t part[2][kSmallThreads / 64];
  const int t = threadIdx.x;
  const int nb = ctr->n_big;
  for (int li = blockIdx.x; li < nb; li += gridDim.x) {  // block-uniform
    const uint2 e = big_list[li];
    const uint2 rg = ranges[e.x];
    const uint32_t x = rg.x + e.y * kSortSmall, nc = (rg.y - rg.x + kSortSmall - 1) / kSortSmall;
    const int m = (int)min(rg.y - x, (uint32_t)kSortSmall);
    if (nc > kMergeChunks) {  // block-uniform
      merge_share(bkey + rg.x, rg.y - rg.x, e.y, keys, part);
      for (int j = t; j < m; j += kSmallThreads) {
        const uint32_t k = (uint32_t)keys[j];
        ival[x + j] = k;
        info_k[x + j] = inst_info[k];
      }
      __syncthreads();
      continue;
    }
    unsigned long long v[kSmallItems];
    uint32_t at[kSmallItems];
#pragma unroll
    for (int q = 0; q < kSmallItems; ++q) {
      const int j = q * kSmallThreads + t;
      v[q] = j < m ? bkey[x + j] : 0ull;
      at[q] = (uint32_t)j;
    }
    for (uint32_t c = 0; c < nc; ++c) {  // block-uniform
      if (c == e.y) continue;
      const uint32_t y = rg.x + c * kSortSmall;
      const int len = (int)min(rg.y - y, (uint32_t)kSortSmall);
#pragma unroll
      for (int q = 0; q < kSmallItems; ++q) {
        const int j = q * kSmallThreads + t;
        keys[j] = j < len ? bkey[y + j] : ~0ull;
      }
      __syncthreads();
      int less[kSmallItems];
#pragma unroll
      for (int q = 0; q < kSmallItems; ++q) less[q] = 0;
#pragma unroll
      for (int s = kSortSmall / 2; s > 0; s >>= 1) {
#pragma unroll
        for (int q = 0; q < kSmallItems; ++q) less[q] += keys[less[q] + s - 1] < v[q] ? s : 0;
      }
#pragma unroll
      for (int q = 0; q < kSmallItems; ++q) at[q] += (uint32_t)(less[q] + (keys[less[q]] < v[q] ? 1 : 0));
      __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < kSmallItems; ++q) {
      if (q * kSmallThreads + t < m) {
        const uint32_t k = (uint32_t)v[q];
        ival[rg.x + at[q]] = k;
        info_k[rg.x + at[q]] = inst_info[k];
      }
    }
  }
}

// One workgroup per tile with 4/PX waves, PX pixels per lane; each 16-lane
// row of a wave covers 4x4 pixel blocks (blend_pixel).  Per batch of
// instances, every row lists the instances whose block mask (k_dup) meets
// its blocks and replays only those, in order: elsewhere alpha < 1/255 at
// every pixel.  The rows of a wave step through their lists together, each on
// its own splat.  The forward records the blocks where some pixel blended an
// instance or stopped on it (event_masks); elsewhere the splat changed
// nothing, which lets the backward skip it there.
// alpha = min(0.99, o e^power), skipped below 1/255; a pixel stops before its
// transmittance would drop below 1e-4.  Splat records are staged in LDS one
// batch per workgroup size and read into registers one list entry ahead; the
// per-pixel steps are written with selects, so the only branches are
// wave-uniform.  The counting variant lists every instance in every row (the
// algorithmic evaluation count: every splat of the tile up to termination).
template <bool COUNT, int PX>
__global__ void __launch_bounds__(256 / PX) k_blend(const ViewConst* __restrict__ vp, const uint2* __restrict__ info_k,
                                                    const Splat* __restrict__ splats, const FrameCounters* ctr,
                                                    const uint4* __restrict__ tile_order, float bg0, float bg1,
                                                    float bg2, float* rgb, uint32_t* event, unsigned long long* work,
                                                    float4* ckpt) {
  constexpr int NT = 256 / PX, NW = 4 / PX;
  const ViewConst v = *vp;
  __shared__ Splat batch[NT];
  __shared__ uint32_t ev[NT];
  __shared__ uint32_t bm[NT];
  __shared__ uint8_t hits[NW][4][NT];  // per row of each wave: the batch slots it replays, in order
  const uint4 place = tile_order[blockIdx.x];
  const int tile = (int)place.x;
  const int tx = tile % v.tiles_x, ty = tile / v.tiles_x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane >> 4;
  int px, pys[PX];
  float fy[PX], T[PX], cr[PX], cg[PX], cb[PX];
  uint32_t pbit[PX];
  bool inside[PX], live[PX];
#pragma unroll
  for (int p = 0; p < PX; ++p) {
    blend_pixel<PX>(tx, ty, wv, lane, p, px, pys[p]);
    pbit[p] = blend_pixel_block<PX>(wv, g, p);
    fy[p] = (float)pys[p] + 0.5f;
    inside[p] = px < v.width && pys[p] < v.height;
    live[p] = inside[p];
    T[p] = 1.0f;
    cr[p] = cg[p] = cb[p] = 0.0f;
  }
  const float fx = (float)px + 0.5f;
  const uint2 rg = make_uint2(place.y, place.z);
  const uint32_t nr = (uint32_t)ctr->n_render;
  const float thr = 1.0f / 255.0f;
  unsigned long long n_eval = 0, n_contrib = 0;
  // the pixels' state before instance k of the list (a segment's first)
  auto checkpoint = [&](uint32_t k) {
    float4* c = ckpt + 256 * (int64_t)(k / kSegment);
#pragma unroll
    for (int p = 0; p < PX; ++p)
      c[16 * (pys[p] & 15) + (px & 15)] = make_float4(live[p] ? T[p] : 0.0f, cr[p], cg[p], cb[p]);
  };
  uint32_t b0 = rg.x;
  for (; b0 < rg.y; b0 += NT) {
    bool active = false;
#pragma unroll
    for (int p = 0; p < PX; ++p) active = active || live[p];
    if (__syncthreads_count(active) == 0) break;
    if (!COUNT && b0 > rg.x && (b0 - rg.x) % kSegment == 0) checkpoint(b0);
    const uint32_t k = b0 + threadIdx.x;
    ev[threadIdx.x] = 0u;
    if (k < rg.y) {
      const uint2 w = info_k[k];
      const uint32_t i = w.x;
      bm[threadIdx.x] = w.y;
      if (i < nr) {
        batch[threadIdx.x] = splats[i];
      } else {  // only reachable if the instance count overflowed (its block mask is 0)
        batch[threadIdx.x].o = 0.0f;
      }
    }
    __syncthreads();
    const int m = (int)min((uint32_t)NT, rg.y - b0);
    int nh[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) nh[r] = wave_hit_list<NT, COUNT>(m, blend_row_blocks<PX>(wv, r), bm, hits[wv][r]);
    __syncthreads();
    const int n = g == 0 ? nh[0] : (g == 1 ? nh[1] : (g == 2 ? nh[2] : nh[3]));  // this row's list
    const int nmax = max(max(nh[0], nh[1]), max(nh[2], nh[3]));
    // one splat (batch slot j of this row's list; has = false past its end)
    // against the row's pixels; true when every pixel of the wave has stopped
    auto step = [&](const Splat& s, int j, bool has) -> bool {
      bool act = false;
      uint32_t eb = 0u;
#pragma unroll
      for (int p = 0; p < PX; ++p) {
        float dx, dy, u1, u2;
        const float power = splat_power(s, fx, fy[p], dx, dy, u1, u2);
        const float alpha = fminf(0.99f, s.o * fexp(power));
        const float tt = T[p] * (1.0f - alpha);
        const bool in = live[p] & has;
        const bool hit = in & (alpha >= thr);
        const bool stop = hit & (tt < 0.0001f);
        const bool con = hit & !stop;
        if (COUNT) {
          n_eval += in ? 1 : 0;
          n_contrib += con ? 1 : 0;
        }
        live[p] = live[p] & !stop;
        const float w = alpha * T[p];
        cr[p] = con ? __builtin_fmaf(s.r, w, cr[p]) : cr[p];
        cg[p] = con ? __builtin_fmaf(s.g, w, cg[p]) : cg[p];
        cb[p] = con ? __builtin_fmaf(s.b, w, cb[p]) : cb[p];
        T[p] = con ? tt : T[p];
        act = act | live[p];
        if (!COUNT && ((ballot(hit) >> (lane & 48)) & 0xFFFFull) != 0ull) eb |= pbit[p];
      }
      if (!COUNT && (lane & 15) == 0 && eb != 0u) atomicOr(&ev[j], eb);
      return !any_lane(act);
    };
    if (any_lane(active) && nmax > 0) {  // wave-uniform
      // two register sets, each loaded one list entry ahead of its use
      const uint8_t* hl = hits[wv][g];
      // (an entry is read unconditionally, within the row's NT bytes, and
      // replaced by 0 past the list's end, so every read is a plain LDS load)
      auto slot = [&](int t) -> int {
        const int e = (int)hl[t & (NT - 1)];
        return t < n ? e : 0;
      };
      Splat sa = batch[slot(0)], sb;
      for (int t = 0;;) {
        const int ja = slot(t);
        const bool ha = t < n;
        sb = batch[slot(t + 1)];
        if (step(sa, ja, ha) || ++t >= nmax) break;
        const int jb = slot(t);
        const bool hb = t < n;
        sa = batch[slot(t + 1)];
        if (step(sb, jb, hb) || ++t >= nmax) break;
      }
    }
    if (!COUNT) {
      __syncthreads();
      // wave w's 64 slots are one event batch: a mask per block
      const uint32_t e = (int)threadIdx.x < m ? ev[threadIdx.x] : 0u;
      unsigned long long mine = 0ull;
#pragma unroll
      for (int b = 0; b < 16; ++b) {
        const unsigned long long x = ballot(((e >> b) & 1u) != 0u);
        mine = lane == b ? x : mine;
      }
      if (lane < 16 && wv * 64 < m) event_masks(event, rg.x, tile)[16 * ((b0 - rg.x) / 64 + wv) + lane] = mine;
    }
  }
  if (!COUNT)  // segments that no pixel reached
    for (uint32_t k = b0 > rg.x ? rg.x + (b0 - rg.x + kSegment - 1) / kSegment * kSegment : rg.x + kSegment; k < rg.y;
         k += kSegment)
      checkpoint(k);
  if (COUNT) {
    for (int d = 32; d > 0; d >>= 1) {
      n_eval += __shfl_xor(n_eval, d, 64);
      n_contrib += __shfl_xor(n_contrib, d, 64);
    }
    if (lane == 0) {
      atomicAdd(work, n_eval);
      atomicAdd(work + 1, n_contrib);
    }
    return;
  }
#pragma unroll
  for (int p = 0; p < PX; ++p) {
    if (!inside[p]) continue;
    float* o = rgb + 3 * ((int64_t)pys[p] * v.width + px);
    o[0] = __builtin_fmaf(T[p], bg0, cr[p]);
    o[1] = __builtin_fmaf(T[p], bg1, cg[p]);
    o[2] = __builtin_fmaf(T[p], bg2, cb[p]);
  }
}

// A tile far longer than the others is blended by 16 waves, one per 4x4 block
// (blend_block_wave), the others by four, one per 8x8 quarter (blend_quarter).
// The waves of a tile run on one XCD (workgroups go to the
// XCDs in turn), so its words and records are read into one L2.
constexpr int kHeavyWgs = 4096;  // single-wave workgroups that take the heavy tiles' blocks in turn

// One wave on an 8x8 quarter of a tile: the wave's rows are the
// quarter's four 4x4 blocks (blend_pixel<1>), lane l its pixel.  The wave
// streams the tile's instances in batches of 64 and replays, row by row, the
// ones whose block mask meets the row's block, as k_blend does.  Instance
// words (owning splat, block mask, in tile order) are loaded two
// batches ahead and the splat records of the instances that reach the quarter
// one batch ahead, into registers, so the loads overlap the blending; the
// waves of a tile never wait for each other, and each stops when its own
// pixels have.  Events: one mask per batch and block (event_masks), zero for
// batches the wave never reached.
struct QuarterLds {
  float4 rec[3][64];    // the batch's records: (mx hi, lo, my hi, lo), (ce, se, h1, h2), (o, r, g, b)
  uint8_t hits[4][64];  // per row: the batch slots it replays, in order
  uint32_t evr[64];     // per slot: this quarter's event bits
};

template <bool LONG>
__device__ __forceinline__ void blend_quarter(const ViewConst& v, int tile, int q, uint2 rg,
                                              const uint2* __restrict__ info_k, const Splat* __restrict__ splats,
                                              uint32_t nr, float bg0, float bg1, float bg2, float* rgb,
                                              uint32_t* event, float4* ckpt, QuarterLds& lds) {
  float4 (&rec)[3][64] = lds.rec;
  uint8_t (&hits)[4][64] = lds.hits;
  uint32_t (&evr)[64] = lds.evr;
  const int tx = tile % v.tiles_x, ty = tile / v.tiles_x;
  const int lane = threadIdx.x, g = lane >> 4;
  const uint64_t lt = lanemask_lt();
  int px, py;
  blend_pixel<1>(tx, ty, q, lane, 0, px, py);
  const uint32_t pbit = blend_pixel_block<1>(q, g, 0);
  const uint32_t qbits = 0xFu << (4 * q);
  const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
  const bool inside = px < v.width && py < v.height;
  bool live = inside;
  float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
  unsigned long long* const ev64 = event_masks(event, rg.x, tile);
  const float thr = 1.0f / 255.0f;
  // pipeline: words of batches b and b + 64, the record of batch b (this lane's slot)
  uint32_t sk0 = 0u, bk0 = 0u, sk1 = 0u, bk1 = 0u;
  if (rg.x + lane < rg.y) {
    const uint2 w = info_k[rg.x + lane];
    sk0 = w.x;
    bk0 = w.y;
  }
  if (rg.x + 64 + lane < rg.y) {
    const uint2 w = info_k[rg.x + 64 + lane];
    sk1 = w.x;
    bk1 = w.y;
  }
  float4 ra = make_float4(0.f, 0.f, 0.f, 0.f), rb = ra, rc = ra;
  if (rg.x + lane < rg.y && sk0 < nr && (bk0 & qbits) != 0u) {
    const float4* r = reinterpret_cast<const float4*>(splats + sk0);
    ra = r[0];
    rb = r[1];
    rc = r[2];
  }
  // the pixels' state before instance k of the list (a segment's first)
  const auto checkpoint = [&](uint32_t k) {
    ckpt[256 * (int64_t)(k / kSegment) + 16 * (py & 15) + (px & 15)] = make_float4(live ? T : 0.0f, cr, cg, cb);
  };
  uint32_t b0 = rg.x;
  for (; b0 < rg.y; b0 += 64) {
    if (!any_lane(live)) break;  // wave-uniform
    if (LONG && b0 > rg.x && (b0 - rg.x) % kSegment == 0) checkpoint(b0);
    const int m = (int)min(64u, rg.y - b0);
    const bool mine = lane < m && sk0 < nr;
    rec[0][lane] = ra;
    rec[1][lane] = rb;
    rec[2][lane] = rc;
    evr[lane] = 0u;
    int nh[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool h = mine && (bk0 & blend_row_blocks<1>(q, r)) != 0u;
      const uint64_t hb = ballot(h);
      if (h) hits[r][__popcll(hb & lt)] = (uint8_t)lane;
      nh[r] = __popcll(hb);
    }
    __syncthreads();
    // prefetch: the records of the next batch, the words of the one after
    ra = rb = rc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (b0 + 64 + lane < rg.y && sk1 < nr && (bk1 & qbits) != 0u) {
      const float4* r = reinterpret_cast<const float4*>(splats + sk1);
      ra = r[0];
      rb = r[1];
      rc = r[2];
    }
    uint32_t sk2 = 0u, bk2 = 0u;
    if (b0 + 128 + lane < rg.y) {
      const uint2 w = info_k[b0 + 128 + lane];
      sk2 = w.x;
      bk2 = w.y;
    }
    const int n = g == 0 ? nh[0] : (g == 1 ? nh[1] : (g == 2 ? nh[2] : nh[3]));  // this row's list
    const int nmax = max(max(nh[0], nh[1]), max(nh[2], nh[3]));
    auto load = [&](int j) -> Splat {
      Splat s;
      const float4 a = rec[0][j], b = rec[1][j], c = rec[2][j];
      s.mxh = a.x; s.mxl = a.y; s.myh = a.z; s.myl = a.w;
      s.ce = b.x; s.se = b.y; s.h1 = b.z; s.h2 = b.w;
      s.o = c.x; s.r = c.y; s.g = c.z; s.b = c.w;
      return s;
    };
    // one splat (slot j of this row's list; has = false past its end) against
    // the lane's pixel; true when every pixel of the wave has stopped
    auto step = [&](const Splat& s, int j, bool has) -> bool {
      float dx, dy, u1, u2;
      const float power = splat_power(s, fx, fy, dx, dy, u1, u2);
      const float alpha = fminf(0.99f, s.o * fexp(power));
      const float tt = T * (1.0f - alpha);
      const bool hit = live & has & (alpha >= thr);
      const bool stop = hit & (tt < 0.0001f);
      const bool con = hit & !stop;
      live = live & !stop;
      const float w = alpha * T;
      cr = con ? __builtin_fmaf(s.r, w, cr) : cr;
      cg = con ? __builtin_fmaf(s.g, w, cg) : cg;
      cb = con ? __builtin_fmaf(s.b, w, cb) : cb;
      T = con ? tt : T;
      const uint64_t hb = ballot(hit);  // all lanes
      if ((lane & 15) == 0 && ((hb >> lane) & 0xFFFFull) != 0ull) atomicOr(&evr[j], pbit);
      return !any_lane(live);
    };
    if (nmax > 0) {
      const uint8_t* hl = hits[g];
      // (an entry is read unconditionally, within the row's 64 bytes, and
      // replaced by 0 past the list's end, so every read is a plain LDS load)
      auto slot = [&](int t) -> int {
        const int e = (int)hl[t & 63];
        return t < n ? e : 0;
      };
      // records one entry ahead of their use, list entries two ahead (so a
      // record's LDS read never waits for the read of its slot index)
      int ja = slot(0), jb = slot(1);
      Splat sa = load(ja), sb;
      for (int t = 0;;) {
        const int jc = slot(t + 2);
        sb = load(jb);
        if (step(sa, ja, t < n) || ++t >= nmax) break;
        const int jd = slot(t + 2);
        sa = load(jc);
        if (step(sb, jb, t < n) || ++t >= nmax) break;
        ja = jc;
        jb = jd;
      }
    }
    __syncthreads();
    // the batch's event masks of the quarter's blocks
    const uint32_t e = lane < m ? evr[lane] >> (4 * q) : 0u;
    unsigned long long own = 0ull;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const unsigned long long x = ballot(((e >> b) & 1u) != 0u);
      own = lane == b ? x : own;
    }
    if (lane < 4) ev64[16 * ((b0 - rg.x) / 64) + 4 * q + lane] = own;
    __syncthreads();
    sk0 = sk1;
    bk0 = bk1;
    sk1 = sk2;
    bk1 = bk2;
  }
  // segments and batches of the tile that this quarter never reached
  for (uint32_t k = b0 > rg.x ? rg.x + (b0 - rg.x + kSegment - 1) / kSegment * kSegment : rg.x + kSegment;
       LONG && k < rg.y; k += kSegment)
    checkpoint(k);
  const uint32_t nb = (rg.y - rg.x + 63) / 64;
  for (uint32_t k = (b0 - rg.x) / 64 + (lane >> 2); k < nb; k += 16) ev64[16 * k + 4 * q + (lane & 3)] = 0ull;
  if (inside) {
    float* o = rgb + 3 * ((int64_t)py * v.width + px);
    o[0] = __builtin_fmaf(T, bg0, cr);
    o[1] = __builtin_fmaf(T, bg1, cg);
    o[2] = __builtin_fmaf(T, bg2, cb);
  }
}

// The values of x in the four 16-lane rows' lanes of the same index, by row.
__device__ __forceinline__ void rows_of(float x, float* y) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);  // rows (0, 0, 2, 2) and (1, 1, 3, 3)
  const auto even = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);
  const auto odd = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);
  y[0] = __uint_as_float(even[0]);
  y[1] = __uint_as_float(odd[0]);
  y[2] = __uint_as_float(even[1]);
  y[3] = __uint_as_float(odd[1]);
}

// One wave on a 4x4 block of a tile, four of the block's splats at a time: row
// r evaluates the (4 s + r)-th one's alpha at the 16 pixels, the rows exchange
// the factors 1 - alpha (1 where the splat is skipped), and every row forms the
// pixel's transmittances in order, so each decision and product is the
// sequential one.  A pixel stops where the transmittance would fall below
// 1e-4: it and everything behind it then stays below, so no stop flag is kept.
// Row c adds up channel c of the four in order.  A step costs about a third
// more instructions than a quarter's (one splat for each of four blocks) and
// retires four of the block's list, which is what bounds a heavy tile: its
// wave is a serial chain of steps.  Records are stored compacted, in list
// order, and read one step ahead.
struct BlockLds {
  float4 a[64], b[64];  // (mx hi, lo, my hi, lo), (ce, se, h1, h2)
  float o[64];
  float col[3][64];     // a step's four colours of a channel are one 16-byte read
};

__device__ __forceinline__ void blend_block_wave(const ViewConst& v, int tile, int blk, uint2 rg,
                                                 const uint2* __restrict__ info_k, const Splat* __restrict__ splats,
                                                 uint32_t nr, float bg0, float bg1, float bg2, float* rgb,
                                                 uint32_t* event, float4* ckpt, BlockLds& lds) {
  const int lane = threadIdx.x, r = lane >> 4, ch = r < 3 ? r : 2;
  const int px = (tile % v.tiles_x) * kTile + 8 * ((blk >> 2) & 1) + 4 * (blk & 1) + (lane & 3);
  const int py = (tile / v.tiles_x) * kTile + 8 * (blk >> 3) + 4 * ((blk >> 1) & 1) + ((lane >> 2) & 3);
  const uint64_t lt = lanemask_lt();
  const uint32_t bit = 1u << blk;
  const float fx = (float)px + 0.5f, fy = (float)py + 0.5f, thr = 1.0f / 255.0f;
  const bool inside = px < v.width && py < v.height;
  unsigned long long* const ev64 = event_masks(event, rg.x, tile) + blk;
  float T = inside ? 1.0f : 0.0f;  // 0 once the pixel has stopped
  float Tout = 1.0f, c = 0.0f;     // the transmittance at the end, this row's channel
  // pipeline: words of batches b0 and b0 + 64, the record of batch b0 (this lane's slot)
  const auto word = [&](uint32_t k) { return k < rg.y ? info_k[k] : make_uint2(0u, 0u); };
  const auto mine = [&](const uint2& w) { return w.x < nr && (w.y & bit) != 0u; };  // (a word past the end has no bit)
  uint2 w0 = word(rg.x + lane), w1 = word(rg.x + 64 + lane);
  float4 ra = make_float4(0.f, 0.f, 0.f, 0.f), rb = ra, rc = ra;
  const auto record = [&](const uint2& w) {
    if (mine(w)) {
      const float4* p = reinterpret_cast<const float4*>(splats + w.x);
      ra = p[0];
      rb = p[1];
      rc = p[2];
    }
  };
  record(w0);
  // the pixels' state before instance k of the list (a segment's first)
  const auto checkpoint = [&](uint32_t k) {
    float* s = reinterpret_cast<float*>(ckpt + 256 * (int64_t)(k / kSegment) + 16 * (py & 15) + (px & 15));
    s[r < 3 ? r + 1 : 0] = r < 3 ? c : T;
  };
  uint32_t b0 = rg.x;
  for (; b0 < rg.y; b0 += 64) {
    if (!any_lane(T > 0.0f)) break;  // wave-uniform
    if (b0 > rg.x && (b0 - rg.x) % kSegment == 0) checkpoint(b0);
    const bool hit0 = mine(w0);
    const uint64_t hb = ballot(hit0);
    const int h = __popcll(hb), at = __popcll(hb & lt);
    if (hit0) {
      lds.a[at] = ra;
      lds.b[at] = rb;
      lds.o[at] = rc.x;
      lds.col[0][at] = rc.y;
      lds.col[1][at] = rc.z;
      lds.col[2][at] = rc.w;
    }
    // prefetch: the records of the next batch, the words of the one after
    record(w1);
    const uint2 w2 = word(b0 + 128 + lane);
    __syncthreads();
    uint64_t evm = 0ull;  // bit e: the e-th listed splat blended or stopped at a pixel of the block
    float4 a = lds.a[r], b = lds.b[r];
    float o = lds.o[r];
#pragma unroll 1
    for (int s = 0; s < h; s += 4) {  // wave-uniform
      const int e = s + r, nx = (e + 4) & 63;
      const float4 na = lds.a[nx], nb = lds.b[nx], col = *reinterpret_cast<const float4*>(&lds.col[ch][s]);
      const float no = lds.o[nx];
      Splat sp;
      sp.mxh = a.x; sp.mxl = a.y; sp.myh = a.z; sp.myl = a.w;
      sp.ce = b.x; sp.se = b.y; sp.h1 = b.z; sp.h2 = b.w;
      float dx, dy, u1, u2;
      const float power = splat_power(sp, fx, fy, dx, dy, u1, u2);
      const float alpha = fminf(0.99f, o * fexp(power));
      const bool hit = (e < h) & (alpha >= thr);
      float f[4], w[4];
      const float own = hit ? 1.0f - alpha : 1.0f;
      rows_of(own, f);
      const float t1 = T * f[0], t2 = t1 * f[1], t3 = t2 * f[2], t4 = t3 * f[3];
      float Tb = r == 0 ? T : t1;  // before this row's splat
      Tb = r >= 2 ? t2 : Tb;
      Tb = r == 3 ? t3 : Tb;
      const bool con = hit & (Tb * own >= 0.0001f);
      const uint64_t hits = ballot(hit & (Tb >= 0.0001f));  // (a pixel that had not stopped)
      rows_of(con ? alpha * Tb : 0.0f, w);
      c = w[0] > 0.0f ? __builtin_fmaf(col.x, w[0], c) : c;
      c = w[1] > 0.0f ? __builtin_fmaf(col.y, w[1], c) : c;
      c = w[2] > 0.0f ? __builtin_fmaf(col.z, w[2], c) : c;
      c = w[3] > 0.0f ? __builtin_fmaf(col.w, w[3], c) : c;
      const uint64_t four = ((hits & 0xFFFFull) ? 1ull : 0ull) | ((hits & 0xFFFF0000ull) ? 2ull : 0ull) |
                            ((hits & 0xFFFF00000000ull) ? 4ull : 0ull) | ((hits >> 48) ? 8ull : 0ull);
      evm |= four << s;
      if (any_lane((T > 0.0f) & (t4 < 0.0001f))) {  // wave-uniform: a pixel stops at one of the four
        float Tl = t1 >= 0.0001f ? t1 : T;
        Tl = t2 >= 0.0001f ? t2 : Tl;
        Tl = t3 >= 0.0001f ? t3 : Tl;
        Tout = ((T > 0.0f) & (t4 < 0.0001f)) ? Tl : Tout;
        T = t4 >= 0.0001f ? t4 : 0.0f;
        if (!any_lane(T > 0.0f)) break;
      } else {
        T = t4;
      }
      a = na;
      b = nb;
      o = no;
    }
    const uint64_t slots = ballot(hit0 && ((evm >> at) & 1ull) != 0ull);
    if (lane == 0) ev64[16 * ((b0 - rg.x) / 64)] = slots;
    __syncthreads();
    w0 = w1;
    w1 = w2;
  }
  // segments and batches of the tile that this block never reached
  for (uint32_t k = b0 > rg.x ? rg.x + (b0 - rg.x + kSegment - 1) / kSegment * kSegment : rg.x + kSegment; k < rg.y;
       k += kSegment)
    checkpoint(k);
  const uint32_t nbt = (rg.y - rg.x + 63) / 64;
  for (uint32_t k = (b0 - rg.x) / 64 + lane; k < nbt; k += 64) ev64[16 * k] = 0ull;
  if (inside && r < 3) {
    const float bg = r == 0 ? bg0 : (r == 1 ? bg1 : bg2);
    rgb[3 * ((int64_t)py * v.width + px) + r] = __builtin_fmaf(T > 0.0f ? T : Tout, bg, c);
  }
}

// Forward blend.  The first kHeavyWgs single-wave workgroups take the heavy
// tiles' blocks in turn, the others the quarters of the other tiles, in the
// tile order.  What bounds it is the longest tile's chain of steps, then the
// instructions.  Blocks shorten the chains and read a tile's list four times as
// often, so they are for tiles that would end after all others: those of at
// least kHeavyTile instances and, where more than kHeavyFew tiles hold that many,
// of a 2048th of the image's (fewer long tiles leave the chip room: 6M leaves at
// 256 x 256 342 us with that share, 224 without).  Quarters alone
// against blocks for tiles of 128, 256 and 512 instances on, us: a 333 x 171
// iteration 67 / 31 / 31 / 38, a 1080p iteration 63 / 42 / 36 / 48.  Blocks from
// 256 instances on against from a 2048th (a 1024th) on, us: a street view at
// 1080p (2.1M instances, tiles of up to 9035) 262 / 220 (217) and at 4K 196 /
// 192 (190), a 1080p iteration 35.0 / 35.1 (35.8); clouds of small splats, whose
// tiles are all long: 2M leaves at 1080p 563 / 229 (236), 6M 1356 / 518 (518), 2M
// at 1024 x 1024 473 / 367 (213).
__global__ void __launch_bounds__(64) k_blend_fwd(const ViewConst* __restrict__ vp,
                                                  const uint2* __restrict__ info_k, const Splat* __restrict__ splats,
                                                  const FrameCounters* ctr, const uint4* __restrict__ tile_order,
                                                  int32_t ntiles, float bg0, float bg1, float bg2, float* rgb,
                                                  uint32_t* event, float4* ckpt) {
  __shared__ union {
    QuarterLds quarter;
    BlockLds block;
  } lds;
  const uint32_t nr = (uint32_t)ctr->n_render;
  const int xcd = blockIdx.x & 7;
  if (blockIdx.x < kHeavyWgs) {
    const int items = (ctr->n_heavy + 7) / 8 * 128;  // eight tiles' blocks for each 16 workgroups of an XCD
    for (int i = blockIdx.x; i < items; i += kHeavyWgs) {
      const int at = (i >> 7) * 8 + xcd, blk = (i >> 3) & 15;
      if (at >= ctr->n_heavy) continue;
      const uint4 o = tile_order[at];
      blend_block_wave(*vp, (int)o.x, blk, make_uint2(o.y, o.z), info_k, splats, nr, bg0, bg1, bg2, rgb, event, ckpt,
                       lds.block);
      __syncthreads();
    }
    return;
  }
  const int i = (int)blockIdx.x - kHeavyWgs, at = (i >> 5) * 8 + xcd, q = (i >> 3) & 3;
  if (at >= ntiles) return;
  const uint4 o = tile_order[at];
  if (o.w != 0u) return;
  if (o.z - o.y > (uint32_t)kSegment)
    blend_quarter<true>(*vp, (int)o.x, q, make_uint2(o.y, o.z), info_k, splats, nr, bg0, bg1, bg2, rgb, event, ckpt,
                        lds.quarter);
  else
    blend_quarter<false>(*vp, (int)o.x, q, make_uint2(o.y, o.z), info_k, splats, nr, bg0, bg1, bg2, rgb, event, ckpt,
                         lds.quarter);
}

template <bool COUNT>
static void launch_blend(lodgs_frame* f, const ViewConst& v, const float bg[3], float* d_rgb, hipStream_t st) {
  const int ntiles = v.tiles_x * v.tiles_y;
  unsigned long long* work = COUNT ? f->work : nullptr;
  uint32_t* event = COUNT ? nullptr : f->inst_event;
  switch (f->blend_px_fwd) {
    case 1:
      if constexpr (COUNT)
        hipLaunchKernelGGL((k_blend<true, 1>), dim3(ntiles), dim3(256), 0, st, f->d_view_ren, f->info_k, f->splats,
                           f->ctr, f->tile_order, bg[0], bg[1], bg[2], d_rgb, event, work, f->ckpt);
      else
        hipLaunchKernelGGL(k_blend_fwd, dim3(kHeavyWgs + 32 * ((ntiles + 7) / 8)), dim3(64), 0, st, f->d_view_ren,
                           f->info_k, f->splats, f->ctr, f->tile_order, ntiles, bg[0], bg[1], bg[2], d_rgb, event,
                           f->ckpt);
      break;
    case 4:
      hipLaunchKernelGGL((k_blend<COUNT, 4>), dim3(ntiles), dim3(64), 0, st, f->d_view_ren,
                         f->info_k, f->splats, f->ctr, f->tile_order, bg[0], bg[1], bg[2],
                         d_rgb, event, work, f->ckpt);
      break;
    default:
      hipLaunchKernelGGL((k_blend<COUNT, 2>), dim3(ntiles), dim3(128), 0, st, f->d_view_ren,
                         f->info_k, f->splats, f->ctr, f->tile_order, bg[0], bg[1], bg[2],
                         d_rgb, event, work, f->ckpt);
      break;
  }
}

int blend_output_arg(const void* func, int* n_args) {
  // k_blend_fwd (..., bg2, rgb, event, ckpt) and k_blend<false, PX> (..., bg2, rgb, event, work, ckpt)
  if (func == reinterpret_cast<const void*>(&k_blend_fwd)) {
    *n_args = 12;
    return 9;
  }
  if (func == reinterpret_cast<const void*>(&k_blend<false, 2>) ||
      func == reinterpret_cast<const void*>(&k_blend<false, 4>)) {
    *n_args = 12;
    return 8;
  }
  return -1;
}

int render_kernel_limits() {
  // the tile counters of k_dup and k_bucket take more than the default 64 KB on large images
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bucket),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, 4 * kBucketLdsTiles);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_dup), hipFuncAttributeMaxDynamicSharedMemorySize,
                            2 * kLdsTiles);
  return e == hipSuccess ? LODGS_OK : hip_fail(e, "lodgs_frame_create: kernel LDS");
}

void launch_render(lodgs_frame* f, const int32_t* d_idx, const int32_t* d_count, const ViewConst& v,
                   const float bg[3], float* d_rgb, hipStream_t st) {
  const SceneDev& S = render_params(f);
  const int64_t cap = f->caps.max_selected, icap = f->caps.max_instances;
  stage_begin(f, LODGS_STAGE_PROJECT, st);
  launch_set_view(v, f->d_view_ren, f->ctr, kViewRender, d_count, cap, f->tile_count, f->run_sums, st);
  const int pgrid = 2048;
  switch (S.sh_degree) {
#define LODGS_PROJECT(D)                                                                                         \
  hipLaunchKernelGGL(k_project<D>, dim3(pgrid), dim3(kBlock), 0, st, S, f->d_view_ren, d_idx, d_count, cap,   \
                     f->splats, f->depth_key, f->tiles, f->rect, f->dcol, f->wave_sums,        \
                     f->run_sums)
    case 0: LODGS_PROJECT(0); break;
    case 1: LODGS_PROJECT(1); break;
    case 2: LODGS_PROJECT(2); break;
    default: LODGS_PROJECT(3); break;
#undef LODGS_PROJECT
  }
  stage_end(f, st);
  const int ntiles = v.tiles_x * v.tiles_y;
  stage_begin(f, LODGS_STAGE_DUPLICATE, st);
  hipLaunchKernelGGL(k_drawn_scan, dim3(512), dim3(kDrawnThreads), 0, st, f->tiles, f->wave_sums, f->run_sums, f->ctr, f->drawn_list,
                     f->inst_off, f->chunk_first, icap);
  const int32_t dup_lds = ntiles <= kLdsTiles ? ntiles : 0;
  hipLaunchKernelGGL(k_dup, dim3(kDupGrid), dim3(kDupThreads), 4 * ((dup_lds + 1) / 2), st, f->ctr, f->drawn_list,
                     f->inst_off, f->chunk_first, v.tiles_x, dup_lds, icap, f->depth_key, f->inst_key, f->inst_info, f->long_list,
                     f->splats, f->tile_count);
  stage_end(f, st);
  stage_begin(f, LODGS_STAGE_RANGES, st);
  hipLaunchKernelGGL(k_tile_scan, dim3(tile_chunks(ntiles)), dim3(kOrderThreads), 0, st,
                     f->tile_count, ntiles, f->ctr, f->ranges, f->tile_cursor, f->tile_order, f->seg_list,
                     f->big_list);
  stage_end(f, st);
  stage_begin(f, LODGS_STAGE_TILE_SORT, st);
  const int32_t bucket_lds = ntiles <= kBucketLdsTiles ? ntiles : 0;
  hipLaunchKernelGGL(k_bucket, dim3(kBucketGrid), dim3(kBucketThreads), 4 * bucket_lds, st, f->ctr, f->inst_key, bucket_lds,
                     f->tile_cursor, f->bucket_key);
  stage_end(f, st);
  stage_begin(f, LODGS_STAGE_DEPTH_SORT, st);
  hipLaunchKernelGGL(k_tile_sort, dim3(kTileSortGrid), dim3(kSmallThreads), 0, st, f->ctr, f->ranges,
                     f->tile_order, ntiles, f->big_list, f->bucket_key, f->inst_info, f->info_k, f->ival);
  hipLaunchKernelGGL(k_tile_merge, dim3(1024), dim3(kSmallThreads), 0, st, f->ctr, f->ranges, f->big_list,
                     f->bucket_key, f->inst_info, f->info_k, f->ival);
  stage_end(f, st);
  stage_begin(f, LODGS_STAGE_BLEND, st);
  launch_blend<false>(f, v, bg, d_rgb, st);
  stage_end(f, st);
}

__global__ void k_zero_work(unsigned long long* w) {
  w[0] = 0;
  w[1] = 0;
}

void launch_blend_count(lodgs_frame* f, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_work, dim3(1), dim3(1), 0, st, f->work);
  const float zero[3] = {0.0f, 0.0f, 0.0f};
  launch_blend<true>(f, f->view, zero, nullptr, st);
}

}  // namespace lodgs
