// Backward of the render (recompute-based): per tile, the forward
// front-to-back pass is replayed with identical FP32 decisions and the
// gradient of every contributing (splat, pixel) pair is formed on the fly,
// using the final pixel colour to obtain the colour behind each splat.  Each
// (splat, tile) instance gets one partial of per-pixel sums (moments about the
// tile centre, dL/do, dL/dRGB), written at its emission index without
// atomics.  The projection backward then forms each drawn splat's 2D sums
// from its partials in FP64 and carries them through the conic inverse, the
// EWA Jacobian, the camera transform, the covariance factorisation, the
// quaternion normalisation, the sigmoid and the SH basis to the raw
// parameters.
#include <algorithm>
#include <type_traits>

#include "lodgs_internal.h"
#include "lodgs_proj.h"

namespace lodgs {

// Reduce-scatter of NP (10 or 11) per-lane values inside each 16-lane row (all lanes
// active): four DPP exchange steps pair lane l with l^1, l^2, l^7 and l^15;
// at each step a lane keeps half of its remaining values (chosen by b0^b2,
// b1^b2, b2^b3 and b3 of l & 15) and adds its partner's copy of that half.
// Lane l then holds its row's sum of value
// slot(l) = (b0^b2) + 2 (b1^b2) + 4 (b2^b3) + 8 b3 (slots NP..15 are zero).
#define LODGS_DPP(x, ctrl) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, false))
#define LODGS_RS_PAIR(out, a, b, k, ctrl)       \
  do {                                          \
    const float keep_ = (k) ? (b) : (a);        \
    const float send_ = (k) ? (a) : (b);        \
    (out) = keep_ + LODGS_DPP(send_, ctrl);     \
  } while (0)

template <int NP>
__device__ __forceinline__ float row_reduce_scatter(const float* g, int lane, int& slot) {
  static_assert(NP == 10 || NP == 11, "10 or 11 values");
  const int b0 = lane & 1, b1 = (lane >> 1) & 1, b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1;
  const bool k1 = (b0 ^ b2) != 0, k2 = (b1 ^ b2) != 0, k3 = (b2 ^ b3) != 0, k4 = b3 != 0;
  float h0, h1, h2, h3, h4, h5;
  LODGS_RS_PAIR(h0, g[0], g[1], k1, 0xB1);  // quad_perm [1,0,3,2]: l^1
  LODGS_RS_PAIR(h1, g[2], g[3], k1, 0xB1);
  LODGS_RS_PAIR(h2, g[4], g[5], k1, 0xB1);
  LODGS_RS_PAIR(h3, g[6], g[7], k1, 0xB1);
  LODGS_RS_PAIR(h4, g[8], g[9], k1, 0xB1);
  if (NP == 11) LODGS_RS_PAIR(h5, g[10], 0.0f, k1, 0xB1);
  else h5 = 0.0f;
  float q0, q1, q2;
  LODGS_RS_PAIR(q0, h0, h1, k2, 0x4E);  // quad_perm [2,3,0,1]: l^2
  LODGS_RS_PAIR(q1, h2, h3, k2, 0x4E);
  LODGS_RS_PAIR(q2, h4, h5, k2, 0x4E);
  float r0, r1;
  LODGS_RS_PAIR(r0, q0, q1, k3, 0x141);  // row_half_mirror: l^7
  LODGS_RS_PAIR(r1, q2, 0.0f, k3, 0x141);
  float z;
  LODGS_RS_PAIR(z, r0, r1, k4, 0x140);  // row_mirror: l^15
  slot = (int)k1 + 2 * (int)k2 + 4 * (int)k3 + 8 * (int)k4;
  return z;
}
#undef LODGS_RS_PAIR
#undef LODGS_DPP

// A wave-uniform 64-bit value, moved to scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32;
}

// Backward of the blend: the forward's decisions, pixel layout blend_pixel.
// Each 16-lane row replays only the splats whose forward event bits cover one
// of its blocks: elsewhere no pixel of the row blended the splat or stopped on
// it in the forward, so the replay would leave every value unchanged.  The
// rows of a wave step through their lists together, each on its own splat.
//
// Per pixel, dL/dalpha = T (G . c) - (G . (C - Q)) / (1 - alpha), with G =
// dL/dC, c the splat colour, C the final colour and Q the colour blended up
// to and including the splat; G . C is fixed per pixel and G . Q is kept as
// one running scalar.  With w = dL/dpower = alpha dL/dalpha, the geometric
// part of a splat's gradient needs sum w d and sum w d d^T over its pixels,
// d = pixel - mean.  They are gathered as moments about the tile centre c_t
// (e = pixel - c_t, |e| <= 7.5): sum w, sum w e, sum w e e^T, so the FP32
// sums stay well conditioned even for a splat whose mean lies far off the
// screen; the projection backward shifts them by c_t - mean in FP64.  Per
// step, each row reduces these NP values of its splat (moments, dL/do, the
// colour gradient and, with NP = 11, the number of pixels it contributes to)
// over its lanes (only when some lane of the wave
// contributes) and adds them to its wave's LDS row of that splat, the four
// rows with one LDS add instruction (the LDS applies the lanes of one
// instruction in lane order, so two rows on the same splat add in row order,
// as adding them one after another does); the workgroup then sums the waves'
// rows in order and writes one NP-float partial per (splat, tile) instance at
// the instance's emission index, with zeros for instances that no pixel
// reached.  No order depends on timing: the result is deterministic.

// LDS of a workgroup of the blend backward (two or four pixels per lane; a batch
// is an instance per thread).
template <int PX, int NP>
struct BlendBwdLds {
  static_assert(PX == 2 || PX == 4, "one pixel per lane: BlocksBwdLds");
  static constexpr int NW = 4 / PX, NB = 256 / PX;
  // the first 12 floats of each splat record (mean, axis, power, opacity,
  // colour): all a replay reads, at a 12-word stride that spreads the rows'
  // reads of different slots over the banks
  struct BatchRec {
    float4 a, b, c;
  };
  BatchRec batch[NB];
  // a row of acc per partial component; slot j's component c sits at column
  // j ^ c, so the ten lanes of a row adding one slot's components hit ten
  // banks (the rows are 128 words apart)
  float acc[NW][NP][NB];
  unsigned long long emask[NB / 64][16];    // the batch's event masks by block
  unsigned long long wave_ev[NW][NB / 64];  // and over each wave's blocks
  uint32_t bid[NB];
  uint32_t wave_active[NW];  // per wave: some pixel still blends
  uint8_t hits[NW][4][NB];   // per row of each wave: the batch slots it replays, in order
};

// Instances [rg.x, rg.y) of the tile whose list begins at `first`: the whole
// list, or a segment of it.
template <int PX, int NP>
__device__ __forceinline__ void blend_bwd_range(const ViewConst& v, int tile, uint32_t first, uint2 rg,
                                                const uint32_t* __restrict__ ival, const uint2* __restrict__ info_k,
                                                const Splat* __restrict__ splats, uint32_t nr,
                                                const float* __restrict__ rgb, const float* __restrict__ dL,
                                                const uint32_t* __restrict__ event, const float4* __restrict__ ckpt,
                                                float* __restrict__ partial, BlendBwdLds<PX, NP>& lds) {
  constexpr int NW = 4 / PX, NB = BlendBwdLds<PX, NP>::NB;
  using BatchRec = typename BlendBwdLds<PX, NP>::BatchRec;
  auto& batch = lds.batch;
  auto& bid = lds.bid;
  auto& emask = lds.emask;
  auto& wave_ev = lds.wave_ev;
  auto& hits = lds.hits;
  auto& acc = lds.acc;
  auto& wave_active = lds.wave_active;
  const int tx = tile % v.tiles_x, ty = tile / v.tiles_x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, row = lane >> 4;
  int px = 0;
  float fy[PX], T[PX], GQ[PX], GC[PX], G0[PX], G1[PX], G2[PX];
  float ey[PX], exx[PX], exy[PX], eyy[PX];  // offsets from the tile centre
  bool live[PX];
#pragma unroll
  for (int p = 0; p < PX; ++p) {
    int py;
    blend_pixel<PX>(tx, ty, wv, lane, p, px, py);
    fy[p] = (float)py + 0.5f;
    live[p] = px < v.width && py < v.height;
    T[p] = 1.0f;
    GQ[p] = GC[p] = G0[p] = G1[p] = G2[p] = 0.0f;
    if (live[p]) {
      const int64_t o = 3 * ((int64_t)py * v.width + px);
      G0[p] = dL[o];
      G1[p] = dL[o + 1];
      G2[p] = dL[o + 2];
      GC[p] = __builtin_fmaf(G2[p], rgb[o + 2], __builtin_fmaf(G1[p], rgb[o + 1], G0[p] * rgb[o]));
      if (rg.x > first) {  // the pixel's state before the segment
        const float4 s = ckpt[256 * (int64_t)(rg.x / kSegment) + 16 * (py & 15) + (px & 15)];
        T[p] = s.x;
        GQ[p] = __builtin_fmaf(G2[p], s.w, __builtin_fmaf(G1[p], s.z, G0[p] * s.y));
        live[p] = s.x > 0.0f;
      }
    }
  }
  const float fx = (float)px + 0.5f;
  const float ex = fx - (float)(16 * tx + 8);
#pragma unroll
  for (int p = 0; p < PX; ++p) {
    ey[p] = fy[p] - (float)(16 * ty + 8);
    exx[p] = ex * ex;
    exy[p] = ex * ey[p];
    eyy[p] = ey[p] * ey[p];
  }
  const float thr = 1.0f / 255.0f;
  for (int t = threadIdx.x; t < NW * NP * NB; t += NB) (&acc[0][0][0])[t] = 0.0f;
  // Thread j holds batch slot j: the words (emission index, splat, whether the
  // instance has an event) of this batch and the next, and the splat record of
  // this batch (only for an instance with events: the others are never
  // replayed), so the loads overlap the replay of the batch before.
  const int ld = (int)threadIdx.x;
  const unsigned long long* const ev64 = event_masks(event, first, tile) + 16 * ((rg.x - first) / 64);
  const uint32_t nbt = (rg.y - rg.x + 63) / 64;
  // e, i of the loaded slot, and lane l % 16's event mask of the 64 slots that
  // this wave loads (block l % 16's)
  auto words = [&](uint32_t b, uint32_t& e, uint32_t& i, unsigned long long& mk) {
    const uint32_t k = b + (uint32_t)ld;
    e = i = 0u;
    mk = 0ull;
    if (k < rg.y) {
      e = ival[k];
      i = info_k[k].x;
    }
    const uint32_t eb = (b - rg.x) / 64 + (uint32_t)(ld >> 6);  // wave-uniform
    if (eb < nbt) mk = ev64[16 * eb + (lane & 15)];
  };
  // whether the loaded slot has an event in any block
  auto any_event = [&](unsigned long long mk) -> bool {
    uint32_t lo = (uint32_t)mk, hi = (uint32_t)(mk >> 32);
#define LODGS_OR16(x, ctrl) x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xf, 0xf, false)
    LODGS_OR16(lo, 0xB1);   // quad_perm [1,0,3,2]
    LODGS_OR16(hi, 0xB1);
    LODGS_OR16(lo, 0x4E);   // quad_perm [2,3,0,1]
    LODGS_OR16(hi, 0x4E);
    LODGS_OR16(lo, 0x141);  // row_half_mirror
    LODGS_OR16(hi, 0x141);
    LODGS_OR16(lo, 0x140);  // row_mirror
    LODGS_OR16(hi, 0x140);
#undef LODGS_OR16
    return (((lane < 32 ? lo : hi) >> (lane & 31)) & 1u) != 0u;
  };
  auto record = [&](uint32_t i, unsigned long long mk, float4& a, float4& b, float4& c) {
    a = b = c = make_float4(0.f, 0.f, 0.f, 0.f);
    if (any_event(mk) && i < nr) {  // i >= nr only follows an instance overflow (no events)
      const float4* r = reinterpret_cast<const float4*>(splats + i);
      a = r[0];
      b = r[1];
      c = r[2];
    }
  };
  uint32_t e0, i0, e1, i1;
  unsigned long long w0, w1;
  words(rg.x, e0, i0, w0);
  words(rg.x + NB, e1, i1, w1);
  float4 ra, rb, rc;
  record(i0, w0, ra, rb, rc);
  uint32_t b0 = rg.x;
  for (; b0 < rg.y; b0 += NB) {
    bool active = false;
#pragma unroll
    for (int p = 0; p < PX; ++p) active = active || live[p];
    // each wave publishes whether a pixel of it still blends with the batch,
    // behind the batch's barrier (no block-wide count, which takes three)
    const bool wave_act = any_lane(active);
    if (lane == 0) wave_active[wv] = wave_act ? 1u : 0u;
    bid[ld] = e0;
    if (lane < 16) emask[ld >> 6][lane] = w0;
    float4* staged = reinterpret_cast<float4*>(&batch[ld]);  // mean, axis, power, opacity, colour
    staged[0] = ra;
    staged[1] = rb;
    staged[2] = rc;
    __syncthreads();
    uint32_t block_act = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) block_act |= wave_active[w];
    if (block_act == 0u) break;  // every pixel of the tile has stopped (the same flags for all threads)
    // the emission index this thread writes out to after the replay
    const uint32_t out_bid = bid[ld];
    record(i1, w1, ra, rb, rc);
    uint32_t e2, i2;
    unsigned long long w2;
    words(b0 + 2 * NB, e2, i2, w2);
    const int m = (int)min((uint32_t)NB, rg.y - b0);
    // every row's list of the batch slots with an event in one of its blocks,
    // in slot order (ranks in the masks)
    const uint64_t lt = lanemask_lt();
    int nh[4];
    uint64_t wave_any[NB / 64];
#pragma unroll
    for (int c = 0; c < NB / 64; ++c) wave_any[c] = 0ull;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int cnt = 0;
#pragma unroll
      for (int c = 0; c < NB / 64; ++c) {
        uint64_t hb = 0ull;
#pragma unroll
        for (int p = 0; p < PX; ++p) hb |= emask[c][31 - __builtin_clz(blend_pixel_block<PX>(wv, r, p))];
        hb = uniform64(hb);
        if ((hb >> lane) & 1ull) hits[wv][r][cnt + __popcll(hb & lt)] = (uint8_t)(c * 64 + lane);
        cnt += __popcll(hb);
        wave_any[c] |= hb;
      }
      nh[r] = cnt;
    }
    if (lane == 0) {
#pragma unroll
      for (int c = 0; c < NB / 64; ++c) wave_ev[wv][c] = wave_any[c];
    }
    // the hit lists are the wave's own (its LDS operations run in order): a
    // wave-level fence and barrier order their writes before the reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int n = row == 0 ? nh[0] : (row == 1 ? nh[1] : (row == 2 ? nh[2] : nh[3]));  // this row's list
    const int nmax = max(max(nh[0], nh[1]), max(nh[2], nh[3]));
    if (any_lane(active) && nmax > 0) {  // wave-uniform
      // one splat (batch slot j of this row's list; has = false past its end)
      // against the row's pixels; true when every pixel of the wave has
      // stopped
      auto step = [&](const Splat& s, int j, bool has) -> bool {
        float dxs[PX], dys[PX], u1s[PX], u2s[PX], es[PX], oes[PX], als[PX], tts[PX];
        bool cons[PX];
        bool any_con = false, act = false;
#pragma unroll
        for (int p = 0; p < PX; ++p) {
          const float power = splat_power(s, fx, fy[p], dxs[p], dys[p], u1s[p], u2s[p]);
          es[p] = fexp(power);
          oes[p] = s.o * es[p];
          als[p] = fminf(0.99f, oes[p]);
          tts[p] = T[p] * (1.0f - als[p]);
          const bool hit = live[p] & has & (als[p] >= thr);
          const bool stop = hit & (tts[p] < 0.0001f);
          cons[p] = hit & !stop;
          live[p] = live[p] & !stop;
          any_con = any_con | cons[p];
          act = act | live[p];
        }
        if (any_lane(any_con)) {  // wave-uniform
          // the first pixel's terms start the sums: only the sign of a zero
          // sum differs from adding them to +0, and the LDS rows (never -0)
          // absorb that
          float g[11];
#pragma unroll
          for (int p = 0; p < PX; ++p) {
            const float alpha = als[p], Tp = T[p];
            const float w = alpha * Tp;
            const float Gc = __builtin_fmaf(G2[p], s.b, __builtin_fmaf(G1[p], s.g, G0[p] * s.r));
            const float gq = __builtin_fmaf(w, Gc, GQ[p]);
            const float ia = __builtin_amdgcn_rcpf(1.0f - alpha);  // gradient values only
            const float dA = Tp * Gc - (GC[p] - gq) * ia;
            const bool con = cons[p];
            const bool unclamped = con & (oes[p] <= 0.99f);
            // the factors are zeroed for pixels without a contribution (the
            // other factors are finite), so the sums need no further selects
            const float dpow = unclamped ? dA * alpha : 0.0f;
            const float dop = unclamped ? dA * es[p] : 0.0f;
            const float wc = con ? w : 0.0f;
            if (p == 0) {
              g[0] = dpow;
              g[1] = dpow * ex;
              g[2] = dpow * ey[p];
              g[3] = dpow * exx[p];
              g[4] = dpow * exy[p];
              g[5] = dpow * eyy[p];
              g[6] = dop;
              g[7] = G0[p] * wc;
              g[8] = G1[p] * wc;
              g[9] = G2[p] * wc;
              g[10] = con ? 1.0f : 0.0f;  // contributing pixels (read only with NP = 11)
            } else {
              g[0] += dpow;
              g[1] = __builtin_fmaf(dpow, ex, g[1]);
              g[2] = __builtin_fmaf(dpow, ey[p], g[2]);
              g[3] = __builtin_fmaf(dpow, exx[p], g[3]);
              g[4] = __builtin_fmaf(dpow, exy[p], g[4]);
              g[5] = __builtin_fmaf(dpow, eyy[p], g[5]);
              g[6] += dop;
              g[7] = __builtin_fmaf(G0[p], wc, g[7]);
              g[8] = __builtin_fmaf(G1[p], wc, g[8]);
              g[9] = __builtin_fmaf(G2[p], wc, g[9]);
              if (NP == 11) g[10] += con ? 1.0f : 0.0f;
            }
            GQ[p] = con ? gq : GQ[p];
            T[p] = con ? tts[p] : Tp;
          }
          int slot;
          const float r = row_reduce_scatter<NP>(g, lane, slot);
          // the rows add into the wave's row of their splats with one LDS
          // add instruction (two rows may be on the same splat: the LDS
          // applies the lanes of one instruction in a fixed order)
          const uint64_t cm = ballot(any_con);
          if (slot < NP && ((cm >> (16 * row)) & 0xFFFFull) != 0ull)
            __hip_atomic_fetch_add(&acc[wv][slot][j ^ slot], r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        return !any_lane(act);
      };
      // two register sets, each loaded one list entry ahead of its use
      static_assert((NB & (NB - 1)) == 0, "a power of two of list entries");
      const uint8_t* hl = hits[wv][row];
      // (an entry is read unconditionally, within the row's NB bytes, and
      // replaced by 0 past the list's end, so every read is a plain LDS load)
      auto slot_at = [&](int t) -> int {
        const int e = (int)hl[t & (NB - 1)];
        return t < n ? e : 0;
      };
      auto rec = [&](int j) -> Splat {
        const BatchRec& q = batch[j];
        Splat sp;
        sp.mxh = q.a.x;
        sp.mxl = q.a.y;
        sp.myh = q.a.z;
        sp.myl = q.a.w;
        sp.ce = q.b.x;
        sp.se = q.b.y;
        sp.h1 = q.b.z;
        sp.h2 = q.b.w;
        sp.o = q.c.x;
        sp.r = q.c.y;
        sp.g = q.c.z;
        sp.b = q.c.w;
        sp.rect_x = sp.rect_y = sp.pad0 = sp.pad1 = 0u;
        return sp;
      };
      // (the list entries themselves two ahead, so a record's LDS read never
      // waits for the read of its slot index)
      int ja = slot_at(0), jb = slot_at(1);
      Splat sa = rec(ja), sb;
      for (int t = 0;;) {
        const int jc = slot_at(t + 2);
        sb = rec(jb);
        if (step(sa, ja, t < n) || ++t >= nmax) break;
        const int jd = slot_at(t + 2);
        sa = rec(jc);
        if (step(sb, jb, t < n) || ++t >= nmax) break;
        ja = jc;
        jb = jd;
      }
    }
    __syncthreads();
    if ((int)threadIdx.x < m) {
      // Only the waves whose blocks hold one of the instance's events replayed
      // it: the other waves' rows of this slot are still +0 and are neither
      // read nor cleared.  Skipping them leaves the sums bit-identical (a row
      // value is never -0: rows start at +0 and x + y is -0 only when both
      // are), and an instance without events is written as zeros.
      float* dst = partial + NP * (int64_t)out_bid;
      float r[NP];
#pragma unroll
      for (int c = 0; c < NP; ++c) r[c] = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        if (((wave_ev[w][threadIdx.x >> 6] >> lane) & 1ull) == 0ull) continue;
#pragma unroll
        for (int c = 0; c < NP; ++c) {
          const int col = (int)threadIdx.x ^ c;
          r[c] += acc[w][c][col];
          acc[w][c][col] = 0.0f;
        }
      }
#pragma unroll
      for (int c = 0; c < NP; ++c) dst[c] = r[c];
    }
    e0 = e1;
    i0 = i1;
    w0 = w1;
    e1 = e2;
    i1 = i2;
    w1 = w2;
  }
  // instances that no pixel of the tile reached
  for (uint32_t k = b0 + threadIdx.x; k < rg.y; k += NB) {
    float* dst = partial + NP * (int64_t)ival[k];
#pragma unroll
    for (int c = 0; c < NP; ++c) dst[c] = 0.0f;
  }
}

// Columns of the blend backward's matrix products, for a wave whose row r is
// the block (r & 1, r >> 1) of a 2 x 2 group (PX = 1).  Columns 0..12 of the
// first product hold the moment factors 1; x of the left and right blocks; y
// of the upper and lower ones; x^2; y^2; x y of the four.  The second holds a
// colour channel of dL/dC of one block in each of twelve columns, placed where
// the first has nothing for that block, so that a row's nine sums lie in nine
// different columns.
constexpr int kMomentColumns = 13;
struct BwdColumns {
  // per column, by 4-bit field from bit 0: for rows 0..3 which sum it holds
  // for the row's splats (0..5 the moments 1, x, y, x^2, x y, y^2; 6..8 the
  // colours; 15 none); the moment's powers (x | y << 2); its block (column |
  // row << 1); the colour's row; its channel (3: none)
  uint32_t col[16];
  // per row, the lanes whose columns hold one of its sums, and a colour
  uint64_t takes[4], colour[4];
};
constexpr BwdColumns bwd_columns() {
  constexpr int colours[4][3] = {{2, 4, 6}, {1, 5, 8}, {3, 7, 12}, {9, 10, 11}};
  BwdColumns t{};
  for (int c = 0; c < 16; ++c) {
    int px = 0, py = 0, b = 0;
    if (c == 1 || c == 2) px = 1, b = c - 1;
    if (c == 3 || c == 4) py = 1, b = 2 * (c - 3);
    if (c == 5 || c == 6) px = 2, b = c - 5;
    if (c == 7 || c == 8) py = 2, b = 2 * (c - 7);
    if (c >= 9 && c < kMomentColumns) px = py = 1, b = c - 9;
    uint32_t crow = 0, ch = 3;
    for (int r = 0; r < 4; ++r) {
      const int m[6] = {0, 1 + (r & 1), 3 + (r >> 1), 5 + (r & 1), 9 + r, 7 + (r >> 1)};
      uint32_t sum = 15;
      for (int k = 0; k < 6; ++k)
        if (m[k] == c) sum = (uint32_t)k;
      for (int k = 0; k < 3; ++k)
        if (colours[r][k] == c) sum = 6u + (uint32_t)k, crow = (uint32_t)r, ch = (uint32_t)k;
      t.col[c] |= sum << (4 * r);
      if (sum < 9) t.takes[r] |= 0x0001000100010001ull << c;
      if (sum >= 6 && sum < 9) t.colour[r] |= 0x0001000100010001ull << c;
    }
    t.col[c] |= (uint32_t)(px | py << 2) << 16 | (uint32_t)b << 20 | crow << 24 | ch << 28;
  }
  return t;
}
constexpr BwdColumns kBwdColumns = bwd_columns();
static_assert(kBwdColumns.takes[0] == 0x02FF02FF02FF02FFull && kBwdColumns.takes[3] == 0x1F551F551F551F55ull,
              "nine columns a row");
__constant__ uint32_t kBwdColumn[16] = {
    kBwdColumns.col[0],  kBwdColumns.col[1],  kBwdColumns.col[2],  kBwdColumns.col[3],
    kBwdColumns.col[4],  kBwdColumns.col[5],  kBwdColumns.col[6],  kBwdColumns.col[7],
    kBwdColumns.col[8],  kBwdColumns.col[9],  kBwdColumns.col[10], kBwdColumns.col[11],
    kBwdColumns.col[12], kBwdColumns.col[13], kBwdColumns.col[14], kBwdColumns.col[15]};
typedef float float4_t __attribute__((ext_vector_type(4)));
// Orders the wave's LDS writes before its later reads (its LDS operations run
// in order: nothing to wait for).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same for PX = 1, the default, in fewer instructions: they and the LDS
// had bounded the kernel.  A wave's rows are the 2 x 2 blocks of a quarter.  A
// lane holds one component of its row's splat, read by the others with a row
// broadcast that is part of the instruction that uses it (one 4-byte LDS read
// a step and one register, instead of three of 16 bytes and twelve).  The sums
// over a block's pixels are matrix products: after four steps the terms of 16
// (step, row) splats at 16 pixels, 16 x 16, times the columns' factors at
// those pixels, in FP32.  The moments are summed without the opacity, which
// multiplies the totals, and about the quarter's centre, which keeps the sums
// small.  The gradients' errors against 64 bits over those of the tree of adds
// about the tile's centre, geometric means over 27 views: scales 0.90, means and
// rotations 0.93, colours 0.99, opacities 1.02.  A single view's lies between
// 0.5 and 3 where one splat, ill-conditioned in that view, decides it.  (The
// moments in two chains as well: 0.87, 0.90, 0.92, 0.99 and 1.01, but such a
// splat's gradients move by 1e-4 with any rounding, so the chains stay.)  A
// step takes 62 vector instructions where it took 110, and the float adds in
// the LDS (3 cycles a lane each) are gone.  96 registers and 31 KB let five
// workgroups run on a CU, which hides part of the batches' waits: with four, 5
// to 10% slower.  What is left: the waits of a workgroup's waves for each
// other at every batch (the vector units issue two thirds of the time).
// Before and after, us: an aerial 1080p view 139 / 117, a 1080p iteration
// 90 / 70, a view of a batch 145 / 96, a street view 318 / 269, a 333 x 171
// iteration 39 / 36.
template <int NP>
struct BlocksBwdLds {
  static constexpr int NW = 4, NB = 64, NA = NP - 1;
  static constexpr int kRow = NB + 20;  // (sums of one slot, and the slots of a write-out, on different banks)
  float rec[NB + 4][16];  // the records' first 12 floats; slots NB.. are splats that reach no pixel
  // per wave, the dL/do terms and the weights of four steps' splats (step,
  // row) at the 16 pixels of the row's block
  float4 fac[NW][2][64];
  float4 grad[NW][64];  // the second product's right operands
  float acc[NW][NA + 1][kRow];  // a row per sum, and one for the columns without
  unsigned long long emask[2][16];  // the event masks of a batch and the next by block
  uint32_t wave_active[NW];      // per wave: some pixel still blends
  uint8_t hits[NW][NB + 4][4];   // per wave and row: the batch slots it replays, in order, then slots NB..
};

template <int N>
__device__ __forceinline__ float row_lane(float x) {  // lane N of the row
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + N, 0xf, 0xf, true));
}

template <int NP>
__device__ __forceinline__ void blend_bwd_blocks(const ViewConst& v, int tile, uint32_t first, uint2 rg,
                                                 const uint32_t* __restrict__ ival, const uint2* __restrict__ info_k,
                                                 const Splat* __restrict__ splats, uint32_t nr,
                                                 const float* __restrict__ rgb, const float* __restrict__ dL,
                                                 const uint32_t* __restrict__ event, const float4* __restrict__ ckpt,
                                                 float* __restrict__ partial, BlocksBwdLds<NP>& lds) {
  constexpr int NW = BlocksBwdLds<NP>::NW, NB = BlocksBwdLds<NP>::NB, NA = BlocksBwdLds<NP>::NA;
  constexpr int kRow = BlocksBwdLds<NP>::kRow;
  const int tx = tile % v.tiles_x, ty = tile / v.tiles_x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, row = lane >> 4;
  // a thread loads part `part` of batch slot `mine`'s record and writes a
  // quarter of its sums
  const int mine = threadIdx.x >> 2, part = threadIdx.x & 3;
  const unsigned long long* const ev64 = event_masks(event, first, tile) + 16 * ((rg.x - first) / 64);
  // the slot's splat, and block (lane % 16)'s event mask of the batch
  const auto words = [&](uint32_t b, uint32_t& i, unsigned long long& mk) {
    i = b + mine < rg.y ? info_k[b + mine].x : 0u;
    mk = b < rg.y ? ev64[16 * ((b - rg.x) / 64) + (lane & 15)] : 0ull;
  };
  // the record's part, if the slot has an event in any block
  const auto record = [&](uint32_t i, unsigned long long mk) -> float4 {
    uint32_t x = wv < 2 ? (uint32_t)mk : (uint32_t)(mk >> 32);
#define LODGS_OR16(ctrl) x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xf, 0xf, true)
    LODGS_OR16(0xB1);   // quad_perm [1,0,3,2]
    LODGS_OR16(0x4E);   // quad_perm [2,3,0,1]
    LODGS_OR16(0x141);  // row_half_mirror
    LODGS_OR16(0x140);  // row_mirror
#undef LODGS_OR16
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    // (i >= nr only follows an instance overflow, without events)
    if (((x >> (mine & 31)) & 1u) != 0u && i < nr && part < 3) r = reinterpret_cast<const float4*>(splats + i)[part];
    return r;
  };
  uint32_t i0, i1;
  unsigned long long mk0, mk1;
  words(rg.x, i0, mk0);
  words(rg.x + NB, i1, mk1);
  int px, py;
  blend_pixel<1>(tx, ty, wv, lane, 0, px, py);
  const float fx = (float)px + 0.5f, fy = (float)py + 0.5f, thr = 1.0f / 255.0f;
  // (a stopped pixel's transmittance is 0: whatever hits it stops it again)
  float T = 0.0f, GQ = 0.0f, GC = 0.0f, G0 = 0.0f, G1 = 0.0f, G2 = 0.0f;
  if (px < v.width && py < v.height) {
    const int64_t o = 3 * ((int64_t)py * v.width + px);
    G0 = dL[o];
    G1 = dL[o + 1];
    G2 = dL[o + 2];
    GC = __builtin_fmaf(G2, rgb[o + 2], __builtin_fmaf(G1, rgb[o + 1], G0 * rgb[o]));
    T = 1.0f;
    if (rg.x > first) {  // the pixel's state before the segment
      const float4 s = ckpt[256 * (int64_t)(rg.x / kSegment) + 16 * (py & 15) + (px & 15)];
      T = s.x;
      GQ = __builtin_fmaf(G2, s.w, __builtin_fmaf(G1, s.z, G0 * s.y));
    }
  }
  // A splat that only stops pixels of a block has weights of 0 there, and 0
  // times a derivative that is not finite is not 0: then its sums go to a slot
  // past the batch.
  const bool odd = any_lane(!((G0 - G0) + (G1 - G1) + (G2 - G2) == 0.0f));
  for (int t = threadIdx.x; t < (int)(sizeof lds.acc / sizeof(float)); t += 256) (&lds.acc[0][0][0])[t] = 0.0f;
  if (threadIdx.x < 64) lds.rec[NB + row][lane & 15] = 0.0f;
  // the right operands (this lane: column lane & 15, pixels (m, row) of the
  // blocks) and, by row, where the column's sums go
  float bm[4];
  uint32_t dest[2];
  {
    const uint32_t cw = kBwdColumn[lane & 15];
    const uint32_t mx = (cw >> 16) & 3u, my = (cw >> 18) & 3u, ch = cw >> 28;
    const float x0 = (float)(4 * (int)((cw >> 20) & 1u)) - 3.5f;
    const float y = (float)(4 * (int)((cw >> 21) & 1u) + row) - 3.5f;
    const float yy = (lane & 15) >= kMomentColumns ? 0.0f : (my == 0u ? 1.0f : (my == 1u ? y : y * y));
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float x = x0 + (float)m;
      bm[m] = yy * (mx == 0u ? 1.0f : (mx == 1u ? x : x * x));
    }
    float* const g = reinterpret_cast<float*>(&lds.fac[wv][0][0]);  // dL/dC by channel
    g[lane] = G0;
    g[64 + lane] = G1;
    g[128 + lane] = G2;
    g[192 + lane] = 0.0f;
    wave_fence();
    lds.grad[wv][lane] = lds.fac[wv][0][16 * ch + 4 * ((cw >> 24) & 3u) + row];
    const auto to = [&](uint32_t c) { return min(c, (uint32_t)NA) * kRow; };
    dest[0] = to(cw & 15u) | to((cw >> 4) & 15u) << 16;
    dest[1] = to((cw >> 8) & 15u) | to((cw >> 12) & 15u) << 16;
    wave_fence();
  }
  float4 rec = record(i0, mk0);
  if (threadIdx.x < 16) lds.emask[0][threadIdx.x] = mk0;
  uint32_t b0 = rg.x, turn = 0;
  for (; b0 < rg.y; b0 += NB, turn ^= 1u) {
    const bool wave_act = any_lane(T > 0.0f);
    if (lane == 0) lds.wave_active[wv] = wave_act ? 1u : 0u;
    reinterpret_cast<float4*>(&lds.rec[mine][0])[part] = rec;
    __syncthreads();
    uint32_t block_act = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) block_act |= lds.wave_active[w];
    if (block_act == 0u) break;  // every pixel of the tile has stopped (the same flags for all threads)
    const int m = (int)min((uint32_t)NB, rg.y - b0);
    const uint32_t out = mine < m ? ival[b0 + mine] : 0u;
    rec = record(i1, mk1);
    if (threadIdx.x < 16) lds.emask[turn ^ 1u][threadIdx.x] = mk1;
    words(b0 + 2 * NB, i1, mk1);
    // every row's list of the batch slots with an event in its block, in slot
    // order (ranks in the masks)
    int nmax = 0, nh[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint64_t hb = uniform64(lds.emask[turn][31 - __builtin_clz(blend_pixel_block<1>(wv, r, 0))]);
      if (__builtin_amdgcn_inverse_ballot_w64(hb))
        lds.hits[wv][__builtin_amdgcn_mbcnt_hi((uint32_t)(hb >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hb, 0u))][r] =
            (uint8_t)lane;
      nh[r] = __popcll(hb);
      nmax = max(nmax, nh[r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      for (int k = nh[r]; k < nmax + 3; k += 64)  // wave-uniform
        if (k + lane < nmax + 3) lds.hits[wv][k + lane][r] = (uint8_t)(NB + (lane & 3));
    wave_fence();
    if (wave_act && nmax > 0) {  // wave-uniform
      float* const fac = reinterpret_cast<float*>(&lds.fac[wv][0][0]) + lane;
      // step st of four: one splat per row (a component a lane) against the
      // row's pixels; false when every pixel of the wave has stopped
      const auto step = [&](float s, int st, int j) -> bool {
        Splat sp;
        sp.mxh = row_lane<0>(s);
        sp.mxl = row_lane<1>(s);
        sp.myh = row_lane<2>(s);
        sp.myl = row_lane<3>(s);
        sp.ce = row_lane<4>(s);
        sp.se = row_lane<5>(s);
        sp.h1 = row_lane<6>(s);
        sp.h2 = row_lane<7>(s);
        float dx, dy, u1, u2;
        const float e = fexp(splat_power(sp, fx, fy, dx, dy, u1, u2));
        const float oe = row_lane<8>(s) * e, alpha = fminf(0.99f, oe), left = 1.0f - alpha, tt = T * left;
        const bool hit = alpha >= thr, con = hit & (tt >= 0.0001f);
        const float Gc = __builtin_fmaf(row_lane<11>(s), G2, __builtin_fmaf(row_lane<10>(s), G1, row_lane<9>(s) * G0));
        const float w = alpha * T, gq = __builtin_fmaf(w, Gc, GQ), wc = con ? w : 0.0f;
        const float ia = __builtin_amdgcn_rcpf(left);  // gradient values only
        const float dA = T * Gc - (GC - gq) * ia;
        GQ = con ? gq : GQ;
        fac[64 * st] = (con & (oe <= 0.99f)) ? dA * e : 0.0f;
        fac[256 + 64 * st] = wc;
        T = con ? tt : (hit ? 0.0f : T);
        if (NP == 11) {  // contributing pixels
          const uint64_t cm = ballot(con);
          if ((lane & 15) == 0 && j < NB)
            __hip_atomic_fetch_add(&lds.acc[wv][NA - 1][j], (float)__popc((uint32_t)(cm >> lane) & 0xFFFFu),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        return any_lane(T > 0.0f);
      };
      // the sums of the four steps from list entry t on (entries past a row's
      // list leave zeros): register r holds row r's, lane (column, step)
      float4_t d1 = {0.f, 0.f, 0.f, 0.f}, d2 = {0.f, 0.f, 0.f, 0.f};
      uint32_t slots = NB * 0x01010101u;  // of the four rows' splats, by byte
      const auto sums = [&](int t) {
        wave_fence();
        const float4 ao = lds.fac[wv][0][4 * (lane & 15) + row], aw = lds.fac[wv][1][4 * (lane & 15) + row];
        const float4 bg = lds.grad[wv][lane];
        if (odd) {  // wave-uniform; bit 4 step + row of `some`: the splat has a weight
          uint64_t some = ballot((aw.x != 0.0f) | (aw.y != 0.0f) | (aw.z != 0.0f) | (aw.w != 0.0f));
          some |= some >> 32;
          some |= some >> 16;
          if (lane < 16 && ((some >> lane) & 1ull) == 0ull)
            lds.hits[wv][t + (lane >> 2)][lane & 3] = (uint8_t)(NB + (lane >> 2));
          wave_fence();
        }
        slots = *reinterpret_cast<const uint32_t*>(&lds.hits[wv][t + row][0]);
        d1 = d2 = float4_t{0.f, 0.f, 0.f, 0.f};
        float4_t d3 = d2;  // (two shorter chains round less)
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ao.x, bm[0], d1, 0, 0, 0);
        d2 = __builtin_amdgcn_mfma_f32_16x16x4f32(aw.x, bg.x, d2, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ao.y, bm[1], d1, 0, 0, 0);
        d2 = __builtin_amdgcn_mfma_f32_16x16x4f32(aw.y, bg.y, d2, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ao.z, bm[2], d1, 0, 0, 0);
        d3 = __builtin_amdgcn_mfma_f32_16x16x4f32(aw.z, bg.z, d3, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ao.w, bm[3], d1, 0, 0, 0);
        d3 = __builtin_amdgcn_mfma_f32_16x16x4f32(aw.w, bg.w, d3, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) d2[r] += d3[r];
      };
      // row r's sums are added to the wave's rows of their splats: a read, an
      // add and a write (a float add in the LDS takes 3 cycles a lane, 195 an
      // instruction; a read and a write 8), the read a step ahead of the
      // write.  The splats of one row's entries differ, and the wave's LDS
      // operations run in order.
      float* const accs = &lds.acc[wv][0][0];
      const auto place = [&](int r) -> float* {
        return accs + ((dest[r >> 1] >> (16 * (r & 1))) & 0xFFFFu) + ((slots >> (8 * r)) & 0xFFu);
      };
      const auto sum = [&](int r) -> float {
        return __builtin_amdgcn_inverse_ballot_w64(kBwdColumns.colour[r]) ? d2[r] : d1[r];
      };
      // records one list entry ahead of their use, entries two ahead, so a
      // record's read never waits for the read of its slot
      const uint8_t* hl = &lds.hits[wv][0][row];
      int ja = hl[0], jb = hl[4];
      float sa = lds.rec[ja][lane & 15], sb;
      bool go = true;
      for (int t = 0; go; t += 4) {
        int end = t;
#pragma unroll
        for (int st = 0; st < 4; st += 2) {
          const int jc = hl[4 * (t + st + 2)];
          sb = lds.rec[jb][lane & 15];
          float* const pa = place(st);
          const float xa = *pa;
          go = step(sa, st, ja);
          *pa = xa + sum(st);
          wave_fence();
          go = ++end < nmax && go;
          if (!go) break;
          const int jd = hl[4 * (t + st + 3)];
          sa = lds.rec[jc][lane & 15];
          float* const pb = place(st + 1);
          const float xb = *pb;
          go = step(sb, st + 1, jb);
          *pb = xb + sum(st + 1);
          wave_fence();
          go = ++end < nmax && go;
          if (!go) break;
          ja = jc;
          jb = jd;
        }
        // (after a last group that is not whole: the steps and rows left)
#pragma unroll
        for (int st = 1; st < 4; ++st)
          if (end - t <= st) {
            fac[64 * st] = fac[256 + 64 * st] = 0.0f;
            *place(st) += sum(st);
            wave_fence();
          }
        sums(t);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        *place(r) += sum(r);
        wave_fence();
      }
    }
    __syncthreads();
    if (mine < m) {
      // The waves' sums in order; the moments, which were summed without the
      // opacity and about the quarters' centres, are moved to the tile's, at
      // (-+4, -+4): with m0, mx, my the zeroth and first ones, x gains cx m0,
      // x^2 2 cx mx + 16 m0, x y cx my + cy mx + cx cy m0.
      float pair[2][3] = {};  // the waves' sums by pairs
      int pt = part;
      asm volatile("" : "+v"(pt));  // keeps the factors from being held in registers over the batches
      const float ax = pt == 1 ? 4.0f : 0.0f, ay = pt == 2 ? 4.0f : 0.0f, aq = pt == 3 ? 16.0f : 0.0f;
      const float bx = pt == 3 ? 8.0f : 0.0f;
      const float cq = pt == 1 ? 16.0f : 0.0f, cxy = pt == 0 ? 16.0f : 0.0f;
      const float c4 = pt == 0 ? 4.0f : 0.0f, cy = pt == 1 ? 8.0f : 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float sx = w & 1 ? 1.0f : -1.0f, sy = w >> 1 ? 1.0f : -1.0f;
        const float m0 = lds.acc[w][0][mine], mx = lds.acc[w][1][mine], my = lds.acc[w][2][mine];
        const float x0 = lds.acc[w][part][mine], x1 = lds.acc[w][part + 4][mine];
        float* const v = pair[w >> 1];
        v[0] += __builtin_fmaf(sx * bx, mx, __builtin_fmaf(sx * ax + sy * ay + aq, m0, x0));
        const float x1c =
            __builtin_fmaf(sx * c4 + sy * cy, my, __builtin_fmaf(sy * c4, mx, __builtin_fmaf(sx * sy * cxy + cq, m0, x1)));
        v[1] += part < 2 ? x1c : x1;
        if (part + 8 < NA) v[2] += lds.acc[w][part + 8][mine];
      }
      const float out_o = lds.rec[mine][8];  // (staged, and staged anew, by this wave)
      wave_fence();  // (a slot's four threads are in one wave)
      float* dst = partial + NP * (int64_t)out;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int c = part + 4 * k;
        if (c >= NA) break;
        const float v = pair[0][k] + pair[1][k];
#pragma unroll
        for (int w = 0; w < NW; ++w) lds.acc[w][c][mine] = 0.0f;
        dst[c < 6 ? c : c + 1] = c < 6 ? v * out_o : v;
        if (c == 0) dst[6] = v;
      }
    }
  }
  // instances that no pixel of the tile reached
  for (uint32_t k = b0 + threadIdx.x; k < rg.y; k += 256) {
    float* dst = partial + NP * (int64_t)ival[k];
#pragma unroll
    for (int c = 0; c < NP; ++c) dst[c] = 0.0f;
  }
}

// The first kSegmentWgs workgroups take the segments of the long tiles in
// turn (their number is known on the device only), the others a tile each, in
// the tile order.
constexpr int kSegmentWgs = 4096;
template <int PX, int NP>
__global__ void __launch_bounds__(256 / PX, PX == 1 ? (NP == 10 ? 5 : 4) : 1) k_blend_bwd(const ViewConst* __restrict__ vp,
                                                        const uint32_t* __restrict__ ival,
                                                        const uint2* __restrict__ info_k,
                                                        const Splat* __restrict__ splats, const FrameCounters* ctr,
                                                        const float* __restrict__ rgb, const float* __restrict__ dL,
                                                        const uint32_t* __restrict__ event,
                                                        const uint4* __restrict__ tile_order,
                                                        const uint4* __restrict__ seg_list,
                                                        const float4* __restrict__ ckpt, float* __restrict__ partial) {
  __shared__ std::conditional_t<PX == 1, BlocksBwdLds<NP>, BlendBwdLds<PX, NP>> lds;
  const bool segments = blockIdx.x < kSegmentWgs;
  const int end = segments ? ctr->n_seg : (int)gridDim.x - kSegmentWgs;
  const uint32_t nr = (uint32_t)ctr->n_render;
  for (int i = segments ? (int)blockIdx.x : (int)blockIdx.x - kSegmentWgs; i < end; i += kSegmentWgs) {
    const uint4 o = segments ? seg_list[i] : tile_order[i];
    const uint2 rg = segments ? make_uint2(o.z, o.w) : make_uint2(o.y, o.z);
    if (!segments && (rg.y - rg.x > (uint32_t)kSegment || rg.x == rg.y)) return;
    if constexpr (PX == 1)
      blend_bwd_blocks<NP>(*vp, (int)o.x, o.y, rg, ival, info_k, splats, nr, rgb, dL, event, ckpt, partial, lds);
    else
      blend_bwd_range<PX, NP>(*vp, (int)o.x, o.y, rg, ival, info_k, splats, nr, rgb, dL, event, ckpt, partial, lds);
    if (!segments) return;
    __syncthreads();
  }
}

// Zeroes the per-selection gradient rows of the selected splats that were not
// drawn (the others' rows are written whole by the colour and projection
// backward): 16 lanes take a row.
template <int NC>
__device__ __forceinline__ void zero_undrawn(const FrameCounters* ctr, const uint32_t* __restrict__ tiles,
                                             const lodgs_grads& sel, int64_t group, int64_t groups) {
  const int64_t n = ctr->n_render;
  const int l = threadIdx.x & 15;
  float* const arr = l < 3 ? sel.d_means : (l < 6 ? sel.d_log_scales : (l < 10 ? sel.d_quats : sel.d_opacity_logits));
  const int w = l < 6 ? 3 : (l < 10 ? 4 : 1), c = l < 3 ? l : (l < 6 ? l - 3 : (l < 10 ? l - 6 : 0));
  for (int64_t i = group; i < n; i += groups) {
    if (tiles[i] != 0u) continue;
    if (arr && l < 11) arr[w * i + c] = 0.0f;
    if (!sel.d_sh) continue;
    if (NC % 4 == 0) {
      if (l < NC / 4) reinterpret_cast<float4*>(sel.d_sh + NC * i)[l] = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
      for (int k = l; k < NC; k += 16) sel.d_sh[NC * i + k] = 0.0f;
    }
  }
}

// Every real SH basis function of degree <= 3 is C L Q with a linear
// monomial L = lx x + ly y + lz z + l1 (one coefficient set) and a quadratic
// form Q = a xx + b yy + g zz + d xy + e yz + f xz + h; row k holds
// (C, lx, ly, lz, l1, a, b, g, d, e, f, h) for basis function k (the same
// functions as sh_basis), so any basis function is evaluated without
// branches.
__constant__ float kShFactors[16][12] = {
    {kSH0, 0, 0, 0, 1, 0, 0, 0, 0, 0, 0, 1},
    {-kSH1, 0, 1, 0, 0, 0, 0, 0, 0, 0, 0, 1},
    {kSH1, 0, 0, 1, 0, 0, 0, 0, 0, 0, 0, 1},
    {-kSH1, 1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 1},
    {kSH2_0, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0},
    {kSH2_1, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0, 0},
    {kSH2_2, 0, 0, 0, 1, -1, -1, 2, 0, 0, 0, 0},
    {kSH2_3, 0, 0, 0, 1, 0, 0, 0, 0, 0, 1, 0},
    {kSH2_4, 0, 0, 0, 1, 1, -1, 0, 0, 0, 0, 0},
    {kSH3_0, 0, 1, 0, 0, 3, -1, 0, 0, 0, 0, 0},
    {kSH3_1, 0, 0, 1, 0, 0, 0, 0, 1, 0, 0, 0},
    {kSH3_2, 0, 1, 0, 0, -1, -1, 4, 0, 0, 0, 0},
    {kSH3_3, 0, 0, 1, 0, -3, -3, 2, 0, 0, 0, 0},
    {kSH3_4, 1, 0, 0, 0, -1, -1, 4, 0, 0, 0, 0},
    {kSH3_5, 0, 0, 1, 0, 1, -1, 0, 0, 0, 0, 0},
    {kSH3_6, 1, 0, 0, 0, 1, -3, 0, 0, 0, 0, 0},
};

// Real SH basis function k at the unit direction (x, y, z).
__device__ __forceinline__ float sh_basis_value(int k, float x, float y, float z) {
  const float* t = kShFactors[k];
  const float L = __builtin_fmaf(t[1], x, __builtin_fmaf(t[2], y, __builtin_fmaf(t[3], z, t[4])));
  float Q = t[11];
  Q = __builtin_fmaf(t[5] * x, x, Q);
  Q = __builtin_fmaf(t[6] * y, y, Q);
  Q = __builtin_fmaf(t[7] * z, z, Q);
  Q = __builtin_fmaf(t[8] * x, y, Q);
  Q = __builtin_fmaf(t[9] * y, z, Q);
  Q = __builtin_fmaf(t[10] * x, z, Q);
  return t[0] * L * Q;
}

// One instance's partial (moments about its tile's centre, dL/do, colour
// gradient) as the splat's 2D sums in FP64: with D = c_t - mean,
//   sum w d = m1 + D m0,  sum w d d^T = m2 + D m1^T + m1 D^T + D D^T m0,
// added into g = [sum w dx, sum w dy, sum w dx^2, sum w dx dy, sum w dy^2,
// dL/do, dL/dr, dL/dg, dL/db, contributing pixels].  l is the instance's index within its splat,
// whose tiles it enumerates row by row over the rectangle q.
template <int NP>
__device__ __forceinline__ void add_instance(double* g, const float* P, uint32_t l, ushort4 q, double mx,
                                             double my) {
  const uint32_t w = (uint32_t)(q.y - q.x);
  const uint32_t tyy = w ? (uint32_t)q.z + l / w : 0u, txx = w ? (uint32_t)q.x + l % w : 0u;
  const double Dx = (double)(16u * txx + 8u) - mx, Dy = (double)(16u * tyy + 8u) - my;
  const double m0 = P[0], m1x = P[1], m1y = P[2];
  g[0] += m1x + Dx * m0;
  g[1] += m1y + Dy * m0;
  g[2] += (double)P[3] + 2.0 * Dx * m1x + Dx * Dx * m0;
  g[3] += (double)P[4] + Dx * m1y + Dy * m1x + Dx * Dy * m0;
  g[4] += (double)P[5] + 2.0 * Dy * m1y + Dy * Dy * m0;
#pragma unroll
  for (int c = 5; c < NP - 1; ++c) g[c] += (double)P[c + 1];
}

__device__ __forceinline__ void splat_mean64(const Splat* splats, int64_t i, double& mx, double& my) {
  const float4 m = *reinterpret_cast<const float4*>(&splats[i].mxh);  // mxh, mxl, myh, myl
  mx = (double)m.x + (double)m.y;
  my = (double)m.z + (double)m.w;
}

// The sum of x over the wave's lanes, in every lane (a fixed order).
__device__ __forceinline__ double wave_sum64(double x) {
  const auto halves = [](double v, uint32_t& lo, uint32_t& hi) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    lo = (uint32_t)u;
    hi = (uint32_t)(u >> 32);
  };
  const auto join = [](uint32_t lo, uint32_t hi) { return __longlong_as_double((long long)((uint64_t)hi << 32 | lo)); };
  uint32_t lo, hi;
#define LODGS_DPP_ADD(ctrl)                                                                                    \
  halves(x, lo, hi);                                                                                           \
  x += join((uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, ctrl, 0xf, 0xf, true),                           \
            (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, ctrl, 0xf, 0xf, true))
  LODGS_DPP_ADD(0xB1);   // quad_perm [1,0,3,2]
  LODGS_DPP_ADD(0x4E);   // quad_perm [2,3,0,1]
  LODGS_DPP_ADD(0x141);  // row_half_mirror
  LODGS_DPP_ADD(0x140);  // row_mirror
#undef LODGS_DPP_ADD
  halves(x, lo, hi);
  const auto l16 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  x = join(l16[0], h16[0]) + join(l16[1], h16[1]);
  halves(x, lo, hi);
  const auto l32 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return join(l32[0], h32[0]) + join(l32[1], h32[1]);
}

// A drawn splat's instances [a, b) in emission order, of which the first is
// number a0, its tile rectangle and its mean.
struct SplatRun {
  uint32_t a, b, a0;
  ushort4 q;
  double mx, my;
};
__device__ __forceinline__ SplatRun splat_run(const FrameCounters* ctr, const uint32_t* inst_off, const Splat* splats,
                                              const ushort4* rect, int64_t r, int64_t i) {
  const uint32_t n_cl = (uint32_t)ctr->n_inst_clamped;
  SplatRun s;
  s.a0 = inst_off[r];
  s.a = min(s.a0, n_cl);
  s.b = min(r + 1 < ctr->n_drawn ? inst_off[r + 1] : (uint32_t)ctr->n_instances, n_cl);
  s.q = rect[i];
  splat_mean64(splats, i, s.mx, s.my);
  return s;
}

// Adds the run's instances from `first` on, every `stride`-th, U loads at a
// time.
template <int NP, int U>
__device__ __forceinline__ void add_run(double* g, const SplatRun& s, const float* __restrict__ partial, uint32_t first,
                                        uint32_t stride) {
  for (uint32_t q0 = s.a + first; q0 < s.b; q0 += U * stride) {  // (below 2^31 + 2^13)
    float t[U][NP];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k = q0 + u * stride;
#pragma unroll
      for (int c = 0; c < NP; ++c) t[u][c] = k < s.b ? partial[NP * (int64_t)k + c] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k = q0 + u * stride;
      if (k < s.b) add_instance<NP>(g, t[u], k - s.a0, s.q, s.mx, s.my);
    }
  }
}

// Every drawn splat's 2D sums from its instance partials (add_instance), into
// grad2d at its rank among the drawn splats (zero for a splat that an instance
// overflow left without instances), and its contributing pixels into contrib.
// FP64 sums in orders that depend on the instance counts alone, so
// deterministic.  By instances:
//   up to kLongSegment     one thread, in selection order, so neighbouring
//                          threads read neighbouring partials;
//   up to kWaveSums        a wave (these and the longer ones from the list that
//                          the duplication kernel made of the splats with more
//                          than kLongSegment tiles whose first instance was
//                          emitted);
//   more                   a workgroup.
// The first kLongWgs workgroups take the list, the others the other splats, at
// the same time: the loops over one splat's instances are chains of loads.
// In two launches, with 256 threads for every longer splat, against this, us:
// 53 / 24 for a 1080p iteration (splats of up to 8160 instances), 90 / 52 for
// a street view, 86 / 29 a view of a batch, 13 / 8 at 333 x 171.  Several loads
// at a time in the one-thread loops (25 / 50 / 63 us for one, two, four), or
// the wave on what has more than 8 or 12 instances, cost more than they hide.
constexpr int kSumThreads = 512, kLongWgs = 512, kWaveSums = 1024;
template <int NP>
__global__ void __launch_bounds__(kSumThreads) k_splat_sums(const FrameCounters* ctr, const uint32_t* long_list,
                                                            const uint32_t* list, const uint32_t* inst_off,
                                                            const float* __restrict__ partial,
                                                            const Splat* __restrict__ splats, const ushort4* rect,
                                                            double* grad2d, int32_t* contrib) {
  constexpr int kWaves = kSumThreads / 64;
  __shared__ double part[kWaves][10];
  __shared__ uint32_t giant[kWaves];  // per wave: the splat it leaves to the workgroup
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (blockIdx.x < kLongWgs) {
    const int64_t nl = ctr->n_long;
    for (int64_t l0 = blockIdx.x; l0 < nl; l0 += (int64_t)kLongWgs * kWaves) {  // block-uniform
      const int64_t li = l0 + (int64_t)wv * kLongWgs;
      uint32_t left = 0xFFFFFFFFu;
      if (li < nl) {  // wave-uniform
        const int64_t r = long_list[li], i = list[r];
        const SplatRun s = splat_run(ctr, inst_off, splats, rect, r, i);
        if (s.b - s.a > (uint32_t)kWaveSums) {
          left = (uint32_t)r;
        } else {
          double g[10] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
          add_run<NP, 2>(g, s, partial, lane, 64);
#pragma unroll
          for (int c = 0; c < NP - 1; ++c) g[c] = wave_sum64(g[c]);
          if (lane == 0) {
#pragma unroll
            for (int c = 0; c < 9; ++c) grad2d[9 * r + c] = g[c];
            if (NP == 11) contrib[i] = (int32_t)g[9];  // a count, exact in FP64
          }
        }
      }
      if (lane == 0) giant[wv] = left;
      __syncthreads();
      for (int w = 0; w < kWaves; ++w) {
        if (giant[w] == 0xFFFFFFFFu) continue;  // block-uniform
        const int64_t r = giant[w], i = list[r];
        const SplatRun s = splat_run(ctr, inst_off, splats, rect, r, i);
        double g[10] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        add_run<NP, 2>(g, s, partial, threadIdx.x, kSumThreads);
#pragma unroll
        for (int c = 0; c < NP - 1; ++c) {
          g[c] = wave_sum64(g[c]);
          if (lane == 0) part[wv][c] = g[c];
        }
        __syncthreads();
        if (threadIdx.x < NP - 1) {
          double sum = part[0][threadIdx.x];
#pragma unroll
          for (int v = 1; v < kWaves; ++v) sum += part[v][threadIdx.x];
          if (threadIdx.x < 9) grad2d[9 * r + threadIdx.x] = sum;
          else contrib[i] = (int32_t)sum;
        }
        __syncthreads();
      }
      __syncthreads();
    }
    return;
  }
  const int64_t n = ctr->n_drawn;
  const int64_t r0 = (int64_t)(blockIdx.x - kLongWgs) * kSumThreads + wv * 64;
  const int64_t step = (int64_t)(gridDim.x - kLongWgs) * kSumThreads;
  for (int64_t rw = r0; rw < n; rw += step) {  // wave-uniform
    const int64_t r = rw + lane;
    const bool in = r < n;
    const int64_t i = in ? list[r] : 0;
    SplatRun s = {0, 0, 0, make_ushort4(0, 0, 0, 0), 0.0, 0.0};
    if (in) s = splat_run(ctr, inst_off, splats, rect, r, i);
    const bool listed = (uint32_t)(s.q.y - s.q.x) * (uint32_t)(s.q.w - s.q.z) > kLongSegment &&
                        s.a0 < (uint32_t)ctr->n_inst_clamped;
    double g[10] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (in && !listed) add_run<NP, 1>(g, s, partial, 0, 1);
    if (in && !listed) {
      double* dst = grad2d + 9 * r;
#pragma unroll
      for (int c = 0; c < 9; ++c) dst[c] = g[c];
      if (NP == 11) contrib[i] = (int32_t)g[9];
    }
  }
}

// Per drawn splat, 16 lanes, in selection order (ascending node index, so
// neighbouring groups read neighbouring nodes): the colour backward.  dL/dRGB
// (the splat's colour sums in grad2d; zero for a channel the forward clamped
// at 0, a decision the forward recorded) goes to the SH coefficients, lane k
// taking basis function k (contiguous reads and writes of the 192-byte
// coefficient block), and, through the forward's d colour / d direction, to
// the view direction; dL/dmean through the view direction then replaces the
// colour sums in grad2d.  The forward's per-splat record holds the view
// direction, 1 / distance and the clamp bits, so no node parameter but the
// coefficients is read.
// With per-selection rows, kZeroWgs further workgroups clear the rows of the
// splats that were not drawn (a launch of its own that cleared all rows took
// 8.8 us for a 1080p iteration and 4.9 at 333 x 171; with it here the kernel
// takes 16.8 and 6.4, without 9.9 and 4.9).
constexpr uint32_t kColorBwdWgs = 16384, kZeroWgs = 2048;
template <int DEG>
__global__ void __launch_bounds__(kBlock) k_color_bwd(const int32_t* idx, const FrameCounters* ctr,
                                                      const uint32_t* drawn_list, const float* __restrict__ dcol,
                                                      double* grad2d, lodgs_grads sel, float* node_sh,
                                                      const uint32_t* __restrict__ tiles) {
  constexpr int nb = (DEG + 1) * (DEG + 1), nc = 3 * nb;
  if (blockIdx.x >= kColorBwdWgs) {  // block-uniform
    zero_undrawn<nc>(ctr, tiles, sel, (int64_t)(blockIdx.x - kColorBwdWgs) * (kBlock / 16) + (threadIdx.x >> 4),
                     (int64_t)(gridDim.x - kColorBwdWgs) * (kBlock / 16));
    return;
  }
  float* const sel_sh = sel.d_sh;
  const int64_t n = ctr->n_drawn;
  const int lane = threadIdx.x & 63, sub = lane & 15;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t waves = ((int64_t)kColorBwdWgs * blockDim.x) >> 6;
  for (int64_t g0 = wave * 4; g0 < n; g0 += waves * 4) {  // wave-uniform
    const int64_t dr = g0 + (lane >> 4);  // drawn rank
    if (dr >= n) continue;
    const int64_t i = drawn_list[dr];
    float gc[3], acc3[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 3; ++c) gc[c] = (float)grad2d[9 * dr + 6 + c];
    const float4* rec = reinterpret_cast<const float4*>(dcol + kColorRec * i);
    const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2], r3 = rec[3];
    const float J[9] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w, r2.x};
    const float d0 = r2.y, d1 = r2.z, d2 = r2.w, il = r3.x;
    const uint32_t clamp = __float_as_uint(r3.y);
    const int64_t node = idx[i];
    // rows of 12 or 48 floats (degree 1 or 3) move as float4s: lane q takes
    // floats 4q .. 4q + 3 of the row, coefficient f / 3 and channel f % 3 of
    // float f; other degrees move one coefficient (3 floats) per lane
    constexpr bool kVec = nc % 4 == 0;
    constexpr int nq = nc / 4;
    float4 acc4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (kVec) {
      if (node_sh && sub < nq) acc4 = *reinterpret_cast<const float4*>(node_sh + (int64_t)nc * node + 4 * sub);
    } else if (node_sh && sub < nb) {
#pragma unroll
      for (int c = 0; c < 3; ++c) acc3[c] = node_sh[(int64_t)nc * node + 3 * sub + c];
    }
    // gradient values only: FP32 throughout
    const float dRGB[3] = {(clamp & 1u) ? 0.0f : gc[0], (clamp & 2u) ? 0.0f : gc[1], (clamp & 4u) ? 0.0f : gc[2]};
    const float Yk = sub < nb ? sh_basis_value(sub, d0, d1, d2) : 0.0f;
    if (kVec) {
      float gk[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {  // every lane of the row takes part in the shuffles
        const int f = 4 * sub + t;
        const int k = f / 3 < nb ? f / 3 : nb - 1, c = f - 3 * (f / 3);
        const float Yf = __shfl(Yk, (lane & ~15) + k, 64);
        gk[t] = (c == 0 ? dRGB[0] : (c == 1 ? dRGB[1] : dRGB[2])) * Yf;
      }
      if (sub < nq) {
        if (sel_sh)
          *reinterpret_cast<float4*>(sel_sh + (int64_t)nc * i + 4 * sub) = make_float4(gk[0], gk[1], gk[2], gk[3]);
        if (node_sh)
          *reinterpret_cast<float4*>(node_sh + (int64_t)nc * node + 4 * sub) =
              make_float4(acc4.x + gk[0], acc4.y + gk[1], acc4.z + gk[2], acc4.w + gk[3]);
      }
    } else if (sub < nb) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float gk = dRGB[c] * Yk;
        if (sel_sh) sel_sh[(int64_t)nc * i + 3 * sub + c] = gk;
        if (node_sh) node_sh[(int64_t)nc * node + 3 * sub + c] = acc3[c] + gk;
      }
    }
    if (sub == 0) {  // dL/ddir, projected onto the sphere's tangent plane, / |mu - pos|
      float dd[3];
#pragma unroll
      for (int a = 0; a < 3; ++a)
        dd[a] = __builtin_fmaf(dRGB[2], J[6 + a], __builtin_fmaf(dRGB[1], J[3 + a], dRGB[0] * J[a]));
      const float dot = __builtin_fmaf(dd[0], d0, __builtin_fmaf(dd[1], d1, dd[2] * d2));
      grad2d[9 * dr + 6] = (double)((dd[0] - d0 * dot) * il);
      grad2d[9 * dr + 7] = (double)((dd[1] - d1 * dot) * il);
      grad2d[9 * dr + 8] = (double)((dd[2] - d2 * dot) * il);
    }
  }
}

// One thread per drawn splat, in selection order (ascending node index, so
// neighbouring lanes touch neighbouring nodes): drawn_list[0 .. n_drawn)
// lists exactly the drawn splats.  The FP64 geometry chain is replayed and
// the 2D gradients of grad2d[r] are carried to the mean, scales, rotation and
// opacity logit; grad2d[r][6..8] already holds dL/dmean through the view
// direction.
// Projection backward, FP64 (per splat): the forward chain is replayed and the
// 2D gradients (mean2D, conic, opacity, colour) are carried to the raw
// parameters.
template <int DEG>
__global__ void __launch_bounds__(kBlock) k_project_bwd(SceneDev S, const ViewConst* __restrict__ vp, const int32_t* idx,
                                                        const FrameCounters* ctr, const uint32_t* drawn_list,
                                                        const double* grad2d, lodgs_grads sel, lodgs_grads nodes,
                                                        float* max_grad2d, ContribStats cs) {
  const int32_t iter = cs.last ? *cs.iteration : 0;
  const ViewConst v = *vp;
  const int64_t n = ctr->n_drawn;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = drawn_list[r];
    const int64_t node = idx[i];
    if (cs.last) {  // pruning statistics: a drawn node is one splat of its view (no races)
      const int32_t c = cs.contrib[i];
      if (c > 0) {
        cs.last[node] = iter;
        if (cs.count) cs.count[node] += c;
      }
    }
    double g2[9];  // 2D sums of the splat, see add_instance
#pragma unroll
    for (int c = 0; c < 9; ++c) g2[c] = grad2d[9 * r + c];
    const double gdir[3] = {g2[6], g2[7], g2[8]};
    double gm[3] = {0, 0, 0}, gls[3] = {0, 0, 0}, gq[4] = {0, 0, 0, 0}, go = 0.0;
    Proj64 P;
    const bool visible = proj_chain64(S.means, S.log_scales, S.quats, v, node, P);
    if (visible) {
      // opacity
      const double o = 1.0 / (1.0 + (double)fexp(-S.opacity_logits[node]));
      go = g2[5] * o * (1.0 - o);
      // d power / d mean2D = Q d, d power / d conic = -(dx^2 / 2, dx dy, dy^2 / 2)
      const double ca = P.C / P.det, cb = -P.B / P.det, cc = P.A / P.det;
      const double gmx = ca * g2[0] + cb * g2[1], gmy = cb * g2[0] + cc * g2[1];
      // the densification statistic: the largest screen-space mean gradient
      // over views (a drawn node is one splat of its view: no races)
      if (max_grad2d) max_grad2d[node] = fmaxf(max_grad2d[node], (float)__builtin_sqrt(gmx * gmx + gmy * gmy));
      // conic -> projected covariance: GS = -Q GQ Q
      const double gq00 = -0.5 * g2[2], gq01 = -0.5 * g2[3], gq11 = -0.5 * g2[4];
      const double qg00 = ca * gq00 + cb * gq01, qg01 = ca * gq01 + cb * gq11;
      const double qg10 = cb * gq00 + cc * gq01, qg11 = cb * gq01 + cc * gq11;
      const double GS00 = -(qg00 * ca + qg01 * cb), GS01 = -(qg00 * cb + qg01 * cc);
      const double GS11 = -(qg10 * cb + qg11 * cc);
      // Sigma' = T Sigma T^T: dL/dT = 2 GS T Sigma, dL/dSigma = T^T GS T
      const double* Tm = P.T;
      const double* Sg = P.Sg;
      double TS[6];
      for (int r = 0; r < 2; ++r) {
        TS[3 * r + 0] = Tm[3 * r] * Sg[0] + Tm[3 * r + 1] * Sg[1] + Tm[3 * r + 2] * Sg[2];
        TS[3 * r + 1] = Tm[3 * r] * Sg[1] + Tm[3 * r + 1] * Sg[3] + Tm[3 * r + 2] * Sg[4];
        TS[3 * r + 2] = Tm[3 * r] * Sg[2] + Tm[3 * r + 1] * Sg[4] + Tm[3 * r + 2] * Sg[5];
      }
      double dT[6];
      for (int c = 0; c < 3; ++c) {
        dT[c] = 2.0 * (GS00 * TS[c] + GS01 * TS[3 + c]);
        dT[3 + c] = 2.0 * (GS01 * TS[c] + GS11 * TS[3 + c]);
      }
      double dS[9];
      for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
          dS[3 * a + b] = Tm[a] * (GS00 * Tm[b] + GS01 * Tm[3 + b]) + Tm[3 + a] * (GS01 * Tm[b] + GS11 * Tm[3 + b]);
      // T = J W
      double dJ00 = 0, dJ02 = 0, dJ11 = 0, dJ12 = 0;
      for (int c = 0; c < 3; ++c) {
        dJ00 += dT[c] * (double)v.R[c];
        dJ02 += dT[c] * (double)v.R[6 + c];
        dJ11 += dT[3 + c] * (double)v.R[3 + c];
        dJ12 += dT[3 + c] * (double)v.R[6 + c];
      }
      const double cx = P.c[0], cy = P.c[1], cz = P.c[2];
      const double fx = v.fx, fy = v.fy;
      const double iz = 1.0 / cz, iz2 = iz * iz, iz3 = iz2 * iz;
      const double dcx = dJ02 * (-fx * iz2) + gmx * fx * iz;
      const double dcy = dJ12 * (-fy * iz2) + gmy * fy * iz;
      const double dcz = dJ00 * (-fx * iz2) + dJ02 * (2.0 * fx * cx * iz3) + dJ11 * (-fy * iz2) +
                         dJ12 * (2.0 * fy * cy * iz3) + gmx * (-fx * cx * iz2) + gmy * (-fy * cy * iz2);
      for (int a = 0; a < 3; ++a)
        gm[a] = (double)v.R[a] * dcx + (double)v.R[3 + a] * dcy + (double)v.R[6 + a] * dcz + gdir[a];
      // Sigma = M M^T, M = Rq diag(s)
      double dRq[9];
      for (int c = 0; c < 3; ++c) {
        double ds = 0.0;
        for (int r = 0; r < 3; ++r) {
          const double dm = 2.0 * (dS[3 * r] * P.M[c] + dS[3 * r + 1] * P.M[3 + c] + dS[3 * r + 2] * P.M[6 + c]);
          ds += dm * P.Rq[3 * r + c];
          dRq[3 * r + c] = dm * P.s[c];
        }
        gls[c] = ds * P.s[c];
      }
      const double w = P.qn[0], x = P.qn[1], y = P.qn[2], z = P.qn[3];
      double dq[4];
      dq[0] = 2.0 * (-z * dRq[1] + y * dRq[2] + z * dRq[3] - x * dRq[5] - y * dRq[6] + x * dRq[7]);
      dq[1] = 2.0 * (y * dRq[1] + z * dRq[2] + y * dRq[3] - 2.0 * x * dRq[4] - w * dRq[5] + z * dRq[6] +
                     w * dRq[7] - 2.0 * x * dRq[8]);
      dq[2] = 2.0 * (-2.0 * y * dRq[0] + x * dRq[1] + w * dRq[2] + x * dRq[3] + z * dRq[5] - w * dRq[6] +
                     z * dRq[7] - 2.0 * y * dRq[8]);
      dq[3] = 2.0 * (-2.0 * z * dRq[0] - w * dRq[1] + x * dRq[2] + w * dRq[3] - 2.0 * z * dRq[4] + y * dRq[5] +
                     x * dRq[6] + y * dRq[7]);
      const double qd = dq[0] * w + dq[1] * x + dq[2] * y + dq[3] * z;
      for (int k = 0; k < 4; ++k) gq[k] = (dq[k] - P.qn[k] * qd) / P.ql;
    }
    if (sel.d_means) for (int k = 0; k < 3; ++k) sel.d_means[3 * i + k] = (float)gm[k];
    if (sel.d_log_scales) for (int k = 0; k < 3; ++k) sel.d_log_scales[3 * i + k] = (float)gls[k];
    if (sel.d_quats) for (int k = 0; k < 4; ++k) sel.d_quats[4 * i + k] = (float)gq[k];
    if (sel.d_opacity_logits) sel.d_opacity_logits[i] = (float)go;
    if (!visible) continue;
    if (nodes.d_means) for (int k = 0; k < 3; ++k) nodes.d_means[3 * node + k] += (float)gm[k];
    if (nodes.d_log_scales) for (int k = 0; k < 3; ++k) nodes.d_log_scales[3 * node + k] += (float)gls[k];
    if (nodes.d_quats) for (int k = 0; k < 4; ++k) nodes.d_quats[4 * node + k] += (float)gq[k];
    if (nodes.d_opacity_logits) nodes.d_opacity_logits[node] += (float)go;
  }
}

// The per-splat 2D sums of the instance partials (frame-local outputs).
template <int NP>
static void launch_splat_sums(lodgs_frame* f, hipStream_t st) {
  // up to half a million threads for the splats that take one each
  const int64_t wgs = std::min<int64_t>((f->caps.max_selected + kSumThreads - 1) / kSumThreads, 1024);
  hipLaunchKernelGGL(k_splat_sums<NP>, dim3((uint32_t)(kLongWgs + std::max<int64_t>(wgs, 1))), dim3(kSumThreads), 0, st,
                     f->ctr, f->long_list, f->drawn_list, f->inst_off, f->inst_grad, f->splats, f->rect, f->grad2d,
                     f->contrib);
}

// Colour and projection backward into the gradient arrays (and the node
// statistics).
template <int DEG>
static void launch_scatter_deg(const SceneDev& S, lodgs_frame* f, const lodgs_grads& sel, const lodgs_grads& nodes,
                               bool contrib, hipStream_t st) {
  // 16 lanes per splat: one pass covers 256k drawn splats, so each 16-lane
  // group runs its latency-bound chain of dependent loads once
  const bool rows = sel.d_means || sel.d_log_scales || sel.d_quats || sel.d_opacity_logits || sel.d_sh;
  hipLaunchKernelGGL(k_color_bwd<DEG>, dim3(kColorBwdWgs + (rows ? kZeroWgs : 0)), dim3(kBlock), 0, st, f->r_idx, f->ctr,
                     f->drawn_list, f->dcol, f->grad2d, sel, nodes.d_sh, f->tiles);
  ContribStats cs{f->contrib, nullptr, nullptr, nullptr};
  if (contrib) cs = ContribStats{f->contrib, f->last_contrib, f->contrib_count, f->contrib_iteration};
  hipLaunchKernelGGL(k_project_bwd<DEG>, dim3(1024), dim3(kBlock), 0, st, S, f->d_view_ren, f->r_idx, f->ctr,
                     f->drawn_list, f->grad2d, sel, nodes, f->rows_mode ? (float*)nullptr : f->max_grad2d, cs);
}

template <int NP>
static void launch_blend_bwd_np(lodgs_frame* f, const float* d_dL, hipStream_t st) {
  const ViewConst& v = f->view;
  const int ntiles = v.tiles_x * v.tiles_y;
  switch (f->blend_px_bwd) {
    case 1:
      hipLaunchKernelGGL((k_blend_bwd<1, NP>), dim3(kSegmentWgs + ntiles), dim3(256), 0, st, f->d_view_ren,
                         f->ival, f->info_k, f->splats, f->ctr, f->r_rgb, d_dL, f->inst_event,
                         f->tile_order, f->seg_list, f->ckpt, f->inst_grad);
      break;
    case 4:
      hipLaunchKernelGGL((k_blend_bwd<4, NP>), dim3(kSegmentWgs + ntiles), dim3(64), 0, st, f->d_view_ren,
                         f->ival, f->info_k, f->splats, f->ctr, f->r_rgb, d_dL, f->inst_event,
                         f->tile_order, f->seg_list, f->ckpt, f->inst_grad);
      break;
    default:
      hipLaunchKernelGGL((k_blend_bwd<2, NP>), dim3(kSegmentWgs + ntiles), dim3(128), 0, st, f->d_view_ren,
                         f->ival, f->info_k, f->splats, f->ctr, f->r_rgb, d_dL, f->inst_event,
                         f->tile_order, f->seg_list, f->ckpt, f->inst_grad);
      break;
  }
}

// LODGS_BWD_PARTIALS: the blend backward and the per-splat 2D sums, which
// write only the frame's own state.  The per-instance partials carry the
// contributing-pixel count (11 values) only while the pruning statistic is
// attached (and not in the rows form).  LODGS_BWD_SCATTER: colour and
// projection backward into the gradient arrays and the node statistics; it
// stamps the pruning statistic only after partials that carried the count.
void launch_backward(lodgs_frame* f, const float* d_dL, const lodgs_grads* sel, const lodgs_grads* nodes,
                     uint32_t phases, hipStream_t st) {
  const bool part = (phases & LODGS_BWD_PARTIALS) != 0, scat = (phases & LODGS_BWD_SCATTER) != 0;
  if (part) {
    f->partials_np = (f->last_contrib && !f->rows_mode) ? kPartial : kPartial - 1;
    stage_begin(f, LODGS_STAGE_BLEND_BWD, st);
    if (f->partials_np == kPartial) launch_blend_bwd_np<kPartial>(f, d_dL, st);
    else launch_blend_bwd_np<kPartial - 1>(f, d_dL, st);
    stage_end(f, st);
  }
  if (!part && !scat) return;
  stage_begin(f, LODGS_STAGE_PROJECT_BWD, st);
  if (part) {
    if (f->partials_np == kPartial) launch_splat_sums<kPartial>(f, st);
    else launch_splat_sums<kPartial - 1>(f, st);
  }
  if (scat) {
    const SceneDev& S = render_params(f);
    const bool contrib = f->partials_np == kPartial && f->last_contrib;
    lodgs_grads none{nullptr, nullptr, nullptr, nullptr, nullptr};
    const lodgs_grads gs = sel ? *sel : none, gn = nodes ? *nodes : none;
    switch (S.sh_degree) {
      case 0: launch_scatter_deg<0>(S, f, gs, gn, contrib, st); break;
      case 1: launch_scatter_deg<1>(S, f, gs, gn, contrib, st); break;
      case 2: launch_scatter_deg<2>(S, f, gs, gn, contrib, st); break;
      default: launch_scatter_deg<3>(S, f, gs, gn, contrib, st); break;
    }
  }
  stage_end(f, st);
}

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
  return x;
}

// L1 loss: grad = sign(img - target) / n, loss = sum |img - target| / n.
__global__ void __launch_bounds__(kBlock) k_l1(const float* img, const float* tgt, int64_t n, float* grad,
                                               float* loss) {
  const float inv = 1.0f / (float)n;
  float acc = 0.0f;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float d = img[i] - tgt[i];
    grad[i] = d > 0.0f ? inv : (d < 0.0f ? -inv : 0.0f);
    acc += fabsf(d);
  }
  if (!loss) return;
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) atomicAdd(loss, acc * inv);
}

__global__ void k_zero_one(float* p) { *p = 0.0f; }

int l1_target_arg(const void* func, int* n_args) {
  if (func != reinterpret_cast<const void*>(&k_l1)) return -1;
  *n_args = 5;  // (img, tgt, n, grad, loss)
  return 1;
}

void launch_l1_loss(const float* img, const float* target, int64_t n, float* grad, float* loss, hipStream_t st) {
  if (loss) hipLaunchKernelGGL(k_zero_one, dim3(1), dim3(1), 0, st, loss);
  int64_t g = (n + kBlock - 1) / kBlock;
  g = g > 4096 ? 4096 : g;
  hipLaunchKernelGGL(k_l1, dim3((int)g), dim3(kBlock), 0, st, img, target, n, grad, loss);
}

}  // namespace lodgs
