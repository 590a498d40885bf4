// LoD cut over the flattened HSPT (Sec. 4.3 two-step cut; Sec. 4.1 Eq. 4 and
// Alg. 2 for the SPTs) and order-preserving stream compaction of the result.
//
// Step 0 (k_select_begin): the view constants and the upper nodes' view tests.
// Step 1 (k_cut_upper): one thread per upper node and per SPT root.  A node is
// reached when no upper ancestor "stops" the descent (stops = culled, or fine
// enough at its own distance); the ancestor chain of the balanced upper
// hierarchy is short, so every thread walks it instead of running a
// level-synchronous BFS.  Reached upper nodes that are not culled and fine
// enough are selected; reached SPT roots that are not culled make their SPT
// visible, and a binary search over the SPT's r_max (descending) gives the
// candidate prefix length high_j = #{r_max > X_j}.  X_j is taken at the root's
// distance times the view's LoD noise factor (1 outside noisy training; the
// upper nodes' own distances are never scaled).  The visible prefixes are
// listed in chunks of kChunk candidates.
// Step 2 (k_cut_count): a wave per chunk counts its selected candidates (r_min
// <= X_j).
// Step 3 (k_cut_write): the selected nodes are written in layout order, a wave
// per run of chunks, at the sum of the counts before it.
// Four launches and no workgroup that waits for another (scenes of more than
// kWideTiles tiles: two more, which scan the tiles' counts).  A small view's cut is
// bound by the launches' latency: 18 us on a 32,767-node scene and 36 on 12M
// nodes, street level (nine launches, with two-kernel scans: 31 and 48).  Tiles numbered by ticket that look back over published
// counts took longer than adding the counts up (a contended ticket costs 0.1
// to 0.2 us a tile here), and a wave per SPT left the SPTs of tens of
// thousands of candidates, which city scenes have, to one wave each.
#include "lodgs_internal.h"

namespace lodgs {

// Writes the view constants for the kernels that follow, clears the cut's
// counters, and evaluates per upper node the two view
// tests of the cut: bit 0 = culled (its sphere is outside the frustum, when
// culling), bit 1 = fine enough (r_min <= X at its own distance).  The descent
// stops at a node with either bit; an upper node is selected when it is
// reached, not culled and fine enough.  (A captured graph is replayed for
// another camera by updating v in this node's arguments.)
__global__ void __launch_bounds__(kBlock) k_select_begin(ViewConst v, ViewConst* dst, FrameCounters* ctr, SceneDev S,
                                                         uint32_t flags, uint8_t* utest) {
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  if (t0 == 0) {
    *dst = v;
    ctr->n_chunks = 0;
  }
  const bool cull = (flags & LODGS_CULL) != 0;
  for (int64_t u = t0; u < S.n_upper; u += stride) {
    const float mx = S.means[3 * u], my = S.means[3 * u + 1], mz = S.means[3 * u + 2];
    const bool culled = cull && sphere_culled(v, mx, my, mz, S.rho[u]);
    const bool fine = S.r_min[u] <= view_distance(v, mx, my, mz) * v.k;
    utest[u] = (uint8_t)((culled ? 1u : 0u) | (fine ? 2u : 0u));
  }
}

namespace {

// Longest ancestor chain a walk follows (a malformed parent array with a
// cycle then reads as "not reached" instead of looping).
constexpr int32_t kMaxWalk = 4096;

// Walk up from a (the first upper ancestor, -1 for none): reached iff no
// upper ancestor stops the descent.
__device__ __forceinline__ bool chain_reached(const SceneDev& S, const uint8_t* utest, int32_t a) {
  for (int32_t steps = 0; a >= 0; ++steps) {
    if (steps >= kMaxWalk || a >= S.n_upper) return false;
    if (utest[a]) return false;
    a = S.upper_parent[a];
  }
  return true;
}

// The same from the ancestor table of element e: sixteen ancestors' tests are
// requested together instead of one dependent load per level.
__device__ __forceinline__ bool table_reached(const SceneDev& S, const uint8_t* utest, int64_t e, int64_t total) {
  constexpr int W = 16;
  for (int32_t d0 = 0; d0 < S.anc_depth; d0 += W) {
    int32_t a[W];
#pragma unroll
    for (int k = 0; k < W; ++k) a[k] = d0 + k < S.anc_depth ? S.anc[(int64_t)(d0 + k) * total + e] : -1;
    uint32_t t[W];
#pragma unroll
    for (int k = 0; k < W; ++k) t[k] = utest[a[k] < 0 ? 0 : a[k]];  // node 0 stands in for missing entries
    bool stop = false, end = false;
#pragma unroll
    for (int k = 0; k < W; ++k) {
      end = end || a[k] < 0;
      stop = stop || (!end && t[k] != 0u);
    }
    if (stop) return false;
    if (end) return true;
  }
  return true;
}

// high = #{i < m : r[i] > X} for r descending, by an 8-ary search: each
// round requests 8 evenly spaced samples together and keeps the interval
// between the last sample above X and the first one not above it.
__device__ __forceinline__ int32_t count_above(const float* r, int32_t m, float X) {
  int32_t lo = 0, hi = m;  // the answer lies in [lo, hi]
  while (hi - lo > 8) {
    const int32_t span = hi - lo;
    int32_t p[8];
    float rv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      p[k] = lo + (int32_t)(((int64_t)(k + 1) * span) / 9);
      rv[k] = r[p[k]];
    }
    int32_t c = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) c += rv[k] > X ? 1 : 0;
    const int32_t nlo = c > 0 ? p[c > 0 ? c - 1 : 0] + 1 : lo;
    const int32_t nhi = c < 8 ? p[c < 8 ? c : 7] : hi;
    lo = nlo;
    hi = nhi;
  }
  float rv[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) rv[k] = lo + k < hi ? r[lo + k] : 0.0f;
  int32_t c = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) c += (lo + k < hi && rv[k] > X) ? 1 : 0;
  return lo + c;
}

__device__ __forceinline__ bool reached(const SceneDev& S, const uint8_t* utest, int64_t e, int64_t total,
                                        int32_t first) {
  return S.anc ? table_reached(S, utest, e, total) : chain_reached(S, utest, first);
}

// Ancestor-table construction: chain lengths (the maximum, or kMaxAncDepth + 1
// for a chain that is too long or leaves the upper node range), then the rows.
__global__ void __launch_bounds__(kBlock) k_anc_depth(SceneDev S, int32_t* depth) {
  const int64_t total = (int64_t)S.n_upper + S.n_spt;
  int32_t dmax = 0;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    int32_t a = e < S.n_upper ? S.upper_parent[e] : S.spt_parent[e - S.n_upper];
    int32_t d = 0;
    while (a >= 0 && d <= kMaxAncDepth) {
      if (a >= S.n_upper) {
        d = kMaxAncDepth + 1;
        break;
      }
      ++d;
      a = S.upper_parent[a];
    }
    dmax = d > dmax ? d : dmax;
  }
  if (dmax) atomicMax(depth, dmax);
}

__global__ void __launch_bounds__(kBlock) k_anc_fill(SceneDev S, int32_t D, int32_t* anc) {
  const int64_t total = (int64_t)S.n_upper + S.n_spt;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    int32_t a = e < S.n_upper ? S.upper_parent[e] : S.spt_parent[e - S.n_upper];
    for (int32_t d = 0; d < D; ++d) {
      anc[(int64_t)d * total + e] = a;
      if (a >= 0) a = S.upper_parent[a];
    }
  }
}

// A tile of the cut: kCutTile upper nodes, or kCutTile SPTs (tiles follow the
// layout order: the upper nodes', then the SPTs').  The SPT prefixes' chunks
// hold at most kChunk candidates.
// A chunk is listed as (SPT, index in the SPT << 10 | selected candidates).
constexpr int32_t kChunk = 512;
constexpr uint32_t kChunkCount = 1023u;  // the count's bits
constexpr uint32_t kManyChunks = 1024, kOwnChunks = 8;  // of a tile, of an SPT
constexpr int kChunkGrid = 1024;  // workgroups over the chunks, four waves each
static_assert(kCutTile == kBlock, "one upper node or SPT per thread");

// Per tile: the upper nodes' decisions and their count, or the SPTs' candidate
// prefixes and their chunks, which a tile appends to the list in order (the tiles in any order: first[tile] is where).
__global__ void __launch_bounds__(kBlock) k_cut_upper(SceneDev S, const ViewConst* __restrict__ vp, uint32_t flags,
                                                      const uint8_t* utest, uint8_t* upper_sel, int32_t* spt_high,
                                                      float* spt_X, FrameCounters* ctr, int32_t n_upper_tiles, uint32_t* selected,
                                                      uint4* sums, uint32_t* first, uint2* chunks, CacheDev C) {
  __shared__ uint32_t wt[kBlock / 64];
  __shared__ uint32_t w3[3][kBlock / 64];
  __shared__ uint32_t s_base;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t total = (int64_t)S.n_upper + S.n_spt;
  const int tile = (int)blockIdx.x;
  const bool upper = tile < n_upper_tiles;  // block-uniform
  uint32_t up = 0, vis = 0, c = 0;
  int32_t high = 0, b = 0;
  float X = 0.0f;
  const int64_t j = upper ? (int64_t)tile * kCutTile + t : (int64_t)(tile - n_upper_tiles) * kCutTile + t;
  if (upper) {
    const bool p = j < S.n_upper && utest[j] == 2u && reached(S, utest, j, total, S.upper_parent[j]);
    if (j < S.n_upper) upper_sel[j] = p ? 1 : 0;
    up = p ? 1u : 0u;
  } else if (j < S.n_spt) {
    const ViewConst v = *vp;
    const bool cull = (flags & LODGS_CULL) != 0;
    const bool conservative = (flags & LODGS_CONSERVATIVE) != 0 && S.spt_radius != nullptr;
    uint8_t vst = 0;
    b = S.spt_begin[j];
    const int32_t m = S.spt_begin[j + 1] - b;
    const float mx = S.means[3 * (int64_t)b], my = S.means[3 * (int64_t)b + 1], mz = S.means[3 * (int64_t)b + 2];
    const float rho = S.rho[b];
    if (reached(S, utest, S.n_upper + j, total, S.spt_parent[j]) && !(cull && sphere_culled(v, mx, my, mz, rho))) {
      const float d = view_distance(v, mx, my, mz) * v.spt_scale;  // the LoD noise (1: none)
      X = conservative ? fmaxf(0.0f, d - S.spt_radius[j]) * v.k : d * v.k;
      if (C.cached) {  // the cache's ratio test (squared, FP32)
        vst = 2;
        if (C.cached[j]) {
          const float r = d / C.dc[j];
          const float r2 = r * r;
          if (C.d_min <= r2 && r2 <= C.d_max) {
            X = C.Xc[j];
            vst = 1;
          }
        }
        C.dcur[j] = d;
      }
      high = count_above(S.r_max + b, m, X);
      vis = 1;
    }
    if (C.cached) {
      C.vstate[j] = vst;
      C.spt_sel[j] = 0u;
    }
    spt_high[j] = high;
    spt_X[j] = X;
    c = (uint32_t)((high + kChunk - 1) / kChunk);
  }
  uint32_t tot;
  const uint32_t at = block_exclusive_scan(c, wt, &tot);
  uint32_t r[3] = {up, vis, (uint32_t)high};
#pragma unroll
  for (int d = 32; d > 0; d >>= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) r[k] += __shfl_xor(r[k], d, 64);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 3; ++k) w3[k][wv] = r[k];
  if (t == 0 && tot) s_base = (uint32_t)atomicAdd(&ctr->n_chunks, (int)tot);
  __syncthreads();
  if (t == 0) {
    uint32_t a[3] = {0u, 0u, 0u};
    for (int w = 0; w < kBlock / 64; ++w)
#pragma unroll
      for (int k = 0; k < 3; ++k) a[k] += w3[k][w];
    selected[tile] = a[0];  // an SPT tile's count comes with its chunks
    sums[tile] = make_uint4(a[0], a[1], a[2], 0u);
    if (!upper) first[tile] = tot ? s_base : 0u;
  }
  if (tot) {
    const uint32_t base = s_base + at;
    const bool many = tot > kManyChunks;  // block-uniform
    if (!many || c <= kOwnChunks) {
      for (uint32_t q = 0; q < c; ++q) chunks[base + q] = make_uint2((uint32_t)j, q << 10);
    }
    if (many) {  // the long ones' by their waves
      for (uint64_t more = __ballot(c > kOwnChunks); more; more &= more - 1) {  // wave-uniform
        const int l = __builtin_ctzll(more);
        const uint32_t to = __shfl(base, l, 64), n = __shfl(c, l, 64), own = __shfl((uint32_t)j, l, 64);
        for (uint32_t q = lane; q < n; q += 64) chunks[to + q] = make_uint2(own, q << 10);
      }
    }
  }
}

// What the waves need of the chunks of a run: a lane holds one of up to 64.
struct LaneChunk {
  uint32_t word;           // as listed
  int32_t node, spt, end;  // first candidate, SPT, end of the SPT's prefix
  float X;
};

// A chunk's first candidate, from its SPT's first node.
__device__ __forceinline__ int32_t chunk_node(int32_t begin, uint32_t word) {
  return begin + (int32_t)(word >> 10) * kChunk;
}

__device__ __forceinline__ LaneChunk load_chunk(const SceneDev& S, const int32_t* __restrict__ spt_high,
                                                const float* __restrict__ spt_X, const uint2* chunks, int g0, int m) {
  const auto load = [&](int c) -> LaneChunk {
    const uint2 ch = chunks[c];
    const int32_t b = S.spt_begin[ch.x];
    return {ch.y, chunk_node(b, ch.y), (int32_t)ch.x, b + spt_high[ch.x], spt_X[ch.x]};
  };
  if (m == 1) return load(g0);  // (by scalar loads, which take less time)
  return load(min(g0 + (int)(threadIdx.x & 63), g0 + m - 1));
}

__device__ __forceinline__ int32_t lane_value(int32_t x, int l) { return __builtin_amdgcn_readlane(x, l); }

// This lane's candidates of a chunk: the q-th one is the chunk's first + 64 q +
// lane.  They are requested together; the selected ones are the bits of
// selected().
struct ChunkNodes {
  int32_t node, end;
  float X, r_min[kChunk / 64];
  __device__ __forceinline__ ChunkNodes(const SceneDev& S, int32_t first, int32_t end_, float X_)
      : node(first + (int32_t)(threadIdx.x & 63)), end(end_), X(X_) {
#pragma unroll
    for (int q = 0; q < kChunk / 64; ++q) r_min[q] = node + 64 * q < end ? S.r_min[(int64_t)node + 64 * q] : 0.0f;
  }
  __device__ __forceinline__ ChunkNodes(const SceneDev& S, const LaneChunk& c, int l)
      : ChunkNodes(S, lane_value(c.node, l), lane_value(c.end, l),
                   __int_as_float(lane_value(__float_as_int(c.X), l))) {}
  __device__ __forceinline__ uint32_t selected() const {
    uint32_t bits = 0u;
#pragma unroll
    for (int q = 0; q < kChunk / 64; ++q) bits |= node + 64 * q < end && r_min[q] <= X ? 1u << q : 0u;
    return bits;
  }
};

__device__ __forceinline__ uint32_t wave_total(uint32_t x) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
  return x;
}

// The chunks' selected candidates, and their sums by run, by tile (and, for
// the cut cache, by SPT).  The list is cut in kCutRuns runs, a wave each; a
// workgroup adds its runs' sum over a tile with one atomic: one per chunk made
// the few visible tiles' words the bound (54 us for a 12M-node street view).
constexpr int kCountThreads = 1024, kCountWaves = kCountThreads / 64, kCountGrid = 256;
static_assert(kCountGrid * kCountWaves == kCutRuns && kChunkGrid * (kBlock / 64) == kCutRuns, "a wave per run");
__device__ __forceinline__ int run_length(int n) { return (n + kCutRuns - 1) / kCutRuns; }

__global__ void __launch_bounds__(kCountThreads) k_cut_count(SceneDev S, const FrameCounters* ctr,
                                                             const int32_t* __restrict__ spt_high,
                                                             const float* __restrict__ spt_X,
                                                             uint2* chunks, int32_t n_upper_tiles, uint32_t* selected,
                                                             uint32_t* runs, uint32_t* spt_sel) {
  __shared__ int32_t w_tile[kCountWaves];   // the wave's last tile (-1: none) ...
  __shared__ uint32_t w_sum[kCountWaves];   // ... and what it has not yet added to it
  const int n = ctr->n_chunks, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int per = run_length(n), run = (int)blockIdx.x * kCountWaves + __builtin_amdgcn_readfirstlane(wv);
  const int c0 = run * per, c1 = min(c0 + per, n);
  if ((int)blockIdx.x * kCountWaves * per >= n) return;  // block-uniform
  int32_t tile = -1;
  uint32_t sum = 0, all = 0;
  for (int g0 = c0; g0 < c1; g0 += 64) {  // wave-uniform
    const int m = min(64, c1 - g0);
    const LaneChunk ch = load_chunk(S, spt_high, spt_X, chunks, g0, m);
    uint32_t mine = 0;
    for (int l = 0; l < m; ++l) {
      const uint32_t bits = ChunkNodes(S, ch, l).selected();
      uint32_t k = 0;
#pragma unroll
      for (int q = 0; q < kChunk / 64; ++q) k += (uint32_t)__popcll(__ballot((bits >> q) & 1u));
      const int32_t own = n_upper_tiles + lane_value(ch.spt, l) / kCutTile;
      if (own != tile && sum != 0u) {
        if (lane == 0) atomicAdd(&selected[tile], sum);
        sum = 0;
      }
      tile = own;
      sum += k;
      all += k;
      mine = lane == l ? k : mine;
    }
    if (lane < m) {
      chunks[g0 + lane].y = ch.word | mine;  // at most kChunk
      if (spt_sel && mine) atomicAdd(&spt_sel[ch.spt], mine);
    }
  }
  if (lane == 0) {
    runs[run] = all;
    w_tile[wv] = tile;
    w_sum[wv] = sum;
  }
  __syncthreads();
  // the first wave of a tile adds the sums of all waves that ended in it
  if (threadIdx.x < kCountWaves && w_tile[threadIdx.x] >= 0) {
    const int32_t mine = w_tile[threadIdx.x];
    uint32_t sums = 0;
    bool lead = true;
    for (int w = 0; w < kCountWaves; ++w) {
      if (w_tile[w] == mine) {
        lead = lead && w >= (int)threadIdx.x;
        sums += w_sum[w];
      }
    }
    if (lead && sums) atomicAdd(&selected[mine], sums);
  }
}

// The first n_upper_tiles workgroups write their tile's selected upper nodes,
// the others take the runs of chunks, a wave each: a tile's place is the sum
// of the counts of the tiles before it, a chunk's that of its tile and of the
// chunks before it there (whole runs by their sums), and is carried on to the
// run's next chunks of that tile.  The last workgroup publishes the totals.
// Up to kWideTiles tiles a wave adds up the tiles before its own itself (at
// most 16 loads a lane); beyond, `place` holds those sums, made by a scan.
// When all waves added up all tiles and every chunk its tile's earlier chunks,
// the cut grew with the square of the scene.  Before / now, whole cuts, us:
// one-node SPTs of 100K leaves 111 / 69, 400K 515 / 233, 1.6M 3225 / 700; one
// SPT of 1.6M leaves 232 / 45.
__global__ void __launch_bounds__(kBlock) k_cut_write(SceneDev S, const uint8_t* __restrict__ upper_sel,
                                                      int32_t n_upper_tiles, int32_t ntiles,
                                                      const uint32_t* __restrict__ selected,
                                                      const uint32_t* __restrict__ place,
                                                      const uint4* __restrict__ sums,
                                                      const uint32_t* __restrict__ first,
                                                      const int32_t* __restrict__ spt_high,
                                                      const float* __restrict__ spt_X,
                                                      const uint2* __restrict__ chunks,
                                                      const uint32_t* __restrict__ runs, int32_t* idx,
                                                      int64_t capacity, FrameCounters* ctr, int32_t* d_count) {
  __shared__ uint32_t wt[kBlock / 64];
  __shared__ uint32_t total[4][kBlock / 64];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint64_t lt = lanemask_lt();
  // selected nodes of the tiles [0, tile), the whole wave adding up
  const auto before = [&](int tile) -> uint32_t {
    if (place) return place[tile];
    uint32_t x = 0;
#pragma unroll 4
    for (int i = lane; i < tile; i += 64) x += selected[i];
    return wave_total(x);
  };
  if ((int)blockIdx.x < n_upper_tiles) {  // block-uniform
    const int tile = (int)blockIdx.x;
    if (selected[tile] == 0u) return;
    const int64_t u = (int64_t)tile * kCutTile + t;
    const bool p = u < S.n_upper && upper_sel[u] != 0;
    const uint32_t base = before(tile);
    uint32_t tot;
    const uint32_t pos = base + block_exclusive_scan(p ? 1u : 0u, wt, &tot);
    if (p && pos < capacity) idx[pos] = (int32_t)u;
    return;
  }
  if (blockIdx.x == gridDim.x - 1) {  // block-uniform: the totals
    const int threads = place ? kBlock : 64;
    if (t >= threads) return;  // whole waves
    uint32_t o[4] = {0u, 0u, 0u, 0u};
#pragma unroll 4
    for (int i = t; i < ntiles; i += threads) {
      const uint4 x = sums[i];
      o[0] += x.x;
      o[1] += x.y;
      o[2] += x.z;
      o[3] += selected[i];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = wave_total(o[k]);
    if (place) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (lane == 0) total[k][wv] = o[k];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = total[k][0] + total[k][1] + total[k][2] + total[k][3];
    }
    if (t == 0) {
      const uint32_t n = o[3];
      ctr->n_selected = (int32_t)n;
      ctr->n_upper_selected = (int32_t)o[0];
      ctr->n_spt_visible = (int32_t)o[1];
      ctr->sum_high = (int32_t)o[2];
      *d_count = (int32_t)n;
      if ((int64_t)n > capacity) ctr->status = LODGS_E_CAPACITY;
    }
    return;
  }
  const int n = ctr->n_chunks, run = ((int)blockIdx.x - n_upper_tiles) * (kBlock / 64) + wv;
  // writes a chunk's selected candidates from place pos0 on, returns the place after them
  const auto write = [&](const ChunkNodes& nodes, uint32_t pos0) -> uint32_t {
    const uint32_t bits = nodes.selected();
#pragma unroll
    for (int q = 0; q < kChunk / 64; ++q) {
      const bool p = (bits >> q) & 1u;
      const uint64_t mask = __ballot(p);
      const uint32_t pos = pos0 + (uint32_t)__popcll(mask & lt);
      if (p && pos < capacity) idx[pos] = nodes.node + 64 * q;
      pos0 += (uint32_t)__popcll(mask);
    }
    return pos0;
  };
  if (n <= kCutRuns) {  // a run is one chunk
    if (run >= n) return;
    const uint2 ch = chunks[run];
    if ((ch.y & kChunkCount) == 0u) return;
    const int32_t b = S.spt_begin[ch.x];
    const ChunkNodes nodes(S, chunk_node(b, ch.y), b + spt_high[ch.x], spt_X[ch.x]);
    const int tile = n_upper_tiles + (int)ch.x / kCutTile;
    uint32_t x = 0;
#pragma unroll 4
    for (int i = (int)first[tile] + lane; i < run; i += 64) x += chunks[i].y & kChunkCount;
    write(nodes, before(tile) + wave_total(x));
    return;
  }
  const int per = run_length(n), r = __builtin_amdgcn_readfirstlane(run);
  const int c0 = r * per, c1 = min(c0 + per, n);
  int32_t tile = -1;
  uint32_t pos0 = 0;
  for (int g0 = c0; g0 < c1; g0 += 64) {  // wave-uniform
    const int m = min(64, c1 - g0);
    const LaneChunk ch = load_chunk(S, spt_high, spt_X, chunks, g0, m);
    for (uint64_t left = __ballot(lane < m && (ch.word & kChunkCount) != 0u); left; left &= left - 1) {
      const int l = __builtin_ctzll(left);
      const int32_t own = n_upper_tiles + lane_value(ch.spt, l) / kCutTile;
      const ChunkNodes nodes(S, ch, l);
      if (own != tile) {
        tile = own;
        // the chunks before this one in the tile: from the tile's first to the
        // next run, whole runs, and this run's
        const int c = g0 + l, a = (int)first[tile];
        const int ra = min((a + per - 1) / per, r);
        uint32_t x = 0;
        for (int i = a + lane; i < min(ra * per, c); i += 64) x += chunks[i].y & kChunkCount;
        for (int i = ra + lane; i < r; i += 64) x += runs[i];
        for (int i = max(a, c0) + lane; i < c; i += 64) x += chunks[i].y & kChunkCount;
        pos0 = before(tile) + wave_total(x);
      }
      pos0 = write(nodes, pos0);
    }
  }
}

}  // namespace

int build_ancestor_table(lodgs_scene* s) {
  SceneDev& S = s->dev;
  const int64_t total = (int64_t)S.n_upper + S.n_spt;
  if (S.n_upper <= 0 || total <= 0) return LODGS_OK;
  int32_t* d_depth = nullptr;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&d_depth), sizeof(int32_t));
  if (e == hipSuccess) e = hipMemset(d_depth, 0, sizeof(int32_t));
  int grid = (int)((total + kBlock - 1) / kBlock);
  grid = grid > 4096 ? 4096 : grid;
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_anc_depth, dim3(grid), dim3(kBlock), 0, 0, S, d_depth);
    e = hipGetLastError();
  }
  int32_t D = 0;
  if (e == hipSuccess) e = hipMemcpy(&D, d_depth, sizeof D, hipMemcpyDeviceToHost);
  if (d_depth) (void)hipFree(d_depth);
  if (e != hipSuccess) return hip_fail(e, "lodgs_scene_create: ancestor table");
  if (D <= 0 || D > kMaxAncDepth) return LODGS_OK;  // the cut walks the parent array instead
  int32_t* anc = nullptr;
  e = hipMalloc(reinterpret_cast<void**>(&anc), sizeof(int32_t) * (size_t)D * (size_t)total);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return LODGS_OK;  // no room: the cut walks the parent array instead
  }
  hipLaunchKernelGGL(k_anc_fill, dim3(grid), dim3(kBlock), 0, 0, S, D, anc);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    (void)hipFree(anc);
    return hip_fail(e, "lodgs_scene_create: ancestor table");
  }
  s->anc_owned = anc;
  S.anc = anc;
  S.anc_depth = D;
  return LODGS_OK;
}

// Radius of each SPT about its root's mean, for the CONSERVATIVE cut: the
// largest |mu_i - mu_root| over the SPT's members (its layout segment), in
// FP64 from the FP32 means (((dx dx + dy dy) + dz dz), correctly rounded
// square root), rounded once to FP32.  One wave per SPT; the maximum is exact,
// so the order does not matter.
__global__ void __launch_bounds__(kBlock) k_spt_radius(SceneDev S, float* radius) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t j = wave; j < S.n_spt; j += waves) {  // wave-uniform
    const int64_t b = S.spt_begin[j], e = S.spt_begin[j + 1];
    const double rx = S.means[3 * b], ry = S.means[3 * b + 1], rz = S.means[3 * b + 2];
    double r = 0.0;
    for (int64_t i = b + lane; i < e; i += 64) {
      const double dx = (double)S.means[3 * i] - rx, dy = (double)S.means[3 * i + 1] - ry,
                   dz = (double)S.means[3 * i + 2] - rz;
      r = fmax(r, __builtin_sqrt((dx * dx + dy * dy) + dz * dz));
    }
    for (int d = 32; d > 0; d >>= 1) r = fmax(r, __shfl_xor(r, d, 64));
    if (lane == 0) radius[j] = (float)r;
  }
}

int build_spt_radius(lodgs_scene* s) {
  SceneDev& S = s->dev;
  if (S.n_spt <= 0) return LODGS_OK;
  float* r = nullptr;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&r), sizeof(float) * (size_t)S.n_spt);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return set_error(LODGS_E_OOM, "lodgs_scene_create: SPT radii");
  }
  int grid = (int)(((int64_t)S.n_spt * 64 + kBlock - 1) / kBlock);
  grid = grid > 4096 ? 4096 : grid;
  hipLaunchKernelGGL(k_spt_radius, dim3(grid), dim3(kBlock), 0, 0, S, r);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    (void)hipFree(r);
    return hip_fail(e, "lodgs_scene_create: SPT radii");
  }
  s->radius_owned = r;
  S.spt_radius = r;
  return LODGS_OK;
}

void launch_select(lodgs_frame* f, const ViewConst& v, uint32_t flags, int32_t* d_idx, int64_t capacity,
                   int32_t* d_count, hipStream_t st, const CacheDev* cache) {
  CacheDev C{};
  if (cache) C = *cache;
  const SceneDev& S = f->scene->dev;
  stage_begin(f, LODGS_STAGE_SELECT, st);
  const int64_t g = ((int64_t)S.n_upper + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(k_select_begin, dim3((int)(g < 1 ? 1 : (g > 4096 ? 4096 : g))), dim3(kBlock), 0, st, v,
                     f->d_view_sel, f->ctr, S, flags, f->upper_test);
  const int32_t n_upper_tiles = (int32_t)upper_tiles(S);
  const int32_t tiles = (int32_t)cut_tiles(S);
  hipLaunchKernelGGL(k_cut_upper, dim3(tiles), dim3(kBlock), 0, st, S, f->d_view_sel, flags, f->upper_test,
                     f->upper_sel, f->spt_high, f->spt_X, f->ctr, n_upper_tiles, f->cut_selected, f->cut_sums,
                     f->cut_first, f->cut_chunks, C);
  hipLaunchKernelGGL(k_cut_count, dim3(kCountGrid), dim3(kCountThreads), 0, st, S, f->ctr, f->spt_high, f->spt_X,
                     f->cut_chunks, n_upper_tiles, f->cut_selected, f->cut_runs, C.spt_sel);
  const bool wide = tiles > kWideTiles;
  if (wide)
    scan_exclusive(LoadArray{f->cut_selected}, &f->ctr->n_cut_tiles, tiles, f->block_sums, f->cut_place, nullptr, st);
  hipLaunchKernelGGL(k_cut_write, dim3(n_upper_tiles + kChunkGrid + 1), dim3(kBlock), 0, st, S, f->upper_sel,
                     n_upper_tiles, tiles, f->cut_selected, wide ? f->cut_place : (const uint32_t*)nullptr, f->cut_sums,
                     f->cut_first, f->spt_high, f->spt_X, f->cut_chunks, f->cut_runs, d_idx, capacity,
                     f->ctr, d_count);
  stage_end(f, st);
}

// ---------------------------------------------------------------- comparator cuts
// The two whole-hierarchy cuts the HSPT replaces (Sec. 4.3): the BFS cut and
// the parallel cut of Eq. 5.  Both mark the selected nodes in a bitmask (bit
// i % 32 of word i / 32); an exclusive scan of the words' popcounts then
// writes the ascending list, so the order of the marking does not matter.
namespace {

__device__ __forceinline__ bool node_fine(const SceneDev& S, const ViewConst& v, int64_t i, float mx, float my,
                                          float mz) {
  return S.r_min[i] <= view_distance(v, mx, my, mz) * v.k;
}

// Clears the bitmask and the BFS level counts (level 0 holds the root alone).
__global__ void __launch_bounds__(kBlock) k_cut_clear(uint32_t* bits, int64_t n_words, int32_t* level_count,
                                                      int32_t n_levels) {
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t w = t0; w < n_words; w += stride) bits[w] = 0u;
  if (level_count)
    for (int64_t l = t0; l < n_levels; l += stride) level_count[l] = l == 0 ? 1 : 0;
}

// Eq. 5 per node: fine at its own distance while its parent is not (the root
// has none); with culling, a node whose own sphere is outside the frustum is
// dropped.  One wave per 64 nodes writes their two bitmask words.
__global__ void __launch_bounds__(kBlock) k_parallel_cut(SceneDev S, const ViewConst* __restrict__ vp, uint32_t flags,
                                                         uint32_t* bits) {
  const ViewConst v = *vp;
  const bool cull = (flags & LODGS_CULL) != 0;
  const int lane = threadIdx.x & 63;
  const int64_t n_waves = (S.n_nodes + 63) / 64;
  for (int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; w < n_waves;
       w += ((int64_t)gridDim.x * blockDim.x) >> 6) {  // wave-uniform
    const int64_t i = w * 64 + lane;
    bool sel = false;
    if (i < S.n_nodes) {
      const float mx = S.means[3 * i], my = S.means[3 * i + 1], mz = S.means[3 * i + 2];
      sel = node_fine(S, v, i, mx, my, mz);
      if (sel) {
        const int64_t p = S.parent[i];
        if (p >= 0 && p < S.n_nodes)
          sel = !node_fine(S, v, p, S.means[3 * p], S.means[3 * p + 1], S.means[3 * p + 2]);
      }
      if (sel && cull) sel = !sphere_culled(v, mx, my, mz, S.rho[i]);
    }
    const uint64_t b = __ballot(sel);
    if (lane == 0) reinterpret_cast<uint2*>(bits)[w] = make_uint2((uint32_t)b, (uint32_t)(b >> 32));
  }
}

// One BFS level: every frontier node is dropped when culled, marked when fine
// at its own distance, else its two children join the next frontier (one
// atomic per wave for their slots).  Level 0 is the root, position 0.  Counts stay even past the root's level,
// and fcap is even, so a pair of children is written whole or not at all; a
// full queue records LODGS_E_CAPACITY and the next level reads only what was
// written.
__global__ void __launch_bounds__(kBlock) k_bfs_level(SceneDev S, const ViewConst* __restrict__ vp, uint32_t flags,
                                                      int32_t level, const int32_t* fin, int32_t* fout,
                                                      int32_t* level_count, int64_t fcap, uint32_t* bits,
                                                      FrameCounters* ctr) {
  const ViewConst v = *vp;
  const bool cull = (flags & LODGS_CULL) != 0;
  const int lane = threadIdx.x & 63;
  const uint64_t lt = lanemask_lt();
  int64_t n_in = level_count[level];
  n_in = level == 0 ? 1 : (n_in < fcap ? n_in : fcap);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63); t0 < n_in; t0 += stride) {
    const int64_t t = t0 + lane;  // t0 is wave-aligned: the loop is wave-uniform
    bool push = false;
    int2 ch = make_int2(-1, -1);
    if (t < n_in) {
      const int64_t u = level == 0 ? 0 : fin[t];
      if (u >= 0 && u < S.n_nodes) {
        const float mx = S.means[3 * u], my = S.means[3 * u + 1], mz = S.means[3 * u + 2];
        if (!(cull && sphere_culled(v, mx, my, mz, S.rho[u]))) {
          if (node_fine(S, v, u, mx, my, mz)) {
            atomicOr(&bits[u >> 5], 1u << (u & 31));
          } else {
            ch = S.child[u];
            push = ch.x >= 0 && ch.x < S.n_nodes && ch.y >= 0 && ch.y < S.n_nodes;
          }
        }
      }
    }
    const uint64_t pb = __ballot(push);
    if (pb) {
      uint32_t base = 0;
      if (lane == 0) base = (uint32_t)atomicAdd(&level_count[level + 1], 2 * __popcll(pb));
      base = __shfl(base, 0, 64);
      if (push) {
        const int64_t pos = (int64_t)base + 2 * __popcll(pb & lt);
        if (pos < fcap) {
          fout[pos] = ch.x;
          fout[pos + 1] = ch.y;
        } else {
          ctr->status = LODGS_E_CAPACITY;
        }
      }
    }
  }
}

struct LoadPopc {
  const uint32_t* bits;
  __device__ uint32_t operator()(int64_t w) const { return (uint32_t)__popc(bits[w]); }
};

// Word w's set bits, lowest first, at idx[prefix ...].
struct StoreBits {
  const uint32_t* bits;
  int32_t* idx;
  int64_t cap;
  __device__ void operator()(int64_t w, uint32_t prefix, uint32_t) const {
    uint32_t b = bits[w];
    int64_t p = prefix;
    while (b) {
      const int k = __ffs(b) - 1;
      b &= b - 1u;
      if (p < cap) idx[p] = (int32_t)(w * 32 + k);
      ++p;
    }
  }
};

// The count, the capacity check and, for the BFS, the depth check: a
// frontier left after the last level means the hierarchy is deeper than its
// stated height.
__global__ void k_cut_finish(FrameCounters* ctr, int32_t* d_count, int64_t capacity, const int32_t* level_count,
                             int32_t height) {
  const int32_t n = ctr->n_selected;
  *d_count = n;
  if ((int64_t)n > capacity) ctr->status = LODGS_E_CAPACITY;
  if (level_count && level_count[height] > 0) ctr->status = LODGS_E_INVALID;
}

}  // namespace

void launch_select_full(lodgs_frame* f, const ViewConst& v, uint32_t flags, int32_t* d_idx, int64_t capacity,
                        int32_t* d_count, hipStream_t st) {
  const SceneDev& S = f->scene->dev;
  const bool bfs = (flags & LODGS_CUT_BFS) != 0;
  const int64_t n_words = cut_bit_words(S.n_nodes);
  stage_begin(f, LODGS_STAGE_SELECT, st);
  launch_set_view(v, f->d_view_sel, f->ctr, kViewSelect, nullptr, 0, nullptr, nullptr, st);
  int cgrid = (int)((n_words + kBlock - 1) / kBlock);
  cgrid = cgrid < 1 ? 1 : (cgrid > 2048 ? 2048 : cgrid);
  hipLaunchKernelGGL(k_cut_clear, dim3(cgrid), dim3(kBlock), 0, st, f->cut_bits, n_words,
                     bfs ? f->level_count : (int32_t*)nullptr, f->cut_height + 1);
  if (bfs) {
    const int64_t fcap = f->caps.max_selected & ~(int64_t)1;
    for (int32_t l = 0; l < f->cut_height; ++l)
      hipLaunchKernelGGL(k_bfs_level, dim3(1024), dim3(kBlock), 0, st, S, f->d_view_sel, flags, l,
                         f->frontier[l & 1], f->frontier[(l + 1) & 1], f->level_count, fcap, f->cut_bits, f->ctr);
  } else {
    int pgrid = (int)((S.n_nodes + kBlock - 1) / kBlock);
    pgrid = pgrid < 1 ? 1 : (pgrid > 8192 ? 8192 : pgrid);
    hipLaunchKernelGGL(k_parallel_cut, dim3(pgrid), dim3(kBlock), 0, st, S, f->d_view_sel, flags, f->cut_bits);
  }
  scan_exclusive(LoadPopc{f->cut_bits}, &f->ctr->n_bit_words, n_words, f->block_sums,
                 StoreBits{f->cut_bits, d_idx, capacity}, &f->ctr->n_selected, st);
  hipLaunchKernelGGL(k_cut_finish, dim3(1), dim3(1), 0, st, f->ctr, d_count, capacity,
                     bfs ? (const int32_t*)f->level_count : (const int32_t*)nullptr, f->cut_height);
  stage_end(f, st);
}

}  // namespace lodgs
