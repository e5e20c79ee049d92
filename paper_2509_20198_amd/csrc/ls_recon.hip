// Tile binning and per-tile interpolated heightmaps (LidarScout Section 3.3,
// Algorithm 1; normalisation of Section 3.4) for gfx950.
//
// Pipeline of ls_recon_tiles, all on one stream, no host round trip:
//   1. k_tile_pos: map linear tile id -> output slot.
//   2. k_bin_count, k_bin_scan, k_bin_scatter: CSR of the points in every
//      listed tile's padded window [c - H, c + H)^2 (a point sits in 1, 2 or
//      4 windows with the paper's 16-texel ring).
//   3. k_bin_sort (only when the caller asks for the CSR): ascending order.
//   4. for as many tiles at a time as the workspace holds face maps, in the
//      caller's list order or by descending window point count, the tiles that
//      cannot hold a triangle at the end:
//      k_recon_prep, one workgroup per tile:
//        a. gather the tile's points to tile-local coordinates and bucket
//           them into a G x G grid over the window (LDS counting sort);
//        b. sort each bucket by (v, u) and drop duplicate positions,
//           keeping the largest (z, R, G, B) -> canonical points; face map
//           reset;
//      k_recon_stars, a list of small runs of points for the whole chip:
//        c. Delaunay triangulation by gift-wrapping around every point (first
//           point hit by a circle growing from a Delaunay edge), with exact
//           orientation and in-circle tests and a symbolic perturbation of
//           the lifted heights (lower canonical index = larger perturbation)
//           that makes the triangulation unique when points are cocircular.
//           A triangle is rasterised by its lowest vertex into a per-texel
//           face map (top-left rule), hull edges by their lower endpoint, so
//           every texel of the closed convex hull gets a containing triangle;
//      k_recon_out, several workgroups per tile:
//        d. nearest point of every texel centre (exact distances, ties by
//           (d^2, v, u)) by scans over the buckets;
//        e. c_z from the centre texel, then per texel: barycentric height and
//           colour inside the hull, nearest point outside it (the paper's
//           corner padding points taken at infinity), normalised and written
//           as one NHWC row of 8 FP32 channels.
// Three launches rather than one workgroup per tile from end to end: the work
// of a tile follows its point count (20 to tens of thousands), and a launch
// over runs of points spreads the largest tile over the chip.  One tile of 400
// points 536 -> 190 us (reconstruction and network), one of 16,000 points
// 16.3 -> 0.78 ms, 1024 tiles of 50-2000 points 2.22 -> 1.51 ms, 16384 tiles of
// 20-5000 points 13.2 -> 7.7 ms.
#include <algorithm>
#include <mutex>

#include "ls_common.hpp"

namespace {

constexpr int RB = 512;                  // threads of a preparation workgroup
constexpr int PREP_INTS = 12000;         // its LDS: windows up to 2,644 points sort there
constexpr int PREP_BATCH = 4;            // points a lane reads at a time
constexpr int MAXG = 76;                 // max buckets per side
constexpr int MAXB = MAXG * MAXG;        // max buckets
static_assert(2 * (MAXB + 1) <= PREP_INTS, "bucket offsets must fit twice in the preparation's LDS");
constexpr int TB = 256;                  // threads of a star or output workgroup
constexpr int OUT_INTS = 7000;           // LDS of an output workgroup for the points and bucket offsets
constexpr int XCDS = 8;                  // chiplets, each with an L2 of its own
constexpr int ITEM_COUNTER = 32;         // integers from a counter to the next: a cache line each
constexpr int N_FLAGS = ITEM_COUNTER * (2 + XCDS);
constexpr int ITEM_MIN = 8, ITEM_MAX = 16;  // points of a work item of the stars
constexpr int CAND = 8;                  // candidates of a star a lane holds
constexpr int CANDS = 8 * CAND;          // and the eight lanes of a star
constexpr int TRI_CAP = 96;              // triangles a wave collects
constexpr int STAR_MAX_STEPS = 1024;     // safeguard on one point's star walk
constexpr uint64_t FACE_NONE = ~0ull;
// First square of a third-vertex search: its centre this share of the edge's
// length beside the midpoint, its half side this share, at least SEARCH_MIN buckets
constexpr float SEARCH_OFFSET = 0.5f, SEARCH_SIZE = 0.9f, SEARCH_MIN = 0.6f;
// First margin, in buckets, of a nearest-point search
constexpr float NEAR_MARGIN = 1.f;
constexpr int SORT_LDS = 16384;          // bin segments up to this size sort in LDS

struct BinParams {
  int64_t ox, oy;
  double invS;  // 1 / S
  int32_t S, H, tiles_x, tiles_y, K;
  int32_t n_tiles;
  int64_t n;
  const int32_t* x;
  const int32_t* y;
  const int32_t* tile_pos;
  int32_t* counts;
  int32_t* fill;
  int32_t* bin_off;
  int32_t* bin_idx;
  int64_t cap;
  int32_t* flags;  // [0]: cap overflow
  int32_t* order;  // recon processing order (tile slots)
  int32_t order_mode;  // LS_ORDER_LIST or LS_ORDER_LONGEST_FIRST
  int32_t n_face;  // most windows that may hold a triangle
};

// floor(a / S) for |a| < 2^53: the double quotient is within one of it
// (a is exact in double), then an exact integer correction.
__device__ __forceinline__ int64_t floordiv_s(int64_t a, int32_t S, double invS) {
  int64_t q = (int64_t)floor((double)a * invS);
  if (q * S > a)
    --q;
  else if ((q + 1) * S <= a)
    ++q;
  return q;
}

// Visit every listed tile whose padded window contains point i.
template <class F>
__device__ __forceinline__ void for_each_window(const BinParams& p, int64_t i, F&& f) {
  const int64_t px = p.x[i], py = p.y[i];
  const int64_t tx0 = floordiv_s(px - p.ox, p.S, p.invS), ty0 = floordiv_s(py - p.oy, p.S, p.invS);
  for (int64_t ty = ty0 - p.K; ty <= ty0 + p.K; ++ty) {
    if (ty < 0 || ty >= p.tiles_y) continue;
    const int64_t cy = p.oy + ty * p.S + p.S / 2;
    if (py < cy - p.H || py >= cy + p.H) continue;
    for (int64_t tx = tx0 - p.K; tx <= tx0 + p.K; ++tx) {
      if (tx < 0 || tx >= p.tiles_x) continue;
      const int64_t cx = p.ox + tx * p.S + p.S / 2;
      if (px < cx - p.H || px >= cx + p.H) continue;
      const int32_t s = p.tile_pos[ty * p.tiles_x + tx];
      if (s >= 0) f(s);
    }
  }
}

__global__ void k_fill_i32(int32_t* __restrict__ a, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    a[i] = v;
}

// Start values of the per-tile arrays, in one launch (five fills took 20 us of
// gaps between launches).
__global__ void k_recon_init(int32_t* __restrict__ tile_pos, int64_t n_all, int32_t* __restrict__ counts,
                             int32_t* __restrict__ fill, int32_t* __restrict__ status, int32_t n_tiles,
                             int32_t* __restrict__ flags) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x, first = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (int64_t i = first; i < n_all; i += step) tile_pos[i] = 0x7fffffff;
  for (int64_t i = first; i <= n_tiles; i += step) {
    counts[i] = 0;
    fill[i] = 0;
    if (i < n_tiles) status[i] = 0;
  }
  for (int64_t i = first; i < N_FLAGS; i += step) flags[i] = 0;
}

__global__ void k_tile_pos(const int32_t* __restrict__ tile_list, int32_t n_tiles, int64_t n_all,
                           int32_t* __restrict__ tile_pos, int32_t* __restrict__ status) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_tiles) return;
  const int32_t t = tile_list[k];
  if (t < 0 || t >= n_all) {
    status[k] = LS_TILE_BADID;
    return;
  }
  // lowest slot wins for a tile listed twice; the others are flagged
  atomicMin(&tile_pos[t], k);
}

// Listed tiles that lost their entry are flagged; entries nobody took become -1.
__global__ void k_tile_pos_fix(const int32_t* __restrict__ tile_list, int32_t n_tiles, int64_t n_all,
                               int32_t* __restrict__ tile_pos, int32_t* __restrict__ status) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x, first = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (int64_t k = first; k < n_tiles; k += step) {
    const int32_t t = tile_list[k];
    if (t >= 0 && t < n_all && tile_pos[t] != k) status[k] = LS_TILE_BADID;
  }
  for (int64_t i = first; i < n_all; i += step)
    if (tile_pos[i] == 0x7fffffff) tile_pos[i] = -1;
}

__global__ void k_bin_count(BinParams p) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < p.n; i += (int64_t)gridDim.x * blockDim.x)
    for_each_window(p, i, [&](int32_t s) { atomicAdd(&p.counts[s], 1); });
}

// Workgroup-private tile histograms: each workgroup bins a contiguous chunk
// of points into an LDS histogram and adds it to the global counts with one
// atomic per tile it touched (instead of one global atomic per membership on
// a few hot counters).
constexpr int BIN_THREADS = 1024;
constexpr int BIN_LDS_TILES = 8192;

__global__ void __launch_bounds__(BIN_THREADS) k_bin_count_lds(BinParams p, int64_t per_block) {
  __shared__ int s_cnt[BIN_LDS_TILES];
  for (int t = threadIdx.x; t < p.n_tiles; t += BIN_THREADS) s_cnt[t] = 0;
  __syncthreads();
  const int64_t i0 = blockIdx.x * per_block, i1 = min(p.n, i0 + per_block);
  for (int64_t i = i0 + threadIdx.x; i < i1; i += BIN_THREADS)
    for_each_window(p, i, [&](int32_t s) { atomicAdd(&s_cnt[s], 1); });
  __syncthreads();
  for (int t = threadIdx.x; t < p.n_tiles; t += BIN_THREADS)
    if (s_cnt[t]) atomicAdd(&p.counts[t], s_cnt[t]);
}

// Scatter with the same chunks: local counts, one global reservation per
// touched tile, then positions from LDS cursors.  Within a tile the order of
// workgroups (and of lanes) is arbitrary; the per-tile sort restores
// ascending order when the caller asks for the CSR.
__global__ void __launch_bounds__(BIN_THREADS) k_bin_scatter_lds(BinParams p, int64_t per_block) {
  __shared__ int s_cnt[BIN_LDS_TILES];
  for (int t = threadIdx.x; t < p.n_tiles; t += BIN_THREADS) s_cnt[t] = 0;
  __syncthreads();
  const int64_t i0 = blockIdx.x * per_block, i1 = min(p.n, i0 + per_block);
  for (int64_t i = i0 + threadIdx.x; i < i1; i += BIN_THREADS)
    for_each_window(p, i, [&](int32_t s) { atomicAdd(&s_cnt[s], 1); });
  __syncthreads();
  for (int t = threadIdx.x; t < p.n_tiles; t += BIN_THREADS) {
    const int c = s_cnt[t];
    if (c) s_cnt[t] = p.bin_off[t] + atomicAdd(&p.fill[t], c);
  }
  __syncthreads();
  for (int64_t i = i0 + threadIdx.x; i < i1; i += BIN_THREADS)
    for_each_window(p, i, [&](int32_t s) {
      const int32_t pos = atomicAdd(&s_cnt[s], 1);
      if (pos < p.cap) p.bin_idx[pos] = (int32_t)i;
    });
}

constexpr int ORDER_KEYS = 4096;
// Points of a window that may hold a triangle.  Smaller windows need no face map:
// they come last in the processing order, behind the launches that hold some.
constexpr int FACE_POINTS = 3;

// Descending window count, in steps of 4 points, as an ascending key.
__device__ __forceinline__ int order_key(int32_t count) {
  return count < FACE_POINTS ? ORDER_KEYS - 1 : ORDER_KEYS - 2 - min(count >> 2, ORDER_KEYS - 2);
}

// Single-workgroup exclusive scan of counts -> bin_off (n_tiles + 1 entries),
// and the recon processing order: the caller's list order (where not all windows
// can hold a triangle, those that do not behind the others, in reverse), or a
// counting sort of the tile slots by order_key (slots with equal keys in any order;
// the results do not depend on the order).
__global__ void __launch_bounds__(1024) k_bin_scan(BinParams p) {
  __shared__ int64_t s_part[1024];
  __shared__ int64_t s_carry;
  __shared__ int s_hist[ORDER_KEYS];
  __shared__ int s_faces[1024 / 64];
  const int tid = threadIdx.x;
  const bool part = p.order_mode == LS_ORDER_LIST && p.n_face < p.n_tiles;
  int faces = 0;  // windows before these that may hold a triangle
  if (tid == 0) s_carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < p.n_tiles; base += 1024) {
    const int64_t i = base + tid;
    const int64_t v = i < p.n_tiles ? p.counts[i] : 0;
    s_part[tid] = v;
    const uint64_t with_face = __ballot(v >= FACE_POINTS);
    if ((tid & 63) == 0) s_faces[tid >> 6] = __popcll(with_face);
    __syncthreads();
    if (part) {
      int before = faces + __popcll(with_face & ((1ull << (tid & 63)) - 1));
      for (int w = 0; w < 1024 / 64; ++w) {
        before += w < (tid >> 6) ? s_faces[w] : 0;
        faces += s_faces[w];
      }
      if (i < p.n_tiles) p.order[v >= FACE_POINTS ? before : p.n_tiles - 1 - ((int)i - before)] = (int)i;
    }
    for (int o = 1; o < 1024; o <<= 1) {
      const int64_t t = tid >= o ? s_part[tid - o] : 0;
      __syncthreads();
      s_part[tid] += t;
      __syncthreads();
    }
    const int64_t excl = s_carry + s_part[tid] - v;
    if (i < p.n_tiles) p.bin_off[i] = (int32_t)(excl < 0x7fffffff ? excl : 0x7fffffff);
    __syncthreads();
    if (tid == 1023) s_carry += s_part[1023];
    __syncthreads();
  }
  if (tid == 0) {
    const int64_t total = s_carry;
    p.bin_off[p.n_tiles] = (int32_t)(total < 0x7fffffff ? total : 0x7fffffff);
    p.flags[0] = total > p.cap ? 1 : 0;
  }
  if (p.order_mode == LS_ORDER_LIST) {
    for (int i = tid; i < p.n_tiles && !part; i += 1024) p.order[i] = i;
    return;
  }
  constexpr int PER = ORDER_KEYS / 1024;
  for (int b = tid; b < ORDER_KEYS; b += 1024) s_hist[b] = 0;
  __syncthreads();
  for (int i = tid; i < p.n_tiles; i += 1024) atomicAdd(&s_hist[order_key(p.counts[i])], 1);
  __syncthreads();
  int run = 0;
  for (int j = 0; j < PER; ++j) run += s_hist[tid * PER + j];
  s_part[tid] = run;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int64_t t = tid >= o ? s_part[tid - o] : 0;
    __syncthreads();
    s_part[tid] += t;
    __syncthreads();
  }
  int excl = (int)(s_part[tid] - run);
  for (int j = 0; j < PER; ++j) {
    const int c = s_hist[tid * PER + j];
    s_hist[tid * PER + j] = excl;
    excl += c;
  }
  __syncthreads();
  for (int i = tid; i < p.n_tiles; i += 1024) p.order[atomicAdd(&s_hist[order_key(p.counts[i])], 1)] = i;
}

__global__ void k_bin_scatter(BinParams p) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < p.n; i += (int64_t)gridDim.x * blockDim.x)
    for_each_window(p, i, [&](int32_t s) {
      const int32_t r = atomicAdd(&p.fill[s], 1);
      const int64_t pos = (int64_t)p.bin_off[s] + r;
      if (pos < p.cap) p.bin_idx[pos] = (int32_t)i;
    });
}

// In-place ascending bitonic sort of one bin segment; segments longer than
// SORT_LDS use `spill` (2 entries per bin entry, so the power-of-two
// padding always fits).
__global__ void __launch_bounds__(RB) k_bin_sort(const int32_t* __restrict__ bin_off, int32_t n_tiles,
                                                 int32_t* __restrict__ bin_idx, int32_t* __restrict__ spill,
                                                 const int32_t* __restrict__ flags) {
  __shared__ int32_t s_buf[SORT_LDS];
  if (flags[0]) return;
  for (int k = blockIdx.x; k < n_tiles; k += gridDim.x) {
    const int32_t off = __builtin_amdgcn_readfirstlane(bin_off[k]);
    const int32_t cnt = __builtin_amdgcn_readfirstlane(bin_off[k + 1]) - off;
    if (cnt <= 1) continue;  // uniform: k comes from blockIdx, the counts are readfirstlane'd
    int n2 = 1;
    while (n2 < cnt) n2 <<= 1;
    int32_t* buf = n2 <= SORT_LDS ? s_buf : spill + 2 * (int64_t)off;
    for (int i = threadIdx.x; i < n2; i += RB) buf[i] = i < cnt ? bin_idx[off + i] : 0x7fffffff;
    __syncthreads();
    for (int kk = 2; kk <= n2; kk <<= 1)
      for (int j = kk >> 1; j > 0; j >>= 1) {
        for (int i = threadIdx.x; i < n2; i += RB) {
          const int l = i ^ j;
          if (l > i) {
            const int32_t a = buf[i], b = buf[l];
            const bool asc = (i & kk) == 0;
            if ((a > b) == asc) {
              buf[i] = b;
              buf[l] = a;
            }
          }
        }
        __syncthreads();
      }
    for (int i = threadIdx.x; i < cnt; i += RB) bin_idx[off + i] = buf[i];
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// per-tile reconstruction
// ---------------------------------------------------------------------------
struct ReconParams {
  int64_t ox, oy;
  int32_t S, tiles_x, C, R, H;
  double scale_z, offset_z, inv_r;
  const int32_t* x;
  const int32_t* y;
  const int32_t* z;
  const uint16_t* rgb;
  const int32_t* tile_list;
  const int32_t* bin_off;
  const int32_t* bin_idx;
  const int32_t* flags;
  // per bin entry: tile-local coordinates and bucket slots, sort keys and
  // entries of windows that do not sort in LDS, canonical points
  int32_t* su;
  int32_t* sv;
  int32_t* sslot;
  uint64_t* skey;
  int32_t* sidx;
  int2* cuv;
  int4* cattr;  // z, R, G, B
  int32_t* boff;   // 2 per bin entry: canonical bucket offsets of a tile from 2 * its bin offset on
  // per tile slot
  int32_t* npts;   // canonical points
  uint64_t* facemap;  // R * R texels of every tile of the launch; null where none has a triangle
  int2* items;        // work items of the stars: position of the tile in the launch, first point
  int32_t* item_n;    // how many, then by XCD how many of its range are taken, ITEM_COUNTER apart
  int32_t item;       // points of an item
  const int32_t* order;  // processing position -> tile slot
  int32_t q0;            // first position of the launch
  float* x_out;
  double* cz_out;
  int32_t* status;
};

// Bucket grid side of a window with cnt points: 1.25 points a bucket (1024 tiles
// of 50-2000 points 1.90 ms, 1.96 with 1.5, 1.91 with 1).
__device__ __forceinline__ int bucket_side(int cnt) {
  const int want = (int)sqrtf((float)cnt * 0.8f);
  return want < 1 ? 1 : (want > MAXG ? MAXG : want);
}

// Pointers into LDS typed as such, so that reads through them are LDS reads
// (a generic pointer that may point to LDS or to global memory compiles to
// flat loads, which wait on both the LDS and the vector-memory counters).
typedef const __attribute__((address_space(3))) int32_t* LdsI32;
typedef const __attribute__((address_space(3))) uint64_t* LdsU64;
// Point coordinates (u, v) as one 8-byte read.
struct UvGlobal {
  const int2* p;
  __device__ __forceinline__ int2 operator[](int i) const { return p[i]; }
};

// A tile's canonical points: coordinates through UVP (UvGlobal or one of the Uvf),
// bucket offsets (G * G + 1, row-major) through BP.
template <class UVP, class BP>
struct TileT {
  UVP uv;
  BP boff;
  int G, H, W2;
  float inv;  // buckets per raw unit
};

// floor(w * G / W2) for 0 <= w < W2 <= 2^19 and G <= 76 (all products below
// 2^26, so the float estimate of a quotient below 76 is off by far less
// than one): a float reciprocal estimate, then an exact integer correction
// by at most one.
__device__ __forceinline__ int bucket_1d(int w, int G, int W2) {
  const int num = w * G;
  int q = (int)((float)num * __builtin_amdgcn_rcpf((float)W2));
  if (q * W2 > num)
    --q;
  else if ((q + 1) * W2 <= num)
    ++q;
  return q;
}

__device__ __forceinline__ double orient_d(double ax, double ay, double bx, double by, double px, double py) {
  // exact: |differences| < 2^19, products < 2^38, result < 2^39
  return (bx - ax) * (py - ay) - (by - ay) * (px - ax);
}

__device__ __forceinline__ int sgn_d(double v) { return (v > 0.0) - (v < 0.0); }

// Exact sign of the in-circle determinant in int128 (|terms| < 2^79), then
// the symbolic perturbation for exactly cocircular points.
__device__ int incircle_exact(int a, int b, int c, int d, int2 pa, int2 pb, int2 pc, int2 pd) {
  const int64_t adx = pa.x - pd.x, ady = pa.y - pd.y;
  const int64_t bdx = pb.x - pd.x, bdy = pb.y - pd.y;
  const int64_t cdx = pc.x - pd.x, cdy = pc.y - pd.y;
  const __int128 e = (__int128)(adx * adx + ady * ady) * (__int128)(bdx * cdy - cdx * bdy) +
                     (__int128)(bdx * bdx + bdy * bdy) * (__int128)(cdx * ady - adx * cdy) +
                     (__int128)(cdx * cdx + cdy * cdy) * (__int128)(adx * bdy - bdx * ady);
  if (e > 0) return 1;
  if (e < 0) return -1;
  int w = a;
  if (b < w) w = b;
  if (c < w) w = c;
  if (d < w) w = d;
  if (w == d) return -1;
  if (w == a) return sgn_d(orient_d(pb.x, pb.y, pc.x, pc.y, pd.x, pd.y));
  if (w == b) return sgn_d(orient_d(pc.x, pc.y, pa.x, pa.y, pd.x, pd.y));
  return sgn_d(orient_d(pa.x, pa.y, pb.x, pb.y, pd.x, pd.y));
}

// Sign of the in-circle determinant of d against CCW (a, b, c): > 0 when d
// is strictly inside.  Floating-point filter first, exact int128 otherwise,
// then the symbolic perturbation for exactly cocircular points.
__device__ __forceinline__ int incircle_sos(int a, int b, int c, int d, int2 pa, int2 pb, int2 pc, int2 pd) {
  const double fadx = (double)(pa.x - pd.x), fady = (double)(pa.y - pd.y);
  const double fbdx = (double)(pb.x - pd.x), fbdy = (double)(pb.y - pd.y);
  const double fcdx = (double)(pc.x - pd.x), fcdy = (double)(pc.y - pd.y);
  const double al = fadx * fadx + fady * fady;
  const double bl = fbdx * fbdx + fbdy * fbdy;
  const double cl = fcdx * fcdx + fcdy * fcdy;
  const double bc = fbdx * fcdy - fcdx * fbdy;
  const double ca = fcdx * fady - fadx * fcdy;
  const double ab = fadx * fbdy - fbdx * fady;
  const double t1 = al * bc, t2 = bl * ca, t3 = cl * ab;
  const double det = t1 + t2 + t3;
  const double perm = fabs(t1) + fabs(t2) + fabs(t3);
  if (fabs(det) > 8.8817841970012523e-16 * perm) return sgn_d(det);  // 8 * 2^-53
  return incircle_exact(a, b, c, d, pa, pb, pc, pd);
}

// ---- stars: a group of eight lanes works on one star
constexpr int STAR_LANES = 8;  // as many as RASTER_LANES
// f over the group: the other lane of a pair, the other pair of a quad, the
// other quad.
template <class V, class F>
__device__ __forceinline__ V group_reduce(V v, F&& f) {
  v = f(v, row_move<0xB1>(v));
  v = f(v, row_move<0x4E>(v));
  return f(v, row_move<0x141>(v));
}
__device__ __forceinline__ float group_min(float v) {
  return group_reduce(v, [](float a, float b) { return fminf(a, b); });
}
// Value of the group's first lane.
__device__ __forceinline__ int group_first(int v) {
  const int lo = row_move<0x150>(v), hi = row_move<0x158>(v);
  return threadIdx.x & STAR_LANES ? hi : lo;
}
// Sum over the lanes of the group before this one.
__device__ __forceinline__ int group_before(int v, int gl) {
  int t, at = v;
  t = row_move<0x111>(at);  // shifts within the sixteen lanes of a row
  at += gl >= 1 ? t : 0;
  t = row_move<0x112>(at);
  at += gl >= 2 ? t : 0;
  t = row_move<0x114>(at);
  at += gl >= 4 ? t : 0;
  return at - v;
}
// Lanes of the group for which the condition holds.
__device__ __forceinline__ uint32_t group_ballot(bool b) {
  return (uint32_t)(__ballot(b) >> (threadIdx.x & 56)) & 0xFF;
}

// Points of the buckets [x0, x1] x [y0, y1] over the lanes of a group (a bucket
// row each, several lanes to one where these are few), four at a time (the last
// of a bucket row again where it has fewer); cut(y, x0, x1) narrows a row's
// columns.
template <class TT, class Cut, class F>
__device__ __forceinline__ void row_scan(const TT& T, int x0, int x1, int y0, int y1, int gl, Cut&& cut, F&& f) {
  int sh = 3;  // log2 of the lanes of a bucket row
  while (sh > 0 && (STAR_LANES >> sh) < y1 - y0 + 1) --sh;
  for (int y = y0 + (gl >> sh); y <= y1; y += STAR_LANES >> sh) {
    int xa = x0, xb = x1;
    cut(y, xa, xb);
    if (xa > xb) continue;
    const int e = T.boff[y * T.G + xb + 1];
    for (int p = T.boff[y * T.G + xa] + (gl & ((1 << sh) - 1)); p < e; p += 4 << sh) {
      int id[4];
      int2 Q[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        id[j] = min(p + (j << sh), e - 1);
        Q[j] = T.uv[id[j]];
      }
      f(id, Q, min(4, ((e - 1 - p) >> sh) + 1));
    }
  }
}

// Nearest neighbour of point a (the smallest index among equals): the square
// around it grows until it holds the circle through the nearest point found.
template <class TT>
__device__ __forceinline__ int nearest_of_point(const TT& T, int a, int gl) {
  const int2 A = T.uv[a];
  const float fx = (float)(A.x + T.H) * T.inv, fy = (float)(A.y + T.H) * T.inv;
  float r = NEAR_MARGIN;
  for (;;) {
    const int x0 = max((int)floorf(fx - r), 0), x1 = min((int)floorf(fx + r), T.G - 1);
    const int y0 = max((int)floorf(fy - r), 0), y1 = min((int)floorf(fy + r), T.G - 1);
    int best = INT_MAX;
    double bd = 1e300;  // squared distance, exact in double (below 2^40)
    row_scan(T, x0, x1, y0, y1, gl, [](int, int&, int&) {}, [&](const int* p, const int2* Q, int) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double dx = Q[j].x - A.x, dy = Q[j].y - A.y;
        const double d = fma(dx, dx, dy * dy);
        const bool less = p[j] != a && (d < bd || (d == bd && p[j] < best));
        bd = less ? d : bd;
        best = less ? p[j] : best;
      }
    });
    const double least = group_reduce(bd, [](double u, double v) { return fmin(u, v); });
    best = group_reduce(bd == least ? best : INT_MAX, [](int u, int v) { return min(u, v); });
    bd = least;
    const float need = best != INT_MAX ? sqrtf((float)bd) * T.inv * 1.000001f + 1e-3f : 2.f * r;
    if ((best != INT_MAX && need <= r) || (x0 == 0 && y0 == 0 && x1 == T.G - 1 && y1 == T.G - 1)) return best;
    r = need;
  }
}

// Coordinates of a tile's points as floats (exact, below 2^18), from LDS with
// three far points behind the last, or from global memory, where an index
// behind the last reads that.
struct UvfLds {
  LdsU64 p;
  __device__ __forceinline__ float2 operator[](int i) const { return __builtin_bit_cast(float2, (uint64_t)p[i]); }
};
struct UvfGlobal {
  const int2* p;
  int last;
  __device__ __forceinline__ float2 operator[](int i) const {
    const int2 P = p[min(i, last)];
    return make_float2((float)P.x, (float)P.y);
  }
};

// Nearest points of an 8 x 8 block of texels, one texel per lane of a wave;
// ties go to the smallest (d^2, v, u).  The 16 lanes of a 4 x 4 texel
// sub-block scan the same buckets, those under the sub-block widened by a
// margin, so their loop is uniform and a point is one LDS broadcast; the
// margin grows until it covers the distance of every lane's answer, which
// proves it.  (i, j) is the lane's texel, inside the grid for every lane that
// counts.
//
// Distances are taken in float (differences exact, squares within 1.2e-7), four
// points at a time without a branch, also those behind the end of a bucket row
// where it is no multiple of four; a lane whose two least are closer than
// NEAR_TIE compares the points within it exactly.
constexpr float NEAR_TIE = 5e-7f;
template <class TT>
__device__ __forceinline__ int nearest_of_texel(const TT& T, int q0, int C, int R, int i0, int j0, int i, int j) {
  const int qx = q0 + j * C, qy = q0 + i * C;
  const float fqx = (float)qx, fqy = (float)qy;
  const bool in_grid = i < R && j < R;
  const float gx0 = (float)(q0 + j0 * C + T.H) * T.inv, gx1 = (float)(q0 + min(j0 + 3, R - 1) * C + T.H) * T.inv;
  const float gy0 = (float)(q0 + i0 * C + T.H) * T.inv, gy1 = (float)(q0 + min(i0 + 3, R - 1) * C + T.H) * T.inv;
  float r = NEAR_MARGIN;
  for (;;) {
    const int x0 = max((int)floorf(gx0 - r), 0), x1 = min((int)floorf(gx1 + r), T.G - 1);
    const int y0 = max((int)floorf(gy0 - r), 0), y1 = min((int)floorf(gy1 + r), T.G - 1);
    int best = -1;
    float bd = 3e38f, second = 3e38f;  // the two least squared distances
    for (int y = y0; y <= y1; ++y) {
      const int e = T.boff[y * T.G + x1 + 1];
      for (int p = T.boff[y * T.G + x0]; p < e; p += 4) {
        float2 P[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) P[k] = T.uv[p + k];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float dx = P[k].x - fqx, dy = P[k].y - fqy;
          const float d = fmaf(dx, dx, dy * dy);
          second = fminf(second, fmaxf(bd, d));
          best = d < bd ? p + k : best;
          bd = fminf(bd, d);
        }
      }
    }
    float need = !in_grid ? 0.f : (best >= 0 ? sqrtf(bd) * T.inv * 1.000001f + 1e-3f : 2.f * r);
    need = group_reduce(need, [](float a, float b) { return fmaxf(a, b); });
    need = fmaxf(need, row_move<0x128>(need));  // the other eight lanes
    if (need > r && !(x0 == 0 && y0 == 0 && x1 == T.G - 1 && y1 == T.G - 1)) {
      r = need;
      continue;
    }
    if (second <= bd + bd * NEAR_TIE) {
      const float lim = bd + bd * NEAR_TIE;
      double ed = 1e300;  // squared distance, exact in double (below 2^40)
      float2 E = make_float2(0.f, 0.f);
      for (int y = y0; y <= y1; ++y) {
        const int e = T.boff[y * T.G + x1 + 1];
        for (int p = T.boff[y * T.G + x0]; p < e; ++p) {
          const float2 P = T.uv[p];
          const float dx = P.x - fqx, dy = P.y - fqy;
          if (fmaf(dx, dx, dy * dy) > lim) continue;
          const double d = fma((double)dx, (double)dx, (double)dy * (double)dy);
          if (d < ed || (d == ed && (P.y < E.y || (P.y == E.y && P.x < E.x)))) {
            ed = d;
            E = P;
            best = p;
          }
        }
      }
    }
    return best;
  }
}

// The third vertex of the Delaunay triangle on the left of edge a->b: the
// first point met by a circle through a and b whose centre moves left; none
// if no point lies strictly left of a->b (a->b is a hull edge).
//
// That point sees the edge under the largest angle, so among the points c with
// cross(b - a, c - a) > 0 it has the smallest cotangent
// dot(c - a, c - b) / cross(b - a, c - a).  Both are integers below 2^40,
// exact in double; their quotient is taken in float, with a relative error
// below 3e-7.  Candidates within COT_NEAR of the least one (nearly always one
// alone) are settled by the exact in-circle test with its symbolic
// perturbation.
constexpr float COT_NONE = 3e38f;
constexpr float COT_NEAR = 1e-6f;
__device__ __forceinline__ float cotangent(double dot, double cross) {
  const float fc = (float)cross;
  return fc > 0.f ? (float)dot * __builtin_amdgcn_rcpf(fc) : COT_NONE;
}
__device__ __forceinline__ float cot_limit(float least) { return fmaf(fabsf(least), COT_NEAR, least); }

// Rectangle in units of buckets.
struct Rect {
  float x0, x1, y0, y1;
};

// Where a better point than one of cotangent t can lie, relative to the edge's
// first point, for an edge (ex, ey) of length len: the circle through the edge
// and that point, of which only the part left of the edge counts (for a centre
// on the right the thin cap between the chord and the parallel tangent).  With n
// the edge turned left by 90 degrees, the circle's centre is mid + n t / 2 and
// its radius |n| sqrt(1 + t^2) / 2.
__device__ __forceinline__ Rect circle_box(float ex, float ey, float len, float t) {
  const float u = sqrtf(1.f + t * t);
  if (t > 0.f) {
    const float ox = 0.5f * (ex - t * ey), oy = 0.5f * (ey + t * ex), rho = 0.5f * len * u;
    const float mg = 1e-3f + 2e-6f * rho;
    return Rect{ox - rho - mg, ox + rho + mg, oy - rho - mg, oy + rho + mg};
  }
  const float k = 0.5f / (u - t);  // height of the cap over |n|
  const float nx = -k * ey, ny = k * ex;
  return Rect{fminf(ex, 0.f) + fminf(nx, 0.f) - 1e-3f, fmaxf(ex, 0.f) + fmaxf(nx, 0.f) + 1e-3f,
              fminf(ey, 0.f) + fminf(ny, 0.f) - 1e-3f, fmaxf(ey, 0.f) + fmaxf(ny, 0.f) + 1e-3f};
}

// The search by the lanes of a group.  `best` is the first point met
// among the points of `known` (-1: none there), an empty rectangle if none was
// looked at.
//
// The points are scanned by bucket rows of a square beside the edge that
// grows until it holds every place a better point than the best so far could
// be (circle_box).  Squares and circles only bound the search, in float
// and in units of buckets, with margins far above the float rounding (2e-5
// buckets at 76 buckets a side); each row is also cut at the edge's line.
template <class TT>
__device__ __forceinline__ int third_left(const TT& T, int a, int b, int best, Rect known, int gl) {
  const int2 A = T.uv[a], B = T.uv[b];
  const int iex = B.x - A.x, iey = B.y - A.y;
  const double ex = iex, ey = iey;
  const float fG = (float)T.G;
  const float fex = (float)iex * T.inv, fey = (float)iey * T.inv;
  const float fax = (float)(A.x + T.H) * T.inv, fay = (float)(A.y + T.H) * T.inv;
  const float mx = fax + 0.5f * fex, my = fay + 0.5f * fey, len = sqrtf(fex * fex + fey * fey);
  const float cx = mx - SEARCH_OFFSET * fey, cy = my + SEARCH_OFFSET * fex;  // the square's centre
  float h = fmaxf(SEARCH_SIZE * len, known.x0 <= known.x1 ? 0.5f * (known.x1 - known.x0) : SEARCH_MIN);  // and half side
  // the edge's line: steep enough, it bounds the columns of a row (its float
  // error stays below 0.03 buckets), else (it rises by less than 0.15 buckets
  // over the window) the rows
  const bool steep = fabsf(fey) * 512.f > fabsf(fex);
  const float slope = steep ? fex / fey : 0.f;
  const float line0 = !steep    ? (iey > 0 ? 1e6f : -1e6f)
                      : iey > 0 ? fax - slope * fay + fmaxf(slope, 0.f) + 0.1f
                                : fax - slope * fay + fminf(slope, 0.f) - 0.1f;
  // where a better point can be: the window, then the circle's left part
  Rect box{0.f, fG, !steep && iex > 0 ? fay - 0.25f : 0.f, !steep && iex <= 0 ? fay + 0.25f : fG};
  auto cot_of = [&](int2 P) {
    const double dx = P.x - A.x, dy = P.y - A.y;
    return cotangent(dx * (dx - ex) + dy * (dy - ey), ex * dy - ey * dx);  // a and b themselves: cross 0
  };
  float cot = best >= 0 ? cot_of(T.uv[best]) : COT_NONE;
  auto narrow = [&]() {
    const Rect c = circle_box(fex, fey, len, cot);
    box = Rect{fmaxf(box.x0, fax + c.x0), fminf(box.x1, fax + c.x1), fmaxf(box.y0, fay + c.y0), fminf(box.y1, fay + c.y1)};
  };
  if (best >= 0) {
    narrow();
    if (known.x0 <= box.x0 && known.x1 >= box.x1 && known.y0 <= box.y0 && known.y1 >= box.y1) return best;
  }
  int x0, x1, y0, y1;
  bool tie;
  auto cut = [&](int y, int& xa, int& xb) {
    const int lim = (int)floorf(fminf(fmaxf(line0 + slope * (float)y, -1.f), fG));
    if (iey > 0)
      xb = min(xb, lim);
    else
      xa = max(xa, lim);
  };
  for (;;) {
    x0 = max((int)floorf(fmaxf(cx - h, box.x0)), 0);
    x1 = min((int)floorf(fminf(cx + h, box.x1)), T.G - 1);
    y0 = max((int)floorf(fmaxf(cy - h, box.y0)), 0);
    y1 = min((int)floorf(fminf(cy + h, box.y1)), T.G - 1);
    // the two least cotangents of a lane and the point of the least
    float second = COT_NONE;
    cot = COT_NONE;
    best = INT_MAX;
    row_scan(T, x0, x1, y0, y1, gl, cut, [&](const int* p, const int2* Q, int n) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float q = j < n ? cot_of(Q[j]) : COT_NONE;
        second = fminf(second, fmaxf(cot, q));
        best = q < cot ? p[j] : best;
        cot = fminf(cot, q);
      }
    });
    const float least = group_min(cot), lim = cot_limit(least);
    const uint32_t near = group_ballot(cot <= lim);
    if (!(least < COT_NONE)) {
      best = -1;
    } else {
      tie = (near & (near - 1)) != 0 || group_ballot(second <= lim) != 0;
      best = group_reduce(cot <= lim ? best : INT_MAX, [](int u, int v) { return min(u, v); });
      cot = least;
      narrow();
    }
    if (cx - h <= box.x0 && cx + h >= box.x1 && cy - h <= box.y0 && cy + h >= box.y1) break;
    h *= 4.f;
  }
  if (best < 0 || !tie) return best;
  // near ties: exactly, one after the other, the same in all lanes of the group
  const float lim = cot_limit(cot);
  best = -1;
  for (int y = y0; y <= y1; ++y) {
    int xa = x0, xb = x1;
    cut(y, xa, xb);
    if (xa > xb) continue;
    const int e = T.boff[y * T.G + xb + 1];
    for (int p = T.boff[y * T.G + xa]; p < e; p += STAR_LANES) {
      const bool near = p + gl < e && cot_of(T.uv[min(p + gl, e - 1)]) <= lim;
      for (uint32_t lanes = group_ballot(near); lanes; lanes &= lanes - 1) {
        const int c = p + __builtin_ctz(lanes);
        if (best < 0 || incircle_sos(a, b, best, c, A, B, T.uv[best], T.uv[c]) > 0) best = c;
      }
    }
  }
  return best;
}

__device__ __forceinline__ uint64_t face_key(int a, int b, int c) {
  // rotate so the lowest index comes first (keeps CCW order)
  if (b < a && b < c) {
    const int t = a;
    a = b;
    b = c;
    c = t;
  } else if (c < a && c < b) {
    const int t = c;
    c = b;
    b = a;
    a = t;
  }
  return ((uint64_t)a << 42) | ((uint64_t)b << 21) | (uint64_t)c;
}

// Top-left ownership of an edge P->Q for points exactly on it: equivalent to
// testing the point nudged by an infinitesimal (-1, -delta).
__device__ __forceinline__ bool edge_owned(int px, int py, int qx, int qy) {
  const int dy = qy - py, dx = qx - px;
  return dy > 0 || (dy == 0 && dx < 0);
}

// floor(x / C) for |x| < 2^20 and quotients below 2^13: a float estimate, off by
// at most one, then corrected exactly.
__device__ __forceinline__ int floor_div_i(int x, int C, float rC) {
  const int q = (int)floorf((float)x * rC), r = x - q * C;
  return q + (r >= C) - (r < 0);
}

// texel index range covering [lo, hi] in tile-local raw coordinates
__device__ __forceinline__ void texel_range(int lo, int hi, int H, int C, int R, int& j0, int& j1) {
  const int q0 = -H + C / 2;
  const float rC = __builtin_amdgcn_rcpf((float)C);
  j0 = -floor_div_i(q0 - lo, C, rC);  // ceil((lo - q0) / C)
  j1 = floor_div_i(hi - q0, C, rC);
  if (j0 < 0) j0 = 0;
  if (j1 > R - 1) j1 = R - 1;
}

// A triangle to rasterise: the box of its texels and its three edge functions,
// e + di * i + dj * j at the box's texel (di, dj).  These are integers below
// 2^53, so stepping them over the box is exact; the top-left rule for a texel on
// an edge is a half unit added or taken off, so a texel is inside where all
// three are positive.
struct RasterTri {
  double ea, ai, aj, eb, bi, bj, ec, ci, cj;
  int i0, j0, h, w;  // w 0: no texel
  uint64_t key;
  __device__ __forceinline__ bool inside(double di, double dj) const {
    return fma(di, ai, fma(dj, aj, ea)) > 0. && fma(di, bi, fma(dj, bj, eb)) > 0. && fma(di, ci, fma(dj, cj, ec)) > 0.;
  }
};

template <class TT>
__device__ __forceinline__ RasterTri raster_tri(const TT& T, uint64_t key, int C, int R) {
  RasterTri t;
  const int2 A = T.uv[(int)(key >> 42)], B = T.uv[(int)((key >> 21) & 0x1FFFFF)], Cc = T.uv[(int)(key & 0x1FFFFF)];
  const int ax = A.x, ay = A.y, bx = B.x, by = B.y, cx = Cc.x, cy = Cc.y;
  int i1, j1;
  texel_range(min(ax, min(bx, cx)), max(ax, max(bx, cx)), T.H, C, R, t.j0, j1);
  texel_range(min(ay, min(by, cy)), max(ay, max(by, cy)), T.H, C, R, t.i0, i1);
  t.key = key;
  t.h = i1 - t.i0 + 1;
  t.w = t.h > 0 ? max(j1 - t.j0 + 1, 0) : 0;
  const double qx = -T.H + C / 2 + t.j0 * C, qy = -T.H + C / 2 + t.i0 * C;  // the box's first texel
  t.ea = orient_d(bx, by, cx, cy, qx, qy) + (edge_owned(bx, by, cx, cy) ? 0.5 : -0.5);
  t.eb = orient_d(cx, cy, ax, ay, qx, qy) + (edge_owned(cx, cy, ax, ay) ? 0.5 : -0.5);
  t.ec = orient_d(ax, ay, bx, by, qx, qy) + (edge_owned(ax, ay, bx, by) ? 0.5 : -0.5);
  const double C_d = C;
  t.ai = (cx - bx) * C_d;
  t.aj = (by - cy) * C_d;
  t.bi = (ax - cx) * C_d;
  t.bj = (cy - ay) * C_d;
  t.ci = (bx - ax) * C_d;
  t.cj = (ay - by) * C_d;
  return t;
}

// e / d and the remainder from a float estimate (e < 2^24), corrected exactly.
__device__ __forceinline__ void divide_small(int e, int d, float rd, int& q, int& r) {
  q = (int)((float)e * rd);
  r = e - q * d;
  q += (r >= d) - (r < 0);
  r = e - q * d;
}

// Triangles are not rasterised by the lanes that find them but by groups of this
// many lanes, so rasterisation does not hold up the walks; triangles whose box
// has more texels than RASTER_MAX are left to the whole wave.
constexpr int RASTER_LANES = 8;
constexpr int RASTER_MAX = 64;

// Write the triangle into every texel whose centre lies in it under the top-left
// rule, by a group of lanes: every texel of the box gets the exact test.
__device__ __forceinline__ void raster_box(const RasterTri& t, int R, uint64_t* __restrict__ fm, int lane) {
  const float rw = __builtin_amdgcn_rcpf((float)t.w);
  for (int e = lane; e < t.h * t.w; e += RASTER_LANES) {
    int di, dj;
    divide_small(e, t.w, rw, di, dj);
    if (t.inside(di, dj)) fm[(t.i0 + di) * R + t.j0 + dj] = t.key;
  }
}

// The same for the triangle of lane src, by the whole wave: 8 x 8 texels at a
// time, without those beyond one of the edges (the slivers along the hull of a
// sparse window have boxes of thousands of texels).
__device__ __forceinline__ void raster_wave(const RasterTri& of, int src, int R, uint64_t* __restrict__ fm, int lane) {
  auto get = [&](int v) -> int { return __builtin_amdgcn_readlane(v, src); };
  auto get_d = [&](double v) -> double {
    const uint64_t w = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, (uint64_t)(uint32_t)get((int)(uint32_t)w) |
                                          ((uint64_t)(uint32_t)get((int)(uint32_t)(w >> 32)) << 32));
  };
  RasterTri t;
  t.ea = get_d(of.ea);
  t.ai = get_d(of.ai);
  t.aj = get_d(of.aj);
  t.eb = get_d(of.eb);
  t.bi = get_d(of.bi);
  t.bj = get_d(of.bj);
  t.ec = get_d(of.ec);
  t.ci = get_d(of.ci);
  t.cj = get_d(of.cj);
  t.i0 = get(of.i0);
  t.j0 = get(of.j0);
  t.h = get(of.h);
  t.w = get(of.w);
  t.key = __builtin_bit_cast(uint64_t, get_d(__builtin_bit_cast(double, of.key)));
  // the largest value of an edge function over a block: at one of its corners
  const double ma = t.ea + fmax(7 * t.ai, 0.) + fmax(7 * t.aj, 0.), mb = t.eb + fmax(7 * t.bi, 0.) + fmax(7 * t.bj, 0.),
               mc = t.ec + fmax(7 * t.ci, 0.) + fmax(7 * t.cj, 0.);
  const int nbj = (t.w + 7) / 8, nb = nbj * ((t.h + 7) / 8);
  const float rn = __builtin_amdgcn_rcpf((float)nbj);
  for (int b0 = 0; b0 < nb; b0 += 64) {
    int q, r;
    divide_small(b0 + lane, nbj, rn, q, r);
    const double di = 8 * q, dj = 8 * r;
    uint64_t near = __ballot(b0 + lane < nb && fma(di, t.ai, fma(dj, t.aj, ma)) > 0. &&
                             fma(di, t.bi, fma(dj, t.bj, mb)) > 0. && fma(di, t.ci, fma(dj, t.cj, mc)) > 0.);
    for (; near; near &= near - 1) {
      const int blk = __builtin_ctzll(near);
      const int ti = 8 * __builtin_amdgcn_readlane(q, blk) + (lane >> 3);
      const int tj = 8 * __builtin_amdgcn_readlane(r, blk) + (lane & 7);
      if (ti < t.h && tj < t.w && t.inside(ti, tj)) fm[(t.i0 + ti) * R + t.j0 + tj] = t.key;
    }
  }
}

// Texels lying exactly on hull edge a->b get the triangle next to it (LANES lanes
// take its rows in turn).  Per texel row the line crosses at most one texel
// centre, found exactly in integers.
template <int LANES, class TT>
__device__ void raster_hull_edge(const TT& T, int a, int b, uint64_t key, int C, int R, uint64_t* __restrict__ fm,
                                 int lane) {
  const int2 A = T.uv[a], B = T.uv[b];
  const int ax = A.x, ay = A.y, bx = B.x, by = B.y;
  int i0, i1, j0, j1;
  texel_range(min(ax, bx), max(ax, bx), T.H, C, R, j0, j1);
  texel_range(min(ay, by), max(ay, by), T.H, C, R, i0, i1);
  const int q0 = -T.H + C / 2;
  const int64_t dx = bx - ax, dy = by - ay;
  if (dy == 0) {
    // the edge lies on a texel row only if ay is a row centre (then i0 == i1)
    if (i0 > i1 || q0 + i0 * C != ay) return;
    for (int j = j0 + lane; j <= j1; j += LANES) fm[i0 * R + j] = key;
    return;
  }
  // x = ax + dx * (y - ay) / dy must be an integer texel centre; every
  // quantity is an integer below 2^39, so the double quotient, its rounding
  // and the check of the product are exact
  const double fdx = (double)dx, fdy = (double)dy;
  for (int i = i0 + lane; i <= i1; i += LANES) {
    const double num = fdx * (double)(q0 + i * C - ay);
    const double xr = rint(num / fdy);
    if (xr * fdy != num) continue;
    const int xo = ax + (int)xr - q0;
    if (xo % C) continue;
    const int j = xo / C;
    if (j >= j0 && j <= j1) fm[i * R + j] = key;
  }
}

__device__ int block_scan_excl(int* s, int n, int* s_tmp) {
  const int tid = threadIdx.x;
  const int per = (n + RB - 1) / RB;
  const int beg = min(n, tid * per), end = min(n, beg + per);
  int sum = 0;
  for (int i = beg; i < end; ++i) sum += s[i];
  const int lane = tid & 63, wid = tid >> 6;
  int v = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  if (lane == 63) s_tmp[wid] = v;
  __syncthreads();
  if (tid == 0) {
    int run = 0;
    for (int w = 0; w < RB / 64; ++w) {
      const int t = s_tmp[w];
      s_tmp[w] = run;
      run += t;
    }
    s_tmp[RB / 64] = run;
  }
  __syncthreads();
  int excl = v - sum + s_tmp[wid];
  for (int i = beg; i < end; ++i) {
    const int t = s[i];
    s[i] = excl;
    excl += t;
  }
  const int total = s_tmp[RB / 64];
  __syncthreads();
  return total;
}

__device__ __forceinline__ void write_zero_tile(const ReconParams& P, int k) {
  const int64_t n8 = (int64_t)P.R * P.R * 2;
  float4* o = reinterpret_cast<float4*>(P.x_out + (int64_t)k * P.R * P.R * 8);
  for (int64_t i = threadIdx.x; i < n8; i += RB) o[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Phases a-b, one workgroup per tile: gather, bucket sort, canonical points.
// Bound by the chains of dependent reads (entry, point, attributes) of a tile's
// 512 lanes, so each pass over the points reads PREP_BATCH of them at a time, and
// attributes follow in a pass of their own instead of bucket by bucket: a window
// of 7,000 points 148 -> 123 us (and 1024 tiles of 50-2000 points 116 -> 100).
__global__ void __launch_bounds__(RB) k_recon_prep(ReconParams P) {
  // the raw bucket offsets at the start, the canonical ones at the end, and
  // between them the sort keys and entries of a window that fits
  __shared__ __align__(16) int s_mem[PREP_INTS];
  __shared__ int s_tmp[RB / 64 + 1];
  __shared__ int s_repeats;  // points at positions that others share
  const int tid = threadIdx.x;
  const int R = P.R, H = P.H, W2 = 2 * P.H;
  const int RR = R * R;
  const int k = __builtin_amdgcn_readfirstlane(P.order[P.q0 + blockIdx.x]);
  const int flags = __builtin_amdgcn_readfirstlane((P.flags[0] ? LS_TILE_CAP : 0) | (P.status[k] & LS_TILE_BADID));
  const int32_t off = __builtin_amdgcn_readfirstlane(P.bin_off[k]);
  const int32_t cnt = __builtin_amdgcn_readfirstlane((flags & (LS_TILE_CAP | LS_TILE_BADID)) ? 0 : P.bin_off[k + 1] - off);
  const int32_t t = __builtin_amdgcn_readfirstlane(P.tile_list[k]);
  __syncthreads();  // the status has been read by every wave
  if (cnt == 0) {
    write_zero_tile(P, k);
    if (tid == 0) {
      P.cz_out[k] = 0.0;
      P.status[k] = flags | LS_TILE_EMPTY;
      P.npts[k] = 0;
    }
    return;
  }
  // texels without a triangle until the stars fill them in
  if (P.facemap) {
    uint64_t* __restrict__ fm = P.facemap + (int64_t)blockIdx.x * RR;
    for (int tt = tid; tt < RR; tt += RB) fm[tt] = FACE_NONE;
  }
  const int64_t cx = P.ox + (int64_t)(t % P.tiles_x) * P.S + P.S / 2;
  const int64_t cy = P.oy + (int64_t)(t / P.tiles_x) * P.S + P.S / 2;
  const int G = bucket_side(cnt), NB = G * G;
  int* s_b = s_mem;
  int* s_k = s_mem + PREP_INTS - (NB + 1);
  // ---- a. gather + bucket histogram
  if (tid == 0) s_repeats = 0;
  for (int b = tid; b <= NB; b += RB) s_b[b] = 0;
  __syncthreads();
  for (int e0 = tid; e0 < cnt; e0 += PREP_BATCH * RB) {
    int32_t gi[PREP_BATCH], x[PREP_BATCH], y[PREP_BATCH];
#pragma unroll
    for (int j = 0; j < PREP_BATCH; ++j) gi[j] = P.bin_idx[off + min(e0 + j * RB, cnt - 1)];
#pragma unroll
    for (int j = 0; j < PREP_BATCH; ++j) {
      x[j] = P.x[gi[j]];
      y[j] = P.y[gi[j]];
    }
#pragma unroll
    for (int j = 0; j < PREP_BATCH; ++j) {
      const int e = e0 + j * RB;
      if (e >= cnt) break;
      const int u = (int)((int64_t)x[j] - cx), v = (int)((int64_t)y[j] - cy);
      P.su[off + e] = u;
      P.sv[off + e] = v;
      const int b = bucket_1d(v + H, G, W2) * G + bucket_1d(u + H, G, W2);
      P.sslot[off + e] = atomicAdd(&s_b[b], 1);
    }
  }
  __syncthreads();
  block_scan_excl(s_b, NB + 1, s_tmp);
  // Scatter (v, u) and the entry into bucket order, sort every bucket by
  // (v, u), drop repeated positions and write the canonical points: of the
  // points at one position the largest (z, R, G, B).
  auto key_of = [](int u, int v) -> uint64_t {
    return ((uint64_t)(uint32_t)(v + (1 << 20)) << 32) | (uint32_t)(u + (1 << 20));
  };
  auto top_of = [&](int32_t gi) -> unsigned long long {  // (z, R, G) as an ascending key
    const uint16_t* c3 = P.rgb + 3 * (int64_t)gi;
    return ((unsigned long long)((uint32_t)P.z[gi] ^ 0x80000000u) << 32) | ((uint32_t)c3[0] << 16) | c3[1];
  };
  auto bucket_sort = [&](uint64_t* __restrict__ key, int* __restrict__ idx) -> int {
    for (int e0 = tid; e0 < cnt; e0 += PREP_BATCH * RB) {
      int u[PREP_BATCH], v[PREP_BATCH], slot[PREP_BATCH];
#pragma unroll
      for (int j = 0; j < PREP_BATCH; ++j) {
        const int e = min(e0 + j * RB, cnt - 1);
        u[j] = P.su[off + e];
        v[j] = P.sv[off + e];
        slot[j] = P.sslot[off + e];
      }
#pragma unroll
      for (int j = 0; j < PREP_BATCH; ++j) {
        const int e = e0 + j * RB;
        if (e >= cnt) break;
        const int b = bucket_1d(v[j] + H, G, W2) * G + bucket_1d(u[j] + H, G, W2);
        const int pos = s_b[b] + slot[j];
        key[pos] = key_of(u[j], v[j]);
        idx[pos] = e;
      }
    }
    __syncthreads();
    // ---- b. per-bucket sort + dedupe
    if (tid == 0) s_k[NB] = 0;
    for (int b = tid; b < NB; b += RB) {
      const int lo = s_b[b], hi = s_b[b + 1];
      int kept = hi > lo ? 1 : 0;
      for (int i = lo + 1; i < hi; ++i) {
        const uint64_t kk = key[i];
        const int e = idx[i];
        int j = i - 1;
        while (j >= lo && kk < key[j]) {
          key[j + 1] = key[j];
          idx[j + 1] = idx[j];
          --j;
        }
        key[j + 1] = kk;
        idx[j + 1] = e;
      }
      for (int i = lo + 1; i < hi; ++i) kept += key[i] != key[i - 1];
      s_k[b] = kept;
    }
    __syncthreads();
    const int mm = __builtin_amdgcn_readfirstlane(block_scan_excl(s_k, NB + 1, s_tmp));
    for (int b = tid; b < NB; b += RB) {
      const int lo = s_b[b], hi = s_b[b + 1];
      int w = off + s_k[b];
      for (int i = lo; i < hi; ++i)
        if (i == lo || key[i] != key[i - 1]) {
          const uint64_t kk = key[i];
          P.cuv[w] = make_int2((int)(uint32_t)kk - (1 << 20), (int)(uint32_t)(kk >> 32) - (1 << 20));
          P.sslot[w] = idx[i];  // the slots have been used
          ++w;
        }
    }
    if (mm < cnt)  // and so have the coordinates: entries at repeated positions and their points
      for (int b = tid; b < NB; b += RB) {
        const int hi = s_b[b + 1];
        for (int i = s_b[b], w = s_k[b]; i < hi; ++w) {
          int j = i + 1;
          while (j < hi && key[j] == key[i]) ++j;
          if (j - i > 1)
            for (int at = off + atomicAdd(&s_repeats, j - i); i < j; ++i, ++at) {
              P.su[at] = idx[i];
              P.sv[at] = w;
            }
          i = j;
        }
      }
    __syncthreads();
    for (int w0 = tid; w0 < mm; w0 += PREP_BATCH * RB) {
      int32_t gi[PREP_BATCH];
      int4 at[PREP_BATCH];
#pragma unroll
      for (int j = 0; j < PREP_BATCH; ++j) gi[j] = P.sslot[off + min(w0 + j * RB, mm - 1)];
#pragma unroll
      for (int j = 0; j < PREP_BATCH; ++j) gi[j] = P.bin_idx[off + gi[j]];
#pragma unroll
      for (int j = 0; j < PREP_BATCH; ++j) {
        const uint16_t* c3 = P.rgb + 3 * (int64_t)gi[j];
        at[j] = make_int4(P.z[gi[j]], c3[0], c3[1], c3[2]);
      }
#pragma unroll
      for (int j = 0; j < PREP_BATCH; ++j)
        if (w0 + j * RB < mm) P.cattr[off + w0 + j * RB] = at[j];
    }
    // Repeated positions: the maximum of (z, R, G) over a position's entries, then
    // of B among those that reach it, in the space of the keys.  1000 points at
    // one position 0.42 ms; sorted with the positions, by one lane a bucket with two
    // dependent reads a comparison, 63 ms.
    if (mm < cnt) {
      const int repeats = s_repeats;
      unsigned long long* top = reinterpret_cast<unsigned long long*>(key);
      for (int r = tid; r < repeats; r += RB) {
        __hip_atomic_store(top + P.sv[off + r], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(idx + P.sv[off + r], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      for (int r = tid; r < repeats; r += RB) atomicMax(top + P.sv[off + r], top_of(P.bin_idx[off + P.su[off + r]]));
      __syncthreads();
      for (int r = tid; r < repeats; r += RB) {
        const int32_t gi = P.bin_idx[off + P.su[off + r]], w = P.sv[off + r];
        if (__hip_atomic_load(top + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == top_of(gi))
          atomicMax(idx + w, (int)P.rgb[3 * (int64_t)gi + 2]);
      }
      __syncthreads();
      for (int r = tid; r < repeats; r += RB) {
        const int w = P.sv[off + r];
        const unsigned long long v = __hip_atomic_load(top + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        P.cattr[off + w] = make_int4((int)((uint32_t)(v >> 32) ^ 0x80000000u), (int)((v >> 16) & 0xFFFF), (int)(v & 0xFFFF),
                                     __hip_atomic_load(idx + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      }
    }
    return mm;
  };
  const int a0 = (NB + 2) & ~1;  // keys 8-byte aligned behind the raw offsets
  int m;
  if (a0 + 3 * cnt <= PREP_INTS - (NB + 1))
    m = bucket_sort(reinterpret_cast<uint64_t*>(s_mem + a0), s_mem + a0 + 2 * cnt);
  else
    m = bucket_sort(P.skey + off, P.sidx + off);
  for (int b = tid; b <= NB; b += RB) P.boff[2 * (int64_t)off + b] = s_k[b];
  __syncthreads();
  // collinearity check
  bool noncol = false;
  if (m >= 3) {
    const int2 p0 = P.cuv[off], p1 = P.cuv[off + 1];
    for (int p = tid; p < m; p += RB) {
      const int2 q = P.cuv[off + p];
      if (orient_d(p0.x, p0.y, p1.x, p1.y, q.x, q.y) != 0.0) noncol = true;
    }
  }
  // face keys pack three point indices in 21 bits each
  const bool big = m >= (1 << 21);
  const bool dt = __syncthreads_or(noncol) != 0 && !big;
  if (tid == 0) {
    P.npts[k] = m;
    P.status[k] = flags | (dt ? 0 : LS_TILE_NN_ONLY) | (big ? LS_TILE_DEGENERATE : 0);
  }
  if (dt) {
    const int n = (m + P.item - 1) / P.item;
    if (tid == 0) s_tmp[0] = atomicAdd(P.item_n, n);
    __syncthreads();
    for (int i = tid; i < n; i += RB) P.items[s_tmp[0] + i] = make_int2(blockIdx.x, i * P.item);
  }
}

// Phase c: the Delaunay triangles and their texels, by work items of P.item
// canonical points that the waves of the launch take from a list.
//
// Eight lanes work on one point.  About forty points around it are gathered
// once, CAND to a lane.  A triangle belongs to the lowest of its vertices, by
// (v, u): so the walk around a point a visits the neighbours above it only,
// counter-clockwise from the first point met by a circle that grows upwards
// from a (tangent to a's row, its inside empty: a Delaunay edge) to the first
// triangle that reaches below a, then clockwise; a hull edge is left to its
// lower end.  Where that start is not proven by the gathered points, the nearest
// neighbour takes its place, and the walk may pass points below a first.
//
// A step takes every candidate's cotangent and its minimum over the group,
// without a branch or a global access on the way; the answer stands if the
// circle through it lies in the gathered square, else third_left goes on from
// it (one step in twenty).  The wave collects its triangles and rasterises them
// together.
//
// Of the 1.15 ms that 1.2 M points of 1024 tiles take, the steps are 0.5, the
// searches beyond the candidates 0.35 and the gather 0.18, all bound by
// instruction issue and by the chain of dependent reads.  A search by one lane
// over the buckets, with the answers shared between stars, takes fewer
// instructions but leaves the lanes of a wave waiting for its longest search
// (1.8 ms); sixteen lanes with 5 candidates each took 1.5 ms, all neighbours
// instead of those above 40 % more steps.  Three waves per SIMD: four spill (8 %
// slower with the largest tiles).  Items of 16 points: 8 and 32 are 1 and 5 %
// slower; with up to 64 tiles 8, what a wave works on at once.
__global__ void __launch_bounds__(TB, 3) k_recon_stars(ReconParams P) {
  __shared__ int2 s_d[TB / STAR_LANES][CANDS];  // candidates: position relative to the centre
  __shared__ int s_id[TB / STAR_LANES][CANDS];  // and index
  __shared__ uint64_t s_tri[TB / 64][TRI_CAP];
  __shared__ int s_ntri[TB / 64];
  const int tid = threadIdx.x, wave = tid >> 6, gl = tid & (STAR_LANES - 1);
  const int R = P.R, C = P.C;
  int2* __restrict__ list_d = s_d[tid / STAR_LANES];
  int* __restrict__ list_id = s_id[tid / STAR_LANES];
  auto wave_sync = []() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if ((tid & 63) == 0) s_ntri[wave] = 0;
  wave_sync();
  const int n_items = __builtin_amdgcn_readfirstlane(P.item_n[0]);
  // The items are cut into a range per XCD (the items of a tile lie together, so
  // its points stay in that XCD's L2).  A wave's first item follows from its
  // number, the others from the range's counter, then from the next ranges'.  One
  // counter for all took 0.8 ms for 75,000 items, unevenly long items in turn
  // without a counter 25 % more than this.
  const int per_range = gridDim.x / XCDS * (TB / 64);  // waves of a range
  int range = blockIdx.x % XCDS, tries = 0;
  auto begin_of = [&](int x) { return (int)((int64_t)n_items * x / XCDS); };
  auto next_item = [&]() -> int {
    if (n_items <= XCDS * per_range) return -1;
    for (; tries < XCDS; ++tries) {
      int i = 0;
      if ((tid & 63) == 0) i = atomicAdd(P.item_n + ITEM_COUNTER * (1 + range), 1);
      i = begin_of(range) + per_range + __builtin_amdgcn_readfirstlane(i);
      if (i < begin_of(range + 1)) return i;
      range = (range + 1) % XCDS;
    }
    return -1;
  };
  int it = begin_of(range) + __builtin_amdgcn_readfirstlane(blockIdx.x / XCDS * (TB / 64) + wave);
  if (it >= begin_of(range + 1)) it = next_item();
  for (; it >= 0; it = next_item()) {
    const int2 item = P.items[it];
    const int pos = __builtin_amdgcn_readfirstlane(item.x), begin = __builtin_amdgcn_readfirstlane(item.y);
    const int k = __builtin_amdgcn_readfirstlane(P.order[P.q0 + pos]);
    const int m = __builtin_amdgcn_readfirstlane(P.npts[k]);
    const int off = __builtin_amdgcn_readfirstlane(P.bin_off[k]);
    const int cnt = __builtin_amdgcn_readfirstlane(P.bin_off[k + 1]) - off;
    uint64_t* __restrict__ fm = P.facemap + (int64_t)pos * R * R;
    typedef TileT<UvGlobal, const int32_t*> TT;
    TT T;
    T.uv = UvGlobal{P.cuv + off};
    T.boff = P.boff + 2 * (int64_t)off;
    T.G = bucket_side(cnt);
    T.H = P.H;
    T.W2 = 2 * P.H;
    T.inv = (float)T.G / (float)T.W2;
    const int G = T.G, end = min(begin + P.item, m);
    for (int a0 = begin; a0 < end; a0 += 64 / STAR_LANES) {
      const int a = a0 + (tid & 63) / STAR_LANES;
      if (a < end) {
        const int2 A = T.uv[a];
        const int bx = bucket_1d(A.x + T.H, G, T.W2), by = bucket_1d(A.y + T.H, G, T.W2);
        // ---- gather: the points of the (2 r + 1)^2 buckets around a, r from
        // the density of 7 x 7 buckets, at most CANDS points
        int r = 3, held = 0, first_p[2], len[2];  // bucket rows gl and gl + 8 of the square
        auto count = [&]() {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int y = by - r + gl + STAR_LANES * h;
            len[h] = 0;
            if (y >= 0 && y <= min(by + r, G - 1)) {
              first_p[h] = T.boff[y * G + max(bx - r, 0)];
              len[h] = T.boff[y * G + min(bx + r, G - 1) + 1] - first_p[h];
            }
          }
          held = group_reduce(len[0] + len[1], [](int u, int v) { return u + v; });
        };
        count();
        r = min(max((int)(3.5f * sqrtf(CANDS * 0.85f / (float)held)), 1), 7);
        for (;; --r) {
          count();
          if (held <= CANDS) break;
          held = 0;
          if (r == 0) break;
        }
        const float fx = (float)(A.x + T.H) * T.inv, fy = (float)(A.y + T.H) * T.inv;
        Rect known{1.f, 0.f, 1.f, 0.f};  // what has been gathered, open at the window's borders
        float reach2 = 0.f;              // squared distance from the centre that it covers
        if (held) {
          const int at = group_before(len[0] + len[1], gl);
          for (int j = 0; j < len[0]; ++j) list_id[at + j] = first_p[0] + j;
          for (int j = 0; j < len[1]; ++j) list_id[at + len[0] + j] = first_p[1] + j;
          known = Rect{bx - r > 0 ? (float)(bx - r) : -16.f, bx + r < G - 1 ? (float)(bx + r + 1) : G + 16.f,
                       by - r > 0 ? (float)(by - r) : -16.f, by + r < G - 1 ? (float)(by + r + 1) : G + 16.f};
          const float reach =
              (fminf(fminf(fx - known.x0, known.x1 - fx), fminf(fy - known.y0, known.y1 - fy)) - 1e-3f) / T.inv;
          reach2 = reach > 0.f ? reach * reach * 0.99999f : 0.f;
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          for (int e = gl; e < held; e += STAR_LANES) {
            const int2 Q = T.uv[list_id[e]];
            list_d[e] = make_int2(Q.x - A.x, Q.y - A.y);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        // ---- walk
        int b0 = -1, b = -1, steps = 0;
        int2 B = make_int2(0, 0), B0 = B;            // b and b0 relative to a
        int f1 = -1, f_prev = -1, f_hull = -1;       // counter-clockwise: first third vertex, last b, b at the hull
        int b1 = -1, b_prev = -1, b_hull = -1;       // and clockwise
        bool back = false, done = false;
        uint64_t rest = FACE_NONE;
        auto above = [](int2 D) { return D.y > 0 || (D.y == 0 && D.x > 0); };
        auto turn = [&]() {
          back = true;
          b = b0;
          B = B0;
        };
        // one step on, c the third vertex of the current edge (-1: none), D its
        // position relative to a
        auto advance = [&](int c, int2 D) {
          const bool up = above(B);
          if (c < 0) {
            if (back) {
              if (up) b_hull = b;
              done = true;
            } else {
              if (up) f_hull = b;
              turn();
            }
            return;
          }
          const bool cup = above(D);
          if (up && cup) {
            const uint64_t key = back ? face_key(b, a, c) : face_key(a, b, c);
            int slot = 0;
            if (gl == 0) slot = atomicAdd(&s_ntri[wave], 1);
            slot = group_first(slot);
            if (slot >= TRI_CAP)
              rest = key;  // no room: rasterised at once
            else if (gl == 0)
              s_tri[wave][slot] = key;
          }
          if (back) {
            b1 = b1 < 0 ? c : b1;
            b_prev = b;
          } else {
            f1 = f1 < 0 ? c : f1;
            f_prev = b;
          }
          b = c;
          B = D;
          if (up && !cup) {  // past the points above a
            if (back || !above(B0))
              done = true;
            else
              turn();
          } else if (!back && b == b0) {
            done = true;
          }
          if (!done && ++steps >= STAR_MAX_STEPS) {
            if (gl == 0) atomicOr(&P.status[k], LS_TILE_DEGENERATE);
            done = true;
          }
        };
        // The candidates are read again after the rare calls below: registers
        // that live across them would halve the waves in flight.
        while (!done) {
          int c = -1;
          bool tie = held == 0;  // near ties: settled by an exact scan of the circle
          if (held) {
            double dx[CAND], dy[CAND], l2[CAND];
#pragma unroll
            for (int s = 0; s < CAND; ++s) {
              const int e = gl + STAR_LANES * s;
              const int2 D = e < held ? list_d[e] : make_int2(0, 0);
              dx[s] = D.x;
              dy[s] = D.y;
              l2[s] = fma(dx[s], dx[s], dy[s] * dy[s]);
            }
            if (b0 < 0) {
              // first edge: the circle's diameter through a candidate is its
              // l2 / dy, the cotangent of a horizontal edge
              float cot[CAND], least = COT_NONE;
#pragma unroll
              for (int s = 0; s < CAND; ++s) {
                cot[s] = cotangent(l2[s], dy[s]);
                least = fminf(least, cot[s]);
              }
              least = group_min(least);
              const float lim = cot_limit(least);
              int n = 0, e = 0;
#pragma unroll
              for (int s = 0; s < CAND; ++s) {
                const bool hit = cot[s] <= lim;
                e = hit ? gl + STAR_LANES * s : e;
                n += hit;
              }
              const uint32_t hits = group_ballot(n > 0), many = group_ballot(n > 1);
              if (least * least <= reach2 && many == 0 && (hits & (hits - 1)) == 0) {
                e = group_reduce(n > 0 ? e : INT_MAX, [](int u, int v) { return min(u, v); });
                b0 = b = list_id[e];
                B = B0 = list_d[e];
              }
            }
            while (b0 >= 0) {
              // the third vertex left of a->b, or of b->a
              const double ex = B.x, ey = B.y, sx = back ? -ex : ex, sy = back ? -ey : ey;
              float cot[CAND], least = COT_NONE;
#pragma unroll
              for (int s = 0; s < CAND; ++s) {
                cot[s] = cotangent(fma(-ex, dx[s], fma(-ey, dy[s], l2[s])), fma(sx, dy[s], -(sy * dx[s])));
                least = fminf(least, cot[s]);
              }
              least = group_min(least);
              c = -1;
              if (!(least < COT_NONE)) break;
              const float lim = cot_limit(least);
              int n = 0, e = 0;
#pragma unroll
              for (int s = 0; s < CAND; ++s) {
                const bool hit = cot[s] <= lim;
                e = hit ? gl + STAR_LANES * s : e;
                n += hit;
              }
              const uint32_t hits = group_ballot(n > 0), many = group_ballot(n > 1);
              e = group_reduce(n > 0 ? e : INT_MAX, [](int u, int v) { return min(u, v); });
              c = list_id[e];
              const int2 D = list_d[e];
              tie = many != 0 || (hits & (hits - 1)) != 0;
              if (tie) break;
              const float len2 = (float)fma(ex, ex, ey * ey);
              if (!(fmaf(len2 * least, least, len2) <= reach2)) {
                const float fex = (float)B.x * T.inv, fey = (float)B.y * T.inv;
                const Rect box = back ? circle_box(-fex, -fey, sqrtf(len2) * T.inv, least)
                                      : circle_box(fex, fey, sqrtf(len2) * T.inv, least);
                const float px = back ? fx + fex : fx, py = back ? fy + fey : fy;
                if (!(known.x0 <= px + box.x0 && known.x1 >= px + box.x1 && known.y0 <= py + box.y0 &&
                      known.y1 >= py + box.y1))
                  break;
              }
              advance(c, D);
              c = -1;
              if (done || rest != FACE_NONE) break;
            }
          }
          if (b0 < 0) {
            b0 = b = nearest_of_point(T, a, gl);
            const int2 Q = T.uv[b];
            B = B0 = make_int2(Q.x - A.x, Q.y - A.y);
            if (held) continue;
          }
          if (!done && rest == FACE_NONE) {
            c = third_left(T, back ? b : a, back ? a : b, c, tie ? Rect{1.f, 0.f, 1.f, 0.f} : known, gl);
            const int2 Q = T.uv[max(c, 0)];
            advance(c, make_int2(Q.x - A.x, Q.y - A.y));
          }
          if (rest != FACE_NONE) {
            raster_box(raster_tri(T, rest, C, R), R, fm, gl);
            rest = FACE_NONE;
          }
        }
        // a hull edge's triangle: the last one before it, or the first of the
        // other direction
        if (f_hull >= 0 && (f_prev >= 0 || b1 >= 0))
          raster_hull_edge<STAR_LANES>(T, a, f_hull, f_prev >= 0 ? face_key(a, f_prev, f_hull) : face_key(b0, a, b1), C, R,
                                       fm, gl);
        if (b_hull >= 0 && (b_prev >= 0 || f1 >= 0))
          raster_hull_edge<STAR_LANES>(T, b_hull, a, b_prev >= 0 ? face_key(b_prev, a, b_hull) : face_key(a, b0, f1), C, R,
                                       fm, gl);
      }
      // ---- raster
      wave_sync();
      const int ntri = min(__builtin_amdgcn_readfirstlane(*(volatile int*)&s_ntri[wave]), TRI_CAP);
      if (ntri >= TRI_CAP / 2 || a0 + 64 / STAR_LANES >= end) {
        for (int i0 = 0; i0 < ntri; i0 += 64 / RASTER_LANES) {
          const int i = i0 + (tid & 63) / RASTER_LANES;
          const RasterTri t = raster_tri(T, s_tri[wave][min(i, ntri - 1)], C, R);
          const bool large = i < ntri && t.h * t.w > RASTER_MAX;
          if (i < ntri && !large) raster_box(t, R, fm, tid & (RASTER_LANES - 1));
          for (uint64_t left = __ballot(large && (tid & (RASTER_LANES - 1)) == 0); left; left &= left - 1)
            raster_wave(t, __builtin_ctzll(left), R, fm, tid & 63);
        }
        wave_sync();
        if ((tid & 63) == 0) s_ntri[wave] = 0;
      }
      wave_sync();
    }
  }
}

// Phases d-e, `parts` workgroups per tile: nearest point of every texel,
// interpolation, normalisation and output, 8 x 8 texels per wave at a time.
// Bound by instruction issue (the 1024-tile batch's 302 MB leave in 217 us, at
// the rate of a fill in 45).  Heights and colours are read from global memory,
// one 16-byte record a point: in LDS with the coordinates they left three waves
// per SIMD (now five), which with the nearest points in double took 407 us.
__global__ void __launch_bounds__(TB) k_recon_out(ReconParams P, int parts) {
  __shared__ __align__(16) int s_mem[OUT_INTS];
  __shared__ double s_cz, s_d[TB];
  __shared__ int s_i[TB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int pos = blockIdx.x / parts, part = blockIdx.x - pos * parts;
  const int k = __builtin_amdgcn_readfirstlane(P.order[P.q0 + pos]);
  const int m = __builtin_amdgcn_readfirstlane(P.npts[k]);
  if (m == 0) return;
  const int off = __builtin_amdgcn_readfirstlane(P.bin_off[k]);
  const int cnt = __builtin_amdgcn_readfirstlane(P.bin_off[k + 1]) - off;
  const int R = P.R, C = P.C;
  const int G = bucket_side(cnt), NB = G * G;
  const bool faces = P.facemap != nullptr;
  const uint64_t* __restrict__ fm = P.facemap + (int64_t)pos * R * R;
  // coordinates, three far points, bucket offsets
  const bool lds = 2 * (m + 3) + NB + 1 <= OUT_INTS;
  int32_t* s_off = s_mem + 2 * (m + 3);
  if (lds) {
    float2* uv = reinterpret_cast<float2*>(s_mem);
    for (int p = tid; p < m; p += TB) {
      const int2 Q = P.cuv[off + p];
      uv[p] = make_float2((float)Q.x, (float)Q.y);
    }
    if (tid < 3) uv[m + tid] = make_float2(1e9f, 1e9f);
    for (int b = tid; b <= NB; b += TB) s_off[b] = P.boff[2 * (int64_t)off + b];
  }
  __syncthreads();
  const int4* __restrict__ attr = P.cattr + off;
  auto run = [&](auto uvp, auto bp) {
    TileT<decltype(uvp), decltype(bp)> T;
    T.uv = uvp;
    T.boff = bp;
    T.G = G;
    T.H = P.H;
    T.W2 = 2 * P.H;
    T.inv = (float)G / (float)T.W2;
    const int q0 = -P.H + C / 2;
    // height (metres) and colours of texel (i, j): linear in its triangle, or
    // its nearest point's
    auto lin_value = [&](int i, int j, uint64_t f, int4 near, double* out4) {
      if (f == FACE_NONE) {
        out4[0] = (double)near.x * P.scale_z + P.offset_z;
        out4[1] = near.y;
        out4[2] = near.z;
        out4[3] = near.w;
        return;
      }
      const int a = (int)(f >> 42), b = (int)((f >> 21) & 0x1FFFFF), c = (int)(f & 0x1FFFFF);
      const float2 A = T.uv[a], B = T.uv[b], Cc = T.uv[c];
      const int4 va = attr[a], vb = attr[b], vc = attr[c];
      const double qx = q0 + j * C, qy = q0 + i * C;
      const double ob = orient_d(Cc.x, Cc.y, A.x, A.y, qx, qy);
      const double oc = orient_d(A.x, A.y, B.x, B.y, qx, qy);
      const double O = orient_d(A.x, A.y, B.x, B.y, Cc.x, Cc.y);
      const double lb = ob / O, lc = oc / O;
      auto mix = [&](double x, double y, double z) { return x + lb * (y - x) + lc * (z - x); };
      out4[0] = mix(va.x, vb.x, vc.x) * P.scale_z + P.offset_z;
      out4[1] = mix(va.y, vb.y, vc.y);
      out4[2] = mix(va.z, vb.z, vc.z);
      out4[3] = mix(va.w, vb.w, vc.w);
    };
    // c_z: the centre texel; outside the hull (sparse windows) its nearest
    // point is searched by all lanes
    const int ic = R / 2;
    const uint64_t fc = faces ? fm[ic * R + ic] : FACE_NONE;
    int pc = -1;
    if (__builtin_amdgcn_readfirstlane((int)(fc == FACE_NONE))) {
      const int qc = q0 + ic * C;
      double bd = 1e300;
      auto less = [&](double d, int p, double d2, int p2) -> bool {
        if (p2 < 0 || d != d2) return p2 < 0 || d < d2;
        const float2 A = T.uv[p], B = T.uv[p2];
        return A.y < B.y || (A.y == B.y && A.x < B.x);
      };
      for (int p = tid; p < m; p += TB) {
        const float2 Q = T.uv[p];
        const double dx = (double)Q.x - qc, dy = (double)Q.y - qc;
        const double d = fma(dx, dx, dy * dy);
        if (less(d, p, bd, pc)) {
          bd = d;
          pc = p;
        }
      }
      s_d[tid] = bd;
      s_i[tid] = pc;
      __syncthreads();
      if (tid == 0)
        for (int i = 1; i < TB; ++i)
          if (s_i[i] >= 0 && less(s_d[i], s_i[i], bd, pc)) {
            bd = s_d[i];
            pc = s_i[i];
          }
    }
    if (tid == 0) {
      double v4[4];
      lin_value(ic, ic, fc, attr[max(pc, 0)], v4);
      s_cz = v4[0];
      if (part == 0) P.cz_out[k] = v4[0];
    }
    __syncthreads();
    const double cz = s_cz;
    float4* __restrict__ out = reinterpret_cast<float4*>(P.x_out + (int64_t)k * R * R * 8);
    const int nbs = (R + 7) / 8;
    // a lane's texel in the wave's 8 x 8 block: 4 x 4 sub-blocks of 16 lanes
    const int sub = lane >> 4, di = 4 * (sub >> 1), dj = 4 * (sub & 1);
    for (int blk = part * (TB / 64) + (tid >> 6); blk < nbs * nbs; blk += parts * (TB / 64)) {
      const int bi = blk / nbs, i0 = 8 * bi + di, j0 = 8 * (blk - bi * nbs) + dj;
      const int i = i0 + ((lane >> 2) & 3), j = j0 + (lane & 3);
      const bool in_grid = i < R && j < R;
      const uint64_t f = in_grid && faces ? fm[i * R + j] : FACE_NONE;
      const int p = nearest_of_texel(T, q0, C, R, min(i0, R - 1), min(j0, R - 1), i, j);
      if (!in_grid) continue;
      const int4 near = attr[p];
      double lv[4];
      lin_value(i, j, f, near, lv);
      const double hn = (double)near.x * P.scale_z + P.offset_z;
      const double k65 = 1.0 / 65535.0;
      const int tt = i * R + j;
      out[2 * tt] = make_float4((float)((lv[0] - cz) * P.inv_r), (float)((hn - cz) * P.inv_r), (float)(lv[1] * k65),
                                (float)(lv[2] * k65));
      out[2 * tt + 1] = make_float4((float)(lv[3] * k65), (float)((double)near.y * k65), (float)((double)near.z * k65),
                                    (float)((double)near.w * k65));
    }
  };
  if (lds)
    run(UvfLds{(LdsU64)s_mem}, (LdsI32)s_off);
  else
    run(UvfGlobal{P.cuv + off, m - 1}, (const int32_t*)(P.boff + 2 * (int64_t)off));
}

int g_num_cu = 0;

int num_cus() {
  if (g_num_cu <= 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    g_num_cu = v;
  }
  return g_num_cu;
}

struct ReconLayout {
  int32_t* tile_pos;
  int32_t* counts;
  int32_t* fill;
  int32_t* flags;
  int32_t* order;
  int32_t* bin_off;
  int32_t* bin_idx;
  int32_t* sort_scratch;
  int32_t *su, *sv, *sslot, *sidx;
  uint64_t* skey;
  int4* cattr;
  int2* cuv;
  uint64_t* facemap;
  int64_t face_tiles;  // tiles whose face maps fit
  int2* items;
  int64_t entries;
};

int64_t max_multiplicity(const LsGridInfo& gi) {
  const int64_t per = (2 * (int64_t)gi.H) / gi.S + 1;
  return per * per;
}

// Output workgroups of a tile, each with a block of 8 x 8 texels for its four waves
// at least: about 4,096 in a launch, so that the largest windows do not end last,
// but no more than 36 of a tile (each copies its window's points first: 64 tiles of
// 224 x 224 texels 257 us, with 64 of a tile 261) unless the launch has fewer than
// 2,048 (one tile of 544 x 544 texels and 400 points: 248 us with 36, 190 with all
// its 1,156; of 100,000 points 4.57 and 4.07 ms).
int recon_out_parts(int nt, int R) {
  const int64_t nbs = (R + 7) / 8, most = (nbs * nbs + TB / 64 - 1) / (TB / 64);
  return (int)std::min<int64_t>(most, std::max({2, std::min(36, 4096 / nt), 2048 / nt}));
}

int recon_wg_count(int32_t n_tiles) {
  const int want = 2 * num_cus();
  return n_tiles < want ? (n_tiles > 0 ? n_tiles : 1) : want;
}

// Workspace bytes for n_tiles tiles and n points: 148 bytes per bin entry
// plus 12 R^2 per tile of a launch (at most two per CU count), and the lists.
// These are the sizes and limits callers know; the arrays take less, and the
// rest of the space holds face maps.
size_t recon_bytes(const LsGridInfo& gi, int32_t n_tiles, int64_t n, int nwg) {
  LsArena A{nullptr, 0, 0};
  const int64_t nall = (int64_t)gi.tx * gi.ty;
  const int64_t E = n * max_multiplicity(gi) + 1;
  const int64_t RR = (int64_t)gi.R * gi.R;
  A.take<int32_t>(nall);
  for (int i = 0; i < 2; ++i) A.take<int32_t>(n_tiles + 1);
  A.take<int32_t>(4);
  A.take<int32_t>(n_tiles);
  A.take<int32_t>(n_tiles + 1);
  A.take<int32_t>(E);
  A.take<int32_t>(2 * E);
  for (int i = 0; i < 7; ++i) A.take<int32_t>(E);
  for (int i = 0; i < 3; ++i) A.take<uint64_t>(E);
  A.take<uint64_t>(2 * E);
  A.take<uint64_t>(8 * E);
  A.take<int32_t>(E);
  A.take<uint64_t>(RR * nwg);
  A.take<int32_t>(RR * nwg);
  return A.used;
}

// The arrays in `bytes` bytes at base, the face maps in what they leave.
void recon_layout(const LsGridInfo& gi, int32_t n_tiles, int64_t n, void* base, size_t bytes, ReconLayout* L) {
  LsArena A{reinterpret_cast<char*>(base), 0, 0};
  const int64_t nall = (int64_t)gi.tx * gi.ty;
  const int64_t E = n * max_multiplicity(gi) + 1;
  const int64_t RR = (int64_t)gi.R * gi.R;
  L->tile_pos = A.take<int32_t>(nall);
  L->counts = A.take<int32_t>(n_tiles + 1);
  L->fill = A.take<int32_t>(n_tiles + 1);
  L->flags = A.take<int32_t>(N_FLAGS);  // too many entries; the work items and how many are taken
  L->order = A.take<int32_t>(n_tiles);
  L->bin_off = A.take<int32_t>(n_tiles + 1);
  L->bin_idx = A.take<int32_t>(E);
  L->sort_scratch = A.take<int32_t>(2 * E);
  L->su = A.take<int32_t>(E);
  L->sv = A.take<int32_t>(E);
  L->sslot = A.take<int32_t>(E);
  L->sidx = A.take<int32_t>(E);
  L->skey = A.take<uint64_t>(E);
  L->cattr = A.take<int4>(E);
  L->cuv = A.take<int2>(E);
  L->items = A.take<int2>(E / 3 + 1);
  L->entries = E;
  const size_t at = ls_align(A.used);
  L->face_tiles = at < bytes ? (int64_t)((bytes - at) / (8 * RR)) : 0;
  L->facemap = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(base) + at);
}

// Enqueue the whole recon pipeline with its workspace of ws_bytes at `ws` (the
// caller has checked that it is large enough).
int recon_enqueue(const LsGridInfo& gi, const int32_t* x, const int32_t* y, const int32_t* z, const uint16_t* rgb,
                  int64_t n, const int32_t* tile_list, int32_t n_tiles, int32_t order, float* x_out, double* cz_out,
                  int32_t* bin_off, int32_t* bin_idx, int64_t bin_cap, int32_t* tile_status, void* ws, size_t ws_bytes,
                  hipStream_t st) {
  ReconLayout L;
  recon_layout(gi, n_tiles, n, ws, ws_bytes, &L);
  if (L.face_tiles < 1) return LS_EWORKSPACE;
  const bool user_csr = bin_off && bin_idx;
  int32_t* boff = user_csr ? bin_off : L.bin_off;
  int32_t* bidx = user_csr ? bin_idx : L.bin_idx;
  const int64_t cap = user_csr ? bin_cap : L.entries;
  const int64_t nall = (int64_t)gi.tx * gi.ty;

  const int T = 256;
  LS_TRACE("recon_all", st);
  auto blocks = [&](int64_t cnt) { return (int)std::min<int64_t>((cnt + T - 1) / T, 65535); };
  const int64_t most = std::max<int64_t>(nall, (int64_t)n_tiles + 1);
  hipLaunchKernelGGL(k_recon_init, dim3(blocks(most)), dim3(T), 0, st, L.tile_pos, nall, L.counts, L.fill, tile_status,
                     n_tiles, L.flags);
  hipLaunchKernelGGL(k_tile_pos, dim3(blocks(n_tiles)), dim3(T), 0, st, tile_list, n_tiles, nall, L.tile_pos,
                     tile_status);
  hipLaunchKernelGGL(k_tile_pos_fix, dim3(blocks(most)), dim3(T), 0, st, tile_list, n_tiles, nall, L.tile_pos,
                     tile_status);
  LS_LAUNCH_CHECK();

  BinParams bp;
  bp.ox = gi.ox;
  bp.oy = gi.oy;
  bp.invS = 1.0 / gi.S;
  bp.S = gi.S;
  bp.H = gi.H;
  bp.tiles_x = gi.tx;
  bp.tiles_y = gi.ty;
  bp.K = 1 + gi.H / gi.S;
  bp.n_tiles = n_tiles;
  bp.n = n;
  bp.x = x;
  bp.y = y;
  bp.tile_pos = L.tile_pos;
  bp.counts = L.counts;
  bp.fill = L.fill;
  bp.bin_off = boff;
  bp.bin_idx = bidx;
  bp.cap = cap;
  bp.flags = L.flags;
  bp.order = L.order;
  bp.order_mode = order;
  const int n_face = (int)std::min<int64_t>(n_tiles, (L.entries - 1) / FACE_POINTS);
  bp.n_face = n_face;
  const int pb = (int)std::min<int64_t>((n + T - 1) / T, 8192);
  // workgroup-private histograms when the tile list fits in LDS
  const bool lds_bins = n_tiles <= BIN_LDS_TILES;
  const int64_t chunk = 4096;
  const int nchunks = (int)std::max<int64_t>(1, (n + chunk - 1) / chunk);
  {
    LS_TRACE("bin_count", st);
    if (n > 0) {
      if (lds_bins)
        hipLaunchKernelGGL(k_bin_count_lds, dim3(nchunks), dim3(BIN_THREADS), 0, st, bp, chunk);
      else
        hipLaunchKernelGGL(k_bin_count, dim3(pb > 0 ? pb : 1), dim3(T), 0, st, bp);
    }
  }
  {
    LS_TRACE("bin_scan", st);
    hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(1024), 0, st, bp);
  }
  {
    LS_TRACE("bin_scatter", st);
    if (n > 0) {
      if (lds_bins)
        hipLaunchKernelGGL(k_bin_scatter_lds, dim3(nchunks), dim3(BIN_THREADS), 0, st, bp, chunk);
      else
        hipLaunchKernelGGL(k_bin_scatter, dim3(pb > 0 ? pb : 1), dim3(T), 0, st, bp);
    }
  }
  if (user_csr)
    hipLaunchKernelGGL(k_bin_sort, dim3(std::min(n_tiles, 4 * num_cus())), dim3(RB), 0, st, boff, n_tiles, bidx,
                       L.sort_scratch, L.flags);
  LS_LAUNCH_CHECK();

  ReconParams rp;
  rp.ox = gi.ox;
  rp.oy = gi.oy;
  rp.S = gi.S;
  rp.tiles_x = gi.tx;
  rp.C = gi.C;
  rp.R = gi.R;
  rp.H = gi.H;
  rp.scale_z = gi.scale_z;
  rp.offset_z = gi.offset_z;
  rp.inv_r = 1.0 / ((double)gi.H * gi.scale_xy);
  rp.x = x;
  rp.y = y;
  rp.z = z;
  rp.rgb = rgb;
  rp.tile_list = tile_list;
  rp.bin_off = boff;
  rp.bin_idx = bidx;
  rp.flags = L.flags;
  rp.su = L.su;
  rp.sv = L.sv;
  rp.sslot = L.sslot;
  rp.skey = L.skey;
  rp.sidx = L.sidx;
  rp.cuv = L.cuv;
  rp.cattr = L.cattr;
  rp.boff = L.sort_scratch;  // free once the caller's CSR is sorted
  rp.npts = L.fill;          // free once the points are binned
  rp.items = L.items;
  rp.item_n = L.flags + ITEM_COUNTER;
  rp.order = L.order;
  rp.x_out = x_out;
  rp.cz_out = cz_out;
  rp.status = tile_status;
  {
    LS_TRACE("recon_tile", st);
    // As many tiles at a time as the workspace holds face maps for.  At most
    // n_face windows hold FACE_POINTS points, and these come first; the others
    // are one launch without face maps (16384 tiles with 1000 points in all:
    // 1.16 ms, 1.84 in rounds over every tile).
    for (int q0 = 0; q0 < n_tiles;) {
      const bool faces = q0 < n_face;
      const int nt = (int)std::min<int64_t>(faces ? std::min<int64_t>(n_face - q0, L.face_tiles) : n_tiles - q0, 1 << 20);
      const int parts = recon_out_parts(nt, gi.R);
      rp.q0 = q0;
      rp.facemap = faces ? L.facemap : nullptr;
      // few tiles: a wave takes the points it works on at once
      rp.item = nt <= 64 ? ITEM_MIN : ITEM_MAX;
      if (q0 && faces)
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(T), 0, st, rp.item_n, (int64_t)(N_FLAGS - ITEM_COUNTER), 0);
      hipLaunchKernelGGL(k_recon_prep, dim3(nt), dim3(RB), 0, st, rp);
      if (faces)
        hipLaunchKernelGGL(k_recon_stars, dim3(3 * ((num_cus() + XCDS - 1) / XCDS * XCDS)), dim3(TB), 0, st, rp);
      hipLaunchKernelGGL(k_recon_out, dim3((unsigned)nt * parts), dim3(TB), 0, st, rp, parts);
      q0 += nt;
    }
  }
  LS_LAUNCH_CHECK();
  return LS_OK;
}

}  // namespace

size_t ls_recon_ws_bytes(const LsGridInfo& gi, int32_t n_tiles, int64_t n) {
  return recon_bytes(gi, n_tiles, n, recon_wg_count(n_tiles));
}

// ---------------------------------------------------------------------------
// Allocation-free variant: the workspace is a fixed array in device memory.
// Host code never passes the array's name to a kernel (in host code it is a
// stand-in, not a device address); it takes the address that
// hipGetSymbolAddress returns on each device, once per device.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[LS_RECON_SCRATCH_BYTES];

namespace {

constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[SCRATCH_MAX_DEVICES] = {};

// Device address of `scratch` on the current device (looked up on the first
// call on that device, with the device current).
int scratch_address(void** out) {
  int dev = -1;
  LS_HOST_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) {
    ls_set_last_message("device ordinal beyond the scratch table");
    return LS_EHIP;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      ls_set_last_error(e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)", __LINE__);
      return LS_EHIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return LS_OK;
}

}  // namespace

int ls_recon_noalloc_impl(const LsGridInfo& gi, const int32_t* x, const int32_t* y, const int32_t* z,
                          const uint16_t* rgb, int64_t n, const int32_t* tile_list, int32_t n_tiles, int32_t order,
                          float* x_out, double* cz_out, int32_t* bin_off, int32_t* bin_idx, int64_t bin_cap,
                          int32_t* tile_status, hipStream_t st) {
  if (n_tiles <= 0) return LS_OK;
  if (recon_bytes(gi, n_tiles, n, 1) > LS_RECON_SCRATCH_BYTES) return LS_ESCRATCH;
  void* ws = nullptr;
  const int rc = scratch_address(&ws);
  if (rc != LS_OK) return rc;
  return recon_enqueue(gi, x, y, z, rgb, n, tile_list, n_tiles, order, x_out, cz_out, bin_off, bin_idx, bin_cap,
                       tile_status, ws, LS_RECON_SCRATCH_BYTES, st);
}

int ls_recon_impl(const LsGridInfo& gi, const int32_t* x, const int32_t* y, const int32_t* z, const uint16_t* rgb,
                  int64_t n, const int32_t* tile_list, int32_t n_tiles, int32_t order, float* x_out, double* cz_out,
                  int32_t* bin_off, int32_t* bin_idx, int64_t bin_cap, int32_t* tile_status, void* ws,
                  size_t ws_bytes, hipStream_t st) {
  if (n_tiles <= 0) return LS_OK;
  if (ws_bytes < recon_bytes(gi, n_tiles, n, recon_wg_count(n_tiles)) || !ws) return LS_EWORKSPACE;
  return recon_enqueue(gi, x, y, z, rgb, n, tile_list, n_tiles, order, x_out, cz_out, bin_off, bin_idx, bin_cap,
                       tile_status, ws, ws_bytes, st);
}
