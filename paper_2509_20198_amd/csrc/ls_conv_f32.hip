// FP32 3x3 convolutions of the refinement networks on the matrix cores of
// gfx950: forward layers and input gradients.
//
// v_mfma_f32_16x16x4_f32 is a chain of four IEEE fused multiply-adds in
// order of k (checked bit by bit against fmaf chains, denormals included),
// so a conv whose steps run over (tap, input channel) in ascending order
// gives the same bits as a scalar fmaf loop in that order, at twice the rate
// of the vector units (157 against 79 TFLOP/s without packed FP32).
//
// The product is D[16 output channels][16 pixels] += W[16][4 k] * I[4 k][16
// pixels].  A wave owns one channel tile and NT pixel tiles of 8 x 2 pixels
// (8 x 2 NT pixels); a workgroup is WX x WY waves side by side times WM waves
// over the channels, and stages the input patch of its pixels (with the
// one-texel halo, all input channels, zero outside the plane) in LDS once.
// Pixel tiles are 8 wide because the planes are 96, 48 and 24 wide: 16-wide
// tiles would spend a quarter of the products of the 24-wide ones on padding.
//
// A lane's operand for step s of a block of KB channels is channel 4 s + g
// (g = lane / 16) of its pixel, one 4-byte LDS read per product; a staged
// pixel takes an odd number of 16-byte quads, which puts the quads of 16
// neighbouring pixels on distinct banks.  (Channels regrouped so that one
// 16-byte read served four steps cost more in the staging writes than it
// saved: 20 against 11 cycles of LDS per product.)  The weights are packed
// in the order of use and read from global memory (L2), one block ahead.
//
// Taps outside the plane are zeros that are multiplied like the others.  With
// an infinite weight that gives NaN where the tap should count for nothing, so
// sums that come out NaN next to the border are taken again without these taps.
//
// Bound: the matrix cores for the layers with 32 and more channels, the
// exposed staging for the others.  Whole forward, 99 tiles of 96 x 96: 0.60
// ms (75 TFLOP/s), one tile 0.14 ms; with the vector kernel this replaced (a
// pixel per lane, weights as wave-uniform scalars) 1.74 and 1.17 ms.
#include <algorithm>

#include "ls_common.hpp"
#include "ls_unet.hpp"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int V>
struct VecOf;
template <>
struct VecOf<4> {
  typedef f32x4 T;
};
template <>
struct VecOf<2> {
  typedef float T __attribute__((ext_vector_type(2)));
};
template <>
struct VecOf<1> {
  typedef float T __attribute__((ext_vector_type(1)));
};

// Floats from one staged pixel to the next: an odd number of quads, so that
// the quads of 16 neighbouring pixels lie on distinct banks.
__host__ __device__ inline int pixel_pitch(int cin) { return (cin >> 2) & 1 ? cin : cin + 4; }

constexpr int STAGE_U = 4;  // patch rows a thread loads at a time

struct ConvGeom {
  int wx, wy, wm;          // waves along x, y and the output channels
  int tiles_x, tiles_y;    // workgroup tiles of one image
  int ntiles;              // of the batch
  int chunk;               // tiles per XCD
  int in_y0, in_y1, in_x0, in_x1;  // pixels that the tensors of both parts hold
};

// The sums of a wave that are NaN, of pixels next to the border, in the order of
// the products: without the taps outside the plane or outside a part's tensor.  A
// sum that is NaN again after a block of channels ends there (99 tiles with one
// weight in a hundred infinite 1.42 ms, channel by channel to the end 5.6; 1.74 with
// a vector kernel that skipped the taps).
// px: the lane's staged pixel at tap (0, 0) of its first pixel tile.
template <int KB, int NT>
__device__ __forceinline__ void sums_within(const ConvArgs& A, const ConvGeom& G, f32x4 (&acc)[NT], const float* px,
                                            int PW, int SP, int mw, int g, int oy, int ox) {
  constexpr int V = KB / 4;
  typedef typename VecOf<V>::T vec;
  const int ca = A.src.a.c, cin = ca + A.src.b.c, co = mw * 16 + 4 * g, x = A.x0 + ox;
  auto holds = [&](const SrcPart& p, int yy, int xx) {
    const int sy = p.up ? yy >> 1 : yy - p.oy, sx = p.up ? xx >> 1 : xx - p.ox;
    return yy >= 0 && xx >= 0 && yy < A.H && xx < A.W && sy >= 0 && sx >= 0 && sy < p.h && sx < p.w;
  };
#pragma unroll 1
  for (int e = 0; e < 4 * NT; ++e, px += e & 3 ? 0 : 2 * PW * SP, oy += e & 3 ? 0 : 2) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < 4 * NT; ++k) v = k == e ? acc[k >> 2][k & 3] : v;
    const int y = A.y0 + oy;
    if (v == v || co >= A.cout || oy >= A.Ho || ox >= A.Wo ||
        (y > G.in_y0 && y + 1 < G.in_y1 && x > G.in_x0 && x + 1 < G.in_x1))
      continue;
    float s = A.bias ? A.bias[co + (e & 3)] : 0.f;
#pragma unroll 1
    for (int tap = 0; tap < 9 && s == s; ++tap) {
      const int ky = tap / 3, kx = tap - 3 * ky;
      const bool in_a = holds(A.src.a, y + ky - 1, x + kx - 1), in_b = holds(A.src.b, y + ky - 1, x + kx - 1);
      const float* in = px + (ky * PW + kx) * SP;
      const vec* wt = reinterpret_cast<const vec*>(A.wt) + (mw * 9 + tap) * (cin / KB) * 64 + 4 * g + (e & 3);
#pragma unroll 1
      for (int c0 = 0; c0 < cin && s == s; c0 += KB, wt += 64) {
        const vec w[4] = {wt[0], wt[16], wt[32], wt[48]};  // channels c0 + k + 4 q
#pragma unroll
        for (int q = 0; q < V; ++q)
          if (c0 + 4 * q < ca ? in_a : in_b) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(in + c0 + 4 * q);
#pragma unroll
            for (int k = 0; k < 4; ++k) s = fmaf(v[k], w[k][q], s);
          }
      }
    }
#pragma unroll
    for (int k = 0; k < 4 * NT; ++k) acc[k >> 2][k & 3] = k == e ? s : acc[k >> 2][k & 3];
  }
}

// At most 96 scalar registers: eight waves per SIMD also with the code for sums
// that are NaN (which never runs otherwise; without the bound 2 % slower).
template <int KB, int NT, bool MASK>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_num_sgpr(96))) k_conv_f32_mfma(ConvArgs A, ConvGeom G) {
  constexpr int V = KB / 4;
  typedef typename VecOf<V>::T vec;
  extern __shared__ __align__(16) float s_in[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  // each XCD takes a contiguous run of tiles, so the halo rows of its
  // neighbours are found in its own L2
  const int tile = (int)(blockIdx.x & 7) * G.chunk + (int)(blockIdx.x >> 3);
  if (tile >= G.ntiles) return;
  const int per_img = G.tiles_x * G.tiles_y;
  const int b = tile / per_img, tt = tile - b * per_img;
  const int ty = tt / G.tiles_x, tx = tt - ty * G.tiles_x;
  const int oy0 = ty * G.wy * 2 * NT, ox0 = tx * G.wx * 8;  // in the output window
  const int cin = A.src.a.c + A.src.b.c, nq = cin >> 2, nblk = cin / KB;
  const int PW = 8 * G.wx + 2, PH = 2 * NT * G.wy + 2, SP = pixel_pitch(cin);
  // ---- stage the patch.  A thread keeps its column (pixel column and channel
  // quad, quads fastest) and walks down the rows, so the address work of an
  // item is a few instructions; the loads of STAGE_U rows are issued before
  // the first is written.
  {
    const int ncol = PW * nq, nthr = blockDim.x;
    const int rows = ncol < nthr ? nthr / ncol : 1;  // rows of one pass
    const int r0 = ncol < nthr ? tid / ncol : 0;
    for (int c = ncol < nthr ? (r0 < rows ? tid - r0 * ncol : ncol) : tid; c < ncol; c += nthr) {
      const int px = c / nq, q = c - px * nq;
      const bool first = 4 * q < A.src.a.c;
      const float* f32 = first ? A.src.a.f32 : A.src.b.f32;
      const float* mask = first ? A.src.a.mask : A.src.b.mask;
      const int up = first ? A.src.a.up : A.src.b.up, h = first ? A.src.a.h : A.src.b.h;
      const int w = first ? A.src.a.w : A.src.b.w, stride = first ? A.src.a.stride : A.src.b.stride;
      const int py0 = first ? A.src.a.oy : A.src.b.oy;
      const int xx = A.x0 + ox0 + px - 1;
      const int sx = up ? xx >> 1 : xx - (first ? A.src.a.ox : A.src.b.ox);
      const bool xok = xx >= 0 && xx < A.W && sx >= 0 && sx < w;
      const int64_t o0 = ((int64_t)b * h * w + (xok ? sx : 0)) * stride +
                         (first ? A.src.a.coff + 4 * q : A.src.b.coff + 4 * q - A.src.a.c);
      const int row = w * stride, yb = A.y0 + oy0 - 1;
      for (int py = r0; py < PH; py += STAGE_U * rows) {
        float4 v[STAGE_U], m[STAGE_U];
        bool ok[STAGE_U];
#pragma unroll
        for (int u = 0; u < STAGE_U; ++u) {
          const int yy = yb + py + u * rows;
          const int sy = up ? yy >> 1 : yy - py0;
          ok[u] = xok && yy >= 0 && yy < A.H && sy >= 0 && sy < h;
          // no branch around the load: outside, the image's first row is read and dropped
          const int64_t o = o0 + (ok[u] ? (int64_t)sy * row : 0);
          v[u] = *reinterpret_cast<const float4*>(f32 + o);
          if (MASK) m[u] = *reinterpret_cast<const float4*>(mask + o);
        }
#pragma unroll
        for (int u = 0; u < STAGE_U; ++u) {
          if (py + u * rows >= PH) break;
          const uint32_t keep = ok[u] ? 0xFFFFFFFFu : 0u;
          uint4 w4 = __builtin_bit_cast(uint4, v[u]);
          w4.x &= !MASK || m[u].x > 0.f ? keep : 0u;
          w4.y &= !MASK || m[u].y > 0.f ? keep : 0u;
          w4.z &= !MASK || m[u].z > 0.f ? keep : 0u;
          w4.w &= !MASK || m[u].w > 0.f ? keep : 0u;
          *reinterpret_cast<uint4*>(s_in + ((py + u * rows) * PW + px) * SP + 4 * q) = w4;
        }
      }
    }
  }
  __syncthreads();
  const int wxy = wave / G.wm, mw = wave - wxy * G.wm;
  const int wyi = wxy / G.wx, wxi = wxy - wyi * G.wx;
  const int co = mw * 16 + 4 * g;  // the lane's first output channel in the result
  f32x4 acc[NT];
  {
    f32x4 bv = {0.f, 0.f, 0.f, 0.f};
    if (A.bias && co < A.cout) {
#pragma unroll
      for (int i = 0; i < 4; ++i) bv[i] = A.bias[co + i];
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = bv;
  }
  // staged position of the lane's pixel at tap (0, 0), channel g
  int P0[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    P0[nt] = ((wyi * 2 * NT + 2 * nt + (r16 >> 3)) * PW + wxi * 8 + (r16 & 7)) * SP + g;
  const int nsteps = 9 * nblk;
  const vec* wp = reinterpret_cast<const vec*>(A.wt) + mw * nsteps * 64 + lane;
  auto load_b = [&](float (&o)[NT][V], int at) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int s = 0; s < V; ++s) o[nt][s] = s_in[P0[nt] + at + 4 * s];
  };
  vec a = wp[0];
  float bf[NT][V];
  load_b(bf, 0);
  int kx = 0, j = 0, at = 0;  // tap column, block, their staged offset
  for (int i = 0; i < nsteps; ++i) {
    // the next block's operands, one block ahead of their use
    at += KB;
    if (++j == nblk) {
      j = 0;
      at += SP - cin;
      if (++kx == 3) {
        kx = 0;
        at += (PW - 3) * SP;
      }
    }
    const bool more = i + 1 < nsteps;
    const vec an = wp[(more ? i + 1 : i) * 64];
    float bn[NT][V];
    load_b(bn, more ? at : 0);
#pragma unroll
    for (int s = 0; s < V; ++s)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], bf[nt][s], acc[nt], 0, 0, 0);
    a = an;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int s = 0; s < V; ++s) bf[nt][s] = bn[nt][s];
  }
  // ---- sums that zeros outside the plane have made NaN, once more without them
  const int by = A.y0 + oy0, bx = A.x0 + ox0;  // the workgroup's first pixel
  if (by <= G.in_y0 || bx <= G.in_x0 || by + 2 * NT * G.wy >= G.in_y1 || bx + 8 * G.wx >= G.in_x1) {
    // NaN if one of the sums is, or if they hold infinities of both signs
    f32x4 any = acc[0];
#pragma unroll
    for (int nt = 1; nt < NT; ++nt) any += acc[nt];
    const float t = any[0] + any[1] + any[2] + any[3];
    if (__ballot(t != t)) {
      const int oy = wyi * 2 * NT + (r16 >> 3), ox = wxi * 8 + (r16 & 7);
      sums_within<KB, NT>(A, G, acc, s_in + (oy * PW + ox) * SP, PW, SP, mw, g, oy0 + oy, ox0 + ox);
    }
  }
  // ---- epilogue: lane = 4 consecutive channels of one pixel per tile
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    f32x4 v = acc[nt];
    if (A.relu) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
    }
    const int oy = oy0 + wyi * 2 * NT + 2 * nt + (r16 >> 3), ox = ox0 + wxi * 8 + (r16 & 7);
    const bool ok = co < A.cout && oy < A.Ho && ox < A.Wo;
    if (ok && A.out)
      *reinterpret_cast<f32x4*>(A.out + (((int64_t)b * A.Ho + oy) * A.Wo + ox) * A.out_stride + A.out_coff + co) = v;
    if (A.pool_out) {
      // 2 x 2 average: a tile holds two rows, eight lanes apart
      f32x4 t;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        t[i] = v[i] + __shfl_xor(v[i], 1, 64);
        t[i] = 0.25f * (t[i] + __shfl_xor(t[i], 8, 64));
      }
      if (ok && (r16 & 9) == 0)
        *reinterpret_cast<f32x4*>(A.pool_out +
                                  (((int64_t)b * (A.Ho >> 1) + (oy >> 1)) * (A.Wo >> 1) + (ox >> 1)) * A.pool_stride +
                                  A.pool_coff + co) = t;
    }
  }
}

constexpr int LDS_MAX = 160 * 1024;

struct ConvPlan {
  int nt, lds;
  ConvGeom g;
};

// A workgroup has one wave per channel tile and four waves in all where that
// leaves room for several pixel blocks: small workgroups overlap one's
// staging with another's products (eight waves were up to 10 % slower, and
// two channel tiles per wave up to 40 % for the 96- and 48-channel inputs,
// whose patches then let only one workgroup into a CU).  A wave takes 8 x 4
// pixels; 8 x 8, whose halo is smaller, where the products per staged byte
// are few (up to 16 input channels: 99 tiles of 96 x 96, 8 -> 16 channels 38
// against 44 us, 16 -> 16 channels 56 against 58.5) and enough waves remain
// (at 24 tiles, 3,500 waves, 22 against 20.6 us).
ConvPlan conv_plan(const ConvArgs& a) {
  const int cin = a.src.a.c + a.src.b.c, mtiles = (a.cout + 15) / 16;
  ConvPlan p;
  p.g.wm = mtiles;
  p.g.wx = mtiles == 1 ? 2 : 1;
  p.g.wy = mtiles <= 2 ? 2 : 1;
  const int64_t waves8x8 = (int64_t)a.B * ((a.Ho + 7) / 8) * ((a.Wo + 7) / 8) * mtiles;
  p.nt = a.tiling == 1 || a.tiling == 3 ? 2 : (a.tiling == 2 || (cin <= 16 && waves8x8 >= 6144) ? 4 : 2);
  if (a.tiling == 3 && 2 * p.g.wx * p.g.wy * p.g.wm <= 8) p.g.wy *= 2;
  p.g.tiles_x = (a.Wo + 8 * p.g.wx - 1) / (8 * p.g.wx);
  p.g.tiles_y = (a.Ho + 2 * p.nt * p.g.wy - 1) / (2 * p.nt * p.g.wy);
  p.lds = (8 * p.g.wx + 2) * (2 * p.nt * p.g.wy + 2) * pixel_pitch(cin) * 4;
  const int64_t tiles = (int64_t)a.B * p.g.tiles_x * p.g.tiles_y;
  p.g.ntiles = (int)std::min<int64_t>(tiles, 0x7fffffff);
  p.g.chunk = (int)((p.g.ntiles + 7LL) / 8);
  p.g.in_y0 = p.g.in_x0 = 0;
  p.g.in_y1 = a.H;
  p.g.in_x1 = a.W;
  for (const SrcPart* q : {&a.src.a, &a.src.b}) {
    if (!q->c) continue;
    p.g.in_y0 = std::max(p.g.in_y0, q->up ? 0 : q->oy);
    p.g.in_x0 = std::max(p.g.in_x0, q->up ? 0 : q->ox);
    p.g.in_y1 = std::min(p.g.in_y1, q->up ? 2 * q->h : q->oy + q->h);
    p.g.in_x1 = std::min(p.g.in_x1, q->up ? 2 * q->w : q->ox + q->w);
  }
  return p;
}

template <int KB, int NT, bool MASK>
int launch(const ConvArgs& a, const ConvPlan& p, hipStream_t st) {
  auto* fn = k_conv_f32_mfma<KB, NT, MASK>;
  // the same limit whatever this launch needs: another thread may set it for its own
  if (p.lds > 65536)
    LS_HOST_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MAX));
  hipLaunchKernelGGL(fn, dim3((unsigned)p.g.chunk * 8), dim3(64u * p.g.wx * p.g.wy * p.g.wm), p.lds, st, a, p.g);
  LS_LAUNCH_CHECK();
  return LS_OK;
}

template <int KB>
int launch_kb(const ConvArgs& a, const ConvPlan& p, bool mask, hipStream_t st) {
  if (p.nt == 4) return mask ? launch<KB, 4, true>(a, p, st) : launch<KB, 4, false>(a, p, st);
  return mask ? launch<KB, 2, true>(a, p, st) : launch<KB, 2, false>(a, p, st);
}

}  // namespace

int ls_conv_f32(const ConvArgs& a, hipStream_t st) {
  const int cin = a.src.a.c + a.src.b.c;
  // channels are staged four at a time from one part, and stored four at a time
  if (a.cout % 4 || a.src.a.c % 4 || a.src.b.c % 4 || cin <= 0 || a.out_stride % 4 || a.out_coff % 4) return LS_ENOTIMPL;
  if (a.pool_out && (a.y0 || a.x0 || a.Ho % 2 || a.Wo % 2 || a.pool_stride % 4 || a.pool_coff % 4)) return LS_ENOTIMPL;
  if (a.B <= 0 || a.Ho <= 0 || a.Wo <= 0) return LS_OK;
  const ConvPlan p = conv_plan(a);
  // up to 8 channel tiles per workgroup; the grid in 32 bits
  if (p.g.wm > 8 || p.lds > LDS_MAX || (int64_t)p.g.ntiles * 64 * p.g.wx * p.g.wy * p.g.wm > 0xFFFF0000LL) return LS_ENOTIMPL;
  const bool mask = a.src.a.mask != nullptr;
  if (a.src.b.c > 0 && (a.src.b.mask != nullptr) != mask) return LS_ENOTIMPL;
  LS_TRACE("conv_f32", st);
  switch (ls_conv_f32_block(cin)) {
    case 16: return launch_kb<16>(a, p, mask, st);
    case 8: return launch_kb<8>(a, p, mask, st);
    default: return launch_kb<4>(a, p, mask, st);
  }
}
