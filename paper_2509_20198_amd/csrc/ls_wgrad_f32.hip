// FP32 weight gradient of a 3x3 conv on the matrix cores of gfx950.
//
// dW[co][n] = sum over output pixels of dZ[p][co] * I[p][n], n = (tap, input
// channel), plus a column of ones for the bias: v_mfma_f32_16x16x4_f32 with
// four pixels as k.  A workgroup owns 16 output channels and one block of CB
// input channels (all nine taps) over the spatial tiles blockIdx.x,
// blockIdx.x + gridDim.x, ..: per tile it stages the masked gradient and the
// input patch in LDS, both pixel-major as they are stored (k runs over the
// lane groups, so no transpose is needed), every element once for its nine
// taps.  Its four waves take every fourth group of four pixels, and their sums
// are added in LDS in a fixed order, so the partial sums are deterministic.
// Tiles are about 256 pixels, 16 to 32 wide, whichever pads the plane least
// (24 x 8 on the 24-wide planes; windows are square, so 8 x 32 would pad as much
// as 32 x 8); several whole images one above the other where a plane has at most
// 10 x 10 texels.
//
// Bound: at small batches the exposed staging of the one or two tiles a
// workgroup gets, else the matrix cores (nine products per ten LDS reads, ten
// where the bias is summed; five per six with 8 input channels).  24
// tiles of 96 x 96, all eleven layers: 0.31 ms (41 TFLOP/s); 0.75 ms with the
// vector kernel this replaced, which staged the im2col columns (each input
// element nine times).  32 output channels per workgroup took 232 registers
// (two waves per SIMD) and the same time; capped at 168 they spilled (0.48 ms).
#include <algorithm>

#include "ls_common.hpp"
#include "ls_unet.hpp"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int WT = 256;         // threads
constexpr int TILE_PX = 256;    // output pixels of a tile at most
constexpr int PATCH_PX = 340;   // and its input patch: 18 x 18, 26 x 10, 34 x 10

struct WgradGeom {
  int tw, th;              // tile, tw a multiple of 4
  int tiles_x, ntiles, per_img;
  int ni;                  // whole images of a tile, one above the other (PACK)
  int ncib;                // input-channel blocks
};

template <int CB, bool PACK>
__global__ void __launch_bounds__(WT) k_wgrad_f32_mfma(WgradArgs A, WgradGeom G) {
  constexpr int NTL = CB == 16 ? 9 : 5;  // column tiles: a tap, or two taps of 8 channels
  constexpr int GP = 16;                 // output channels of a workgroup
  constexpr int NGI = 4, NXI = (PATCH_PX * (CB / 4) + WT - 1) / WT;  // staged quads per thread
  static_assert((NTL + 1) * 256 <= TILE_PX * GP + PATCH_PX * CB, "the reduction fits the staging");
  __shared__ __align__(16) float s_mem[TILE_PX * GP + PATCH_PX * CB];
  float* s_g = s_mem;
  float* s_x = s_mem + TILE_PX * GP;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int cin = A.src.a.c + A.src.b.c;
  const int cib = blockIdx.y % G.ncib, co0 = (blockIdx.y / G.ncib) * GP;
  const int c0 = cib * CB;
  const bool bias = cib == 0;
  const SrcPart S = c0 < A.src.a.c ? A.src.a : A.src.b;  // the block lies in one part
  const int sc = S.coff + (c0 < A.src.a.c ? c0 : c0 - A.src.a.c);
  const int ni = PACK ? G.ni : 1;
  const int PW = G.tw + 2, npx = G.tw * G.th * ni, npatch = PW * (G.th + 2) * ni;
  // staged offset of the lane's column in column tile t
  int off[NTL];
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    const int tap = min(CB == 16 ? t : 2 * t + (r16 >> 3), 8);  // the tenth tap of the last pair is not stored
    off[t] = ((tap / 3) * PW + tap % 3) * CB + (CB == 16 ? r16 : (r16 & 7));
  }
  f32x4 acc[NTL + 1];
#pragma unroll
  for (int t = 0; t <= NTL; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int tile = blockIdx.x; tile < G.ntiles; tile += gridDim.x) {
    const int b = PACK ? tile * G.ni : tile / G.per_img, tt = PACK ? 0 : tile - b * G.per_img;
    const int ty0 = (tt / G.tiles_x) * G.th, tx0 = (tt % G.tiles_x) * G.tw;
    const int nb = PACK ? min(G.ni, A.B - b) : 1;  // images
    // every load of the tile before its LDS writes: one memory round trip
    float4 gv[NGI], gm[NGI], xv[NXI];
    bool gok[NGI], xok[NXI];
#pragma unroll
    for (int i = 0; i < NGI; ++i) {
      const int e = tid + WT * i, px = e >> 2, q = e & 3;
      const int vr = px / G.tw, c = px - vr * G.tw;
      const int im = PACK ? vr / G.th : 0, r = vr - im * G.th;
      gok[i] = px < npx && im < nb && ty0 + r < A.Ho && tx0 + c < A.Wo && co0 + 4 * q < A.cout;
      const int64_t o = gok[i] ? (((int64_t)(b + im) * A.Ho + ty0 + r) * A.Wo + tx0 + c) * A.d_stride + co0 + 4 * q : 0;
      gv[i] = *reinterpret_cast<const float4*>(A.dA + o);
      if (A.mask) gm[i] = *reinterpret_cast<const float4*>(A.mask + o);
    }
#pragma unroll
    for (int i = 0; i < NXI; ++i) {
      const int e = tid + WT * i, px = e / (CB / 4), q = e % (CB / 4);
      const int vr = px / PW, c = px - vr * PW;
      const int im = PACK ? vr / (G.th + 2) : 0, r = vr - im * (G.th + 2);
      const int yy = A.y0 + ty0 + r - 1, xx = A.x0 + tx0 + c - 1;
      const int sy = S.up ? yy >> 1 : yy - S.oy, sx = S.up ? xx >> 1 : xx - S.ox;
      xok[i] = px < npatch && im < nb && yy >= 0 && xx >= 0 && yy < A.H && xx < A.W && sy >= 0 && sx >= 0 && sy < S.h && sx < S.w;
      const int64_t o = (xok[i] ? (((int64_t)(b + im) * S.h + sy) * S.w + sx) * S.stride : 0) + sc + 4 * q;
      xv[i] = *reinterpret_cast<const float4*>(S.f32 + o);
    }
#pragma unroll
    for (int i = 0; i < NGI; ++i) {
      const int e = tid + WT * i;
      const float4 v = gv[i];
      const float4 m = A.mask ? gm[i] : make_float4(1.f, 1.f, 1.f, 1.f);
      const bool k = gok[i];
      if (e < npx * 4)
        reinterpret_cast<float4*>(s_g)[e] = make_float4(k && m.x > 0.f ? v.x : 0.f, k && m.y > 0.f ? v.y : 0.f,
                                                        k && m.z > 0.f ? v.z : 0.f, k && m.w > 0.f ? v.w : 0.f);
    }
#pragma unroll
    for (int i = 0; i < NXI; ++i) {
      const int e = tid + WT * i;
      const float4 v = xv[i];
      const bool k = xok[i];
      if (e < npatch * (CB / 4))
        reinterpret_cast<float4*>(s_x)[e] = make_float4(k ? v.x : 0.f, k ? v.y : 0.f, k ? v.z : 0.f, k ? v.w : 0.f);
    }
    __syncthreads();
    // groups of four pixels (4 c .. 4 c + 3 of a row) inside the window: a padding
    // pixel's gradient is zero, but its products with infinite inputs are not
    const int vw = min(G.tw, A.Wo - tx0), w4 = (vw + 3) >> 2, ngrp = w4 * min(G.th, A.Ho - ty0) * nb;
    int row = 0, c = wave;
    for (; c >= w4; c -= w4) ++row;
    for (int s = wave; s < ngrp; s += 4) {
      const float af = s_g[(row * G.tw + 4 * c + g) * GP + r16];
      const float* xa = s_x + ((PACK ? row + 2 * (row / G.th) : row) * PW + 4 * c + g) * CB;
      float bf[NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t) bf[t] = xa[off[t]];
      if (4 * c + 4 > vw) {  // the last group of a row
#pragma unroll
        for (int t = 0; t < NTL; ++t) bf[t] = 4 * c + g < vw ? bf[t] : 0.f;
      }
#pragma unroll
      for (int t = 0; t < NTL; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(af, bf[t], acc[t], 0, 0, 0);
      if (bias) acc[NTL] = __builtin_amdgcn_mfma_f32_16x16x4f32(af, 1.f, acc[NTL], 0, 0, 0);
      for (c += 4; c >= w4; c -= w4) ++row;
    }
    __syncthreads();  // every wave is done with the staged tile
  }
  // the four waves' sums in a fixed order
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int t = 0; t <= NTL; ++t) {
        f32x4* q = reinterpret_cast<f32x4*>(s_mem) + t * 64 + lane;
        *q = w == 0 ? acc[t] : *q + acc[t];
      }
    }
    __syncthreads();
  }
  const int N = 9 * cin;
  float* out = A.partial + (int64_t)blockIdx.x * ((int64_t)A.cout * N + A.cout);
  for (int e = tid; e < (NTL + 1) * 64; e += WT) {
    const int l = e & 63, t = e >> 6;
    const int col = l & 15, tap = CB == 16 ? t : 2 * t + (col >> 3);
    const f32x4 v = reinterpret_cast<const f32x4*>(s_mem)[e];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int co = co0 + 4 * (l >> 4) + i;
      if (co >= A.cout) continue;
      if (t == NTL) {
        if (bias && col == 0) out[(int64_t)A.cout * N + co] = v[i];
      } else if (tap < 9) {
        out[(int64_t)co * N + tap * cin + c0 + (CB == 16 ? col : (col & 7))] = v[i];
      }
    }
  }
}

}  // namespace

// Partial sums of the FP32 weight gradient; sets the number of chunks written
// (at most a.nchunk).
int ls_wgrad_f32_partials(const WgradArgs& a, int* nchunk, hipStream_t st) {
  const int cin = a.src.a.c + a.src.b.c;
  // blocks of 8 or 16 input channels within one part, quads of the gradient
  if (a.src.a.c % 8 || a.src.b.c % 8 || a.cout % 4 || a.d_stride % 4 || !a.dA) return LS_ENOTIMPL;
  const int cb = a.src.a.c % 16 == 0 && a.src.b.c % 16 == 0 ? 16 : 8;
  WgradGeom g;
  int64_t best = 0;
  for (int tw : {16, 24, 32}) {
    const int th = tw == 24 ? 8 : TILE_PX / tw;
    const int64_t padded = (int64_t)((a.Wo + tw - 1) / tw) * tw * (((a.Ho + th - 1) / th) * th);
    if (best == 0 || padded < best) {
      best = padded;
      g.tw = tw;
      g.th = th;
    }
  }
  // planes of which a tile holds several: as many as fit (a backward of 2,000
  // images of 4 x 4, 2 x 2 and 1 x 1 texels 1.11 ms; with a tile for each 2.70 ms)
  const int pw = (a.Wo + 3) & ~3;
  g.ni = std::min(TILE_PX / std::max(1, pw * a.Ho), PATCH_PX / ((pw + 2) * (a.Ho + 2)));
  const bool pack = g.ni > 1;
  if (pack) {
    g.tw = pw;
    g.th = a.Ho;
  }
  g.tiles_x = (a.Wo + g.tw - 1) / g.tw;
  g.per_img = g.tiles_x * ((a.Ho + g.th - 1) / g.th);
  const int64_t ntiles = pack ? (a.B + g.ni - 1LL) / g.ni : (int64_t)a.B * g.per_img;
  if (ntiles > 0x7fffffff) return LS_ENOTIMPL;
  g.ntiles = (int)ntiles;
  g.ncib = cin / cb;
  const int groups = g.ncib * ((a.cout + 15) / 16);
  // equal numbers of tiles for the workgroups
  const int per = std::max(1, (g.ntiles + a.nchunk - 1) / a.nchunk);
  *nchunk = std::max(1, (g.ntiles + per - 1) / per);
  const dim3 grid((unsigned)*nchunk, (unsigned)groups);
  auto* fn = cb == 16 ? (pack ? k_wgrad_f32_mfma<16, true> : k_wgrad_f32_mfma<16, false>)
                      : (pack ? k_wgrad_f32_mfma<8, true> : k_wgrad_f32_mfma<8, false>);
  hipLaunchKernelGGL(fn, grid, dim3(WT), 0, st, a, g);
  LS_LAUNCH_CHECK();
  return LS_OK;
}
