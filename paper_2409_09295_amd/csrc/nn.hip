// Kernels of the learned Gaussian initialiser: a small U-Net over BF16 NHWC
// activations with FP32 accumulation on MFMA (v_mfma_f32_16x16x32_bf16).
//
// conv3x3 (forward and, with flipped/transposed weights, backward-data) is a direct
// convolution on spatial tiles, conv3x3_patch_kernel; its inputs' channels come in
// eights.  They may come from two tensors, which is how the decoder's skip
// concatenation is read without materialising it, and an optional mask tensor zeroes
// input entries whose mask value is <= 0 (the ReLU backward fused into the
// backward-data pass).
//
// conv3x3_wgrad: dW[tap][co][ci] = sum_p dz[p][co] x[p + tap][ci] as a GEMM
// with M = Cout, N = Cin, K = pixels, split over runs of pixels with float32
// atomics: conv3x3_wgrad_strip_kernel for channels in eights, which reads the
// tiles transposed from LDS; conv3x3_wgrad_kernel and conv3x3_wgrad32_kernel for
// the others, which write them transposed.
//
// MFMA 16x16x32 operand layout (lane l, 8 values each): A row l % 16, B
// column l % 16, both covering k = 8 (l / 16) .. 8 (l / 16) + 7; result D row
// 4 (l / 16) + j, column l % 16, j = 0..3.
#include <cmath>

#include "gs_internal.h"
#include "gs_nn.h"

namespace gsmi {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// round-to-nearest-even float -> bf16 (inputs are finite)
__device__ __forceinline__ uint16_t f2bf(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint32_t r = u + 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(r >> 16);
}

// Two floats as bf16 in one word, rounded as f2bf rounds.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef float float2v __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){lo, hi}, bf16x2));
}

struct ActView {
  const uint16_t* p;
  int32_t c, stride, offset;
};

// Zeroes the bf16 elements of v whose mask element is <= 0 (as int16, -0 among
// them: 0 - x saturates, so its sign is set exactly where x > 0).
__device__ __forceinline__ uint32_t mask_word(uint32_t v, uint32_t mk) {
  typedef short short2v __attribute__((ext_vector_type(2)));
  const short2v m = __builtin_elementwise_sub_sat(short2v{0, 0}, __builtin_bit_cast(short2v, mk));
  return v & __builtin_bit_cast(uint32_t, (short2v)(m >> (short)15));
}

__device__ __forceinline__ uint4 apply_mask8(uint4 v, uint4 mk) {
  return make_uint4(mask_word(v.x, mk.x), mask_word(v.y, mk.y), mask_word(v.z, mk.z),
                    mask_word(v.w, mk.w));
}

// Loads 8 consecutive channels [c0, c0 + 8) of pixel (n, y, x) from a
// two-source channel concatenation; zero outside the image or beyond the
// channel count.  mask (optional, same layout as the concatenation) zeroes
// elements whose mask is <= 0.
__device__ __forceinline__ uint4 load8(const ActView& a, const ActView& b, const ActView& m,
                                       int64_t pix, bool inb, int c0) {
  uint4 v = make_uint4(0, 0, 0, 0);
  if (!inb) return v;
  const ActView* s = &a;
  int c = c0;
  if (c0 >= a.c) {
    s = &b;
    c = c0 - a.c;
  }
  if (s->p == nullptr || c >= s->c) return v;
  v = *reinterpret_cast<const uint4*>(s->p + pix * s->stride + s->offset + c);
  if (m.p) {
    const uint4 mk = *reinterpret_cast<const uint4*>(m.p + pix * m.stride + m.offset + c0);
    v = apply_mask8(v, mk);
  }
  return v;
}

// Direct 3x3 convolution on spatial tiles.  A workgroup computes 16 x 16
// pixel tiles of one image for 16 JN output channels; wavefront w of eight
// computes output rows 2w and 2w + 1 for all of them (four rows in four
// wavefronts read fewer fragments but held two or three wavefronts per SIMD).  Input channels go in chunks of 32:
// the chunk's 18 x 18 input patch (the tile and its one-pixel halo; zero outside
// the image) and its 9 x 16 JN x 32 weights are staged in LDS once, and every
// tap reads the patch at its offset, so each input value is loaded from memory
// about 1.3 times instead of nine.  Workgroups are persistent: those of
// column c take tiles c, c + columns, ..., and the next (tile, chunk) pair's patch and
// weights are loaded into registers while this pair's 18 JN MFMAs per wavefront
// run, so a layer with a single chunk overlaps the next tile's loads with this
// tile's products and stores.
//
// The weights are the A operand and 16 pixels of a row the B operand, so a lane
// ends with 4 JN consecutive channels of one pixel (A row 4 g + r of block j holds
// channel 4 JN g + 4 j + r) and stores them 16 bytes at a time; four patch rows
// per tap column serve its three taps.  LDS pixels and weight rows are 64 bytes,
// their four 16-byte pieces permuted by a function of the pixel's column (the
// weight's row) that leaves the 16 lanes of an LDS read cycle, {0-3, 12-15, 20-27}
// and so on, on different banks.
//
// 4 x 640x480, forward: 32 -> 32 channels 33 us (65 with pixels as the A operand, a
// 16-channel span per lane group and 2-byte stores), 96 -> 32 100 (133), 64 -> 64 121
// (197); with a mask, 96 of 32 channels 139 (232), 32 of 64 109 (131).  157 MB and 315 MB
// of activations would take 33 and 66 us at the 4.7 TB/s of a copy: one chunk is bound
// by memory, several by the LDS reads of the fragments (eight bytes per pixel and
// channel block for 2 x 16 x 32 products) and the two barriers of a chunk.
constexpr int PT = 16;                  // output tile side
constexpr int PP = PT + 2;              // patch side (with halo)
constexpr int PCC = 32;                 // input channels per chunk
constexpr int PPITCH = 20;              // LDS pixels per patch row
constexpr int PR = 2;                   // output rows per wavefront
constexpr int PATCH_CHUNKS = PP * PP * (PCC / 8);   // 16-byte pieces of a patch (1,296)

// Byte offset of 16-byte piece c of the 64-byte record i of a row of records.
__device__ __forceinline__ int cv_piece(int i, int c) {
  return i * 64 + ((c ^ (-(i >> 2) & 3)) << 4);
}

// MASKED: the input is multiplied by a ReLU mask (mask > 0) as it is staged.
// ONE: a single chunk (cin <= 32), whose weights stay in LDS.
template <int JN, bool MASKED, bool ONE>
__global__ __launch_bounds__(64 * PT / PR, 4) void conv3x3_patch_kernel(
    ActView x1, ActView x2, ActView mask, int N, int H, int W, const uint16_t* __restrict__ wk,
    int cout, int cin, const float* __restrict__ bias, int relu, uint16_t* __restrict__ y,
    int y_stride, int y_offset, float* __restrict__ yf, int yf_stride, int columns) {
  constexpr int BNT = 16 * JN;
  constexpr int NT = 64 * PT / PR;                  // threads
  constexpr int W_CHUNKS = 9 * BNT * (PCC / 8);     // 16-byte pieces of a chunk's weights
  constexpr int PA = (PATCH_CHUNKS + NT - 1) / NT;    // per thread
  constexpr int PB = (W_CHUNKS + NT - 1) / NT;
  __shared__ __attribute__((aligned(16))) char sP[PP * PPITCH * 64];
  __shared__ __attribute__((aligned(16))) char sW[9 * BNT * 64];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tiles_x = (W + PT - 1) / PT, tiles_y = (H + PT - 1) / PT;
  const int n_tiles = N * tiles_x * tiles_y;
  // the channel groups of a column of tiles on one XCD (workgroups go round the eight
  // of them), close in time: they read it through one L2
  const int groups = (cout + BNT - 1) / BNT, slot = (int)blockIdx.x >> 3;
  const int column = slot / groups * 8 + ((int)blockIdx.x & 7), n0 = slot % groups * BNT;
  if (column >= columns) return;   // the whole workgroup
  const int nchunks = ONE ? 1 : (cin + PCC - 1) / PCC;
  // this thread's pieces hold channels pc .. pc + 7 of a chunk
  const int pc = (t & 3) * 8;
  uint4 ra[PA], rm[MASKED ? PA : 1], rb[PB];
  int img = 0, ty0 = 0, tx0 = 0;   // of the tile last located
  auto locate = [&](int tile) {
    img = tile / (tiles_x * tiles_y);
    const int trem = tile - img * tiles_x * tiles_y;
    ty0 = (trem / tiles_x) * PT;
    tx0 = (trem % tiles_x) * PT;
  };
  auto fetch = [&](int chunk, bool weights) {   // of the tile last located
    const int c = chunk * PCC + pc;
    const bool first = c < x1.c;
    const ActView& s = first ? x1 : x2;
    const int64_t base = (int64_t)img * H * W;
    const uint16_t* src = s.p + s.offset + (first ? c : c - x1.c) + base * s.stride;
    const uint16_t* msrc = MASKED ? mask.p + mask.offset + c + base * mask.stride : nullptr;
#pragma unroll
    for (int u = 0; u < PA; ++u) {
      const int pp = (t + NT * u) >> 2;    // patch pixel
      const int py = pp / PP, sy = ty0 + py - 1, sx = tx0 + (pp - py * PP) - 1;
      ra[u] = make_uint4(0, 0, 0, 0);
      if constexpr (MASKED) rm[u] = ra[u];
      if (pp < PP * PP && (unsigned)sy < (unsigned)H && (unsigned)sx < (unsigned)W && c < cin) {
        const int64_t pix = sy * W + sx;
        ra[u] = *reinterpret_cast<const uint4*>(src + pix * s.stride);
        if constexpr (MASKED) rm[u] = *reinterpret_cast<const uint4*>(msrc + pix * mask.stride);
      }
    }
    if (!weights) return;
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      const int tn = (t + NT * u) >> 2;    // (tap, LDS row): row 16 j + 4 g + r of a tap
      const int tap = tn / BNT, row = tn - tap * BNT;
      const int co = n0 + 4 * JN * ((row >> 2) & 3) + 4 * (row >> 4) + (row & 3);
      rb[u] = make_uint4(0, 0, 0, 0);
      if (tn < 9 * BNT && co < cout && c < cin)
        rb[u] = *reinterpret_cast<const uint4*>(wk + ((int64_t)tap * cout + co) * cin + c);
    }
  };
  f32x4 acc[PR][JN];
#pragma unroll
  for (int i = 0; i < PR; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // registers -> LDS: the patch, and the weights when they are (re)loaded
  auto stage = [&](bool weights) {
#pragma unroll
    for (int u = 0; u < PA; ++u) {
      const int pp = (t + NT * u) >> 2, py = pp / PP;
      uint4 v = ra[u];
      if constexpr (MASKED) v = apply_mask8(v, rm[u]);
      if (pp < PP * PP)
        *reinterpret_cast<uint4*>(sP + py * PPITCH * 64 + cv_piece(pp - py * PP, t & 3)) = v;
    }
    if (!weights) return;
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      const int tn = (t + NT * u) >> 2;
      if (tn < 9 * BNT)
        *reinterpret_cast<uint4*>(sW + (tn & ~15) * 64 + cv_piece(tn & 15, t & 3)) = rb[u];
    }
  };
  const char* w_base = sW + cv_piece(lane & 15, lane >> 4);
  const char* p_base = sP + PR * wv * PPITCH * 64;
  auto multiply = [&]() {
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      bf16x8 p[PR + 2];
      const char* pl = p_base + cv_piece((lane & 15) + dx, lane >> 4);
#pragma unroll
      for (int i = 0; i < PR + 2; ++i) p[i] = *reinterpret_cast<const bf16x8*>(pl + i * PPITCH * 64);
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          const bf16x8 w = *reinterpret_cast<const bf16x8*>(w_base + ((3 * dy + dx) * BNT + 16 * j) * 64);
#pragma unroll
          for (int i = 0; i < PR; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, p[i + dy], acc[i][j], 0, 0, 0);
        }
    }
  };
  // bias, ReLU, bf16 (or float32) store, accumulators cleared; acc[i][j][r] is
  // output row PR wv + i, column lane % 16, channel c0 + 4 j + r
  const int c0 = n0 + 4 * JN * (lane >> 4);
  const bool wide = cout % 8 == 0 && y_stride % 8 == 0 && y_offset % 8 == 0 &&
                    (reinterpret_cast<uintptr_t>(y) & 15) == 0;
  static_assert(JN % 2 == 0, "eight channels to a store");
  auto epilogue = [&](int tile) {
    const int timg = tile / (tiles_x * tiles_y);
    const int trem = tile - timg * tiles_x * tiles_y;
    const int oy0 = (trem / tiles_x) * PT + PR * wv, ox = (trem % tiles_x) * PT + (lane & 15);
    const int64_t base = (int64_t)timg * H * W;
#pragma unroll
    for (int j = 0; j < JN; j += 2) {   // channels c0 + 4 j .. + 7
      float b[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) b[c] = bias && c0 + 4 * j + c < cout ? bias[c0 + 4 * j + c] : 0.f;
#pragma unroll
      for (int i = 0; i < PR; ++i) {
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          v[c] = acc[i][j + (c >> 2)][c & 3] + b[c];
          if (relu) v[c] = fmaxf(v[c], 0.f);
        }
        acc[i][j] = acc[i][j + 1] = (f32x4){0.f, 0.f, 0.f, 0.f};
        const int oy = oy0 + i;
        if (oy >= H || ox >= W) continue;
        const int64_t p = base + oy * W + ox;
        uint16_t* o = y + p * y_stride + y_offset + c0 + 4 * j;
        if (y && wide) {
          if (c0 + 4 * j < cout)
            *reinterpret_cast<uint4*>(o) = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]),
                                                      pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
        } else if (y) {
#pragma unroll
          for (int c = 0; c < 8; ++c)
            if (c0 + 4 * j + c < cout) o[c] = f2bf(v[c]);
        }
        if (yf) {
          float* of = yf + p * yf_stride + c0 + 4 * j;
#pragma unroll
          for (int c = 0; c < 8; ++c)
            if (c0 + 4 * j + c < cout) of[c] = v[c];
        }
      }
    }
  };
  int tile = column, chunk = 0;   // columns never exceed the tiles
  locate(tile);
  fetch(0, true);
  for (bool first = true;; first = false) {
    __syncthreads();   // the previous pair's fragments have been read
    stage(first || !ONE);
    __syncthreads();
    // the next (tile, chunk) pair, loaded while this one is multiplied
    int next_tile = tile, next_chunk = chunk + 1;
    if (next_chunk == nchunks) {
      next_chunk = 0;
      next_tile = tile + columns;
    }
    const bool more = next_tile < n_tiles;
    if (more) {
      if (next_tile != tile) locate(next_tile);
      fetch(next_chunk, !ONE);
    }
    multiply();
    if (chunk == nchunks - 1) epilogue(tile);
    if (!more) break;
    tile = next_tile;
    chunk = next_chunk;
  }
}

// Weight-gradient tile: 64 output channels x 64 input channels for one row
// of three taps (dy fixed, dx = -1, 0, 1: one load of dz serves three taps),
// pixels [kbeg, kbeg + kchunk) of the K dimension.  Each stage covers 64
// pixels: thread t loads pixels 2 (t % 32) and 2 (t % 32) + 1, channels
// 8 (t / 32) .. +8, of both dz (output-channel tile) and the tap-shifted
// inputs (input-channel tile) with 16-byte loads, and writes them transposed
// ([channel][pixel], two pixels per 32-bit write) into LDS; each wavefront
// then issues two K steps of four MFMAs per tap.
constexpr int BM = 64, BN = 64;      // channels of a tile
constexpr int WBK = 64;              // pixels per stage
constexpr int WLDK = WBK + 8;        // LDS row pitch in bf16 (16-byte aligned rows)
constexpr int kWgradBlocks = 512;    // pixel chunks are sized for about this many workgroups
constexpr int kWgrad32Blocks = 512;  // the narrow kernel: two resident workgroups per CU


__global__ __launch_bounds__(256) void conv3x3_wgrad_kernel(
    ActView x1, ActView x2, ActView dz, ActView mask, int N, int H, int W, int cout, int cin,
    int64_t kchunk, float* __restrict__ dw, float* __restrict__ dbias) {
  __shared__ __attribute__((aligned(16))) uint16_t sA[BM * WLDK];   // [co][pixel]
  __shared__ __attribute__((aligned(16))) uint16_t sB[3][BN * WLDK];   // per tap [ci][pixel]
  __shared__ float s_bias[BM][33];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t npix = (int64_t)N * H * W;
  const int co0 = blockIdx.x * BM;
  const int row = blockIdx.y % 3;
  const int ci0 = (blockIdx.y / 3) * BN;
  const int64_t kbeg = (int64_t)blockIdx.z * kchunk;
  const int64_t kend = min(npix, kbeg + kchunk);
  const int dy = row - 1;
  f32x4 acc[3][2][2];
  for (int u = 0; u < 3; ++u)
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j) acc[u][i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const bool do_bias = dbias != nullptr && row == 1 && ci0 == 0;
  float bacc[8];
  for (int q = 0; q < 8; ++q) bacc[q] = 0.f;
  const int wm = (wv & 1) * 32, wn = (wv >> 1) * 32;
  // this thread stages pixels k0 + 2 pp and k0 + 2 pp + 1, channels 8 cg .. +8
  const int pp = t & 31, cg = t >> 5;
  const ActView none = {nullptr, 0, 0, 0};
  // image coordinates of the first pixel, advanced by WBK pixels per stage
  int64_t p0 = kbeg + 2 * pp;
  int img = 0, py = 0, px = 0;
  if (p0 < npix) {
    img = (int)(p0 / ((int64_t)H * W));
    const int rem = (int)(p0 - (int64_t)img * H * W);
    py = rem / W;
    px = rem - py * W;
  }
  // loads of the stage at p0 (the thread's two pixels: (img, py, px) and the
  // next one); issued one stage ahead, before the MFMAs of the current one
  // the mask is applied when the stage is written to LDS, so no load waits on another
  const bool masked = mask.p != nullptr;
  uint4 z0, z1, m0, m1, xa[3], xb[3];
  auto fetch = [&]() {
    int img1 = img, py1 = py, px1 = px + 1;
    if (px1 == W) {
      px1 = 0;
      if (++py1 == H) {
        py1 = 0;
        ++img1;
      }
    }
    const bool v0 = p0 < kend, v1 = p0 + 1 < kend;
    z0 = load8(dz, none, none, p0, v0, co0 + 8 * cg);
    z1 = load8(dz, none, none, p0 + 1, v1, co0 + 8 * cg);
    if (masked) {
      m0 = load8(mask, none, none, p0, v0, co0 + 8 * cg);
      m1 = load8(mask, none, none, p0 + 1, v1, co0 + 8 * cg);
    }
    const int sy0 = py + dy, sy1 = py1 + dy;
    const bool r0 = v0 && sy0 >= 0 && sy0 < H, r1 = v1 && sy1 >= 0 && sy1 < H;
    const int64_t row0 = ((int64_t)img * H + sy0) * W, row1 = ((int64_t)img1 * H + sy1) * W;
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int sx0 = px + u - 1, sx1 = px1 + u - 1;
      xa[u] = load8(x1, x2, none, row0 + sx0, r0 && sx0 >= 0 && sx0 < W, ci0 + 8 * cg);
      xb[u] = load8(x1, x2, none, row1 + sx1, r1 && sx1 >= 0 && sx1 < W, ci0 + 8 * cg);
    }
    // advance to the next stage (WBK pixels on; rows may be narrower)
    p0 += WBK;
    px += WBK;
    while (px >= W) {
      px -= W;
      if (++py == H) {
        py = 0;
        ++img;
      }
    }
  };
  fetch();
  for (int64_t k0 = kbeg; k0 < kend; k0 += WBK) {
    const uint4 zz0 = masked ? apply_mask8(z0, m0) : z0, zz1 = masked ? apply_mask8(z1, m1) : z1;
    const uint32_t za[4] = {zz0.x, zz0.y, zz0.z, zz0.w}, zb[4] = {zz1.x, zz1.y, zz1.z, zz1.w};
    __syncthreads();
    // transposed into [channel][pixel], two pixels per 32-bit write
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int sh = 16 * (q & 1);
      const uint32_t lo_z = (za[q >> 1] >> sh) & 0xFFFFu, hi_z = (zb[q >> 1] >> sh) & 0xFFFFu;
      *reinterpret_cast<uint32_t*>(&sA[(8 * cg + q) * WLDK + 2 * pp]) = lo_z | (hi_z << 16);
      if (do_bias) bacc[q] += bf2f((uint16_t)lo_z) + bf2f((uint16_t)hi_z);
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const uint32_t xw0[4] = {xa[u].x, xa[u].y, xa[u].z, xa[u].w};
      const uint32_t xw1[4] = {xb[u].x, xb[u].y, xb[u].z, xb[u].w};
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int sh = 16 * (q & 1);
        const uint32_t lo_x = (xw0[q >> 1] >> sh) & 0xFFFFu, hi_x = (xw1[q >> 1] >> sh) & 0xFFFFu;
        *reinterpret_cast<uint32_t*>(&sB[u][(8 * cg + q) * WLDK + 2 * pp]) = lo_x | (hi_x << 16);
      }
    }
    __syncthreads();
    if (k0 + WBK < kend) fetch();
#pragma unroll
    for (int ks = 0; ks < WBK / 32; ++ks) {
      bf16x8 a[2];
      for (int i = 0; i < 2; ++i)
        a[i] = *reinterpret_cast<const bf16x8*>(
            &sA[(wm + i * 16 + (lane & 15)) * WLDK + 32 * ks + 8 * (lane >> 4)]);
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        bf16x8 b[2];
        for (int j = 0; j < 2; ++j)
          b[j] = *reinterpret_cast<const bf16x8*>(
              &sB[u][(wn + j * 16 + (lane & 15)) * WLDK + 32 * ks + 8 * (lane >> 4)]);
        for (int i = 0; i < 2; ++i)
          for (int j = 0; j < 2; ++j)
            acc[u][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[u][i][j], 0, 0, 0);
      }
    }
  }
  for (int u = 0; u < 3; ++u)
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j) {
        const int ci = ci0 + wn + j * 16 + (lane & 15);
        if (ci >= cin) continue;
        for (int r = 0; r < 4; ++r) {
          const int co = co0 + wm + i * 16 + 4 * (lane >> 4) + r;
          if (co >= cout) continue;
          unsafeAtomicAdd(&dw[((int64_t)(3 * row + u) * cout + co) * cin + ci], acc[u][i][j][r]);
        }
      }
  if (do_bias) {   // block-uniform
    for (int q = 0; q < 8; ++q) s_bias[8 * cg + q][pp] = bacc[q];
    __syncthreads();
    if (t < BM && co0 + t < cout) {
      float sum = 0.f;
      for (int k = 0; k < 32; ++k) sum += s_bias[t][k];
      unsafeAtomicAdd(&dbias[co0 + t], sum);
    }
  }
}

// Weight gradient: dW[tap][co][ci] = sum over pixels p of dz[p][co] x[p + tap][ci]
// (dz masked by the ReLU of the layer's output), the pixels being the K dimension
// of the MFMAs.
//
// A workgroup owns 32 NCO output and 32 NCI input channels and all nine taps. It
// walks down strips of the images, 32 pixels wide, 4 NR rows a step: the step's
// new rows of dz and of the input (34 pixels) go to LDS as they lie in memory,
// [pixel][32 channels], with 16-byte loads and writes; the input's rows stay in a
// ring, so only columns are read twice (34 of 32). The ring and the two dz buffers
// hold the next step beside this one: one barrier a step, the loads of the next
// step in flight while this one is multiplied.
//
// The fragments (8 pixels of one channel per lane) come out of LDS by transposing
// reads (ds_read_b64_tr_b16: four pixels of 16 channels per 16 lanes), so a tap is
// an address offset, and nothing is transposed by the VALU or stored shifted. The
// two 16-channel halves of a pixel swap places every four pixels, so the eight
// pixels that a read takes at a time cover all banks.
//
// A wavefront takes one column of taps (dx) of one 32 x 32 channel pair and four
// of the step's rows: 48 accumulator registers instead of the 144 of nine taps at
// about the same LDS reads per MFMA, since an input row's fragments serve the
// three taps of the column against three rows of dz held in registers.
//
// 4 x 640x480, 96 -> 32 channels: 139 us (402 MB needed, 85 at this card's copy
// rate), 276 on 16 x 8 tiles transposed by the VALU with three shifted copies of
// the input. 8 x 160x120, 128 -> 128: 81 us, 31 of them the closing adds, 147
// with a row of taps per workgroup. What is left is issue and LDS latency at three
// wavefronts per SIMD: without the loads 128 and 84 us, without the MFMAs 152 and
// 78 (before the row halves met in LDS, which took 10 us off the first).
constexpr int WG_W = 32, WG_XW = WG_W + 2;
constexpr int WG_XPITCH = 40;                   // pixels per input row in LDS
constexpr int WG_ZROW = WG_W * 64, WG_XROW = WG_XPITCH * 64;   // bytes per row and 32-channel group
constexpr int WG_SKEW = 128;                    // between the groups of a pixel: other banks

typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));

// Byte offset of 16-byte piece c (of 4) of pixel p of a row in LDS.
__device__ __forceinline__ int wg_piece(int p, int c) {
  return p * 64 + ((c ^ (((p >> 2) & 1) << 1)) << 4);
}

// Fragment: this lane's channel (of the 16 at the address) at pixels 4 g .. 4 g
// + 3 and 16 + 4 g .. of a 32-pixel row, g = lane / 16; dz and the input use
// the same order of pixels.
__device__ __forceinline__ bf16x8 wg_fragment(const char* p, const char* p16) {
  using lds = __attribute__((address_space(3))) short4v*;
  const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds)p);
  const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds)p16);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ bf16x8 wg_fragment(const char* p) { return wg_fragment(p, p + 16 * 64); }

// EDGE: a strip or a step may reach beyond the image, whose last rows in a wavefront's
// four are REM = H % 4. dz is zero there, but the taps that look back pair its first
// column and row beside the image with the input's last, and zero times an infinite
// input is NaN in a sum that has no such term. So the column's address moves on by one
// pixel (zero) and the row's fragment is cleared. Images of whole strips and steps need
// neither and go without: 160x121 of 32 -> 32 channels takes 13.4 us instead of 13.3,
// 242x186 of 256 -> 256 79.5 instead of 77.3.
template <int NCO, int NCI, int NR, bool EDGE, int REM>
__global__ __launch_bounds__(64 * 3 * NCO * NCI * NR, 3) void conv3x3_wgrad_strip_kernel(
    ActView x1, ActView x2, ActView dz, ActView mask, int N, int H, int W, int cout, int cin,
    int n_pairs, int ci_groups, int steps_per_wg, float* __restrict__ dw,
    float* __restrict__ dbias) {
  constexpr int NT = 64 * 3 * NCO * NCI * NR;
  constexpr int SR = 4 * NR;                            // rows per step
  constexpr int RING = 2 * SR + 2;                      // input rows held
  constexpr int ZP = 4 * NCO, XP = 4 * NCI;             // 16-byte pieces per pixel
  static_assert(NT % ZP == 0 && NT % XP == 0, "a thread's pieces share their channels");
  constexpr int ZIT = (SR * WG_W * ZP + NT - 1) / NT;
  constexpr int XIT = (SR * WG_XW * XP + NT - 1) / NT;
  constexpr int HIT = (2 * WG_XW * XP + NT - 1) / NT;   // the two rows above a run or strip
  constexpr int ZGROUP = 2 * SR * WG_ZROW + WG_SKEW, XGROUP = RING * WG_XROW + WG_SKEW;
  __shared__ __attribute__((aligned(16))) char s_z[NCO * ZGROUP];
  __shared__ __attribute__((aligned(16))) char s_x[NCI * XGROUP];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  // an eighth of the (run of steps, channel pair) list to each XCD (workgroups go
  // round the eight of them): the pairs of a run, but for those at an eighth's end,
  // share what they read in its L2
  const int item = ((int)blockIdx.x & 7) * (int)(gridDim.x >> 3) + ((int)blockIdx.x >> 3);
  const int run = item / n_pairs, pair = item % n_pairs;
  const int co0 = (pair / ci_groups) * 32 * NCO, ci0 = (pair % ci_groups) * 32 * NCI;
  const int strips = (W + WG_W - 1) / WG_W, strip_steps = (H + SR - 1) / SR;
  const int n_steps = N * strips * strip_steps;
  const int64_t k_beg64 = (int64_t)run * steps_per_wg;
  if (k_beg64 >= n_steps) return;   // the whole workgroup
  const int k_beg = (int)k_beg64, k_end = min(n_steps, k_beg + steps_per_wg);

  // this thread's pieces: channels 8 zc .. of dz (and mask), 8 xc .. of the input
  const int zc = t % ZP, xc = t % XP;
  const bool z_ok = co0 + 8 * zc < cout;
  const uint16_t* zp = dz.p + dz.offset + co0 + 8 * zc;
  const uint16_t* mp = mask.p ? mask.p + mask.offset + co0 + 8 * zc : nullptr;
  const int xch = ci0 + 8 * xc;
  const bool x_ok = xch < cin, from_1 = xch < x1.c;
  const uint16_t* xp = from_1 ? x1.p + x1.offset + xch : x2.p + x2.offset + (xch - x1.c);
  const int x_stride = from_1 ? x1.stride : x2.stride;
  char* z_dst = s_z + (zc >> 2) * ZGROUP;
  char* x_dst = s_x + (xc >> 2) * XGROUP;
  int img = 0, tx0 = 0, r0 = 0;   // of the step: image, first column, first row
  int64_t base = 0;               // of the image: its first pixel
  auto locate = [&](int k) {
    const int strip = k / strip_steps;
    img = strip / strips;
    tx0 = (strip - img * strips) * WG_W;
    r0 = (k - strip * strip_steps) * SR;
    base = (int64_t)img * H * W;
  };
  // piece p of 34-pixel input rows from row r on (rows of the image only)
  auto load_x = [&](int p, int rows, int r) {
    const int i = p / WG_XW, sy = r + i, sx = tx0 + (p - i * WG_XW) - 1;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (x_ok && i < rows && (unsigned)sy < (unsigned)H && (unsigned)sx < (unsigned)W)
      v = *reinterpret_cast<const uint4*>(xp + (base + sy * W + sx) * x_stride);
    return v;
  };
  // its place when the first of the rows is in ring slot s (< 2 RING - rows)
  auto x_place = [&](int p, int s) {
    const int i = p / WG_XW, c = p - i * WG_XW;
    int at = s + i;
    if (at >= RING) at -= RING;
    return x_dst + at * WG_XROW + wg_piece(c, xc & 3);
  };
  uint4 rz[ZIT], rm[ZIT], rx[XIT];
  auto fetch = [&]() {   // the step's dz rows r0 .. and input rows r0 + 1 ..
#pragma unroll
    for (int u = 0; u < ZIT; ++u) {
      const int p = (t + NT * u) / ZP;
      const int oy = r0 + p / WG_W, ox = tx0 + p % WG_W;
      const int64_t pix = base + oy * W + ox;
      rz[u] = rm[u] = make_uint4(0, 0, 0, 0);
      if (z_ok && p < SR * WG_W && oy < H && ox < W) {
        rz[u] = *reinterpret_cast<const uint4*>(zp + pix * dz.stride);
        if (mp) rm[u] = *reinterpret_cast<const uint4*>(mp + pix * mask.stride);
      }
    }
#pragma unroll
    for (int u = 0; u < XIT; ++u) rx[u] = load_x((t + NT * u) / XP, SR, r0 + 1);
  };
  const int dx = wv % 3, rw = (wv / 3) % NR, ciw = (wv / (3 * NR)) % NCI, cow = wv / (3 * NR * NCI);
  // transposing reads: lane 16 g + i reads 8 bytes of pixel 4 g + i / 4
  const int px = 4 * (lane >> 4) + ((lane >> 2) & 3), ch = (lane & 3) * 8;
  const char* a_base[2];
  const char* b_base[2];
  const char* b_base16[2];   // of the fragment's second half
  auto set_b = [&](int cols) {   // columns of the image from the strip's first on
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const char* group = s_x + ciw * XGROUP + ch;
      const bool back = EDGE && dx == 0;
      b_base[h] = group + wg_piece(px + dx + (back && px == cols ? 1 : 0), 2 * h);
      b_base16[h] = EDGE ? group + wg_piece(px + 16 + dx + (back && px + 16 == cols ? 1 : 0), 2 * h)
                         : b_base[h] + 16 * 64;
    }
  };
  if constexpr (!EDGE) set_b(0);
#pragma unroll
  for (int h = 0; h < 2; ++h)
    a_base[h] = s_z + cow * ZGROUP + rw * 4 * WG_ZROW + wg_piece(px, 2 * h) + ch;
  const bool do_bias = dbias != nullptr && ci0 == 0 && ciw == 0 && dx == 1;   // wavefront-uniform
  f32x4 acc[3][2][2], bacc[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    bacc[a] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[dy][a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const short one = 0x3F80;   // bf16
  const bf16x8 ones = __builtin_bit_cast(bf16x8, (short8v){one, one, one, one, one, one, one, one});

  locate(k_beg);
  fetch();
  int first = 0;   // ring slot of input row r0 - 1
  bool start = true;   // the first step of the run or of a strip
  for (int k = k_beg, zbuf = 0; k < k_end; ++k, zbuf ^= 1) {
    if (start) {   // rows r0 - 1 and r0 as well
      if constexpr (EDGE) set_b(W - tx0);
      __syncthreads();   // the previous strip's fragments have been read
#pragma unroll
      for (int u = 0; u < HIT; ++u) {
        const int p = (t + NT * u) / XP;
        const uint4 v = load_x(p, 2, r0 - 1);
        if (p < 2 * WG_XW) *reinterpret_cast<uint4*>(x_place(p, first)) = v;
      }
    }
#pragma unroll
    for (int u = 0; u < ZIT; ++u) {
      const int p = (t + NT * u) / ZP;
      uint4 v = rz[u];
      if (mp) v = apply_mask8(v, rm[u]);
      if (p < SR * WG_W)
        *reinterpret_cast<uint4*>(z_dst + (zbuf * SR + p / WG_W) * WG_ZROW + wg_piece(p % WG_W, zc & 3)) = v;
    }
#pragma unroll
    for (int u = 0; u < XIT; ++u) {
      const int p = (t + NT * u) / XP;
      if (p < SR * WG_XW) *reinterpret_cast<uint4*>(x_place(p, first + 2)) = rx[u];
    }
    __syncthreads();
    const int rows = H - r0 - 4 * rw;   // of dz in the image, from the wavefront's first
    if (k + 1 < k_end) {
      locate(k + 1);
      start = r0 == 0;
      fetch();
    }
    // input row j of the wavefront's six meets dz row j - dy in tap (dy, dx)
    bf16x8 a[3][2];
    const int a_off = zbuf * SR * WG_ZROW;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      if (j < 4) {
#pragma unroll
        for (int h = 0; h < 2; ++h) a[j % 3][h] = wg_fragment(a_base[h] + a_off + j * WG_ZROW);
      }
      int at = first + 4 * rw + j;
      if (at >= RING) at -= RING;
      bf16x8 b[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) b[h] = wg_fragment(b_base[h] + at * WG_XROW, b_base16[h] + at * WG_XROW);
#pragma unroll
      for (int dy = 2; dy >= 0; --dy) {
        const int i = j - dy;
        if (i < 0 || i >= 4) continue;
        if (EDGE && dy == 0 && j == REM && (REM > 0 || NR > 1)) {
          typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
          const uint32_t keep = rows == REM ? 0u : ~0u;
#pragma unroll
          for (int h = 0; h < 2; ++h)
            b[h] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(uint4v, b[h]) & keep);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 2; ++q)
            acc[dy][h][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i % 3][h], b[q], acc[dy][h][q], 0, 0, 0);
      }
    }
    if (do_bias) {   // apart, so that the loop above stays one block for the scheduler
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          bacc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              wg_fragment(a_base[h] + a_off + j * WG_ZROW), ones, bacc[h], 0, 0, 0);
    }
    first += SR;
    if (first >= RING) first -= RING;
  }
  // acc[dy][h][q][r]: output channel 16 h + 4 (lane / 16) + r, input channel 16 q +
  // lane % 16.  The odd 16-lane rows of q = 0 change places with the even ones of
  // q = 1, so that an atomic instruction covers 32 input channels (a whole
  // 128-byte line) of two output channels instead of 16 of four.
  const int co = co0 + 32 * cow, ci = ci0 + 32 * ciw + (lane & 31);
  const int rows = cout - co - 8 * (lane >> 5);   // valid channels from this lane's first
  float* d0 = dw + ((int64_t)dx * cout + co + 8 * (lane >> 5)) * cin + ci;
  auto add = [&](int dy, int h, int r) {
    const auto sw = __builtin_amdgcn_permlane16_swap(   // by all lanes
        __float_as_uint(acc[dy][h][0][r]), __float_as_uint(acc[dy][h][1][r]), false, false);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int c = 16 * h + 4 * e + r;   // and 8 (lane / 32)
      if (c < rows && ci < cin)
        unsafeAtomicAdd(d0 + ((int64_t)3 * dy * cout + c) * cin, __uint_as_float(sw[e]));
    }
  };
  // the wavefronts that shared the rows of a step meet in LDS first: the adds to dw
  // go through at about one element per clock and memory channel
  if constexpr (NR > 1) {
    static_assert(NCO == 1 && NCI == 1 && 3 * 48 * 64 * 4 <= XGROUP, "the partial sums fit the ring");
    float* s_sum = reinterpret_cast<float*>(s_x) + dx * 48 * 64 + lane;
    for (int k = 1; k < NR; ++k) {
      __syncthreads();   // fragments, or the previous sums, have been read
#pragma unroll
      for (int e = 0; e < 48; ++e)
        if (rw == k) s_sum[e * 64] = acc[e / 16][(e >> 3) & 1][(e >> 2) & 1][e & 3];
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 48; ++e)
        if (rw == 0) acc[e / 16][(e >> 3) & 1][(e >> 2) & 1][e & 3] += s_sum[e * 64];
    }
  }
  if (rw == 0) {
#pragma unroll
    for (int k = 0; k < 24; ++k) add(k / 8, (k >> 2) & 1, k & 3);
  }
  if (do_bias && (lane & 15) == 0) {   // every column holds the row's sum
#pragma unroll
    for (int h = 0; h < 2; ++h)
      for (int r = 0; r < 4; ++r)
        if (co + 16 * h + 4 * (lane >> 4) + r < cout)
          unsafeAtomicAdd(dbias + co + 16 * h + 4 * (lane >> 4) + r, bacc[h][r]);
  }
}

// Narrow weight gradient (cout <= 32): a 32 x 32 channel tile for one row
// of three taps (dy fixed, dx = -1, 0, 1), so each stage's dz and mask loads
// serve three taps.  The four wavefronts split the workgroup's pixels (wave
// w takes every fourth 64-pixel stage), each staging through its own LDS
// region, so only wave-level ordering is needed; the four partial tiles are
// summed once at the end.  Lane l stages pixels 2 (l % 32), 2 (l % 32) + 1
// and channel groups (l / 32) + 2 g, g = 0, 1, of dz and of the three
// shifted inputs.
__global__ __launch_bounds__(256) void conv3x3_wgrad32_kernel(
    ActView x1, ActView x2, ActView dz, ActView mask, int N, int H, int W, int cout, int cin,
    int64_t kchunk, float* __restrict__ dw, float* __restrict__ dbias) {
  __shared__ __attribute__((aligned(16))) union {
    struct {
      uint16_t a[4][32 * WLDK];      // per wave [co][pixel]
      uint16_t b[4][3][32 * WLDK];   // per wave and tap [ci][pixel]
    } st;
    float red[4][3][32][33];         // after the pixel loop: the four waves' tiles
  } sm;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t npix = (int64_t)N * H * W;
  const int row = blockIdx.y % 3;
  const int ci0 = (blockIdx.y / 3) * 32;
  const int64_t kbeg = (int64_t)blockIdx.z * kchunk;
  const int64_t kend = min(npix, kbeg + kchunk);
  const int dy = row - 1;
  const bool do_bias = dbias != nullptr && row == 1 && ci0 == 0;
  const int pp = lane & 31, gh = lane >> 5;
  const ActView none = {nullptr, 0, 0, 0};
  f32x4 acc[3][2][2];
  for (int u = 0; u < 3; ++u)
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j) acc[u][i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float bacc[16];
  for (int q = 0; q < 16; ++q) bacc[q] = 0.f;
  uint16_t* a_s = sm.st.a[wv];
  const bool masked = mask.p != nullptr;
  // image coordinates of the lane's first pixel, advanced by 4 WBK pixels
  // per stage (the stride of one wavefront)
  int64_t p0 = kbeg + (int64_t)wv * WBK + 2 * pp;
  int img = 0, py = 0, px = 0;
  if (p0 < npix) {
    img = (int)(p0 / ((int64_t)H * W));
    const int rem = (int)(p0 - (int64_t)img * H * W);
    py = rem / W;
    px = rem - py * W;
  }
  // [pixel][group] ([tap][pixel][group] for the input), loaded one stage
  // ahead; the mask is applied when the stage is written to LDS, so no load
  // waits on another
  uint4 z[2][2], zm[2][2], xv[3][2][2];
  auto fetch = [&]() {
    int img1 = img, py1 = py, px1 = px + 1;
    if (px1 == W) {
      px1 = 0;
      if (++py1 == H) {
        py1 = 0;
        ++img1;
      }
    }
    const bool v0 = p0 < kend, v1 = p0 + 1 < kend;
    const int sy0 = py + dy, sy1 = py1 + dy;
    const bool r0 = v0 && sy0 >= 0 && sy0 < H, r1 = v1 && sy1 >= 0 && sy1 < H;
    const int64_t row0 = ((int64_t)img * H + sy0) * W, row1 = ((int64_t)img1 * H + sy1) * W;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int cg = gh + 2 * g;   // channel group 0..3
      z[0][g] = load8(dz, none, none, p0, v0, 8 * cg);
      z[1][g] = load8(dz, none, none, p0 + 1, v1, 8 * cg);
      if (masked) {
        zm[0][g] = load8(mask, none, none, p0, v0, 8 * cg);
        zm[1][g] = load8(mask, none, none, p0 + 1, v1, 8 * cg);
      }
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int sx0 = px + u - 1, sx1 = px1 + u - 1;
        xv[u][0][g] = load8(x1, x2, none, row0 + sx0, r0 && sx0 >= 0 && sx0 < W, ci0 + 8 * cg);
        xv[u][1][g] = load8(x1, x2, none, row1 + sx1, r1 && sx1 >= 0 && sx1 < W, ci0 + 8 * cg);
      }
    }
    p0 += 4 * WBK;
    px += 4 * WBK;
    while (px >= W) {
      px -= W;
      if (++py == H) {
        py = 0;
        ++img;
      }
    }
  };
  fetch();
  for (int64_t k0 = kbeg + (int64_t)wv * WBK; k0 < kend; k0 += 4 * WBK) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int cg = gh + 2 * g;
      const uint4 z0 = masked ? apply_mask8(z[0][g], zm[0][g]) : z[0][g];
      const uint4 z1 = masked ? apply_mask8(z[1][g], zm[1][g]) : z[1][g];
      const uint32_t za[4] = {z0.x, z0.y, z0.z, z0.w};
      const uint32_t zb[4] = {z1.x, z1.y, z1.z, z1.w};
      // transposed into [channel][pixel], two pixels per 32-bit write
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int sh = 16 * (q & 1);
        const uint32_t lo_z = (za[q >> 1] >> sh) & 0xFFFFu, hi_z = (zb[q >> 1] >> sh) & 0xFFFFu;
        *reinterpret_cast<uint32_t*>(&a_s[(8 * cg + q) * WLDK + 2 * pp]) = lo_z | (hi_z << 16);
        if (do_bias) bacc[8 * g + q] += bf2f((uint16_t)lo_z) + bf2f((uint16_t)hi_z);
      }
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const uint32_t xa[4] = {xv[u][0][g].x, xv[u][0][g].y, xv[u][0][g].z, xv[u][0][g].w};
        const uint32_t xb[4] = {xv[u][1][g].x, xv[u][1][g].y, xv[u][1][g].z, xv[u][1][g].w};
        uint16_t* b_s = sm.st.b[wv][u];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int sh = 16 * (q & 1);
          const uint32_t lo_x = (xa[q >> 1] >> sh) & 0xFFFFu, hi_x = (xb[q >> 1] >> sh) & 0xFFFFu;
          *reinterpret_cast<uint32_t*>(&b_s[(8 * cg + q) * WLDK + 2 * pp]) = lo_x | (hi_x << 16);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (k0 + 4 * WBK < kend) fetch();
#pragma unroll
    for (int ks = 0; ks < WBK / 32; ++ks) {
      bf16x8 a[2];
      for (int i = 0; i < 2; ++i)
        a[i] = *reinterpret_cast<const bf16x8*>(&a_s[(i * 16 + (lane & 15)) * WLDK + 32 * ks + 8 * (lane >> 4)]);
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const uint16_t* b_s = sm.st.b[wv][u];
        bf16x8 b[2];
        for (int j = 0; j < 2; ++j)
          b[j] = *reinterpret_cast<const bf16x8*>(&b_s[(j * 16 + (lane & 15)) * WLDK + 32 * ks + 8 * (lane >> 4)]);
        for (int i = 0; i < 2; ++i)
          for (int j = 0; j < 2; ++j)
            acc[u][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[u][i][j], 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();   // fragments read before the next stage's writes
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  // sum the four wavefronts' tiles: red[w][u][co][ci] (over the staging buffers)
  __syncthreads();
  float(*s_red)[3][32][33] = sm.red;
  for (int u = 0; u < 3; ++u)
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j)
        for (int r = 0; r < 4; ++r)
          s_red[wv][u][i * 16 + 4 * (lane >> 4) + r][j * 16 + (lane & 15)] = acc[u][i][j][r];
  __syncthreads();
  for (int e = t; e < 3 * 32 * 32; e += 256) {
    const int u = e >> 10, co = (e >> 5) & 31, ci = e & 31;
    if (co >= cout || ci0 + ci >= cin) continue;
    const float v = s_red[0][u][co][ci] + s_red[1][u][co][ci] + s_red[2][u][co][ci] + s_red[3][u][co][ci];
    unsafeAtomicAdd(&dw[((int64_t)(3 * row + u) * cout + co) * cin + ci0 + ci], v);
  }
  if (do_bias) {   // block-uniform
    __syncthreads();   // s_red is reused for the per-wave channel sums
    float* sb = &s_red[0][0][0][0];
    for (int q = 0; q < 16; ++q) {
      float v = bacc[q];
      for (int d = 1; d < 32; d <<= 1) v += __shfl_xor(v, d, 64);   // over the 32 pixel pairs
      bacc[q] = v;
    }
    if (pp == 0)
      for (int g = 0; g < 2; ++g)
        for (int q = 0; q < 8; ++q) sb[wv * 32 + 8 * (gh + 2 * g) + q] = bacc[8 * g + q];
    __syncthreads();
    if (t < 32 && t < cout)
      unsafeAtomicAdd(&dbias[t], sb[t] + sb[32 + t] + sb[64 + t] + sb[96 + t]);
  }
}

// w [9][cout][cin] -> wt [9][cin][cout] with taps mirrored (backward data)
__global__ void flip_weights_kernel(const uint16_t* __restrict__ w, int cout, int cin,
                                    uint16_t* __restrict__ wt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = 9LL * cout * cin;
  if (i >= total) return;
  const int tap = (int)(i / ((int64_t)cout * cin));
  const int rem = (int)(i - (int64_t)tap * cout * cin);
  const int co = rem / cin, ci = rem % cin;
  wt[((int64_t)(8 - tap) * cin + ci) * cout + co] = w[i];
}

__device__ __forceinline__ void unpack8(uint4 u, float* v) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
  for (int k = 0; k < 4; ++k) {
    v[2 * k] = bf2f((uint16_t)(w[k] & 0xFFFFu));
    v[2 * k + 1] = bf2f((uint16_t)(w[k] >> 16));
  }
}

__device__ __forceinline__ uint4 pack8(const float* v) {
  uint32_t w[4];
  for (int k = 0; k < 4; ++k) w[k] = (uint32_t)f2bf(v[2 * k]) | ((uint32_t)f2bf(v[2 * k + 1]) << 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// 8 channels per thread (channel counts, strides and offsets are multiples of 8)
__global__ void avgpool2_kernel(ActView x, int N, int H, int W, uint16_t* __restrict__ y,
                                int y_stride) {
  const int Ho = H / 2, Wo = W / 2;
  const int c8n = x.c / 8;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)N * Ho * Wo * c8n;
  if (i >= total) return;
  const int c = (int)(i % c8n) * 8;
  const int64_t q = i / c8n;
  const int n = (int)(q / ((int64_t)Ho * Wo));
  const int r = (int)(q - (int64_t)n * Ho * Wo);
  const int yo = r / Wo, xo = r % Wo;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) {
      const int64_t p = ((int64_t)n * H + 2 * yo + a) * W + 2 * xo + b;
      float v[8];
      unpack8(*reinterpret_cast<const uint4*>(x.p + p * x.stride + x.offset + c), v);
      for (int k = 0; k < 8; ++k) s[k] += v[k];
    }
  for (int k = 0; k < 8; ++k) s[k] *= 0.25f;
  *reinterpret_cast<uint4*>(y + q * y_stride + c) = pack8(s);
}

// dx[p][c] (+)= dy[pool(p)][c] / 4 (dx may be a channel slice; accumulate adds)
// 8 channels per thread (see upsample2_kernel)
__global__ void avgpool2_bwd_kernel(ActView dy, int N, int H, int W, uint16_t* __restrict__ dx,
                                    int dx_stride, int dx_offset, int accumulate,
                                    const uint16_t* __restrict__ add_src, int add_stride,
                                    int add_offset) {
  const int c8n = dy.c / 8;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)N * H * W * c8n;
  if (i >= total) return;
  const int c = (int)(i % c8n) * 8;
  const int64_t p = i / c8n;
  const int n = (int)(p / ((int64_t)H * W));
  const int r = (int)(p - (int64_t)n * H * W);
  const int yy = r / W, xx = r % W;
  const int Ho = H / 2, Wo = W / 2;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (yy / 2 < Ho && xx / 2 < Wo) {
    const int64_t q = ((int64_t)n * Ho + yy / 2) * Wo + xx / 2;
    unpack8(*reinterpret_cast<const uint4*>(dy.p + q * dy.stride + dy.offset + c), v);
    for (int k = 0; k < 8; ++k) v[k] *= 0.25f;
  }
  if (add_src) {
    float a[8];
    unpack8(*reinterpret_cast<const uint4*>(add_src + p * add_stride + add_offset + c), a);
    for (int k = 0; k < 8; ++k) v[k] += a[k];
  }
  uint4* o = reinterpret_cast<uint4*>(dx + p * dx_stride + dx_offset + c);
  if (accumulate) {
    float cur[8];
    unpack8(*o, cur);
    for (int k = 0; k < 8; ++k) v[k] = cur[k] + v[k];
  }
  *o = pack8(v);
}

// 8 channels (16 bytes) per thread; channel counts, strides and offsets are
// multiples of 8.
__global__ void upsample2_kernel(ActView x, int N, int H, int W, uint16_t* __restrict__ y,
                                 int y_stride, int y_offset) {
  // x is (H/2) x (W/2); y is H x W
  const int c8n = x.c / 8;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)N * H * W * c8n;
  if (i >= total) return;
  const int c = (int)(i % c8n) * 8;
  const int64_t p = i / c8n;
  const int n = (int)(p / ((int64_t)H * W));
  const int r = (int)(p - (int64_t)n * H * W);
  const int yy = r / W, xx = r % W;
  const int64_t q = ((int64_t)n * (H / 2) + yy / 2) * (W / 2) + xx / 2;
  *reinterpret_cast<uint4*>(y + p * y_stride + y_offset + c) =
      *reinterpret_cast<const uint4*>(x.p + q * x.stride + x.offset + c);
}

// 8 channels per thread (see avgpool2_kernel)
__global__ void upsample2_bwd_kernel(ActView dy, int N, int H, int W, uint16_t* __restrict__ dx,
                                     int dx_stride) {
  // dy is H x W, dx is (H/2) x (W/2): dx = sum of the 2x2 block
  const int Ho = H / 2, Wo = W / 2;
  const int c8n = dy.c / 8;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)N * Ho * Wo * c8n;
  if (i >= total) return;
  const int c = (int)(i % c8n) * 8;
  const int64_t q = i / c8n;
  const int n = (int)(q / ((int64_t)Ho * Wo));
  const int r = (int)(q - (int64_t)n * Ho * Wo);
  const int yo = r / Wo, xo = r % Wo;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) {
      const int64_t p = ((int64_t)n * H + 2 * yo + a) * W + 2 * xo + b;
      float v[8];
      unpack8(*reinterpret_cast<const uint4*>(dy.p + p * dy.stride + dy.offset + c), v);
      for (int k = 0; k < 8; ++k) s[k] += v[k];
    }
  *reinterpret_cast<uint4*>(dx + q * dx_stride + c) = pack8(s);
}

// planar float32 RGB [N][3][H][W] -> NHWC bf16 with `stride` channels (zero padded)
__global__ void rgb_to_nhwc_kernel(const float* __restrict__ rgb, int N, int H, int W,
                                   uint16_t* __restrict__ x, int stride) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t npix = (int64_t)N * H * W;
  if (p >= npix) return;
  const int n = (int)(p / ((int64_t)H * W));
  const int64_t r = p - (int64_t)n * H * W;
  for (int c = 0; c < stride; ++c)
    x[p * stride + c] = c < 3 ? f2bf(rgb[((int64_t)n * 3 + c) * H * W + r]) : (uint16_t)0;
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ src, uint16_t* __restrict__ dst,
                                   int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = f2bf(src[i]);
}

// Per-pixel head on float32 features [p][2] (a 1x1 conv already applied by
// conv3x3 with a 1x1 kernel would waste 8/9 of the work; the head is a 1x1
// conv): out[n][k][y][x] = b[k] + sum_c w[k][c] f[p][c].
__global__ void head_fwd_kernel(ActView f, int N, int H, int W, const float* __restrict__ w,
                                const float* __restrict__ b, float* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t npix = (int64_t)N * H * W;
  if (p >= npix) return;
  float o0 = b[0], o1 = b[1];
  for (int c = 0; c < f.c; ++c) {
    const float v = bf2f(f.p[p * f.stride + f.offset + c]);
    o0 += w[c] * v;
    o1 += w[f.c + c] * v;
  }
  const int n = (int)(p / ((int64_t)H * W));
  const int64_t r = p - (int64_t)n * H * W;
  out[((int64_t)n * 2 + 0) * H * W + r] = o0;
  out[((int64_t)n * 2 + 1) * H * W + r] = o1;
}

// The same with 16-byte loads when the channels come in whole groups of 8
// (count, stride and offset multiples of 8): a thread reads its pixel's
// features 8 at a time, the sums run over the channels in the same order.
__global__ __launch_bounds__(256) void head_fwd8_kernel(ActView f, int N, int H, int W,
                                                        const float* __restrict__ w,
                                                        const float* __restrict__ b,
                                                        float* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t npix = (int64_t)N * H * W;
  if (p >= npix) return;
  const uint16_t* src = f.p + p * f.stride + f.offset;
  float o0 = b[0], o1 = b[1];
  for (int c = 0; c < f.c; c += 8) {
    const uint4 v = *reinterpret_cast<const uint4*>(src + c);
    const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float lo = __uint_as_float(wd[i] << 16), hi = __uint_as_float(wd[i] & 0xFFFF0000u);
      o0 += w[c + 2 * i] * lo;
      o1 += w[f.c + c + 2 * i] * lo;
      o0 += w[c + 2 * i + 1] * hi;
      o1 += w[f.c + c + 2 * i + 1] * hi;
    }
  }
  const int n = (int)(p / ((int64_t)H * W));
  const int64_t r = p - (int64_t)n * H * W;
  out[((int64_t)n * 2 + 0) * H * W + r] = o0;
  out[((int64_t)n * 2 + 1) * H * W + r] = o1;
}

// Head backward: dF[p][c] = sum_k w[k][c] dout[k][p] masked by the feature's
// ReLU (f > 0); dW, db accumulated with per-block reductions and atomics.
// Threads (channel lane t % 32, pixel group t / 32): each thread walks every
// eighth pixel of the workgroup's 256-pixel chunks (grid-stride), handling
// channels t % 32 + 32 k; the weight and bias partials stay in registers and
// are reduced over the eight groups once per workgroup.
constexpr int kHeadMaxSlots = 2;   // channels per thread: up to 64 feature channels (the C ABI limit)

__global__ __launch_bounds__(256) void head_bwd_kernel(ActView f, int N, int H, int W,
                                                       const float* __restrict__ w,
                                                       const float* __restrict__ dout,
                                                       uint16_t* __restrict__ df, int df_stride,
                                                       float* __restrict__ dw,
                                                       float* __restrict__ db) {
  __shared__ float s_red[8][2 * 32 * kHeadMaxSlots + 2];
  const int t = threadIdx.x, cl = t & 31, pg = t >> 5;
  const int64_t npix = (int64_t)N * H * W;
  const int64_t hw = (int64_t)H * W;
  const int slots = (f.c + 31) / 32;
  float a0[kHeadMaxSlots], a1[kHeadMaxSlots], w0[kHeadMaxSlots], w1[kHeadMaxSlots];
  for (int k = 0; k < kHeadMaxSlots; ++k) {
    a0[k] = a1[k] = 0.f;
    const int c = cl + 32 * k;
    w0[k] = (k < slots && c < f.c) ? w[c] : 0.f;
    w1[k] = (k < slots && c < f.c) ? w[f.c + c] : 0.f;
  }
  float b0 = 0.f, b1 = 0.f;
  for (int64_t base = (int64_t)blockIdx.x * 256; base < npix; base += (int64_t)gridDim.x * 256) {
    for (int j = pg; j < 256; j += 8) {
      const int64_t p = base + j;
      if (p >= npix) break;
      const int n = (int)(p / hw);
      const int64_t r = p - (int64_t)n * hw;
      const float g0 = dout[((int64_t)n * 2 + 0) * hw + r];
      const float g1 = dout[((int64_t)n * 2 + 1) * hw + r];
      if (cl == 0) {
        b0 += g0;
        b1 += g1;
      }
      for (int k = 0; k < kHeadMaxSlots; ++k) {
        const int c = cl + 32 * k;
        if (k >= slots || c >= f.c) break;
        const float v = bf2f(f.p[p * f.stride + f.offset + c]);
        a0[k] += g0 * v;
        a1[k] += g1 * v;
        df[p * df_stride + c] = f2bf(v > 0.f ? (w0[k] * g0 + w1[k] * g1) : 0.f);
      }
    }
  }
  for (int k = 0; k < kHeadMaxSlots; ++k) {
    s_red[pg][32 * k + cl] = a0[k];
    s_red[pg][32 * kHeadMaxSlots + 32 * k + cl] = a1[k];
  }
  if (cl == 0) {
    s_red[pg][64 * kHeadMaxSlots] = b0;
    s_red[pg][64 * kHeadMaxSlots + 1] = b1;
  }
  __syncthreads();
  for (int k = t; k < 2 * f.c + 2; k += 256) {
    // k < f.c: dw row 0; f.c <= k < 2 f.c: dw row 1; then the two biases
    const int col = k < f.c ? k : k < 2 * f.c ? 32 * kHeadMaxSlots + (k - f.c)
                                              : 64 * kHeadMaxSlots + (k - 2 * f.c);
    float sum = 0.f;
    for (int g = 0; g < 8; ++g) sum += s_red[g][col];
    if (k < 2 * f.c)
      unsafeAtomicAdd(&dw[k], sum);
    else
      unsafeAtomicAdd(&db[k - 2 * f.c], sum);
  }
}

// Head backward with 16-byte accesses (channel counts, strides and offsets
// multiples of 8): thread t owns channel group t % G (8 channels, G = C / 8)
// of pixel t / G of each 256 / G-pixel step (grid-stride), loads and stores
// its 8 features and gradients at once, and keeps 16 weight partials in
// registers; the partials of a group are summed over the workgroup in LDS
// once, then added with one atomic per weight.
constexpr int kHead8Groups = 8;   // up to 64 channels

__global__ __launch_bounds__(256) void head_bwd8_kernel(ActView f, int N, int H, int W,
                                                        const float* __restrict__ w,
                                                        const float* __restrict__ dout,
                                                        uint16_t* __restrict__ df, int df_stride,
                                                        float* __restrict__ dw,
                                                        float* __restrict__ db) {
  __shared__ float s_red[256][19];
  const int t = threadIdx.x;
  const int G = f.c / 8;
  const int per = 256 / G;          // pixels per step
  const int cg = t % G, pix = t / G;
  const bool active = pix < per;    // 256 not a multiple of G: the last threads idle
  const int64_t npix = (int64_t)N * H * W;
  const int64_t hw = (int64_t)H * W;
  float w0[8], w1[8], a0[8], a1[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    w0[i] = w[8 * cg + i];
    w1[i] = w[f.c + 8 * cg + i];
    a0[i] = a1[i] = 0.f;
  }
  float b0 = 0.f, b1 = 0.f;
  if (active) {
    for (int64_t p = (int64_t)blockIdx.x * per + pix; p < npix; p += (int64_t)gridDim.x * per) {
      const int n = (int)(p / hw);
      const int64_t r = p - (int64_t)n * hw;
      const float g0 = dout[((int64_t)n * 2 + 0) * hw + r];
      const float g1 = dout[((int64_t)n * 2 + 1) * hw + r];
      if (cg == 0) {
        b0 += g0;
        b1 += g1;
      }
      const uint4 v = *reinterpret_cast<const uint4*>(f.p + p * f.stride + f.offset + 8 * cg);
      const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
      uint32_t od[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float lo = __uint_as_float(wd[i] << 16), hi = __uint_as_float(wd[i] & 0xFFFF0000u);
        a0[2 * i] += g0 * lo;
        a1[2 * i] += g1 * lo;
        a0[2 * i + 1] += g0 * hi;
        a1[2 * i + 1] += g1 * hi;
        const uint16_t dlo = f2bf(lo > 0.f ? (w0[2 * i] * g0 + w1[2 * i] * g1) : 0.f);
        const uint16_t dhi = f2bf(hi > 0.f ? (w0[2 * i + 1] * g0 + w1[2 * i + 1] * g1) : 0.f);
        od[i] = (uint32_t)dlo | ((uint32_t)dhi << 16);
      }
      *reinterpret_cast<uint4*>(df + p * df_stride + 8 * cg) = make_uint4(od[0], od[1], od[2], od[3]);
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    s_red[t][i] = a0[i];
    s_red[t][8 + i] = a1[i];
  }
  s_red[t][16] = b0;   // nonzero in the group-0 threads only
  s_red[t][17] = b1;
  __syncthreads();
  // weight (row, channel 8 g + i): the sum over the threads of group g;
  // bias k: the sum over the group-0 threads
  for (int k = t; k < 2 * f.c + 2; k += 256) {
    float sum = 0.f;
    if (k < 2 * f.c) {
      const int row = k / f.c, c = k - row * f.c, g = c / 8, i = c % 8;
      for (int u = g; u < per * G; u += G) sum += s_red[u][8 * row + i];
      unsafeAtomicAdd(&dw[k], sum);
    } else {
      for (int u = 0; u < per * G; u += G) sum += s_red[u][16 + (k - 2 * f.c)];
      unsafeAtomicAdd(&db[k - 2 * f.c], sum);
    }
  }
}

// Depth supervision: pred [N][2][H][W] = (log depth, log scale); target depth
// [N][H][W] (<= 0 marks invalid); log-scale target log(depth / fx).
// loss = mean over valid of |pred0 - log d| + |pred1 - log(d / fx)|.
__global__ __launch_bounds__(256) void depth_loss_kernel(const float* __restrict__ pred,
                                                         const float* __restrict__ depth, int N,
                                                         int H, int W, float fx,
                                                         const int* __restrict__ count,
                                                         float* __restrict__ dpred,
                                                         double* __restrict__ loss) {
  __shared__ float s_acc[4];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t npix = (int64_t)N * H * W;
  float l = 0.f;
  if (p < npix) {
    const int n = (int)(p / ((int64_t)H * W));
    const int64_t r = p - (int64_t)n * H * W;
    const float d = depth[p];
    const float inv = 1.0f / (float)max(*count, 1);
    float g0 = 0.f, g1 = 0.f;
    if (d > 0.f) {
      const float ld = logf(d), ls = logf(d / fx);
      const float e0 = pred[((int64_t)n * 2 + 0) * H * W + r] - ld;
      const float e1 = pred[((int64_t)n * 2 + 1) * H * W + r] - ls;
      l = (fabsf(e0) + fabsf(e1)) * inv;
      g0 = e0 > 0.f ? inv : (e0 < 0.f ? -inv : 0.f);
      g1 = e1 > 0.f ? inv : (e1 < 0.f ? -inv : 0.f);
    }
    dpred[((int64_t)n * 2 + 0) * H * W + r] = g0;
    dpred[((int64_t)n * 2 + 1) * H * W + r] = g1;
  }
  for (int d = 32; d > 0; d >>= 1) l += __shfl_xor(l, d, 64);
  if ((threadIdx.x & 63) == 0) s_acc[threadIdx.x >> 6] = l;
  __syncthreads();
  if (threadIdx.x == 0 && loss) atomicAdd(loss, (double)(s_acc[0] + s_acc[1] + s_acc[2] + s_acc[3]));
}

__global__ void count_valid_kernel(const float* __restrict__ depth, int64_t n,
                                   int* __restrict__ count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int c = (i < n && depth[i] > 0.f) ? 1 : 0;
  for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d, 64);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(count, c);
}

__global__ void zero_kernel(uint32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

ActView view(const gs_act* a) {
  ActView v{nullptr, 0, 0, 0};
  if (a) {
    v.p = static_cast<const uint16_t*>(a->data);
    v.c = a->c;
    v.stride = a->stride;
    v.offset = a->offset;
  }
  return v;
}

unsigned blocks(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// The patch convolution is persistent: as many workgroups as the device holds at
// once (split over the channel tiles), never more than there are tiles.
template <int JN, bool MASKED, bool ONE>
hipError_t launch_patch(ActView x1, ActView x2, ActView mask, int n, int h, int w,
                        const uint16_t* wp, int cout, int cin, const float* bias, int relu,
                        uint16_t* yp, int ys, int yo, float* yf, int yf_stride, unsigned tiles,
                        hipStream_t s) {
  const unsigned gy = (unsigned)((cout + 16 * JN - 1) / (16 * JN));
  const int resident = resident_workgroups((const void*)conv3x3_patch_kernel<JN, MASKED, ONE>, 64 * PT / PR);
  // as many columns of tiles as the CUs hold at once with all their channel groups: a
  // workgroup that has to wait for a place comes on top (518 for 325 us, 384 of 128
  // channels at 4 x 320x240, with 516 of them for 512 places)
  unsigned columns = tiles;
  if (resident > 0) {
    const unsigned most = (unsigned)resident / 8 / gy * 8;
    columns = std::min(tiles, most ? most : std::max(1u, (unsigned)resident / gy));
  }
  const unsigned grid = (columns + 7) / 8 * 8 * gy;
  hipLaunchKernelGGL((conv3x3_patch_kernel<JN, MASKED, ONE>), dim3(grid), dim3(64 * PT / PR), 0, s, x1, x2,
                     mask, n, h, w, wp, cout, cin, bias, relu, yp, ys, yo, yf, yf_stride, (int)columns);
  return hipGetLastError();
}

}  // namespace

hipError_t nn_conv3x3(const gs_act* x1, const gs_act* x2, const gs_act* mask, const void* w,
                      int cout, const float* bias, int relu, gs_act* y, float* yf, int yf_stride,
                      hipStream_t s) {
  const int cin = x1->c + (x2 ? x2->c : 0);
  auto* yp = y ? static_cast<uint16_t*>(y->data) : nullptr;
  const int ys = y ? y->stride : 0, yo = y ? y->offset : 0;
  const auto* wp = static_cast<const uint16_t*>(w);
  const unsigned tiles = (unsigned)(x1->n * ((x1->h + PT - 1) / PT) * ((x1->w + PT - 1) / PT));
  // 32 output channels per workgroup up to 32 channels, for an odd number of
  // 32-channel groups (96 in 64-channel workgroups would waste a quarter of the
  // products), and where 64-channel workgroups would number fewer than 1,024, two for
  // each of the 512 places: half as much to a workgroup fills the places of a small
  // layer and leaves less in the last turn of a middling one, while in a large one
  // both halves of the channels would read the input.  The line at 512, 1,024 or
  // 2,048 (us): 320x240, 128 -> 128 31, 28, 28; 8 x 160x120, 64 -> 64 21, 18, 18 and
  // 384 -> 128 133, 130, 155.
  const bool narrow =
      cout <= 32 || cout % 64 == 32 || tiles * (unsigned)((cout + 63) / 64) < 1024u;
  const bool one = cin <= PCC;
#define GS_PATCH(J, M, O)                                                                     \
  launch_patch<J, M, O>(view(x1), view(x2), view(mask), x1->n, x1->h, x1->w, wp, cout, cin, bias, \
                        relu, yp, ys, yo, yf, yf_stride, tiles, s)
  if (narrow && one) return mask ? GS_PATCH(2, true, true) : GS_PATCH(2, false, true);
  if (narrow) return mask ? GS_PATCH(2, true, false) : GS_PATCH(2, false, false);
  return mask ? GS_PATCH(4, true, false) : GS_PATCH(4, false, false);
#undef GS_PATCH
}

hipError_t nn_conv3x3_wgrad(const gs_act* x1, const gs_act* x2, const gs_act* dz,
                            const gs_act* mask, float* dw, float* dbias, hipStream_t s) {
  const int cin = x1->c + (x2 ? x2->c : 0);
  const int cout = dz->c;
  const int64_t npix = (int64_t)x1->n * x1->h * x1->w;
  if (cin % 8 == 0 && x1->c % 8 == 0 && cout % 8 == 0) {
    // 32 x 32 channels per workgroup up to 32 output channels and for little work:
    // fewer runs share a pair then, and with them go the closing adds, which bound
    // small layers; else 64 output channels, and 64 input channels unless these are
    // an odd number of 32-channel groups, which halves what is staged per product.
    // 32 x 32 against 64 x 64 (us, millions of pixels and channel pairs): 160x120,
    // 128 -> 128 (0.3) 23 and 30; 320x240, 128 -> 128 (1.2) 50 and 58; 160x120, 256 ->
    // 256 (1.2) 48 and 51, as four 80x60 58 and 55; 8 x 160x120, 192 -> 64 (1.8) 70
    // and 67, 128 -> 128 (2.5) 86 and 81; 320x240, 256 -> 256 (4.9) 159 and 106.
    const int64_t work = npix * ((cin + 31) / 32) * ((cout + 31) / 32);
    const bool one_co = cout <= 32 || work <= 1250000, one_ci = one_co || (cin + 31) / 32 % 2 == 1;
    const int rows = one_co ? 8 : 4;   // per step
    const int steps = x1->n * ((x1->w + WG_W - 1) / WG_W) * ((x1->h + rows - 1) / rows);
    const int ci_groups = one_ci ? (cin + 31) / 32 : (cin + 63) / 64;
    const int pairs = ci_groups * (one_co ? (cout + 31) / 32 : (cout + 63) / 64);
    // B workgroups share the steps S pairs, about 3 us each, and every one closes with
    // 9,216 adds per 32 x 32 channel pair of its `own`, which the memory channels that
    // hold dw (36 KB per pair) take at some 60 per ns and pair, 200 in all: the sum of
    // both is least at B^2 = S pairs / own by 16 per pair of dw, at most 50.  From one
    // to one per CU: a second on some CUs makes these the last (8 x 160x120, 96 -> 32:
    // 45 us with 424 workgroups, 32 with 256), one on each costs as much in adds as it
    // hides (4 x 640x480, 32 -> 32: 94 and 72 us).
    const int own = one_co ? 1 : one_ci ? 2 : 4;
    const double ratio = std::min(50.0, 16.0 * own * pairs);
    const int blocks = std::min(256, (int)std::sqrt(ratio * steps * pairs / own));
    const int runs_wanted = std::max(1, blocks / pairs);
    const int per = (steps + runs_wanted - 1) / runs_wanted;
    const int runs = (steps + per - 1) / per;
    const unsigned grid = (unsigned)((runs * (int64_t)pairs + 7) / 8 * 8);
#define GS_WGRAD_EDGE(O, I, R, E, M)                                                            \
  hipLaunchKernelGGL((conv3x3_wgrad_strip_kernel<O, I, R, E, M>), dim3(grid),                   \
                     dim3(64 * 3 * O * I * R), 0, s, view(x1), view(x2), view(dz), view(mask),  \
                     x1->n, x1->h, x1->w, cout, cin, pairs, ci_groups, per, dw, dbias)
#define GS_WGRAD(O, I, R)                                                                       \
  do {                                                                                          \
    const int rem = x1->h % 4;                                                                  \
    if (x1->w % WG_W == 0 && x1->h % rows == 0) GS_WGRAD_EDGE(O, I, R, false, 0);               \
    else if (rem == 0) GS_WGRAD_EDGE(O, I, R, true, 0);                                         \
    else if (rem == 1) GS_WGRAD_EDGE(O, I, R, true, 1);                                         \
    else if (rem == 2) GS_WGRAD_EDGE(O, I, R, true, 2);                                         \
    else GS_WGRAD_EDGE(O, I, R, true, 3);                                                       \
  } while (0)
    if (one_co) GS_WGRAD(1, 1, 2);
    else if (one_ci) GS_WGRAD(2, 1, 1);
    else GS_WGRAD(2, 2, 1);
#undef GS_WGRAD_EDGE
#undef GS_WGRAD
    return hipGetLastError();
  }
  // pixel chunks: enough workgroups to fill the chip, each long enough that
  // its 4096 atomic adds into dw are few next to its MFMA work
  if (cout <= 32) {   // 32 x 32 channel tiles, a row of taps each (see conv3x3_wgrad32_kernel)
    const int64_t tiles = 3 * (int64_t)((cin + 31) / 32);
    const int64_t nk = std::max<int64_t>(1, kWgrad32Blocks / tiles);
    int64_t kchunk = (npix + nk - 1) / nk;
    kchunk = std::max<int64_t>(4 * WBK, (kchunk + 4 * WBK - 1) / (4 * WBK) * (4 * WBK));
    const dim3 grid(1, (unsigned)(3 * ((cin + 31) / 32)), (unsigned)((npix + kchunk - 1) / kchunk));
    hipLaunchKernelGGL(conv3x3_wgrad32_kernel, grid, dim3(256), 0, s, view(x1), view(x2),
                       view(dz), view(mask), x1->n, x1->h, x1->w, cout, cin, kchunk, dw, dbias);
    return hipGetLastError();
  }
  const int64_t tiles = (int64_t)((cout + BM - 1) / BM) * 3 * ((cin + BN - 1) / BN);
  const int64_t nk = std::max<int64_t>(1, kWgradBlocks / tiles);
  int64_t kchunk = (npix + nk - 1) / nk;
  kchunk = std::max<int64_t>(WBK, (kchunk + WBK - 1) / WBK * WBK);
  const dim3 grid((unsigned)((cout + BM - 1) / BM), (unsigned)(3 * ((cin + BN - 1) / BN)),
                  (unsigned)((npix + kchunk - 1) / kchunk));
  hipLaunchKernelGGL(conv3x3_wgrad_kernel, grid, dim3(256), 0, s, view(x1), view(x2), view(dz),
                     view(mask), x1->n, x1->h, x1->w, cout, cin, kchunk, dw, dbias);
  return hipGetLastError();
}

hipError_t nn_flip_weights(const void* w, int cout, int cin, void* wt, hipStream_t s) {
  hipLaunchKernelGGL(flip_weights_kernel, dim3(blocks(9LL * cout * cin)), dim3(256), 0, s,
                     static_cast<const uint16_t*>(w), cout, cin, static_cast<uint16_t*>(wt));
  return hipGetLastError();
}

hipError_t nn_avgpool2(const gs_act* x, gs_act* y, hipStream_t s) {
  const int64_t total = (int64_t)x->n * (x->h / 2) * (x->w / 2) * (x->c / 8);
  hipLaunchKernelGGL(avgpool2_kernel, dim3(blocks(total)), dim3(256), 0, s, view(x), x->n, x->h,
                     x->w, static_cast<uint16_t*>(y->data) + y->offset, y->stride);
  return hipGetLastError();
}

hipError_t nn_avgpool2_bwd(const gs_act* dy, const gs_act* add, gs_act* dx, int accumulate,
                           hipStream_t s) {
  const int64_t total = (int64_t)dx->n * dx->h * dx->w * (dy->c / 8);
  hipLaunchKernelGGL(avgpool2_bwd_kernel, dim3(blocks(total)), dim3(256), 0, s, view(dy), dx->n,
                     dx->h, dx->w, static_cast<uint16_t*>(dx->data), dx->stride, dx->offset,
                     accumulate, add ? static_cast<const uint16_t*>(add->data) : nullptr,
                     add ? add->stride : 0, add ? add->offset : 0);
  return hipGetLastError();
}

hipError_t nn_upsample2(const gs_act* x, gs_act* y, hipStream_t s) {
  const int64_t total = (int64_t)y->n * y->h * y->w * (x->c / 8);
  hipLaunchKernelGGL(upsample2_kernel, dim3(blocks(total)), dim3(256), 0, s, view(x), y->n, y->h,
                     y->w, static_cast<uint16_t*>(y->data), y->stride, y->offset);
  return hipGetLastError();
}

hipError_t nn_upsample2_bwd(const gs_act* dy, gs_act* dx, hipStream_t s) {
  const int64_t total = (int64_t)dx->n * dx->h * dx->w * (dy->c / 8);
  hipLaunchKernelGGL(upsample2_bwd_kernel, dim3(blocks(total)), dim3(256), 0, s, view(dy), dy->n,
                     dy->h, dy->w, static_cast<uint16_t*>(dx->data) + dx->offset, dx->stride);
  return hipGetLastError();
}

hipError_t nn_rgb_to_nhwc(const float* rgb, gs_act* x, hipStream_t s) {
  const int64_t npix = (int64_t)x->n * x->h * x->w;
  hipLaunchKernelGGL(rgb_to_nhwc_kernel, dim3(blocks(npix)), dim3(256), 0, s, rgb, x->n, x->h,
                     x->w, static_cast<uint16_t*>(x->data), x->stride);
  return hipGetLastError();
}

hipError_t nn_f32_to_bf16(const float* src, void* dst, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(f32_to_bf16_kernel, dim3(blocks(n)), dim3(256), 0, s, src,
                     static_cast<uint16_t*>(dst), n);
  return hipGetLastError();
}

hipError_t nn_head(const gs_act* f, const float* w, const float* b, float* out, hipStream_t s) {
  const int64_t npix = (int64_t)f->n * f->h * f->w;
  if (f->c % 8 == 0 && f->stride % 8 == 0 && f->offset % 8 == 0)
    hipLaunchKernelGGL(head_fwd8_kernel, dim3(blocks(npix)), dim3(256), 0, s, view(f), f->n, f->h,
                       f->w, w, b, out);
  else
    hipLaunchKernelGGL(head_fwd_kernel, dim3(blocks(npix)), dim3(256), 0, s, view(f), f->n, f->h,
                       f->w, w, b, out);
  return hipGetLastError();
}

hipError_t nn_head_bwd(const gs_act* f, const float* w, const float* dout, gs_act* df, float* dw,
                       float* db, hipStream_t s) {
  const int64_t npix = (int64_t)f->n * f->h * f->w;
  if (f->c > 32 * kHeadMaxSlots) return hipErrorInvalidValue;
  if (f->c % 8 == 0 && f->c <= 8 * kHead8Groups && f->stride % 8 == 0 && f->offset % 8 == 0 &&
      df->stride % 8 == 0 && df->offset % 8 == 0) {
    const int per = 256 / (f->c / 8);
    const unsigned nb = (unsigned)std::min<int64_t>((npix + per - 1) / per, 2048);
    hipLaunchKernelGGL(head_bwd8_kernel, dim3(nb), dim3(256), 0, s, view(f), f->n, f->h, f->w, w,
                       dout, static_cast<uint16_t*>(df->data) + df->offset, df->stride, dw, db);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(head_bwd_kernel, dim3(std::min<unsigned>(blocks(npix), 1024u)), dim3(256), 0,
                     s, view(f), f->n, f->h,
                     f->w, w, dout, static_cast<uint16_t*>(df->data) + df->offset, df->stride, dw,
                     db);
  return hipGetLastError();
}

hipError_t nn_depth_loss(const float* pred, const float* depth, int N, int H, int W, float fx,
                         float* dpred, double* loss, int* count_ws, hipStream_t s) {
  const int64_t npix = (int64_t)N * H * W;
  hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(count_ws),
                     (int64_t)1);
  if (loss) hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(64), 0, s,
                               reinterpret_cast<uint32_t*>(loss), (int64_t)2);
  hipLaunchKernelGGL(count_valid_kernel, dim3(blocks(npix)), dim3(256), 0, s, depth, npix, count_ws);
  hipLaunchKernelGGL(depth_loss_kernel, dim3(blocks(npix)), dim3(256), 0, s, pred, depth, N, H, W,
                     fx, count_ws, dpred, loss);
  return hipGetLastError();
}

}  // namespace gsmi
