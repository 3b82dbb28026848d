// gs_bp_labels: loopy min-sum belief propagation over the photometric cost
// volume (Sec. III-A2; Felzenszwalb and Huttenlocher's formulation) on the
// 4-connected grid with the truncated linear smoothness min(lam |l - l'|, trunc).
//
// A pixel's 64 labels lie side by side in memory, in its data costs and in
// each message it receives.  A message is the lower envelope of the sender's
// costs under the cone lam |l - l'|: the prefix minimum of h(l) - lam l and the
// suffix minimum of h(l) + lam l, then cut at min h + trunc and shifted to a
// zero minimum.  Minima do not depend on their order, so any split of the
// labels gives the same bits.
//
// kLanes = 8 lanes share a pixel, each holding 8 consecutive labels: the scans
// run over a lane's own registers (one minimum a label, no lane exchange) and
// only the 8 partial minima cross lanes, by DPP.  One label per lane instead
// pays a 6-step DPP scan for every label, twice per message, and bound the
// iteration by the half-rate lane exchanges.  Iterations are synchronous (every message of an
// iteration from the previous iteration's), with two message buffers in turn;
// the messages before the first iteration and those from outside the grid are
// zero and are not stored.
#include "gs_internal.h"
#include "gs_nn.h"

namespace gsmi {

namespace {

constexpr int kL = 64;           // labels = hypotheses
constexpr int kLanes = 8;        // lanes per pixel
constexpr int kOwn = kL / kLanes;   // consecutive labels per lane
constexpr int kBpPixels = 256 / kLanes;   // pixels per workgroup
constexpr int kTileW = 8, kTileH = 4;     // pixels of a two-iteration tile
constexpr int kTilePixels = kTileW * kTileH;
static_assert(2 * (kTileW + kTileH) <= kTilePixels, "one edge pixel per group of lanes");

// x of another lane of the same 8-lane group by DPP
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// the same, +inf (the identity of min) where the row has no such lane
template <int CTRL>
__device__ __forceinline__ float dpp_or_inf(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(INFINITY), __float_as_int(x), CTRL,
                                                    0xf, 0xf, false));
}

// Minimum over the group's 8 lanes, in every lane.
__device__ __forceinline__ float group_min(float x) {
  x = fminf(x, dpp<0xb1>(x));    // quad_perm [1,0,3,2]
  x = fminf(x, dpp<0x4e>(x));    // quad_perm [2,3,0,1]
  return fminf(x, dpp<0x141>(x));   // row_half_mirror: lane 7 - i of the group
}

// Minimum over the group's lanes before (after) this one, +inf in the first
// (last): Hillis-Steele by row shifts, cut at the group's edge (a row holds two).
__device__ __forceinline__ float before_min(float x, int g) {
  float y = dpp_or_inf<0x111>(x);          // row_shr:1
  y = g >= 1 ? y : INFINITY;
  float z = dpp_or_inf<0x111>(y);
  y = fminf(y, g >= 2 ? z : INFINITY);     // lanes g - 1, g - 2
  z = dpp_or_inf<0x112>(y);                // row_shr:2
  y = fminf(y, g >= 3 ? z : INFINITY);     // .. g - 4
  z = dpp_or_inf<0x114>(y);                // row_shr:4
  return fminf(y, g >= 5 ? z : INFINITY);
}
__device__ __forceinline__ float after_min(float x, int g) {
  float y = dpp_or_inf<0x101>(x);          // row_shl:1
  y = g <= 6 ? y : INFINITY;
  float z = dpp_or_inf<0x101>(y);
  y = fminf(y, g <= 5 ? z : INFINITY);
  z = dpp_or_inf<0x102>(y);                // row_shl:2
  y = fminf(y, g <= 4 ? z : INFINITY);
  z = dpp_or_inf<0x104>(y);                // row_shl:4
  return fminf(y, g <= 2 ? z : INFINITY);
}

struct Labels {
  float v[kOwn];
};

// 16 bytes that need only a float's alignment (the workspace is the caller's)
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ Labels load_labels(const float* __restrict__ p) {
  Labels r;
#pragma unroll
  for (int k = 0; k < kOwn; k += 4) {
    const float4u x = *reinterpret_cast<const float4u*>(p + k);
    r.v[k] = x.x;
    r.v[k + 1] = x.y;
    r.v[k + 2] = x.z;
    r.v[k + 3] = x.w;
  }
  return r;
}

__device__ __forceinline__ Labels zero_labels() {
  Labels r;
#pragma unroll
  for (int k = 0; k < kOwn; ++k) r.v[k] = 0.0f;
  return r;
}

__device__ __forceinline__ void store_labels(float* __restrict__ p, const Labels& x) {
#pragma unroll
  for (int k = 0; k < kOwn; k += 4)
    *reinterpret_cast<float4u*>(p + k) = float4u{x.v[k], x.v[k + 1], x.v[k + 2], x.v[k + 3]};
}

__device__ __forceinline__ float own_min(const Labels& x) {
  float m = fminf(fminf(x.v[0], x.v[1]), x.v[2]);
#pragma unroll
  for (int k = 3; k + 1 < kOwn; k += 2) m = fminf(fminf(m, x.v[k]), x.v[k + 1]);
  return fminf(m, x.v[kOwn - 1]);
}

// A pixel's message to one neighbour, this lane's labels: min over l of
// h(l) + min(lam |l - l'|, trunc), h = tot - in (in: what that neighbour sent),
// shifted so that its minimum over l' is 0.
__device__ __forceinline__ Labels message(const Labels& tot, const Labels& in, int g, float lam,
                                          float trunc) {
  const float l0 = (float)(g * kOwn);
  Labels h, a, b;
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {
    h.v[k] = tot.v[k] - in.v[k];
    a.v[k] = __builtin_fmaf(-lam, l0 + (float)k, h.v[k]);
    b.v[k] = __builtin_fmaf(lam, l0 + (float)k, h.v[k]);
  }
  const float cut = group_min(own_min(h)) + trunc;
  a.v[0] = fminf(a.v[0], before_min(own_min(a), g));
  b.v[kOwn - 1] = fminf(b.v[kOwn - 1], after_min(own_min(b), g));
#pragma unroll
  for (int k = 1; k < kOwn; ++k) {
    a.v[k] = fminf(a.v[k], a.v[k - 1]);
    b.v[kOwn - 1 - k] = fminf(b.v[kOwn - 1 - k], b.v[kOwn - k]);
  }
#pragma unroll
  for (int k = 0; k < kOwn; ++k)
    a.v[k] = fminf(fminf(__builtin_fmaf(lam, l0 + (float)k, a.v[k]),
                         __builtin_fmaf(-lam, l0 + (float)k, b.v[k])), cut);
  const float r = group_min(own_min(a));
#pragma unroll
  for (int k = 0; k < kOwn; ++k) a.v[k] -= r;
  return a;
}

// What a pixel knows: its data costs, the messages received from its left (0),
// right (1), upper (2) and lower (3) neighbour (zero from outside the grid)
// and their sum.
struct Pixel {
  Labels tot, in[4];
};

template <typename Load>
__device__ __forceinline__ void receive(Pixel& P, const Labels& data, int x, int y, int H, int W,
                                        Load load) {
  P.in[0] = x > 0 ? load(0) : zero_labels();
  P.in[1] = x + 1 < W ? load(1) : zero_labels();
  P.in[2] = y > 0 ? load(2) : zero_labels();
  P.in[3] = y + 1 < H ? load(3) : zero_labels();
#pragma unroll
  for (int k = 0; k < kOwn; ++k)
    P.tot.v[k] = data.v[k] + P.in[0].v[k] + P.in[1].v[k] + P.in[2].v[k] + P.in[3].v[k];
}

__device__ __forceinline__ void receive_none(Pixel& P, const Labels& data) {
  P.tot = data;
#pragma unroll
  for (int k = 0; k < 4; ++k) P.in[k] = zero_labels();
}

// The four messages of pixel (x, y) to global memory: message k of a pixel
// lies at plane k.
__device__ __forceinline__ void send_all(const Pixel& P, int x, int y, int H, int W, int g,
                                         float lam, float trunc, float* __restrict__ mout) {
  const int64_t plane = (int64_t)H * W * kL;
  float* o = mout + ((int64_t)y * W + x) * kL + g * kOwn;
  const Labels r = message(P.tot, P.in[1], g, lam, trunc);
  if (x + 1 < W) store_labels(o + kL, r);
  const Labels l = message(P.tot, P.in[0], g, lam, trunc);
  if (x > 0) store_labels(o + plane - kL, l);
  const Labels d = message(P.tot, P.in[3], g, lam, trunc);
  if (y + 1 < H) store_labels(o + 2 * plane + (int64_t)W * kL, d);
  const Labels u = message(P.tot, P.in[2], g, lam, trunc);
  if (y > 0) store_labels(o + 3 * plane - (int64_t)W * kL, u);
}

// D[p][l] from cost[l][p], 64 pixels per workgroup through LDS (a pitch of 65
// words: reading a column touches every bank once); +inf (no valid view)
// becomes `invalid`.
__global__ __launch_bounds__(256) void bp_init_kernel(const float* __restrict__ cost, int64_t np,
                                                      float invalid, float* __restrict__ D) {
  __shared__ float s_c[kL][65];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t p0 = (int64_t)blockIdx.x * 64;
#pragma unroll 4
  for (int l = w; l < kL; l += 4)
    if (p0 + lane < np) s_c[l][lane] = cost[(int64_t)l * np + p0 + lane];
  __syncthreads();
#pragma unroll 4
  for (int q = w; q < 64; q += 4) {
    if (p0 + q >= np) break;
    const float c = s_c[lane][q];
    D[(p0 + q) * kL + lane] = isfinite(c) ? c : invalid;
  }
}

// The first of an odd number of iterations: no message has been sent yet.
__global__ __launch_bounds__(256) void bp_first_kernel(const float* __restrict__ D,
                                                       float* __restrict__ mout, int H, int W,
                                                       float lam, float trunc) {
  const int p = (int)blockIdx.x * kBpPixels + (int)(threadIdx.x / kLanes);
  const int g = threadIdx.x % kLanes;
  if (p >= H * W) return;   // whole 8-lane groups leave together
  Pixel P;
  receive_none(P, load_labels(D + (int64_t)p * kL + g * kOwn));
  send_all(P, p % W, p / W, H, W, g, lam, trunc, mout);
}

// Two synchronous iterations on tiles of kTileW x kTileH pixels.  The first one's messages
// into the tile stay in LDS: those its own pixels send each other and those
// the pixels along its edge send in (computed from the same inputs by the
// edge pixel's own workgroup as well, to the same bits); the second one's go to
// mout.  FIRST: no message has been sent yet.
// All of a launch's wavefronts run at once, so loading, computing and storing
// follow one another instead of overlapping: one iteration per launch took
// 10.8 us at 160x120 (44 MB), two take 14.6 us together (the loads of the
// second and the stores of the first stay on the chip; 15.5 us on 8x8 tiles,
// 300 workgroups that leave two on some CUs and one on others, 14.6 on 4x4).
// One label per lane had taken 17 us an iteration.
template <bool FIRST>
__global__ __launch_bounds__(kTilePixels * kLanes) void bp_pair_kernel(const float* __restrict__ D,
                                                      const float* __restrict__ min_,
                                                      float* __restrict__ mout, int H, int W,
                                                      float lam, float trunc) {
  __shared__ __align__(16) float s_m[4][kTilePixels][kL];   // messages into the tile's pixels
  const int g = threadIdx.x % kLanes, q = threadIdx.x / kLanes;
  const int x0 = blockIdx.x * kTileW, y0 = blockIdx.y * kTileH;
  const int64_t plane = (int64_t)H * W * kL;
  auto at = [&](int x, int y) { return ((int64_t)y * W + x) * kL + g * kOwn; };
  auto into = [&](int k, int lx, int ly) { return &s_m[k][ly * kTileW + lx][g * kOwn]; };
  auto from_memory = [&](Pixel& P, int x, int y) {
    const Labels data = load_labels(D + at(x, y));
    if constexpr (FIRST)
      receive_none(P, data);
    else
      receive(P, data, x, y, H, W,
              [&](int k) { return load_labels(min_ + k * plane + at(x, y)); });
  };
  const int lx = q % kTileW, ly = q / kTileW, x = x0 + lx, y = y0 + ly;
  const bool in_grid = x < W && y < H;
  Pixel P;
  if (in_grid) {
    from_memory(P, x, y);
    const Labels r = message(P.tot, P.in[1], g, lam, trunc);
    if (lx < kTileW - 1) store_labels(into(0, lx + 1, ly), r);
    const Labels l = message(P.tot, P.in[0], g, lam, trunc);
    if (lx > 0) store_labels(into(1, lx - 1, ly), l);
    const Labels d = message(P.tot, P.in[3], g, lam, trunc);
    if (ly < kTileH - 1) store_labels(into(2, lx, ly + 1), d);
    const Labels u = message(P.tot, P.in[2], g, lam, trunc);
    if (ly > 0) store_labels(into(3, lx, ly - 1), u);
  }
  // edge pixel i of side k sends into the tile: k = 0 from the left, 1 from the
  // right, 2 from above, 3 from below
  if (q < 2 * (kTileW + kTileH)) {
    const int side = q < kTileH ? 0 : q < 2 * kTileH ? 1 : q < 2 * kTileH + kTileW ? 2 : 3;
    const int i = q - (side == 0 ? 0 : side == 1 ? kTileH : side == 2 ? 2 * kTileH : 2 * kTileH + kTileW);
    const int ex = side == 0 ? x0 - 1 : side == 1 ? x0 + kTileW : x0 + i;
    const int ey = side == 2 ? y0 - 1 : side == 3 ? y0 + kTileH : y0 + i;
    if (ex >= 0 && ey >= 0 && ex < W && ey < H) {
      Pixel E;
      from_memory(E, ex, ey);
      // what the tile's pixel sent to the edge pixel
      Labels back;
#pragma unroll
      for (int k = 0; k < kOwn; ++k)
        back.v[k] = side == 0   ? E.in[1].v[k]
                    : side == 1 ? E.in[0].v[k]
                    : side == 2 ? E.in[3].v[k]
                                : E.in[2].v[k];
      store_labels(into(side, side == 0 ? 0 : side == 1 ? kTileW - 1 : i,
                        side == 2 ? 0 : side == 3 ? kTileH - 1 : i),
                   message(E.tot, back, g, lam, trunc));
    }
  }
  Labels data = zero_labels();
  if (in_grid) data = load_labels(D + at(x, y));   // again, rather than held in registers
  __syncthreads();
  if (!in_grid) return;
  receive(P, data, x, y, H, W, [&](int k) { return load_labels(into(k, lx, ly)); });
  send_all(P, x, y, H, W, g, lam, trunc, mout);
}

// Belief = data + the four incoming messages (m == NULL: none were sent);
// label = its first minimum.
__global__ __launch_bounds__(256) void bp_label_kernel(const float* __restrict__ D,
                                                       const float* __restrict__ m, int H, int W,
                                                       int32_t* __restrict__ labels,
                                                       float* __restrict__ depth) {
  const int np = H * W;
  const int p = (int)blockIdx.x * kBpPixels + (int)(threadIdx.x / kLanes);
  const int g = threadIdx.x % kLanes;
  if (p >= np) return;
  const int y = p / W, x = p - y * W;
  const int64_t o = (int64_t)p * kL + g * kOwn;
  Pixel P;
  const Labels data = load_labels(D + o);
  if (m)
    receive(P, data, x, y, H, W,
            [&](int k) { return load_labels(m + (int64_t)k * np * kL + o); });
  else
    receive_none(P, data);
  const float mn = group_min(own_min(P.tot));
  int own = kL;   // this lane's first label at the minimum
#pragma unroll
  for (int k = kOwn - 1; k >= 0; --k) own = P.tot.v[k] == mn ? g * kOwn + k : own;
#pragma unroll
  for (int d = 1; d < kLanes; d <<= 1) own = min(own, __shfl_xor(own, d, kLanes));
  if (g == 0) {
    if (labels) labels[p] = own;
    // the hypothesis depth exactly as the cost volume evaluates it
    if (depth) depth[p] = 0.25f + (25.0f - 0.25f) * (float)own / (float)(kL - 1);
  }
}

}  // namespace

size_t bp_ws_bytes(int h, int w) {
  const size_t np = (size_t)h * w;
  return (np * kL + 2 * 4 * np * kL) * sizeof(float);   // data costs + two message sets
}

hipError_t launch_bp(const float* cost, int h, int w, float lam, float trunc, int iters,
                     float invalid, int32_t* labels, float* depth, void* ws, hipStream_t s) {
  const int64_t np = (int64_t)h * w;
  float* D = static_cast<float*>(ws);
  float* mA = D + np * kL;
  float* mB = mA + 4 * np * kL;
  hipLaunchKernelGGL(bp_init_kernel, dim3((unsigned)((np + 63) / 64)), dim3(256), 0, s, cost, np,
                     invalid, D);
  const dim3 grid((unsigned)((np + kBpPixels - 1) / kBpPixels));
  const dim3 tiles((unsigned)((w + kTileW - 1) / kTileW), (unsigned)((h + kTileH - 1) / kTileH));
  int done = 0;
  if (iters & 1) {
    hipLaunchKernelGGL(bp_first_kernel, grid, dim3(256), 0, s, D, mB, h, w, lam, trunc);
    std::swap(mA, mB);
    done = 1;
  }
  for (; done < iters; done += 2) {
    if (done == 0)
      hipLaunchKernelGGL(bp_pair_kernel<true>, tiles, dim3(kTilePixels * kLanes), 0, s, D, mA, mB, h, w, lam, trunc);
    else
      hipLaunchKernelGGL(bp_pair_kernel<false>, tiles, dim3(kTilePixels * kLanes), 0, s, D, mA, mB, h, w, lam, trunc);
    std::swap(mA, mB);
  }
  hipLaunchKernelGGL(bp_label_kernel, grid, dim3(256), 0, s, D, iters > 0 ? mA : nullptr, h, w,
                     labels, depth);
  return hipGetLastError();
}

}  // namespace gsmi
