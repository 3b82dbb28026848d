// gs_bin_sort: tile binning and (tile, depth) ordering of the splats.
//
// The order wanted is, per global tile, the splats whose rectangles cover it
// by ascending (float32 depth bits, entry).  It is built as a counting sort
// on the tile (the tiles are few: 38,400 for 32 views at 640x480) followed by
// a sort of each tile's own short list.  No step uses global atomics on the
// tile counters, which contend badly on tiles many splats cover:
//
//   compact   the splats of each view that touch a tile are appended to a
//             per-view list as {u, v, radius, depth} records (one global
//             atomic per workgroup of 1,024 entries); the walks below read
//             only these (a tenth of the entries in a mapping batch)
//   hist      each workgroup of 512 threads takes chunks of 512 listed
//             splats of one view and counts, in an LDS histogram over that
//             view's tiles, the keys they emit (each splat's tile rectangle
//             in float64 from its float32 centre), then stores the whole
//             histogram as row `chunk` of a dense chunk x tile matrix.
//             Splats with large rectangles do not serialise one lane: a
//             wavefront walks its 64 splats' keys 64 at a time, each lane
//             finding its splat by a prefix maximum over start marks.
//   column    per tile, an exclusive scan down its matrix column (each
//             chunk's first slot within the tile's segment) and the total
//   scan      exclusive scan of the per-tile totals: every tile's [start,
//             end) in the sorted keys, and the key count (in 64 bits)
//   emit      the same walk per chunk places each key's (depth bits,
//             entry) pair in its tile's segment, at the chunk's slots
//             (LDS atomics hand out the slots within a chunk)
//   segment   one wavefront per tile sorts its segment by (depth bits,
//             entry) with a bitonic network in registers (lists of up to
//             kSegShort pairs) and writes the entries (and keys); in the
//             same launch, the first workgroups sort the longer lists with
//             all their wavefronts (registers and LDS), or, beyond kSegLong
//             pairs, by a stable LSD radix sort over the 64-bit pair
//   order     optional: the tiles stably sorted by list length group,
//             longest first (the launch order of the compositing grids)
//
// Small batches take a short path of five launches with the same results (see
// run_bin_sort).  Views with more tiles than the LDS histogram holds are processed in tile
// windows (one walk per window).  Nothing here needs a host synchronisation
// unless the caller asks for the key count.
#include <immintrin.h>

#include <atomic>
#include <type_traits>

#include "gs_internal.h"

namespace gsmi {

namespace {

// Words of pinned host memory that the scan kernel writes key counts to, for the calls
// that return them: one block for the process, of which a call holds a word from its
// launches until the count is there.  (A word per thread had to be given back when the
// thread ended, and freeing pinned memory invalidates a graph that another thread
// records.)  A call that finds none free copies its count instead.
constexpr uint64_t kNoCount = ~0ull;
constexpr int kCountWords = 64;
constexpr int kCountStride = 8;   // in words: a cache line each

// While it lives, this thread's calls may do what another thread's recording of a graph
// forbids in the default mode; they leave that recording alone.
class RelaxedCapture {
 public:
  RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  RelaxedCapture(const RelaxedCapture&) = delete;
  RelaxedCapture& operator=(const RelaxedCapture&) = delete;

 private:
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

struct CountBlock {
  uint64_t *host = nullptr, *dev = nullptr;   // dev NULL: no pinned memory to be had
  std::atomic<uint64_t> free{~0ull};          // bit per word
  CountBlock() {
    RelaxedCapture relaxed;
    void *h = nullptr, *d = nullptr;
    if (hipHostMalloc(&h, sizeof(uint64_t) * kCountWords * kCountStride,
                      hipHostMallocMapped | hipHostMallocPortable) == hipSuccess) {
      host = static_cast<uint64_t*>(h);
      if (hipHostGetDevicePointer(&d, h, 0) == hipSuccess) dev = static_cast<uint64_t*>(d);
    }
    if (!dev) (void)hipGetLastError();
  }
};

static_assert(std::is_trivially_destructible_v<CountBlock>);

// The process's block, allocated by the first call that wants a word and kept to its end.
CountBlock& count_block() {
  static CountBlock block;   // trivially destroyed: no call of the runtime at exit
  return block;
}

// A call's word of the block.
class CountWord {
 public:
  explicit CountWord(hipStream_t s) : s_(s) {}
  CountWord(const CountWord&) = delete;
  CountWord& operator=(const CountWord&) = delete;
  // The device's address of a free word, NULL if there is none.
  uint64_t* take() {
    CountBlock& block = count_block();
    if (!block.dev) return nullptr;
    uint64_t bits = block.free.load(std::memory_order_relaxed);
    do {
      if (!bits) return nullptr;
    } while (!block.free.compare_exchange_weak(bits, bits & (bits - 1), std::memory_order_acquire,
                                               std::memory_order_relaxed));
    word_ = __builtin_ctzll(bits);
    __atomic_store_n(block.host + word_ * kCountStride, kNoCount, __ATOMIC_RELEASE);
    return block.dev + word_ * kCountStride;
  }
  // The count once the kernel on the stream has written it; an error of the stream, or
  // its end, ends the wait.
  hipError_t wait(uint64_t& count) {
    const uint64_t* host = count_block().host + word_ * kCountStride;
    for (unsigned spin = 1;; ++spin) {
      count = __atomic_load_n(host, __ATOMIC_ACQUIRE);
      if (count != kNoCount) break;
      _mm_pause();
      if (spin % 256) continue;
      const hipError_t e = hipStreamQuery(s_);
      if (e == hipErrorNotReady) {
        (void)hipGetLastError();
        continue;
      }
      if (e != hipSuccess) return e;
      count = __atomic_load_n(host, __ATOMIC_ACQUIRE);   // all of the stream is done
      if (count != kNoCount) break;
      return hipErrorUnknown;
    }
    written_ = true;
    return hipSuccess;
  }
  // A call that returns without its count waits for its stream first: the kernel may
  // still write the word, and another call would take that count for its own.
  ~CountWord() {
    if (word_ < 0) return;
    if (!written_) {
      RelaxedCapture relaxed;
      if (hipStreamSynchronize(s_) != hipSuccess) return;   // then it is not given back
    }
    count_block().free.fetch_or(uint64_t(1) << word_, std::memory_order_release);
  }

 private:
  hipStream_t s_;
  int word_ = -1;
  bool written_ = false;
};

// The key count in 64 bits, its 32-bit clamp and, unless NULL, the host's copy.
__device__ __forceinline__ void write_count(uint64_t count, uint64_t* total, uint32_t* n_keys,
                                            uint64_t* host) {
  *total = count;
  *n_keys = count > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)count;
  if (host) __hip_atomic_store(host, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

constexpr int kBinThreads = 512;                         // threads of a binning workgroup
constexpr int kBinWaves = kBinThreads / 64;
constexpr int kBinChunk = kBinThreads;                  // splats per binning chunk
constexpr int kBinGrid = 64;                             // binning workgroups per view
constexpr int kLdsTiles = 8192;                          // largest LDS histogram (tiles)
constexpr int kSegShort = 1024;                          // longest list of the wavefront sort
constexpr int kSegFew = 256, kSegFewTiles = 1536;         // the same up to so many tiles
constexpr int kSegLong = 4096;                           // longest list of the workgroup sort
constexpr int kSortThreads = 512;                        // threads of a sort workgroup
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kLongSlots = 512;                          // most sort workgroups that take the long lists

// The short path (see run_bin_sort): at most kFewGaussians Gaussians,
// kFewEntries (view, Gaussian) entries and kFewTiles tiles.
constexpr int kFewThreads = 256;                         // threads of its binning workgroups
constexpr int64_t kFewEntries = 1 << 20;
constexpr int64_t kFewGaussians = 1 << 18;
constexpr int kFewTiles = 16384;
constexpr int kFewRows = 256;                            // most chunks of a view
constexpr int kFewColWaves = 16;                         // wavefronts that share a column's rows

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63; }

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
  const uint32_t lane = lane_id();
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const T y = __shfl_up(x, d, 64);
    if (lane >= (uint32_t)d) x += y;
  }
  return x;
}

// ---------------------------------------------------------------------------
// the key walk
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t* __restrict__ p, uint32_t value,
                                                       int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

// Inclusive prefix maximum over the 64 lanes of a wavefront (DPP row shifts,
// then the row broadcasts; lanes without a source see 0, the identity here).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, 0xf, true);
}

__device__ __forceinline__ uint32_t wave_prefix_max(uint32_t x) {
  x = max(x, dpp_u32<0x111, 0xf>(x));   // row_shr:1
  x = max(x, dpp_u32<0x112, 0xf>(x));   // row_shr:2
  x = max(x, dpp_u32<0x114, 0xf>(x));   // row_shr:4
  x = max(x, dpp_u32<0x118, 0xf>(x));   // row_shr:8
  x = max(x, dpp_u32<0x142, 0xa>(x));   // row_bcast:15 into rows 1 and 3
  x = max(x, dpp_u32<0x143, 0xc>(x));   // row_bcast:31 into rows 2 and 3
  return x;
}

// Inclusive prefix sum over the 64 lanes (the same DPP pattern).
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t x) {
  x += dpp_u32<0x111, 0xf>(x);
  x += dpp_u32<0x112, 0xf>(x);
  x += dpp_u32<0x114, 0xf>(x);
  x += dpp_u32<0x118, 0xf>(x);
  x += dpp_u32<0x142, 0xa>(x);
  x += dpp_u32<0x143, 0xc>(x);
  return x;
}

// Per wavefront: its 64 entries' key ranges and rectangles while it walks them.
struct WalkLds {
  uint4 rect[64];      // first key in the wave's run, first tile (view-local), width, tiles per row
  uint32_t ent[64];
  uint32_t dep[64];    // float32 depth bits (emission only)
  uint32_t mark[64];
};

// q = jj / w for jj < 2^20 and 1 <= w < 2^11: a float reciprocal estimate
// corrected by one step either way (exact: the estimate is within one).
__device__ __forceinline__ uint32_t div_small(uint32_t jj, uint32_t w) {
  uint32_t q = (uint32_t)((float)jj * __builtin_amdgcn_rcpf((float)w));
  if (q * w > jj) --q;
  else if ((q + 1) * w <= jj) ++q;
  return q;
}

// A splat's keys: their number, and its first tile | rectangle width << 21 (a
// view has at most 2^20 tiles, a rectangle at most 1,024 columns).
struct SplatKeys {
  uint32_t cnt, rect;
};

__device__ __forceinline__ SplatKeys splat_keys(const uint4& c, const ViewInfo& vi) {
  SplatKeys k{0u, 1u << 21};
  Rect rc;
  if (tile_rect(__uint_as_float(c.x), __uint_as_float(c.y), (int32_t)c.z, vi.width, vi.height, rc)) {
    k.cnt = (uint32_t)((rc.x1 - rc.x0) * (rc.y1 - rc.y0));
    k.rect = (uint32_t)(rc.y0 * vi.tiles_x + rc.x0) | ((uint32_t)(rc.x1 - rc.x0) << 21);
  }
  return k;
}

// Calls op(view-local tile, entry, depth bits) once for every key of a
// wavefront's 64 splats (one per lane; cnt 0: none): the wavefront walks the
// keys 64 at a time, every lane taking the key at its position and finding the
// splat that owns it as the last splat whose first key is at or before it (a
// prefix maximum over start marks), so large rectangles spread over the lanes.
template <bool kDepth, typename Op>
__device__ __forceinline__ void walk_wave(const SplatKeys& k, uint32_t id, uint32_t dep,
                                          const ViewInfo& vi, WalkLds& L, Op op) {
  const uint32_t lane = lane_id();
  const uint32_t inc = wave_prefix_sum(k.cnt);
  const uint32_t start = inc - k.cnt;
  const uint32_t wend = __builtin_amdgcn_readlane(inc, 63);
  if (wend == 0) return;   // uniform within the wavefront
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  L.rect[lane] = make_uint4(start, k.rect & 0x1FFFFFu, k.rect >> 21, (uint32_t)vi.tiles_x);
  if constexpr (kDepth) {
    L.ent[lane] = id;
    L.dep[lane] = dep;
  }
  uint32_t carry = 0;   // 1 + lane of the entry owning the position before the window
  for (uint32_t w0 = 0; w0 < wend; w0 += 64) {
    L.mark[lane] = 0;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    if (k.cnt > 0 && start >= w0 && start - w0 < 64) L.mark[start - w0] = lane + 1;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    const uint32_t m = wave_prefix_max(max(L.mark[lane], carry));
    carry = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
    const uint32_t pos = w0 + lane;
    if (pos < wend) {   // then m >= 1: the owner's first key is at or before pos
      const uint4 rc = L.rect[m - 1];
      const uint32_t jj = pos - rc.x;
      const uint32_t row = div_small(jj, rc.z);
      if constexpr (kDepth)
        op(rc.y + row * rc.w + (jj - row * rc.z), L.ent[m - 1], L.dep[m - 1]);
      else
        op(rc.y + row * rc.w + (jj - row * rc.z), 0u, 0u);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  }
}

// walk_wave over splats j0 .. j0 + kBinChunk of a view's compacted list (count
// splats in all), one per thread.  (Two per thread, 1,024 to a chunk, left the
// chip short of wavefronts: the whole binning took 124 us instead of 109 for 32
// views of 640x480 over 200,000 Gaussians, 81 instead of 73 for 12.)
template <bool kDepth, typename Op>
__device__ __forceinline__ void walk_keys(const uint4* __restrict__ rec,
                                          const uint32_t* __restrict__ ids, uint32_t count,
                                          uint32_t j0, const ViewInfo& vi, WalkLds* L, Op op) {
  const uint32_t j = j0 + threadIdx.x;
  const uint32_t jc = j < count ? j : count - 1;
  uint4 c = rec[jc];
  uint32_t id = 0;
  if constexpr (kDepth) id = ids[jc];
  if (j >= count) c.z = 0u;   // past the list: radius 0, no keys
  walk_wave<kDepth>(splat_keys(c, vi), id, c.w, vi, L[threadIdx.x >> 6], op);
}

// ---------------------------------------------------------------------------
// compaction, counts: chunk x tile matrix, column scan
// ---------------------------------------------------------------------------

constexpr int kCompactItems = 4;                 // entries per thread (256 threads)
constexpr int kCompactChunk = 256 * kCompactItems;

// Grid (entries / kCompactChunk, views): the splats of view v that touch a
// tile (stored count > 0, or radius > 0 when counts are not stored) are
// appended to the view's list, [v n, v n + list_count[v]), as {u, v, radius,
// depth bits} records with their entries (v n + i) beside them.  One global
// atomic per workgroup reserves its run; the list order is the order of the
// reservations, which the per-tile sort makes irrelevant.
__global__ __launch_bounds__(256) void bin_compact_kernel(const float2* __restrict__ xy,
                                                          const int32_t* __restrict__ radius,
                                                          const float4* __restrict__ rd,
                                                          const uint32_t* __restrict__ stored,
                                                          int64_t n,
                                                          uint32_t* __restrict__ list_count,
                                                          uint4* __restrict__ rec,
                                                          uint32_t* __restrict__ ids) {
  __shared__ uint32_t s_wave[4];
  __shared__ uint32_t s_base;
  const int v = blockIdx.y;
  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * kCompactChunk;
  bool keep[kCompactItems];
  uint32_t mine = 0;
#pragma unroll
  for (int q = 0; q < kCompactItems; ++q) {
    const int64_t i = i0 + q * 256 + threadIdx.x;
    const int64_t e = (int64_t)v * n + (i < n ? i : n - 1);
    const uint32_t x = stored ? stored[e] : (uint32_t)max(radius[e], 0);
    keep[q] = i < n && x > 0u;
    mine += keep[q] ? 1u : 0u;
  }
  // the kept splats' data, loaded while the run is reserved (entries not
  // kept read the view's first entry instead, one cached line)
  float2 c[kCompactItems];
  int32_t r[kCompactItems];
  float z[kCompactItems];
#pragma unroll
  for (int q = 0; q < kCompactItems; ++q) {
    const int64_t e = (int64_t)v * n + (keep[q] ? i0 + q * 256 + threadIdx.x : 0);
    c[q] = xy[e];
    r[q] = radius[e];
    z[q] = rd[e].w;
  }
  const uint32_t inc = wave_prefix_sum(mine);
  if (lane == 63) s_wave[w] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t tot = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    s_base = tot ? atomicAdd(&list_count[v], tot) : 0u;
  }
  __syncthreads();
  uint32_t pos = s_base + inc - mine;
  for (uint32_t k = 0; k < w; ++k) pos += s_wave[k];
  uint4* vrec = rec + (int64_t)v * n;
  uint32_t* vids = ids + (int64_t)v * n;
#pragma unroll
  for (int q = 0; q < kCompactItems; ++q) {
    if (keep[q]) {
      vrec[pos] = make_uint4(__float_as_uint(c[q].x), __float_as_uint(c[q].y), (uint32_t)r[q],
                             __float_as_uint(z[q]));
      vids[pos] = (uint32_t)((int64_t)v * n + i0 + q * 256 + threadIdx.x);
      ++pos;
    }
  }
}

__device__ __forceinline__ uint32_t list_chunks(uint32_t count) {
  return (count + kBinChunk - 1) / kBinChunk;
}

// Grid (kBinGrid, views): workgroup x takes chunks x, x + kBinGrid, ... of
// view y's list; row `chunk` of `matrix` ([chunks][n_tiles]), over the
// view's columns, receives the keys the chunk emits per tile.
__global__ __launch_bounds__(kBinThreads) void bin_hist_kernel(const uint4* __restrict__ rec,
                                                               const uint32_t* __restrict__ list_count,
                                                               int64_t n, ViewTable vt,
                                                               int lds_tiles,
                                                               uint32_t* __restrict__ matrix) {
  extern __shared__ uint32_t s_hist[];
  __shared__ WalkLds L[kBinWaves];
  const int v = blockIdx.y;
  const ViewInfo& vi = vt.v[v];
  const uint32_t count = list_count[v];
  const int vtiles = vi.tiles_x * vi.tiles_y;
  const uint4* vrec = rec + (int64_t)v * n;
  for (uint32_t ch = blockIdx.x; ch < list_chunks(count); ch += gridDim.x) {
    uint32_t* row = matrix + (int64_t)ch * vt.n_tiles + vi.tile_base;
    for (int tw = 0; tw < vtiles; tw += lds_tiles) {   // tile windows (one unless the view is huge)
      const uint32_t span = (uint32_t)min(lds_tiles, vtiles - tw);
      for (uint32_t t = threadIdx.x; t < span; t += kBinThreads) s_hist[t] = 0u;
      __syncthreads();
      walk_keys<false>(vrec, nullptr, count, ch * kBinChunk, vi, L,
                       [&](uint32_t tile, uint32_t, uint32_t) {
                         const uint32_t k = tile - (uint32_t)tw;
                         if (k < span) atomicAdd(&s_hist[k], 1u);
                       });
      __syncthreads();
      for (uint32_t t = threadIdx.x; t < span; t += kBinThreads) row[tw + t] = s_hist[t];
      __syncthreads();
    }
  }
}

// Grid (view tiles / 256, views), one thread per tile: exclusive scan down
// its column over the view's chunks (in place) and the column total.
__global__ __launch_bounds__(256) void bin_column_kernel(uint32_t* __restrict__ matrix,
                                                         const uint32_t* __restrict__ list_count,
                                                         ViewTable vt,
                                                         uint32_t* __restrict__ counts) {
  const int v = blockIdx.y;
  const ViewInfo& vi = vt.v[v];
  const int tl = blockIdx.x * 256 + threadIdx.x;
  if (tl >= vi.tiles_x * vi.tiles_y) return;
  const int64_t T = vt.n_tiles;
  const int t = vi.tile_base + tl;
  const int chunks = (int)list_chunks(list_count[v]);
  uint32_t run = 0;
  int c = 0;
  for (; c + 8 <= chunks; c += 8) {
    uint32_t x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = matrix[(int64_t)(c + q) * T + t];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      matrix[(int64_t)(c + q) * T + t] = run;
      run += x[q];
    }
  }
  for (; c < chunks; ++c) {
    const uint32_t x = matrix[(int64_t)c * T + t];
    matrix[(int64_t)c * T + t] = run;
    run += x;
  }
  counts[t] = run;
}

// ---------------------------------------------------------------------------
// exclusive scan of the per-tile counts: segments, key count
// ---------------------------------------------------------------------------

constexpr int kScanBlock = 1024;   // tiles per scan workgroup (256 threads x 4)

__global__ __launch_bounds__(256) void bin_scan_reduce_kernel(const uint32_t* __restrict__ counts,
                                                              int n_tiles,
                                                              uint64_t* __restrict__ partial,
                                                              uint32_t* __restrict__ n_long,
                                                              uint32_t* __restrict__ queue) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *n_long = 0u;   // the down-sweep queues long lists
  // the compositing calls' tile counters start from zero
  if (queue && blockIdx.x == 0)
    for (int w = threadIdx.x; w < GS_QUEUE_WORDS; w += 256) queue[w] = 0u;
  __shared__ uint64_t s_wave[4];
  const int base = blockIdx.x * kScanBlock + threadIdx.x;
  uint64_t acc = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) acc += base + q * 256 < n_tiles ? counts[base + q * 256] : 0u;
  for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
  if (lane_id() == 0) s_wave[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
}

// Each workgroup adds the totals of the blocks before it and scans its own
// 1,024 tiles (4 consecutive per thread): ranges [start, end) ([0, 0) for an
// empty tile, and for all on overflow) and every tile's first slot, and
// queues the tiles with more than kSegShort keys; block 0 also writes the
// key count in 64 bits and its 32-bit clamp.
__global__ __launch_bounds__(256) void bin_scan_down_kernel(const uint32_t* __restrict__ counts,
                                                            int n_tiles,
                                                            const uint64_t* __restrict__ partial,
                                                            int n_blocks, int64_t capacity,
                                                            uint32_t* __restrict__ ranges,
                                                            uint32_t* __restrict__ starts,
                                                            uint64_t* __restrict__ total,
                                                            uint32_t* __restrict__ n_keys,
                                                            uint64_t* __restrict__ host_count,
                                                            uint32_t* __restrict__ long_list,
                                                            uint32_t* __restrict__ n_long) {
  __shared__ uint64_t s_red[2][4];
  __shared__ uint32_t s_wave[4];
  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  uint64_t pre = 0, tot = 0;
  for (int b = threadIdx.x; b < n_blocks; b += 256) {
    const uint64_t x = partial[b];
    tot += x;
    pre += b < (int)blockIdx.x ? x : 0u;
  }
  for (int d = 32; d >= 1; d >>= 1) {
    pre += __shfl_xor(pre, d, 64);
    tot += __shfl_xor(tot, d, 64);
  }
  if (lane == 0) {
    s_red[0][w] = pre;
    s_red[1][w] = tot;
  }
  const int t0 = blockIdx.x * kScanBlock + 4 * threadIdx.x;
  uint32_t c[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) c[q] = t0 + q < n_tiles ? counts[t0 + q] : 0u;
  const uint32_t mine = c[0] + c[1] + c[2] + c[3];
  const uint32_t inc = wave_inclusive_scan(mine);
  if (lane == 63) s_wave[w] = inc;
  __syncthreads();
  pre = s_red[0][0] + s_red[0][1] + s_red[0][2] + s_red[0][3];
  tot = s_red[1][0] + s_red[1][1] + s_red[1][2] + s_red[1][3];
  const bool ok = tot <= (uint64_t)capacity;
  uint32_t st = (uint32_t)pre + inc - mine;   // exact whenever ok
  for (uint32_t k = 0; k < w; ++k) st += s_wave[k];
  if (blockIdx.x == 0 && threadIdx.x == 0) write_count(tot, total, n_keys, host_count);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int t = t0 + q;
    if (t < n_tiles) {
      const bool used = ok && c[q] > 0;
      ranges[2 * (int64_t)t] = used ? st : 0u;
      ranges[2 * (int64_t)t + 1] = used ? st + c[q] : 0u;
      starts[t] = st;
    }
    st += c[q];
  }
  // queue the long lists: one atomic per wavefront and item; lane 0's
  // reservation reaches the other lanes through LDS (every lane reads what
  // lane 0 wrote, whatever the compiler does with the lanes' control flow)
  __shared__ uint32_t s_qbase[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int t = t0 + q;
    const bool lng = ok && t < n_tiles && c[q] > (uint32_t)kSegShort;
    const uint64_t m = __ballot(lng);
    if (m) {
      if (lane == 0) s_qbase[w] = atomicAdd(n_long, (uint32_t)__popcll(m));
      const uint32_t base = s_qbase[w];
      if (lng) long_list[base + (uint32_t)__popcll(m & ((uint64_t(1) << lane) - 1))] = (uint32_t)t;
    }
  }
}

// ---------------------------------------------------------------------------
// emission
// ---------------------------------------------------------------------------

// Grid (kBinGrid, views), chunks as in the histogram: every key's (depth
// bits, entry) pair goes to its tile's segment at slot start + (the chunk's
// offset in the column) + (its rank among the chunk's keys of that tile, in
// no particular order).  Nothing on overflow.
__global__ __launch_bounds__(kBinThreads) void bin_emit_kernel(
    const uint4* __restrict__ rec, const uint32_t* __restrict__ ids,
    const uint32_t* __restrict__ list_count, int64_t n, ViewTable vt, int lds_tiles,
    const uint32_t* __restrict__ matrix, const uint32_t* __restrict__ starts,
    const uint64_t* __restrict__ total, int64_t capacity, uint64_t* __restrict__ staged) {
  extern __shared__ uint32_t s_slot[];
  __shared__ WalkLds L[kBinWaves];
  if (*total > (uint64_t)capacity) return;
  const int v = blockIdx.y;
  const ViewInfo& vi = vt.v[v];
  const uint32_t count = list_count[v];
  const int vtiles = vi.tiles_x * vi.tiles_y;
  const uint4* vrec = rec + (int64_t)v * n;
  const uint32_t* vids = ids + (int64_t)v * n;
  const uint32_t* st = starts + vi.tile_base;
  for (uint32_t ch = blockIdx.x; ch < list_chunks(count); ch += gridDim.x) {
    const uint32_t* row = matrix + (int64_t)ch * vt.n_tiles + vi.tile_base;
    for (int tw = 0; tw < vtiles; tw += lds_tiles) {
      const uint32_t span = (uint32_t)min(lds_tiles, vtiles - tw);
      for (uint32_t t = threadIdx.x; t < span; t += kBinThreads) s_slot[t] = st[tw + t] + row[tw + t];
      __syncthreads();
      walk_keys<true>(vrec, vids, count, ch * kBinChunk, vi, L,
                      [&](uint32_t tile, uint32_t ent, uint32_t dep) {
                        const uint32_t k = tile - (uint32_t)tw;
                        if (k < span) staged[atomicAdd(&s_slot[k], 1u)] = ((uint64_t)dep << 32) | ent;
                      });
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// per-tile sort by (depth bits, entry)
// ---------------------------------------------------------------------------

template <typename K>
__device__ __forceinline__ void seg_store(K* keys, uint32_t* vals, int64_t pos, uint32_t tile,
                                          uint64_t k) {
  vals[pos] = (uint32_t)k;
  if constexpr (sizeof(K) == 8) {
    if (keys) keys[pos] = ((uint64_t)tile << 32) | (k >> 32);
  }
}

// The value of lane (this lane ^ jl), 64 bits: DPP quad permutations for 1
// and 2, a row rotation by 8 for 8, a lane permute otherwise.
__device__ __forceinline__ uint64_t lane_xor(uint64_t x, int jl) {
  const int lo = (int)(uint32_t)x, hi = (int)(uint32_t)(x >> 32);
  int a, b;
  switch (jl) {
    case 1:   // quad_perm [1, 0, 3, 2]
      a = __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xf, 0xf, true);
      b = __builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xf, 0xf, true);
      break;
    case 2:   // quad_perm [2, 3, 0, 1]
      a = __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xf, 0xf, true);
      b = __builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xf, 0xf, true);
      break;
    case 8:   // row_ror:8
      a = __builtin_amdgcn_update_dpp(0, lo, 0x128, 0xf, 0xf, true);
      b = __builtin_amdgcn_update_dpp(0, hi, 0x128, 0xf, 0xf, true);
      break;
    default:
      a = __shfl_xor(lo, jl, 64);
      b = __shfl_xor(hi, jl, 64);
      break;
  }
  return ((uint64_t)(uint32_t)b << 32) | (uint32_t)a;
}

// One stage (block size kk, partner distance j) of an ascending bitonic sort
// of the pairs whose indices are gbase + lane R + k, held in x[k] (R
// consecutive pairs per lane).  Partners closer than R are in the same lane;
// partners up to 64 R apart are exchanged across lanes.
template <int R>
__device__ __forceinline__ void bitonic_stage_wave(uint64_t (&x)[R], uint32_t lane, uint32_t gbase,
                                                   int kk, int j) {
  if (j < R) {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if ((k & j) == 0) {
        const bool up = ((gbase + lane * R + k) & kk) == 0;
        const uint64_t a = x[k], b = x[k + j];
        const bool sw = (b < a) == up;
        x[k] = sw ? b : a;
        x[k + j] = sw ? a : b;
      }
    }
  } else {
    const int jl = j / R;
    const bool up = ((gbase + lane * R) & kk) == 0;
    const bool keep_min = up == ((lane & jl) == 0);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint64_t y = lane_xor(x[k], jl);
      x[k] = ((y < x[k]) == keep_min) ? y : x[k];
    }
  }
}

// One wavefront sorts a list of at most 64 R pairs in registers.
template <int R, typename K>
__device__ __forceinline__ void wave_segment_sort(const uint64_t* __restrict__ staged, uint32_t s,
                                                  int len, uint32_t tile, K* keys, uint32_t* vals) {
  const uint32_t lane = lane_id();
  uint64_t x[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int i = (int)lane * R + k;
    x[k] = i < len ? staged[s + i] : ~0ull;
  }
#pragma unroll
  for (int kk = 2; kk <= 64 * R; kk <<= 1) {
#pragma unroll
    for (int j = kk >> 1; j > 0; j >>= 1) bitonic_stage_wave<R>(x, lane, 0u, kk, j);
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int i = (int)lane * R + k;
    if (i < len) seg_store(keys, vals, (int64_t)s + i, tile, x[k]);
  }
}

// The kSortWaves wavefronts of a workgroup sort a list of at most
// kSortWaves 64 R pairs: wavefront w holds indices w 64 R + lane R + k;
// partners 64 R or more apart are exchanged through LDS (s_x).
template <int R, typename K>
__device__ __forceinline__ void block_segment_sort(const uint64_t* __restrict__ staged, uint32_t s,
                                                   int len, uint32_t tile, K* keys, uint32_t* vals,
                                                   uint64_t* s_x) {
  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  const uint32_t gbase = w * 64 * R;
  uint64_t x[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int i = (int)(gbase + lane * R) + k;
    x[k] = i < len ? staged[s + i] : ~0ull;
  }
#pragma unroll
  for (int kk = 2; kk <= kSortWaves * 64 * R; kk <<= 1) {
#pragma unroll
    for (int j = kk >> 1; j > 0; j >>= 1) {
      if (j >= 64 * R) {
#pragma unroll
        for (int k = 0; k < R; ++k) s_x[gbase + lane * R + k] = x[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const uint32_t i = gbase + lane * R + k;
          const uint64_t y = s_x[i ^ (uint32_t)j];
          const bool keep_min = ((i & (uint32_t)kk) == 0) == ((i & (uint32_t)j) == 0);
          x[k] = ((y < x[k]) == keep_min) ? y : x[k];
        }
        __syncthreads();
      } else {
        bitonic_stage_wave<R>(x, lane, gbase, kk, j);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int i = (int)(gbase + lane * R) + k;
    if (i < len) seg_store(keys, vals, (int64_t)s + i, tile, x[k]);
  }
}

// Stable LSD radix sort of a long segment by its 64-bit (depth, entry) pair,
// one workgroup, 8 passes of 8 bits between buffers a and b (an even number:
// the result ends in a).  Per kSortThreads-key round, keys are ranked within
// their wavefront by match masks of equal digits and across wavefronts by
// their digit counts, which keeps equal digits in input order.
__device__ void radix_segment_sort(uint64_t* a, uint64_t* b, int64_t len, uint32_t* s_cnt,
                                   uint32_t* s_wdig /* [kSortWaves][256] */) {
  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  for (int pass = 0; pass < 8; ++pass) {
    const int shift = 8 * pass;
    if (threadIdx.x < 256) s_cnt[threadIdx.x] = 0u;
    __syncthreads();
    for (int64_t i = threadIdx.x; i < len; i += kSortThreads)
      atomicAdd(&s_cnt[(uint32_t)(a[i] >> shift) & 255u], 1u);
    __syncthreads();
    if (threadIdx.x == 0) {   // first output slot of every digit
      uint32_t run = 0;
      for (int d = 0; d < 256; ++d) {
        const uint32_t c = s_cnt[d];
        s_cnt[d] = run;
        run += c;
      }
    }
    __syncthreads();
    for (int64_t c0 = 0; c0 < len; c0 += kSortThreads) {
      const int64_t i = c0 + threadIdx.x;
      const bool valid = i < len;
      const uint64_t k = valid ? a[i] : 0ull;
      const uint32_t dig = valid ? (uint32_t)(k >> shift) & 255u : 0u;
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const uint64_t m = __ballot((dig >> bit) & 1u);
        peers &= ((dig >> bit) & 1u) ? m : ~m;
      }
      const uint32_t below = (uint32_t)__popcll(peers & ((uint64_t(1) << lane) - 1));
      for (int d = threadIdx.x; d < kSortWaves * 256; d += kSortThreads) s_wdig[d] = 0u;
      __syncthreads();
      if (valid && below == 0) s_wdig[w * 256 + dig] = (uint32_t)__popcll(peers);
      __syncthreads();
      if (valid) {
        uint32_t off = s_cnt[dig] + below;
        for (uint32_t q = 0; q < w; ++q) off += s_wdig[q * 256 + dig];
        b[off] = k;
      }
      __syncthreads();
      if (threadIdx.x < 256) {
        uint32_t add = 0;
        for (int q = 0; q < kSortWaves; ++q) add += s_wdig[q * 256 + threadIdx.x];
        s_cnt[threadIdx.x] += add;
      }
      __syncthreads();
    }
    uint64_t* t = a;
    a = b;
    b = t;
    __syncthreads();
  }
}

// Grid long_slots + T / kSortWaves.  The first long_slots workgroups take
// the queued lists longer than seg_short (all wavefronts of a workgroup up to
// kSegLong pairs, else the radix sort, whose pair buffers are `staged` itself
// and `spare`); they are dispatched first, so the long lists run beside the
// short ones.  In every later workgroup each wavefront sorts one tile's list
// of up to seg_short <= kSegShort pairs in registers.
template <typename K>
__global__ __launch_bounds__(kSortThreads) void seg_sort_kernel(const uint32_t* __restrict__ ranges,
                                                                int n_tiles,
                                                                uint64_t* __restrict__ staged,
                                                                uint64_t* __restrict__ spare,
                                                                K* __restrict__ keys,
                                                                uint32_t* __restrict__ vals,
                                                                const uint32_t* __restrict__ long_list,
                                                                const uint32_t* __restrict__ n_long,
                                                                int long_slots,
                                                                int seg_short) {
  __shared__ uint64_t s_mem[kSegLong + 128];   // pairs, or the radix sort's digit counts
  if (blockIdx.x < (unsigned)long_slots) {
    uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_mem + kSegLong);
    uint32_t* s_wdig = reinterpret_cast<uint32_t*>(s_mem);
    const uint32_t count = *n_long;
    for (uint32_t q = blockIdx.x; q < count; q += (uint32_t)long_slots) {
      const uint32_t tile = long_list[q];
      const uint32_t s = ranges[2 * (int64_t)tile], e = ranges[2 * (int64_t)tile + 1];
      const int64_t len = (int64_t)e - (int64_t)s;
      if (len <= kSortThreads) {
        block_segment_sort<1>(staged, s, (int)len, tile, keys, vals, s_mem);
      } else if (len <= 2 * kSortThreads) {
        block_segment_sort<2>(staged, s, (int)len, tile, keys, vals, s_mem);
      } else if (len <= kSegLong / 2) {
        block_segment_sort<kSegLong / (2 * kSortThreads)>(staged, s, (int)len, tile, keys, vals, s_mem);
      } else if (len <= kSegLong) {
        block_segment_sort<kSegLong / kSortThreads>(staged, s, (int)len, tile, keys, vals, s_mem);
      } else {
        radix_segment_sort(staged + s, spare + s, len, s_cnt, s_wdig);
        for (int64_t i = threadIdx.x; i < len; i += kSortThreads)
          seg_store(keys, vals, (int64_t)s + i, tile, staged[s + i]);
      }
      __syncthreads();   // LDS reused by the next list
    }
    return;
  }
  const int tile = (int)(blockIdx.x - long_slots) * kSortWaves + (int)(threadIdx.x >> 6);
  if (tile >= n_tiles) return;
  const uint32_t s = ranges[2 * (int64_t)tile], e = ranges[2 * (int64_t)tile + 1];
  const int64_t len = (int64_t)e - (int64_t)s;   // 0 for every tile on overflow
  const uint32_t t = (uint32_t)tile;
  if (len <= 0 || len > seg_short) return;
  if (len <= 64) wave_segment_sort<1>(staged, s, (int)len, t, keys, vals);
  else if (len <= 128) wave_segment_sort<2>(staged, s, (int)len, t, keys, vals);
  else if (len <= 256) wave_segment_sort<4>(staged, s, (int)len, t, keys, vals);
  else if (len <= 512) wave_segment_sort<8>(staged, s, (int)len, t, keys, vals);
  else wave_segment_sort<16>(staged, s, (int)len, t, keys, vals);
}

// ---------------------------------------------------------------------------
// tile order, longest lists first
// ---------------------------------------------------------------------------

// A stable sort of the tiles by 32 list length groups (0, then half
// octaves), longest group first and ascending tile index within a group, so
// that tiles running side by side stay close in the image.  Three passes over
// blocks of kOrderBlock tiles: group counts per block, per-(block, group)
// output offsets, stable scatter.
constexpr int kOrderGroups = 32;
constexpr int kOrderBlock = 256;

__device__ __forceinline__ int length_group(uint32_t len) {   // ascending in len
  if (len == 0) return 0;
  const int lg = 31 - __clz(len);
  const int half = lg > 0 ? (int)((len >> (lg - 1)) & 1u) : 0;
  return min(kOrderGroups - 1, 1 + 2 * lg + half);
}

__device__ __forceinline__ int tile_group(const uint32_t* ranges, int t) {
  return length_group(ranges[2 * (int64_t)t + 1] - ranges[2 * (int64_t)t]);
}

// Group of this thread's tile (-1 past the end), its rank among the block's
// earlier tiles of the same group, and the block's count of every group.
__device__ __forceinline__ int block_group_ranks(const uint32_t* ranges, int n_tiles,
                                                 uint32_t* s_wcnt /* [4][32] */,
                                                 uint32_t* s_cnt /* [32] */, uint32_t& rank) {
  const int t = blockIdx.x * kOrderBlock + (int)threadIdx.x;
  const int g = t < n_tiles ? tile_group(ranges, t) : -1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint64_t peers = 0;
  for (int h = 0; h < kOrderGroups; ++h) {
    const uint64_t m = __ballot(g == h);
    if (g == h) peers = m;
    if (lane == 0) s_wcnt[wave * kOrderGroups + h] = (uint32_t)__popcll(m);
  }
  __syncthreads();
  if (threadIdx.x < kOrderGroups) {
    uint32_t c = 0;
    for (int w = 0; w < kOrderBlock / 64; ++w) c += s_wcnt[w * kOrderGroups + threadIdx.x];
    s_cnt[threadIdx.x] = c;
  }
  rank = 0;
  if (g >= 0) {
    for (int w = 0; w < wave; ++w) rank += s_wcnt[w * kOrderGroups + g];
    rank += (uint32_t)__popcll(peers & ((uint64_t(1) << lane) - 1));
  }
  __syncthreads();
  return g;
}

__global__ __launch_bounds__(kOrderBlock) void order_count_kernel(
    const uint32_t* __restrict__ ranges, int n_tiles, uint32_t* __restrict__ blk) {
  __shared__ uint32_t s_wcnt[4 * kOrderGroups];
  __shared__ uint32_t s_cnt[kOrderGroups];
  uint32_t rank;
  block_group_ranks(ranges, n_tiles, s_wcnt, s_cnt, rank);
  if (threadIdx.x < kOrderGroups) blk[blockIdx.x * kOrderGroups + threadIdx.x] = s_cnt[threadIdx.x];
}

// One workgroup: blk[b][g] (counts) -> output offset of block b's group-g
// tiles.  Thread (g, j) owns the blocks of chunk j for group g.
__global__ __launch_bounds__(1024) void order_offsets_kernel(uint32_t* __restrict__ blk, int nblk) {
  __shared__ uint32_t s_part[kOrderGroups][33];
  __shared__ uint32_t s_start[kOrderGroups];
  const int g = threadIdx.x & 31, j = threadIdx.x >> 5;
  const int chunk = (nblk + 31) / 32;
  const int b0 = min(nblk, j * chunk), b1 = min(nblk, b0 + chunk);
  uint32_t sum = 0;
  for (int b = b0; b < b1; ++b) sum += blk[b * kOrderGroups + g];
  s_part[g][j] = sum;
  __syncthreads();
  if (threadIdx.x < kOrderGroups) {   // chunk prefix per group, then group totals
    uint32_t run = 0;
    for (int k = 0; k < 32; ++k) {
      const uint32_t v = s_part[threadIdx.x][k];
      s_part[threadIdx.x][k] = run;
      run += v;
    }
    s_part[threadIdx.x][32] = run;
  }
  __syncthreads();
  if (threadIdx.x == 0) {   // longest group first
    uint32_t run = 0;
    for (int h = kOrderGroups - 1; h >= 0; --h) {
      s_start[h] = run;
      run += s_part[h][32];
    }
  }
  __syncthreads();
  uint32_t off = s_start[g] + s_part[g][j];
  for (int b = b0; b < b1; ++b) {
    const uint32_t c = blk[b * kOrderGroups + g];
    blk[b * kOrderGroups + g] = off;
    off += c;
  }
}

__global__ __launch_bounds__(kOrderBlock) void order_scatter_kernel(
    const uint32_t* __restrict__ ranges, int n_tiles, const uint32_t* __restrict__ blk,
    uint32_t* __restrict__ order) {
  __shared__ uint32_t s_wcnt[4 * kOrderGroups];
  __shared__ uint32_t s_cnt[kOrderGroups];
  uint32_t rank;
  const int g = block_group_ranks(ranges, n_tiles, s_wcnt, s_cnt, rank);
  if (g >= 0)
    order[blk[blockIdx.x * kOrderGroups + g] + rank] = (uint32_t)(blockIdx.x * kOrderBlock + threadIdx.x);
}

// ---------------------------------------------------------------------------
// the short path: few entries, few tiles
// ---------------------------------------------------------------------------

// Calls walk_wave for a chunk's splats, dealt evenly to the workgroup's
// wavefronts: load(j) gives splat j's record and entry.
template <bool kDepth, typename Load, typename Op>
__device__ __forceinline__ void few_walk(uint32_t count, const ViewInfo& vi, WalkLds* L, Load load,
                                         Op op) {
  constexpr uint32_t kWaves = kFewThreads / 64;
  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  const uint32_t per = (count + kWaves - 1) / kWaves;
  const uint32_t end = min(count, (w + 1) * per);
  for (uint32_t j0 = w * per; j0 < end; j0 += 64) {
    uint32_t id = 0;
    uint4 c = make_uint4(0u, 0u, 0u, 0u);
    SplatKeys k{0u, 1u << 21};
    if (j0 + lane < end) {
      c = load(j0 + lane, id);
      k = splat_keys(c, vi);
    }
    walk_wave<kDepth>(k, id, c.w, vi, L[w], op);
  }
}

// Grid (chunks, views), chunks of kEntries entries: the chunk's splats that
// touch a tile go to its part of the list (and their number to few_count), and
// the keys they emit are counted per tile into the chunk's row of the matrix.
// Chunk b takes every gridDim.x-th run of 64 entries from run b on: neighbours
// in a map are neighbours in space, and chunks of consecutive entries would be
// all visible or not at all.
template <int kEntries>
__global__ __launch_bounds__(kFewThreads) void few_gather_kernel(
    const float2* __restrict__ xy, const int32_t* __restrict__ radius,
    const float4* __restrict__ rd, const uint32_t* __restrict__ stored, int n, ViewTable vt,
    uint32_t* __restrict__ few_count, uint4* __restrict__ rec, uint32_t* __restrict__ ids,
    uint32_t* __restrict__ matrix) {
  constexpr int kWaves = kFewThreads / 64;
  constexpr int kItems = (kEntries + kFewThreads - 1) / kFewThreads;
  extern __shared__ uint32_t s_hist[];
  __shared__ WalkLds L[kWaves];
  __shared__ uint4 s_rec[kEntries];
  __shared__ uint32_t s_wave[kWaves];
  const int v = blockIdx.y;
  const ViewInfo& vi = vt.v[v];
  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  const int vtiles = vi.tiles_x * vi.tiles_y;
  bool keep[kItems];
  uint4 c[kItems];
  int64_t entry[kItems];
  uint32_t mine = 0;
#pragma unroll
  for (int q = 0; q < kItems; ++q) {
    const int run = q * kWaves + (int)w;   // of the chunk's kEntries / 64
    const int64_t i = ((int64_t)run * gridDim.x + blockIdx.x) * 64 + lane;
    const bool mine_q = run < kEntries / 64 && i < n;
    entry[q] = (int64_t)v * n + (mine_q ? i : 0);
    const int32_t r = radius[entry[q]];
    const uint32_t x = stored ? stored[entry[q]] : (uint32_t)max(r, 0);
    const float2 m = xy[entry[q]];
    c[q] = make_uint4(__float_as_uint(m.x), __float_as_uint(m.y), (uint32_t)r,
                      __float_as_uint(rd[entry[q]].w));
    keep[q] = mine_q && x > 0u;
    mine += keep[q] ? 1u : 0u;
  }
  for (int t = threadIdx.x; t < vtiles; t += kFewThreads) s_hist[t] = 0u;
  const uint32_t inc = wave_prefix_sum(mine);
  if (lane == 63) s_wave[w] = inc;
  __syncthreads();
  uint32_t pos = inc - mine, count = 0;
#pragma unroll
  for (uint32_t k = 0; k < kWaves; ++k) {
    pos += k < w ? s_wave[k] : 0u;
    count += s_wave[k];
  }
  const int64_t seg = ((int64_t)v * gridDim.x + blockIdx.x) * kEntries;
#pragma unroll
  for (int q = 0; q < kItems; ++q) {
    if (keep[q]) {
      s_rec[pos] = c[q];
      rec[seg + pos] = c[q];
      ids[seg + pos] = (uint32_t)entry[q];
      ++pos;
    }
  }
  if (threadIdx.x == 0) few_count[v * gridDim.x + blockIdx.x] = count;
  __syncthreads();
  few_walk<false>(count, vi, L, [&](uint32_t j, uint32_t&) { return s_rec[j]; },
                  [&](uint32_t tile, uint32_t, uint32_t) { atomicAdd(&s_hist[tile], 1u); });
  __syncthreads();
  uint32_t* row = matrix + (int64_t)blockIdx.x * vt.n_tiles + vi.tile_base;
  for (int t = threadIdx.x; t < vtiles; t += kFewThreads) row[t] = s_hist[t];
}

// Grid T / 64: the wavefronts of a workgroup share the rows of 64 columns
// (kFewRows / kFewColWaves each, all in registers): every column's exclusive
// scan down the rows, in place, and its total.
__global__ __launch_bounds__(64 * kFewColWaves) void few_column_kernel(
    uint32_t* __restrict__ matrix, int rows, int n_tiles, uint32_t* __restrict__ counts) {
  constexpr int kOwn = kFewRows / kFewColWaves;
  __shared__ uint32_t s_sum[kFewColWaves][64];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  const int t = (int)blockIdx.x * 64 + lane;
  const int per = (rows + kFewColWaves - 1) / kFewColWaves;
  const int r0 = w * per, r1 = min(rows, r0 + per);
  uint32_t x[kOwn], sum = 0;
#pragma unroll
  for (int k = 0; k < kOwn; ++k)
    x[k] = r0 + k < r1 && t < n_tiles ? matrix[(int64_t)(r0 + k) * n_tiles + t] : 0u;
#pragma unroll
  for (int k = 0; k < kOwn; ++k) sum += x[k];
  s_sum[w][lane] = sum;
  __syncthreads();
  if (t >= n_tiles) return;
  uint32_t run = 0;
  for (int k = 0; k < w; ++k) run += s_sum[k][lane];
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {
    if (r0 + k < r1) matrix[(int64_t)(r0 + k) * n_tiles + t] = run;
    run += x[k];
  }
  if (w == kFewColWaves - 1) counts[t] = run;
}

// One workgroup, at most kFewTiles tiles: the segments and the key count (as
// bin_scan_down_kernel writes them), the queue of long lists, cleared tile
// counters and, when wanted, the tile order (as the order_* kernels write it).
__global__ __launch_bounds__(1024) void few_scan_kernel(
    const uint32_t* __restrict__ counts, int n_tiles, int64_t capacity,
    uint32_t* __restrict__ ranges, uint32_t* __restrict__ starts, uint64_t* __restrict__ total,
    uint32_t* __restrict__ n_keys, uint64_t* __restrict__ host_count,
    uint32_t* __restrict__ long_list, uint32_t* __restrict__ n_long, uint32_t* __restrict__ queue,
    uint32_t* __restrict__ order, uint32_t seg_short) {
  constexpr int kPer = kFewTiles / 1024;   // tile c 1024 + thread, c < kPer
  constexpr int kWaves = 16;
  constexpr int kCells = kOrderGroups * kPer * kWaves;   // (group, c, wave), longest group first
  __shared__ uint32_t s_tot[kPer * kWaves];   // per (c, wave): keys, then keys before it
  __shared__ uint32_t s_cell[kCells];
  __shared__ uint32_t s_wave[kWaves];
  __shared__ uint64_t s_all;
  __shared__ uint32_t s_long;
  const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
  if (queue)
    for (int k = threadIdx.x; k < GS_QUEUE_WORDS; k += 1024) queue[k] = 0u;
  if (threadIdx.x == 0) s_long = 0u;
  for (int k = threadIdx.x; k < kCells; k += 1024) s_cell[k] = 0u;
  uint32_t cnt[kPer], inc[kPer];
#pragma unroll
  for (int c = 0; c < kPer; ++c) {
    const int t = c * 1024 + (int)threadIdx.x;
    cnt[c] = t < n_tiles ? counts[t] : 0u;
  }
#pragma unroll
  for (int c = 0; c < kPer; ++c) {
    inc[c] = wave_prefix_sum(cnt[c]);
    if (lane == 63) s_tot[c * kWaves + w] = inc[c];
  }
  __syncthreads();
  if (w == 0) {
    constexpr int kOwn = kPer * kWaves / 64;   // totals per lane (below 2^26 together)
    uint32_t a[kOwn], sum = 0;
#pragma unroll
    for (int k = 0; k < kOwn; ++k) sum += a[k] = s_tot[kOwn * lane + k];
    const uint64_t p = wave_inclusive_scan<uint64_t>(sum);
    uint32_t run = (uint32_t)p - sum;   // exact whenever the keys fit the capacity's 32 bits
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      s_tot[kOwn * lane + k] = run;
      run += a[k];
    }
    if (lane == 63) {
      s_all = p;
      write_count(p, total, n_keys, host_count);
    }
  }
  __syncthreads();
  const bool ok = s_all <= (uint64_t)capacity;
  uint32_t rank[kPer];
#pragma unroll
  for (int c = 0; c < kPer; ++c) {
    const int t = c * 1024 + (int)threadIdx.x;
    if (c * 1024 >= n_tiles) break;   // uniform
    const uint32_t len = ok ? cnt[c] : 0u;
    const uint32_t st = s_tot[c * kWaves + w] + inc[c] - cnt[c];
    if (t < n_tiles) {
      ranges[2 * (int64_t)t] = len ? st : 0u;
      ranges[2 * (int64_t)t + 1] = len ? st + len : 0u;
      starts[t] = st;
      if (len > seg_short) long_list[atomicAdd(&s_long, 1u)] = (uint32_t)t;
    }
    // the lanes of this wavefront whose tiles share the length group
    const uint32_t g = (uint32_t)length_group(len);
    uint64_t peers = __ballot(t < n_tiles);
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      const uint64_t m = __ballot((g >> b) & 1u);
      peers &= ((g >> b) & 1u) ? m : ~m;
    }
    rank[c] = (uint32_t)__popcll(peers & ((uint64_t(1) << lane) - 1));
    if (t < n_tiles && rank[c] == 0)
      s_cell[((kOrderGroups - 1 - g) * kPer + c) * kWaves + w] = (uint32_t)__popcll(peers);
  }
  __syncthreads();
  if (threadIdx.x == 0) *n_long = s_long;
  if (!order) return;
  constexpr int kOwnCells = kCells / 1024;
  uint32_t cell[kOwnCells], mine = 0;
#pragma unroll
  for (int k = 0; k < kOwnCells; ++k) {
    cell[k] = s_cell[kOwnCells * threadIdx.x + k];
    mine += cell[k];
  }
  const uint32_t cinc = wave_prefix_sum(mine);
  if (lane == 63) s_wave[w] = cinc;
  __syncthreads();
  uint32_t off = cinc - mine;
  for (uint32_t k = 0; k < w; ++k) off += s_wave[k];
#pragma unroll
  for (int k = 0; k < kOwnCells; ++k) {
    s_cell[kOwnCells * threadIdx.x + k] = off;
    off += cell[k];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kPer; ++c) {
    const int t = c * 1024 + (int)threadIdx.x;
    if (c * 1024 >= n_tiles) break;
    if (t < n_tiles) {
      const uint32_t g = (uint32_t)length_group(ok ? cnt[c] : 0u);
      order[s_cell[((kOrderGroups - 1 - g) * kPer + c) * kWaves + w] + rank[c]] = (uint32_t)t;
    }
  }
}

// Grid (chunks, views): bin_emit_kernel on the short path's chunks.
__global__ __launch_bounds__(kFewThreads) void few_emit_kernel(
    const uint4* __restrict__ rec, const uint32_t* __restrict__ ids,
    const uint32_t* __restrict__ few_count, int entries, ViewTable vt,
    const uint32_t* __restrict__ matrix, const uint32_t* __restrict__ starts,
    const uint64_t* __restrict__ total, int64_t capacity, uint64_t* __restrict__ staged) {
  extern __shared__ uint32_t s_slot[];
  __shared__ WalkLds L[kFewThreads / 64];
  const int v = blockIdx.y;
  const uint32_t count = few_count[v * gridDim.x + blockIdx.x];
  if (count == 0 || *total > (uint64_t)capacity) return;
  const ViewInfo& vi = vt.v[v];
  const int vtiles = vi.tiles_x * vi.tiles_y;
  const uint32_t* row = matrix + (int64_t)blockIdx.x * vt.n_tiles + vi.tile_base;
  for (int t = threadIdx.x; t < vtiles; t += kFewThreads) s_slot[t] = starts[vi.tile_base + t] + row[t];
  const int64_t seg = ((int64_t)v * gridDim.x + blockIdx.x) * entries;
  __syncthreads();
  few_walk<true>(count, vi, L,
                 [&](uint32_t j, uint32_t& id) {
                   id = ids[seg + j];
                   return rec[seg + j];
                 },
                 [&](uint32_t tile, uint32_t ent, uint32_t dep) {
                   staged[atomicAdd(&s_slot[tile], 1u)] = ((uint64_t)dep << 32) | ent;
                 });
}

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

int64_t bin_chunks(int64_t n) { return (n + kBinChunk - 1) / kBinChunk; }   // at most

}  // namespace

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, value,
                     n);
  return hipGetLastError();
}

namespace {

// What the two paths need in different measure (elements).
struct BinScratch {
  size_t matrix;        // chunk x tile matrix
  size_t list;          // compacted splats
  size_t list_counts;   // their numbers, per view or per (view, chunk)
};

// For n Gaussians in n_views views of n_tiles tiles in all; few_entries: entries of a
// chunk on the short path, 0 on the general one.
BinScratch bin_scratch(int64_t n, int few_entries, int n_views, int64_t n_tiles) {
  if (few_entries == 0)
    return {(size_t)bin_chunks(n) * (size_t)n_tiles, (size_t)n * n_views, GS_MAX_VIEWS};
  const size_t chunks = (size_t)((n + few_entries - 1) / few_entries);
  return {chunks * (size_t)n_tiles, chunks * few_entries * n_views,
          std::max<size_t>(GS_MAX_VIEWS, chunks * n_views)};
}

// The most (view, Gaussian) entries of a call in chunks of 64, 256 and 1,024: the smallest
// chunks that number at most about 256 over all views (a small map fills the GPU, a larger
// one keeps the matrix small).
constexpr int kFewChunk[3] = {64, 256, 1024};
constexpr int64_t kFewChunkEntries[3] = {256 * 64, 256 * 256, kFewEntries};

void lay_out(BinSortPlan& P, const BinScratch& need) {
  const size_t nt = sizeof(uint32_t) * (size_t)std::max(P.n_tiles, 1);
  size_t off = 0;
  P.off_matrix = off;    off += align_up(sizeof(uint32_t) * need.matrix);
  P.off_list = off;      off += align_up(sizeof(uint4) * need.list);      // compacted splats
  P.off_ids = off;       off += align_up(sizeof(uint32_t) * need.list);   // their entries
  P.off_list_count = off; off += align_up(sizeof(uint32_t) * need.list_counts);
  P.off_counts = off;    off += align_up(nt);   // keys per tile
  P.off_starts = off;    off += align_up(nt);   // first slot of every tile's segment
  P.off_long = off;      off += align_up(nt);   // tiles whose lists the long grid sorts
  P.off_flag = off;      off += align_up(sizeof(uint64_t) * 2);   // key count, long-list count
  P.off_partial = off;   // per scan block: its tiles' key count
  off += align_up(sizeof(uint64_t) * (size_t)std::max(1, (P.n_tiles + kScanBlock - 1) / kScanBlock));
  P.off_order = off;     // tile order: per-(block, group) counts, then offsets
  off += align_up(sizeof(uint32_t) * kOrderGroups * ((P.n_tiles + kOrderBlock - 1) / kOrderBlock));
  P.off_staged = off;    off += align_up(sizeof(uint64_t) * (size_t)P.capacity);   // (depth, entry) pairs
  P.off_spare = off;     off += align_up(sizeof(uint64_t) * (size_t)P.capacity);   // radix partner
  P.total = off;
}

}  // namespace

BinSortPlan make_bin_sort_plan(int64_t n, const ViewTable& vt, int64_t capacity) {
  BinSortPlan P{};
  P.n_entries = n * vt.n_views;
  P.capacity = capacity;
  P.n_tiles = vt.n_tiles;
  P.chunks = bin_chunks(n);
  P.lds_tiles = 1;
  P.max_view_tiles = 1;
  for (int v = 0; v < vt.n_views; ++v) {
    P.max_view_tiles = std::max(P.max_view_tiles, vt.v[v].tiles_x * vt.v[v].tiles_y);
    P.lds_tiles = std::max(P.lds_tiles, std::min(kLdsTiles, vt.v[v].tiles_x * vt.v[v].tiles_y));
  }
  P.few_entries = 0;
  if (n > 0 && n <= kFewGaussians && P.n_entries <= kFewEntries && vt.n_tiles <= kFewTiles &&
      P.max_view_tiles <= kLdsTiles) {
    int k = 0;
    while (P.n_entries > kFewChunkEntries[k]) ++k;
    P.few_entries = kFewChunk[k];
    P.chunks = (n + P.few_entries - 1) / P.few_entries;
  }
  lay_out(P, bin_scratch(n, P.few_entries, vt.n_views, vt.n_tiles));
  return P;
}

size_t bin_sort_workspace_bound(int64_t n, const ViewTable& vt, int64_t capacity) {
  BinSortPlan P = make_bin_sort_plan(n, vt, capacity);
  // A smaller call can need more: its chunks are smaller, so its matrix has more rows.
  // The most that each chunk size needs over up to n Gaussians in any of the views, each
  // at most as large as it is (views sorted by tiles, the largest first).
  int tiles[GS_MAX_VIEWS];
  for (int v = 0; v < vt.n_views; ++v)
    tiles[v] = std::min(kLdsTiles, vt.v[v].tiles_x * vt.v[v].tiles_y);
  std::sort(tiles, tiles + vt.n_views, [](int a, int b) { return a > b; });
  BinScratch most = bin_scratch(n, P.few_entries, vt.n_views, vt.n_tiles);
  int64_t sum = 0;
  for (int V = 1; V <= vt.n_views; ++V) {
    sum = std::min<int64_t>(kFewTiles, sum + tiles[V - 1]);
    for (int k = 0; k < 3; ++k) {
      const int64_t m = std::min({n, kFewGaussians, kFewChunkEntries[k] / V});
      if (k > 0 && m * V <= kFewChunkEntries[k - 1]) break;   // no call has such chunks
      const BinScratch few = bin_scratch(m, kFewChunk[k], V, sum);
      most = {std::max(most.matrix, few.matrix), std::max(most.list, few.list),
              std::max(most.list_counts, few.list_counts)};
    }
  }
  lay_out(P, most);
  return P.total;
}

int run_bin_sort(const gs_projected& p, int64_t n, const ViewTable& vt, const gs_bins& bins,
                 uint32_t* n_keys_host, char* ws, const BinSortPlan& P, hipStream_t s) {
  auto* matrix = reinterpret_cast<uint32_t*>(ws + P.off_matrix);
  auto* list = reinterpret_cast<uint4*>(ws + P.off_list);
  auto* ids = reinterpret_cast<uint32_t*>(ws + P.off_ids);
  auto* list_count = reinterpret_cast<uint32_t*>(ws + P.off_list_count);
  auto* counts = reinterpret_cast<uint32_t*>(ws + P.off_counts);
  auto* starts = reinterpret_cast<uint32_t*>(ws + P.off_starts);
  auto* long_list = reinterpret_cast<uint32_t*>(ws + P.off_long);
  auto* total = reinterpret_cast<uint64_t*>(ws + P.off_flag);
  auto* n_long = reinterpret_cast<uint32_t*>(ws + P.off_flag + sizeof(uint64_t));
  auto* partial = reinterpret_cast<uint64_t*>(ws + P.off_partial);
  auto* order_blk = reinterpret_cast<uint32_t*>(ws + P.off_order);
  auto* staged = reinterpret_cast<uint64_t*>(ws + P.off_staged);
  auto* spare = reinterpret_cast<uint64_t*>(ws + P.off_spare);
  const auto* xy = reinterpret_cast<const float2*>(p.xy);
  const auto* rd = reinterpret_cast<const float4*>(p.rgb_depth);
  const int T = vt.n_tiles;
  const size_t lds = sizeof(uint32_t) * (size_t)P.lds_tiles;
  hipError_t e;

  kernel_event_start(GS_KERNEL_BIN_SORT, s);
  if (T == 0) {
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, s, bins.n_keys, 0u, (int64_t)1);
    if (bins.queue)
      hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, s, bins.queue, 0u,
                         (int64_t)GS_QUEUE_WORDS);
    kernel_event_stop(GS_KERNEL_BIN_SORT, s);
    return (e = hipGetLastError()) == hipSuccess ? GS_OK : hip_fail(e, "bin sort launch");
  }
  const dim3 bin_grid((unsigned)std::min<int64_t>(kBinGrid, std::max<int64_t>(P.chunks, 1)),
                      (unsigned)vt.n_views);
  // Short path: few entries and tiles, where launches and idle CUs are most of
  // the time.  Fixed chunks need no list shared by a view (its counter, clearing
  // and compaction), and one workgroup does the scans and the order: five
  // launches instead of eleven.  Whole call, short | general: 2,000 entries on
  // 80 tiles 23 | 41 us, 65,536 on 1,200 28 | 53, 262,144 on 3,225 38 | 56,
  // 600,000 on 14,400 58 | 105.  The limits are where the two meet (4 x 262,144
  // entries on 12,900 tiles: 64 | 67) and where one workgroup holds the tiles and
  // the column kernel a column's 256 rows.
  const bool few = P.few_entries != 0;
  // A caller that wants the key count gets it from the scan kernel by way of a word of
  // host memory, and the placement and the sort, which do nothing beyond the capacity,
  // are launched before it is waited for: after a copy of the count and a
  // synchronisation the GPU stood idle for these, their launches and the caller's next
  // (2,000 Gaussians rendered at 160x120: 87 us a call, and 43 so; 200,000 at 640x480,
  // forward and backward: 202 and 161).  A stream that is being recorded refuses the
  // synchronisation, as it always did.
  uint64_t* host_count = nullptr;
  CountWord word(s);
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (n_keys_host && hipStreamIsCapturing(s, &capture) == hipSuccess &&
      capture == hipStreamCaptureStatusNone)
    host_count = word.take();
  // Lists that a whole workgroup sorts: with few tiles from 256 pairs up, where a
  // wavefront alone takes 10 to 20 us while CUs idle (whole call, 256 | 1,024: 300 tiles
  // of 600 pairs 28 | 38 us, 1,200 of 230 34 | 36; 2,400 of 350 63 | 57, 9,600 of 290
  // 129 | 90).
  const int seg_short = few && T <= kSegFewTiles ? kSegFew : kSegShort;
  const dim3 few_grid((unsigned)P.chunks, (unsigned)vt.n_views);
  if (few) {
#define GS_GATHER(E)                                                                          \
  hipLaunchKernelGGL(few_gather_kernel<E>, few_grid, dim3(kFewThreads), lds, s, xy, p.radius, rd, \
                     p.tiles, (int)n, vt, list_count, list, ids, matrix)
    if (P.few_entries == 64) GS_GATHER(64);
    else if (P.few_entries == 256) GS_GATHER(256);
    else GS_GATHER(1024);
#undef GS_GATHER
    hipLaunchKernelGGL(few_column_kernel, dim3((unsigned)((T + 63) / 64)), dim3(64 * kFewColWaves),
                       0, s, matrix, (int)P.chunks, T, counts);
    hipLaunchKernelGGL(few_scan_kernel, dim3(1), dim3(1024), 0, s, counts, T, P.capacity,
                       bins.ranges, starts, total, bins.n_keys, host_count, long_list, n_long,
                       bins.queue, bins.order, (uint32_t)seg_short);
  } else {
    // 1. the splats that touch a tile, per view; keys per (chunk, tile), per
    // tile, the segments and the key count
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, s, list_count, 0u,
                       (int64_t)vt.n_views);
    if (n > 0) {
      hipLaunchKernelGGL(bin_compact_kernel, dim3((unsigned)((n + kCompactChunk - 1) / kCompactChunk),
                         (unsigned)vt.n_views), dim3(256), 0, s, xy, p.radius, rd, p.tiles, n,
                         list_count, list, ids);
      hipLaunchKernelGGL(bin_hist_kernel, bin_grid, dim3(kBinThreads), lds, s, list, list_count, n,
                         vt, P.lds_tiles, matrix);
    }
    hipLaunchKernelGGL(bin_column_kernel, dim3((unsigned)((P.max_view_tiles + 255) / 256),
                       (unsigned)vt.n_views), dim3(256), 0, s, matrix, list_count, vt, counts);
    const int nsb = (T + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(bin_scan_reduce_kernel, dim3((unsigned)nsb), dim3(256), 0, s, counts, T,
                       partial, n_long, bins.queue);
    hipLaunchKernelGGL(bin_scan_down_kernel, dim3((unsigned)nsb), dim3(256), 0, s, counts, T,
                       partial, nsb, P.capacity, bins.ranges, starts, total, bins.n_keys, host_count,
                       long_list, n_long);
  }
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "bin count launch");

  // 2. placement into the segments, then each segment sorted by (depth, entry)
  if (n > 0) {
    if (few)
      hipLaunchKernelGGL(few_emit_kernel, few_grid, dim3(kFewThreads), lds, s, list, ids,
                         list_count, P.few_entries, vt, matrix, starts, total,
                         P.capacity, staged);
    else
      hipLaunchKernelGGL(bin_emit_kernel, bin_grid, dim3(kBinThreads), lds, s, list, ids,
                         list_count, n, vt, P.lds_tiles, matrix, starts, total, P.capacity, staged);
    const int long_slots = std::min(kLongSlots, T);
    const unsigned sblocks = (unsigned)(long_slots + (T + kSortWaves - 1) / kSortWaves);
    if (bins.keys)
      hipLaunchKernelGGL(seg_sort_kernel<uint64_t>, dim3(sblocks), dim3(kSortThreads), 0, s,
                         bins.ranges, T, staged, spare, bins.keys, bins.values, long_list, n_long,
                         long_slots, seg_short);
    else
      hipLaunchKernelGGL(seg_sort_kernel<uint32_t>, dim3(sblocks), dim3(kSortThreads), 0, s,
                         bins.ranges, T, staged, spare, (uint32_t*)nullptr, bins.values, long_list,
                         n_long, long_slots, seg_short);
  }
  // 3. launch order of the compositing grids (from the ranges; on overflow
  // they are all empty and this is the identity)
  if (bins.order && !few) {
    const int nblk = (T + kOrderBlock - 1) / kOrderBlock;
    hipLaunchKernelGGL(order_count_kernel, dim3((unsigned)nblk), dim3(kOrderBlock), 0, s,
                       bins.ranges, T, order_blk);
    hipLaunchKernelGGL(order_offsets_kernel, dim3(1), dim3(1024), 0, s, order_blk, nblk);
    hipLaunchKernelGGL(order_scatter_kernel, dim3((unsigned)nblk), dim3(kOrderBlock), 0, s,
                       bins.ranges, T, order_blk, bins.order);
  }
  kernel_event_stop(GS_KERNEL_BIN_SORT, s);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "bin sort launch");
  if (!n_keys_host) return GS_OK;
  uint64_t tot = 0;
  if (host_count) {
    if ((e = word.wait(tot)) != hipSuccess) return hip_fail(e, "wait for the key count");
  } else {
    if ((e = hipMemcpyAsync(&tot, total, sizeof(uint64_t), hipMemcpyDeviceToHost, s)) != hipSuccess)
      return hip_fail(e, "read key count");
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "synchronise key count");
  }
  *n_keys_host = tot > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)tot;
  if (tot <= (uint64_t)P.capacity) return GS_OK;
  // the ranges are all empty and the order the identity; nothing of this call is under
  // way when the caller hears of it
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "synchronise bin sort");
  set_error("gs_bin_sort: %llu keys exceed capacity %lld", (unsigned long long)tot,
            (long long)P.capacity);
  return GS_ERR_CAPACITY;
}

}  // namespace gsmi
