// Segmenting on the GPU: validate matches, give each its canonical camera
// pair (i < j, keypoints swapped when needed), stable-sort by pair with an
// LSD radix sort, find the pair runs and gather the structure-of-arrays
// device layout.  This is the data marshalling that precedes the epipolar
// adjustment iterations (FastMap, Experiments: marshalling done on the GPU
// with tensor indexing); here every step is an integer kernel so the result
// is bit-exact and deterministic.
//
// All of it is bound by memory.  The matches arrive in any order, so one
// pass has to reach into memory at random: validation packs each match's
// four coordinates, already in the pair's orientation, into one 16-byte
// record, so that the gather after the sort makes one random access per
// match instead of six of 4 bytes (30M matches in random order, 1,000
// cameras: gather 3,447 -> 821 us).  The sort moves 8 bytes per match and
// pass (key; input index with the swap flag in its top bit) and takes the
// fewest passes of at most 8 bits; a tile of 4,096 keys is first sorted in
// LDS so that a digit's keys leave as one run (five 4-bit passes 2,070 ->
// three 7-bit passes 590 us).  Records and keys live in the two buffers
// that hold the filtered layouts of later rounds and are free until then.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "fea_ctx.h"
#include "fea_device.h"

namespace fea {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanPer = 8;
constexpr int kScanTile = kScanThreads * kScanPer;
constexpr int kMaxRadixBits = 8;
constexpr int kMaxRadixBins = 1 << kMaxRadixBits;
constexpr int kRsThreads = 256;
constexpr int kRsWaves = kRsThreads / kWave;
constexpr int kRsPer = 16;
constexpr int kRsTile = kRsThreads * kRsPer;
constexpr int kRsWaveTile = kRsPer * kWave;  // consecutive keys of one wave of a tile
static_assert(kRsThreads == kMaxRadixBins, "one thread per digit in the tile's scan");
constexpr int32_t kSwapBit = INT32_MIN;      // of a sort value: the match's cameras were exchanged

// Exclusive scan of a 256-thread block's values; returns this thread's
// exclusive prefix and writes the block total to *total.
__device__ int block_exclusive_scan(int v, int* total, int* s_w) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int inc = wave_inclusive_scan(v);
  if (lane == 63) s_w[wid] = inc;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) {
    const int x = s_w[w];
    before += (w < wid) ? x : 0;
    all += x;
  }
  __syncthreads();
  *total = all;
  return before + inc - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_tile(int* __restrict__ data, int64_t n,
                                                             int* __restrict__ tile_sums) {
  __shared__ int s_w[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
  int v[kScanPer];
  int sum = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = (base + k < n) ? data[base + k] : 0;
    sum += v[k];
  }
  int total;
  int run = block_exclusive_scan(sum, &total, s_w);
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    if (base + k < n) data[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 0 && tile_sums) tile_sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_add(int* __restrict__ data, int64_t n,
                                                            const int* __restrict__ offs) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
  const int o = offs[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kScanPer; ++k)
    if (base + k < n) data[base + k] += o;
}

// In-place exclusive scan of n ints; scratch must hold scan_scratch_ints(n).
int64_t scan_scratch_ints(int64_t n) {
  int64_t need = 0;
  while (n > kScanTile) {
    n = (n + kScanTile - 1) / kScanTile;
    need += n;
  }
  return need + 1;
}

hipError_t device_exclusive_scan(int* data, int64_t n, int* scratch, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t tiles = (n + kScanTile - 1) / kScanTile;
  if (tiles == 1) {
    k_scan_tile<<<1, kScanThreads, 0, st>>>(data, n, nullptr);
    return hipGetLastError();
  }
  k_scan_tile<<<(unsigned)tiles, kScanThreads, 0, st>>>(data, n, scratch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = device_exclusive_scan(scratch, tiles, scratch + tiles, st);
  if (e != hipSuccess) return e;
  k_scan_add<<<(unsigned)tiles, kScanThreads, 0, st>>>(data, n, scratch);
  return hipGetLastError();
}

// Validation, canonical keys (key = i * N + j with i < j), sort values (input
// index, top bit set when the cameras are exchanged) and the coordinates in
// the pair's orientation, one record per match.
__global__ void k_validate(int64_t n, int N, const int32_t* __restrict__ cam1, const int32_t* __restrict__ cam2,
                           const float* __restrict__ x1, const float* __restrict__ y1,
                           const float* __restrict__ x2, const float* __restrict__ y2,
                           uint32_t* __restrict__ keys, int32_t* __restrict__ vals, float4* __restrict__ rec,
                           int* __restrict__ err) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n) return;
  const int c1 = cam1[m], c2 = cam2[m];
  const float a = x1[m], b = y1[m], c = x2[m], d = y2[m];
  int bits = 0;
  if (c1 < 0 || c1 >= N || c2 < 0 || c2 >= N)
    bits |= kErrRange;
  else if (c1 == c2)
    bits |= kErrSameCam;
  if (!isfinite(a) || !isfinite(b) || !isfinite(c) || !isfinite(d)) bits |= kErrNonFinite;
  if (bits) atomicOr(err, bits);
  // ids out of range are clamped: the call fails once the error bits are read
  const uint32_t i = (uint32_t)min(max(min(c1, c2), 0), N - 1);
  const uint32_t j = (uint32_t)min(max(max(c1, c2), 0), N - 1);
  const bool s = c1 > c2;
  keys[m] = i * (uint32_t)N + j;
  vals[m] = (int32_t)m | (s ? kSwapBit : 0);
  rec[m] = s ? make_float4(c, d, a, b) : make_float4(a, b, c, d);
}

// Digit counts of every tile, digit-major: hist[digit * n_tiles + tile].
__global__ __launch_bounds__(kRsThreads) void k_radix_hist(const uint32_t* __restrict__ keys, int64_t n,
                                                           int shift, int bits, int n_tiles, int* __restrict__ hist) {
  __shared__ int h[kMaxRadixBins];
  const int bins = 1 << bits, tid = threadIdx.x;
  h[tid] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kRsTile + tid;
  uint32_t key[kRsPer];
#pragma unroll
  for (int k = 0; k < kRsPer; ++k) key[k] = keys[min(base + k * kRsThreads, n - 1)];  // all in flight together
#pragma unroll
  for (int k = 0; k < kRsPer; ++k)
    if (base + k * kRsThreads < n) atomicAdd(&h[(key[k] >> shift) & (bins - 1)], 1);
  __syncthreads();
  if (tid < bins) hist[(int64_t)tid * n_tiles + blockIdx.x] = h[tid];
}

// Stable scatter of one radix pass.  Wave w of a tile owns its kRsWaveTile
// consecutive keys from w * kRsWaveTile and takes them 64 at a time in input
// order: the lanes holding the same digit find each other with one ballot
// per digit bit, a key's rank is the number of such lanes below it plus the
// wave's count of that digit so far.  The tile is then laid out by digit in
// LDS and written from there, consecutive lanes to consecutive places of a
// digit's run.
__global__ __launch_bounds__(kRsThreads) void k_radix_scatter(const uint32_t* __restrict__ kin,
                                                              const int32_t* __restrict__ vin,
                                                              uint32_t* __restrict__ kout,
                                                              int32_t* __restrict__ vout, int64_t n, int shift,
                                                              int bits, int n_tiles, const int* __restrict__ offs) {
  __shared__ uint32_t s_key[kRsTile];
  __shared__ int32_t s_val[kRsTile];
  __shared__ int s_cnt[kRsWaves][kMaxRadixBins];
  __shared__ int s_off[kMaxRadixBins];  // global place of a digit's run minus its place in the tile
  __shared__ int s_w[kRsWaves];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint32_t dmask = (1u << bits) - 1u;
  const int64_t tile0 = (int64_t)blockIdx.x * kRsTile;
  const int64_t base = tile0 + wid * kRsWaveTile + lane;
  uint32_t key[kRsPer];
  int32_t val[kRsPer];
#pragma unroll
  for (int r = 0; r < kRsPer; ++r) {
    const bool ok = base + r * kWave < n;
    const int64_t p = ok ? base + r * kWave : n - 1;  // n >= 1; the last key's copies are not used
    key[r] = kin[p];
    val[r] = vin[p];
  }
  for (int d = tid; d < kRsWaves * kMaxRadixBins; d += kRsThreads) (&s_cnt[0][0])[d] = 0;
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
  int rank[kRsPer];
#pragma unroll
  for (int r = 0; r < kRsPer; ++r) {
    const bool ok = base + r * kWave < n;
    const uint32_t d = (key[r] >> shift) & dmask;
    uint64_t peers = __ballot(ok);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    // every lane reads the wave's count before the digit's first lane
    // raises it (one wave, LDS operations in order)
    const int before = __hip_atomic_load(&s_cnt[wid][d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    const int mine = __popcll(peers & below);
    __builtin_amdgcn_wave_barrier();
    if (ok && mine == 0)
      __hip_atomic_store(&s_cnt[wid][d], before + __popcll(peers), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    __builtin_amdgcn_wave_barrier();
    rank[r] = before + mine;
  }
  __syncthreads();
  {
    // per digit: the waves' counts to exclusive prefixes, then the digits'
    // starts within the tile (digits past the pass's bins count zero)
    int c[kRsWaves], sum = 0;
#pragma unroll
    for (int w = 0; w < kRsWaves; ++w) {
      c[w] = sum;
      sum += s_cnt[w][tid];
    }
    int total;
    const int start = block_exclusive_scan(sum, &total, s_w);
#pragma unroll
    for (int w = 0; w < kRsWaves; ++w) s_cnt[w][tid] = start + c[w];
    s_off[tid] = tid <= (int)dmask ? offs[(int64_t)tid * n_tiles + blockIdx.x] - start : 0;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRsPer; ++r) {
    if (base + r * kWave >= n) continue;
    const int q = s_cnt[wid][(key[r] >> shift) & dmask] + rank[r];
    s_key[q] = key[r];
    s_val[q] = val[r];
  }
  __syncthreads();
  const int cnt_tile = (int)min((int64_t)kRsTile, n - tile0);
  for (int q = tid; q < cnt_tile; q += kRsThreads) {
    const uint32_t k = s_key[q];
    const int64_t dst = (int64_t)s_off[(k >> shift) & dmask] + q;
    kout[dst] = k;
    vout[dst] = s_val[q];
  }
}

// The first position of every pair's run ("head") in a wave's kRsWaveTile
// sorted keys, 64 at a time: bit l of heads[r] for position base + 64 r + l.
// Returns how many there are.
__device__ __forceinline__ int wave_heads(const uint32_t* __restrict__ sk, int64_t base, int64_t n, int lane,
                                          uint32_t (&key)[kRsPer], uint64_t (&heads)[kRsPer]) {
  int c = 0;
#pragma unroll
  for (int r = 0; r < kRsPer; ++r) {
    const int64_t p = base + r * kWave + lane;
    key[r] = sk[min(p, n - 1)];  // n >= 1
    const uint32_t prev = sk[max(min(p, n) - 1, (int64_t)0)];
    heads[r] = __ballot(p < n && (p == 0 || key[r] != prev));
    c += __popcll(heads[r]);
  }
  return c;
}

// Heads before this wave's keys: the tile's (exclusive scan over the tiles)
// plus the tile's waves below.
__device__ __forceinline__ int heads_before(int mine, int tile_base, int wid, int lane, int* s_w) {
  if (lane == 0) s_w[wid] = mine;
  __syncthreads();
  int b = tile_base;
#pragma unroll
  for (int w = 0; w < kRsWaves; ++w) b += w < wid ? s_w[w] : 0;
  return b;
}

__global__ __launch_bounds__(kRsThreads) void k_head_count(const uint32_t* __restrict__ sk, int64_t n,
                                                           int* __restrict__ tile_heads) {
  __shared__ int s_w[kRsWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t key[kRsPer];
  uint64_t heads[kRsPer];
  const int c = wave_heads(sk, (int64_t)blockIdx.x * kRsTile + wid * kRsWaveTile, n, lane, key, heads);
  if (lane == 0) s_w[wid] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < kRsWaves; ++w) t += s_w[w];
    tile_heads[blockIdx.x] = t;
  }
}

// Pair table: key and first sorted position of every run, in order.
__global__ __launch_bounds__(kRsThreads) void k_heads(const uint32_t* __restrict__ sk, int64_t n,
                                                      const int* __restrict__ tile_base,
                                                      uint32_t* __restrict__ pair_key,
                                                      int32_t* __restrict__ seg_start, int* __restrict__ n_pairs) {
  __shared__ int s_w[kRsWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kRsTile + wid * kRsWaveTile;
  uint32_t key[kRsPer];
  uint64_t heads[kRsPer];
  const int c = wave_heads(sk, base, n, lane, key, heads);
  int id = heads_before(c, tile_base[blockIdx.x], wid, lane, s_w);
  if (blockIdx.x == gridDim.x - 1 && wid == kRsWaves - 1 && lane == 0) *n_pairs = id + c;
#pragma unroll
  for (int r = 0; r < kRsPer; ++r) {
    if ((heads[r] >> lane) & 1ull) {
      const int k = id + __popcll(heads[r] & ((1ull << lane) - 1ull));
      pair_key[k] = key[r];
      seg_start[k] = (int32_t)(base + r * kWave + lane);
    }
    id += __popcll(heads[r]);
  }
}

// The layout: position p of pair k goes to slot p + shift[k] (the pair's
// aligned start minus its first position).
__global__ __launch_bounds__(kRsThreads) void k_gather(const uint32_t* __restrict__ sk, int64_t n,
                                                       const int* __restrict__ tile_base,
                                                       const int32_t* __restrict__ sv,
                                                       const int32_t* __restrict__ shift,
                                                       const float4* __restrict__ rec, float* __restrict__ ox1,
                                                       float* __restrict__ oy1, float* __restrict__ ox2,
                                                       float* __restrict__ oy2, int32_t* __restrict__ opos,
                                                       int32_t* __restrict__ perm, uint8_t* __restrict__ swp) {
  __shared__ int s_w[kRsWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kRsTile + wid * kRsWaveTile;
  uint32_t key[kRsPer];
  uint64_t heads[kRsPer];
  const int c = wave_heads(sk, base, n, lane, key, heads);
  int id = heads_before(c, tile_base[blockIdx.x], wid, lane, s_w) - 1;
  const uint64_t upto = lane == 63 ? ~0ull : (1ull << (lane + 1)) - 1ull;
#pragma unroll 4
  for (int r = 0; r < kRsPer; ++r) {
    const int64_t p = base + r * kWave + lane;
    const int k = id + __popcll(heads[r] & upto);
    id += __popcll(heads[r]);
    if (p >= n) continue;
    const int32_t v = sv[p];
    const int32_t m = v & ~kSwapBit;
    const float4 q = rec[m];
    const int64_t dst = p + shift[k];
    __builtin_nontemporal_store(q.x, ox1 + dst);
    __builtin_nontemporal_store(q.y, oy1 + dst);
    __builtin_nontemporal_store(q.z, ox2 + dst);
    __builtin_nontemporal_store(q.w, oy2 + dst);
    __builtin_nontemporal_store((int32_t)p, opos + dst);
    __builtin_nontemporal_store(m, perm + p);
    __builtin_nontemporal_store((uint8_t)(v < 0 ? 1 : 0), swp + p);
  }
}

// The alignment padding after every pair's run (fewer than kAlign slots):
// zero coordinates, position -1.  One thread per (pair, slot).
__global__ void k_pad(int64_t n_pairs, const int32_t* __restrict__ shift, const int32_t* __restrict__ seg_end,
                      float* __restrict__ ox1, float* __restrict__ oy1, float* __restrict__ ox2,
                      float* __restrict__ oy2, int32_t* __restrict__ opos) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t k = t / kAlign;
  if (k >= n_pairs) return;
  const int64_t end = (int64_t)seg_end[k] + shift[k];  // slot past the pair's last match
  const int64_t s = end + t % kAlign;
  if (s >= (end + kAlign - 1) / kAlign * kAlign) return;
  ox1[s] = oy1[s] = ox2[s] = oy2[s] = 0.f;
  opos[s] = -1;
}

#define FEA_TRY(expr)                    \
  do {                                   \
    hipError_t _e = (expr);              \
    if (_e != hipSuccess) return _e;     \
  } while (0)

hipError_t alloc_dbuf(DBuf& b, size_t bytes) {
  if (b.p && b.bytes >= bytes) return hipSuccess;
  if (b.p) (void)hipFree(b.p);
  b.p = nullptr;
  b.bytes = 0;
  FEA_TRY(hipMalloc(&b.p, std::max<size_t>(bytes, 16)));
  b.bytes = bytes;
  return hipSuccess;
}

// Export, pass 1: the coordinates of every real slot of the full layout to
// its sorted position (padding slots hold lpos = -1).
__global__ void k_export_coords(int64_t n_slots, const int32_t* __restrict__ lpos, const float* __restrict__ x1,
                                const float* __restrict__ y1, const float* __restrict__ x2,
                                const float* __restrict__ y2, float* __restrict__ ox1, float* __restrict__ oy1,
                                float* __restrict__ ox2, float* __restrict__ oy2) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_slots) return;
  const int32_t q = lpos[s];
  if (q < 0) return;
  ox1[q] = x1[s];
  oy1[q] = y1[s];
  ox2[q] = x2[s];
  oy2[q] = y2[s];
}

// Export, pass 2: one workgroup per pair writes the pair's camera ids
// (offset by cam_base) over its sorted range.
__global__ void k_export_cams(const int64_t* __restrict__ seg_off, const int32_t* __restrict__ pair_i,
                              const int32_t* __restrict__ pair_j, int32_t cam_base, int32_t* __restrict__ c1,
                              int32_t* __restrict__ c2) {
  const int n = blockIdx.x;
  const int32_t a = pair_i[n] + cam_base, b = pair_j[n] + cam_base;
  for (int64_t q = seg_off[n] + threadIdx.x; q < seg_off[n + 1]; q += blockDim.x) {
    c1[q] = a;
    c2[q] = b;
  }
}

}  // namespace

// The loaded matches in sorted order (each canonical, lower camera first),
// into device arrays [n_matches] of the context's device: coordinates as
// loaded, camera ids offset by cam_base.  seg_off_dev: the pair ranges
// [P + 1] on the device (caller-provided scratch).
hipError_t export_sorted(fea_ctx* c, int32_t cam_base, const int64_t* seg_off_dev, float* x1, float* y1,
                         float* x2, float* y2, int32_t* cam1, int32_t* cam2) {
  int64_t slots = 0;
  for (int64_t n = 0; n < c->P; ++n)
    slots += (c->seg_off[n + 1] - c->seg_off[n] + kAlign - 1) / kAlign * kAlign;
  if (slots > 0)
    k_export_coords<<<(unsigned)((slots + 255) / 256), 256, 0, c->stream>>>(
        slots, c->lpos[0].as<int32_t>(), c->lay[0][0].as<float>(), c->lay[0][1].as<float>(),
        c->lay[0][2].as<float>(), c->lay[0][3].as<float>(), x1, y1, x2, y2);
  if (c->P > 0)
    k_export_cams<<<(unsigned)c->P, 256, 0, c->stream>>>(seg_off_dev, c->d_pair_i.as<int32_t>(),
                                                       c->d_pair_j.as<int32_t>(), cam_base, cam1, cam2);
  return hipGetLastError();
}

// The filtered layouts' buffers (1 and 2) for `slots` slots each: one block
// per layout, its four coordinate arrays views into it.
hipError_t alloc_filtered_layouts(fea_ctx* c, int64_t slots) {
  const size_t each = (std::max<int64_t>(slots, 1) * sizeof(float) + 255) / 256 * 256;
  for (int b = 1; b < 3; ++b) {
    if (!(c->lay_block[b].p && c->lay_block[b].bytes >= 4 * each)) {
      for (int a = 0; a < 4; ++a) c->lay[b][a] = DBuf();
      FEA_TRY(alloc_dbuf(c->lay_block[b], 4 * each));
    }
    const size_t part = c->lay_block[b].bytes / 4 / 256 * 256;
    for (int a = 0; a < 4; ++a) {
      c->lay[b][a].p = c->lay_block[b].as<uint8_t>() + a * part;
      c->lay[b][a].bytes = part;
    }
    FEA_TRY(alloc_dbuf(c->lpos[b], each));
  }
  return hipSuccess;
}

hipError_t segment_matches(fea_ctx* c, const float* x1, const float* y1, const float* x2, const float* y2,
                           const int32_t* cam1, const int32_t* cam2, int* bad_bits) {
  hipStream_t st = c->stream;
  const int64_t M = c->M;
  const int N = c->N;
  *bad_bits = 0;
  // the fewest LSD passes of at most kMaxRadixBits over the keys' bits
  const uint64_t max_key = (uint64_t)N * (uint64_t)N;
  int bits = 1;
  while (bits < 32 && (1ull << bits) < max_key) ++bits;
  const int passes = (bits + kMaxRadixBits - 1) / kMaxRadixBits;
  const int digit = (bits + passes - 1) / passes;
  const int64_t n_tiles = (M + kRsTile - 1) / kRsTile;
  const int64_t hist_n = ((int64_t)1 << digit) * std::max<int64_t>(n_tiles, 1);
  // the filtered layouts hold the sort meanwhile: records in the first one's
  // block, keys and values (double-buffered) in the second's, the pair table
  // in their position arrays.  Pairs of 1,000 matches need M / 64 slots of
  // padding at most; a layout that turns out larger is allocated again below
  const int64_t max_pairs = std::min<int64_t>(M, (int64_t)N * (N - 1) / 2);
  FEA_TRY(alloc_filtered_layouts(c, M + std::min<int64_t>(M / 64, (kAlign - 1) * max_pairs)));
  float4* rec = c->lay_block[1].as<float4>();
  uint32_t *kin = c->lay[2][0].as<uint32_t>(), *kout = c->lay[2][1].as<uint32_t>();
  int32_t *vin = c->lay[2][2].as<int32_t>(), *vout = c->lay[2][3].as<int32_t>();
  uint32_t* pair_key = c->lpos[1].as<uint32_t>();
  int32_t* seg_start = c->lpos[2].as<int32_t>();
  const int64_t scr_n = scan_scratch_ints(std::max<int64_t>(hist_n, n_tiles));
  FEA_TRY(alloc_dbuf(c->seg_ws, (size_t)(2 + n_tiles + 1 + hist_n + scr_n) * sizeof(int)));
  int* err = c->seg_ws.as<int>();  // error bits, pair count
  int *tile_heads = err + 2, *hist = tile_heads + n_tiles + 1, *scan_scr = hist + hist_n;
  int h_head[2] = {0, 0};
  if (M > 0) {
    FEA_TRY(hipMemsetAsync(err, 0, 2 * sizeof(int), st));
    k_validate<<<(unsigned)((M + 255) / 256), 256, 0, st>>>(M, N, cam1, cam2, x1, y1, x2, y2, kin, vin, rec, err);
    FEA_TRY(hipGetLastError());
    for (int ps = 0; ps < passes; ++ps) {
      const int shift = ps * digit;
      k_radix_hist<<<(unsigned)n_tiles, kRsThreads, 0, st>>>(kin, M, shift, digit, (int)n_tiles, hist);
      FEA_TRY(hipGetLastError());
      FEA_TRY(device_exclusive_scan(hist, hist_n, scan_scr, st));
      k_radix_scatter<<<(unsigned)n_tiles, kRsThreads, 0, st>>>(kin, vin, kout, vout, M, shift, digit, (int)n_tiles,
                                                                hist);
      FEA_TRY(hipGetLastError());
      std::swap(kin, kout);
      std::swap(vin, vout);
    }
    // pair runs
    k_head_count<<<(unsigned)n_tiles, kRsThreads, 0, st>>>(kin, M, tile_heads);
    FEA_TRY(hipGetLastError());
    FEA_TRY(device_exclusive_scan(tile_heads, n_tiles, scan_scr, st));
    k_heads<<<(unsigned)n_tiles, kRsThreads, 0, st>>>(kin, M, tile_heads, pair_key, seg_start, err + 1);
    FEA_TRY(hipGetLastError());
    FEA_TRY(hipMemcpyAsync(h_head, err, 2 * sizeof(int), hipMemcpyDeviceToHost, st));
    FEA_TRY(hipStreamSynchronize(st));
    if (h_head[0]) {
      *bad_bits = h_head[0];
      return hipSuccess;
    }
  }
  const int64_t P = h_head[1];
  std::vector<uint32_t> h_key(P);
  std::vector<int32_t> h_start(P);
  if (P > 0) {
    FEA_TRY(hipMemcpyAsync(h_key.data(), pair_key, P * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    FEA_TRY(hipMemcpyAsync(h_start.data(), seg_start, P * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    FEA_TRY(hipStreamSynchronize(st));
  }
  c->P = P;
  c->pair_i.resize(P);
  c->pair_j.resize(P);
  c->seg_off.resize(P + 1);
  c->phys_off.resize(P);
  c->cur_len.resize(P);
  std::vector<int32_t> h_shift(2 * P);  // per pair: slot minus position, then the pairs' ends
  int64_t off = 0;
  for (int64_t k = 0; k < P; ++k) {
    c->pair_i[k] = (int32_t)(h_key[k] / (uint32_t)N);
    c->pair_j[k] = (int32_t)(h_key[k] % (uint32_t)N);
    c->seg_off[k] = h_start[k];
    const int64_t end = (k + 1 < P) ? (int64_t)h_start[k + 1] : M, len = end - h_start[k];
    c->cur_len[k] = len;
    c->phys_off[k] = off;
    h_shift[k] = (int32_t)(off - h_start[k]);
    h_shift[P + k] = (int32_t)end;
    off += (len + kAlign - 1) / kAlign * kAlign;
  }
  c->seg_off[P] = M;
  c->layout_len = off;
  c->cur = 0;
  if (off >= (int64_t)1 << 31) return hipSuccess;  // refused by the caller
  // the full device layout (buffer 0; the filtered rounds use buffers 1, 2)
  const size_t cap = (size_t)std::max<int64_t>(off, 1);
  for (int a = 0; a < 4; ++a) FEA_TRY(alloc_dbuf(c->lay[0][a], cap * sizeof(float)));
  FEA_TRY(alloc_dbuf(c->lpos[0], cap * sizeof(int32_t)));
  FEA_TRY(alloc_dbuf(c->perm, std::max<int64_t>(M, 1) * sizeof(int32_t)));
  FEA_TRY(alloc_dbuf(c->swp, std::max<int64_t>(M, 1)));
  if (P > 0) {
    float *o1 = c->lay[0][0].as<float>(), *o2 = c->lay[0][1].as<float>(), *o3 = c->lay[0][2].as<float>(),
          *o4 = c->lay[0][3].as<float>();
    int32_t* opos = c->lpos[0].as<int32_t>();
    // the shifts and ends take the pair table's place (its copy is on the host)
    FEA_TRY(hipMemcpyAsync(c->lpos[1].p, h_shift.data(), P * sizeof(int32_t), hipMemcpyHostToDevice, st));
    FEA_TRY(hipMemcpyAsync(c->lpos[2].p, h_shift.data() + P, P * sizeof(int32_t), hipMemcpyHostToDevice, st));
    const int32_t *shift = c->lpos[1].as<int32_t>(), *ends = c->lpos[2].as<int32_t>();
    k_gather<<<(unsigned)n_tiles, kRsThreads, 0, st>>>(kin, M, tile_heads, vin, shift, rec, o1, o2, o3, o4, opos,
                                                       c->perm.as<int32_t>(), c->swp.as<uint8_t>());
    FEA_TRY(hipGetLastError());
    k_pad<<<(unsigned)((P * kAlign + 255) / 256), 256, 0, st>>>(P, shift, ends, o1, o2, o3, o4, opos);
    FEA_TRY(hipGetLastError());
  }
  FEA_TRY(hipStreamSynchronize(st));
  return alloc_filtered_layouts(c, off);
}

namespace {

constexpr int kItThreads = 256;
// A launch takes fewer than 2^32 threads, and a layout up to 2^31 / kAlign
// pairs: a wavefront for each and two threads for its camera entries would be
// more, so past kItPairBlocks workgroups the wavefronts take further pairs.
constexpr int64_t kItPairBlocks = 1 << 23;
constexpr int64_t kItMaxPairs = (int64_t(1) << 31) / kAlign;
static_assert((kItPairBlocks + 2 * kItMaxPairs / kItThreads + 1) * kItThreads < int64_t(1) << 32, "one launch");

// The tables of a layout from its pairs' runs: the first pair_blocks
// workgroups, one wavefront per pair, write the work items (runs of at most
// `tile` matches) {pair, start, count, 1 for a stopped scene}; the others, one
// thread each, the camera entries {2n + side, first item, end item, other
// camera}.  12,000 items and 21,000 entries: 4.7 us; the host, which wrote
// and copied them before, kept the device waiting (30 million matches loaded
// and a first round begun, three layouts: 3.48 -> 3.20 ms).
__global__ __launch_bounds__(kItThreads) void k_items(
    int P, int pair_blocks, int tile, const int32_t* __restrict__ first, const int32_t* __restrict__ start,
    const int32_t* __restrict__ len, const int32_t* __restrict__ pair_scene, const int32_t* __restrict__ done,
    int4* __restrict__ items, const int32_t* __restrict__ cam_code, const int32_t* __restrict__ pair_i,
    const int32_t* __restrict__ pair_j, int4* __restrict__ cam_ent) {
  if ((int)blockIdx.x < pair_blocks) {
    constexpr int kWaves = kItThreads / 64;
    for (int n = blockIdx.x * kWaves + (threadIdx.x >> 6); n < P; n += pair_blocks * kWaves) {
      const int b = first[n], e = first[n + 1], s = start[n], l = len[n];
      const int flag = done != nullptr && done[pair_scene[n]] != 0 ? 1 : 0;
      for (int it = b + (threadIdx.x & 63); it < e; it += 64) {
        const int at = (it - b) * tile;
        items[it] = make_int4(n, s + at, min(tile, l - at), flag);
      }
    }
    return;
  }
  const int64_t e = ((int64_t)blockIdx.x - pair_blocks) * kItThreads + threadIdx.x;
  if (e >= 2 * (int64_t)P) return;
  const int code = cam_code[e], n = code >> 1;
  cam_ent[e] = make_int4(code, first[n], first[n + 1], (code & 1) ? pair_i[n] : pair_j[n]);
}

// A compaction's new layout from the items' survivor counts, one wavefront
// per pair: the pair's new length, and that rounded up to whole aligned
// groups (whose exclusive scan is where its run starts).
__global__ __launch_bounds__(kItThreads) void k_filter_lengths(int P, const int32_t* __restrict__ first,
                                                               const int32_t* __restrict__ keep,
                                                               int32_t* __restrict__ len, int32_t* __restrict__ off) {
  const int n = blockIdx.x * (kItThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (n >= P) return;
  int s = 0;
  for (int it = first[n] + lane; it < first[n + 1]; it += 64) s += keep[it];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m);
  if (lane == 0) {
    len[n] = s;
    off[n] = (s + kAlign - 1) / kAlign * kAlign;
  }
}

// Where each item's first survivor goes, and, for a pair's last item, the
// aligned end of its run, up to which it clears the padding (-1: not the
// last).
__global__ __launch_bounds__(kItThreads) void k_filter_offsets(int P, const int32_t* __restrict__ first,
                                                               const int32_t* __restrict__ keep,
                                                               const int32_t* __restrict__ len,
                                                               const int32_t* __restrict__ off,
                                                               int2* __restrict__ base) {
  const int n = blockIdx.x * (kItThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (n >= P) return;
  const int b = first[n], e = first[n + 1];
  int run = off[n];
  const int end = run + (len[n] + kAlign - 1) / kAlign * kAlign;
  for (int k = b; k < e; k += 64) {
    const int it = k + lane;
    const int mine = it < e ? keep[it] : 0;
    const int inc = wave_inclusive_scan(mine);
    if (it < e) base[it] = make_int2(run + inc - mine, it == e - 1 ? end : -1);
    run += __shfl(inc, 63);
  }
}

unsigned pair_waves(int64_t P) { return (unsigned)((P + kItThreads / 64 - 1) / (kItThreads / 64)); }

}  // namespace

// Work items and camera entries of the layout that pair_runs describes;
// flags: items of converged scenes are marked to be skipped by the steps.
hipError_t launch_items(fea_ctx* c, bool flags) {
  const int64_t P = c->P;
  if (P == 0) return hipSuccess;
  const unsigned pair_blocks = (unsigned)std::min<int64_t>(pair_waves(P), kItPairBlocks);
  const int32_t* runs = c->pair_runs.as<int32_t>();
  k_items<<<pair_blocks + (unsigned)((2 * P + kItThreads - 1) / kItThreads), kItThreads, 0, c->stream>>>(
      (int)P, (int)pair_blocks, (int)tile_matches_of(c->tile_cfg), runs, runs + P + 1, runs + 2 * P + 1,
      c->d_pair_scene.as<int32_t>(), flags ? c->d_scene_done.as<int32_t>() : nullptr, c->item_rec.as<int4>(),
      c->d_cam_code.as<int32_t>(), c->d_pair_i.as<int32_t>(), c->d_pair_j.as<int32_t>(), c->d_cam_ent.as<int4>());
  return hipGetLastError();
}

// pair_ws: new lengths [P], new offsets [P], scratch of their scan.
int64_t filter_offsets_ints(int64_t n_pairs) { return 2 * n_pairs + scan_scratch_ints(n_pairs); }

hipError_t launch_filter_lengths(fea_ctx* c) {
  const int64_t P = c->P;
  if (P == 0) return hipSuccess;
  int32_t* ws = c->pair_ws.as<int32_t>();
  k_filter_lengths<<<pair_waves(P), kItThreads, 0, c->stream>>>((int)P, c->pair_runs.as<int32_t>(),
                                                                c->item_keep.as<int32_t>(), ws, ws + P);
  return hipGetLastError();
}

hipError_t launch_filter_offsets(fea_ctx* c) {
  const int64_t P = c->P;
  if (P == 0) return hipSuccess;
  int32_t* ws = c->pair_ws.as<int32_t>();
  const hipError_t e = device_exclusive_scan(ws + P, P, ws + 2 * P, c->stream);
  if (e != hipSuccess) return e;
  k_filter_offsets<<<pair_waves(P), kItThreads, 0, c->stream>>>(
      (int)P, c->pair_runs.as<int32_t>(), c->item_keep.as<int32_t>(), ws, ws + P, c->item_base.as<int2>());
  return hipGetLastError();
}

}  // namespace fea
