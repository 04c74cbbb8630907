// Per-frame culling and ray/primitive intervals for the primitive ray marcher.
//
// Built with -ffp-contract=off and IEEE division/square root: every written
// float operation below is exactly one binary32 operation, so the hit
// decisions and sample intervals are reproducible bit for bit.
//
// Pipeline (one frame, V views of W x H pixels, N primitives):
//   prep       per primitive: world-to-local rows A = diag(1/s) R^T (Sec. 3.1.2:
//              t, R, s are the model-to-world transform), and per view a
//              conservative rectangle of 16x16 screen tiles covering the
//              projected box; counts tile entries.
//   tile_fill  writes each primitive into the culling list of every tile of its
//              rectangle.  These lists take the role of the paper's per-frame
//              BVH (Sec. 3.2.1): a ray only looks at its tile's list.
//   pairs      per ray: slab test against every primitive of the tile's list
//              (staged in LDS), then the fixed-step sample interval [jlo, jhi]
//              inside each hit box.  The resulting per-ray list of
//              (sample interval, list position), sorted by first sample and
//              then primitive id, is the "primitives each ray intersects" and
//              their domain of integration (Sec. 3.2.1); the local ray of a
//              pair is rebuilt from its entry's frame (A, a = A (o - t)) and
//              b = A d.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "internal.h"
#include "pairs.h"

namespace mvp {

// ---------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------

__global__ void k_zero_u32(uint32_t *p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0u;
}

__global__ void k_zero_counters(unsigned long long *c, int first, int n) {
  for (int i = threadIdx.x; i < kCntSlots * n; i += blockDim.x) c[(i / n) * kCntStride + first + i % n] = 0ull;
}
hipError_t launch_zero_counters(unsigned long long *counters, int first, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_counters, dim3(1), dim3(256), 0, s, counters, first, n);
  return hipGetLastError();
}

// Start of a build, in one launch: clear the tile counts and cursors and the
// counters, and bring the cameras from the build's pinned host block.
__global__ __launch_bounds__(256) void k_build_init(uint32_t *tiles, size_t n_tiles, unsigned long long *counters,
                                                    DevCam *cams, const DevCam *host_cams, int n_cams) {
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = i0; i < n_tiles; i += stride) tiles[i] = 0u;
  if (i0 < kCntSlots * kCntStride) counters[i0] = 0ull;
  if (host_cams) {
    constexpr int kWords = sizeof(DevCam) / 4;
    for (size_t i = i0; i < (size_t)n_cams * kWords; i += stride) ((uint32_t *)cams)[i] = ((const uint32_t *)host_cams)[i];
  }
}

static unsigned grid_for(size_t n, unsigned block) {
  size_t g = (n + block - 1) / block;
  if (g > 65535u * 8u) g = 65535u * 8u;
  return (unsigned)(g < 1 ? 1 : g);
}

hipError_t launch_zero_u32(uint32_t *p, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_u32, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_build_init(uint32_t *tiles, size_t n_tiles, unsigned long long *counters, DevCam *cams,
                             const DevCam *host_cams, int n_cams, hipStream_t s) {
  const unsigned g = std::min(1024u, std::max(grid_for(n_tiles, 256), (unsigned)(kCntSlots * kCntStride / 256)));
  hipLaunchKernelGGL(k_build_init, dim3(g), dim3(256), 0, s, tiles, n_tiles, counters, cams, host_cams, n_cams);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// exclusive scan: n counts -> n+1 offsets (the last one is the total)
// ---------------------------------------------------------------------------

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanBlock = kScanThreads * kScanItems;

__device__ inline uint64_t wave_incl_scan(uint64_t v) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    uint64_t o = __shfl_up(v, d, kWave);
    if (lane >= d) v += o;
  }
  return v;
}

// block-wide exclusive scan of one value per thread; returns the prefix, *total the sum
__device__ inline uint64_t block_excl_scan(uint64_t v, uint64_t *total) {
  __shared__ uint64_t s_wave[kScanThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  uint64_t incl = wave_incl_scan(v);
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  uint64_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / kWave; ++w) {
    if (w < wave) base += s_wave[w];
    tot += s_wave[w];
  }
  __syncthreads();
  *total = tot;
  return base + incl - v;
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_block(const T *in, size_t n, uint64_t *out,
                                                             uint64_t *partial) {
  // logical input has n+1 elements, element n reads as 0
  const size_t b0 = (size_t)blockIdx.x * kScanBlock + (size_t)threadIdx.x * kScanItems;
  uint64_t v[kScanItems];
  uint64_t sum = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    size_t idx = b0 + i;
    v[i] = idx < n ? (uint64_t)in[idx] : 0ull;
    sum += v[i];
  }
  uint64_t total;
  uint64_t pre = block_excl_scan(sum, &total);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    size_t idx = b0 + i;
    if (idx <= n) out[idx] = pre;
    pre += v[i];
  }
  if (threadIdx.x == 0 && partial) partial[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_add(uint64_t *out, size_t n1, const uint64_t *base) {
  const uint64_t add = base[blockIdx.x];
  const size_t b0 = (size_t)blockIdx.x * kScanBlock;
  for (int i = threadIdx.x; i < kScanBlock; i += kScanThreads) {
    size_t idx = b0 + i;
    if (idx < n1) out[idx] += add;
  }
}

static size_t scan_blocks(size_t n) { return (n + 1 + kScanBlock - 1) / kScanBlock; }

size_t scan_scratch_bytes(size_t n) {
  size_t bytes = 0;
  size_t nb = scan_blocks(n);
  while (nb > 1) {
    bytes += (2 * nb + 1) * sizeof(uint64_t);
    nb = scan_blocks(nb);
  }
  return bytes + 64;
}

template <typename T>
static hipError_t scan_rec(const T *in, uint64_t *out, size_t n, uint64_t *scratch, hipStream_t s) {
  size_t nb = scan_blocks(n);
  uint64_t *partial = nb > 1 ? scratch : nullptr;
  hipLaunchKernelGGL(k_scan_block<T>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, out, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nb == 1) return e;
  uint64_t *pout = scratch + nb;
  e = scan_rec<uint64_t>(partial, pout, nb, scratch + 2 * nb + 1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kScanThreads), 0, s, out, n + 1, pout);
  return hipGetLastError();
}

// Small scans in one workgroup of 1024 threads: each thread takes a
// contiguous run of the n+1 inputs (its loads in flight together), the run
// sums are scanned across the workgroup, then each thread reads its run again
// and writes its prefixes.  One launch instead of the three of the
// block-recursive scan; used up to 8 inputs per thread, beyond which the one
// workgroup's uncoalesced reads make it the slower of the two.
constexpr int kScanOneThreads = 1024;
constexpr int kScanOneBatch = 8;
constexpr size_t kScanOneMax = (size_t)kScanOneThreads * kScanOneBatch;

__global__ __launch_bounds__(kScanOneThreads) void k_scan_one(const uint32_t *__restrict__ in, size_t n,
                                                              uint64_t *__restrict__ out) {
  __shared__ uint64_t s_wave[kScanOneThreads / kWave];
  const size_t per = (n + 1 + kScanOneThreads - 1) / kScanOneThreads;
  const size_t b = (size_t)threadIdx.x * per, e = min(n + 1, b + per);
  uint64_t sum = 0;
  for (size_t c = b; c < e; c += kScanOneBatch) {
    uint32_t x[kScanOneBatch];
#pragma unroll
    for (int i = 0; i < kScanOneBatch; ++i) x[i] = (c + i < e && c + i < n) ? in[c + i] : 0u;
#pragma unroll
    for (int i = 0; i < kScanOneBatch; ++i) sum += x[i];
  }
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint64_t incl = wave_incl_scan(sum);
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  uint64_t pre = incl - sum;
  for (int w = 0; w < wave; ++w) pre += s_wave[w];
  for (size_t c = b; c < e; c += kScanOneBatch) {
    uint32_t x[kScanOneBatch];
#pragma unroll
    for (int i = 0; i < kScanOneBatch; ++i) x[i] = (c + i < e && c + i < n) ? in[c + i] : 0u;
#pragma unroll
    for (int i = 0; i < kScanOneBatch; ++i) {
      if (c + i < e) out[c + i] = pre;
      pre += x[i];
    }
  }
}

hipError_t launch_scan_u32_u64(const uint32_t *in, uint64_t *out, size_t n, void *scratch, hipStream_t s) {
  if (n + 1 <= kScanOneMax) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanOneThreads), 0, s, in, n, out);
    return hipGetLastError();
  }
  return scan_rec<uint32_t>(in, out, n, (uint64_t *)scratch, s);
}

// ---------------------------------------------------------------------------
// tile offsets: culling-list offsets, pair bases and the sizes, from the counts
// ---------------------------------------------------------------------------

// A tile's pair capacity is its culling-list length times its rays (256, or
// its share of a ray subset), saturated at 32 bits so that a product beyond
// them cannot wrap to a small one.  Up to kScanOneMax tiles one workgroup scans
// lengths and capacities together and writes the sizes (one launch in place of
// four); more tiles take three: sums per block of tiles, their scan, offsets.
__device__ __forceinline__ uint64_t tile_capacity(uint32_t len, const uint32_t *rays, size_t t) {
  const uint64_t c = (uint64_t)len * (rays ? rays[t] : (uint32_t)kTileThreads);
  return c > 0xffffffffull ? 0xffffffffull : c;   // integer compare (no FP64 on the device)
}

// the build's sizes, for the host: entries, capacity, ray-subset flags, the two
// statistics of the boxes (kCntSizes + 3, + 4, from k_prep) and the tiles with entries
__device__ __forceinline__ void write_sizes(uint64_t *out, uint64_t entries, uint64_t capacity, uint64_t full,
                                            const uint32_t *flag, const unsigned long long *counters) {
  out[0] = entries;
  out[1] = capacity;
  out[2] = flag ? (uint64_t)*flag : 0ull;
  out[3] = counters[kCntSizes + 3];
  out[4] = counters[kCntSizes + 4];
  out[5] = full;
  __threadfence_system();   // out may be pinned host memory
}

// exclusive scan of two values per thread over a workgroup of W waves
template <int W>
__device__ inline void block_scan2(uint64_t &a, uint64_t &b, uint64_t &ta, uint64_t &tb) {
  __shared__ uint64_t s_a[W], s_b[W];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint64_t ia = wave_incl_scan(a), ib = wave_incl_scan(b);
  __syncthreads();
  if (lane == kWave - 1) {
    s_a[wave] = ia;
    s_b[wave] = ib;
  }
  __syncthreads();
  uint64_t pa = 0, pb = 0;
  ta = tb = 0;
  for (int w = 0; w < W; ++w) {
    if (w < wave) {
      pa += s_a[w];
      pb += s_b[w];
    }
    ta += s_a[w];
    tb += s_b[w];
  }
  a = pa + ia - a;
  b = pb + ib - b;
}

__global__ __launch_bounds__(kScanOneThreads) void k_tile_offsets_one(const uint32_t *__restrict__ cnt,
                                                                      const uint32_t *__restrict__ rays, size_t n,
                                                                      uint64_t *__restrict__ off, uint64_t *__restrict__ base,
                                                                      const uint32_t *__restrict__ flag,
                                                                      const unsigned long long *__restrict__ counters,
                                                                      uint64_t *sizes) {
  __shared__ uint32_t s_full;
  if (threadIdx.x == 0) s_full = 0;
  __syncthreads();
  const size_t t0 = (size_t)threadIdx.x * kScanOneBatch;
  uint32_t len[kScanOneBatch], full = 0;
  uint64_t cap[kScanOneBatch], a = 0, b = 0;
#pragma unroll
  for (int i = 0; i < kScanOneBatch; ++i) {
    len[i] = t0 + i < n ? cnt[t0 + i] : 0u;
    cap[i] = t0 + i < n ? tile_capacity(len[i], rays, t0 + i) : 0ull;
    a += len[i];
    b += cap[i];
    full += (uint32_t)__popcll(__ballot(len[i] != 0));
  }
  if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&s_full, full);
  uint64_t ta, tb;
  block_scan2<kScanOneThreads / kWave>(a, b, ta, tb);   // (its barriers order s_full)
#pragma unroll
  for (int i = 0; i < kScanOneBatch; ++i) {
    if (t0 + i < n) {
      off[t0 + i] = a;
      base[t0 + i] = b;
    }
    a += len[i];
    b += cap[i];
  }
  if (threadIdx.x == 0) {
    off[n] = ta;
    base[n] = tb;
    write_sizes(sizes, ta, tb, s_full, flag, counters);
  }
}

// WRITE == false: part[2 b], part[2 b + 1] = the sums of block b; true: the
// block's offsets from its scanned sums.
template <bool WRITE>
__global__ __launch_bounds__(kScanThreads) void k_tile_offsets(const uint32_t *__restrict__ cnt,
                                                               const uint32_t *__restrict__ rays, size_t n,
                                                               uint64_t *__restrict__ part, uint64_t *__restrict__ off,
                                                               uint64_t *__restrict__ base,
                                                               unsigned long long *__restrict__ counters) {
  const size_t t0 = (size_t)blockIdx.x * kScanBlock + (size_t)threadIdx.x * kScanItems;
  uint32_t len[kScanItems], full = 0;
  uint64_t cap[kScanItems], a = 0, b = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    len[i] = t0 + i < n ? cnt[t0 + i] : 0u;
    cap[i] = t0 + i < n ? tile_capacity(len[i], rays, t0 + i) : 0ull;
    a += len[i];
    b += cap[i];
    full += (uint32_t)__popcll(__ballot(len[i] != 0));
  }
  uint64_t ta, tb;
  block_scan2<kScanThreads / kWave>(a, b, ta, tb);
  if (!WRITE) {
    if (threadIdx.x == 0) {
      part[2 * blockIdx.x] = ta;
      part[2 * blockIdx.x + 1] = tb;
    }
    if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&counters[kCntTiles], (unsigned long long)full);
    return;
  }
  a += part[2 * blockIdx.x];
  b += part[2 * blockIdx.x + 1];
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (t0 + i < n) {
      off[t0 + i] = a;
      base[t0 + i] = b;
    }
    a += len[i];
    b += cap[i];
  }
}

__global__ __launch_bounds__(kScanOneThreads) void k_tile_offsets_parts(uint64_t *__restrict__ part, size_t nb, size_t n,
                                                                        uint64_t *__restrict__ off,
                                                                        uint64_t *__restrict__ base,
                                                                        const uint32_t *__restrict__ flag,
                                                                        const unsigned long long *__restrict__ counters,
                                                                        uint64_t *sizes) {
  const size_t per = (nb + kScanOneThreads - 1) / kScanOneThreads;
  const size_t p0 = (size_t)threadIdx.x * per, p1 = min(nb, p0 + per);
  uint64_t a = 0, b = 0;
  for (size_t p = p0; p < p1; ++p) {
    a += part[2 * p];
    b += part[2 * p + 1];
  }
  uint64_t ta, tb;
  block_scan2<kScanOneThreads / kWave>(a, b, ta, tb);
  for (size_t p = p0; p < p1; ++p) {
    const uint64_t x = part[2 * p], y = part[2 * p + 1];
    part[2 * p] = a;
    part[2 * p + 1] = b;
    a += x;
    b += y;
  }
  if (threadIdx.x == 0) {
    off[n] = ta;
    base[n] = tb;
    write_sizes(sizes, ta, tb, counters[kCntTiles], flag, counters);
  }
}

size_t tile_offsets_scratch_bytes(size_t ntile) { return (ntile / kScanBlock + 1) * 2 * sizeof(uint64_t); }

hipError_t launch_tile_offsets(const uint32_t *cnt, const uint32_t *rays, size_t n, uint64_t *off, uint64_t *base,
                               const uint32_t *flag, unsigned long long *counters, uint64_t *sizes, void *scratch,
                               hipStream_t s) {
  if (n <= kScanOneMax) {
    hipLaunchKernelGGL(k_tile_offsets_one, dim3(1), dim3(kScanOneThreads), 0, s, cnt, rays, n, off, base, flag, counters,
                       sizes);
    return hipGetLastError();
  }
  const size_t nb = (n + kScanBlock - 1) / kScanBlock;
  uint64_t *part = (uint64_t *)scratch;
  hipLaunchKernelGGL(k_tile_offsets<false>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, cnt, rays, n, part, off, base, counters);
  hipLaunchKernelGGL(k_tile_offsets_parts, dim3(1), dim3(kScanOneThreads), 0, s, part, nb, n, off, base, flag, counters,
                     sizes);
  hipLaunchKernelGGL(k_tile_offsets<true>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, cnt, rays, n, part, off, base, counters);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// prep: local frames and conservative screen rectangles
// ---------------------------------------------------------------------------

// A workgroup takes 64 primitives, one per lane, and its four waves the views
// in turn; the tiles of each rectangle are then counted by the whole wave,
// rectangle after rectangle (a lane per rectangle left the launch waiting for
// the largest one: 48 us for 4096 primitives in 4 views).
constexpr int kPrepWaves = 4;

__global__ __launch_bounds__(kPrepWaves *kWave) void k_prep(int N, const float *__restrict__ pos,
                                              const float *__restrict__ rot,
                                              const float *__restrict__ scale, AccelView av,
                                              float4 *__restrict__ xf, int4 *__restrict__ rect,
                                              uint32_t *__restrict__ depth, uint32_t *__restrict__ tile_cnt,
                                              unsigned long long *__restrict__ counters) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int k0 = blockIdx.x * kWave + lane;
  const bool live = k0 < N;
  const int k = live ? k0 : N - 1;   // the lanes past the end work on the last primitive and write nothing
  float inv_s = 0.f, far_s = 0.f;    // the largest 1 / s and distance / s over the boxes (for the backward)
  float R[9], s[3], t[3];
#pragma unroll
  for (int i = 0; i < 9; ++i) R[i] = rot[9 * (size_t)k + i];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    s[i] = scale[3 * (size_t)k + i];
    t[i] = pos[3 * (size_t)k + i];
  }
  float A[9];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    float is = 1.0f / s[i];
#pragma unroll
    for (int j = 0; j < 3; ++j) A[3 * i + j] = R[3 * j + i] * is;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (live && wave == 0) xf[3 * (size_t)k + i] = make_float4(A[3 * i], A[3 * i + 1], A[3 * i + 2], t[i]);
  inv_s = 1.0f / fminf(s[0], fminf(s[1], s[2]));

  // half-extent axes of the box in world space: h_j = s_j R[:, j]
  float h[3][3];
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int m = 0; m < 3; ++m) h[j][m] = R[3 * m + j] * s[j];

  const int T = av.tiles_x * av.tiles_y;
  for (int v = wave; v < av.V; v += kPrepWaves) {
    const DevCam &c = av.cams[v];
    // homogeneous pixel coordinates w = Pinv (x - o) of the centre and axes
    float rel[3] = {t[0] - c.o[0], t[1] - c.o[1], t[2] - c.o[2]};
    float wc[3], wh[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      wc[i] = c.Pinv[3 * i] * rel[0] + c.Pinv[3 * i + 1] * rel[1] + c.Pinv[3 * i + 2] * rel[2];
#pragma unroll
      for (int j = 0; j < 3; ++j)
        wh[j][i] = c.Pinv[3 * i] * h[j][0] + c.Pinv[3 * i + 1] * h[j][1] + c.Pinv[3 * i + 2] * h[j][2];
    }
    float zmin = INFINITY, zmax = -INFINITY, mag = fabsf(wc[2]);
    float umin = INFINITY, umax = -INFINITY, vmin = INFINITY, vmax = -INFINITY;
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) {
      const float sx = (cc & 1) ? 1.0f : -1.0f, sy = (cc & 2) ? 1.0f : -1.0f, sz = (cc & 4) ? 1.0f : -1.0f;
      float w0 = wc[0] + sx * wh[0][0] + sy * wh[1][0] + sz * wh[2][0];
      float w1 = wc[1] + sx * wh[0][1] + sy * wh[1][1] + sz * wh[2][1];
      float w2 = wc[2] + sx * wh[0][2] + sy * wh[1][2] + sz * wh[2][2];
      zmin = fminf(zmin, w2);
      zmax = fmaxf(zmax, w2);
      mag = fmaxf(mag, fabsf(w0) + fabsf(w1) + fabsf(w2));
      float iw = 1.0f / w2;
      umin = fminf(umin, w0 * iw);
      umax = fmaxf(umax, w0 * iw);
      vmin = fminf(vmin, w1 * iw);
      vmax = fmaxf(vmax, w1 * iw);
    }
    int4 r;
    const float eps = 1e-4f * mag;
    if (zmax < -eps) {
      r = make_int4(1, 1, 0, 0);                       // entirely behind the camera
    } else if (zmin <= eps) {
      r = make_int4(0, 0, av.tiles_x - 1, av.tiles_y - 1);  // straddles the camera plane
    } else {
      // pixels whose centre lies within the projected box, plus a margin
      const float lim = 1e7f;
      umin = fmaxf(umin, -lim); umax = fminf(umax, lim);
      vmin = fmaxf(vmin, -lim); vmax = fminf(vmax, lim);
      int px0 = (int)floorf(umin - 2.0f), px1 = (int)ceilf(umax + 1.0f);
      int py0 = (int)floorf(vmin - 2.0f), py1 = (int)ceilf(vmax + 1.0f);
      px0 = max(px0, 0); py0 = max(py0, 0);
      px1 = min(px1, av.W - 1); py1 = min(py1, av.H - 1);
      if (px0 > px1 || py0 > py1) r = make_int4(1, 1, 0, 0);
      else r = make_int4(px0 / kTile, py0 / kTile, px1 / kTile, py1 / kTile);
    }
    if (!live) r = make_int4(1, 1, 0, 0);
    if (live) rect[(size_t)v * N + k] = r;
    // order key of the box along the rays of this view: its distance from the
    // camera less its half diagonal (a lower bound of where rays enter it),
    // as float bits mapped to an unsigned order
    const float dist = sqrtf(rel[0] * rel[0] + rel[1] * rel[1] + rel[2] * rel[2]);
    const float dk = dist - sqrtf(s[0] * s[0] + s[1] * s[1] + s[2] * s[2]);
    const uint32_t bits = __float_as_uint(dk);
    if (live) depth[(size_t)v * N + k] = (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
    far_s = fmaxf(far_s, dist * inv_s);
    for (int q = 0; q < kWave; ++q) {
      const int x0 = __builtin_amdgcn_readlane(r.x, q), y0 = __builtin_amdgcn_readlane(r.y, q);
      const int w = __builtin_amdgcn_readlane(r.z, q) - x0 + 1, h = __builtin_amdgcn_readlane(r.w, q) - y0 + 1;
      if (w <= 0 || h <= 0) continue;
      for (int i = lane; i < w * h; i += kWave)
        atomicAdd(&tile_cnt[(size_t)v * T + (size_t)(y0 + i / w) * av.tiles_x + x0 + i % w], 1u);
    }
  }
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    inv_s = fmaxf(inv_s, __shfl_xor(inv_s, d, kWave));
    far_s = fmaxf(far_s, __shfl_xor(far_s, d, kWave));
  }
  if (lane == 0) {   // non-negative floats order like their bits
    if (far_s > 0.f) atomicMax(&counters[kCntSizes + 3], (unsigned long long)__float_as_uint(far_s));
    if (wave == 0) atomicMax(&counters[kCntSizes + 4], (unsigned long long)__float_as_uint(inv_s));
  }
}

hipError_t launch_prep(const mvp_prims &p, const AccelView &av, float4 *xf, int4 *rect, uint32_t *depth,
                       uint32_t *tile_cnt, unsigned long long *counters, hipStream_t s) {
  if (p.n_prim == 0) return hipSuccess;
  hipLaunchKernelGGL(k_prep, dim3((p.n_prim + kWave - 1) / kWave), dim3(kPrepWaves *kWave), 0, s, p.n_prim, p.pos, p.rot,
                     p.scale, av, xf, rect, depth, tile_cnt, counters);
  return hipGetLastError();
}

// Each primitive's id into the culling list of every tile of its rectangles.  A
// wave takes kFillRects rectangles, its lanes their tiles, and asks for the
// slots of all of them before it stores (a lane per rectangle took one atomic
// after another: 131 us for 2048 primitives at 1920 x 1080, 267 us for 64 large
// ones).
constexpr int kFillRects = 4;

__global__ __launch_bounds__(256) void k_tile_fill(AccelView av, const int4 *__restrict__ rect,
                                                   uint32_t *__restrict__ cursor,
                                                   uint32_t *__restrict__ list) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t wv = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const int64_t i0 = wv * kFillRects, n = (int64_t)av.V * av.N;
  const int T = av.tiles_x * av.tiles_y;
  int4 r[kFillRects];
  int area[kFillRects], most = 0;
#pragma unroll
  for (int q = 0; q < kFillRects; ++q) {
    r[q] = i0 + q < n ? rect[i0 + q] : make_int4(1, 1, 0, 0);
    area[q] = r[q].x <= r[q].z && r[q].y <= r[q].w ? (r[q].z - r[q].x + 1) * (r[q].w - r[q].y + 1) : 0;
    most = max(most, area[q]);
  }
  for (int t = lane; t < most; t += kWave) {
    size_t tile[kFillRects];
    uint32_t slot[kFillRects];
#pragma unroll
    for (int q = 0; q < kFillRects; ++q) {
      if (t >= area[q]) continue;
      const int w = r[q].z - r[q].x + 1;
      tile[q] = (size_t)((i0 + q) / av.N) * T + (size_t)(r[q].y + t / w) * av.tiles_x + r[q].x + t % w;
      slot[q] = atomicAdd(&cursor[tile[q]], 1u);
    }
#pragma unroll
    for (int q = 0; q < kFillRects; ++q)
      if (t < area[q]) list[av.tile_off[tile[q]] + slot[q]] = (uint32_t)((i0 + q) % av.N);
  }
}

hipError_t launch_tile_fill(const AccelView &av, const int4 *rect, uint32_t *cursor,
                            uint32_t *tile_list, hipStream_t s) {
  const size_t n = (size_t)av.V * av.N;
  if (n == 0) return hipSuccess;
  const size_t waves = (n + kFillRects - 1) / kFillRects;
  hipLaunchKernelGGL(k_tile_fill, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, av, rect, cursor, tile_list);
  return hipGetLastError();
}

// Transposed lists without atomics: the entries of primitive k come from the
// tiles of its screen rectangles, view by view and row by row, so the place of
// entry g (tile (v, tx, ty), primitive k) in k's list follows from the
// rectangles alone and the lists come out ascending in g.
__global__ __launch_bounds__(256) void k_prim_entry_place(AccelView av, const int4 *__restrict__ rect, uint64_t n,
                                                          const uint64_t *__restrict__ off,
                                                          uint32_t *__restrict__ out) {
  const int T = av.tiles_x * av.tiles_y;
  uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (; g < n; g += stride) {
    // tile of entry g: last tile t with tile_off[t] <= g
    int lo = 0, hi = av.V * T - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (av.tile_off[mid] <= g) lo = mid; else hi = mid - 1;
    }
    const int v = lo / T, tt = lo - v * T, tx = tt % av.tiles_x, ty = tt / av.tiles_x;
    const uint32_t k = av.tile_list[g];
    uint64_t p = 0;
    for (int w = 0; w < v; ++w) {
      const int4 r = rect[(size_t)w * av.N + k];
      if (r.x <= r.z && r.y <= r.w) p += (uint64_t)(r.z - r.x + 1) * (uint64_t)(r.w - r.y + 1);
    }
    const int4 r = rect[(size_t)v * av.N + k];
    p += (uint64_t)(ty - r.y) * (uint64_t)(r.z - r.x + 1) + (uint64_t)(tx - r.x);
    out[off[k] + p] = (uint32_t)g;
  }
}

// Work items of the p-th primitive in the backward's order (prim[p]; the
// identity when prim is null).
__global__ __launch_bounds__(256) void k_item_count(const uint64_t *__restrict__ off, const uint32_t *__restrict__ prim,
                                                    int n, int per_item, uint32_t *__restrict__ cnt) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const int k = prim ? (int)prim[p] : p;
  cnt[p] = (uint32_t)((off[k + 1] - off[k] + per_item - 1) / per_item);
}

// The backward's order of the primitives: by screen position, so that
// consecutive work items read the per-ray data of neighbouring rays.  A
// primitive's key is the Morton code (6 bits a side) of the centre of its tile
// rectangle in the first view that sees it (the last key if none does); the
// primitives are counted into the kPrimBuckets keys, and scattered by key.
// The order within a key follows the atomics and carries no meaning: the
// order only schedules the work items.  Also the primitive's culling-list
// entries: the area of its rectangles.
__device__ __forceinline__ uint32_t prim_key(const int4 *__restrict__ rect, int k, int N, int V, int tiles_x,
                                             int tiles_y, uint32_t *entries) {
  uint32_t kk = kPrimBuckets - 1, n = 0;
  bool seen = false;
  for (int v = 0; v < V; ++v) {
    const int4 r = rect[(size_t)v * N + k];
    if (r.x <= r.z && r.y <= r.w) {
      n += (uint32_t)(r.z - r.x + 1) * (uint32_t)(r.w - r.y + 1);
      if (seen) continue;
      seen = true;
      const uint32_t cx = (uint32_t)min(63, (int)(((int64_t)r.x + r.z) * 32 / max(tiles_x, 1)));
      const uint32_t cy = (uint32_t)min(63, (int)(((int64_t)r.y + r.w) * 32 / max(tiles_y, 1)));
      kk = 0;
      for (int b = 0; b < 6; ++b) kk |= (((cx >> b) & 1u) << (2 * b)) | (((cy >> b) & 1u) << (2 * b + 1));
    }
  }
  *entries = n;
  return kk;
}

__global__ __launch_bounds__(256) void k_prim_key(const int4 *__restrict__ rect, int N, int V, int tiles_x,
                                                  int tiles_y, uint32_t *__restrict__ key, uint32_t *__restrict__ cnt,
                                                  uint32_t *__restrict__ entries) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= N) return;
  uint32_t n;
  const uint32_t kk = prim_key(rect, k, N, V, tiles_x, tiles_y, &n);
  key[k] = kk;
  entries[k] = n;
  atomicAdd(&cnt[kk], 1u);
}

// All of it in one workgroup for up to kScanOneMax primitives: entry offsets,
// order, work-item offsets (one launch in place of nine).
__global__ __launch_bounds__(kScanOneThreads) void k_prim_lists_one(const int4 *__restrict__ rect, int N, int V, int tiles_x,
                                                                    int tiles_y, int per_item,
                                                                    uint64_t *__restrict__ entry_off,
                                                                    uint32_t *__restrict__ prim,
                                                                    uint64_t *__restrict__ item_off) {
  __shared__ uint32_t s_hist[kPrimBuckets];
  __shared__ uint32_t s_items[kScanOneMax];
  for (int i = threadIdx.x; i < kPrimBuckets; i += kScanOneThreads) s_hist[i] = 0u;
  __syncthreads();
  const int k0 = threadIdx.x * kScanOneBatch;
  uint32_t n[kScanOneBatch], key[kScanOneBatch];
  uint64_t a = 0, b = 0, ta, tb;
#pragma unroll
  for (int i = 0; i < kScanOneBatch; ++i) {
    n[i] = 0;
    key[i] = 0;
    if (k0 + i < N) {
      key[i] = prim_key(rect, k0 + i, N, V, tiles_x, tiles_y, &n[i]);
      atomicAdd(&s_hist[key[i]], 1u);
    }
    a += n[i];
  }
  __syncthreads();
  constexpr int kPer = kPrimBuckets / kScanOneThreads;
  uint32_t h[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    h[i] = s_hist[threadIdx.x * kPer + i];
    b += h[i];
  }
  block_scan2<kScanOneThreads / kWave>(a, b, ta, tb);
#pragma unroll
  for (int i = 0; i < kPer; ++i) {   // (each thread writes the buckets it read)
    s_hist[threadIdx.x * kPer + i] = (uint32_t)b;
    b += h[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kScanOneBatch; ++i) {
    if (k0 + i < N) {
      entry_off[k0 + i] = a;
      const uint32_t p = atomicAdd(&s_hist[key[i]], 1u);
      prim[p] = (uint32_t)(k0 + i);
      s_items[p] = (n[i] + per_item - 1) / per_item;
    }
    a += n[i];
  }
  if (threadIdx.x == 0) entry_off[N] = ta;
  __syncthreads();
  a = b = 0;
#pragma unroll
  for (int i = 0; i < kScanOneBatch; ++i) {
    n[i] = k0 + i < N ? s_items[k0 + i] : 0u;
    a += n[i];
  }
  block_scan2<kScanOneThreads / kWave>(a, b, ta, tb);
#pragma unroll
  for (int i = 0; i < kScanOneBatch; ++i) {
    if (k0 + i < N) item_off[k0 + i] = a;
    a += n[i];
  }
  if (threadIdx.x == 0) item_off[N] = ta;
}

__global__ __launch_bounds__(256) void k_prim_scatter(const uint32_t *__restrict__ key, int N,
                                                      unsigned long long *__restrict__ boff,
                                                      uint32_t *__restrict__ prim) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < N) prim[atomicAdd(&boff[key[k]], 1ull)] = (uint32_t)k;
}

hipError_t launch_prim_lists(const AccelView &av, const int4 *rect, uint64_t n_entries, uint32_t *cnt, uint32_t *key,
                             uint32_t *bcnt, uint64_t *boff, void *scan_scratch, uint64_t *entry_off, uint32_t *entries,
                             uint32_t *prim, uint64_t *item_off, hipStream_t s) {
  const int N = av.N;
  hipError_t e = hipSuccess;
  const dim3 pg((unsigned)((N + 255) / 256));
  if ((size_t)N <= kScanOneMax) {
    hipLaunchKernelGGL(k_prim_lists_one, dim3(1), dim3(kScanOneThreads), 0, s, rect, N, av.V, av.tiles_x, av.tiles_y,
                       av.item_entries, entry_off, prim, item_off);
  } else {
    e = launch_zero_u32(bcnt, kPrimBuckets, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_prim_key, pg, dim3(256), 0, s, rect, N, av.V, av.tiles_x, av.tiles_y, key, bcnt, cnt);
    e = launch_scan_u32_u64(cnt, entry_off, N, scan_scratch, s);
    if (e != hipSuccess) return e;
    e = launch_scan_u32_u64(bcnt, boff, kPrimBuckets, scan_scratch, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_prim_scatter, pg, dim3(256), 0, s, key, N, (unsigned long long *)boff, prim);
    hipLaunchKernelGGL(k_item_count, pg, dim3(256), 0, s, entry_off, prim, N, av.item_entries, cnt);
    e = launch_scan_u32_u64(cnt, item_off, N, scan_scratch, s);
    if (e != hipSuccess) return e;
  }
  if (n_entries)
    hipLaunchKernelGGL(k_prim_entry_place, dim3(grid_for(n_entries, 256)), dim3(256), 0, s, av, rect, n_entries, entry_off,
                       entries);
  return hipGetLastError();
}

// Sort segments [off[i], off[i+1]) of 32-bit values ascending: plain values
// (depth == nullptr), or culling-list entries (primitive ids) of segment =
// tile i by (depth[v N + id], id) with v = i / tiles_per_view, so that each
// tile's list runs from near to far and a ray meets its primitives nearly in
// the order of their first samples; ties and the order itself are
// independent of the order of the fill atomics.  Bitonic sort in LDS;
// segments longer than kSortMax are sorted by the same network in device
// memory.
constexpr int kSortMax = 4096;

__device__ __forceinline__ uint64_t sort_key(uint32_t x, const uint32_t *depth, uint64_t vN) {
  return depth ? ((uint64_t)depth[vN + x] << 32) | x : (uint64_t)x;
}

__global__ __launch_bounds__(256) void k_segment_sort(const uint64_t *__restrict__ off, uint32_t *__restrict__ list,
                                                      const uint32_t *__restrict__ depth, int N, int tiles_per_view) {
  __shared__ uint64_t s[kSortMax];
  const int64_t seg = blockIdx.x;
  const uint64_t b = off[seg];
  const int64_t n = (int64_t)(off[seg + 1] - b);
  if (n < 2) return;
  const uint64_t vN = depth ? (uint64_t)(seg / tiles_per_view) * (uint64_t)N : 0;
  if (n <= kSortMax) {
    int np = 2;
    while (np < n) np <<= 1;
    for (int i = threadIdx.x; i < np; i += blockDim.x) s[i] = i < n ? sort_key(list[b + i], depth, vN) : ~0ull;
    __syncthreads();
    for (int k = 2; k <= np; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = threadIdx.x; i < np; i += blockDim.x) {
          const int ixj = i ^ j;
          if (ixj > i) {
            const uint64_t x = s[i], y = s[ixj];
            const bool up = (i & k) == 0;
            if ((x > y) == up) {
              s[i] = y;
              s[ixj] = x;
            }
          }
        }
        __syncthreads();
      }
    }
    for (int i = threadIdx.x; i < n; i += blockDim.x) list[b + i] = (uint32_t)s[i];
    return;
  }
  // Longer segments: the same sort over the segment in device memory (in place,
  // keys looked up as they are compared), in the form of the bitonic network
  // whose comparators all put the smaller key first, so that the entries past
  // n act as +infinity and never move.  Each stage's comparators are
  // independent, so a thread issues several at once; a barrier separates the
  // stages (the workgroup's writes are visible to it after the barrier).
  uint32_t *a = list + b;
  int64_t np = 2;
  while (np < n) np <<= 1;
  const int64_t half = np >> 1;
  auto cmpx = [&](int64_t i, int64_t q) {
    if (q >= n) return;
    const uint32_t x = a[i], y = a[q];
    if (sort_key(x, depth, vN) > sort_key(y, depth, vN)) {
      a[i] = y;
      a[q] = x;
    }
  };
  for (int64_t k = 2; k <= np; k <<= 1) {
    const int64_t hk = k >> 1;
    for (int64_t c = threadIdx.x; c < half; c += blockDim.x) {   // flip: i against its mirror in the k-block
      const int64_t i = (c / hk) * k + (c % hk);
      cmpx(i, (i / k) * k + (k - 1 - (i % k)));
    }
    __syncthreads();
    for (int64_t j = hk >> 1; j > 0; j >>= 1) {   // half-cleaners
#pragma unroll 4
      for (int64_t c = threadIdx.x; c < half; c += blockDim.x) {
        const int64_t i = (c / j) * 2 * j + (c % j);
        cmpx(i, i + j);
      }
      __syncthreads();
    }
  }
}

hipError_t launch_segment_sort(const uint64_t *off, uint32_t *data, int64_t n_seg, const uint32_t *depth, int N,
                               int tiles_per_view, hipStream_t s) {
  if (n_seg <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_segment_sort, dim3((unsigned)n_seg), dim3(256), 0, s, off, data, depth, N, tiles_per_view);
  return hipGetLastError();
}

// Ray subsets: bin the sampled rays (pixel ids) into screen tiles.
__global__ __launch_bounds__(256) void k_ray_bin(AccelView av, uint32_t *__restrict__ tile_cnt,
                                                 uint32_t *__restrict__ flag) {
  const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= av.n_slots) return;
  const int64_t pix = av.ray_pix[slot];
  if (pix < 0 || pix >= (int64_t)av.V * av.W * av.H) {
    atomicOr(flag, 1u);
    return;
  }
  const int64_t hw = (int64_t)av.W * av.H;
  const int v = (int)(pix / hw);
  const int64_t r = pix - v * hw;
  const int px = (int)(r % av.W), py = (int)(r / av.W);
  const size_t tile = (size_t)v * av.tiles_x * av.tiles_y + (size_t)(py / kTile) * av.tiles_x + px / kTile;
  if (atomicAdd(&tile_cnt[tile], 1u) >= (uint32_t)kTileThreads) atomicOr(flag, 2u);
}

__global__ __launch_bounds__(256) void k_ray_fill(AccelView av, uint32_t *__restrict__ cursor,
                                                  uint32_t *__restrict__ tile_rays) {
  const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= av.n_slots) return;
  const int64_t pix = av.ray_pix[slot];
  if (pix < 0 || pix >= (int64_t)av.V * av.W * av.H) return;
  const int64_t hw = (int64_t)av.W * av.H;
  const int v = (int)(pix / hw);
  const int64_t r = pix - v * hw;
  const int px = (int)(r % av.W), py = (int)(r / av.W);
  const size_t tile = (size_t)v * av.tiles_x * av.tiles_y + (size_t)(py / kTile) * av.tiles_x + px / kTile;
  const uint32_t k = atomicAdd(&cursor[tile], 1u);
  const uint64_t pos = av.tile_ray_off[tile] + k;
  if (pos < av.tile_ray_off[tile + 1]) tile_rays[pos] = (uint32_t)slot;
}

hipError_t launch_ray_bin(const AccelView &av, uint32_t *tile_cnt, uint32_t *flag, hipStream_t s) {
  if (av.n_slots == 0) return hipSuccess;
  hipLaunchKernelGGL(k_ray_bin, dim3((unsigned)((av.n_slots + 255) / 256)), dim3(256), 0, s, av, tile_cnt, flag);
  return hipGetLastError();
}

hipError_t launch_ray_fill(const AccelView &av, uint32_t *cursor, uint32_t *tile_rays, hipStream_t s) {
  if (av.n_slots == 0) return hipSuccess;
  hipLaunchKernelGGL(k_ray_fill, dim3((unsigned)((av.n_slots + 255) / 256)), dim3(256), 0, s, av, cursor, tile_rays);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// per-ray hit lists
// ---------------------------------------------------------------------------

template <bool SUBSET>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(SUBSET ? 4 : 5))) void k_pairs(AccelView av,
                                                                                                PairsOut o) {
  tile_pairs<SUBSET>(av, blockIdx.x, o);
}

hipError_t launch_pairs(const AccelView &av, const PairsOut &o, hipStream_t s) {
  const int ntile = av.V * av.tiles_x * av.tiles_y;
  if (ntile == 0) return hipSuccess;
  if (av.tile_rays)
    hipLaunchKernelGGL((k_pairs<true>), dim3(ntile), dim3(kTileThreads), 0, s, av, o);
  else
    hipLaunchKernelGGL((k_pairs<false>), dim3(ntile), dim3(kTileThreads), 0, s, av, o);
  return hipGetLastError();
}

// Debug hit sets: per ray the number of slab hits against its tile's list
// (with or without samples).
__global__ __launch_bounds__(kTileThreads) void k_hit_count(AccelView av, uint32_t *__restrict__ ray_cnt) {
  __shared__ Staged sm;
  const int tile = blockIdx.x;
  int v, px, py;
  size_t slot;
  const bool valid = tile_ray(av, tile, threadIdx.x, &slot, &v, &px, &py);
  const DevCam &cam = av.cams[v];
  float d[3];
  pixel_ray(cam, px, py, d);
  const uint64_t lb = av.tile_off[tile], le = av.tile_off[tile + 1];
  uint32_t cnt = 0;
  for (uint64_t c0 = lb; c0 < le; c0 += kStage) {
    const int n = (int)min<uint64_t>(kStage, le - c0);
    __syncthreads();
    stage_chunk(sm, av, cam, c0, n);
    __syncthreads();
    for (int e = 0; e < n; ++e) {
      float a[3], b[3], t0, t1;
      local_ray(sm, e, d, a, b);
      cnt += (valid && slab_test(a, b, av.t_near, &t0, &t1)) ? 1u : 0u;
    }
  }
  if (valid) ray_cnt[slot] = cnt;
}

hipError_t launch_hit_count(const AccelView &av, uint32_t *ray_cnt, hipStream_t s) {
  const int ntile = av.V * av.tiles_x * av.tiles_y;
  if (ntile == 0) return hipSuccess;
  hipLaunchKernelGGL(k_hit_count, dim3(ntile), dim3(kTileThreads), 0, s, av, ray_cnt);
  return hipGetLastError();
}

// ... and their primitive ids in increasing order at ids[off[ray] ..] (each
// id inserted into the ray's sorted run as it is found).
__global__ __launch_bounds__(kTileThreads) void k_hit_ids(AccelView av, const uint64_t *__restrict__ off,
                                                           int32_t *__restrict__ ids) {
  __shared__ Staged sm;
  const int tile = blockIdx.x;
  int v, px, py;
  size_t slot;
  const bool valid = tile_ray(av, tile, threadIdx.x, &slot, &v, &px, &py);
  const DevCam &cam = av.cams[v];
  float d[3];
  pixel_ray(cam, px, py, d);
  const uint64_t lb = av.tile_off[tile], le = av.tile_off[tile + 1];
  const uint64_t o0 = valid ? off[slot] : 0;
  uint64_t o = o0;
  for (uint64_t c0 = lb; c0 < le; c0 += kStage) {
    const int n = (int)min<uint64_t>(kStage, le - c0);
    __syncthreads();
    stage_chunk(sm, av, cam, c0, n);
    __syncthreads();
    for (int e = 0; e < n; ++e) {
      float a[3], b[3], t0, t1;
      local_ray(sm, e, d, a, b);
      if (valid && slab_test(a, b, av.t_near, &t0, &t1)) {
        const int32_t id = sm.id[e];
        uint64_t at = o++;
        while (at > o0 && ids[at - 1] > id) {
          ids[at] = ids[at - 1];
          --at;
        }
        ids[at] = id;
      }
    }
  }
}

hipError_t launch_hit_ids(const AccelView &av, const uint64_t *off, int32_t *ids, hipStream_t s) {
  const int ntile = av.V * av.tiles_x * av.tiles_y;
  if (ntile == 0) return hipSuccess;
  hipLaunchKernelGGL(k_hit_ids, dim3(ntile), dim3(kTileThreads), 0, s, av, off, ids);
  return hipGetLastError();
}

}  // namespace mvp
