// Forward and backward ray march through the per-ray primitive lists.
//
// Forward (Sec. 3.2.2): for each sample t_j = j*dt inside at least one
// primitive of the ray's list, every containing primitive is sampled
// trilinearly (Sec. 3.2.1) and the samples are combined by the sum rule
//   sigma_j = sum_k sigma_kj,   C_j = sum_k sigma_kj c_kj
// (the global colour/opacity field), then accumulated with the clamp
//   T + sigma_j dt <= 1 :  T += sigma_j dt,  I += C_j dt
//   otherwise           :  I += C_j (1 - T) / sigma_j,  T = 1   (stop)
// and the march stops once T > 1 - eps_early.  With the sequential combine
// (combine == 1) a sample whose summed step saturates is instead taken one
// primitive at a time in increasing id, each with its own clamp step: the
// primitives before the clamping one k* add sigma_k c_k dt, k* adds
// c_k* (1 - T) and the rest nothing; every other sample is the sum rule.
//
// Backward: the additive rule makes every sample's contribution independent
// of the others except through the clamp, so the backward replays each
// (ray, primitive) pair from the ray's stored final state (last sample j_end
// and, if clamped, T before the clamp) without any per-sample storage:
//   Tdot = dL/dA (unclamped)  or  -g . C_S / sigma_S (clamped at sample S)
//   dL/dsigma_kj = dt (Tdot + g . c_kj),   dL/dc_kj = dt sigma_kj g      (j < S)
//   dL/dsigma_kS = (1 - T_{S-1}) (g . c_kS + Tdot) / sigma_S
//   dL/dc_kS     = (1 - T_{S-1}) (sigma_kS / sigma_S) g
// and for the sequential combine Tdot = -g . c_k*S, the primitives before k*
// at S take the j < S formulas, dL/dc_k*S = (1 - T*) g with T* the opacity
// just before k*, and dL/dsigma_k*S = 0.
// The pairs are replayed by work items, each 16 to 128 culling-list entries
// (screen tile, primitive) of one primitive: channel adjoints go to the 8
// voxel corners with the trilinear weights, formed over a run of samples in one
// cell and then added to an LDS copy of the primitive's gradient (or of a slab
// of it) held in 64-bit fixed point (LDS 64-bit integer atomic adds run about 25
// times faster than FP32 ones on gfx950, and integer sums do not depend on the
// order of the additions), which is added to device memory once per item; the
// pose gradient (through y = A (o + t d - pos)) is reduced over the workgroup.
// The fixed-point scale of an item is chosen from a bound on what any one of its
// pairs can add to one gradient value: every single addend then fits 32 bits (50
// where it is converted in two parts) and no 64-bit sum can overflow.
//
// Built with -ffp-contract=off; fused multiply-adds are written explicitly.
#include <hip/hip_runtime.h>
#include <stdlib.h>

#include <algorithm>
#include <type_traits>
#include <climits>
#include <cmath>

#include "internal.h"
#include "pairs.h"

namespace mvp {

// Largest number of culling-list entries per backward work item of 256 or 512
// threads (the build picks the number per structure, see backward_item_entries),
// the shape of those of sparse rays (64 threads), and how the pairs of an item
// too large for the ordering buffer (below) are dealt to its threads.
constexpr int kItemEntries = 64;
constexpr int kSparseMaxM = 10;   // largest payload for it
constexpr int kSparseThreads = kWave, kSparseEntries = 128, kSparseSort = 1024;   // (the last: pairs it orders)
constexpr bool kChunkedPairs = true;
// Lanes accumulate in cell coordinates mirrored by (lane mod 8), so lanes that
// flush the same cell add to different corners in each instruction.
constexpr bool kRotateFlush = true;
// The pairs of a work item are ordered by their number of samples (longest
// first) and dealt round-robin, so the lanes of a wave replay pairs of about
// the same length together; pairs without samples are dropped.
#ifndef MVP_SORT_PAIRS
#define MVP_SORT_PAIRS 1
#endif
constexpr bool kSortPairs = MVP_SORT_PAIRS;
constexpr int kLenBuckets = 64;

template <bool BF16>
struct Voxels;

template <>
struct Voxels<false> {
  static __device__ __forceinline__ float4 load(const void *p, size_t i) {
    return ((const float4 *)p)[i];
  }
};

template <>
struct Voxels<true> {
  static __device__ __forceinline__ float4 load(const void *p, size_t i) {
    const uint2 w = ((const uint2 *)p)[i];
    return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u),
                       __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u));
  }
};

// Position of sample tau in a primitive's voxel grid (align-corners): index of
// the lower corner of the cell and the fractional offsets.
struct Cell {
  int idx;      // (iz*M + iy)*M + ix of corner (0,0,0)
  int i[3];     // ix, iy, iz of corner (0,0,0)
  float f[3];
};

// Index of voxel (q0, q1, q2), whole numbers below M <= 1024 held as floats.  A
// float holds every step exactly up to M = 256; above (BIG) only the inner
// multiply-add (below 2^20) is, and the index, which reaches 2^30, is formed in
// integers: one conversion more, 0.9% of a march that is bound by the VALU (2048 x
// 12^3 BF16 at 1920 x 1080), so the small ones keep the floats.
constexpr int kFloatIndexM = 256;
template <bool BIG>
__device__ __forceinline__ int voxel_index(float q0, float q1, float q2, int M, float Mf) {
  const float zy = fmaf(q2, Mf, q1);
  if (BIG) return (int)(__umul24((unsigned)zy, (unsigned)M) + (unsigned)q0);
  return (int)fmaf(zy, Mf, q0);
}

template <bool BIG>
__device__ __forceinline__ Cell locate(const float4 &A, const float4 &B, float tau, int M, float hM) {
  const float y[3] = {fmaf(tau, B.x, A.x), fmaf(tau, B.y, A.y), fmaf(tau, B.z, A.z)};
  const float top = (float)(M - 2), Mf = (float)M;
  Cell c;
  float qf[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    // u is in [0, M-1] (fma(-1, hM, hM) is exactly 0), so the lower corner is
    // floor(u), except u = M-1, which belongs to the last cell with offset 1
    const float yc = fminf(fmaxf(y[i], -1.0f), 1.0f);
    const float u = fmaf(yc, hM, hM);
    qf[i] = fminf(floorf(u), top);
    c.i[i] = (int)qf[i];
    c.f[i] = u - qf[i];
  }
  c.idx = voxel_index<BIG>(qf[0], qf[1], qf[2], M, Mf);
  return c;
}


// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------

// Trilinear RGBA from the 8 cached corners of a cell (corner q = dx + 2 dy + 4 dz):
// the 8 corner weights once, then one weighted sum per channel.
__device__ __forceinline__ float4 trilerp(const float4 (&v)[8], const Cell &c) {
  const float fx = c.f[0], fy = c.f[1], fz = c.f[2];
  const float gx = 1.0f - fx, gy = 1.0f - fy, gz = 1.0f - fz;
  const float yz[4] = {gy * gz, fy * gz, gy * fz, fy * fz};
  float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float w = ((q & 1) ? fx : gx) * yz[q >> 1];
    r.x = fmaf(w, v[q].x, r.x);
    r.y = fmaf(w, v[q].y, r.y);
    r.z = fmaf(w, v[q].z, r.z);
    r.w = fmaf(w, v[q].w, r.w);
  }
  return r;
}

template <bool BF16>
__device__ __forceinline__ void load_corners(const void *pay, size_t b0, int M, float4 (&v)[8]) {
  const size_t MM = (size_t)M * M;
  v[0] = Voxels<BF16>::load(pay, b0);
  v[1] = Voxels<BF16>::load(pay, b0 + 1);
  v[2] = Voxels<BF16>::load(pay, b0 + M);
  v[3] = Voxels<BF16>::load(pay, b0 + M + 1);
  v[4] = Voxels<BF16>::load(pay, b0 + MM);
  v[5] = Voxels<BF16>::load(pay, b0 + MM + 1);
  v[6] = Voxels<BF16>::load(pay, b0 + MM + M);
  v[7] = Voxels<BF16>::load(pay, b0 + MM + M + 1);
}

__device__ __forceinline__ int prim_of(const float4 &A) { return __float_as_int(A.w); }

// Opacity fade window of Sec. 3.1.3 at the voxel centres of one axis,
// w(i) = exp(-alpha |x_i|^beta), x_i = -1 + 2i/(M-1); W(ix,iy,iz) = w(ix) w(iy) w(iz).
__device__ __forceinline__ void fill_fade(float *tab, int M, float alpha, float beta) {
  for (int i = threadIdx.x; i < M; i += blockDim.x) {
    const float x = fabsf(-1.0f + 2.0f * (float)i / (float)(M - 1));
    // |x|^beta (beta > 0) as exp2(beta log2 |x|), all in FP32
    const float xb = x > 0.0f ? exp2f(beta * log2f(x)) : 0.0f;
    tab[i] = expf(-alpha * xb);
  }
}

// Window of the 8 corners of a cell (corner q = dx + 2 dy + 4 dz).
__device__ __forceinline__ void corner_fade(const float *tab, const Cell &c, float (&wq)[8]) {
  const float wx[2] = {tab[c.i[0]], tab[c.i[0] + 1]};
  const float wy[2] = {tab[c.i[1]], tab[c.i[1] + 1]};
  const float wz[2] = {tab[c.i[2]], tab[c.i[2] + 1]};
#pragma unroll
  for (int q = 0; q < 8; ++q) wq[q] = wx[q & 1] * wy[(q >> 1) & 1] * wz[q >> 2];
}

// The local ray y(t) = a + t b of the pair formed by a ray of direction d with
// culling-list entry g: b = A d in the build's canonical arithmetic, so sample
// positions and the pair's sample interval come from the same values.  A.w
// holds the primitive id (as int bits).
__device__ __forceinline__ void entry_ray(const AccelView &av, uint64_t g, const float d[3], float4 &A, float4 &B) {
  const float4 f0 = av.ef[3 * g], f1 = av.ef[3 * g + 1], f2 = av.ef[3 * g + 2];
  const int k = (int)av.tile_list[g];
  A = make_float4(f0.w, f1.w, f2.w, __int_as_float(k));
  B = make_float4(row_dot(f0.x, f0.y, f0.z, d), row_dot(f1.x, f1.y, f1.z, d), row_dot(f2.x, f2.y, f2.z, d), 0.f);
}

// Tile of a ray slot.
__device__ __forceinline__ int slot_tile(const AccelView &av, size_t slot) {
  int v, px, py;
  slot_pixel(av, slot, &v, &px, &py);
  return (v * av.tiles_y + py / kTile) * av.tiles_x + px / kTile;
}

// RGBA at tau of the pair with local ray (A, B) (primitive id in A.w):
// trilinear payload of its primitive (opacity times the fade window when FADE).
template <bool BF16, bool FADE>
__device__ __forceinline__ float4 sample_pair(const AccelView &av, const void *pay, const float *fade, const float4 &A,
                                              const float4 &B, float tau) {
  const int M = av.M;
  const float hM = 0.5f * (float)(M - 1);
  const Cell c = locate<true>(A, B, tau, M, hM);
  float4 v[8];
  load_corners<BF16>(pay, (size_t)prim_of(A) * M * M * M + c.idx, M, v);
  if (FADE) {
    float wq[8];
    corner_fade(fade, c, wq);
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q].w *= wq[q];
  }
  return trilerp(v, c);
}

// Accumulated state of one ray.
struct RayState {
  float T, I0, I1, I2, t_prev;
};

// Among the ray's pairs [0, n) (sorted by first sample) that contain sample
// j, the one with the smallest primitive id above `after`; n if none.
__device__ __forceinline__ int next_by_id(const AccelView &av, uint32_t seg, int stride, int n, int j, int after) {
  int best = INT_MAX, bi = n;
  for (int i = 0; i < n; ++i) {
    const int4 r = av.pr[seg + i * stride];
    if (r.x > j) break;
    if (r.y < j) continue;
    if (r.w > after && r.w < best) {
      best = r.w;
      bi = i;
    }
  }
  return bi;
}

// Sequential combine at sample j, whose summed step saturates: the
// primitives containing j in increasing id, each with its own clamp step.
// Returns true to stop.
template <bool BF16, bool FADE>
__device__ bool seq_sample(const AccelView &av, uint64_t lb, const void *pay, const float *fade, uint32_t seg,
                           int stride, int n, const float d[3], int j, RayState &st) {
  const float dt = av.step;
  const float tau = (float)j * dt;
  const float T0 = st.T;
  int last = -1;
  for (int i = next_by_id(av, seg, stride, n, j, last); i < n; i = next_by_id(av, seg, stride, n, j, last)) {
    const int4 r = av.pr[seg + i * stride];
    float4 A, B;
    entry_ray(av, lb + (uint64_t)r.z, d, A, B);
    const float4 s = sample_pair<BF16, FADE>(av, pay, fade, A, B, tau);
    const float Tn = st.T + s.w * dt;
    if (Tn <= 1.0f) {
      st.T = Tn;
      st.I0 = fmaf(s.w * s.x, dt, st.I0);
      st.I1 = fmaf(s.w * s.y, dt, st.I1);
      st.I2 = fmaf(s.w * s.z, dt, st.I2);
    } else {
      const float u = 1.0f - st.T;
      st.I0 = fmaf(s.x, u, st.I0);
      st.I1 = fmaf(s.y, u, st.I1);
      st.I2 = fmaf(s.z, u, st.I2);
      st.t_prev = T0;
      st.T = 1.0f;
      return true;
    }
    last = r.w;
  }
  // rounding kept every per-primitive step at or below 1: an ordinary sample
  return st.T > 1.0f - av.eps;
}

// The forward gives each ray kWin lanes of a wave, one lane per sample of a
// window of kWin consecutive samples: a wave marches 64 / kWin = 8 rays (4 x 2
// pixels).  Every lane evaluates its own sample for each pair of the ray that
// overlaps the window, pair by pair in the list's order, so that a sample's
// sums take the primitives in one fixed order; then the window is composited
// across the ray's lanes.  The pairs of a ray are sorted by (first sample,
// primitive id): a window visits only a run of the list.
//
// Why lanes are samples: with one ray per lane the lanes of a wave change
// voxel cells at different samples, so the corner loads were issued for 8 of
// 64 lanes on average, and a gather costs the L1 at least 16 cycles however
// few lanes it serves (46% of the lanes did work per VALU instruction; 70% do
// now); and a picture gave the chip one wave per 64 rays, each a long serial
// chain (256 waves of 4 for 256 x 256 pixels).  The march is now bound by the
// L1's data return (one 128-byte line per four neighbouring lanes and cycle:
// about 20 cycles per corner load) with FP32 payloads and by the VALU with
// BF16 ones.  8 samples rather than 16: a window of 16 leaves 6% more lanes
// idle at the ends of the pairs and takes more pairs per window.
// Measured (march and pairs kernels together, one ray per lane -> this):
// 512 x 16^3 BF16 at 256^2 1.40 -> 0.26 ms, 4096 x 8^3 FP32 at 1024^2
// 4.15 -> 2.05 ms and four such views 8.0 -> 7.75 ms, 2048 x 12^3 BF16 at
// 1920 x 1080 5.8 -> 4.15 ms, 32768 x 16^3 BF16 at 2 x 2048^2 21.0 -> 13.8 ms,
// 16384 sampled rays of four 1024^2 views 2.6 -> 0.53 ms.
constexpr int kWin = 8;
constexpr int kRaysPerWave = kWave / kWin;
// Pairs staged per ray in LDS: a ring, refilled kBatch at a time (each lane
// takes kBatch / kWin of them), whose slot after the last pair holds a
// sentinel.  A refill waits for device memory twice (the records, then the
// frames they name): 16 pairs at a time beat 8 by 4 to 15%.
constexpr int kRing = 32, kBatch = 16;

// Orders this wave's LDS accesses for its other lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ int dpp(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }
constexpr int kShr1 = 0x111, kXor1 = 0xb1, kXor2 = 0x4e, kMirror8 = 0x141;

// maximum and minimum over the 8 lanes of a ray, in every one of them
__device__ __forceinline__ int max8(int v) {
  v = max(v, dpp<kXor1>(v));
  v = max(v, dpp<kXor2>(v));
  return max(v, dpp<kMirror8>(v));
}
__device__ __forceinline__ int min8(int v) {
  v = min(v, dpp<kXor1>(v));
  v = min(v, dpp<kXor2>(v));
  return min(v, dpp<kMirror8>(v));
}

// The ordinary steps of a window, sample by sample in order: T += x,
// I = fma(c, dt, I), taken by all 8 lanes of a ray alike (the roundings are
// those of a serial loop).  Step k reads lane k of the ray: lane k or k + 8 of
// the row of 16 that two rays share, each with the other ray's banks masked.
// Inline because the compiler does not fold a bank-masked move into the
// arithmetic; the leading wait covers a write of an operand just before.
#define MVP_STEP(K, H)                                                                \
  "v_add_f32_dpp %0, %4, %0 row_newbcast:" #K " row_mask:0xf bank_mask:0x3\n\t"       \
  "v_fmac_f32_dpp %1, %5, %8 row_newbcast:" #K " row_mask:0xf bank_mask:0x3\n\t"      \
  "v_fmac_f32_dpp %2, %6, %8 row_newbcast:" #K " row_mask:0xf bank_mask:0x3\n\t"      \
  "v_fmac_f32_dpp %3, %7, %8 row_newbcast:" #K " row_mask:0xf bank_mask:0x3\n\t"      \
  "v_add_f32_dpp %0, %4, %0 row_newbcast:" #H " row_mask:0xf bank_mask:0xc\n\t"       \
  "v_fmac_f32_dpp %1, %5, %8 row_newbcast:" #H " row_mask:0xf bank_mask:0xc\n\t"      \
  "v_fmac_f32_dpp %2, %6, %8 row_newbcast:" #H " row_mask:0xf bank_mask:0xc\n\t"      \
  "v_fmac_f32_dpp %3, %7, %8 row_newbcast:" #H " row_mask:0xf bank_mask:0xc\n\t"
__device__ __forceinline__ void window_steps(float &T, float &I0, float &I1, float &I2, float x, float c0, float c1,
                                             float c2, float dt) {
  asm("s_nop 1\n\t" MVP_STEP(0, 8) MVP_STEP(1, 9) MVP_STEP(2, 10) MVP_STEP(3, 11) MVP_STEP(4, 12) MVP_STEP(5, 13)
          MVP_STEP(6, 14) MVP_STEP(7, 15)
      : "+v"(T), "+v"(I0), "+v"(I1), "+v"(I2)
      : "v"(x), "v"(c0), "v"(c1), "v"(c2), "v"(dt));
}
#undef MVP_STEP

// The 8 voxel corners of a cell whose corner (0,0,0) is at byte address p.
template <bool BF16>
__device__ __forceinline__ void corners_at(const char *p, size_t row, size_t slice, float4 (&v)[8]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const char *q = p + ((r & 1) ? row : 0) + ((r & 2) ? slice : 0);
    if (BF16) {   // both voxels of an x edge in one load (8-byte aligned)
      typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(8)));
      const u4 w = *(const u4 *)q;
      v[2 * r] = make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u),
                             __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u));
      v[2 * r + 1] = make_float4(__uint_as_float(w.z << 16), __uint_as_float(w.z & 0xffff0000u),
                                 __uint_as_float(w.w << 16), __uint_as_float(w.w & 0xffff0000u));
    } else {
      v[2 * r] = *(const float4 *)q;
      v[2 * r + 1] = *(const float4 *)(q + 16);
    }
  }
}

// The march's schedule over full frames.  Unit u of the launch (one workgroup
// of one wave: larger workgroups hold their slots until their slowest wave
// ends, 4 to 10% slower) runs on XCD u mod 8.  The tiles of a view are cut into
// blocks of kMarchBlock x kMarchBlock (edge blocks padded); blocks are dealt
// to the XCDs in turn, with an offset that moves from turn to turn, so that
// every XCD gets blocks from all over the view (the rays that meet primitives
// usually fill its middle), and an XCD takes the units of one block after
// another, so that its L2 serves a compact patch of the screen at a time.
// Blocks of 2 x 2 tiles against 4 x 4: a 256 x 256 picture 0.21 against 0.36 ms
// (4 x 4 gives each XCD two blocks), 32768 x 16^3 12.6 against 14.5 ms, one
// 1024^2 view of 4096 x 8^3 1.90 against 1.80 ms.
//
// A ray subset's units (8 rays each, in the order of their tiles) go to the XCDs
// in runs of kSubsetRun, likewise dealt in turn: 131072 rays over 16384 tiles of
// 4096 x 8^3 616 against 644 us with neighbours on different XCDs, 16384 rays 412
// against 424.
constexpr int kSubsetRun = 16;
constexpr int kMarchBlock = 2;
constexpr int kUnitW = 4, kUnitH = 2;   // pixels of a unit
constexpr int kUnitsPerTile = kTileThreads / kRaysPerWave;
constexpr int kUnitsPerBlock = kMarchBlock * kMarchBlock * kUnitsPerTile;

__host__ __device__ __forceinline__ int64_t march_units(const AccelView &av) {
  if (av.tile_rays) {   // whole runs for every XCD
    constexpr int64_t turn = kXcd * kSubsetRun * kRaysPerWave;
    return (av.n_slots + turn - 1) / turn * (kXcd * kSubsetRun);
  }
  const int64_t bx = (av.tiles_x + kMarchBlock - 1) / kMarchBlock, by = (av.tiles_y + kMarchBlock - 1) / kMarchBlock;
  const int64_t blocks = bx * by * av.V;
  return (blocks + kXcd - 1) / kXcd * kXcd * kUnitsPerBlock;
}

// Tile and unit within the tile of unit u; false for a padding unit.
__device__ __forceinline__ bool march_tile(const AccelView &av, int64_t u, int *tile, int *sub) {
  const int bx = (av.tiles_x + kMarchBlock - 1) / kMarchBlock, by = (av.tiles_y + kMarchBlock - 1) / kMarchBlock;
  const int x = (int)(u % kXcd);
  const int m = (int)(u / kXcd / kUnitsPerBlock), r = (int)(u / kXcd % kUnitsPerBlock);
  const int blk = m * kXcd + ((x + 3 * m) & (kXcd - 1));
  const int v = blk / (bx * by), b = blk - v * bx * by;
  const int t = r / kUnitsPerTile;
  const int ty = (b / bx) * kMarchBlock + t / kMarchBlock, tx = (b % bx) * kMarchBlock + t % kMarchBlock;
  *sub = r % kUnitsPerTile;
  *tile = (v * av.tiles_y + ty) * av.tiles_x + tx;
  return v < av.V && ty < av.tiles_y && tx < av.tiles_x;
}

// 4 waves per SIMD: 5 spill and crowd the L1 (32768 x 16^3: 23 against 16 ms).
// GENERAL: payloads above 256^3 (voxel_index) and nearly empty pictures (skip), kept
// out of the kernel for the others, which they cost up to 1%.
template <bool BF16, bool FADE, bool SEQ, bool GENERAL>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_march_fwd(
    AccelView av, const char *__restrict__ pay, const float *__restrict__ bg, float4 *__restrict__ rgba,
    mvp_ray_aux *__restrict__ aux, unsigned long long *__restrict__ counters, int64_t n_units, int skip) {
  __shared__ float4 pa[kRing][kRaysPerWave];     // a, first sample (int bits)
  __shared__ float4 pb[kRing][kRaysPerWave];     // b, last sample (int bits)
  __shared__ uint64_t pp[kRing][kRaysPerWave];   // address of the primitive's payload
  extern __shared__ float s_fade[];   // [M] when FADE
  if (FADE) {
    fill_fade(s_fade, av.M, av.fade_alpha, av.fade_beta);
    wave_sync();
  }
  const int lane = threadIdx.x;
  const int w = lane & (kWin - 1), rl = lane / kWin;   // sample of the window, ray of the wave
  const int M = av.M;
  const float hM = 0.5f * (float)(M - 1), top = (float)(M - 2), Mf = (float)M;
  constexpr int kVox = BF16 ? 8 : 16;
  const uint32_t row = (uint32_t)M * kVox, slice = row * (uint32_t)M;   // bytes
  const uint64_t prim_bytes = (uint64_t)slice * (uint64_t)M;
  const float dt = av.step, lim = 1.0f - av.eps;
  uint32_t n_ray = 0, n_prim = 0, n_cell = 0, n_pj = 0;

  // skip: nearly all tiles are empty (see launch_march_fwd).  The wave's units, at
  // most one per lane, are looked at together, and those in empty tiles written eight
  // at a time.
  uint64_t full = ~0ull;
  if (GENERAL && skip) {
    auto unit_tile = [&](int i, int *tile, int *sub) {   // unit i of the wave: 0 no unit, 1 in an empty tile, 2 in another
      const int64_t u = blockIdx.x + (int64_t)i * gridDim.x;
      if (u >= n_units || !march_tile(av, u, tile, sub)) return 0;
      return av.tile_off[*tile] == av.tile_off[*tile + 1] ? 1 : 2;
    };
    int tile, sub;
    const int kind = unit_tile(lane, &tile, &sub);
    full = ballot(kind == 2);
    const uint64_t none = ballot(kind == 1);
    for (int g = 0; g < kWave / kRaysPerWave; ++g) {
      if (!((none >> (g * kRaysPerWave)) & 0xffu)) continue;
      size_t ray;
      int v, px, py;
      if (unit_tile(g * kRaysPerWave + rl, &tile, &sub) != 1) continue;
      constexpr int kAcross = kTile / kUnitW;
      const int x = (sub % kAcross) * kUnitW + (w & 3), y = (sub / kAcross) * kUnitH + (w >> 2);
      if (!tile_ray(av, tile, y * kTile + x, &ray, &v, &px, &py)) continue;
      rgba[ray] = bg ? make_float4(bg[3 * ray], bg[3 * ray + 1], bg[3 * ray + 2], 0.f) : make_float4(0.f, 0.f, 0.f, 0.f);
      if (aux) aux[ray] = mvp_ray_aux{-1, -1.0f};
    }
  }
  for (int64_t u = blockIdx.x; u < n_units; u += gridDim.x) {
    if (GENERAL && skip) {
      const bool take = full & 1;
      full >>= 1;
      if (!take) continue;
    }
    // the ray of this lane's group of kWin lanes
    size_t ray = 0;
    int tile = 0, v = 0, px = 0, py = 0;
    bool valid;
    if (av.tile_rays) {   // ray subset: consecutive entries of the tiles' ray lists
      const int64_t i = u / kXcd, m = i / kSubsetRun;
      const int64_t p = ((m * kXcd + ((u + 3 * m) & (kXcd - 1))) * kSubsetRun + i % kSubsetRun) * kRaysPerWave + rl;
      valid = p < av.n_slots;
      if (valid) {
        ray = av.tile_rays[p];
        slot_pixel(av, ray, &v, &px, &py);
        tile = (v * av.tiles_y + py / kTile) * av.tiles_x + px / kTile;
      }
    } else {
      int sub;
      if (!march_tile(av, u, &tile, &sub)) continue;
      constexpr int kAcross = kTile / kUnitW;
      const int x = (sub % kAcross) * kUnitW + (rl & 3), y = (sub / kAcross) * kUnitH + (rl >> 2);
      valid = tile_ray(av, tile, y * kTile + x, &ray, &v, &px, &py);
    }
    int n = 0, stride = 0;
    uint32_t seg = 0;
    float d[3] = {0.f, 0.f, 1.f};
    if (valid) {
      n = av.ray_nj[ray].x;
      seg = (uint32_t)av.ray_seg[ray];
      stride = tile_ray_count(av, tile);
      pixel_ray(av.cams[v], px, py, d);
    }
    const uint64_t lb = av.tile_off[tile];
    float T = 0.f, t_prev = -1.0f;
    float I0 = 0.f, I1 = 0.f, I2 = 0.f;
    int j_last = -1;                      // the last sample this lane took
    bool act = n > 0;
    int e0 = 0;                // pairs before e0 have ended before the window
    int base = 0, ready = 0;   // pairs [base, ready) are staged; slot `ready` of the ring is the sentinel
    // stage pairs [ready, ready + kBatch) of the ray: kBatch / kWin per lane
    auto stage = [&]() {
      constexpr int kB = kBatch / kWin;
      const int i0 = ready + w;
      int4 r[kB];
#pragma unroll
      for (int b = 0; b < kB; ++b) r[b] = av.pr[seg + (uint32_t)min(i0 + b * kWin, n - 1) * (uint32_t)stride];
      ready = min(n, ready + kBatch);
      base = max(base, ready + 1 - kRing);
#pragma unroll
      for (int b = 0; b < kB; ++b) {
        const int i = i0 + b * kWin, at = i & (kRing - 1);
        float4 A, B;
        entry_ray(av, lb + (uint64_t)r[b].z, d, A, B);
        if (i < n) {
          pp[at][rl] = (uint64_t)(uint32_t)r[b].w * prim_bytes + (uint64_t)pay;
          pa[at][rl] = make_float4(A.x, A.y, A.z, __int_as_float(r[b].x));
          pb[at][rl] = make_float4(B.x, B.y, B.z, __int_as_float(r[b].y));
          ++n_pj;
        }
      }
      if (w == 0) {   // no pair: starts after every window, ends after every window
        pa[ready & (kRing - 1)][rl].w = __int_as_float(INT_MAX);
        pb[ready & (kRing - 1)][rl].w = __int_as_float(INT_MAX);
      }
    };
    wave_sync();   // the ring's last readers (the previous rays) are done
    if (act) stage();
    wave_sync();
    int J = act ? __float_as_int(pa[0][rl].w) : 0;
    while (ballot(act)) {
      // keep the pairs of a window staged ahead: once a ray runs short, every
      // ray of the wave with room is refilled
      if (ballot(act && ready < n && ready - e0 < kWin)) {
        if (act && ready < n && ready - e0 <= kRing - 1 - kBatch) stage();
        wave_sync();
      }
      const int j = J + w, J1 = J + kWin;
      const int j_end = act ? J1 : INT_MIN;
      const float tau = (float)j * dt;
      float as = 0.f, ar = 0.f, ag = 0.f, ab = 0.f;   // the sample's sums over its primitives
      uint32_t cnt = 0;                               // the number of those
      int i = e0;
      while (true) {
        while (true) {
          const int at = i & (kRing - 1);
          const float4 A = pa[at][rl];
          const int jlo = __float_as_int(A.w);
          const bool more = jlo < j_end;
          if (!ballot(more)) break;
          const float4 B = pb[at][rl];
          i += more ? 1 : 0;
          if (more && j >= jlo && j <= __float_as_int(B.w)) {
            const float y0 = fmaf(tau, B.x, A.x), y1 = fmaf(tau, B.y, A.y), y2 = fmaf(tau, B.z, A.z);
            const float u0 = fmaf(__builtin_amdgcn_fmed3f(y0, -1.0f, 1.0f), hM, hM),
                        u1 = fmaf(__builtin_amdgcn_fmed3f(y1, -1.0f, 1.0f), hM, hM),
                        u2 = fmaf(__builtin_amdgcn_fmed3f(y2, -1.0f, 1.0f), hM, hM);
            const float q0 = __builtin_amdgcn_fmed3f(floorf(u0), 0.0f, top),
                        q1 = __builtin_amdgcn_fmed3f(floorf(u1), 0.0f, top),
                        q2 = __builtin_amdgcn_fmed3f(floorf(u2), 0.0f, top);
            Cell c;
            c.f[0] = u0 - q0;
            c.f[1] = u1 - q1;
            c.f[2] = u2 - q2;
            c.idx = voxel_index<GENERAL>(q0, q1, q2, M, Mf);
            float4 vx[8];
            corners_at<BF16>((const char *)(pp[at][rl] + (uint64_t)(uint32_t)c.idx * kVox), row, slice, vx);
            if (FADE) {
              c.i[0] = (int)q0;
              c.i[1] = (int)q1;
              c.i[2] = (int)q2;
              float wq[8];
              corner_fade(s_fade, c, wq);
#pragma unroll
              for (int q = 0; q < 8; ++q) vx[q].w *= wq[q];
            }
            const float4 sv = trilerp(vx, c);
            as += sv.w;
            ar = fmaf(sv.w, sv.x, ar);
            ag = fmaf(sv.w, sv.y, ag);
            ab = fmaf(sv.w, sv.z, ab);
            ++cnt;
          }
        }
        // a ray that ran out of staged pairs within the window
        const bool dry = act && i == ready && ready < n;
        if (!ballot(dry)) break;
        if (dry) stage();
        wave_sync();
      }
      n_cell += cnt;
      // Composite the window's samples in order (a sample outside every
      // primitive adds 0).  Where none of its opacities is negative, a ray stops
      // in this window iff its last sum exceeds the limit.
      const float x = as * dt;
      float Tw = T, J0 = I0, J1c = I1, J2 = I2;
      window_steps(Tw, J0, J1c, J2, x, ar, ag, ab, dt);
      const bool mine = cnt > 0;
      if (!ballot(act && (!(Tw <= lim) || x < 0.f))) {   // no ray of the wave stops here
        T = Tw;
        I0 = J0;
        I1 = J1c;
        I2 = J2;
        n_ray += mine ? 1 : 0;
        n_prim += cnt;
        j_last = mine ? j : j_last;
      } else {
        // A ray's stopping sample is the first whose sum exceeds the limit.  A
        // sample whose summed step saturates under the sequential combine is
        // taken primitive by primitive, and the rest of the window after it.
        int from = 0;   // samples before it are done
        while (true) {
          // the opacity after each sample, on its lane: each step adds the
          // previous lane's sum
          const float xs = w >= from ? x : 0.f;
          const float t0 = T + xs;
          float t = t0;
#pragma unroll
          for (int s = 1; s < kWin; ++s) {
            const float up = dpp<kShr1>(t) + xs;
            t = w == 0 ? t0 : up;
          }
          const int ws = min8(act && w >= from && !(t <= lim) ? w : kWin);
          const int src = (lane & ~(kWin - 1)) | min(ws, kWin - 1);
          const float tw = __shfl(t, src, kWave);          // after the stopping (or the last) sample
          const bool over = ws < kWin && !(tw <= 1.0f);   // it is not an ordinary step
          if (act && mine && w >= from && w <= ws) {
            ++n_ray;
            n_prim += cnt;
            j_last = j;
          }
          // the ordinary steps
          const bool ord = act && w >= from && (w < ws || (w == ws && !over));
          float Tn = T;
          window_steps(Tn, I0, I1, I2, ord ? x : 0.f, ord ? ar : 0.f, ord ? ag : 0.f, ord ? ab : 0.f, dt);
          const float s0 = __shfl(ar, src, kWave), s1 = __shfl(ag, src, kWave), s2 = __shfl(ab, src, kWave),
                      ss = __shfl(as, src, kWave);
          bool again = false;
          if (act) {
            T = Tn;
            if (!over) {
              act = ws == kWin;
            } else if (!SEQ) {
              const float wgt = (1.0f - T) / ss;
              I0 = fmaf(s0, wgt, I0);
              I1 = fmaf(s1, wgt, I1);
              I2 = fmaf(s2, wgt, I2);
              t_prev = T;
              T = 1.0f;
              act = false;
            } else {   // every lane of the ray takes the same walk
              RayState st{T, I0, I1, I2, -1.0f};
              const bool stop = seq_sample<BF16, FADE>(av, lb, pay, s_fade, seg, stride, n, d, J + ws, st);
              const bool nan = tw != tw;   // a NaN density: so is the colour, as under the sum rule
              T = st.T;
              I0 = nan ? tw : st.I0;
              I1 = nan ? tw : st.I1;
              I2 = nan ? tw : st.I2;
              if (stop) {
                t_prev = st.t_prev;
                act = false;
              } else {
                again = ws + 1 < kWin;
              }
            }
          }
          from = again ? ws + 1 : kWin;   // kWin: done with this window
          if (!SEQ || !ballot(again)) break;
        }
      }
      // next window: the first pair that reaches past this one, or the first
      // sample of the next pair (all pairs after e0 start no earlier than e0 does)
      while (true) {
        if (ballot(act && e0 < base)) {   // pushed out by a window over more pairs than the ring holds
          if (act && e0 < base) {
            ready = e0;
            base = e0;
            stage();
          }
          wave_sync();
        }
        const int c = min(e0 + w, ready);
        const bool past = __float_as_int(pb[c & (kRing - 1)][rl].w) >= J1;
        const int f = min8(past ? c : INT_MAX);
        const bool none = f == INT_MAX;        // all kWin pairs have ended
        if (act) e0 = none ? e0 + kWin : f;
        const bool dry = act && !none && e0 == ready;
        if (dry && ready == n) act = false;
        if (ballot(dry && act)) {
          if (dry && act) stage();
          wave_sync();
        } else if (!ballot(act && none)) {
          break;
        }
      }
      J = max(J1, __float_as_int(pa[e0 & (kRing - 1)][rl].w));
    }
    const int j_end = max8(j_last);
    if (valid && w == 0) {
      if (bg) {   // composite over the background: I + (1 - A) B
        const float b = 1.0f - T;
        I0 = fmaf(b, bg[3 * ray], I0);
        I1 = fmaf(b, bg[3 * ray + 1], I1);
        I2 = fmaf(b, bg[3 * ray + 2], I2);
      }
      rgba[ray] = make_float4(I0, I1, I2, T);
      if (aux) aux[ray] = mvp_ray_aux{j_end, t_prev};
    }
  }
  if (counters && ballot(n_pj != 0)) {
    const unsigned long long c[5] = {wave_sum_u64(n_ray), wave_sum_u64(n_prim), wave_sum_u64(n_cell),
                                     wave_sum_u64(n_pj), wave_sum_u64(n_pj)};
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < 5; ++i) atomicAdd(counter_slot(counters) + i, c[i]);
    }
  }
}

hipError_t launch_march_fwd(const AccelView &av, const mvp_prims &p, const float *bg, float *rgba,
                            mvp_ray_aux *aux, unsigned long long *counters, hipStream_t s) {
  const int64_t ntile = (int64_t)av.V * av.tiles_x * av.tiles_y;
  if (ntile == 0 || av.n_slots == 0) return hipSuccess;
  const int64_t units = march_units(av);
  // At least 7 of 8 tiles empty: a wave takes several units (as many as there are
  // tiles for each one with primitives, at most one per lane, and no more than leave
  // every SIMD 4 waves), of which it looks at the tiles together.  One
  // wave per unit takes 0.57 ns of the chip for an empty one: 1.16 ms for a 4096^2
  // picture of a few small primitives, 0.28 ms at 2048^2.
  int64_t per = 1;
  if (!av.tile_rays && av.full_tiles * 8 <= ntile)
    per = std::max<int64_t>(1, std::min<int64_t>({kWave, ntile / std::max<int64_t>(av.full_tiles, 1), units / 4096}));
  const int64_t waves = std::min<int64_t>((units + per - 1) / per, 1 << 22);
  const int grid = (int)((waves + kXcd - 1) / kXcd * kXcd);   // a multiple of kXcd
  const int skip = per > 1 && (units + grid - 1) / grid <= kWave ? 1 : 0;
  const bool fade = av.fade_alpha > 0.f;
  const size_t shm = fade ? (size_t)av.M * sizeof(float) : 0;
  const bool general = skip || av.M > kFloatIndexM;
#define MVP_FWD(B, F, S, G)                                                                               \
  hipLaunchKernelGGL((k_march_fwd<B, F, S, G>), dim3(grid), dim3(kWave), shm, s, av,                    \
                     (const char *)p.payload, bg, (float4 *)rgba, aux, counters, units, skip)
#define MVP_FWD_S(B, F)                                                               \
  do {                                                                                \
    if (av.combine) { if (general) MVP_FWD(B, F, true, true); else MVP_FWD(B, F, true, false); }   \
    else { if (general) MVP_FWD(B, F, false, true); else MVP_FWD(B, F, false, false); }   \
  } while (0)
  if (p.payload_dtype == MVP_BF16) {
    if (fade) MVP_FWD_S(true, true); else MVP_FWD_S(true, false);
  } else {
    if (fade) MVP_FWD_S(false, true); else MVP_FWD_S(false, false);
  }
#undef MVP_FWD_S
#undef MVP_FWD
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------

// Per-ray constants of the adjoint.  Tdot is dL/dA for an unclamped ray and
// -g . C_S/sigma_S for a ray clamped at its last sample S, with the weight
// (1 - T_{S-1}) / sigma_S (recomputed here from the pairs open at S).  For
// the sequential combine the clamping primitive k* is found again by
// replaying the per-primitive steps of S from T_{S-1} with the forward's
// arithmetic; then Tdot = -g . c_k*, the weight is 1 - T* and kstar = k*.
// With a background B the output colour is I + (1 - A) B: the upstream of A
// becomes dL/dA - g . B, and dL/dB = (1 - A) g is accumulated here.
//
// Also the ray's bounds for the fixed-point accumulation (RayBound): a replayed
// sample adds to one gradient value of a corner at most its trilinear weight
// (<= 1) times dL/dsigma_k or dL/dc_k.  Away from the clamp
// |dL/dsigma_k| <= dt (|Tdot| + |g|_1 Cmax) and |dL/dc_k| <= dt sigma_max |g|_inf
// (Cmax, sigma_max: the payload's largest colour and opacity magnitudes; the
// fade window only lowers them); at the clamping sample dL/dsigma_k has the
// weight (1 - T_{S-1}) / sigma_S < dt in place of dt and the colour adjoint is
// at most |g|_inf (sum rule: (1 - T_{S-1}) sigma_k / sigma_S <= 1; sequential:
// 1 - T* <= 1).
// Rays per workgroup of k_bwd_rays (4 per thread).  Only the clamped rays
// (about one in eight on a typical frame) replay a sample; they are gathered
// in LDS first, so that the replay runs on full waves instead of on the few
// lanes of every wave whose ray clamped.
constexpr int kBwdRaysPerBlock = 1024;

template <bool BF16, bool FADE>
__global__ __launch_bounds__(256) void k_bwd_rays(AccelView av, const void *__restrict__ pay,
                                                  const mvp_ray_aux *__restrict__ aux,
                                                  const float4 *__restrict__ grad_rgba,
                                                  const float *__restrict__ bg, const float4 *__restrict__ rgba,
                                                  RayConst *__restrict__ rc, RayBound *__restrict__ rbd,
                                                  const uint32_t *__restrict__ pmax, uint32_t *__restrict__ odd,
                                                  float *__restrict__ g_bg, size_t R) {
  extern __shared__ float s_fade[];
  __shared__ uint32_t s_clamped[kBwdRaysPerBlock];
  __shared__ int s_nc;
  if (threadIdx.x == 0) s_nc = 0;
  if (blockIdx.x == 0 && threadIdx.x < 2) av.item_lists[threadIdx.x] = 0u;   // (for k_item_split)
  if (FADE) fill_fade(s_fade, av.M, av.fade_alpha, av.fade_beta);
  __syncthreads();
  const float cmax = __uint_as_float(pmax[0]), smax = __uint_as_float(pmax[1]);
  const size_t base = (size_t)blockIdx.x * kBwdRaysPerBlock;
  // dL/dA of the ray (with a background, of the composite over it)
  auto base_tdot = [&](size_t r, const float4 &g) {
    float t = g.w;
    if (bg) t -= g.x * bg[3 * r] + g.y * bg[3 * r + 1] + g.z * bg[3 * r + 2];
    return t;
  };
  auto write = [&](size_t r, const float4 &g, float tdot, float wsig, int kstar, bool clamped) {
    rc[r] = RayConst{tdot, wsig, kstar, 0};
    const float g1 = fabsf(g.x) + fabsf(g.y) + fabsf(g.z);
    const float gi = fmaxf(fabsf(g.x), fmaxf(fabsf(g.y), fabsf(g.z)));
    const RayBound b{av.step * (fabsf(tdot) + g1 * cmax + smax * gi), clamped ? gi : 0.f};
    rbd[r] = b;
    if (!(b.per_sample <= 1e30f && b.clamp <= 1e30f)) atomicOr(odd, 1u);   // times 2^24 samples it may overflow
  };
  for (int o = 0; o < kBwdRaysPerBlock; o += 256) {
    const size_t r = base + o + threadIdx.x;
    if (r >= R) break;
    const mvp_ray_aux ax = aux[r];
    const float4 g = grad_rgba[r];
    if (bg && g_bg) {
      const float u = 1.0f - rgba[r].w;
      g_bg[3 * r] += u * g.x;
      g_bg[3 * r + 1] += u * g.y;
      g_bg[3 * r + 2] += u * g.z;
    }
    if (ax.j_end >= 0 && ax.t_prev >= 0.f) s_clamped[atomicAdd(&s_nc, 1)] = (uint32_t)(o + threadIdx.x);
    else write(r, g, base_tdot(r, g), 0.f, -1, false);
  }
  __syncthreads();
  const int nc = s_nc;
  for (int ci = threadIdx.x; ci < nc; ci += blockDim.x) {
    const size_t r = base + s_clamped[ci];
    const mvp_ray_aux ax = aux[r];
    const float4 g = grad_rgba[r];
    float tdot = base_tdot(r, g), wsig = 0.f;
    int kstar = -1;
    // the ray's pairs open at its last sample, in increasing primitive id as
    // the forward visited them
    const float tau = (float)ax.j_end * av.step;
    const int tile = slot_tile(av, r);
    const uint64_t lb = av.tile_off[tile];
    int v, px, py;
    slot_pixel(av, r, &v, &px, &py);
    float d[3];
    pixel_ray(av.cams[v], px, py, d);
    const uint32_t seg = (uint32_t)av.ray_seg[r];
    const int stride = tile_ray_count(av, tile);
    const int n = av.ray_nj[r].x;
    if (av.combine) {
      float T = ax.t_prev;
      int last = -1;
      for (int i = next_by_id(av, seg, stride, n, ax.j_end, last); i < n; i = next_by_id(av, seg, stride, n, ax.j_end, last)) {
        const int4 pq = av.pr[seg + i * stride];
        float4 A, B;
        entry_ray(av, lb + (uint64_t)pq.z, d, A, B);
        const float4 s = sample_pair<BF16, FADE>(av, pay, s_fade, A, B, tau);
        const float Tn = T + s.w * av.step;
        last = pq.w;
        if (Tn > 1.0f) {
          kstar = prim_of(A);
          tdot = -(g.x * s.x + g.y * s.y + g.z * s.z);
          wsig = 1.0f - T;
          break;
        }
        T = Tn;
      }
    } else {
      // the pairs open at S, in list order (the order the forward summed them
      // in); their records are read four at a time, so that the scan does not
      // wait for one record before asking for the next
      float sig = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
      constexpr int kB = 4;
      for (int i0 = 0; i0 < n; i0 += kB) {
        int4 q[kB];
#pragma unroll
        for (int k = 0; k < kB; ++k)
          q[k] = i0 + k < n ? av.pr[seg + (i0 + k) * stride] : make_int4(INT_MAX, INT_MIN, 0, 0);
#pragma unroll
        for (int k = 0; k < kB; ++k) {
          if (q[k].x > ax.j_end || q[k].y < ax.j_end) continue;
          float4 A, B;
          entry_ray(av, lb + (uint64_t)q[k].z, d, A, B);
          const float4 s = sample_pair<BF16, FADE>(av, pay, s_fade, A, B, tau);
          sig += s.w;
          c0 = fmaf(s.w, s.x, c0);
          c1 = fmaf(s.w, s.y, c1);
          c2 = fmaf(s.w, s.z, c2);
        }
        if (q[kB - 1].x > ax.j_end) break;   // sorted by first sample: no later pair is open
      }
      tdot = -(g.x * (c0 / sig) + g.y * (c1 / sig) + g.z * (c2 / sig));
      wsig = (1.0f - ax.t_prev) / sig;
    }
    write(r, g, tdot, wsig, kstar, !av.combine || kstar >= 0);
  }
}

// Largest colour and opacity magnitudes of the payload, as float bits in
// pmax[0] and pmax[1] (which start at zero; non-negative floats order like
// their bit patterns).  A value that is not finite raises *odd.
template <bool BF16>
__global__ __launch_bounds__(256) void k_payload_bound(const void *__restrict__ pay, size_t n_vox,
                                                       uint32_t *__restrict__ pmax, uint32_t *__restrict__ odd) {
  float c = 0.f, sg = 0.f;
  bool finite = true;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_vox; i += (size_t)gridDim.x * blockDim.x) {
    const float4 v = Voxels<BF16>::load(pay, i);
    c = fmaxf(c, fmaxf(fabsf(v.x), fmaxf(fabsf(v.y), fabsf(v.z))));
    sg = fmaxf(sg, fabsf(v.w));
    finite = finite && fabsf(v.x) + fabsf(v.y) + fabsf(v.z) + fabsf(v.w) < INFINITY;
  }
  if (__ballot(!finite) && (threadIdx.x & (kWave - 1)) == 0) atomicOr(odd, 1u);
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    c = fmaxf(c, __shfl_xor(c, d, kWave));
    sg = fmaxf(sg, __shfl_xor(sg, d, kWave));
  }
  // one pair of atomics per workgroup: atomics on one address are serialised
  // at the L2, so their number, not the payload read, sets this kernel's time
  __shared__ float s_c[256 / kWave], s_s[256 / kWave];
  const int wave = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    s_c[wave] = c;
    s_s[wave] = sg;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 256 / kWave; ++w) {
      c = fmaxf(c, s_c[w]);
      sg = fmaxf(sg, s_s[w]);
    }
    atomicMax(&pmax[0], __float_as_uint(c));
    atomicMax(&pmax[1], __float_as_uint(sg));
  }
}

struct BwdOut {
  float *pay, *pos, *rot, *scale;
};


// The LDS copy of a primitive's payload gradient is planar: channel ch of
// voxel (ix, iy, iz) at ch * plane + ix + iy * sy + iz * sz.  A wave adds one
// channel of one corner per instruction, and the lanes working in one cell add
// to its 8 different corners (see the mirrored lanes in bwd_pair); with 64-bit
// words a bank pair is a word index mod 16, so the strides are padded until
// the 8 corner offsets {0, 1} + {0, sy} + {0, sz} fall on 8 different bank
// pairs (8^3: sy = 8, sz = 66), when the padded copy fits the LDS; otherwise
// the copy is packed (sy = M, sz = M^2, plane = M^3 + 1).
struct LdsMap {
  int sy, sz, plane;
};

__host__ __device__ inline LdsMap lds_map(int M, bool padded) {
  if (!padded) return LdsMap{M, M * M, M * M * M + 1};
  auto distinct = [](int a, int b) {   // {0, 1, a, a + 1, b, b + 1, a + b, a + b + 1} mod 16
    int seen = 0;
    const int v[8] = {0, 1, a, a + 1, b, b + 1, a + b, a + b + 1};
    for (int i = 0; i < 8; ++i) {
      const int bit = 1 << (v[i] & 15);
      if (seen & bit) return false;
      seen |= bit;
    }
    return true;
  };
  int sy = M;
  while ((sy & 15) == 0 || (sy & 15) == 1 || (sy & 15) == 15) ++sy;
  int sz = sy * M;
  while (!distinct(sy, sz)) ++sz;
  return LdsMap{sy, sz, sz * M};
}

// One addend of the fixed-point accumulator: v rounded to the nearest integer
// (|v| < 2^30 by the choice of scale), sign-extended to the 64-bit two's
// complement word that the LDS atomic adds.  (Rounding down v + 1/2, formed in
// one fma, saves an instruction but is biased where v has no fraction bits left.)
//
// WIDE (payloads taken in slabs, sparse rays): |v| < 2^50, converted in two
// exact parts.  The scale follows the largest bound of an item's pairs, which
// may be thousands of times what most voxels get (a ray that saturates in a
// faint sample): with 30 bits the rounding of every addend then shows in the
// gradient (970 x 24^3 with the fade window: over 1e-6 of it), with 50 bits only
// the FP32 rounding of the run's own sums is left (the voxels beside one ray with 2^18
// times the others' upstream gradient: under 2e-6, 3e-6 to 7e-6 with 44 bits).
template <bool WIDE>
__device__ __forceinline__ unsigned long long fixed_addend(float v) {
  if constexpr (WIDE) {
    const float h = rintf(v * 0x1p-20f);
    const float l = fmaf(h, -0x1p20f, v);
    return (unsigned long long)((long long)(int)h * (1ll << 20) + (long long)__float2int_rn(l));
  }
  return (unsigned long long)(long long)__float2int_rn(v);
}

// The scale of a work item's fixed-point gradient as a product of two powers of
// two of about its root: one goes into the rays' upstream colour gradients, the
// other into the sums they multiply, so that neither overflows where the
// product does not and a cell's 32 addends need no scaling of their own.
struct FixedScale {
  float g, w, both;
};
__device__ __forceinline__ FixedScale split_scale(float scale) {
  if (!(scale > 0.f)) return FixedScale{0.f, 0.f, 0.f};
  int e;
  (void)frexpf(scale, &e);   // scale = 2^(e-1)
  const int h = (e - 1) / 2;
  return FixedScale{ldexpf(1.0f, h), ldexpf(1.0f, e - 1 - h), scale};
}

// Adds a run's corner adjoints: of the colours g times bw, of the opacity b3
// (LDS_ACC: scaled, see FixedScale).
template <bool LDS_ACC, bool FADE, bool WIDE, typename T>
__device__ __forceinline__ void flush_cell(T *dst, size_t cell, int M, const LdsMap &lm, const float (&g)[3],
                                           const float (&bw)[8], const float (&b3)[8], const float (&wq)[8], unsigned m) {
  // cell: LDS slot of corner (0,0,0) (LDS_ACC) or its voxel index in device memory
  const size_t sy = LDS_ACC ? (size_t)lm.sy : (size_t)M, sz = LDS_ACC ? (size_t)lm.sz : (size_t)M * M;
  const size_t plane = (size_t)lm.plane;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const unsigned r = (unsigned)q ^ m;
    const size_t vox = cell + (r & 1u) + ((r >> 1) & 1u) * sy + (r >> 2) * sz;
    if constexpr (LDS_ACC) {
#pragma unroll
      for (int c = 0; c < 3; ++c) atomicAdd(dst + c * plane + vox, fixed_addend<WIDE>(g[c] * bw[q]));
      atomicAdd(dst + 3 * plane + vox, fixed_addend<WIDE>(FADE ? b3[q] * wq[q] : b3[q]));
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) unsafeAtomicAdd(dst + vox * 4 + c, g[c] * bw[q]);
      unsafeAtomicAdd(dst + vox * 4 + 3, FADE ? b3[q] * wq[q] : b3[q]);
    }
  }
}

// A trilinear function along a run: the samples of one cell lie on a line, at
// (x, y, z) + n (p, q, r) with n the sample's distance from the run's middle,
// so in the monomial basis f = sum_q F[q] m_q of the cell offsets it is the
// cubic c0 + c1 n + c2 n^2 + c3 n^3, and its derivative along an axis the
// quadratic d[axis][0] + d[axis][1] n + d[axis][2] n^2.
struct LineFn {
  float c0, c1, c2, c3;
  float d[3][3];
};

__device__ __forceinline__ LineFn along(const float (&F)[8], float x, float y, float z, float p, float q, float r,
                                        float pq, float pr, float qr, float pqr) {
  LineFn f;
  const float u0 = fmaf(F[4], z, F[0]), u1 = fmaf(F[5], z, F[1]), u2 = fmaf(F[6], z, F[2]), u3 = fmaf(F[7], z, F[3]);
  const float v5 = fmaf(F[7], y, F[5]), v6 = fmaf(F[7], x, F[6]);
  f.d[0][0] = fmaf(u3, y, u1);
  f.d[1][0] = fmaf(u3, x, u2);
  f.d[2][0] = fmaf(v6, y, fmaf(F[5], x, F[4]));
  f.d[0][1] = fmaf(u3, q, v5 * r);
  f.d[1][1] = fmaf(u3, p, v6 * r);
  f.d[2][1] = fmaf(v5, p, v6 * q);
  f.d[0][2] = F[7] * qr;
  f.d[1][2] = F[7] * pr;
  f.d[2][2] = F[7] * pq;
  f.c0 = fmaf(y, f.d[1][0], fmaf(x, u1, u0));
  f.c1 = fmaf(r, f.d[2][0], fmaf(q, f.d[1][0], p * f.d[0][0]));
  f.c2 = fmaf(qr, v6, fmaf(pr, v5, pq * u3));
  f.c3 = F[7] * pqr;
  return f;
}

constexpr unsigned kSlabGrid = 4096;   // workgroups over the listed items (most may not be there)

// Longest run taken at once (a longer one is taken in parts).
constexpr int kRunMax = 64;

// Cell layers [z0, z1) of a primitive that a work item handles: all of them,
// or one slab of a payload whose gradient does not fit the LDS.
struct Slab {
  int z0, z1;
};

// The samples of [lo, hi] of a pair whose cells lie in the slab (z of the local
// ray: a, b).  The layer of a sample is locate's, and monotone along the ray:
// the ends are predicted, then settled with locate's own arithmetic, so that
// every sample belongs to exactly one slab.
__device__ __forceinline__ void clip_to_slab(const Slab &sl, float a, float b, float dt, int M, float hM, int &lo,
                                             int &hi) {
  const float top = (float)(M - 2);
  auto layer = [&](int j) {
    const float y = fmaf((float)j * dt, b, a);
    return (int)fminf(floorf(fmaf(fminf(fmaxf(y, -1.0f), 1.0f), hM, hM)), top);
  };
  if (lo > hi) return;
  const bool up = b >= 0.f;
  // first sample at or past the entry face, last one before the exit face
  const float step = b * hM * dt;
  const float is = fabsf(step) > 1e-12f ? 1.0f / step : 0.f;
  const float u0 = fmaf(a, hM, hM);
  const float te = ((float)(up ? sl.z0 : sl.z1) - u0) * is, tx = ((float)(up ? sl.z1 : sl.z0) - u0) * is;
  auto in = [&](int j) { return up ? layer(j) >= sl.z0 : layer(j) < sl.z1; };      // past the entry face
  auto out = [&](int j) { return up ? layer(j) >= sl.z1 : layer(j) < sl.z0; };     // past the exit face
  int e = (int)fminf(fmaxf(is != 0.f ? ceilf(te) : (float)lo, (float)lo), (float)hi);
  while (e > lo && in(e - 1)) --e;
  while (e <= hi && !in(e)) ++e;
  int x = (int)fminf(fmaxf(is != 0.f ? floorf(tx) : (float)hi, (float)lo), (float)hi);
  while (x < hi && !out(x + 1)) ++x;
  while (x >= lo && out(x)) --x;
  lo = e;
  hi = x;
}

// How a pair is replayed: sample by sample, or by runs in closed form, whose
// samples are equidistant if dt is a power of two.  Otherwise their times fl(j dt)
// are off by a rounding each, which the sample loop takes as it comes and the closed
// form to first order (a payload gradient of 46^3 at 574 samples per unit: 1.0e-6
// from that in 64 bits, 1.1e-5 if they are left out; 1.1e-6 by the loop).
enum class Replay { kLoop, kRuns, kRounded };

// Replay one (ray, primitive k) pair backward: channel adjoints to the 8
// voxel corners (registers over a run of samples in one cell, then gdst:
// the LDS copy of k's gradient or device memory) and the pair's pose sums
// added to P (12 values, see the end and pose_from_sums).
//
// Closed form (R): a run is not taken sample by sample.  g . c and the
// opacity are cubics in n (LineFn), an ordinary sample's adjoints are dt times
// them (plus a constant), so their moments sum_n n^k (.) over the run follow
// from the power sums of n, and every sum over the run's samples (corner
// adjoints, G, H) is a fixed combination of those moments: about 450 VALU
// instructions per run, whatever its length, where the sample loop takes 108 per
// sample and 240 per run and leaves the lanes with shorter runs idle.  4096 x
// 8^3, four 1024^2 views (5 samples per run): 6.5 -> 4.2 ms; 512 x 16^3 at
// 667 x 1024: 4.4 -> 1.9 ms.  At 2 samples per run the two are equal (32768 x
// 16^3 at 2 x 2048^2: 26.8 and 27.0 ms): see backward_by_runs.
template <bool BF16, bool LDS_ACC, bool FADE, Replay R, bool SLABS, bool PREFETCH, bool WIDE, typename GAcc>
__device__ __forceinline__ void bwd_pair(const AccelView &av, const char *__restrict__ payk,
                                         const mvp_ray_aux *__restrict__ aux, const float4 *__restrict__ grad_rgba,
                                         const RayConst *__restrict__ rc, const uint2 rec, uint64_t gent, int tile,
                                         int k, const float (&t)[3], const Slab &slab, GAcc *gdst, const LdsMap &lm, const FixedScale &fxs,
                                         const float *s_fade, bool pose,
                                         float (&P)[12], uint32_t &runs) {
  constexpr bool kBig = !LDS_ACC;   // (a gradient in the LDS: M of at most 45)
  const int M = av.M;
  const float hM = 0.5f * (float)(M - 1);
  const float dt = av.step;
  int2 jr = make_int2((int)(rec.x & 0xffffffu), (int)rec.y);
  size_t ray;
  int rv, px, py;
  (void)tile_ray(av, tile, (int)(rec.x >> 24), &ray, &rv, &px, &py);
  float d[3];
  pixel_ray(av.cams[rv], px, py, d);
  float4 A, B;   // the pair's local ray, from the frame of its culling-list entry gent
  entry_ray(av, gent, d, A, B);
  const mvp_ray_aux ax = aux[ray];
  const float4 g = grad_rgba[ray];
  const RayConst rcv = rc[ray];
  const float tdot = rcv.tdot, wsig = rcv.w;
  // sum rule: sample S uses the clamp formulas; sequential: only k* does
  // (primitives before it are ordinary steps, those after it add nothing)
  const bool seq = av.combine != 0;
  const bool clamped = ax.t_prev >= 0.f && (!seq || rcv.kstar >= 0);
  int jh = min(jr.y, ax.j_end);
  if (SLABS) clip_to_slab(slab, A.z, B.z, dt, M, hM, jr.x, jh);
  float G0 = 0.f, G1 = 0.f, G2 = 0.f, H0 = 0.f, H1 = 0.f, H2 = 0.f;
  const float gsc[3] = {g.x * fxs.g, g.y * fxs.g, g.z * fxs.g};
  float4 cv[8];
  float wq[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) wq[q] = 1.0f;
  // Into LDS, lane L works in the cell coordinates mirrored along the axes
  // named by the bits of m = L mod 8: its register slot q holds corner q ^ m,
  // so lanes of one wave that flush the same cell add to different voxels in
  // each instruction (instead of serialising on one address) at no cost in
  // register moves.  Mirroring an axis maps its offset f to 1 - f and flips
  // the sign of the derivative along it.
  const unsigned m = (LDS_ACC && kRotateFlush) ? (threadIdx.x & 7u) : 0u;
  const bool mx = m & 1u, my = (m >> 1) & 1u, mz = (m >> 2) & 1u;
  const float sgx = mx ? -1.0f : 1.0f, sgy = my ? -1.0f : 1.0f, sgz = mz ? -1.0f : 1.0f;
  const float offx = mx ? 1.0f : 0.0f, offy = my ? 1.0f : 0.0f, offz = mz ? 1.0f : 0.0f;
  const float hMx = sgx * hM, hMy = sgy * hM, hMz = sgz * hM;
  // byte offsets of the register slots' voxels in the primitive's payload
  constexpr int kVox = BF16 ? 8 : 16;
  const int MMi = M * M;
  const int so0 = kVox * ((mx ? 1 : 0) + (my ? M : 0) + (mz ? MMi : 0));
  const int sx = mx ? -kVox : kVox, sy = my ? -kVox * M : kVox * M, sz = mz ? -kVox * MMi : kVox * MMi;
  auto load_cell = [&](int cell) {
    if constexpr (LDS_ACC) {   // (a primitive whose gradient fits the LDS is far below 4 GiB)
      const int b0 = cell * kVox + so0;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        cv[q] = Voxels<BF16>::load(payk + (uint32_t)(b0 + ((q & 1) ? sx : 0) + ((q & 2) ? sy : 0) + ((q & 4) ? sz : 0)), 0);
    } else {
      const char *b0 = payk + (size_t)cell * kVox + so0;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        cv[q] = Voxels<BF16>::load(b0 + (ptrdiff_t)((q & 1) ? sx : 0) + ((q & 2) ? sy : 0) + ((q & 4) ? sz : 0), 0);
    }
  };
  // The pair's reference sample time: the sums of the pose gradient take sample
  // times from it and positions from the primitive's centre, which keeps them
  // free of the cancellation of camera distances (60 box sizes on the 4096 x 8^3
  // scene).
  const float tref = 0.5f * (float)(jr.x + jh) * dt;
  if constexpr (R != Replay::kLoop) {
    // offsets per sample, signed by direction and (p, q, r) mirrored; samples per
    // unit of offset
    const float s0 = B.x * hM * dt, s1 = B.y * hM * dt, s2 = B.z * hM * dt;
    const float p = sgx * s0, q = sgy * s1, r = sgz * s2;
    const float pq = p * q, pr = p * r, qr = q * r, pqr = pq * r;
    auto inv = [](float s) { return fminf(__builtin_amdgcn_rcpf(fabsf(s)), 1e20f); };
    const float i0 = inv(s0), i1 = inv(s1), i2 = inv(s2);
    // What keeps a predicted sample inside the cell by more than the rounding of
    // locate's position (about 2e-7 M offset units) and of the sample times (one
    // part in 2^24): a run that ends a sample early goes on in the next one.
    const float slack = 1e-6f * (float)M, jslack = fmaf(2.4e-7f, (float)jh, 1e-3f);
    int j = jr.x;
    Cell c;
    if (j <= jh) {
      c = locate<kBig>(A, B, (float)j * dt, M, hM);
      if (PREFETCH) load_cell(c.idx);
    }
    while (j <= jh) {
      const int cell = c.idx;
      const int ci0 = c.i[0], ci1 = c.i[1], ci2 = c.i[2];
      ++runs;
      if (!PREFETCH) load_cell(cell);
      // the run's last sample
      const float e0 = ((s0 > 0.f ? 1.0f - c.f[0] : c.f[0]) - slack) * i0, e1 = ((s1 > 0.f ? 1.0f - c.f[1] : c.f[1]) - slack) * i1,
                  e2 = ((s2 > 0.f ? 1.0f - c.f[2] : c.f[2]) - slack) * i2;
      const float ex = fminf(fmaxf(fminf(fminf(e0, e1), e2) - jslack, 0.0f), (float)(kRunMax - 1));
      const int jl = min(j + (int)ex, jh);
      const bool sp = clamped && jl == ax.j_end && (!seq || k >= rcv.kstar);   // it is the clamping sample
      const int j0 = j, L = jl - j + (sp ? 0 : 1);   // first and number of the run's ordinary samples
      const float jm = 0.5f * (float)(j + j + L - 1);   // their middle
      const float tm = jm * dt;
      // offsets from the cell's own corner ((M-1)/2 - index is exact): rounded once,
      // at their own size, where the whole coordinate's rounding would be shared by
      // all of the run's samples
      const float x = fmaf(fmaf(tm, B.x, A.x), hMx, fmaf(sgx, hM - (float)ci0, offx)),
                  y = fmaf(fmaf(tm, B.y, A.y), hMy, fmaf(sgy, hM - (float)ci1, offy)),
                  z = fmaf(fmaf(tm, B.z, A.z), hMz, fmaf(sgz, hM - (float)ci2, offz));
      if (FADE) {
        const float wx[2] = {s_fade[ci0 + (mx ? 1 : 0)], s_fade[ci0 + (mx ? 0 : 1)]};
        const float wy[2] = {s_fade[ci1 + (my ? 1 : 0)], s_fade[ci1 + (my ? 0 : 1)]};
        const float wz[2] = {s_fade[ci2 + (mz ? 1 : 0)], s_fade[ci2 + (mz ? 0 : 1)]};
  #pragma unroll
        for (int q8 = 0; q8 < 8; ++q8) {
          wq[q8] = wx[q8 & 1] * wy[(q8 >> 1) & 1] * wz[q8 >> 2];
          cv[q8].w *= wq[q8];
        }
      }
      // The cell's field in the monomial basis (m_q the product of the offsets
      // named by the bits of q).  The ray's upstream colour gradient g is fixed
      // along the run, and every colour term of a sample (g . rgb, the colour
      // adjoint ws g and its position derivative) involves the colours only
      // through g . c: the run keeps g . c and the opacity, and sums the colour
      // adjoint as g times sum_s m_q ws.
      float gcf[8], sf[8];
  #pragma unroll
      for (int q8 = 0; q8 < 8; ++q8) {
        gcf[q8] = fmaf(g.z, cv[q8].z, fmaf(g.y, cv[q8].y, g.x * cv[q8].x));
        sf[q8] = cv[q8].w;
      }
      // the next run's first sample, and its corners
      j = jl + 1;
      if (j <= jh) {
        c = locate<kBig>(A, B, (float)j * dt, M, hM);
        if (PREFETCH) load_cell(c.idx);
      }
  #pragma unroll
      for (int bit = 1; bit < 8; bit <<= 1)
  #pragma unroll
        for (int q8 = 0; q8 < 8; ++q8)
          if (q8 & bit) {
            gcf[q8] -= gcf[q8 ^ bit];
            sf[q8] -= sf[q8 ^ bit];
          }
      const LineFn fg = along(gcf, x, y, z, p, q, r, pq, pr, qr, pqr), fs = along(sf, x, y, z, p, q, r, pq, pr, qr, pqr);
      // moments of the samples' factors: ws (of g in dL/d(rgb)) and a3 (dL/dsigma)
      float W0, W1, W2, W3, V0, V1, V2, V3;
      {
        // power sums of n = -(L-1)/2 .. (L-1)/2 (odd ones vanish), times dt
        const float l = (float)L, l2 = l * l;
        const float S0 = l * dt, S2 = S0 * (l2 - 1.0f) * (1.0f / 12), S4 = S2 * fmaf(3.0f, l2, -7.0f) * (1.0f / 20),
                    S6 = S2 * fmaf(fmaf(3.0f, l2, -18.0f), l2, 31.0f) * (1.0f / 112);
        const float h0 = tdot + fg.c0;
        W0 = fmaf(S2, fs.c2, S0 * fs.c0);
        W1 = fmaf(S4, fs.c3, S2 * fs.c1);
        W2 = fmaf(S4, fs.c2, S2 * fs.c0);
        W3 = fmaf(S6, fs.c3, S4 * fs.c1);
        V0 = fmaf(S2, fg.c2, S0 * h0);
        V1 = fmaf(S4, fg.c3, S2 * fg.c1);
        V2 = fmaf(S4, fg.c2, S2 * h0);
        V3 = fmaf(S6, fg.c3, S4 * fg.c1);
      }
      if constexpr (R == Replay::kRounded) {
        // A sample at n + e / dt in place of n adds e f'(n) to a moment dt sum f(n) of
        // the monomials up to n^3 times a cubic: the sums of e n^k up to n^5 take all of
        // it to first order (e / dt is below 1e-3).
        float E0 = 0.f, E1 = 0.f, E2 = 0.f, E3 = 0.f, E4 = 0.f, E5 = 0.f;
        for (int i = 0; i < L; ++i) {
          const float n = (float)(j0 + i) - jm;
          float e = fmaf(-n, dt, (float)(j0 + i) * dt - tm);
          E0 += e;
          e *= n;
          E1 += e;
          e *= n;
          E2 += e;
          e *= n;
          E3 += e;
          e *= n;
          E4 += e;
          E5 = fmaf(e, n, E5);
        }
        E1 *= 2.0f;
        E2 *= 3.0f;
        E3 *= 4.0f;
        E4 *= 5.0f;
        E5 *= 6.0f;
        auto shift = [&](float c0, float c1, float c2, float c3, float &M0, float &M1, float &M2, float &M3) {
          M0 = fmaf(c1, E0, fmaf(c2, E1, fmaf(c3, E2, M0)));
          M1 = fmaf(c0, E0, fmaf(c1, E1, fmaf(c2, E2, fmaf(c3, E3, M1))));
          M2 = fmaf(c0, E1, fmaf(c1, E2, fmaf(c2, E3, fmaf(c3, E4, M2))));
          M3 = fmaf(c0, E2, fmaf(c1, E3, fmaf(c2, E4, fmaf(c3, E5, M3))));
        };
        shift(fs.c0, fs.c1, fs.c2, fs.c3, W0, W1, W2, W3);
        shift(tdot + fg.c0, fg.c1, fg.c2, fg.c3, V0, V1, V2, V3);
      }
      if (sp) {
        float n = (float)jl - jm;
        if constexpr (R == Replay::kRounded) n = fmaf(fmaf(-n, dt, (float)jl * dt - tm), __builtin_amdgcn_rcpf(dt), n);
        const float gc = fmaf(n, fmaf(n, fmaf(n, fg.c3, fg.c2), fg.c1), fg.c0);
        const float sg = fmaf(n, fmaf(n, fmaf(n, fs.c3, fs.c2), fs.c1), fs.c0);
        float a3 = seq ? 0.f : wsig * (gc + tdot);
        float ws = seq ? (k == rcv.kstar ? wsig : 0.f) : wsig * sg;
        W0 += ws;
        V0 += a3;
        ws *= n;
        a3 *= n;
        W1 += ws;
        V1 += a3;
        ws *= n;
        a3 *= n;
        W2 += ws;
        V2 += a3;
        W3 = fmaf(ws, n, W3);
        V3 = fmaf(a3, n, V3);
      }
      // gradient with respect to the cell offsets, and its first moment (the
      // factor dx/dy = hM, signed on mirrored axes, is applied to the pair's sums)
      if (pose) {
        float gs[3], hs[3];
  #pragma unroll
        for (int i = 0; i < 3; ++i) {
          gs[i] = fmaf(fs.d[i][2], V2, fmaf(fs.d[i][1], V1, fmaf(fs.d[i][0], V0,
                  fmaf(fg.d[i][2], W2, fmaf(fg.d[i][1], W1, fg.d[i][0] * W0)))));
          hs[i] = fmaf(fs.d[i][2], V3, fmaf(fs.d[i][1], V2, fmaf(fs.d[i][0], V1,
                  fmaf(fg.d[i][2], W3, fmaf(fg.d[i][1], W2, fg.d[i][0] * W1)))));
        }
        G0 += gs[0];
        G1 += gs[1];
        G2 += gs[2];
        const float tr = tm - tref;
        H0 = fmaf(tr, gs[0], fmaf(dt, hs[0], H0));
        H1 = fmaf(tr, gs[1], fmaf(dt, hs[1], H1));
        H2 = fmaf(tr, gs[2], fmaf(dt, hs[2], H2));
      }
      if (gdst) {
        // adjoint of the monomial coefficients, sum_n m_q(n) (.): from the
        // moments and the monomials' own coefficients in n
        const float xy = x * y, xz = x * z, yz = y * z;
        const float xy1 = fmaf(x, q, y * p), xz1 = fmaf(x, r, z * p), yz1 = fmaf(y, r, z * q);
        const float xyz0 = xy * z, xyz1 = fmaf(xy, r, xy1 * z), xyz2 = fmaf(xy1, r, pq * z);
        float bw[8], b3[8];
        auto adjoint = [&](float (&o)[8], float M0, float M1, float M2, float M3) {
          o[0] = M0;
          o[1] = fmaf(p, M1, x * M0);
          o[2] = fmaf(q, M1, y * M0);
          o[3] = fmaf(pq, M2, fmaf(xy1, M1, xy * M0));
          o[4] = fmaf(r, M1, z * M0);
          o[5] = fmaf(pr, M2, fmaf(xz1, M1, xz * M0));
          o[6] = fmaf(qr, M2, fmaf(yz1, M1, yz * M0));
          o[7] = fmaf(pqr, M3, fmaf(xyz2, M2, fmaf(xyz1, M1, xyz0 * M0)));
          // to the corners: the transpose of the basis change
  #pragma unroll
          for (int bit = 1; bit < 8; bit <<= 1)
  #pragma unroll
            for (int q8 = 0; q8 < 8; ++q8)
              if (!(q8 & bit)) o[q8] -= o[q8 | bit];
        };
        adjoint(bw, W0 * fxs.w, W1 * fxs.w, W2 * fxs.w, W3 * fxs.w);
        adjoint(b3, V0 * fxs.both, V1 * fxs.both, V2 * fxs.both, V3 * fxs.both);
        const size_t fc = LDS_ACC ? (size_t)((unsigned)ci0 + __umul24((unsigned)ci1, (unsigned)lm.sy) +
                                             __umul24((unsigned)(SLABS ? ci2 - slab.z0 : ci2), (unsigned)lm.sz))
                                  : (size_t)cell;
        flush_cell<LDS_ACC, FADE, WIDE>(gdst, fc, M, lm, gsc, bw, b3, wq, m);
      }
    }
  } else {
    int j = jr.x;
    Cell c;
    if (j <= jh) {
      c = locate<kBig>(A, B, (float)j * dt, M, hM);
      if (PREFETCH) load_cell(c.idx);
    }
    while (j <= jh) {
      const int cell = c.idx;
      const int ci0 = c.i[0], ci1 = c.i[1], ci2 = c.i[2];
      ++runs;
      if (!PREFETCH) load_cell(cell);
      if (FADE) {
        const float wx[2] = {s_fade[ci0 + (mx ? 1 : 0)], s_fade[ci0 + (mx ? 0 : 1)]};
        const float wy[2] = {s_fade[ci1 + (my ? 1 : 0)], s_fade[ci1 + (my ? 0 : 1)]};
        const float wz[2] = {s_fade[ci2 + (mz ? 1 : 0)], s_fade[ci2 + (mz ? 0 : 1)]};
  #pragma unroll
        for (int q = 0; q < 8; ++q) {
          wq[q] = wx[q & 1] * wy[(q >> 1) & 1] * wz[q >> 2];
          cv[q].w *= wq[q];
        }
      }
      // The cell's field in the monomial basis: f = sum_q cf[q] m_q with m_q the
      // product of the offsets (x, y, z) named by the bits of q.  The ray's
      // upstream colour gradient g is fixed along the run, and every colour term
      // of a sample (g . rgb, the colour adjoint ws g and its position
      // derivative) involves the colours only through g . c: the run keeps
      // gcf[q] = g . cf[q][rgb] and the opacity coefficients sf[q] (the basis
      // change is linear, so gcf comes from the corners' g . c), and sums the
      // colour adjoint as g times sum_s m_q ws.
      float gcf[8], sf[8], bw[8], b3[8];
  #pragma unroll
      for (int q = 0; q < 8; ++q) {
        gcf[q] = fmaf(g.z, cv[q].z, fmaf(g.y, cv[q].y, g.x * cv[q].x));
        sf[q] = cv[q].w;
        bw[q] = b3[q] = 0.f;
      }
  #pragma unroll
      for (int bit = 1; bit < 8; bit <<= 1)
  #pragma unroll
        for (int q = 0; q < 8; ++q)
          if (q & bit) {
            gcf[q] -= gcf[q ^ bit];
            sf[q] -= sf[q ^ bit];
          }
      do {
        const float tau = (float)j * dt;
        // offsets, mirrored where the lane's axis is: |0 - f| = f, |1 - f| = 1 - f
        // (0 <= f <= 1; the absolute value folds into the instructions that use it)
        const float fx = fabsf(offx - c.f[0]), fy = fabsf(offy - c.f[1]), fz = fabsf(offz - c.f[2]);
        const float mxy = fx * fy, mxz = fx * fz, myz = fy * fz, mxyz = mxy * fz;
        const float mq[8] = {1.0f, fx, fy, mxy, fz, mxz, myz, mxyz};
        float gc = gcf[0], sg = sf[0];
  #pragma unroll
        for (int q = 1; q < 8; ++q) {
          gc = fmaf(mq[q], gcf[q], gc);
          sg = fmaf(mq[q], sf[q], sg);
        }
        float a3, ws;   // dL/dsigma and the factor of g in dL/d(rgb) for this prim-sample
        if (clamped && j == ax.j_end && (!seq || k >= rcv.kstar)) {
          a3 = seq ? 0.f : wsig * (gc + tdot);
          ws = seq ? (k == rcv.kstar ? wsig : 0.f) : wsig * sg;
        } else {
          a3 = dt * (tdot + gc);
          ws = dt * sg;
        }
        // adjoint of the monomial coefficients; the corners' are formed at the flush
        const float wsf = ws * fxs.w, a3f = a3 * fxs.both;
  #pragma unroll
        for (int q = 0; q < 8; ++q) {
          bw[q] = fmaf(mq[q], wsf, bw[q]);
          b3[q] = fmaf(mq[q], a3f, b3[q]);
        }
        // gradient with respect to the cell offsets of the interpolant of the
        // adjoint-weighted channels: al[q] = a . cf[q], d/dx of sum al[q] m_q
        // (the factor dx/dy = hM, signed on mirrored axes, is applied to the
        // pair's sums G and H)
        float al[8];
  #pragma unroll
        for (int q = 1; q < 8; ++q) al[q] = fmaf(ws, gcf[q], a3 * sf[q]);
        const float gx = fmaf(al[7], myz, fmaf(al[5], fz, fmaf(al[3], fy, al[1])));
        const float gyv = fmaf(al[7], mxz, fmaf(al[6], fz, fmaf(al[3], fx, al[2])));
        const float gz = fmaf(al[7], mxy, fmaf(al[6], fy, fmaf(al[5], fx, al[4])));
        G0 += gx;
        G1 += gyv;
        G2 += gz;
        H0 = fmaf(tau, gx, H0);
        H1 = fmaf(tau, gyv, H1);
        H2 = fmaf(tau, gz, H2);
        ++j;
        if (j > jh) break;
        c = locate<kBig>(A, B, (float)j * dt, M, hM);
      } while (c.idx == cell);
      if (PREFETCH && j <= jh) load_cell(c.idx);
      // monomial adjoint -> corner adjoint (transpose of the basis change), on
      // the two sums before the colour adjoint is spread over the channels
  #pragma unroll
      for (int bit = 1; bit < 8; bit <<= 1)
  #pragma unroll
        for (int q = 0; q < 8; ++q)
          if (!(q & bit)) {
            bw[q] -= bw[q | bit];
            b3[q] -= b3[q | bit];
          }
      if (gdst) {
        const size_t fc = LDS_ACC ? (size_t)((unsigned)ci0 + __umul24((unsigned)ci1, (unsigned)lm.sy) +
                                             __umul24((unsigned)(SLABS ? ci2 - slab.z0 : ci2), (unsigned)lm.sz))
                                  : (size_t)cell;
        flush_cell<LDS_ACC, FADE, WIDE>(gdst, fc, M, lm, gsc, bw, b3, wq, m);
      }
    }
  }
  if (!pose) return;
  // y = A (x - t), x = o + tau d, A = diag(1/s) R^T, d the unit pixel ray.  The
  // pose gradient is linear in the pair's sums G = sum dL/dy and
  // H = sum (tau - tref) dL/dy, and the primitive is the same for every pair of
  // a work item, so the pair adds only sum G (P[0..2]) and (P[3 + 3m + i])
  // sum (x - t)_m dL/dy_i = (o + tref d - t)_m G_i + d_m H_i, or for the sample
  // loop (tref = 0) sum x_m dL/dy_i = o_m G_i + d_m H_i; the primitive's A, t, R
  // and s are applied once per item (pose_from_sums).
  const DevCam &cam = av.cams[rv];
  const float G[3] = {hMx * G0, hMy * G1, hMz * G2}, H[3] = {hMx * H0, hMy * H1, hMz * H2};
#pragma unroll
  for (int mm = 0; mm < 3; ++mm) {
    const float w = R != Replay::kLoop ? fmaf(tref, d[mm], cam.o[mm] - t[mm]) : cam.o[mm];
#pragma unroll
    for (int i = 0; i < 3; ++i) P[3 + 3 * mm + i] = fmaf(w, G[i], fmaf(d[mm], H[i], P[3 + 3 * mm + i]));
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) P[i] += G[i];
}

// Output i (0-2 dL/dt, 3-11 dL/dR row-major, 12-14 dL/ds) of primitive k's
// pose gradient from the sums of its pairs (bwd_pair): SG = sum G and
// S[m][i] = sum (x - t)_m dL/dy_i (CENTRED, the closed form) or sum x_m dL/dy_i.  With
// P_mi = S_mi, or S_mi - t_m SG_i: dL/dt_m = -sum_i A_im SG_i,
// dL/dR_mi = P_mi / s_i, dL/ds_i = -sum_m R_mi P_mi / s_i^2.
template <bool CENTRED>
__device__ __forceinline__ float pose_from_sums(const AccelView &av, const float *__restrict__ rot,
                                                const float *__restrict__ scale, int k, const float *sums,
                                                int i) {
  float Am[9], t[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const float4 row = av.xf[3 * (size_t)k + r];
    Am[3 * r] = row.x; Am[3 * r + 1] = row.y; Am[3 * r + 2] = row.z; t[r] = row.w;
  }
  auto rel = [&](int m, int c) { return CENTRED ? sums[3 + 3 * m + c] : sums[3 + 3 * m + c] - t[m] * sums[c]; };
  if (i < 3) return -fmaf(Am[6 + i], sums[2], fmaf(Am[3 + i], sums[1], Am[i] * sums[0]));
  if (i < 12) return rel((i - 3) / 3, (i - 3) % 3) / scale[3 * (size_t)k + (i - 3) % 3];
  const int c = i - 12;
  const float sk = scale[3 * (size_t)k + c];
  float rp = 0.f;
#pragma unroll
  for (int m = 0; m < 3; ++m) rp = fmaf(rot[9 * (size_t)k + 3 * m + c], rel(m, c), rp);
  return -rp / (sk * sk);
}


// Samples the backward replays for the pair of entry record rec (of a
// culling-list entry of `tile`): its samples up to the ray's last.  Raises
// `bound` to the pair's bound on what it adds to any one payload gradient
// value (see RayBound), if larger.
// Maximum that propagates NaN (a non-finite bound must reach fixed_scale).
__device__ __forceinline__ float nan_max(float a, float b) {
  return (a == a && b == b) ? fmaxf(a, b) : __builtin_nanf("");
}

template <bool SLABS>
__device__ __forceinline__ int pair_len(const AccelView &av, const mvp_ray_aux *__restrict__ aux,
                                        const RayBound *__restrict__ rbd, const uint2 rec, uint64_t gent, int tile,
                                        const Slab &slab, float &bound) {
  int lo = (int)(rec.x & 0xffffffu);
  size_t ray;
  int rv, px, py;
  (void)tile_ray(av, tile, (int)(rec.x >> 24), &ray, &rv, &px, &py);
  const int je = aux[ray].j_end;
  int hi = min((int)rec.y, je);
  if (SLABS && lo <= hi) {
    float d[3];
    pixel_ray(av.cams[rv], px, py, d);
    const float4 f = av.ef[3 * gent + 2];
    clip_to_slab(slab, f.w, row_dot(f.x, f.y, f.z, d), av.step, av.M, 0.5f * (float)(av.M - 1), lo, hi);
  }
  const int n = max(0, hi - lo + 1);
  if (n > 0) {
    const RayBound rb = rbd[ray];
    const float b = (float)n * rb.per_sample + (hi >= je ? rb.clamp : 0.f);
    bound = nan_max(bound, b);
  }
  return n;
}

// Fixed-point scale of a work item of `total` pairs none of which adds more than
// `bound` to any one gradient value.  A cell run adds part of one pair's share,
// so with the scale below every addend is under 2^29 (half of that covers the
// rounding of the run's sums) and fits 32 bits; an item has at most 128
// entries x 256 rays = 2^15 pairs, so a 64-bit sum stays under 2^44.  WIDE:
// addends under 2^49, or less where so many pairs could take a sum past 2^62
// (more than 2^13).
// 0 for a non-finite bound (the item's gradient is then written as NaN).
template <bool WIDE>
__device__ __forceinline__ float fixed_scale(float bound, uint32_t total) {
  if (!(bound < INFINITY)) return 0.0f;
  if (!(bound > 0.0f)) return 1.0f;
  const int bits = WIDE ? min(50, 63 - (32 - __clz((int)total))) : 30;   // 32 - clz: total < 2^(32 - clz)
  int e;
  (void)frexpf(2.0f * bound, &e);   // 2 bound = m 2^e, 0.5 <= m < 1, so bound < 2^(e-1)
  return ldexpf(1.0f, min(max(bits - e, -126), 126));
}

// Payloads taken in slabs: which work items are worth it.  Every slab of an item
// costs its workgroup some 16 us however few pairs there are (128 KB of LDS to
// clear and to read back, one workgroup per CU), a pair taken with device
// atomics some 13 ns of the device.  The items of at least `few` pairs are listed
// from the front of item_lists, the others (if they have any) from its back, and
// the latter go to device memory where they would be more than kSlabsAtLeast slabs
// (about eight for each CU; fewer are hidden better than another kernel's
// latency).  64 x 32^3, 1000 rays: backward of 300 us, 3000 all in slabs; 4000 x
// 32^3 at 64 x 64: 1.5 against 6.4 ms.  Both ways take as long at 25 pairs an item
// with 2 slabs (17^3, 18^3), 30 with 3 (20^3), 36 to 50 with 4 (24^3), 55 to 85 with
// 11 (32^3) and 60 to 140 with 39 (40^3): few = 20 + 4 for each slab, up to 100.
constexpr uint32_t kSlabsAtLeast = 2048;
__global__ __launch_bounds__(kWave) void k_item_split(AccelView av, uint32_t few, uint32_t n_list) {
  const uint32_t it = blockIdx.x * (uint32_t)kWave + threadIdx.x;
  uint32_t total = 0;
  if (it < av.item_off[av.N]) {
    int lo = 0, hi = av.N - 1;   // primitive of the item: the p-th in item order, last p with item_off[p] <= it
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (av.item_off[mid] <= it) lo = mid; else hi = mid - 1;
    }
    const uint32_t k = av.item_prim[lo];
    const uint64_t eb = av.prim_entry_off[k] + (it - av.item_off[lo]) * (uint64_t)av.item_entries;
    const int nent = (int)min<uint64_t>((uint64_t)av.item_entries, av.prim_entry_off[k + 1] - eb);
    constexpr int kB = 16;   // entries asked for together
    for (int q0 = 0; q0 < nent; q0 += kB) {
      uint32_t g[kB];
      uint4 c[kB];
#pragma unroll
      for (int q = 0; q < kB; ++q) g[q] = av.prim_entries[eb + min(q0 + q, nent - 1)];
#pragma unroll
      for (int q = 0; q < kB; ++q) c[q] = ((const uint4 *)av.ent_n)[g[q]];
#pragma unroll
      for (int q = 0; q < kB; ++q) total += q0 + q < nent ? c[q].x + c[q].y + c[q].z + c[q].w : 0u;
    }
  }
  const int lane = threadIdx.x;
  const unsigned long long lt = (1ull << lane) - 1ull;
  const unsigned long long many = __ballot(total >= few), some = __ballot(total > 0 && total < few);
  uint32_t at_many = 0, at_some = 0;
  if (lane == 0) {
    if (many) at_many = atomicAdd(&av.item_lists[0], (uint32_t)__popcll(many));
    if (some) at_some = atomicAdd(&av.item_lists[1], (uint32_t)__popcll(some));
  }
  at_many = __builtin_amdgcn_readfirstlane(at_many);
  at_some = __builtin_amdgcn_readfirstlane(at_some);
  if (total >= few) av.item_lists[2 + at_many + (uint32_t)__popcll(many & lt)] = it;
  else if (total > 0) av.item_lists[2 + n_list - 1 - (at_some + (uint32_t)__popcll(some & lt))] = it;
}

// Length classes for ordering pairs: exact below 32 samples, then 4 wide.
__device__ __forceinline__ int len_bucket(int n) { return n < 32 ? n : min(kLenBuckets - 1, 32 + ((n - 32) >> 2)); }

// Backward, one workgroup per work item: up to kItemEntries (for sparse rays
// kSparseEntries) culling-list entries (tile, primitive k) of one primitive.  The pairs of those entries
// (at most one per ray of each tile) are spread over the workgroup's threads;
// the payload gradient of k is accumulated in LDS (LDS_ACC, 64-bit fixed point
// with the item's scale) and added to device memory once per item, the pose
// gradient is reduced over the workgroup and added with 15 atomics.
//
// WAVES > 1 asks the compiler for that many waves per SIMD (it then keeps the
// kernel within 512 / WAVES registers, spilling a few); it is used when the
// LDS gradient leaves room for that many workgroups per CU.  THREADS is the
// workgroup size: 512 when the LDS gradient leaves room for only one
// workgroup per CU, so that the CU still runs two waves per SIMD.
template <bool BF16, bool LDS_ACC, bool FADE, Replay R, int WAVES, int THREADS, bool SLABS = false>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_bwd_items(
    AccelView av, const float *__restrict__ rot, const float *__restrict__ scale, const void *__restrict__ pay,
    const mvp_ray_aux *__restrict__ aux, const float4 *__restrict__ grad_rgba, const RayConst *__restrict__ rc,
    const RayBound *__restrict__ rbd, BwdOut out, uint32_t sort_cap, int padded, int slab_cells, uint32_t n_list,
    unsigned long long *__restrict__ counters) {
  // loads of this thread: pairs visited by the ordering / bound pass, pairs
  // replayed, their cell runs (one voxel-corner set each), and the non-zero
  // gradient values it adds to device memory at the end of an item
  uint32_t n_visit = 0, n_rep = 0, n_run = 0, n_nz = 0;
  // gradient (LDS_ACC), fade window (FADE), pair order and classes
  extern __shared__ unsigned long long s_dyn[];
  using GAcc = typename std::conditional<LDS_ACC, unsigned long long, float>::type;
  __shared__ uint32_t s_live;
  __shared__ uint32_t s_cls[kLenBuckets];
  __shared__ uint32_t s_base[2][kLenBuckets];
  __shared__ uint32_t s_wcnt[2][THREADS / kWave][kLenBuckets];
  __shared__ float s_pose[THREADS / kWave][16];
  __shared__ float s_bnd[THREADS / kWave];
  // the pairs of an item come in sub-lists, four per entry (the rays of each
  // wave of its tile): their starts in ent_rec and their prefix sums
  constexpr bool kWide = SLABS || THREADS == kSparseThreads;
  constexpr int kEnt = THREADS == kSparseThreads ? kSparseEntries : kItemEntries;
  constexpr int kSub = 4 * kEnt;
  constexpr int kSubRounds = (kSub + THREADS - 1) / THREADS;
  __shared__ uint64_t s_start[kSub];
  __shared__ uint32_t s_pre[kSub + 1];
  __shared__ uint32_t s_wsum[kSub / kWave];
  __shared__ uint64_t s_gent[kEnt];
  __shared__ int s_tile[kEnt];
  __shared__ int s_prim, s_pos;
  const int M = av.M;
  const size_t M3 = (size_t)M * M * M;
  // SLABS: an item is taken once per slab of slab_cells cell layers, whose voxel
  // layers are the LDS copy
  const uint32_t n_slab = SLABS ? (uint32_t)((M - 2 + slab_cells) / slab_cells) : 1u;
  const LdsMap lm = SLABS ? LdsMap{M, M * M, M * M * (slab_cells + 1) + 1} : lds_map(M, padded != 0);
  const int nlds = 4 * lm.plane;                  // their planar LDS copy
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const bool pose = out.pos || out.rot || out.scale;
  GAcc *s_grad = (GAcc *)s_dyn;
  float *s_fade = (float *)((char *)s_dyn + ((LDS_ACC && out.pay) ? (size_t)nlds * sizeof(GAcc) : 0));
  uint16_t *s_sort = (uint16_t *)(s_fade + (FADE ? M : 0));   // [sort_cap] pair order
  uint8_t *s_pcls = (uint8_t *)(s_sort + sort_cap);              // [sort_cap] length class of pair i
  if (FADE) {
    fill_fade(s_fade, M, av.fade_alpha, av.fade_beta);
    __syncthreads();
  }
  // A payload taken in slabs (slab_cells > 0; !LDS_ACC is the kernel beside them that
  // goes to device memory).  n_list > 0: the items of k_item_split's lists (of at
  // most n_list items).  Values that fixed point cannot hold (*odd: infinities, NaN,
  // bounds that overflow) leave every item to device memory.
  uint32_t n_many = 0, n_few = 0;
  bool listed = false;
  if (SLABS || (!LDS_ACC && slab_cells > 0)) {
    const bool odd = *(const uint32_t *)(counters + kCntOdd) != 0u;
    if (odd ? SLABS : !SLABS && n_list == 0) return;
    listed = n_list != 0 && !odd;
    if (listed) {
      n_many = av.item_lists[0];
      n_few = av.item_lists[1];
      const uint32_t slabs = (uint32_t)((M - 2 + slab_cells) / slab_cells);
      if (((uint64_t)n_few * slabs <= kSlabsAtLeast) != SLABS) n_few = 0;   // they are the other kernel's
      if (!SLABS) n_many = 0;
    }
  }
  const uint64_t n_items = (listed ? (uint64_t)n_many + n_few : av.item_off[av.N]) * n_slab;
  for (uint64_t is = blockIdx.x; is < n_items; is += gridDim.x) {
    uint64_t it = SLABS ? is / n_slab : is;
    if (listed) it = av.item_lists[2 + (it < n_many ? it : n_list - 1 - (it - n_many))];
    Slab slab{0, M - 1};
    if (SLABS) {
      slab.z0 = (int)(is % n_slab) * slab_cells;
      slab.z1 = min(slab.z0 + slab_cells, M - 1);
    }
    if (threadIdx.x == 0) {   // primitive of the item: the p-th in item order, last p with item_off[p] <= it
      int lo = 0, hi = av.N - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (av.item_off[mid] <= it) lo = mid; else hi = mid - 1;
      }
      s_pos = lo;
      s_prim = av.item_prim ? (int)av.item_prim[lo] : lo;
    }
    __syncthreads();
    const int k = __builtin_amdgcn_readfirstlane(s_prim);
    const char *payk = (const char *)pay + (size_t)k * M3 * (BF16 ? 8 : 16);
    const float t[3] = {av.xf[3 * (size_t)k].w, av.xf[3 * (size_t)k + 1].w, av.xf[3 * (size_t)k + 2].w};
    const uint64_t chunk = it - av.item_off[s_pos];
    const uint64_t eb = av.prim_entry_off[k] + chunk * (uint64_t)av.item_entries;
    const int nent = (int)min<uint64_t>((uint64_t)av.item_entries, av.prim_entry_off[k + 1] - eb);
    const int nsub = 4 * nent;
    uint32_t incl[kSubRounds];
#pragma unroll
    for (int r = 0; r < kSubRounds; ++r) {
      const int u = r * THREADS + (int)threadIdx.x;   // sub-list u = 4 q + w: entry q, wave w of its tile
      if (u >= kSub) break;                           // (whole waves)
      const int q = u >> 2, w = u & 3;
      uint32_t cnt = 0;
      if (u < nsub) {
        const uint32_t g = av.prim_entries[eb + q];
        s_start[u] = av.ent_base[g] + (uint64_t)w * kWave;
        cnt = av.ent_n[4 * (uint64_t)g + w];
        if (w == 0) {
          s_gent[q] = g;
          s_tile[q] = (int)av.ent_tile[g];
        }
      }
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(cnt, d, kWave);
        if (lane >= d) cnt += o;
      }
      incl[r] = cnt;
      if (lane == kWave - 1) s_wsum[u / kWave] = cnt;
    }
    if (LDS_ACC && out.pay)
      for (int i = threadIdx.x; i < nlds; i += THREADS) s_grad[i] = (GAcc)0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSubRounds; ++r) {   // prefix sums over the sub-lists
      const int u = r * THREADS + (int)threadIdx.x;
      if (u >= kSub) break;
      uint32_t base = 0;
#pragma unroll
      for (int w = 0; w < kSub / kWave; ++w) base += w < u / kWave ? s_wsum[w] : 0u;
      if (u == 0) s_pre[0] = 0;
      s_pre[u + 1] = base + incl[r];
    }
    __syncthreads();
    const uint32_t total = s_pre[nsub];
    GAcc *gdst = nullptr;
    if constexpr (LDS_ACC) {
      if (out.pay) gdst = s_grad;
    } else {
      if (out.pay) gdst = out.pay + (size_t)k * M3 * 4;
    }
    float P[12];   // the pose sums of this thread's pairs (see bwd_pair)
#pragma unroll
    for (int i = 0; i < 12; ++i) P[i] = 0.f;
    float bound = 0.f;   // largest bound of this thread's pairs, then of the item's
    float fscale = 1.0f;
    FixedScale fxs{1.0f, 1.0f, 1.0f};
    if (kSortPairs && total <= sort_cap) {
      // Counting sort of the item's pairs by length class, longest first, in a
      // fixed order (class, then round r = the r-th pair of every thread's
      // contiguous chunk, then wave, then lane), so the replay order, and with
      // it every rounding, is the same from run to run; pairs of one class that
      // are replayed together come from rays a chunk apart.  A histogram pass
      // (which also sums the pairs' bounds) and a scan give the class bases;
      // the scatter ranks each round by ballot within a wave and by per-wave
      // counts across waves (double-buffered, one barrier per round).
      const uint32_t per = (total + THREADS - 1) / THREADS;
      const uint32_t c0 = threadIdx.x * per, c1 = min(total, c0 + per);
      int q0 = 0;
      if (c0 < c1) {
        int hi = nsub - 1;
        while (q0 < hi) {
          const int mid = (q0 + hi + 1) >> 1;
          if (s_pre[mid] <= c0) q0 = mid; else hi = mid - 1;
        }
      }
      if (threadIdx.x < kLenBuckets) s_cls[threadIdx.x] = 0;
      __syncthreads();
      for (uint32_t i = c0, q = q0; i < c1; ++i) {
        while (s_pre[q + 1] <= i) ++q;
        const int n = pair_len<SLABS>(av, aux, rbd, av.ent_rec[s_start[q] + (i - s_pre[q])], s_gent[q >> 2], s_tile[q >> 2], slab, bound);
        ++n_visit;
        const int b = n > 0 ? len_bucket(n) : 0xff;
        s_pcls[i] = (uint8_t)b;
        if (n > 0) atomicAdd(&s_cls[b], 1u);
      }
#pragma unroll
      for (int d = kWave / 2; d > 0; d >>= 1) bound = nan_max(bound, __shfl_xor(bound, d, kWave));
      if (lane == 0) s_bnd[wave] = bound;
      __syncthreads();
      bound = 0.f;
#pragma unroll
      for (int w = 0; w < THREADS / kWave; ++w) bound = nan_max(bound, s_bnd[w]);
      fscale = fixed_scale<kWide>(bound, total);
      if (LDS_ACC) fxs = split_scale(fscale);
      if (wave == 0) {   // exclusive scan over the classes from the longest down
        const uint32_t c = s_cls[kLenBuckets - 1 - lane];
        uint32_t incl = c;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
          const uint32_t o = __shfl_up(incl, d, kWave);
          if (lane >= d) incl += o;
        }
        s_base[0][kLenBuckets - 1 - lane] = incl - c;
        if (lane == kWave - 1) s_live = incl;
      }
      const unsigned long long lt = (1ull << lane) - 1ull;
      for (uint32_t r = 0; r < per; ++r) {
        const int cur = r & 1;
        const uint32_t i = c0 + r;
        int b = -1;
        if (i < c1) {
          const int pb_ = s_pcls[i];
          if (pb_ != 0xff) b = pb_;
        }
        s_wcnt[cur][wave][lane] = 0;   // kLenBuckets == kWave
        uint32_t rank = 0;
        unsigned long long todo = __ballot(b >= 0);
        while (todo) {   // one class at a time: its lanes and their order
          const int src = __ffsll((long long)todo) - 1;
          const int bb = __shfl(b, src, kWave);
          const unsigned long long mm = __ballot(b == bb);
          if (b == bb) rank = (uint32_t)__popcll(mm & lt);
          if (lane == src) s_wcnt[cur][wave][bb] = (uint32_t)__popcll(mm);
          todo &= ~mm;
        }
        __syncthreads();
        if (b >= 0) {
          uint32_t pos = s_base[cur][b] + rank;
          for (int w = 0; w < wave; ++w) pos += s_wcnt[cur][w][b];
          s_sort[pos] = (uint16_t)i;
        }
        if (threadIdx.x < kLenBuckets) {
          uint32_t add = 0;
#pragma unroll
          for (int w = 0; w < THREADS / kWave; ++w) add += s_wcnt[cur][w][threadIdx.x];
          s_base[cur ^ 1][threadIdx.x] = s_base[cur][threadIdx.x] + add;
        }
      }
      __syncthreads();
      const uint32_t live = s_live;
      for (uint32_t p = threadIdx.x; p < live; p += THREADS) {
        const uint32_t i = s_sort[p];
        int q = 0, hi = nsub - 1;    // entry of flattened pair i: last q with s_pre[q] <= i
        while (q < hi) {
          const int mid = (q + hi + 1) >> 1;
          if (s_pre[mid] <= i) q = mid; else hi = mid - 1;
        }
        const uint2 rec = av.ent_rec[s_start[q] + (i - s_pre[q])];
        bwd_pair<BF16, LDS_ACC, FADE, R, SLABS, WAVES == 1, kWide>(av, payk, aux, grad_rgba, rc, rec, s_gent[q >> 2], s_tile[q >> 2], k, t, slab, gdst,
                                      lm, fxs, s_fade, pose, P, n_run);
        ++n_rep;
      }
    } else {
      // list order (more pairs than the ordering buffer holds).
      // kChunkedPairs: each thread replays a contiguous run of the flattened
      // pairs, so the lanes of a wave follow rays some pixels apart, which flush
      // into different voxel cells at once; otherwise pair i goes to thread
      // i mod 256 (neighbouring pixels on neighbouring lanes).
      const uint32_t per = kChunkedPairs ? (total + THREADS - 1) / THREADS : 1;
      const uint32_t stride = kChunkedPairs ? 1 : THREADS;
      const uint32_t i0 = kChunkedPairs ? threadIdx.x * per : threadIdx.x;
      const uint32_t iend = kChunkedPairs ? min(total, i0 + per) : total;
      int q0 = 0;
      if (i0 < iend) {
        int hi = nsub - 1;    // entry of flattened pair i0: last q with s_pre[q] <= i0
        while (q0 < hi) {
          const int mid = (q0 + hi + 1) >> 1;
          if (s_pre[mid] <= i0) q0 = mid; else hi = mid - 1;
        }
      }
      if (LDS_ACC && out.pay) {   // the item's bound, for the fixed-point scale
        for (uint32_t i = i0, q = q0; i < iend; i += stride) {
          while (s_pre[q + 1] <= i) ++q;
          (void)pair_len<SLABS>(av, aux, rbd, av.ent_rec[s_start[q] + (i - s_pre[q])], s_gent[q >> 2], s_tile[q >> 2], slab, bound);
          ++n_visit;
        }
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) bound = nan_max(bound, __shfl_xor(bound, d, kWave));
        if (lane == 0) s_bnd[wave] = bound;
        __syncthreads();
        bound = 0.f;
#pragma unroll
        for (int w = 0; w < THREADS / kWave; ++w) bound = nan_max(bound, s_bnd[w]);
        fscale = fixed_scale<kWide>(bound, total);
      if (LDS_ACC) fxs = split_scale(fscale);
      }
      for (uint32_t i = i0, q = q0; i < iend; i += stride) {
        while (s_pre[q + 1] <= i) ++q;
        const uint2 rec = av.ent_rec[s_start[q] + (i - s_pre[q])];
        bwd_pair<BF16, LDS_ACC, FADE, R, SLABS, WAVES == 1, kWide>(av, payk, aux, grad_rgba, rc, rec, s_gent[q >> 2], s_tile[q >> 2], k, t, slab, gdst,
                                      lm, fxs, s_fade, pose, P, n_run);
        ++n_rep;
      }
    }
    if (pose) {
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        float x = P[i];
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d, kWave);
        if (lane == 0) s_pose[wave][i] = x;
      }
    }
    __syncthreads();
    if (pose && threadIdx.x < 12) {   // the item's sums (each thread reads and writes its own column)
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < THREADS / kWave; ++w) x += s_pose[w][threadIdx.x];
      s_pose[0][threadIdx.x] = x;
    }
    __syncthreads();
    if (pose && threadIdx.x < 15 && total > 0) {
      const int i = threadIdx.x;
      const float x = pose_from_sums<R != Replay::kLoop>(av, rot, scale, k, s_pose[0], i);
      if (i < 3) {
        if (out.pos) unsafeAtomicAdd(out.pos + 3 * (size_t)k + i, x);
      } else if (i < 12) {
        if (out.rot) unsafeAtomicAdd(out.rot + 9 * (size_t)k + (i - 3), x);
      } else {
        if (out.scale) unsafeAtomicAdd(out.scale + 3 * (size_t)k + (i - 12), x);
      }
    }
    if (LDS_ACC && out.pay && total > 0) {
      float *dst = out.pay + (M3 * (size_t)k + (size_t)slab.z0 * M * M) * 4;
      const int nacc = (slab.z1 - slab.z0 + 1) * M * M * 4;   // gradient values of the slab (shared layers: added by both)
      const bool ok = fscale > 0.0f;
      const float inv = ok ? 1.0f / fscale : __builtin_nanf("");   // exact: a power of two
      for (int i = threadIdx.x; i < nacc; i += THREADS) {   // device order: voxel i/4, channel i%4
        const int vx = i >> 2, ix = vx % M, iy = (vx / M) % M, iz = vx / (M * M);
        const long long v = (long long)s_grad[(i & 3) * lm.plane + ix + iy * lm.sy + iz * lm.sz];
        if (v != 0 || !ok) {
          unsafeAtomicAdd(dst + i, (float)v * inv);
          ++n_nz;
        }
      }
    }
    __syncthreads();   // LDS is reused by the next item
  }
  if (counters) {
    const unsigned long long c[4] = {wave_sum_u64(n_visit), wave_sum_u64(n_rep), wave_sum_u64(n_run),
                                     wave_sum_u64(n_nz)};
    if (lane == 0 && (c[0] | c[1] | c[3])) {
#pragma unroll
      for (int i = 0; i < 4; ++i) atomicAdd(counter_slot(counters) + kCntBwdVisit + i, c[i]);
    }
  }
}

// Static LDS of k_bwd_items by its workgroup size: the tables' bytes, and the
// bound that room for the dynamic part is reckoned with.
constexpr size_t bwd_items_tables(int threads) {
  const size_t waves = threads / kWave, ent = threads == kSparseThreads ? kSparseEntries : kItemEntries, sub = 4 * ent;
  return 16 + kLenBuckets * 4 * (1 + 2 + 2 * waves) + waves * (64 + 4) + sub * (8 + 4) + 4 + sub / kWave * 4 + ent * (8 + 4) +
         64;   // (alignment)
}
constexpr size_t bwd_items_static(int threads) {
  return threads == kTileThreads ? 8 * 1024 : threads == kSparseThreads ? 10 * 1024 : 16 * 1024;
}
static_assert(bwd_items_tables(kTileThreads) <= bwd_items_static(kTileThreads) &&
              bwd_items_tables(2 * kTileThreads) <= bwd_items_static(2 * kTileThreads) &&
              bwd_items_tables(kSparseThreads) <= bwd_items_static(kSparseThreads), "static LDS of k_bwd_items");

// The work-item kernel for 3 waves per SIMD, 2 workgroups per CU, one of 512
// threads, one of 512 threads in slabs, or of 64 threads for sparse rays.
enum class BwdShape { kThree, kTwo, kOne, kSlabs, kSparse };
typedef void (*BwdItemsFn)(AccelView, const float *, const float *, const void *, const mvp_ray_aux *, const float4 *,
                           const RayConst *, const RayBound *, BwdOut, uint32_t, int, int, uint32_t, unsigned long long *);
template <bool B, bool L, bool F, Replay R>
static BwdItemsFn bwd_items_fn(BwdShape shape) {
  if (shape == BwdShape::kThree) return k_bwd_items<B, L, F, R, 3, kTileThreads>;
  if (shape == BwdShape::kSparse) return k_bwd_items<B, L, F, R, 1, kSparseThreads>;
  if constexpr (L) {
    if (shape == BwdShape::kSlabs) return k_bwd_items<B, L, F, R, 1, 2 * kTileThreads, true>;
    if (shape == BwdShape::kOne) return k_bwd_items<B, L, F, R, 1, 2 * kTileThreads>;
    return k_bwd_items<B, L, F, R, 1, kTileThreads>;
  }
  return nullptr;   // without the LDS copy three workgroups fit
}
template <bool B, bool L, bool F>
static BwdItemsFn bwd_items_fn(Replay r, BwdShape shape) {
  return r == Replay::kRuns ? bwd_items_fn<B, L, F, Replay::kRuns>(shape)
         : r == Replay::kRounded ? bwd_items_fn<B, L, F, Replay::kRounded>(shape) : bwd_items_fn<B, L, F, Replay::kLoop>(shape);
}
static BwdItemsFn bwd_items_fn(bool bf16, bool lds, bool fade, Replay r, BwdShape shape) {
  if (bf16)
    return lds ? (fade ? bwd_items_fn<true, true, true>(r, shape) : bwd_items_fn<true, true, false>(r, shape))
               : (fade ? bwd_items_fn<true, false, true>(r, shape) : bwd_items_fn<true, false, false>(r, shape));
  return lds ? (fade ? bwd_items_fn<false, true, true>(r, shape) : bwd_items_fn<false, true, false>(r, shape))
             : (fade ? bwd_items_fn<false, false, true>(r, shape) : bwd_items_fn<false, false, false>(r, shape));
}

// Whether the backward takes cell runs in closed form (bwd_pair).  Two lines:
// - at least 3 samples per voxel cell across the smallest box (7 for 4096 x 8^3
//   at 1/512: 1.6 times as fast as the sample loop; 10 for 512 x 16^3: 2.4
//   times; 2.7 for 32768 x 16^3 at 1/1024: equal);
// - no box smaller than 1/90 of its distance.  This line is for continuity, not
//   for speed or accuracy: the sample loop's sums of the rotation and scale
//   gradients run over camera distances, and their FP32 rounding grows with this
//   ratio (about 1.0e-5 of the gradient at 86, 2.2e-5 at 210) where the closed
//   form's does not (1e-6), so far from the camera its results would differ from
//   the sample loop's, which they have always had, by more than 2e-5.
bool backward_by_runs(const AccelView &av, int M) {
  const float cell = 2.0f / (av.max_inv_scale * (float)(M - 1));
  return cell >= 3.0f * av.step && av.max_dist_ratio <= 90.0f;
}

hipError_t launch_march_bwd(const AccelView &av, const mvp_prims &p, int64_t n_items_max,
                            const mvp_ray_aux *aux, const float *grad_rgba, const float *bg,
                            const float *rgba, void *scratch, float *g_pay, float *g_pos, float *g_rot,
                            float *g_scale, float *g_bg, unsigned long long *counters, bool clean, hipStream_t s,
                            hipEvent_t t0, hipEvent_t t1) {
  const size_t R = (size_t)av.n_slots;
  if (!clean) {
    hipError_t ez = launch_zero_counters(counters, kCntBwdVisit, 4, s);
    if (ez == hipSuccess) ez = launch_zero_counters(counters, kCntPayMax, 1, s);
    if (ez != hipSuccess) return ez;
  }
  if (R == 0) return hipSuccess;
  RayConst *rc = (RayConst *)scratch;
  RayBound *rbd = (RayBound *)(rc + R);
  uint32_t *pmax = (uint32_t *)(counters + kCntPayMax), *odd = (uint32_t *)(counters + kCntOdd);
  const bool bf16 = p.payload_dtype == MVP_BF16;
  const bool fade = av.fade_alpha > 0.f;
  const size_t fade_shm = fade ? (size_t)p.M * sizeof(float) : 0;
  hipError_t e = hipSuccess;
  const size_t n_vox = (size_t)p.n_prim * p.M * p.M * p.M;
  if (n_vox) {
    const unsigned pg = (unsigned)std::min<size_t>((n_vox + 255) / 256, 1024);
    if (bf16)
      hipLaunchKernelGGL((k_payload_bound<true>), dim3(pg), dim3(256), 0, s, p.payload, n_vox, pmax, odd);
    else
      hipLaunchKernelGGL((k_payload_bound<false>), dim3(pg), dim3(256), 0, s, p.payload, n_vox, pmax, odd);
  }
  const unsigned rb = (unsigned)((R + kBwdRaysPerBlock - 1) / kBwdRaysPerBlock);
#define MVP_RAYS(B, F)                                                                                        \
  hipLaunchKernelGGL((k_bwd_rays<B, F>), dim3(rb), dim3(256), fade_shm, s, av, p.payload, aux,               \
                     (const float4 *)grad_rgba, bg, (const float4 *)rgba, rc, rbd, pmax, odd, g_bg, R)
  if (bf16) {
    if (fade) MVP_RAYS(true, true); else MVP_RAYS(true, false);
  } else {
    if (fade) MVP_RAYS(false, true); else MVP_RAYS(false, false);
  }
#undef MVP_RAYS
  e = hipGetLastError();
  if (e != hipSuccess || p.n_prim == 0 || n_items_max == 0) return e;
  // the planar 64-bit LDS gradient, when one workgroup's copy fits a CU; its
  // padded layout unless only the packed one fits
  const size_t kStatic = bwd_items_static(kTileThreads), kStaticWide = bwd_items_static(2 * kTileThreads);
  auto lds_bytes = [&](bool pad) { return (size_t)lds_map(p.M, pad).plane * 4 * sizeof(unsigned long long); };
  const int padded = lds_bytes(true) + fade_shm + kStaticWide <= 160 * 1024 ? 1 : 0;
  size_t lds = lds_bytes(padded != 0);
  bool in_lds = g_pay && lds + fade_shm + kStaticWide <= 160 * 1024;
  // A larger payload (up to 45^3): slabs of as many cell layers as fit beside
  // the ordering buffer of 4096 pairs, each replaying the samples in it; every
  // pair is set up once per slab (11 of 3 layers for 32^3), but adds to the LDS.
  // Device atomics in their place, 32 per cell run, ran at 46 G/s: 64 x 32^3 at
  // 667 x 1024 48.4 ms against 3.4; items of few pairs are left to them (k_item_split).
  int slab_cells = 0;
  // The items' length was chosen at the build, for its payload size and way
  // through a pair; this call's payload may be of another size.  Items of more
  // than kItemEntries entries only fit the tables of the shape for sparse rays,
  // which takes any payload and either way, but no slabs.
  const bool sparse = av.item_entries > kItemEntries;
  if (g_pay && !in_lds && !sparse) {
    const size_t layer = (size_t)p.M * p.M * 4 * sizeof(unsigned long long);
    const int layers = (int)((160 * 1024 - kStaticWide - fade_shm - 4096 * 3 - 64) / layer);
    if (layers >= 2) {
      const int n_slab = (p.M - 2 + layers - 1) / (layers - 1);
      slab_cells = (p.M - 2 + n_slab) / n_slab;
      lds = ((size_t)p.M * p.M * (slab_cells + 1) + 1) * 4 * sizeof(unsigned long long);
      in_lds = true;
    }
  }
  auto wgs_per_cu = [&](size_t grad) {
    for (int w = 3; w > 1; --w)
      if ((size_t)w * (grad + fade_shm + kStatic) <= 160 * 1024) return w;
    return 1;
  };
  // 3 waves per SIMD when 3 workgroups' LDS fits a CU; 512-thread workgroups
  // when only one does (16^3 payloads: 131 KB)
  const int wgs_fit = in_lds ? wgs_per_cu(lds) : 3;
  BwdShape shape = sparse ? BwdShape::kSparse : slab_cells ? BwdShape::kSlabs : wgs_fit >= 3 ? BwdShape::kThree : wgs_fit == 2 ? BwdShape::kTwo : BwdShape::kOne;
  auto wide = [&] { return shape == BwdShape::kOne || shape == BwdShape::kSlabs; };
  const int64_t n_slab = slab_cells ? (p.M - 2 + slab_cells) / slab_cells : 1;
  // items of few pairs are left out of the slabs where there may be many of them
  uint32_t n_list = n_items_max * n_slab > kSlabsAtLeast && slab_cells ? (uint32_t)n_items_max : 0u;
  const unsigned grid = (unsigned)std::min<int64_t>(n_items_max * n_slab, n_list ? kSlabGrid : 1 << 20);
  BwdOut out{g_pay, g_pos, g_rot, g_scale};
  size_t shm = (in_lds ? lds : 0) + fade_shm;
  // the pair-ordering buffer takes what is left of the LDS share of a
  // workgroup at the occupancy chosen above (items with more pairs than it
  // holds keep their pairs in list order)
  uint32_t sort_cap = 0;
  if (kSortPairs) {
    const size_t fixed = bwd_items_static(sparse ? kSparseThreads : wide() ? 2 * kTileThreads : kTileThreads);
    const size_t wgs = shape == BwdShape::kThree ? 3 : (shm + fixed <= 80 * 1024 ? 2 : 1);
    const size_t share = 160 * 1024 / wgs - fixed;
    const size_t room = share > shm ? (share - shm) / (sizeof(uint16_t) + 1) : 0;
    const size_t want = sparse ? kSparseSort : (size_t)av.item_entries * kTileThreads;
    sort_cap = (uint32_t)(std::min(room, want) / kTileThreads * kTileThreads);
    shm += (size_t)sort_cap * (sizeof(uint16_t) + 1);
  }
  int exponent;
  const Replay runs = !backward_by_runs(av, p.M) ? Replay::kLoop
                      : std::frexp(av.step, &exponent) == 0.5f ? Replay::kRuns : Replay::kRounded;
  BwdItemsFn fn = bwd_items_fn(bf16, in_lds, fade, runs, shape);
  if (shm > 64 * 1024) {
    // allow more than the default dynamic LDS per workgroup (gfx950 has 160 KB)
    if (hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) != hipSuccess) {
      (void)hipGetLastError();
      // gradients straight to device memory, pairs in list order
      shape = sparse ? BwdShape::kSparse : BwdShape::kThree;
      slab_cells = 0;
      n_list = 0;
      sort_cap = 0;
      shm = fade_shm;
      fn = bwd_items_fn(bf16, false, fade, runs, shape);
    }
  }
  if (t0) (void)hipEventRecord(t0, s);
  if (slab_cells) {
    const uint32_t few = (uint32_t)std::min<int64_t>(20 + 4 * n_slab, 100);
    if (n_list)
      hipLaunchKernelGGL(k_item_split, dim3((unsigned)((n_items_max + kWave - 1) / kWave)), dim3(kWave), 0, s, av, few, n_list);
    hipLaunchKernelGGL(bwd_items_fn(bf16, false, fade, runs, BwdShape::kThree),
                       dim3((unsigned)std::min<int64_t>(n_items_max, kSlabGrid)), dim3(kTileThreads),
                       fade_shm + kTileThreads * (sizeof(uint16_t) + 1), s, av, p.rot, p.scale, p.payload, aux,
                       (const float4 *)grad_rgba, rc, rbd, out, (uint32_t)kTileThreads, 0, slab_cells, n_list, counters);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, dim3(grid), dim3(sparse ? kSparseThreads : wide() ? 2 * kTileThreads : kTileThreads), shm, s, av, p.rot, p.scale, p.payload,
                     aux, (const float4 *)grad_rgba, rc, rbd, out, sort_cap, padded, slab_cells, n_list, counters);
  e = hipGetLastError();
  if (t1) (void)hipEventRecord(t1, s);
  return e;
}

// Entries per backward work item.
//
// Up to 8^3: 32.  The scale of the 30-bit sums follows the item's largest pair,
// so a longer item leaves the others fewer bits, and it is no faster either (4096 of
// them at 4 x 1024^2: a step of 12.36 ms with 32, 12.47 with 64; at 667 x 1024 the
// backward takes 690 us with both and 699 with 16).
//
// To 16^3 with closed-form runs: a long item zeroes and flushes its primitive's
// gradient less often, but where there are few primitives, long items leave
// workgroups idle at the end (512 of 16^3, 56 entries each, one workgroup per CU:
// 1953 us with 64 entries, 1625 with 32, 1315 with 16, 1388 with 8).  So an item
// takes 64 entries, or fewer, down to 16, where that is under 8 items for each CU.
//
// Sparse rays (n_slots, the rays of all entries' tiles, few per entry) leave
// most of 256 threads without a pair: 128 entries for 64 threads, of which
// more workgroups fit a CU, up to 8 rays per entry (4096 x 8^3: 1 ray 247 against
// 518 us, 4 rays 363 against 563, 6 rays 448 against 577, 8 rays 603 and 597), to
// 10^3 with fewer workgroups per CU up to 5 (1 ray 411 against 610, 4 rays 581
// against 663, 6 rays 708 against 679); larger ones leave room for three or less.
//
// The sample loop keeps items of fixed length, 32 entries to 8^3 and 64 to 16^3:
// the rounding of its pose sums depends on how they are grouped (see
// backward_by_runs), and the largest case is fastest at 64 (32768 of 16^3: 28.3
// ms with 32, 27.4 with 64).  Payloads taken in slabs have items of at most 4096
// pairs, the ordering buffer's size beside a slab (64 of 32^3: 3.6 ms with 16
// entries, 4.8 with 8 or 32).  Larger ones, in device memory, take 16 too (8 x 64^3 at
// 667 x 1024: 24 ms, 59 with 64 and the sample loop).
int backward_item_entries(const AccelView &av, int M, uint64_t n_entries, uint64_t n_slots) {
  if (M > 16) return 16;
  if (!backward_by_runs(av, M)) return M <= 8 ? 32 : kItemEntries;
  if (M <= kSparseMaxM && n_slots < (M <= 8 ? 8 : 5) * n_entries) return kSparseEntries;
  if (M <= 8) return 32;
  int n = kItemEntries;
  while (n > 16 && n_entries / n + (uint64_t)av.N < 8 * 256) n /= 2;
  return n;
}

}  // namespace mvp
