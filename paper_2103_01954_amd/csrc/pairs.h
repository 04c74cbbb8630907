// The per-ray pair lists of one screen tile: the canonical FP32 geometry
// (slab test, sample intervals) and the per-tile pairs pass of the pairs kernel.
//
// Built with -ffp-contract=off and IEEE division/square root: every written
// float operation below is exactly one binary32 operation, so the hit
// decisions and sample intervals are reproducible bit for bit.
#pragma once

#include <climits>

#include "internal.h"

namespace mvp {

// ---------------------------------------------------------------------------
// canonical FP32 geometry (one rounding per written operation)
// ---------------------------------------------------------------------------

// Slab test of the local ray y(t) = a + t b against [-1,1]^3, clipped to t >= t_near.
// An axis with b_i = 0 excludes the ray if a_i lies outside [-1, 1] and
// otherwise does not constrain t.  Written without branches (the quotients of
// a zero b_i are computed and discarded), so the three axes' correctly rounded
// divisions are independent and can overlap.
__device__ inline bool slab_test(const float a[3], const float b[3], float t_near, float *t_in,
                                 float *t_out) {
  float lo = t_near, hi = INFINITY;
  bool miss = false;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float n0 = -1.0f - a[i];
    const float n1 = 1.0f - a[i];
    const float q0 = n0 / b[i];
    const float q1 = n1 / b[i];
    const bool par = b[i] == 0.0f;
    lo = par ? lo : fmaxf(lo, fminf(q0, q1));
    hi = par ? hi : fminf(hi, fmaxf(q0, q1));
    miss = miss || (par && !(a[i] >= -1.0f && a[i] <= 1.0f));
  }
  *t_in = lo;
  *t_out = hi;
  return !miss && lo <= hi;
}

__device__ inline float sample_pos(int j, float dt) { return (float)j * dt; }

// smallest j >= 0 with fl(j dt) >= t (kJMax + 1 if none)
__device__ inline int first_sample_not_before(float t, float dt) {
  const float q = t / dt;
  int j;
  if (!(q <= 16777216.0f)) {
    j = kJMax + 1;
  } else {
    float c = ceilf(q);
    j = c < 0.0f ? 0 : (int)c;
  }
  for (int it = 0; it < 4 && j > 0 && sample_pos(j - 1, dt) >= t; ++it) --j;
  for (int it = 0; it < 4 && j <= kJMax && sample_pos(j, dt) < t; ++it) ++j;
  return j;
}

// largest j <= kJMax with fl(j dt) <= t (-1 if none)
__device__ inline int last_sample_not_after(float t, float dt) {
  const float q = t / dt;
  int j;
  if (!(q < 16777215.0f)) {
    j = (q == q) ? kJMax : -1;
  } else {
    float f = floorf(q);
    j = f < -1.0f ? -1 : (int)f;
  }
  for (int it = 0; it < 4 && j < kJMax && sample_pos(j + 1, dt) <= t; ++it) ++j;
  for (int it = 0; it < 4 && j >= 0 && sample_pos(j, dt) > t; ++it) --j;
  return j;
}

// Correctly rounded n / b from a reciprocal kept for several numerators
// (Markstein's method): Newton's step on the hardware's reciprocal, then the
// quotient corrected twice by its exact residual.  These are the very steps of
// the compiler's division without its scaling, which does nothing while both
// operands lie within 2^-40 .. 2^40.
constexpr float kDivLo = 0x1p-40f, kDivHi = 0x1p40f;
__device__ __forceinline__ float refined_rcp(float b) {
  const float r = __builtin_amdgcn_rcpf(b);
  return __builtin_fmaf(__builtin_fmaf(-b, r, 1.0f), r, r);
}
__device__ __forceinline__ float div_with(float n, float b, float r) {
  const float q = n * r;
  const float q1 = __builtin_fmaf(__builtin_fmaf(-b, q, n), r, q);
  return __builtin_fmaf(__builtin_fmaf(-b, q1, n), r, q1);
}

// The slab test and, of a ray that hits, the first and last sample in the box:
// the results of slab_test and the two functions above.  The quotients of an
// axis come from one reciprocal, without the cases of a ray parallel to an axis
// and without scaling, where every lane's operands allow it (those of a NaN are
// NaN either way).  The sample numbers come from t times the reciprocal rdt of
// the step, and are checked against their definition; only if a lane's fails
// (its quotient is within rounding of a whole number) are they searched for.
__device__ __forceinline__ bool ray_samples(const float a[3], const float b[3], float t_near, float dt, float rdt,
                                            int *jlo, int *jhi) {
  float n[6], mn = INFINITY, mx = 0.f;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    n[2 * i] = -1.0f - a[i];
    n[2 * i + 1] = 1.0f - a[i];
    mn = fminf(fminf(mn, fabsf(b[i])), fminf(fabsf(n[2 * i]), fabsf(n[2 * i + 1])));
    mx = fmaxf(fmaxf(mx, fabsf(b[i])), fmaxf(fabsf(n[2 * i]), fabsf(n[2 * i + 1])));
  }
  float lo = t_near, hi = INFINITY;
  bool hit;
  if (__ballot(!(mn >= kDivLo && mx <= kDivHi)) == 0ull) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const float r = refined_rcp(b[i]);
      const float q0 = div_with(n[2 * i], b[i], r);
      const float q1 = div_with(n[2 * i + 1], b[i], r);
      lo = fmaxf(lo, fminf(q0, q1));
      hi = fminf(hi, fmaxf(q0, q1));
    }
    hit = lo <= hi;
  } else {
    hit = slab_test(a, b, t_near, &lo, &hi);
  }
  if (hit) {   // 0 <= lo <= hi
    const float c = ceilf(lo * rdt), f = floorf(hi * rdt);   // exact as floats below 2^23
    const bool good = f < 8388608.0f && (c - 1.0f) * dt < lo && c * dt >= lo && (f + 1.0f) * dt > hi && f * dt <= hi;
    if (__ballot(!good) == 0ull) {
      *jlo = (int)c;
      *jhi = (int)f;
    } else {
      *jlo = first_sample_not_before(lo, dt);
      *jhi = last_sample_not_after(hi, dt);
    }
    hit = *jlo <= *jhi;
  }
  return hit;
}

// One workgroup per screen tile, one thread per pixel.  The tile's culling
// list is staged through LDS in chunks of kStage primitives: the rows of A,
// each with its coordinate of the local ray origin a = A (o - t), which is the
// same for every ray of a view.
struct Staged {
  float4 row[kStage][3];
  int32_t id[kStage];
};

__device__ inline void stage_chunk(Staged &sm, const AccelView &av, const DevCam &cam, uint64_t lb,
                                   int cnt) {
  const int e = threadIdx.x;
  if (e < cnt) {
    const int k = (int)av.tile_list[lb + e];
    float4 r[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) r[i] = av.xf[3 * (size_t)k + i];
    const float p[3] = {cam.o[0] - r[0].w, cam.o[1] - r[1].w, cam.o[2] - r[2].w};
#pragma unroll
    for (int i = 0; i < 3; ++i) sm.row[e][i] = make_float4(r[i].x, r[i].y, r[i].z, row_dot(r[i].x, r[i].y, r[i].z, p));
    sm.id[e] = k;
  }
}

// Local ray y(t) = a + t b of staged entry e for direction d.
__device__ __forceinline__ void local_ray(const Staged &sm, int e, const float d[3], float a[3], float b[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float4 r = sm.row[e][i];
    a[i] = r.w;
    b[i] = row_dot(r.x, r.y, r.z, d);
  }
}

// Conservative test of a pixel block against a staged entry: can the ray
// through any pixel centre of the block hit the entry's box?  The unnormalised
// directions e(u, v) = P (u, v, 1) of the block's pixel centres span the
// parallelogram of its four corner directions, so their local directions
// A e lie, componentwise, within the bounds [bl, bh] of the four corners' A e.
// A ray that hits at some t >= 0 meets, with that t, a + t bl <= 1 and
// a + t bh >= -1 on every axis (positive scaling of the direction changes no
// hit), so an empty intersection of those t-intervals excludes the whole
// block.  The bounds are widened by far more than the rounding of the per-ray
// canonical test and of this one (the box by 1e-5 (1 + max |a|), the direction
// bounds by 1e-5 |A_i|_1 max |e|), and anything non-finite never excludes.
__device__ __forceinline__ bool block_may_hit(const Staged &sm, int e, const float (*E)[3], float emax) {
  float a[3], bl[3], bh[3], amax = 0.f;
  bool sane = true;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float4 r = sm.row[e][i];
    a[i] = r.w;
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float b = r.x * E[c][0] + r.y * E[c][1] + r.z * E[c][2];
      lo = fminf(lo, b);
      hi = fmaxf(hi, b);
    }
    const float eta = 1e-5f * (fabsf(r.x) + fabsf(r.y) + fabsf(r.z)) * emax;
    bl[i] = lo - eta;
    bh[i] = hi + eta;
    amax = fmaxf(amax, fabsf(a[i]));
    sane = sane && fabsf(bl[i]) < 1e30f && fabsf(bh[i]) < 1e30f;
  }
  const float lim = 1.0f + 1e-5f * (1.0f + amax);
  float lo = 0.0f, hi = INFINITY;
  bool ok = true;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float nu = lim - a[i];    // a + t bl <= lim
    const float tu = nu * __builtin_amdgcn_rcpf(bl[i]);
    hi = bl[i] > 0.0f ? fminf(hi, tu) : hi;
    lo = bl[i] < 0.0f ? fmaxf(lo, tu) : lo;
    ok = ok && !(bl[i] == 0.0f && nu < 0.0f);
    const float nl = -lim - a[i];   // a + t bh >= -lim
    const float tl = nl * __builtin_amdgcn_rcpf(bh[i]);
    hi = bh[i] < 0.0f ? fminf(hi, tl) : hi;
    lo = bh[i] > 0.0f ? fmaxf(lo, tl) : lo;
    ok = ok && !(bh[i] == 0.0f && nl > 0.0f);
  }
  return !(sane && amax < 1e30f) || (ok && !(lo > hi));
}

// The pairs of one screen tile, computed by a workgroup of kTileThreads
// threads, one per ray (every thread must call it: it has barriers).  The tile's
// culling list (ordered near to far) is staged through LDS in chunks of
// kStage entries; every ray runs the canonical slab test against each staged
// entry, and each pair with at least one sample is inserted into the ray's
// slots in (jlo, primitive id) order.  The list order leaves few pairs out of
// place, and those only by a few places, so the ray keeps its last kTail
// pairs sorted in registers and writes the first of them to device memory when
// one more arrives; a pair that belongs before the written ones moves those
// up by one.  The same pair is listed under its entry: the rays of each wave
// that hit the entry are ranked by a ballot into the wave's 64 slots of the
// entry's list (unless ent_n is null: a structure for the forward only).  A
// wave's rays are an 8 x 8 block of pixels (about 7% fewer entries than with 16 x 4; those are
// kept for a backward by the sample loop, whose sums' rounding depends on the
// order of the pairs), and its lanes first test the staged
// entries, one each, against that block (block_may_hit): the wave then walks
// only the entries that one of its rays may hit, about half of a list.
//
// Bound by instructions where the chip is full and by the chain of one entry
// after another where it is not, so what counts is the instructions per entry
// and wave.  16384 x 8^3 at 512^2: 225 us (453 with waves of 16 x 4 pixels that
// pass over the entries they skip, six full divisions per slab test, searched
// sample numbers and a tail of counted length), 4096 x 8^3 at 4 x 1024^2 397
// (770), 512 x 16^3 at 256^2 52 (109).
constexpr int kTail = 4;

__device__ __forceinline__ bool pair_before(const int4 &a, const int4 &b) {
  return a.x < b.x || (a.x == b.x && a.w < b.w);
}

// The pairs of a tile with few rays (of a ray subset) and at most kStage
// entries, staged in sm, by one wave: ray after ray, one lane per entry.  A hit's
// place in its ray's list is the number of hits before it.  16384 rays over
// 16384 tiles of 21 entries: 115 us, 380 with one lane per ray.
__device__ inline uint32_t sparse_tile_pairs(const Staged &sm, const AccelView &av, int tile, const PairsOut &o,
                                             uint64_t lb, int len, int rays, uint64_t pbase, float rdt) {
  constexpr int kBlocks = kStage / kWave;
  const int lane = threadIdx.x;
  uint32_t cnt[kBlocks], total = 0;   // hits of this lane's entries so far
#pragma unroll
  for (int q = 0; q < kBlocks; ++q) cnt[q] = 0;
  for (int t = 0; t < rays; ++t) {
    int v, px, py;
    size_t ray;
    (void)tile_ray(av, tile, t, &ray, &v, &px, &py);
    float d[3];
    pixel_ray(av.cams[v], px, py, d);
    int jlo[kBlocks], jhi[kBlocks], id[kBlocks];
    uint32_t rank[kBlocks], n = 0;
    unsigned long long m[kBlocks];
#pragma unroll
    for (int q = 0; q < kBlocks; ++q) {
      const int e = min(q * kWave + lane, len - 1);
      float a[3], b[3];
      jlo[q] = jhi[q] = 0;
      rank[q] = 0;
      m[q] = 0;
      id[q] = sm.id[e];
      if (q * kWave < len) {   // the same for every lane
        local_ray(sm, e, d, a, b);
        const bool hit = ray_samples(a, b, av.t_near, av.step, rdt, &jlo[q], &jhi[q]);
        m[q] = __ballot(hit && q * kWave + lane < len);
      }
      n += (uint32_t)__popcll(m[q]);
    }
#pragma unroll
    for (int p = 0; p < kBlocks; ++p)
      for (unsigned long long todo = m[p]; todo; todo &= todo - 1) {
        const int k = __builtin_ctzll(todo);
        const int sj = __builtin_amdgcn_readlane(jlo[p], k), si = __builtin_amdgcn_readlane(id[p], k);
#pragma unroll
        for (int q = 0; q < kBlocks; ++q) rank[q] += (sj < jlo[q] || (sj == jlo[q] && si < id[q])) ? 1u : 0u;
      }
#pragma unroll
    for (int q = 0; q < kBlocks; ++q)
      if ((m[q] >> lane) & 1ull) {
        const int e = q * kWave + lane;
        o.pr[pbase + (uint64_t)t + (uint64_t)rank[q] * (uint64_t)rays] = make_int4(jlo[q], jhi[q], e, id[q]);
        if (rank[q] == 0) o.ray_nj[ray] = make_int2((int)n, jlo[q]);
        if (o.ent_n)
          o.ent_rec[pbase + (uint64_t)e * (uint64_t)rays + cnt[q]] = make_uint2((uint32_t)jlo[q] | ((uint32_t)t << 24), (uint32_t)jhi[q]);
        ++cnt[q];
      }
    if (lane == 0) {
      o.ray_seg[ray] = pbase + (uint64_t)t;
      if (n == 0) o.ray_nj[ray] = make_int2(0, INT_MAX);
    }
    total += n;
  }
  if (o.ent_n) {
#pragma unroll
    for (int q = 0; q < kBlocks; ++q)
      if (q * kWave + lane < len)
        ((uint4 *)o.ent_n)[lb + (uint64_t)(q * kWave + lane)] = make_uint4(cnt[q], 0u, 0u, 0u);
  }
  return total;
}

template <bool SUBSET>
__device__ inline void tile_pairs(const AccelView &av, int tile, const PairsOut &o) {
  __shared__ Staged sm;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // the ray of this thread: its number in the tile
  const bool square = !SUBSET && o.square;
  const int x0 = square ? (wave & 1) * 8 : 0, y0 = square ? (wave >> 1) * 8 : SUBSET ? 0 : wave * (kWave / kTile);
  const int t = square ? (y0 + (lane >> 3)) * kTile + x0 + (lane & 7) : (int)threadIdx.x;
  const uint64_t lb = av.tile_off[tile], le = av.tile_off[tile + 1];
  const uint64_t len = le - lb;
  const uint64_t rays = SUBSET ? av.tile_ray_off[tile + 1] - av.tile_ray_off[tile] : (uint64_t)kTileThreads;
  // read once: a load inside the entry loop would wait for all of the wave's
  // earlier stores (the wait counter counts stores too)
  const uint64_t pbase = av.pair_base[tile];
  const float rdt = 1.0f / av.step;
  // Few rays for the length of the list: one lane per entry instead of one per
  // ray.  The one takes rays x blocks of 64 entries in turn, the other the
  // entries, each in about a quarter of the time (no ranks of the hits to count).
  // 4096 x 8^3 in one 1024^2 view, 64 rays a tile: 116 us, 342 with the line at
  // rays x blocks = len (a wave took 64 rays in turn), 227 with one lane per ray
  // throughout; 16 rays a tile 98, 155 and 201 us, 4 rays 85, 83 and 193 us.
  constexpr uint32_t kRayCost = 4;
  const bool sparse = SUBSET && len <= kStage && rays <= kWave &&
                      kRayCost * (uint32_t)rays * (((uint32_t)len + kWave - 1) / kWave) <= (uint32_t)len;
  int v, px, py;
  size_t ray;
  const bool valid = tile_ray(av, tile, t, &ray, &v, &px, &py);
  const DevCam &cam = av.cams[tile / (av.tiles_x * av.tiles_y)];
  // corner directions of the wave's pixel block (a ray subset: of the tile)
  float E[4][3], emax = 0.f;
  if (!sparse) {
    const int x1 = x0 + (square ? 8 : kTile) - 1, y1 = y0 + (square ? 8 : SUBSET ? kTile : kWave / kTile) - 1;
    const int T = av.tiles_x * av.tiles_y, tt = tile % T;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float u = (float)((tt % av.tiles_x) * kTile + ((c & 1) ? x1 : x0)) + 0.5f;
      const float w = (float)((tt / av.tiles_x) * kTile + ((c & 2) ? y1 : y0)) + 0.5f;
      float nrm = 0.f;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        E[c][i] = cam.P[3 * i] * u + cam.P[3 * i + 1] * w + cam.P[3 * i + 2];
        nrm = fmaxf(nrm, fabsf(E[c][i]));
      }
      emax = fmaxf(emax, nrm * 1.7320508f);   // bounds |e| of the corner directions
    }
  }
  float d[3];
  pixel_ray(cam, px, py, d);
  const bool lists = o.ent_n != nullptr;   // the per-entry lists (for the backward) are wanted
  const bool any = __ballot(valid) != 0ull;
  const uint64_t seg = pbase + (uint64_t)t;   // pair q at seg + q * rays
  const unsigned long long lt = (1ull << lane) - 1ull;
  int nw = 0;         // pairs written to device memory, in order
  int nh = 0;         // pairs so far
  int first = INT_MAX;
  int4 tb[kTail];     // the last pairs, sorted, all after the written ones (jlo < 0: none yet)
#pragma unroll
  for (int q = 0; q < kTail; ++q) tb[q] = make_int4(-1, 0, 0, 0);
  int4 wl = make_int4(-1, 0, 0, 0);   // the last written pair (its key)
  for (uint64_t c0 = lb; c0 < le; c0 += kStage) {
    const int nc = (int)min<uint64_t>(kStage, le - c0);
    __syncthreads();
    stage_chunk(sm, av, cam, c0, nc);
    if ((int)threadIdx.x < nc) {   // the entry's frame and where its pair list goes
      const int e = threadIdx.x;
      const uint64_t g = c0 + e;
#pragma unroll
      for (int r = 0; r < 3; ++r) o.ef[3 * g + r] = sm.row[e][r];
      if (lists) {
        o.ent_base[g] = pbase + (g - lb) * rays;
        o.ent_tile[g] = (uint32_t)tile;
      }
    }
    __syncthreads();
    if (sparse) {
      if (wave == 0) {
        const uint32_t n = sparse_tile_pairs(sm, av, tile, o, lb, nc, (int)rays, pbase, rdt);
        if (lane == 0 && n) atomicAdd(counter_slot(o.counters) + kCntPairs, (unsigned long long)n);
      }
      return;
    }
    for (int b0 = 0; b0 < nc; b0 += kWave) {
      unsigned long long may = 0;   // entries of this block that a ray of the wave may hit
      if (any) may = __ballot(block_may_hit(sm, min(b0 + lane, nc - 1), E, emax) && b0 + lane < nc);
      uint32_t cnt = 0;             // lane k: hits of entry b0 + k
      while (may) {
        const int k = __builtin_ctzll(may), e = b0 + k;
        may &= may - 1;
        const uint64_t g = c0 + e;
        float a[3], b[3];
        int jlo = 0, jhi = 0;
        local_ray(sm, e, d, a, b);
        const bool hit = ray_samples(a, b, av.t_near, av.step, rdt, &jlo, &jhi) && valid;
        const unsigned long long m = __ballot(hit);
        if (lane == k) cnt = (uint32_t)__popcll(m);
        if (hit) {
          const int4 rec = make_int4(jlo, jhi, (int)(g - lb), sm.id[e]);
          ++nh;
          first = min(first, jlo);
          if (pair_before(rec, wl)) {
            // before every written pair still after it: those move up by one
            int at = nw;
            while (at > 0) {
              const int4 p = o.pr[seg + (uint64_t)(at - 1) * rays];
              if (!pair_before(rec, p)) break;
              o.pr[seg + (uint64_t)at * rays] = p;
              --at;
            }
            o.pr[seg + (uint64_t)at * rays] = rec;
            ++nw;
          } else {   // into the tail; the first of the kTail + 1 pairs is final among the written ones
            int4 x = rec;
#pragma unroll
            for (int q = kTail - 1; q >= 0; --q) {
              const int4 y = tb[q];
              const bool below = pair_before(x, y);
              tb[q] = make_int4(below ? y.x : x.x, below ? y.y : x.y, below ? y.z : x.z, below ? y.w : x.w);
              x = make_int4(below ? x.x : y.x, below ? x.y : y.y, below ? x.z : y.z, below ? x.w : y.w);
            }
            if (x.x >= 0) {
              o.pr[seg + (uint64_t)nw * rays] = x;
              wl = x;
              ++nw;
            }
          }
          if (lists)
            o.ent_rec[pbase + (g - lb) * rays + (uint64_t)wave * kWave + (uint32_t)__popcll(m & lt)] =
                make_uint2((uint32_t)jlo | ((uint32_t)t << 24), (uint32_t)jhi);
        }
      }
      if (lists && b0 + lane < nc) o.ent_n[4 * (c0 + (uint64_t)(b0 + lane)) + wave] = cnt;
    }
  }
#pragma unroll
  for (int q = 0; q < kTail; ++q)
    if (tb[q].x >= 0) o.pr[seg + (uint64_t)(nw++) * rays] = tb[q];
  if (valid) {
    o.ray_seg[ray] = seg;
    o.ray_nj[ray] = make_int2(nh, first);
  }
  const unsigned long long c = wave_sum_u64((unsigned long long)nh);
  if (lane == 0 && c) atomicAdd(counter_slot(o.counters) + kCntPairs, c);
}


}  // namespace mvp
