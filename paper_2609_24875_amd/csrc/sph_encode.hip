// Spherical encoder and codebook initialisation on the device (Sec. 3.1, Eq. 3 and 5-7;
// Sec. 4.1 for the k-means settings).
//
// Every decision is the fp64 one, from fp32 weights, so that each integer (a direction index, a radius
// level, a sampled vector) is the one a plain fp64 implementation of the equations takes. Sums whose
// order fixes the bits of a stored value (the squared radius, the least-squares radius of Eq. 6, the
// norm of a k-means centre) use the pairwise order ((p0+p1)+(p2+p3))+((p4+p5)+(p6+p7)) with the
// products rounded first, never fused. Every reduction runs in a fixed order or on integers, so
// repeated calls give bitwise identical results.
//
// Work layout:
//   Eq. 5 search a wave takes 64 vectors (or samples); the matrix cores score them against all
//                entries within a known error, and only entries within that error of the best are
//                compared in fp64 (see scan_entries, nearest_of and nearest_small).
//   encoder      16 neighbouring lanes form one 128-weight group; the fp16 codebook sits in LDS.
//   k-means      squared radii and their running sum (three-pass scan), inverse-CDF sampling by
//                binary search, then per iteration: assignment (the centre range split over
//                workgroups, splits combined in ascending order) and a count per centre, the
//                samples listed by centre, and one workgroup per centre that adds its samples in
//                exact fixed point (integers, so the order of the list does not matter) and
//                renormalises.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "sph_fp.h"
#include "sph_host.h"
#include "sph_layout.h"

namespace {

constexpr double kEps = 1e-12;  // Eq. 3's guard against a zero radius
constexpr int kThreads = 256;
constexpr int kScanItems = 8;    // vectors per thread in the radius scan
constexpr int kScanBlock = kThreads * kScanItems;

// Pairwise sum of the eight rounded products a[j] * b[j].
__device__ __forceinline__ double dot8_pairwise(const double* a, const double* b) {
#pragma clang fp contract(off)
  double p[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) p[j] = a[j] * b[j];
  return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
}

// Eq. 3's unit direction a / max(||a||, eps) of magnitudes a. Returns the radius.
__device__ __forceinline__ double unit_direction(const double a[8], double d[8]) {
#pragma clang fp contract(off)
  const double r = sqrt(dot8_pairwise(a, a));
  const double rr = r < kEps ? kEps : r;
#pragma unroll
  for (int j = 0; j < 8; ++j) d[j] = a[j] / rr;
  return r;
}

// Eq. 3 on one fp32 vector: magnitudes |w_j| (w_+), sign bits (set where w_j < 0) and the
// unit direction w_+ / max(||w||, eps). Returns the radius.
__device__ __forceinline__ double decompose(const float* __restrict__ w, int64_t ldw, int64_t nv, int64_t i,
                                            double a[8], double d[8], uint32_t& neg) {
#pragma clang fp contract(off)
  const int64_t row = i / nv, v = i - row * nv;
  const float4* p = reinterpret_cast<const float4*>(w + row * ldw + v * 8);
  const float4 x0 = p[0], x1 = p[1];
  const float f[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
  neg = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    neg |= (f[j] < 0.0f ? 1u : 0u) << j;
    a[j] = fabs((double)f[j]);
  }
  return unit_direction(a, d);
}

// ------------------------------------------------------------------------------------ Eq. 5

typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));

// A unit direction times kUp as two fp16 words per pair of coordinates, hi + lo up to 2^-22 of a coordinate or, where
// fp16 ends, 2^-25 (2^-40 of the unit direction: unscaled it would be 2^-25, which an entry's coordinate of
// 6e4 made 2e-3 of a score).
constexpr float kUp = 0x1p15f, kSlack = 1e-5f * kUp;

struct DirWords {
  uint32_t hi[4], lo[4];
};

__device__ __forceinline__ DirWords split_dir(const float (&d)[8]) {
  DirWords w;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // taken as they are: folded into the product that made them, the two uses of hi could be
    // rounded differently (once from the product, or by way of fp32)
    float x = d[2 * i], y = d[2 * i + 1];
    asm("" : "+v"(x), "+v"(y));
    h2v h, l;
    h[0] = (_Float16)x;
    h[1] = (_Float16)y;
    l[0] = (_Float16)(x - (float)h[0]);
    l[1] = (_Float16)(y - (float)h[1]);
    w.hi[i] = __builtin_bit_cast(uint32_t, h);
    w.lo[i] = __builtin_bit_cast(uint32_t, l);
  }
  return w;
}

// (x, y) of the wave -> x = {lower half of x, lower half of y}, y = {upper half of x, upper half of y}.
__device__ __forceinline__ void swap_halves(uint32_t& x, uint32_t& y) {
  const bool low = (threadIdx.x & 32) == 0;
  const uint32_t o = __shfl_xor(low ? y : x, 32, 64);
  if (low) y = o;
  else x = o;
}

// Scores are compared through their bit patterns as signed integers: for non-negative floats the
// order is the same, and integer max needs no NaN canonicalisation.
__device__ __forceinline__ int fbits(float x) { return __builtin_bit_cast(int, x); }
__device__ __forceinline__ int max3i(int a, int b, int c) { return max(max(a, b), c); }
__device__ __forceinline__ int med3i(int a, int b, int c) { return max(min(a, b), min(max(a, b), c)); }

// The three best keys among a lane's entries, largest first. A key is the best score of a block of
// entries with its low bits replaced by the block's number.
struct Top3 {
  int k[3];
};

// Screening by the matrix cores. Entry c (fp16, in LDS; LO: fp64 centres as two fp16 words, a second
// array) against direction d: one v_mfma_f32_32x32x16_f16 forms c . d_hi + c . d_lo for 32 entries and
// 32 vectors (K = 16, the lower lanes' operand d_hi, the upper ones' d_lo, the same entry for both),
// with LO a second one adds c_lo . (d_hi + d_lo). Products are exact and the fp32 sums of up to 32
// non-negative terms err by less than 2e-6 of the score, d's split by 2^-22 of it (and by 2^-25 times the entry a
// coordinate where fp16 ends, 1e-6 of kUp at most). A lane holds 16 of each 32 entries (rows 8 (i / 4) + 4 (lane / 32) + i % 4)
// for vector lane % 32 of two blocks of 32, block b = 0 the wave's vectors 0..31. It keeps the three
// best keys of blocks of GR * 32 entries. The scan is bound by the vector ALU's maxima
// (a v_max3_i32 per two scores, 4 cycles; 20 instructions per 64 entries and 32 vectors) on top of the
// products (64 cycles), which overlap with them only in part: issuing the next block's products
// first gained 2%. GR = 2 spares the key's four instructions on every second product where one
// product covers 32 entries; GR = 1 where two do halves the entries looked at again.
template <int GR, bool LO>
__device__ __forceinline__ void scan_entries(const uint4* cb, const uint4* cl, int nblk, const DirWords& w, Top3& p, Top3& q) {
  const int lane = threadIdx.x & 63;
  constexpr int kMask = GR == 2 ? 127 : 63;   // block numbers: up to 128 blocks of 64, 64 of 32
  uint32_t b0[4], b1[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    b0[i] = w.hi[i];
    b1[i] = w.lo[i];
    swap_halves(b0[i], b1[i]);
  }
  const h8v bop[2] = {__builtin_bit_cast(h8v, make_uint4(b0[0], b0[1], b0[2], b0[3])),
                      __builtin_bit_cast(h8v, make_uint4(b1[0], b1[1], b1[2], b1[3]))};
  int k[2][3];
#pragma unroll
  for (int b = 0; b < 2; ++b) k[b][0] = k[b][1] = k[b][2] = INT_MIN;
  const uint4* ca = cb + (lane & 31);
  const uint4* cla = LO ? cl + (lane & 31) : nullptr;
  f16v zero;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero[i] = 0.0f;
  for (int blk = 0; blk < nblk; ++blk) {
    f16v d[2][GR];
#pragma unroll
    for (int g = 0; g < GR; ++g) {
      const h8v aop = __builtin_bit_cast(h8v, ca[(blk * GR + g) * 32]);
#pragma unroll
      for (int b = 0; b < 2; ++b) d[b][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop, bop[b], zero, 0, 0, 0);
      if constexpr (LO) {
        const h8v alo = __builtin_bit_cast(h8v, cla[(blk * GR + g) * 32]);
#pragma unroll
        for (int b = 0; b < 2; ++b) d[b][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(alo, bop[b], d[b][g], 0, 0, 0);
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      int m = INT_MIN;
#pragma unroll
      for (int g = 0; g < GR; ++g)
#pragma unroll
        for (int i = 0; i < 16; i += 2) m = max3i(m, fbits(d[b][g][i]), fbits(d[b][g][i + 1]));
      m = (m & ~kMask) | blk;
      k[b][2] = med3i(k[b][1], k[b][2], m);
      k[b][1] = med3i(k[b][0], k[b][1], m);
      k[b][0] = max(k[b][0], m);
    }
  }
  // both halves' keys of the lane's own vector: p from the rows of the lower lanes, q of the upper ones
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    uint32_t x = (uint32_t)k[0][t], y = (uint32_t)k[1][t];
    swap_halves(x, y);
    p.k[t] = (int)x;
    q.k[t] = (int)y;
  }
}

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(h2v, a), __builtin_bit_cast(h2v, b), c, false);
}

// The score of one entry on the vector ALU, with the matrix cores' error bound.
template <bool LO>
__device__ __forceinline__ float score_of(const uint4* cb, const uint4* cl, int e, const DirWords& w) {
  const uint4 c = cb[e];
  const uint32_t cw[4] = {c.x, c.y, c.z, c.w};
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) s = dot2(cw[i], w.lo[i], s);
  if constexpr (LO) {
    const uint4 l = cl[e];
    const uint32_t lw[4] = {l.x, l.y, l.z, l.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) s = dot2(lw[i], w.hi[i], s);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) s = dot2(cw[i], w.hi[i], s);
  return s;
}

__device__ __forceinline__ double cosine(const double (&d)[8], const double (&c)[8]) {
  double s = d[0] * c[0];
#pragma unroll
  for (int t = 1; t < 8; ++t) s = fma(d[t], c[t], s);
  return s;
}

// The entry of [0, cnt) with the largest fp64 cosine to the direction of lane src, the lowest index among
// equals, by the whole wave: each lane compares the entries scoring at least thr of its share. d: the
// lanes' fp64 directions. 0 without a result (non-finite weights).
template <bool LO, class EntF>
__device__ __forceinline__ int wave_scan(const uint4* cb, const uint4* cl, int cnt, const DirWords& w, const double (&d)[8],
                                         float thr, int src, EntF entry) {
  const int lane = threadIdx.x & 63;
  DirWords v;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v.hi[i] = __shfl(w.hi[i], src, 64);
    v.lo[i] = __shfl(w.lo[i], src, 64);
  }
  double dv[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) dv[i] = __shfl(d[i], src, 64);
  const float tv = __shfl(thr, src, 64);
  double bs = -INFINITY;
  int be = INT_MAX;
  for (int e = lane; e < cnt; e += 64)
    if (score_of<LO>(cb, cl, e, v) >= tv) {
      double c[8];
      entry(e, c);
      const double sc = cosine(dv, c);
      if (sc > bs) {
        bs = sc;
        be = e;
      }
    }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const double os = __shfl_xor(bs, o, 64);
    const int oe = __shfl_xor(be, o, 64);
    if (os > bs || (os == bs && oe < be)) {
      bs = os;
      be = oe;
    }
  }
  return be < cnt ? be : 0;
}

// The same for all lanes whose thr is finite, by scoring the entries on the matrix cores once more: cheaper than
// wave_scan for one lane after the other where many lanes need it (codebooks with equal or nearly equal
// entries: 1000x1024 with each of 8192 entries four times 1.00 -> 0.35 ms; two k-means iterations with each centre
// sixteen times 1.57 -> 0.73 ms, 64 centres 0.22 -> 0.12). On 16x16x16 products, whose four scores a lane leave the
// registers of the first scan as they are (32x32x16 ones cost every W3 encode 1.6%).
template <bool LO, class EntF>
__device__ __forceinline__ int rescan(const uint4* cb, const uint4* cl, int cnt, const DirWords& w, const double (&d)[8], float thr,
                                      EntF entry) {
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  int own = 0;
#pragma unroll 1
  for (int b = 0; b < 4; ++b) {   // vectors 16 b + col
    const int src = 16 * b + col;
    const float tv = __shfl(thr, src, 64);
    if (!__any(tv < INFINITY)) continue;
    uint32_t x[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t h0 = __shfl(w.hi[i], src, 64), h1 = __shfl(w.hi[2 + i], src, 64), l0 = __shfl(w.lo[i], src, 64), l1 = __shfl(w.lo[2 + i], src, 64);
      x[i] = grp == 0 ? h0 : grp == 1 ? h1 : grp == 2 ? l0 : l1;
    }
    const h4v bop = __builtin_bit_cast(h4v, make_uint2(x[0], x[1]));
    double dv[8], bs = -INFINITY;
#pragma unroll
    for (int i = 0; i < 8; ++i) dv[i] = __shfl(d[i], src, 64);
    int be = INT_MAX;
#pragma unroll 1
    for (int e0 = 0; e0 < cnt; e0 += 16) {
      const int at = 2 * (e0 + col) + (grp & 1);   // four of the entry's coordinates
      f4v s = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(h4v, ((const uint2*)cb)[at]), bop, f4v{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
      if constexpr (LO) s = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(h4v, ((const uint2*)cl)[at]), bop, s, 0, 0, 0);
      uint32_t hits = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) hits |= (s[i] >= tv ? 1u : 0u) << i;
#pragma unroll 1
      while (__any(hits != 0)) {
        const int e = e0 + 4 * grp + (hits ? __builtin_ctz(hits) : 0);
        if (hits && e < cnt) {
          double c[8];
          entry(e, c);
          const double sc = cosine(dv, c);
          if (sc > bs) {
            bs = sc;
            be = e;
          }
        }
        hits &= hits - 1;
      }
    }
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const double os = __shfl_xor(bs, o, 64);
      const int oe = __shfl_xor(be, o, 64);
      if (os > bs || (os == bs && oe < be)) {
        bs = os;
        be = oe;
      }
    }
    if (grp == b) own = be < cnt ? be : 0;
  }
  return own;
}

// The entry of [0, cnt) with the largest fp64 cosine (an FMA chain in coordinate order), the lowest
// index among equals, for the lane's vector. `active` lanes hold a non-zero direction in w; dir(d)
// gives it in fp64 and entry(e, c) an entry in fp64. Every entry whose fp64 cosine could be the
// largest scores within the slack of the best key: twice the score's error (4e-6 of it and 1e-6 of
// kUp), the key's cut-off bits (2^-16 of it) and a margin. One survivor needs no fp64 at all; two are compared;
// more, or more candidate blocks than were kept, go to a scan of all entries by the whole wave. Lanes
// without a result (non-finite weights) get 0. The LDS holds nblk whole blocks.
template <int GR, bool LO, class DirF, class EntF>
__device__ __forceinline__ int nearest_of(const uint4* cb, const uint4* cl, int cnt, int nblk, const DirWords& w, bool active,
                                          DirF dir, EntF entry) {
  constexpr int kMask = GR == 2 ? 127 : 63;
  Top3 p, q;
  scan_entries<GR, LO>(cb, cl, nblk, w, p, q);
  const float best = __builtin_bit_cast(float, max(p.k[0], q.k[0]) & ~kMask);
  const float thr = best - (kSlack + 3e-5f * best);
  const int thr_i = thr < 0.0f ? INT_MIN : fbits(thr);
  int e1 = 0, e2 = 0, n = 0;
  // the candidate blocks: each lane's best first, then (rarely) the others
  const int first = max(p.k[0], q.k[0]), first_half = p.k[0] >= q.k[0] ? 0 : 1;
  const int second = min(p.k[0], q.k[0]);
#pragma unroll 1
  for (int t = 0; t < 4; ++t) {
    const int key = t == 0 ? first : t == 1 ? second : t == 2 ? p.k[1] : q.k[1];
    const int half = t == 0 ? first_half : t == 1 ? first_half ^ 1 : t - 2;
    const bool on = active && key >= thr_i;
    if (!__any(on)) continue;
    const int base = (key & kMask) * (32 * GR) + 4 * half;
    // four entries at a time, their LDS reads and dot products independent of each other (lanes
    // that are not `on` read some block as well)
#pragma unroll 2
    for (int g = 0; g < 4 * GR; ++g) {
      uint4 c[4], l[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        c[x] = cb[base + 8 * g + x];
        if constexpr (LO) l[x] = cl[base + 8 * g + x];
      }
      float a[4] = {0.0f, 0.0f, 0.0f, 0.0f}, b[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const uint32_t cw = i == 0 ? c[x].x : i == 1 ? c[x].y : i == 2 ? c[x].z : c[x].w;
          a[x] = dot2(cw, w.hi[i], a[x]);
          b[x] = dot2(cw, w.lo[i], b[x]);
          if constexpr (LO) b[x] = dot2(i == 0 ? l[x].x : i == 1 ? l[x].y : i == 2 ? l[x].z : l[x].w, w.hi[i], b[x]);
        }
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int e = base + 8 * g + x;
        const bool hit = on && e < cnt && a[x] + b[x] >= thr;
        e2 = hit && n == 1 ? e : e2;
        e1 = hit && n == 0 ? e : e1;
        n += hit ? 1 : 0;
      }
    }
  }
  const bool wide = active && (p.k[2] >= thr_i || q.k[2] >= thr_i || n == 0 || n > 2);
  if (__any(wide || (active && n == 2))) {
    double d[8];
    dir(d);
    if (active && n == 2) {
      double c1[8], c2[8];
      entry(e1, c1);
      entry(e2, c2);
      const double s1 = cosine(d, c1), s2 = cosine(d, c2);
      if (s2 > s1 || (s2 == s1 && e2 < e1)) e1 = e2;
    }
    uint64_t todo = __ballot(wide);
    if (__builtin_expect(__builtin_popcountll(todo) > 8, 0)) {
      const int e = rescan<LO>(cb, cl, cnt, w, d, wide ? thr : INFINITY, entry);
      if (wide) e1 = e;
      todo = 0;
    }
    for (; todo; todo &= todo - 1) {
      const int src = (int)__builtin_ctzll(todo);
      const int e = wave_scan<LO>(cb, cl, cnt, w, d, thr, src, entry);
      if ((int)(threadIdx.x & 63) == src) e1 = e;
    }
  }
  return active ? e1 : 0;
}

// The same for a small codebook (at most 256 entries): keys carry the entry itself, so the best key
// names the entry, and where the second best lies outside the slack nothing is left to decide (all
// but about one vector in a thousand at 64 entries). Three instructions per score instead of half of one, but
// no second look at a block of entries, which would cost more than the scan.
template <class DirF, class EntF>
__device__ __forceinline__ int nearest_small(const uint4* cb, int cnt, const DirWords& w, bool active, DirF dir, EntF entry) {
  const int lane = threadIdx.x & 63;
  const int mask = max(cnt, 32) - 1;   // cnt is a power of two
  uint32_t b0[4], b1[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    b0[i] = w.hi[i];
    b1[i] = w.lo[i];
    swap_halves(b0[i], b1[i]);
  }
  const h8v bop[2] = {__builtin_bit_cast(h8v, make_uint4(b0[0], b0[1], b0[2], b0[3])),
                      __builtin_bit_cast(h8v, make_uint4(b1[0], b1[1], b1[2], b1[3]))};
  f16v zero;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero[i] = 0.0f;
  int k[2][2] = {{INT_MIN, INT_MIN}, {INT_MIN, INT_MIN}};
  for (int e0 = 0; e0 < cnt; e0 += 32) {
    const h8v aop = __builtin_bit_cast(h8v, cb[e0 + (lane & 31)]);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const f16v d = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop, bop[b], zero, 0, 0, 0);
      int m1 = INT_MIN, m2 = INT_MIN;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = (fbits(d[i]) & ~mask) | (8 * (i / 4) + i % 4);
        m2 = med3i(m1, m2, key);
        m1 = max(m1, key);
      }
      m1 |= e0;
      m2 |= e0;
      k[b][1] = max(med3i(k[b][0], k[b][1], m1), m2);
      k[b][0] = max(k[b][0], m1);
    }
  }
  uint32_t x1 = (uint32_t)k[0][0], y1 = (uint32_t)k[1][0], x2 = (uint32_t)k[0][1], y2 = (uint32_t)k[1][1];
  swap_halves(x1, y1);
  swap_halves(x2, y2);
  const int p1 = (int)x1, q1 = (int)y1 | 4, p2 = (int)x2, q2 = (int)y2 | 4;   // bit 2: the rows' half
  const int k1 = max(p1, q1), k2 = max(min(p1, q1), max(p2, q2));
  const float best = __builtin_bit_cast(float, k1 & ~mask);
  const float thr = best - (kSlack + best * (1e-5f + (float)(mask + 1) * 0x1p-23f));
  const int thr_i = thr < 0.0f ? INT_MIN : fbits(thr);
  int e1 = k1 & mask;
  const bool wide = active && !(k2 < thr_i && e1 < cnt);
  if (__any(wide)) {
    double d[8];
    dir(d);
    uint64_t todo = __ballot(wide);
    // equal or nearly equal entries for many lanes: every lane compares them all in fp64 (1000x1024 with each entry
    // twice, 64 entries 83 -> 14 us, 256 110 -> 41)
    if (5 * __builtin_popcountll(todo) > cnt) {
      double bs = -INFINITY;
      int be = 0;
      for (int e = 0; e < cnt; ++e) {
        double c[8];
        entry(e, c);
        const double sc = cosine(d, c);
        if (sc > bs) {
          bs = sc;
          be = e;
        }
      }
      if (wide) e1 = be;
      todo = 0;
    }
    for (; todo; todo &= todo - 1) {
      const int src = (int)__builtin_ctzll(todo);
      const int e = wave_scan<false>(cb, nullptr, cnt, w, d, thr, src, entry);
      if (lane == src) e1 = e;
    }
  }
  return active ? e1 : 0;
}

// ------------------------------------------------------------------------------------ encoder

struct EncArgs {
  const float* w;
  int64_t ldw, nv, nvec;
  uint32_t nv_m;   // division by nv below 2^31, as (x * nv_m) >> nv_k; 0 for more vectors
  int nv_k;
  const uint16_t* cb;
  int ncb, vmax;
  uint8_t* signs;
  uint16_t* dir;
  uint8_t* q;
  uint16_t* gmin;
  uint16_t* gstep;
};

typedef uint32_t u4a2 __attribute__((ext_vector_type(4), aligned(2)));   // codebooks are 2-byte aligned

// Minimum and maximum over 16-lane rows by DPP rotations.
template <int CTRL>
__device__ __forceinline__ double row_ror(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ void row_min_max(double& lo, double& hi) {
  lo = fmin(lo, row_ror<0x128>(lo));
  hi = fmax(hi, row_ror<0x128>(hi));
  lo = fmin(lo, row_ror<0x124>(lo));
  hi = fmax(hi, row_ror<0x124>(hi));
  lo = fmin(lo, row_ror<0x122>(lo));
  hi = fmax(hi, row_ror<0x122>(hi));
  lo = fmin(lo, row_ror<0x121>(lo));
  hi = fmax(hi, row_ror<0x121>(hi));
}

// Eq. 3, 5, 6 and 7: a wave encodes 64 consecutive vectors at a time, with the codebook (at most
// MAXE entries) in LDS, rows past it zero. Groups of 16 vectors never straddle a row (k is a multiple of 128) and start at multiples of 16 in the flat
// vector index, so each is 16 aligned lanes, all inside or all outside [0, nvec).
//
// The direction is normalised in fp32 for the screening, after scaling by a power of two so that no
// square leaves its range: a common factor of d's coordinates (the rounded norm, Eq. 3's floor of
// the radius) does not change which entry is nearest, and fp64 decides among survivors with Eq. 3's own.
//
// Measured (MI355X): 12288x4096 W2 (64 entries) 235 -> 107 us, of which the bytes take 45, the rest
// vector-ALU work (about 2700 cycles per 64 vectors: a third the search, the rest Eq. 3, 6 and 7);
// 4096x4096 W3 (8192 entries) 2.61 -> 0.61 ms, the scan. Before, every vector was compared with
// every entry in fp64 (W2), or scored twice on 16x16x16 products with fp64 on the candidates (W3).
template <int MAXE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(4))) void k_encode(EncArgs a, int64_t units) {
  constexpr bool SMALL = MAXE <= 256;
  static_assert(MAXE % 64 == 0, "whole blocks of entries");
  __shared__ uint4 cbl[MAXE];
  const int nthreads = (int)blockDim.x;
  for (int t = threadIdx.x; t < MAXE; t += nthreads) {
    uint4 c = make_uint4(0, 0, 0, 0);
    if (t < a.ncb) {
      const u4a2 v = *(const u4a2*)(a.cb + (int64_t)t * 8);
      c = make_uint4(v[0], v[1], v[2], v[3]);
    }
    cbl[t] = c;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wpb = nthreads >> 6;
  auto entry = [&](int e, double (&c)[8]) {
    const uint4 v = cbl[e];
    const uint32_t cw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int t = 0; t < 8; ++t) c[t] = h2d((uint16_t)(cw[t / 2] >> (16 * (t & 1))));
  };
  for (int64_t unit = (int64_t)blockIdx.x * wpb + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); unit < units; unit += (int64_t)gridDim.x * wpb) {
    // the wave's first row and vector by one scalar division, the lanes' from there
    const int64_t i0 = unit * 64, i = i0 + lane;
    const bool ok = i < a.nvec;
    int64_t row = a.nv_m ? (int64_t)(((uint64_t)(uint32_t)i0 * a.nv_m) >> a.nv_k) : i0 / a.nv;
    int v = (int)(i0 - row * a.nv) + lane;
    const int nv = (int)a.nv;
    if (v >= nv) {
      const int more = nv >= 64 ? 1 : v / nv;
      row += more;
      v -= more * nv;
    }
    float f[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (ok) {
      const float4* p = reinterpret_cast<const float4*>(a.w + row * a.ldw + (int64_t)v * 8);
      const float4 x0 = p[0], x1 = p[1];
      f[0] = x0.x; f[1] = x0.y; f[2] = x0.z; f[3] = x0.w; f[4] = x1.x; f[5] = x1.y; f[6] = x1.z; f[7] = x1.w;
    }
    uint32_t neg = 0;
    float most = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      neg |= (f[j] < 0.0f ? 1u : 0u) << j;
      f[j] = fabsf(f[j]);
      most = fmaxf(most, f[j]);
    }
    const bool active = ok && most > 0.0f;   // a zero vector's cosines are all 0: the first entry
    float d[8], ss = 0.0f;
    const int ex = -__builtin_amdgcn_frexp_expf(most);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      d[j] = ldexpf(f[j], ex);
      ss = fmaf(d[j], d[j], ss);
    }
    const float inv = active ? kUp * __builtin_amdgcn_rsqf(ss) : 0.0f;   // ss is in [1/4, 8)
#pragma unroll
    for (int j = 0; j < 8; ++j) d[j] *= inv;
    const DirWords w = split_dir(d);
    auto dir = [&](double (&dd)[8]) {
      double av[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) av[j] = (double)f[j];
      unit_direction(av, dd);
    };
    int bz;
    if constexpr (SMALL) bz = nearest_small(cbl, a.ncb, w, active, dir, entry);
    else bz = nearest_of<2, false>(cbl, nullptr, a.ncb, (a.ncb + 63) / 64, w, active, dir, entry);
    double av[8], c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) av[j] = (double)f[j];
    entry(bz, c);
    const double rt = dot8_pairwise(av, c);  // Eq. 6
    double lo = rt, hi = rt;
    row_min_max(lo, hi);
    const uint16_t lo16 = d2h(lo), st16 = d2h((hi - lo) / (double)a.vmax);
    const double lod = h2d(lo16), std_ = h2d(st16);
    int q = 0;
    if (std_ > 0.0) q = (int)fmin(fmax(rint((rt - lod) / std_), 0.0), (double)a.vmax);
    if (ok) {
      a.signs[i] = (uint8_t)neg;
      a.dir[i] = (uint16_t)bz;
      a.q[i] = (uint8_t)q;
      if ((lane & 15) == 0) {
        a.gmin[i >> 4] = lo16;
        a.gstep[i >> 4] = st16;
      }
    }
  }
}

// ------------------------------------------------------------------------------------ k-means

// Block-wide exclusive prefix of one value per thread, in a fixed order; also returns the block
// total. `sh` holds kThreads doubles.
__device__ __forceinline__ double block_exclusive(double v, double* sh, double& total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) sh[wv] = incl;
  __syncthreads();
  double woff = 0.0;
  for (int k = 0; k < wv; ++k) woff += sh[k];
  double tot = 0.0;
  for (int k = 0; k < kThreads / 64; ++k) tot += sh[k];
  __syncthreads();
  total = tot;
  return woff + (incl - v);
}

// Squared radius r^2 of every vector (r from Eq. 3), stored in cdf[], and each block's total. The
// vectors are read in order across the block (8 consecutive ones per thread, as they are summed, would
// touch eight times the lines at once: 50 us for 4096x4096) and handed over through LDS.
__global__ __launch_bounds__(kThreads) void k_r2(const float* __restrict__ w, int64_t ldw, int64_t nv,
                                                 int64_t nvec, double* __restrict__ cdf,
                                                 double* __restrict__ bsum) {
  __shared__ double sh[kThreads / 64];
  __shared__ double val[kThreads * (kScanItems + 1)];   // one double of padding per thread's run
  const int64_t b0 = (int64_t)blockIdx.x * kScanBlock;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    const int o = j * kThreads + (int)threadIdx.x;
    const int64_t i = b0 + o;
    double r2 = 0.0;
    if (i < nvec) {
      double av[8], d[8];
      uint32_t neg;
      const double r = decompose(w, ldw, nv, i, av, d, neg);
      r2 = r * r;
      cdf[i] = r2;
    }
    val[o + o / kScanItems] = r2;
  }
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) s += val[threadIdx.x * (kScanItems + 1) + j];
  double total;
  block_exclusive(s, sh, total);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// Exclusive running sum of the nb block totals, in place, by one block.
__global__ __launch_bounds__(kThreads) void k_scan_blocks(double* __restrict__ bsum, int64_t nb) {
  __shared__ double sh[kThreads / 64];
  const int64_t per = (nb + kThreads - 1) / kThreads;
  const int64_t b0 = (int64_t)threadIdx.x * per, b1 = min(nb, b0 + per);
  double s = 0.0;
  for (int64_t b = b0; b < b1; ++b) s += bsum[b];
  double total;
  double run = block_exclusive(s, sh, total);
  for (int64_t b = b0; b < b1; ++b) {
    const double v = bsum[b];
    bsum[b] = run;
    run += v;
  }
}

// Running sum of r^2 in storage order: cdf[i] = sum of r^2 over vectors 0..i.
__global__ __launch_bounds__(kThreads) void k_scan_apply(double* __restrict__ cdf, const double* __restrict__ boff,
                                                         int64_t nvec) {
  __shared__ double sh[kThreads / 64];
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems;
  double v[kScanItems];
  double s = 0.0;
  for (int j = 0; j < kScanItems; ++j) {
    const int64_t i = i0 + j;
    v[j] = i < nvec ? cdf[i] : 0.0;
    s += v[j];
  }
  double total;
  const double off = boff[blockIdx.x] + block_exclusive(s, sh, total);
  double run = 0.0;
  for (int j = 0; j < kScanItems; ++j) {
    const int64_t i = i0 + j;
    run += v[j];
    if (i < nvec) cdf[i] = off + run;
  }
}

// Inverse-CDF draw (Sec. 3.1): sample j takes the first vector whose running r^2 exceeds
// u_j * total, clamped to the last vector; its unit direction goes to ds[j][0..8).
__global__ __launch_bounds__(kThreads) void k_sample(const float* __restrict__ w, int64_t ldw, int64_t nv,
                                                     int64_t nvec, const double* __restrict__ cdf,
                                                     const double* __restrict__ u, int64_t ns,
                                                     double* __restrict__ ds, int64_t* __restrict__ sidx) {
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (j >= ns) return;
  const double target = u[j] * cdf[nvec - 1];
  int64_t lo = 0, hi = nvec;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (cdf[mid] > target)
      hi = mid;
    else
      lo = mid + 1;
  }
  const int64_t idx = lo < nvec ? lo : nvec - 1;
  if (sidx) sidx[j] = idx;
  double av[8], d[8];
  uint32_t neg;
  decompose(w, ldw, nv, idx, av, d, neg);
#pragma unroll
  for (int c = 0; c < 8; ++c) ds[j * 8 + c] = d[c];
}

__device__ __forceinline__ void store_words(uint4* words, int ncb, int c, int e, double v);

__global__ __launch_bounds__(kThreads) void k_init_centres(const uint16_t* __restrict__ init, int64_t count,
                                                           double* __restrict__ cen, uint4* __restrict__ words) {
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t >= count) return;
  const double v = h2d(init[t]);
  cen[t] = v;
  store_words(words, (int)(count / 8), (int)(t / 8), (int)(t & 7), v);
}

// Eq. 5 for every sample against centres [split * per, (split + 1) * per): the best cosine and its
// index per sample and split (blockIdx.y is the split). The centres go through LDS kCentres at a
// time as two fp16 words per coordinate (error 2^-22 of it, inside nearest_of's bound), kept beside the
// fp64 ones by whoever moves a centre; a later chunk wins only with a strictly larger cosine. 65,536 samples, 8192 centres: 236 us
// (fp64 against every centre) -> 44 us.
constexpr int kCentres = 2048;   // 64 KiB of LDS

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(4))) void k_assign_split(const double* __restrict__ ds, int64_t ns,
                                                             const double* __restrict__ cen, const uint4* __restrict__ words, int ncb,
                                                             int per, double* __restrict__ sbest, int32_t* __restrict__ sidx) {
  constexpr int MAXE = WAVES == 16 ? kCentres : 256;
  __shared__ uint4 ch[MAXE], cl[MAXE];
  const int lane = threadIdx.x & 63;
  const int64_t j = ((int64_t)blockIdx.x * WAVES + (threadIdx.x >> 6)) * 64 + lane;
  const int c0 = blockIdx.y * per, c1 = min(ncb, c0 + per);
  double d[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) d[c] = j < ns ? ds[j * 8 + c] : 0.0;
  float f[8], most = 0.0f;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    f[c] = kUp * (float)d[c];
    most = fmaxf(most, f[c]);
  }
  const bool active = most > 0.0f;   // a zero vector's cosines are all 0: the first centre
  const DirWords w = split_dir(f);
  double best = -INFINITY;
  int bz = c0;
  for (int base = c0; base < c1; base += MAXE) {
    const int cnt = min(MAXE, c1 - base), nblk = (cnt + 31) / 32;
    __syncthreads();
    for (int t = threadIdx.x; t < nblk * 32; t += 64 * WAVES) {
      ch[t] = t < cnt ? words[base + t] : make_uint4(0, 0, 0, 0);
      cl[t] = t < cnt ? words[ncb + base + t] : make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    auto entry = [&](int e, double (&c)[8]) {
      const double2* p = reinterpret_cast<const double2*>(cen + (int64_t)(base + e) * 8);
      const double2 x0 = p[0], x1 = p[1], x2 = p[2], x3 = p[3];
      c[0] = x0.x; c[1] = x0.y; c[2] = x1.x; c[3] = x1.y; c[4] = x2.x; c[5] = x2.y; c[6] = x3.x; c[7] = x3.y;
    };
    const int z = nearest_of<1, true>(
        ch, cl, cnt, nblk, w, active,
        [&](double (&dd)[8]) {
#pragma unroll
          for (int c = 0; c < 8; ++c) dd[c] = d[c];
        },
        entry);
    double c[8];
    entry(z, c);
    const double s = cosine(d, c);
    if (s > best) {
      best = s;
      bz = base + z;
    }
  }
  if (j < ns) {
    sbest[blockIdx.y * ns + j] = best;
    sidx[blockIdx.y * ns + j] = bz;
  }
}

// The splits combined in ascending order with a strict comparison (the same decision as one scan
// over all centres): z[j] gets the nearest centre, rank[j] its place among that centre's samples of this
// block's chunk of ch samples (in whatever order they arrive), hist[block][centre] their number. Each
// 256 samples' cosines to their centres are summed (each in pairwise order, then in a fixed order) into
// opart. Counted in LDS: a few centres take thousands of samples each (weight vectors with an outlier),
// and global atomics on them took 30 us. rank may be sidx's first split. Without hist nothing is counted.
constexpr int kFinalThreads = 1024;

__global__ __launch_bounds__(kFinalThreads) void k_assign_final(const double* __restrict__ ds, int64_t ns, int64_t ch,
                                                                const double* __restrict__ cen, int ncb, int nsplit,
                                                                const double* __restrict__ sbest, const int32_t* sidx,
                                                                int32_t* __restrict__ z, int32_t* rank,
                                                                uint32_t* __restrict__ hist, double* __restrict__ opart) {
  __shared__ uint32_t cnt[8192];
  __shared__ double wsum[kFinalThreads / 64];
  if (hist)
    for (int t = threadIdx.x; t < ncb; t += kFinalThreads) cnt[t] = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t j0 = blockIdx.x * ch, j1 = min(ns, j0 + ch);
  for (int64_t base = j0; base < j1; base += kFinalThreads) {   // ch is a multiple of kFinalThreads
    const int64_t j = base + threadIdx.x;
    double v = 0.0;
    if (j < j1) {
      double best = sbest[j];
      int bz = sidx[j];
      for (int t = 1; t < nsplit; ++t) {
        const double b = sbest[t * ns + j];
        if (b > best) {
          best = b;
          bz = sidx[t * ns + j];
        }
      }
      z[j] = bz;
      if (hist) rank[j] = (int32_t)atomicAdd(&cnt[bz], 1u);
      double d[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) d[c] = ds[j * 8 + c];
      v = dot8_pairwise(d, cen + (int64_t)bz * 8);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double t = __shfl_up(v, o, 64);
      if (lane >= o) v += t;
    }
    __syncthreads();
    if (lane == 63) wsum[wv] = v;
    __syncthreads();
    if (threadIdx.x < kFinalThreads / 256 && base + threadIdx.x * 256 < ns) {
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) s += wsum[4 * threadIdx.x + k];
      opart[base / 256 + threadIdx.x] = s;
    }
  }
  __syncthreads();
  if (hist)
    for (int t = threadIdx.x; t < ncb; t += kFinalThreads) hist[(int64_t)blockIdx.x * ncb + t] = cnt[t];
}

// Per centre, the running sum of the chunks' counts over the nch chunks, in place, and their total;
// the last block adds up the objective of the assignment (if wanted) over its nblk partial sums,
// lane-strided in block order and then by a fixed lane tree.
__global__ __launch_bounds__(kThreads) void k_offsets(uint32_t* __restrict__ hist, int nch, int ncb, uint32_t* __restrict__ count,
                                                      const double* __restrict__ opart, int64_t nblk, double* __restrict__ out) {
  if (blockIdx.x + 1 == gridDim.x) {
    if (!out || threadIdx.x >= 64) return;
    double s = 0.0;
    for (int64_t b = threadIdx.x; b < nblk; b += 64) s += opart[b];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    if (threadIdx.x == 0) *out = s;
    return;
  }
  const int c = blockIdx.x * kThreads + threadIdx.x;
  if (c >= ncb) return;
  uint32_t run = 0;
  for (int b0 = 0; b0 < nch; b0 += 16) {
    uint32_t v[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) v[t] = b0 + t < nch ? hist[(int64_t)(b0 + t) * ncb + c] : 0u;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      if (b0 + t < nch) hist[(int64_t)(b0 + t) * ncb + c] = run;
      run += v[t];
    }
  }
  count[c] = run;
}

// The samples listed by centre, perm[start of the centre + the chunk's offset in it + rank] = sample,
// the starts being the running sum of the counts, which every block forms for itself in LDS. Block 0
// keeps them, and the list of centres with more than kBig samples.
constexpr int kListThreads = 1024;
constexpr int kBig = 256;          // samples up to which one wave adds up a centre
constexpr int kMaxBig = 1024;      // big centres kept; more are left to their waves

__global__ __launch_bounds__(kListThreads) void k_list(const int32_t* __restrict__ z, const int32_t* __restrict__ rank,
                                                       int64_t ns, int64_t ch, const uint32_t* __restrict__ hist,
                                                       const uint32_t* __restrict__ count, int ncb,
                                                       uint32_t* __restrict__ start, uint32_t* __restrict__ big,
                                                       int32_t* __restrict__ perm) {
  __shared__ uint32_t at[8192];
  __shared__ uint32_t wsum[kListThreads / 64];
  __shared__ uint32_t nbig;
  const int per = (ncb + kListThreads - 1) / kListThreads;   // 1..8 consecutive centres per thread
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int e0 = (int)threadIdx.x * per;
  if (threadIdx.x == 0) nbig = 0;
  uint32_t own[8], s = 0;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    own[t] = t < per && e0 + t < ncb ? count[e0 + t] : 0u;
    s += own[t];
  }
  uint32_t incl = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(incl, o, 64);
    if (lane >= o) incl += u;
  }
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  uint32_t run = incl - s;
  for (int k = 0; k < wv; ++k) run += wsum[k];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    if (t < per && e0 + t < ncb) {
      at[e0 + t] = run;
      if (blockIdx.x == 0) {
        start[e0 + t] = run;
        if (own[t] > kBig) {
          const uint32_t b = atomicAdd(&nbig, 1u);
          if (b < kMaxBig) big[1 + b] = (uint32_t)(e0 + t);
        }
      }
    }
    run += own[t];
  }
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) big[0] = nbig <= kMaxBig ? nbig : 0;
  for (int64_t j = (int64_t)blockIdx.x * kListThreads + threadIdx.x; j < ns; j += (int64_t)gridDim.x * kListThreads) {
    const int c = z[j];
    perm[at[c] + hist[j / ch * ncb + c] + (uint32_t)rank[j]] = (int32_t)j;
  }
}

// Centre sums by exact fixed-point accumulation. A direction component v in [0, 1 + 2^-52] is
// truncated to T = floor(v * 2^100) in a 128-bit integer. Integer addition is associative, so the
// sums do not depend on the order in which samples are listed, and 2^24 samples cannot overflow. The sum
// is exact up to the 2^-100 truncation of each term.
constexpr int kFixBits = 100;
constexpr int kLimbBits = 40;
constexpr uint64_t kLimbMask = (1ull << kLimbBits) - 1;

__device__ __forceinline__ unsigned __int128 to_fixed(double v) {
  const uint64_t bits = __builtin_bit_cast(uint64_t, v);
  const int ex = (int)(bits >> 52);  // components are >= 0; 0 for zero and subnormals
  unsigned __int128 t = 0;
  if (ex != 0) {
    const uint64_t m = (bits & 0xFFFFFFFFFFFFFull) | 0x10000000000000ull;
    const int sh = ex - 1075 + kFixBits;  // v = m * 2^(ex - 1075)
    if (sh >= 0)
      t = (unsigned __int128)m << sh;
    else if (sh > -64)
      t = m >> -sh;
  }
  return t;
}

// The fp16 words of centre c's coordinate e (lanes 0..7 of a wave hold the coordinates): the same split
// as split_dir's, for k_assign_split.
__device__ __forceinline__ void store_words(uint4* words, int ncb, int c, int e, double v) {
  const float f = (float)v;
  const _Float16 h = (_Float16)f, l = (_Float16)(f - (float)h);
  ((_Float16*)(words + c))[e] = h;
  ((_Float16*)(words + ncb + c))[e] = l;
}

// Centre c's sum of component lane % 8 (the same in all of the wave's lanes of that component) converted
// to fp64, and the sums normalised to unit length; a centre without directions keeps its position.
__device__ __forceinline__ void finish_centre(unsigned __int128 sum, int ncb, int c, int lane, double* cen, uint4* words) {
#pragma clang fp contract(off)
  const int e = lane & 7;
  // limbs of 40 bits convert exactly; two roundings combine them
  const uint64_t l0 = (uint64_t)sum & kLimbMask, l1 = (uint64_t)(sum >> kLimbBits) & kLimbMask, l2 = (uint64_t)(sum >> (2 * kLimbBits));
  const double hi = ((double)l2 * 0x1p40 + (double)l1) * 0x1p40;
  const double mine = (hi + (double)l0) * 0x1p-100;
  double s[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) s[t] = __shfl(mine, t, 64);
  const double norm = sqrt(dot8_pairwise(s, s));
  if (norm > 0.0 && lane < 8) {
    const double v = mine / norm;
    cen[(int64_t)c * 8 + e] = v;
    store_words(words, ncb, c, e, v);
  }
}

// Up to 256 centres are summed without a list: block p adds chunk p's samples with 64-bit LDS atomics,
// three 40-bit limbs a component, and stores 128-bit sums; a wave per centre adds the chunks'.
// A list gives such a codebook only as many blocks as it has centres. k-means of 4096x4096, 65,536
// samples, 20 iterations, by lists -> by chunks: 936 -> 514 us (16 entries), 921 -> 541 (64), 958 -> 629
// (256). With 2^13 centres the chunks' sums are more bytes than the samples, and the list wins (101 + 30
// us an iteration against 10 + 22).
constexpr int kAccMax = 256;
constexpr int kLimbs = 8 * 3;

__global__ __launch_bounds__(kThreads) void k_accumulate(const double* __restrict__ ds, int64_t ns, const int32_t* __restrict__ z,
                                                         int ncb, int64_t ch, ulonglong2* __restrict__ part) {
  __shared__ unsigned long long la[kAccMax * kLimbs];
  for (int t = threadIdx.x; t < ncb * kLimbs; t += kThreads) la[t] = 0;
  __syncthreads();
  const int64_t j0 = (int64_t)blockIdx.x * ch, j1 = min(ns, j0 + ch);
  for (int64_t j = j0 + threadIdx.x; j < j1; j += kThreads) {
    unsigned long long* a = la + z[j] * kLimbs;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const unsigned __int128 t = to_fixed(ds[j * 8 + e]);
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        const uint64_t v = (uint64_t)(t >> (l * kLimbBits)) & kLimbMask;
        if (v) atomicAdd(a + 3 * e + l, (unsigned long long)v);
      }
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < ncb * 8; t += kThreads) {
    const unsigned __int128 v = (unsigned __int128)la[3 * t] + ((unsigned __int128)la[3 * t + 1] << kLimbBits) +
                                ((unsigned __int128)la[3 * t + 2] << (2 * kLimbBits));
    part[(int64_t)blockIdx.x * ncb * 8 + t] = make_ulonglong2((uint64_t)v, (uint64_t)(v >> 64));
  }
}

__global__ __launch_bounds__(64) void k_update_chunks(const ulonglong2* __restrict__ part, int np, int ncb, double* __restrict__ cen,
                                                      uint4* __restrict__ words) {
  const int lane = threadIdx.x, c = blockIdx.x;
  unsigned __int128 sum = 0;
#pragma unroll 8
  for (int p = lane >> 3; p < np; p += 8) {
    const ulonglong2 v = part[((int64_t)p * ncb + c) * 8 + (lane & 7)];
    sum += ((unsigned __int128)v.y << 64) | v.x;
  }
#pragma unroll
  for (int o = 8; o <= 32; o <<= 1) {
    const uint64_t lo = __shfl_xor((uint64_t)sum, o, 64), hi = __shfl_xor((uint64_t)(sum >> 64), o, 64);
    sum += ((unsigned __int128)hi << 64) | lo;
  }
  finish_centre(sum, ncb, c, lane, cen, words);
}

// New centres of large codebooks: eight lanes per sample, one for each component, add a centre's listed
// samples. One wave per centre of at most kBig samples (blocks of 16), and one block for each of the
// big ones, which the last gridDim.x - (ncb + 15) / 16 blocks share. (65,536 samples, 8192 centres,
// a few of them with thousands: 101 + 30 us with LDS atomics in passes over all samples per centre range,
// 10 + 22 us with the list; 148 us with one wave per centre whatever its size.)
__global__ __launch_bounds__(1024) void k_update(const double* __restrict__ ds, const int32_t* __restrict__ perm,
                                                 const uint32_t* __restrict__ start, const uint32_t* __restrict__ count,
                                                 const uint32_t* __restrict__ big, int ncb, double* __restrict__ cen,
                                                 uint4* __restrict__ words) {
#pragma clang fp contract(off)
  __shared__ uint64_t part[16][8][2];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, e = lane & 7;
  const int small = (ncb + 15) / 16;
  const bool one = (int)blockIdx.x < small;   // a wave per centre
  const uint32_t nbig = big[0];
  for (uint32_t b = one ? 0u : blockIdx.x - small; one || b < nbig; b += gridDim.x - small) {
    const int c = one ? (int)blockIdx.x * 16 + wv : (int)big[1 + b];
    const bool have = c < ncb && !(one && nbig > 0 && count[c] > kBig);   // wave-uniform
    unsigned __int128 sum = 0;
    if (have) {
      const uint32_t len = count[c], first = start[c];
      const uint32_t t0 = one ? lane >> 3 : threadIdx.x >> 3, step = one ? 8 : 128;
#pragma unroll 4
      for (uint32_t t = t0; t < len; t += step) sum += to_fixed(ds[(int64_t)perm[first + t] * 8 + e]);
#pragma unroll
      for (int o = 8; o <= 32; o <<= 1) {
        const uint64_t lo = __shfl_xor((uint64_t)sum, o, 64), hi = __shfl_xor((uint64_t)(sum >> 64), o, 64);
        sum += ((unsigned __int128)hi << 64) | lo;
      }
    }
    if (!one) {
      if (lane < 8) {
        part[wv][e][0] = (uint64_t)sum;
        part[wv][e][1] = (uint64_t)(sum >> 64);
      }
      __syncthreads();
      sum = 0;
      for (int k = 0; k < 16; ++k) sum += ((unsigned __int128)part[k][e][1] << 64) | part[k][e][0];
      __syncthreads();
    }
    if (have && (one || wv == 0)) {
      finish_centre(sum, ncb, c, lane, cen, words);
    }
    if (one) break;
  }
}

__global__ __launch_bounds__(kThreads) void k_centres_to_f16(const double* __restrict__ cen, int64_t count,
                                                             uint16_t* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t < count) out[t] = d2h(cen[t]);
}

// ------------------------------------------------------------------------------------ host side

inline uint64_t align256(uint64_t x) { return (x + 255) / 256 * 256; }

struct KmPlan {
  int64_t nvec, nb, nfb, ch;
  int ncb, nsplit, per, waves, nch;
  int np;           // chunks of chp samples summed without a list, 0: by lists
  int64_t chp;
  uint64_t off_cdf, off_bsum, off_ds, off_z, off_opart, off_cen, off_words, off_count, off_hist, off_sbest, off_sidx, total;
};

// The workspace size that the interface states, per sample, per codebook entry and chunk and per split.
// The layout of km_plan takes no more (its 12 * nsplit bytes per sample, and 32 bytes of words and 8 to 12 of
// counts per entry with 4 per entry and chunk, or 32 with 128 per entry and chunk, stay within the 12
// and 192 bytes of more splits and chunks here);
// the size stays what callers have sized their buffers by.
uint64_t stated_bytes(int64_t nvec, int64_t nb, int64_t ns, int64_t ncb) {
  const int64_t nab = (ns + 1023) / 1024, nr = (ncb + 511) / 512;
  int64_t sp = std::min<int64_t>((1024 + nab - 1) / nab, std::max<int64_t>(1, ncb / 64));
  const int64_t per = (ncb + sp - 1) / sp;
  sp = (ncb + per - 1) / per;
  int64_t np = std::min<int64_t>((128 + nr - 1) / nr, (ns + kThreads - 1) / kThreads);
  const int64_t ch = (ns + np - 1) / np;
  np = (ns + ch - 1) / ch;
  uint64_t p = 0;
  for (const int64_t bytes : {nvec * 8, nb * 8, ns * 64, ns * 4, (ns + kThreads - 1) / kThreads * 8, ncb * 64, np * ncb * 192,
                              sp * ns * 8, sp * ns * 4})
    p = align256(p + (uint64_t)bytes);
  return p;
}

KmPlan km_plan(const sph_format* fmt, int64_t n, int64_t k, int64_t ns) {
  KmPlan P{};
  P.nvec = n * (k / SPH_VEC);
  P.nb = (P.nvec + kScanBlock - 1) / kScanBlock;
  P.nfb = (ns + kThreads - 1) / kThreads;
  P.ncb = 1 << fmt->dir_bits;
  // Waves per workgroup of the assignment: 16 share the staged centres where there are many, 4 spread
  // a small codebook's samples over more CUs. Centre splits: enough waves for four per SIMD, at
  // least 256 centres each, and no more than 2^20 + ns split results altogether.
  P.waves = P.ncb > 256 ? 16 : 4;
  const int64_t units = (ns + 63) / 64;
  int64_t sp = (4096 + units - 1) / units;
  sp = std::min<int64_t>(sp, std::max(1, P.ncb / 256));
  sp = std::max<int64_t>(1, std::min<int64_t>(sp, ((1 << 20) + ns) / ns));
  P.per = (int)((P.ncb + sp - 1) / sp);
  P.nsplit = (P.ncb + P.per - 1) / P.per;
  // sample chunks of the counting: whole rounds of kFinalThreads samples, at most 64 chunks
  P.ch = ((ns + 63) / 64 + kFinalThreads - 1) / kFinalThreads * kFinalThreads;
  P.nch = (int)((ns + P.ch - 1) / P.ch);
  if (P.ncb <= kAccMax) {   // at most 128 chunks, a thread per sample at least
    P.np = (int)std::min<int64_t>(128, (ns + kThreads - 1) / kThreads);
    P.chp = (ns + P.np - 1) / P.np;
    P.np = (int)((ns + P.chp - 1) / P.chp);
    P.ch = kFinalThreads;
    P.nch = (int)((ns + P.ch - 1) / P.ch);
  }
  uint64_t p = 0;
  P.off_cdf = p;
  p = align256(p + (uint64_t)P.nvec * 8);
  P.off_bsum = p;
  p = align256(p + (uint64_t)P.nb * 8);
  P.off_ds = p;
  p = align256(p + (uint64_t)ns * 64);
  P.off_z = p;
  p = align256(p + (uint64_t)ns * 4);
  P.off_opart = p;
  p = align256(p + (uint64_t)P.nfb * 8);
  P.off_cen = p;
  p = align256(p + (uint64_t)P.ncb * 64);
  P.off_words = p;
  p = align256(p + (uint64_t)P.ncb * 32);
  P.off_count = p;   // counts, list starts, big centres
  if (P.np == 0) p = align256(p + ((uint64_t)P.ncb * 2 + 1 + std::min(P.ncb, kMaxBig)) * 4);
  P.off_hist = p;    // or the chunks' sums
  p = align256(p + (P.np > 0 ? (uint64_t)P.np * P.ncb * 128 : (uint64_t)P.nch * P.ncb * 4));
  P.off_sbest = p;   // after a split's results are combined, the samples listed by centre
  p = align256(p + (uint64_t)P.nsplit * ns * 8);
  P.off_sidx = p;    // likewise the samples' ranks
  p = align256(p + (uint64_t)P.nsplit * ns * 4);
  P.total = std::max(p, stated_bytes(P.nvec, P.nb, ns, P.ncb));
  return P;
}

constexpr int64_t kMaxSamples = int64_t(1) << 24;
constexpr int32_t kMaxIters = 10000;

// The encoder and k-means handle 8-D vectors (the 4-D and 16-D formats are decode-only).
int check_fmt8(const sph_format* fmt) {
  const int st = sph_host_check_format(fmt);
  if (st) return st;
  return fmt->vec_dim == SPH_VEC ? SPH_OK : SPH_ERR_UNSUPPORTED_FORMAT;
}

int check_common(const sph_format* fmt, int64_t n, int64_t k, const float* d_w, int64_t ldw) {
  int st = check_fmt8(fmt);
  if (st) return st;
  st = sph_host_check_shape(n, k);
  if (st) return st;
  if (!d_w) return SPH_ERR_NULL;
  if (ldw < k || ldw % 4 != 0 || (uintptr_t)d_w % 16 != 0) return SPH_ERR_SHAPE;
  return SPH_OK;
}

constexpr int kSmallEntries = 256, kMaxEntries = 8192;   // direction bits are 4..8 or 13

int num_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    return 256;
  return cus;
}

template <typename... A>
bool launch_ok(const void* fn, dim3 grid, dim3 block, hipStream_t s, A... args) {
  void* kargs[] = {(void*)&args...};
  if (hipLaunchKernel(fn, grid, block, kargs, 0, s) != hipSuccess) return false;
  return hipGetLastError() == hipSuccess;
}

}  // namespace

extern "C" {

sph_status sph_encode(const sph_format* fmt, int64_t n, int64_t k, const float* d_w, int64_t ldw,
                      const uint16_t* d_codebook, uint8_t* d_signs, uint16_t* d_dir_idx,
                      uint8_t* d_radius_code, uint16_t* d_group_min, uint16_t* d_group_step,
                      void* stream) {
  if (!fmt || !d_codebook || !d_signs || !d_dir_idx || !d_radius_code || !d_group_min || !d_group_step)
    return SPH_ERR_NULL;
  const int st = check_common(fmt, n, k, d_w, ldw);
  if (st) return (sph_status)st;
  if ((uintptr_t)d_codebook % 2 || (uintptr_t)d_dir_idx % 2 || (uintptr_t)d_group_min % 2 ||
      (uintptr_t)d_group_step % 2)
    return SPH_ERR_SHAPE;
  EncArgs a{};
  a.w = d_w;
  a.ldw = ldw;
  a.nv = k / SPH_VEC;
  a.nvec = n * a.nv;
  a.cb = d_codebook;
  a.ncb = 1 << fmt->dir_bits;
  a.vmax = (1 << fmt->radius_bits) - 1;
  if (a.nvec < (1ll << 31)) {
    // exact below 2^31: m = ceil(2^k / nv) with k = 31 + ceil(log2 nv) exceeds 2^k / nv by less than 2^(k - 31) / nv
    int l = 0;
    while ((1ll << l) < a.nv) ++l;
    a.nv_k = 31 + l;
    a.nv_m = (uint32_t)(((1ull << a.nv_k) + (uint64_t)a.nv - 1) / (uint64_t)a.nv);
  }
  a.signs = d_signs;
  a.dir = d_dir_idx;
  a.q = d_radius_code;
  a.gmin = d_group_min;
  a.gstep = d_group_step;
  const int64_t units = (a.nvec + 63) / 64;
  if (a.ncb <= kSmallEntries) {
    if (!launch_ok((const void*)k_encode<kSmallEntries, kEncodeWaves>, dim3(sph_encode_blocks(units)), dim3(64 * kEncodeWaves), (hipStream_t)stream, a, units))
      return SPH_ERR_HIP;
    return SPH_OK;
  }
  // the 2^13-entry codebook: one 128 KiB copy per CU, shared by up to 16 waves (at least 4, which
  // load it)
  const int cus = num_cus();
  const int64_t waves = std::min<int64_t>(16, std::max<int64_t>(4, (units + cus - 1) / cus));
  const int64_t grid = std::min<int64_t>(cus, (units + waves - 1) / waves);
  if (!launch_ok((const void*)k_encode<kMaxEntries, 16>, dim3((unsigned)grid), dim3((unsigned)(64 * waves)), (hipStream_t)stream, a, units))
    return SPH_ERR_HIP;
  return SPH_OK;
}

sph_status sph_kmeans_workspace_bytes(const sph_format* fmt, int64_t n, int64_t k, int64_t n_samples,
                                      size_t* bytes) {
  if (!fmt || !bytes) return SPH_ERR_NULL;
  int st = check_fmt8(fmt);
  if (st) return (sph_status)st;
  st = sph_host_check_shape(n, k);
  if (st) return (sph_status)st;
  if (n_samples < 1 || n_samples > kMaxSamples) return SPH_ERR_SHAPE;
  *bytes = (size_t)km_plan(fmt, n, k, n_samples).total;
  return SPH_OK;
}

sph_status sph_kmeans_codebook(const sph_format* fmt, int64_t n, int64_t k, const float* d_w, int64_t ldw,
                               const double* d_u, int64_t n_samples, int32_t iters,
                               const uint16_t* d_init, uint16_t* d_codebook, double* d_objective,
                               int64_t* d_sample_idx, void* d_ws, size_t ws_bytes, void* stream) {
  if (!fmt || !d_u || !d_init || !d_codebook || !d_ws) return SPH_ERR_NULL;
  const int st = check_common(fmt, n, k, d_w, ldw);
  if (st) return (sph_status)st;
  if (n_samples < 1 || n_samples > kMaxSamples || iters < 0 || iters > kMaxIters) return SPH_ERR_SHAPE;
  if ((uintptr_t)d_u % 8 || (uintptr_t)d_init % 2 || (uintptr_t)d_codebook % 2 ||
      (uintptr_t)d_objective % 8 || (uintptr_t)d_sample_idx % 8 || (uintptr_t)d_ws % 256)
    return SPH_ERR_SHAPE;
  const KmPlan P = km_plan(fmt, n, k, n_samples);
  if (ws_bytes < P.total) return SPH_ERR_BUFFER_TOO_SMALL;
  hipStream_t s = (hipStream_t)stream;
  uint8_t* ws = (uint8_t*)d_ws;
  double* cdf = (double*)(ws + P.off_cdf);
  double* bsum = (double*)(ws + P.off_bsum);
  double* ds = (double*)(ws + P.off_ds);
  int32_t* z = (int32_t*)(ws + P.off_z);
  double* opart = (double*)(ws + P.off_opart);
  double* cen = (double*)(ws + P.off_cen);
  uint32_t* count = (uint32_t*)(ws + P.off_count);
  uint32_t* start = count + P.ncb;
  uint32_t* big = start + P.ncb;
  uint32_t* hist = (uint32_t*)(ws + P.off_hist);
  uint4* words = (uint4*)(ws + P.off_words);
  double* sbest = (double*)(ws + P.off_sbest);
  int32_t* sidx = (int32_t*)(ws + P.off_sidx);
  int32_t* perm = (int32_t*)sbest;
  int32_t* rank = sidx;
  const int64_t ns = n_samples, nv = k / SPH_VEC, ncb8 = (int64_t)P.ncb * 8;
  const dim3 blk(kThreads);
  const unsigned g_cb = (unsigned)((ncb8 + kThreads - 1) / kThreads);
  const unsigned g_s = (unsigned)((ns + kThreads - 1) / kThreads);
  bool ok = launch_ok((const void*)k_r2, dim3((unsigned)P.nb), blk, s, d_w, ldw, nv, P.nvec, cdf, bsum) &&
            launch_ok((const void*)k_scan_blocks, dim3(1), blk, s, bsum, P.nb) &&
            launch_ok((const void*)k_scan_apply, dim3((unsigned)P.nb), blk, s, cdf, (const double*)bsum, P.nvec) &&
            launch_ok((const void*)k_sample, dim3(g_s), blk, s, d_w, ldw, nv, P.nvec, (const double*)cdf, d_u, ns,
                      ds, d_sample_idx) &&
            launch_ok((const void*)k_init_centres, dim3(g_cb), blk, s, d_init, ncb8, cen, words);
  const int64_t units = (ns + 63) / 64;
  const dim3 g_split((unsigned)((units + P.waves - 1) / P.waves), (unsigned)P.nsplit);
  const void* assign = P.waves == 16 ? (const void*)k_assign_split<16> : (const void*)k_assign_split<4>;
  const unsigned g_list = (unsigned)((ns + kListThreads - 1) / kListThreads);
  const unsigned g_upd = (unsigned)((P.ncb + 15) / 16 + std::min(P.ncb, 256));
  const unsigned g_off = (unsigned)((P.ncb + kThreads - 1) / kThreads + 1);
  for (int32_t it = 0; ok && it <= iters; ++it) {
    ok = launch_ok(assign, g_split, dim3(64 * P.waves), s, (const double*)ds, ns, (const double*)cen, (const uint4*)words, P.ncb,
                   P.per, sbest, sidx) &&
         launch_ok((const void*)k_assign_final, dim3((unsigned)P.nch), dim3(kFinalThreads), s, (const double*)ds, ns, P.ch,
                   (const double*)cen, P.ncb, P.nsplit, (const double*)sbest, (const int32_t*)sidx, z, rank,
                   P.np > 0 ? (uint32_t*)nullptr : hist, opart);
    if (P.np > 0) {
      if (ok && d_objective)
        ok = launch_ok((const void*)k_offsets, dim3(1), blk, s, hist, 0, 0, count, (const double*)opart, P.nfb, d_objective + it);
      if (ok && it < iters)
        ok = launch_ok((const void*)k_accumulate, dim3((unsigned)P.np), blk, s, (const double*)ds, ns, (const int32_t*)z, P.ncb, P.chp,
                       (ulonglong2*)hist) &&
             launch_ok((const void*)k_update_chunks, dim3((unsigned)P.ncb), dim3(64), s, (const ulonglong2*)hist, P.np, P.ncb, cen,
                       words);
      continue;
    }
    if (ok && (d_objective || it < iters))
      ok = launch_ok((const void*)k_offsets, dim3(g_off), blk, s, hist, P.nch, P.ncb, count, (const double*)opart, P.nfb,
                     d_objective ? d_objective + it : (double*)nullptr);
    if (ok && it < iters)
      ok = launch_ok((const void*)k_list, dim3(g_list), dim3(kListThreads), s, (const int32_t*)z, (const int32_t*)rank, ns, P.ch,
                     (const uint32_t*)hist, (const uint32_t*)count, P.ncb, start, big, perm) &&
           launch_ok((const void*)k_update, dim3(g_upd), dim3(1024), s, (const double*)ds, (const int32_t*)perm,
                     (const uint32_t*)start, (const uint32_t*)count, (const uint32_t*)big, P.ncb, cen, words);
  }
  if (ok) ok = launch_ok((const void*)k_centres_to_f16, dim3(g_cb), blk, s, (const double*)cen, ncb8, d_codebook);
  return ok ? SPH_OK : SPH_ERR_HIP;
}

}  // extern "C"
