// Training side of SPHQuant on the device: the angular codebook (Sec. 3.3, Eq. 9-10) and the
// pseudo-quantised weight of a linear module (Sec. 3.3; App. A steps 7-8 and 10): radius
// r = softplus(rho), group-wise V-bit fake quantisation with a straight-through estimator, and
// w^_i = r^_i s_i (.) c_{z_i}. The radius, its group offset and step (rounded to fp16, as the
// finalised codes store them) and the level are computed in fp64, so each level is decided in
// fp64; weights, gradients and the angular codebook are fp32, the precision of the fine-tuning.
//
// Work layout:
//   angular kernels   one thread per codebook entry (at most 8192).
//   fake quantisation a block takes whole groups of 16 vectors (128 weights); the radii of a group's
//                     smallest and largest parameter in fp64, one per thread, then levels and weights.
//   gradients         codebooks of up to 256 entries on matrices large enough for them: one pass in storage
//                     order, each wave adding its vectors to sums of its own per centre on the matrix cores.
//                     Otherwise the radius gradient one thread per vector; the vectors are pre-sorted by
//                     direction (a stable counting sort on the host, once per module, since the indices
//                     stay fixed) and the lanes of a centre's slice add its list in fp64. A last
//                     kernel adds the waves' or slices' sums in a fixed order. No sum crosses waves by
//                     atomics: repeated calls are bitwise equal.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "sph_fp.h"
#include "sph_host.h"
#include "sph_layout.h"

namespace {

constexpr int kThreads = 256;
constexpr float kHalfPi = 1.57079632679489662f;

__device__ __forceinline__ float sigmoidf(float x) { return 1.0f / (1.0f + expf(-x)); }

// softplus in fp64 as log(e^0 + e^x) without overflow: log1p(e^x) for x < 0, x + log1p(e^-x) for
// x > 0, log 2 at 0
__device__ __forceinline__ double softplus_d(double x) {
  if (x < 0.0) return log1p(exp(x));
  if (x > 0.0) return x + log1p(exp(-x));
  return 0.69314718055994530942;
}

__device__ __forceinline__ float sum8_pairwise(const float* p) {
  return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
}

// ------------------------------------------------------------------ angular codebook (Eq. 9-10)

// c = C(theta(phi)) for each entry: theta_j = eps + (pi/2 - 2 eps) sigmoid(phi_j),
// c_1 = cos t_1, c_i = (prod_{j<i} sin t_j) cos t_i, c_8 = prod_j sin t_j.
__global__ __launch_bounds__(kThreads) void k_angular_fwd(const float* __restrict__ phi, int ncb, float eps,
                                                          float* __restrict__ cb) {
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (e >= ncb) return;
  const float span = kHalfPi - 2.0f * eps;
  float sprod = 1.0f;
#pragma unroll
  for (int j = 0; j < 7; ++j) {
    float s, c;
    sincosf(eps + span * sigmoidf(phi[e * 7 + j]), &s, &c);
    cb[e * 8 + j] = sprod * c;
    sprod *= s;
  }
  cb[e * 8 + 7] = sprod;
}

// dL/dphi from dL/dc: dc_i/dt_j = c_i cot t_j for j < i (including c_8), -(prod_{k<i} sin t_k)
// sin t_i for j = i <= 7, and 0 for j > i; dt_j/dphi_j = (pi/2 - 2 eps) s (1 - s).
__global__ __launch_bounds__(kThreads) void k_angular_bwd(const float* __restrict__ phi, int ncb, float eps,
                                                          const float* __restrict__ gc, float* __restrict__ gphi) {
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (e >= ncb) return;
  const float span = kHalfPi - 2.0f * eps;
  float sg[7], sn[7], cs[7], c[8], pre[7];
  float sprod = 1.0f;
#pragma unroll
  for (int j = 0; j < 7; ++j) {
    sg[j] = sigmoidf(phi[e * 7 + j]);
    sincosf(eps + span * sg[j], &sn[j], &cs[j]);
    pre[j] = sprod;
    c[j] = sprod * cs[j];
    sprod *= sn[j];
  }
  c[7] = sprod;
  float g[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) g[i] = gc[e * 8 + i];
  float later = g[7] * c[7];  // sum over i > j of g_i c_i, built from the back
#pragma unroll
  for (int j = 6; j >= 0; --j) {
    const float dth = later * cs[j] / sn[j] - g[j] * pre[j] * sn[j];
    gphi[e * 7 + j] = dth * span * sg[j] * (1.0f - sg[j]);
    later += g[j] * c[j];
  }
}

// Inverse of Eq. 9-10 for a non-negative unit direction: theta_i = atan2(||c_{i+1..8}||, c_i),
// t = clamp((theta - eps) / (pi/2 - 2 eps), 1e-6, 1 - 1e-6), phi = log t - log(1 - t).
__global__ __launch_bounds__(kThreads) void k_angular_logits(const float* __restrict__ cb, int ncb, float eps,
                                                             float* __restrict__ phi) {
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (e >= ncb) return;
  const float span = kHalfPi - 2.0f * eps;
  float c[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) c[i] = cb[e * 8 + i];
  float tail2 = c[7] * c[7];
#pragma unroll
  for (int j = 6; j >= 0; --j) {
    const float th = atan2f(sqrtf(tail2), c[j]);
    const float t = fminf(fmaxf((th - eps) / span, 1e-6f), 1.0f - 1e-6f);
    phi[e * 7 + j] = logf(t) - log1pf(-t);
    tail2 += c[j] * c[j];
  }
}

// ------------------------------------------------------------------ pseudo-quantised weights

struct FqArgs {
  int64_t nv, nvec;
  const float* rho;
  const uint8_t* signs;
  const uint16_t* dir;
  const float* cb;
  int vmax;
  float* w_hat;
  int64_t ldw;
  float* r_hat;
  uint8_t* q;
  uint16_t* gmin;
  uint16_t* gstep;
};

// softplus in fp32 with a relative error of a few 2^-24 (times 1 + |x| for e^x): log1p(y) as
// log(u) * y / (u - 1) for u = 1 + y, where the two roundings of u cancel.
__device__ __forceinline__ float softplus_f(float x) {
  const float y = __expf(-fabsf(x));
  const float u = 1.0f + y;
  const float l = u == 1.0f ? y : __logf(u) * (y / (u - 1.0f));
  return fmaxf(x, 0.0f) + l;
}

template <int CTRL>
__device__ __forceinline__ float row_ror(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// r = softplus(rho); per group of 16 vectors the offset min r and the step (max - min)/(2^V - 1),
// both rounded to fp16; q = clip(round((r - min)/step), 0, 2^V - 1), half to even (0 for a zero
// step); r^ = min + q step; w^ = r^ s (.) c_z, stored as fp32 with r^. Every decision is the fp64 one:
// softplus is increasing, so a group's offset and step come from its smallest and largest rho, two
// fp64 evaluations per 16 vectors, one per thread of the block; a level is rounded from fp32 unless the
// quotient lies within its error of a rounding boundary, and then from fp64 (about one vector in 10^4).
// The weights' products are single fp32 roundings of exact factors (fp64 where r^ needs more than 24 bits).
// Optional outputs: r^, and the finalised codes (levels, fp16 offsets and steps).
//
// Bound by memory: 43 bytes per vector, 32 of them written, so the weights go out 16 bytes per lane in
// address order through LDS (32 contiguous bytes per thread, as they are computed, touch every line twice). 12288x4096 W2: 80 us
// with fp64 softplus for every vector -> 71 us.
template <int VPT>   // vectors per thread
__global__ __launch_bounds__(kThreads) void k_fq_forward(FqArgs a) {
  constexpr int NVB = VPT * kThreads, NG = NVB / 16;
  __shared__ float ext[NG][2];       // smallest and largest rho of a group
  __shared__ float par[NG][2];       // offset and step
  __shared__ float rad[NVB], low[NVB];   // r^ as two fp32 words
  __shared__ uint32_t dz[NVB];       // direction and signs
  __shared__ int wide;               // some r^ needs its second word
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * NVB;
  if (tid == 0) wide = 0;
  float x[VPT];
#pragma unroll
  for (int t = 0; t < VPT; ++t) {
    const int64_t i = base + t * kThreads + tid;   // whole groups are inside or outside together
    x[t] = i < a.nvec ? a.rho[i] : 0.0f;
    if (i < a.nvec) dz[t * kThreads + tid] = (uint32_t)a.dir[i] | ((uint32_t)a.signs[i] << 16);
  }
#pragma unroll
  for (int t = 0; t < VPT; ++t) {
    if (x[t] != x[t]) x[t] = 0.0f;   // softplus_d's value without a number, log 2, is softplus(0)
    float lo = x[t], hi = x[t];
    lo = fminf(lo, row_ror<0x128>(lo));
    hi = fmaxf(hi, row_ror<0x128>(hi));
    lo = fminf(lo, row_ror<0x124>(lo));
    hi = fmaxf(hi, row_ror<0x124>(hi));
    lo = fminf(lo, row_ror<0x122>(lo));
    hi = fmaxf(hi, row_ror<0x122>(hi));
    lo = fminf(lo, row_ror<0x121>(lo));
    hi = fmaxf(hi, row_ror<0x121>(hi));
    if ((tid & 15) == 0) {
      ext[(t * kThreads + tid) >> 4][0] = lo;
      ext[(t * kThreads + tid) >> 4][1] = hi;
    }
  }
  __syncthreads();
  if (tid < 2 * NG) {
    const int g = tid >> 1;
    const double r = softplus_d((double)ext[g][tid & 1]);
    const double o = __shfl_xor(r, 1, 64);
    const double lo = (tid & 1) ? o : r, hi = (tid & 1) ? r : o;
    const uint16_t lo16 = d2h(lo), st16 = d2h((hi - lo) / (double)a.vmax);
    const int64_t grp = (base >> 4) + g;
    if ((tid & 1) == 0) {
      par[g][0] = (float)h2d(lo16);
      par[g][1] = (float)h2d(st16);
      if (a.gmin && grp * 16 < a.nvec) {
        a.gmin[grp] = lo16;
        a.gstep[grp] = st16;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < VPT; ++t) {
    const int o = t * kThreads + tid;
    const int64_t i = base + o;
    const float lo = par[o >> 4][0], st = par[o >> 4][1];
    int q = 0;
    bool close = false;
    if (st > 0.0f) {
      const float r = softplus_f(x[t]), inv = 1.0f / st;
      const float v = (r - lo) * inv;
      const float err = fmaf(4e-6f * (1.0f + fabsf(x[t])) * (r + fabsf(lo)), inv, 1e-5f);
      const float k = rintf(v);
      close = !(fabsf(fabsf(v - k) - 0.5f) > err);   // also where an overflow leaves no number
      q = (int)fminf(fmaxf(k, 0.0f), (float)a.vmax);
    }
    if (__any(close) && close)
      q = (int)fmin(fmax(rint((softplus_d((double)x[t]) - (double)lo) / (double)st), 0.0), (double)a.vmax);
    const double rh = (double)lo + (double)q * (double)st;
    const float rf = (float)rh, rl = (float)(rh - (double)rf);
    rad[o] = rf;
    low[o] = rl;
    if (rl != 0.0f) wide = 1;
    if (i < a.nvec) {
      if (a.r_hat) a.r_hat[i] = rf;
      if (a.q) a.q[i] = (uint8_t)q;
    }
  }
  __syncthreads();
  const bool two = wide != 0;
  const bool packed = a.ldw == a.nv * 8;
  const float4* cb4 = reinterpret_cast<const float4*>(a.cb);
#pragma unroll 4
  for (int t = 0; t < 2 * VPT; ++t) {
    const int o = t * kThreads + tid, v = o >> 1, half = o & 1;
    const int64_t i = base + v;
    if (i >= a.nvec) break;
    const uint32_t zs = dz[v], s = zs >> (16 + 4 * half);
    const float4 c = cb4[(int64_t)(zs & 0xFFFFu) * 2 + half];
    const float rf = rad[v];
    float m[4] = {rf * c.x, rf * c.y, rf * c.z, rf * c.w};
    if (two) {
      const double rh = (double)rf + (double)low[v];
      m[0] = (float)(rh * (double)c.x);
      m[1] = (float)(rh * (double)c.y);
      m[2] = (float)(rh * (double)c.z);
      m[3] = (float)(rh * (double)c.w);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if ((s >> j) & 1) m[j] = -m[j];
    const int64_t row = packed ? 0 : i / a.nv;
    *reinterpret_cast<float4*>(a.w_hat + row * a.ldw + (i - row * a.nv) * 8 + half * 4) = make_float4(m[0], m[1], m[2], m[3]);
  }
}

// rho from Eq. 6's radius r~ = <|w|, c_z> (floored at 1e-6) through the inverse of softplus.
__global__ __launch_bounds__(kThreads) void k_fq_init_rho(const float* __restrict__ w, int64_t ldw, int64_t nv,
                                                          int64_t nvec, const uint16_t* __restrict__ dir,
                                                          const float* __restrict__ cb, float* __restrict__ rho) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= nvec) return;
  const int64_t row = i / nv, v = i - row * nv;
  const float4* p = reinterpret_cast<const float4*>(w + row * ldw + v * 8);
  const float4* c4 = reinterpret_cast<const float4*>(cb + (int64_t)dir[i] * 8);
  const float4 x0 = p[0], x1 = p[1], c0 = c4[0], c1 = c4[1];
  const float pr[8] = {fabsf(x0.x) * c0.x, fabsf(x0.y) * c0.y, fabsf(x0.z) * c0.z, fabsf(x0.w) * c0.w,
                       fabsf(x1.x) * c1.x, fabsf(x1.y) * c1.y, fabsf(x1.z) * c1.z, fabsf(x1.w) * c1.w};
  const float rt = fmaxf(sum8_pairwise(pr), 1e-6f);
  rho[i] = rt > 20.0f ? rt + log1pf(-expf(-rt)) : logf(expm1f(rt));
}

__host__ __device__ __forceinline__ int64_t stretch_begin(int64_t nvec, int b, int nblk);

// dL/drho_i = sigmoid(rho_i) * sum_j dL/dw^_ij s_ij c_{z_i, j} (straight-through: dr^/dr = 1).
__global__ __launch_bounds__(kThreads) void k_fq_grad_rho(int64_t nv, int64_t nvec, const float* __restrict__ rho,
                                                          const uint8_t* __restrict__ signs,
                                                          const uint16_t* __restrict__ dir,
                                                          const float* __restrict__ cb, const float* __restrict__ gw,
                                                          int64_t ldg, int first, int nblk, float* __restrict__ grho) {
  // all vectors, or with nblk > 0 the first `first` of each of nblk stretches (see k_fq_grad_pass)
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (nblk > 0) {
    if (i >= (int64_t)first * nblk) return;
    i = stretch_begin(nvec, (int)(i / first), nblk) + i % first;
  }
  if (i >= nvec) return;
  const int64_t row = i / nv, v = i - row * nv;
  const float4* g4 = reinterpret_cast<const float4*>(gw + row * ldg + v * 8);
  const float4* c4 = reinterpret_cast<const float4*>(cb + (int64_t)dir[i] * 8);
  const float4 g0 = g4[0], g1 = g4[1], c0 = c4[0], c1 = c4[1];
  const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
  const float c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
  const uint32_t s = signs[i];
  float p[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) p[j] = ((s >> j) & 1) ? -g[j] * c[j] : g[j] * c[j];
  grho[i] = sum8_pairwise(p) * sigmoidf(rho[i]);
}

// Slice sl of a centre's direction-sorted vector list: sum of r^_i s_i (.) dL/dw^_i, two lanes per vector
// (16 bytes of the gradient each) and U vectors at a time, in fp64, then over the lanes by a fixed
// tree; stored as fp32 in part[slice][centre][8]. A block holds G centres, 256 / G lanes each, and then takes
// those of them together whose slice is longer than `most`: weight vectors with one large coordinate lie near an
// axis and crowd into a few centres, and eight lanes alone take as long as such a list is (W3, the sums in
// the workspace: 1024x4096 encoded 47 -> 30 us, 1024x1024 with nine vectors in ten in one centre 4.7 -> 0.21 ms).
//
// G = 32 where the radius gradient's array holds eight slices or more, G = 4 for 2^13 centres otherwise (a
// wave per centre: 1024x4096 encoded 30 us against 31 with G = 1 and 47 with 32, 256x1024 12 against
// 25 and 11), G = 1 for up to 256 centres, which have no more blocks to offer.
//
// The gradient's 32 bytes per vector are gathered in list order; neighbouring vectors belong to
// different centres, so a cache line is read by up to four of them. A slice covers about one
// stretch of the matrix for all centres, and block ids that are equal modulo 8 share an L2, so a
// slice's blocks take ids of one residue: its lines come from memory once. (The finest useful slices: a
// step of 12288x4096 W3, 8192 centres, 500 us with one block of 256 threads per centre -> 348 us.)
constexpr int kXcd = 8;

template <int G>
__global__ __launch_bounds__(kThreads) void k_fq_grad_cb_part(int64_t nv, const float* __restrict__ r_hat,
                                                              const uint8_t* __restrict__ signs,
                                                              const float* __restrict__ gw, int64_t ldg,
                                                              const int32_t* __restrict__ perm,
                                                              const int64_t* __restrict__ off, int ncb, int nslice, int most,
                                                              float* __restrict__ part) {
  constexpr int L = kThreads / G;          // lanes per centre
  constexpr int U = G == 1 ? 8 : 4;        // vectors in flight per pair of lanes
  static_assert(G == 1 || (L >= 8 && L <= 64), "a block, or lanes of one wave");
  __shared__ double sh[kThreads / 64][8];
  const int ncblk = (ncb + G - 1) / G;
  const int nx = nslice % kXcd == 0 ? kXcd : 1;
  const int xcd = blockIdx.x % nx, seq = blockIdx.x / nx;
  const int sl = seq / ncblk * nx + xcd, cfirst = seq % ncblk * G;
  const int half = threadIdx.x & 1;
  const bool packed = ldg == nv * 8;
  double acc[4];
  auto add = [&](float rh, uint32_t s, const float4 g) {
    const float p[4] = {rh * g.x, rh * g.y, rh * g.z, rh * g.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] += (double)(((s >> (4 * half + j)) & 1) ? -p[j] : p[j]);
  };
  auto grad = [&](int64_t i) {
    const int64_t row = packed ? 0 : i / nv;
    return *reinterpret_cast<const float4*>(gw + row * ldg + (i - row * nv) * 8 + 4 * half);
  };
  // every step-th vector of the list's places [t, b1)
  auto walk = [&](int64_t t, int64_t b1, int step) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = 0.0;
    for (; t + step * (U - 1) < b1; t += step * U) {
      int64_t i[U];
      float rh[U];
      uint32_t s[U];
      float4 g[U];
#pragma unroll
      for (int u = 0; u < U; ++u) i[u] = perm[t + step * u];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        rh[u] = r_hat[i[u]];
        s[u] = signs[i[u]];
        g[u] = grad(i[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) add(rh[u], s[u], g[u]);
    }
    for (; t < b1; t += step) {
      const int64_t i = perm[t];
      add(r_hat[i], signs[i], grad(i));
    }
  };
  auto over_lanes = [&](int lanes) {
#pragma unroll
    for (int o = 2; o < 64; o <<= 1)
      if (o < lanes)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] += __shfl_xor(acc[j], o, 64);
  };
  auto bounds = [&](int c, int64_t& b0, int64_t& b1) {
    const int64_t a0 = off[c], len = off[c + 1] - a0;
    b0 = a0 + len * sl / nslice;
    b1 = a0 + len * (sl + 1) / nslice;
  };
  auto store = [&](int c, const double (&v)[4]) {
    *reinterpret_cast<float4*>(part + ((int64_t)sl * ncb + c) * 8 + 4 * half) = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
  };
  if constexpr (G > 1) {
    const int c = cfirst + (int)threadIdx.x / L;
    int64_t b0 = 0, b1 = 0;
    if (c < ncb) bounds(c, b0, b1);
    const bool mine = c < ncb && b1 - b0 <= most;
    walk(b0 + (threadIdx.x % L >> 1), mine ? b1 : b0, L / 2);
    over_lanes(L);
    if (mine && threadIdx.x % L < 2) store(c, acc);
    if (!__syncthreads_or(c < ncb && !mine)) return;
  }
  const int cend = min(ncb, cfirst + G);
  for (int c = cfirst; c < cend; ++c) {   // the same for all threads
    int64_t b0, b1;
    bounds(c, b0, b1);
    if (G > 1 && b1 - b0 <= most) continue;
    walk(b0 + (threadIdx.x >> 1), b1, kThreads / 2);
    over_lanes(64);
    __syncthreads();                      // the last centre's sums have been read
    if ((threadIdx.x & 63) < 2)
#pragma unroll
      for (int j = 0; j < 4; ++j) sh[threadIdx.x >> 6][4 * half + j] = acc[j];
    __syncthreads();
    if (threadIdx.x < 2) {
      double v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (sh[0][4 * half + j] + sh[1][4 * half + j]) + (sh[2][4 * half + j] + sh[3][4 * half + j]);
      store(c, v);
    }
  }
}

// Both gradients in one pass over dL/dW^, for codebooks of at most NCB entries (16, 64 or 256). A wave walks its
// stretch of the vectors in storage order, 32 at a time (two lanes per vector, 16 bytes of the gradient
// each): dL/drho directly, and r^ s (.) dL/dw^ summed per centre on the matrix cores, as the product of
// a one-hot matrix (16 centres x 32 vectors; exact ones and zeros) with the 32 x 8 products. Each
// product is cut into three bfloat16 words (8 + 8 + 8 bits: exactly its 24): the high and middle words of the
// 8 coordinates are the 16 columns of one operand, the low words half of another. The words and the
// directions reach the operands' layout through a few LDS rows of the wave's own. Adding an
// exact zero rounds nothing, so a sum is rounded as often as a centre's vectors are added. Products
// that are not finite would spoil every centre (0 times infinity); a wave that meets one takes its vectors again
// and adds such products to their centre in LDS instead.
//
// The matrix cores take subnormal bfloat16 words as zero, which unscaled would cost products below 2^-110 their low
// words (gradients of 1e-33: error 8e-7 of the sums, of 1e-37: 8e-3). The radius carries a factor of 2^24 into the
// products, so that the low words of every normal fp32 product stay normal. A wave that meets a product beyond
// 2^80 takes its vectors again with 2^-40, so that no sum of finite products overflows before its own size does. (The
// same loop with that case inside it took 3% longer.)
//
// The waves' sums are added in order (fp64) per block and stored as fp32, in d_ws where it holds all
// blocks' sums, else in the radius gradient's first ncb * 8 values of the block's stretch, which
// k_fq_grad_rho fills afterwards.
//
// 47 bytes per vector, read and written once and in order. The gather of the lists by centre (above)
// moved a 128-byte line into L1 for each 32-byte gradient, each radius and each sign byte: 2.4 GB for
// 12288x4096, 244 us, and the radius gradient took another 55 us; this pass takes 96
// us, the vector ALUs busy 73% of it (the cuts and the one-hot words). Additions to
// the wave's sums in LDS (ds_add_f32) took 260 us, one lane every three cycles.
constexpr int kPassWaves = 8;
constexpr float kPassUp = 0x1p24f, kPassDown = 0x1p-40f, kPassMost = 0x1p104f;
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint16_t u2s __attribute__((ext_vector_type(2)));

struct PassArgs {
  int64_t nv, nvec;
  const float* rho;
  const uint8_t* signs;
  const uint16_t* dir;
  const float* cb;
  const float* r_hat;
  const float* gw;
  int64_t ldg;
  float* grho;
  float* part;     // [blocks][ncb * 8], or null: the first values of each block's stretch of grho
  int ncb;
};

// Block b's stretch: whole groups of 16 vectors, nearly equal.
__host__ __device__ __forceinline__ int64_t stretch_begin(int64_t nvec, int b, int nblk) { return nvec / 16 * b / nblk * 16; }

template <int NCB>
__global__ __launch_bounds__(64 * kPassWaves) void k_fq_grad_pass(PassArgs a) {
  constexpr int NT = NCB / 16;                    // tiles of 16 centres
  constexpr int ROW = 40;                         // bf16 words per row of 32 vectors, padded against bank conflicts
  __shared__ __align__(16) uint16_t words[kPassWaves][24 * ROW];   // rows: word (high, middle, low) x coordinate
  __shared__ __align__(16) uint16_t zs[kPassWaves][32];
  __shared__ float sums[kPassWaves][NCB * 8];     // the waves' sums, at the end (added one wave after the
                                                  // other in one array, the tail took 8 to 75 us more)
  __shared__ float odd[NCB * 8];                  // products that are not finite
  __shared__ float4 cbl[NCB * 2];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nval = a.ncb * 8;
  for (int t = tid; t < a.ncb * 2; t += 64 * kPassWaves) cbl[t] = reinterpret_cast<const float4*>(a.cb)[t];
  for (int t = tid; t < NCB * 8; t += 64 * kPassWaves) odd[t] = 0.0f;
  __syncthreads();
  const int64_t b0 = stretch_begin(a.nvec, blockIdx.x, gridDim.x), b1 = stretch_begin(a.nvec, blockIdx.x + 1, gridDim.x);
  const int64_t keep = a.part ? b0 : b0 + nval;   // radius gradients before it are left for later
  const int64_t per = ((b1 - b0 + kPassWaves - 1) / kPassWaves + 31) / 32 * 32;
  const int64_t w0 = min(b1, b0 + wv * per), w1 = min(b1, w0 + per);
  const int half = lane & 1, own = lane >> 1;
  const int r = lane & 15, kb = lane >> 4;        // row (or column) and block of 8 vectors of an operand
  const bool packed = a.ldg == a.nv * 8;
  uint16_t* wr = words[wv] + 4 * half * ROW + own;
  const uint16_t* rd1 = words[wv] + r * ROW + kb * 8;
  const uint16_t* rd2 = words[wv] + (16 + (r & 7)) * ROW + kb * 8;
  f4v hm[NT], lw[NT];   // sums of their own for the low words: chained into the others they cost 10%
  bool again = false;
  // the wave's vectors; CAREFUL: the small scale, and products that are not finite apart
  auto run = [&](auto careful) {
    constexpr bool CAREFUL = decltype(careful)::value;
    constexpr float up = CAREFUL ? kPassDown : kPassUp;
    constexpr int U = 2;
#pragma unroll
    for (int t = 0; t < NT; ++t) hm[t] = lw[t] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
    for (int64_t i0 = w0; i0 < w1; i0 += 32 * U) {
      float4 g[U];
      float rho[U], rh[U];
      uint32_t z[U], s[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = min(i0 + 32 * u + own, w1 - 1);   // past the end: the last vector again, not counted
        const int64_t row = packed ? 0 : i / a.nv;
        g[u] = *reinterpret_cast<const float4*>(a.gw + row * a.ldg + (i - row * a.nv) * 8 + 4 * half);
        rho[u] = a.rho[i];
        rh[u] = a.r_hat[i];
        z[u] = a.dir[i];
        s[u] = (uint32_t)a.signs[i] >> (4 * half);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + 32 * u + own;
        const bool ok = i < w1;
        const float4 c = cbl[z[u] * 2 + half];
        const float gg[4] = {g[u].x, g[u].y, g[u].z, g[u].w};
        const float cc[4] = {c.x, c.y, c.z, c.w};
        float p[4], q[4];
        [[maybe_unused]] bool fine = true;
        const float rs = rh[u] * up;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float sg = ((s[u] >> j) & 1) ? -gg[j] : gg[j];
          p[j] = sg * cc[j];
          q[j] = ok ? rs * sg : 0.0f;
          if constexpr (CAREFUL) {
            const float raw = ok ? rh[u] * sg : 0.0f;
            if (!(fabsf(raw) <= 3.402823466e38f)) {
              atomicAdd(&odd[z[u] * 8 + 4 * half + j], raw);
              q[j] = 0.0f;
            }
          } else {
            fine = fine && fabsf(q[j]) <= kPassMost;
          }
        }
        if constexpr (!CAREFUL) {
          again = again || !fine;
          const float mysum = (p[0] + p[1]) + (p[2] + p[3]);
          const float total = mysum + __shfl_xor(mysum, 1, 64);   // the pairwise order of eight terms
          if (half == 0 && ok && i >= keep) a.grho[i] = total * sigmoidf(rho[u]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t b = __builtin_bit_cast(uint32_t, q[j]);
          const float r1 = q[j] - __builtin_bit_cast(float, b & 0xFFFF0000u);
          const uint32_t m = __builtin_bit_cast(uint32_t, r1);
          const float r2 = r1 - __builtin_bit_cast(float, m & 0xFFFF0000u);
          wr[j * ROW] = (uint16_t)(b >> 16);
          wr[(8 + j) * ROW] = (uint16_t)(m >> 16);
          wr[(16 + j) * ROW] = (uint16_t)(__builtin_bit_cast(uint32_t, r2) >> 16);
        }
        if (half == 0) zs[wv][own] = (uint16_t)z[u];
        // the LDS performs a wave's operations in issue order: these reads see the writes above, and
        // the next vectors' writes come after them
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint4 zq = *(const uint4*)(zs[wv] + kb * 8);
        const bf8v x1 = *(const bf8v*)rd1;
        uint4 x2w = *(const uint4*)rd2;
        if (r >= 8) x2w = make_uint4(0, 0, 0, 0);
        const bf8v x2 = __builtin_bit_cast(bf8v, x2w);
        const uint32_t zw[4] = {zq.x, zq.y, zq.z, zq.w};
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const uint32_t c2 = (uint32_t)(16 * t + r) * 0x10001u;
          uint32_t o[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const u2s d = __builtin_elementwise_min(__builtin_bit_cast(u2s, zw[k] ^ c2), u2s{1, 1});
            o[k] = __builtin_bit_cast(uint32_t, (u2s)(u2s{0x3F80, 0x3F80} - d * u2s{0x3F80, 0x3F80}));   // 1.0 where equal
          }
          const bf8v one = __builtin_bit_cast(bf8v, make_uint4(o[0], o[1], o[2], o[3]));
          hm[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(one, x1, hm[t], 0, 0, 0);
          lw[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(one, x2, lw[t], 0, 0, 0);
        }
      }
    }
  };
  run(std::false_type{});
  const bool redo = __any(again);
  if (redo) run(std::true_type{});
  const double down = redo ? 1.0 / kPassDown : 1.0 / kPassUp;
  // lane (column, rows 4 * kb + e) of tile t: high words in columns 0..7, middle in 8..15, low in 0..7
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float mid = __shfl_xor(hm[t][e], 8, 64);
      if (r < 8) sums[wv][(16 * t + 4 * kb + e) * 8 + r] = (float)(((double)hm[t][e] + ((double)mid + (double)lw[t][e])) * down);
    }
  __syncthreads();
  float* out = a.part ? a.part + (int64_t)blockIdx.x * nval : a.grho + b0;
  for (int t = tid; t < nval; t += 64 * kPassWaves) {
    double sum = (double)odd[t];
#pragma unroll
    for (int k = 0; k < kPassWaves; ++k) sum += (double)sums[k][t];
    out[t] = (float)sum;
  }
}

// The sums of 32 consecutive values per block, 32 lanes over the slices (or blocks of k_fq_grad_pass,
// whose sums lie in their stretches of nvec vectors if that is not 0) in fp64, added in a fixed order.
__global__ __launch_bounds__(1024) void k_fq_grad_cb_final(const float* __restrict__ part, int nval, int nslice, int64_t nvec,
                                                           float* __restrict__ gcb) {
  __shared__ double sh[32][33];
  const int v = threadIdx.x & 31, l = threadIdx.x >> 5;
  const int64_t o = (int64_t)blockIdx.x * 32 + v;
  double s = 0.0;
  if (o < nval) {
#pragma unroll 4
    for (int t = l; t < nslice; t += 32) s += (double)part[(nvec ? stretch_begin(nvec, t, nslice) : (int64_t)t * nval) + o];
  }
  sh[l][v] = s;
  __syncthreads();
  if (l == 0 && o < nval) {
#pragma unroll
    for (int k = 1; k < 32; ++k) s += sh[k][v];
    gcb[o] = (float)s;
  }
}

// ------------------------------------------------------------------------------------ host side

// Slices of every centre's list: enough groups of eight lanes to fill the chip (65,536), at least 32 so that
// a slice's stretch of a large matrix stays near an XCD's 4 MiB of L2.
int slices_for(int ncb) { return std::max(32, std::min(1024, 65536 / ncb)); }

// Slices the caller's workspace holds (its size is part of the interface). Most matrices use the
// radius gradient's array instead, which is written last.
int ws_slices(int ncb) { return std::max(1, std::min(64, (1024 + ncb - 1) / ncb)); }

template <typename... A>
bool launch_ok(const void* fn, dim3 grid, dim3 block, hipStream_t s, A... args) {
  void* kargs[] = {(void*)&args...};
  if (hipLaunchKernel(fn, grid, block, kargs, 0, s) != hipSuccess) return false;
  return hipGetLastError() == hipSuccess;
}

bool dir_bits_ok(int32_t d) { return d >= 1 && d <= 13; }

// The fine-tuning kernels handle 8-D vectors (the 4-D and 16-D formats are decode-only).
int check_fq(const sph_format* fmt, int64_t n, int64_t k) {
  int st = sph_host_check_format(fmt);
  if (st) return st;
  if (fmt->vec_dim != SPH_VEC) return SPH_ERR_UNSUPPORTED_FORMAT;
  return sph_host_check_shape(n, k);
}

bool a16(const void* p) { return (uintptr_t)p % 16 == 0; }

}  // namespace

extern "C" {

sph_status sph_angular_codebook(int32_t dir_bits, const float* d_phi, float eps, float* d_codebook, void* stream) {
  if (!d_phi || !d_codebook) return SPH_ERR_NULL;
  if (!dir_bits_ok(dir_bits) || !(eps >= 0.0f && eps < 0.25f)) return SPH_ERR_SHAPE;
  const int ncb = 1 << dir_bits;
  return launch_ok((const void*)k_angular_fwd, dim3((ncb + kThreads - 1) / kThreads), dim3(kThreads),
                   (hipStream_t)stream, d_phi, ncb, eps, d_codebook)
             ? SPH_OK
             : SPH_ERR_HIP;
}

sph_status sph_angular_codebook_backward(int32_t dir_bits, const float* d_phi, float eps, const float* d_grad_codebook,
                                         float* d_grad_phi, void* stream) {
  if (!d_phi || !d_grad_codebook || !d_grad_phi) return SPH_ERR_NULL;
  if (!dir_bits_ok(dir_bits) || !(eps >= 0.0f && eps < 0.25f)) return SPH_ERR_SHAPE;
  const int ncb = 1 << dir_bits;
  return launch_ok((const void*)k_angular_bwd, dim3((ncb + kThreads - 1) / kThreads), dim3(kThreads),
                   (hipStream_t)stream, d_phi, ncb, eps, d_grad_codebook, d_grad_phi)
             ? SPH_OK
             : SPH_ERR_HIP;
}

sph_status sph_angular_logits(int32_t dir_bits, const float* d_codebook, float eps, float* d_phi, void* stream) {
  if (!d_phi || !d_codebook) return SPH_ERR_NULL;
  if (!dir_bits_ok(dir_bits) || !(eps >= 0.0f && eps < 0.25f)) return SPH_ERR_SHAPE;
  const int ncb = 1 << dir_bits;
  return launch_ok((const void*)k_angular_logits, dim3((ncb + kThreads - 1) / kThreads), dim3(kThreads),
                   (hipStream_t)stream, d_codebook, ncb, eps, d_phi)
             ? SPH_OK
             : SPH_ERR_HIP;
}

sph_status sph_direction_groups(int32_t dir_bits, int64_t count, const uint16_t* dir_idx, int32_t* perm,
                                int64_t* offsets) {
  if (!dir_idx || !perm || !offsets) return SPH_ERR_NULL;
  if (!dir_bits_ok(dir_bits) || count < 1 || count > INT32_MAX) return SPH_ERR_SHAPE;
  const int64_t ncb = int64_t(1) << dir_bits;
  std::vector<int64_t> cnt(ncb + 1, 0);
  for (int64_t i = 0; i < count; ++i) {
    if (dir_idx[i] >= ncb) return SPH_ERR_CODE_RANGE;
    ++cnt[dir_idx[i] + 1];
  }
  for (int64_t c = 0; c < ncb; ++c) cnt[c + 1] += cnt[c];
  for (int64_t c = 0; c <= ncb; ++c) offsets[c] = cnt[c];
  for (int64_t i = 0; i < count; ++i) perm[cnt[dir_idx[i]]++] = (int32_t)i;
  return SPH_OK;
}

sph_status sph_fake_quant_init_rho(const sph_format* fmt, int64_t n, int64_t k, const float* d_w, int64_t ldw,
                                   const uint16_t* d_dir_idx, const float* d_codebook, float* d_rho, void* stream) {
  if (!fmt || !d_w || !d_dir_idx || !d_codebook || !d_rho) return SPH_ERR_NULL;
  const int st = check_fq(fmt, n, k);
  if (st) return (sph_status)st;
  if (ldw < k || ldw % 4 || !a16(d_w) || !a16(d_codebook) || (uintptr_t)d_dir_idx % 2 || (uintptr_t)d_rho % 4)
    return SPH_ERR_SHAPE;
  const int64_t nv = k / SPH_VEC, nvec = n * nv;
  return launch_ok((const void*)k_fq_init_rho, dim3((unsigned)((nvec + kThreads - 1) / kThreads)), dim3(kThreads),
                   (hipStream_t)stream, d_w, ldw, nv, nvec, d_dir_idx, d_codebook, d_rho)
             ? SPH_OK
             : SPH_ERR_HIP;
}

sph_status sph_fake_quant_forward(const sph_format* fmt, int64_t n, int64_t k, const float* d_rho,
                                  const uint8_t* d_signs, const uint16_t* d_dir_idx, const float* d_codebook,
                                  float* d_w_hat, int64_t ldw, float* d_r_hat, uint8_t* d_radius_code,
                                  uint16_t* d_group_min, uint16_t* d_group_step, void* stream) {
  if (!fmt || !d_rho || !d_signs || !d_dir_idx || !d_codebook || !d_w_hat) return SPH_ERR_NULL;
  const int st = check_fq(fmt, n, k);
  if (st) return (sph_status)st;
  if ((d_radius_code || d_group_min || d_group_step) && !(d_radius_code && d_group_min && d_group_step))
    return SPH_ERR_NULL;
  if (ldw < k || ldw % 4 || !a16(d_w_hat) || !a16(d_codebook) || (uintptr_t)d_rho % 4 || (uintptr_t)d_dir_idx % 2 ||
      (uintptr_t)d_r_hat % 4 || (uintptr_t)d_group_min % 2 || (uintptr_t)d_group_step % 2)
    return SPH_ERR_SHAPE;
  FqArgs a{};
  a.nv = k / SPH_VEC;
  a.nvec = n * a.nv;
  a.rho = d_rho;
  a.signs = d_signs;
  a.dir = d_dir_idx;
  a.cb = d_codebook;
  a.vmax = (1 << fmt->radius_bits) - 1;
  a.w_hat = d_w_hat;
  a.ldw = ldw;
  a.r_hat = d_r_hat;
  a.q = d_radius_code;
  a.gmin = d_group_min;
  a.gstep = d_group_step;
  // eight vectors per thread fill the chip from 1024 blocks on; smaller matrices take two
  const int64_t big = (a.nvec + 8 * kThreads - 1) / (8 * kThreads);
  const bool two = big < 1024;
  const int64_t grid = two ? (a.nvec + 2 * kThreads - 1) / (2 * kThreads) : big;
  return launch_ok(two ? (const void*)k_fq_forward<2> : (const void*)k_fq_forward<8>, dim3((unsigned)grid), dim3(kThreads),
                   (hipStream_t)stream, a)
             ? SPH_OK
             : SPH_ERR_HIP;
}

sph_status sph_fake_quant_backward_workspace_bytes(int32_t dir_bits, size_t* bytes) {
  if (!bytes) return SPH_ERR_NULL;
  if (!dir_bits_ok(dir_bits)) return SPH_ERR_SHAPE;
  const int ncb = 1 << dir_bits;
  *bytes = (size_t)ncb * ws_slices(ncb) * 8 * sizeof(float);
  return SPH_OK;
}

sph_status sph_fake_quant_backward(const sph_format* fmt, int64_t n, int64_t k, const float* d_rho,
                                   const uint8_t* d_signs, const uint16_t* d_dir_idx, const float* d_codebook,
                                   const float* d_r_hat, const float* d_grad_w, int64_t ldg, const int32_t* d_perm,
                                   const int64_t* d_offsets, float* d_grad_rho, float* d_grad_codebook, void* d_ws,
                                   size_t ws_bytes, void* stream) {
  if (!fmt || !d_rho || !d_signs || !d_dir_idx || !d_codebook || !d_r_hat || !d_grad_w || !d_perm || !d_offsets ||
      !d_grad_rho || !d_grad_codebook || !d_ws)
    return SPH_ERR_NULL;
  const int st = check_fq(fmt, n, k);
  if (st) return (sph_status)st;
  if (ldg < k || ldg % 4 || !a16(d_grad_w) || !a16(d_codebook) || (uintptr_t)d_rho % 4 || (uintptr_t)d_r_hat % 4 ||
      (uintptr_t)d_dir_idx % 2 || (uintptr_t)d_perm % 4 || (uintptr_t)d_offsets % 8 || (uintptr_t)d_grad_rho % 4 ||
      (uintptr_t)d_grad_codebook % 4 || (uintptr_t)d_ws % 16)
    return SPH_ERR_SHAPE;
  const int ncb = 1 << fmt->dir_bits;
  const int64_t nv = k / SPH_VEC, nvec = n * nv;
  if (ws_bytes < (size_t)ncb * ws_slices(ncb) * 8 * sizeof(float)) return SPH_ERR_BUFFER_TOO_SMALL;
  hipStream_t s = (hipStream_t)stream;
  const int nval = ncb * 8;
  // The radius gradient's array may hold sums until it is written, unless it is one of the inputs, or
  // the codebook's gradient replaces the codebook, which the radius gradient reads.
  auto apart = [](const void* p, size_t np, const void* q, size_t nq) {
    return (const char*)p + np <= (const char*)q || (const char*)q + nq <= (const char*)p;
  };
  const size_t rho_bytes = (size_t)nvec * 4, cb_bytes = (size_t)nval * 4;
  const bool free_rho = apart(d_grad_rho, rho_bytes, d_rho, rho_bytes) && apart(d_grad_rho, rho_bytes, d_r_hat, rho_bytes) &&
                        apart(d_grad_codebook, cb_bytes, d_codebook, cb_bytes);
  const dim3 g_final((unsigned)((nval + 31) / 32));
  // One pass: two blocks per CU on the largest matrices, at least max(128, ncb) vectors per wave (so that a
  // block's sums fit its stretch of the radius gradient), where there is memory for their sums (in place of
  // an input only the workspace: 16 blocks for 64 centres, 12288x4096 1.58 ms against 0.13 by lists) and it is
  // the faster way. Its work per vector grows with the centres, the lists' does not: whole calls, us, encoded
  // directions, before the pass / lists / pass: 64 centres 2^15 vectors 9.5 / 9.2 / 11.9, 2^18 17.0 / 12.0 / 15.1,
  // 2^21 92 / 52 / 42; 128 centres 2^19 27.5 / 18.7 / 43, 2^21 101 / 59 / 98; 256 centres 2^17 10.8 / 11.1 / 30, 2^19
  // 30 / 29 / 35, 2^20 57 / 54 / 65, 2^21 112 / 107 / 102; 16 and 32 centres never behind the former kernels.
  // The lists slow down where most vectors share one centre (2^21 vectors, nine in ten: 0.25 ms for 64 centres,
  // 1.3 ms for 256; the pass 0.04 and 0.10), which is why the lines are not drawn higher.
  const int64_t least = (int64_t)kPassWaves * std::max(128, ncb);
  const int64_t nblk = std::max<int64_t>(1, std::min<int64_t>(512, nvec / least));
  const bool in_ws = nblk <= ws_slices(ncb);
  if (ncb <= 256 && free_rho && (ncb <= 32 || nvec >= (ncb <= 64 ? 3ll << 16 : 1ll << 21))) {
    PassArgs a{nv, nvec, d_rho, d_signs, d_dir_idx, d_codebook, d_r_hat, d_grad_w, ldg, d_grad_rho, in_ws ? (float*)d_ws : nullptr, ncb};
    bool ok = launch_ok(ncb <= 16 ? (const void*)k_fq_grad_pass<16> : ncb <= 64 ? (const void*)k_fq_grad_pass<64> : (const void*)k_fq_grad_pass<256>, dim3((unsigned)nblk),
                        dim3(64 * kPassWaves), s, a) &&
              launch_ok((const void*)k_fq_grad_cb_final, g_final, dim3(1024), s, in_ws ? (const float*)d_ws : (const float*)d_grad_rho,
                        nval, (int)nblk, in_ws ? (int64_t)0 : nvec, d_grad_codebook);
    if (ok && !in_ws)
      ok = launch_ok((const void*)k_fq_grad_rho, dim3((unsigned)(((int64_t)nval * nblk + kThreads - 1) / kThreads)), dim3(kThreads), s,
                     nv, nvec, d_rho, d_signs, d_dir_idx, d_codebook, d_grad_w, ldg, nval, (int)nblk, d_grad_rho);
    return ok ? SPH_OK : SPH_ERR_HIP;
  }
  // By lists, in as many slices as the workspace holds. The slices' sums of 2^13 centres go to the radius
  // gradient's array while it is not yet written, where it holds more of them; each slice then keeps
  // at least 16 vectors per centre on average.
  int group = 1;
  int64_t ns = ws_slices(ncb);
  float* part = (float*)d_ws;
  if (ncb > 256) {
    group = 4;
    const int64_t room = std::min<int64_t>(std::min<int64_t>(slices_for(ncb), nvec / (8 * ncb)), nvec / ncb / 16) / kXcd * kXcd;
    if (room > ns && free_rho && a16(d_grad_rho)) {
      ns = room;
      part = d_grad_rho;
      group = 32;
    }
  }
  // lists up to four times the mean stay with their lanes
  const int most = (int)std::min<int64_t>(1 << 30, std::max<int64_t>(group == 32 ? 256 : 1024, 4 * (nvec / ncb / ns)));
  const int ncblk = (ncb + group - 1) / group;
  const void* fn = group == 1 ? (const void*)k_fq_grad_cb_part<1> : group == 32 ? (const void*)k_fq_grad_cb_part<32> : (const void*)k_fq_grad_cb_part<4>;
  // the lists' sums before the radius gradient (which may be written over r^), that before the
  // codebook's (which may be written over the codebook) unless the sums wait in its array
  auto sums = [&] {
    return launch_ok((const void*)k_fq_grad_cb_final, g_final, dim3(1024), s, (const float*)part, nval, (int)ns, (int64_t)0,
                     d_grad_codebook);
  };
  auto radii = [&] {
    return launch_ok((const void*)k_fq_grad_rho, dim3((unsigned)((nvec + kThreads - 1) / kThreads)), dim3(kThreads), s, nv,
                     nvec, d_rho, d_signs, d_dir_idx, d_codebook, d_grad_w, ldg, 0, 0, d_grad_rho);
  };
  const bool ok =
      launch_ok(fn, dim3((unsigned)(ncblk * ns)), dim3(kThreads), s, nv, d_r_hat, d_signs, d_grad_w, ldg, d_perm, d_offsets, ncb, (int)ns,
                most, part) &&
      (part == d_grad_rho ? sums() && radii() : radii() && sums());
  return ok ? SPH_OK : SPH_ERR_HIP;
}

}  // extern "C"
