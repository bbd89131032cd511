// k-means clustering of the corpus (Sections 3.2, 3.3.2): Lloyd iterations.
//
// Assignment = argmin_j |x - mu_j|^2 decided in FP64 with ties to the smaller
// j.  The distances come from a split bf16 MFMA product (g_j = |mu_j|^2 -
// 2 x.mu_j, the |x|^2 term is common to all j).  When the best and second-best
// values are closer than a rigorous rounding-error bound allows, the point is
// queued for the same product in FP64 (assign_f64_kernel); one that its bound
// cannot decide either (ties, in effect) has all its distances formed
// sequentially in FP64 (sum over dimensions of (x_l - mu_l)^2, no contraction),
// which is the definition itself.
//
// Update = FP64 mean of each cluster's members summed in ascending id order,
// rounded once to fp32; an empty cluster keeps its centroid.

#include <algorithm>

#include "lider_internal.hpp"

namespace lider {

__global__ void zero_i32_kernel2(int32_t* p, int64_t cnt) {
  for (int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; t < cnt;
       t += int64_t(gridDim.x) * blockDim.x)
    p[t] = 0;
}

__global__ void fill_i32_kernel(int32_t* p, int64_t cnt, int32_t v) {
  for (int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; t < cnt;
       t += int64_t(gridDim.x) * blockDim.x)
    p[t] = v;
}

// Centroids per column tile of the assignment product (and rows per tile).
constexpr int kAsgTile = 256;

__host__ __device__ inline int32_t asg_steps(int32_t d) { return (d + 31) / 32; }

__device__ inline void split8(const float (&v)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 h = (__bf16)v[e];
    hi[e] = h;
    lo[e] = (__bf16)(v[e] - float(h));  // the difference is exact
  }
}

// Zeros past dim d of the eight values from dim k on.
__device__ inline void mask8(float (&v)[8], int32_t k, int32_t d) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = k + e < d ? v[e] : 0.f;
}

// The centroids split into h = bf16(mu) and l = bf16(mu - h) in the operand
// order of the assignment product: per 16-centroid block and 32-dim step the
// h part and the l part, 1 KB each, lane i + 16 s holding dims [8 s, 8 s + 8)
// of centroid i (zeros past d and past C).  One wave per centroid; it also
// writes |mu_j|^2 in fp32 (+inf for the centroids past C, which are never
// nearest) and in FP64, and an upper bound of max_j |mu_j| (as float bits,
// atomicMax).
__global__ __launch_bounds__(256) void cent_split_kernel(const float* __restrict__ cent, int32_t C,
                                                         int32_t d, bf16x8* __restrict__ out,
                                                         float* __restrict__ cnorm,
                                                         double* __restrict__ cn64,
                                                         uint32_t* __restrict__ maxbits) {
  const int lane = threadIdx.x & 63;
  const int64_t j = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int32_t nk = asg_steps(d);
  const float* mu = cent + j * d;
  bf16x8* o = out + (j >> 4) * (int64_t(nk) * 128) + (j & 15);
  float s = 0.f;
  double s64 = 0.0;
  for (int32_t u = lane; u < 4 * nk; u += 64) {  // eight dims per lane
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = j < C && 8 * u + e < d ? mu[8 * u + e] : 0.f;
      s += v[e] * v[e];
      s64 += double(v[e]) * double(v[e]);
    }
    bf16x8 h, l;
    split8(v, h, l);
    bf16x8* q = o + (u >> 2) * 128 + 16 * (u & 3);
    q[0] = h;
    q[64] = l;
  }
  for (int x = 32; x > 0; x >>= 1) {
    s += __shfl_xor(s, x);
    s64 += __shfl_xor(s64, x);
  }
  if (lane == 0) {
    cnorm[j] = j < C ? s : INFINITY;
    cn64[j] = j < C ? s64 : double(INFINITY);
    if (j < C) {
      atomicMax(maxbits, __float_as_uint(float(norm_above(s, d))));
    }
  }
}

// Smallest value, its centroid, and the second smallest (equal to the smallest
// on a tie, whichever centroid is kept: a tie is always recomputed).
struct Best {
  float bv;
  int32_t bi;
  float sv;
};

__device__ inline void best_push(Best& b, float g, int32_t j) {
  b.sv = fminf(b.sv, fmaxf(b.bv, g));
  b.bi = g < b.bv ? j : b.bi;
  b.bv = fminf(b.bv, g);
}

__device__ inline Best best_merge(const Best& a, const Best& b) {
  Best r;
  r.sv = fminf(fminf(a.sv, b.sv), fmaxf(a.bv, b.bv));
  r.bi = b.bv < a.bv ? b.bi : a.bi;
  r.bv = fminf(a.bv, b.bv);
  return r;
}

// The other lane's entry of a butterfly over the 16 lanes of a DPP row
// (rotation by N).
template <int N>
__device__ inline Best best_ror(const Best& b) {
  Best p;
  p.bv = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(b.bv), 0x120 + N, 0xf, 0xf, false));
  p.bi = __builtin_amdgcn_update_dpp(0, b.bi, 0x120 + N, 0xf, 0xf, false);
  p.sv = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(b.sv), 0x120 + N, 0xf, 0xf, false));
  return p;
}

// Where a point's assignment goes.
struct AssignOut {
  int32_t d, C;
  const uint32_t* maxbits;
  int32_t* assign;
  const int32_t* prev;
  int32_t* changed;
  int64_t* amb;
  int32_t* amb_count;
};

// Bound of the error of a value g_j of the split product for a point with
// |x| <= xn and centroids with |mu| <= M: x.mu within split_err_coef(d) |x| |mu|
// plus absolute terms for parts below 2^-126; |mu|^2 in fp32 is within
// dot_err_coef(d) |mu|^2, the fp32 combination adds 2^-22, and the FP64 reference
// has its own rounding.  Two values further apart than 2 E are in the exact
// order; assign_decide asks for 4 E.
__device__ inline double assign_err(int32_t d, double xn, double M) {
  return (dot_err_coef(d) + 2.384185791015625e-07) * M * M +
         2.0 * (split_err_coef(d) + 2.384185791015625e-07) * xn * M +
         6.0 * sqrt(double(d)) * 1.1754943508222875e-38 * (xn + M) +
         double(d + 2) * 8.881784197001252e-16 * (xn + M) * (xn + M) +
         6.0 * double(d) * 7.888609052210118e-31;
}

// Decides one point from its best and second-best value and |x|^2 (fp32), or
// queues it.
__device__ inline void assign_decide(const AssignOut& o, int64_t row, const Best& b, float ssr) {
  const double E = assign_err(o.d, norm_above(ssr, o.d), double(__uint_as_float(*o.maxbits)));
  const double gap = double(b.sv) - double(b.bv);
  if (o.C == 1 || gap > 4.0 * E) {
    const int32_t bi = o.C == 1 ? 0 : b.bi;
    o.assign[row] = bi;
    if (o.prev && o.prev[row] != bi) atomicAdd(o.changed, 1);
  } else {
    const int32_t slot = atomicAdd(o.amb_count, 1);
    o.amb[slot] = row;
  }
}

// Assignment product.  A workgroup of 8 waves owns 256 points and sweeps the
// column tiles of 256 centroids of its group (blockIdx.y), 32 dimensions per
// step; wave (wr, wc) owns 64 points x 128 centroids (4 x 8 blocks of
// v_mfma_f32_16x16x32_bf16, three products each).  Points: read in fp32
// straight into the operand layout one step ahead (a wave's points are its
// own, and the 4 lanes of a point cover one 128-byte line of it) and split in
// registers.  Centroids: split beforehand (cent_split_kernel), 32 KB per step
// staged through one of two LDS slots, lane-contiguous on both sides.  64 x
// 128 per wave keeps the LDS reads (16 KB per 96 MFMAs) below the MFMA time,
// and 256 points per workgroup read the centroids from L2 n / 256 times and
// the points C / 256 times; the matrix cores bound it (points served from L2:
// 6% faster).  120,000 x 768 points, 1,000 centroids: 3,374 us by the fp32
// product of 16 points per wave straight from L2, 740 us by this one with its
// loads under conditions, 650 us now (850 TFLOP/s of bf16 products; a plain
// 8192^3 library product reaches 1,145 on the same card).
// The values of a tile are reduced over the wave's columns (registers, then
// DPP rotations over the 16 lanes of a point) and merged into the point's
// best in LDS, so no value is stored.  Decided here without `part`, else part
// receives each group's best (value, centroid, second value, |x|^2).
// MODE 2: rows of whole 32-dimension steps at 16-byte addresses, 1: d a
// multiple of 4 there, 0: any.
template <int MODE>
__global__ __launch_bounds__(512, 2) void assign_kernel(
    const float* __restrict__ X, int64_t n, int32_t d, const bf16x8* __restrict__ cs,
    const float* __restrict__ cnorm, int32_t ntiles, AssignOut o, float4* __restrict__ part) {
  __shared__ bf16x8 sb[2][16 * 128];
  __shared__ float sbv[2][kAsgTile], ssv[2][kAsgTile], sss[kAsgTile];
  __shared__ int32_t sbi[2][kAsgTile];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, s = lane >> 4;
  const int wr = wave >> 1, wc = wave & 1;
  const int64_t row0 = int64_t(blockIdx.x) * kAsgTile;
  const int32_t G = int32_t(gridDim.y), g = int32_t(blockIdx.y);
  const int32_t t0 = int32_t(int64_t(ntiles) * g / G), t1 = int32_t(int64_t(ntiles) * (g + 1) / G);
  const int32_t nk = asg_steps(d);
  // offsets within the tile (at most 256 x 65,536 values) from a uniform base
  const float* xt = X + row0 * d;
  const int32_t rlast = int32_t(min(n - row0, int64_t(kAsgTile))) - 1;
  int32_t xo[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) xo[a] = min(64 * wr + 16 * a + i, rlast) * d + 8 * s;
  float4 xa[4][2];
  bf16x8 st[4];
  auto load_points = [&](int32_t kc) {
    const float* xk = xt + 32 * kc;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int32_t at = xo[a] + 4 * h, kd = 32 * kc + 8 * s + 4 * h;
        // inside the point; values past it become zeros where they are used (at
        // the load that would wait for the load)
        if (MODE == 2) {  // d % 32 == 0
          xa[a][h] = *reinterpret_cast<const float4*>(xk + at);
        } else if (MODE == 1) {  // d % 4 == 0: a whole float4 lies inside the point or past it
          xa[a][h] = *reinterpret_cast<const float4*>(xk + at - max(kd - (d - 4), 0));
        } else {
          const float* p = xk + at;
          xa[a][h].x = p[-max(kd - (d - 1), 0)];
          xa[a][h].y = p[1 - max(kd + 1 - (d - 1), 0)];
          xa[a][h].z = p[2 - max(kd + 2 - (d - 1), 0)];
          xa[a][h].w = p[3 - max(kd + 3 - (d - 1), 0)];
        }
      }
  };
  auto load_cents = [&](int32_t t, int32_t kc) {
    const bf16x8* ck = cs + (int64_t(t) * 16 * nk + kc) * 128;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int32_t p = tid + 512 * j;
      st[j] = ck[(p >> 7) * (nk * 128) + (p & 127)];
    }
  };
  auto store_cents = [&](int slot) {
#pragma unroll
    for (int j = 0; j < 4; ++j) sb[slot][tid + 512 * j] = st[j];
  };
  floatx4 acc[4][8];
  float ss[4] = {0.f, 0.f, 0.f, 0.f};
  load_cents(t0, 0);
  load_points(0);
  store_cents(0);
  __syncthreads();
  int slot = 0;
  for (int32_t t = t0; t < t1; ++t) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 8; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int32_t kc = 0; kc < nk; ++kc) {
      bf16x8 ah[4], al[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        float v[8] = {xa[a][0].x, xa[a][0].y, xa[a][0].z, xa[a][0].w,
                      xa[a][1].x, xa[a][1].y, xa[a][1].z, xa[a][1].w};
        if (MODE != 2) mask8(v, 32 * kc + 8 * s, d);
        split8(v, ah[a], al[a]);
        if (t == t0) {
#pragma unroll
          for (int e = 0; e < 8; ++e) ss[a] += v[e] * v[e];
        }
      }
      const bool last = kc + 1 == nk;
      // the next step's operands, in flight during this one (after the last
      // step some again: a load under a condition would make the compiler wait
      // for all loads at the next use)
      load_cents(last ? min(t + 1, t1 - 1) : t, last ? 0 : kc + 1);
      load_points(last ? 0 : kc + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const bf16x8 bh = sb[slot][(8 * wc + b) * 128 + lane];
        const bf16x8 bl = sb[slot][(8 * wc + b) * 128 + 64 + lane];
#pragma unroll
        for (int a = 0; a < 4; ++a)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[a], bh, acc[a][b], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[a], bl, acc[a][b], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[a], bh, acc[a][b], 0, 0, 0);
      }
      store_cents(slot ^ 1);
      __syncthreads();
      slot ^= 1;
    }
    // D layout: acc[a][b][e] = point 64 wr + 16 a + 4 s + e, centroid
    // 128 wc + 16 b + i of the tile
    const int32_t c0 = t * kAsgTile + 128 * wc + i;
    float cn[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) cn[b] = cnorm[c0 + 16 * b];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        Best v{INFINITY, 0x7fffffff, INFINITY};
#pragma unroll
        for (int b = 0; b < 8; ++b) best_push(v, cn[b] - 2.f * acc[a][b][e], c0 + 16 * b);
        v = best_merge(v, best_ror<8>(v));
        v = best_merge(v, best_ror<4>(v));
        v = best_merge(v, best_ror<2>(v));
        v = best_merge(v, best_ror<1>(v));
        const int r = 64 * wr + 16 * a + 4 * s + e;
        if (i == 0) {  // this wave's own entries
          if (t > t0) v = best_merge(Best{sbv[wc][r], sbi[wc][r], ssv[wc][r]}, v);
          sbv[wc][r] = v.bv;
          sbi[wc][r] = v.bi;
          ssv[wc][r] = v.sv;
        }
      }
  }
  if (wc == 0) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      float q = ss[a];  // over the four dimension slots
      q += __shfl_xor(q, 16);
      q += __shfl_xor(q, 32);
      if (s == 0) sss[64 * wr + 16 * a + i] = q;
    }
  }
  __syncthreads();
  if (tid < kAsgTile && row0 + tid < n) {
    const Best v = best_merge(Best{sbv[0][tid], sbi[0][tid], ssv[0][tid]},
                              Best{sbv[1][tid], sbi[1][tid], ssv[1][tid]});
    if (!part)
      assign_decide(o, row0 + tid, v, sss[tid]);
    else
      part[int64_t(g) * n + row0 + tid] = float4{v.bv, __int_as_float(v.bi), v.sv, sss[tid]};
  }
}

// The product for few centroids (C <= 16 NB <= 128): the wide tile would
// multiply mostly padding, and the points' rows, read once, bound the time.  A
// workgroup of 4 waves owns 64 RB points, a wave 16 RB of them and every
// column; its rows are in flight four steps ahead (a ring of register sets),
// the step's centroids go through two LDS slots, staged two steps ahead, and
// no load stands under a condition.  A call with 66,872 x 768 points and 18
// centroids: 133 us by the fp32 product of 16 points per wave, 171 by the wide
// tile, 75 now; 97,695 points and 60 centroids 206 -> 91, 128 374 -> 113.
template <int MODE, int NB, int RB>
__global__ __launch_bounds__(256) void assign_narrow_kernel(
    const float* __restrict__ X, int64_t n, int32_t d, const bf16x8* __restrict__ cs,
    const float* __restrict__ cnorm, AssignOut o, float4* __restrict__ part) {
  constexpr int ROWS = 64 * RB, P = 4, NS = (NB * 128 + 255) / 256;
  __shared__ bf16x8 sb[2][NB * 128];
  __shared__ float sbv[ROWS], ssv[ROWS], sss[ROWS];
  __shared__ int32_t sbi[ROWS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, s = lane >> 4;
  const int64_t row0 = int64_t(blockIdx.x) * ROWS;
  const int32_t nk = asg_steps(d);
  const float* xt = X + row0 * d;
  const int32_t rlast = int32_t(min(n - row0, int64_t(ROWS))) - 1;
  int32_t xo[RB];
#pragma unroll
  for (int a = 0; a < RB; ++a) xo[a] = min(16 * (RB * wave + a) + i, rlast) * d + 8 * s;
  float4 xa[P][RB][2];
  bf16x8 st[2][NS];
  auto load_points = [&](int32_t kc, float4 (&x)[RB][2]) {
    kc = min(kc, nk - 1);
    const float* xk = xt + 32 * kc;
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int32_t at = xo[a] + 4 * h, kd = 32 * kc + 8 * s + 4 * h;
        if (MODE == 2) {
          x[a][h] = *reinterpret_cast<const float4*>(xk + at);
        } else if (MODE == 1) {
          x[a][h] = *reinterpret_cast<const float4*>(xk + at - max(kd - (d - 4), 0));
        } else {
          const float* p = xk + at;
          x[a][h].x = p[-max(kd - (d - 1), 0)];
          x[a][h].y = p[1 - max(kd + 1 - (d - 1), 0)];
          x[a][h].z = p[2 - max(kd + 2 - (d - 1), 0)];
          x[a][h].w = p[3 - max(kd + 3 - (d - 1), 0)];
        }
      }
  };
  auto load_cents = [&](int32_t kc, bf16x8 (&v)[NS]) {
    const bf16x8* ck = cs + int64_t(min(kc, nk - 1)) * 128;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int32_t p = (tid + 256 * j) & (NB * 128 - 1);  // the same piece twice where threads are left
      v[j] = ck[(p >> 7) * (nk * 128) + (p & 127)];
    }
  };
  auto store_cents = [&](int slot, const bf16x8 (&v)[NS]) {
#pragma unroll
    for (int j = 0; j < NS; ++j) sb[slot][(tid + 256 * j) & (NB * 128 - 1)] = v[j];
  };
  floatx4 acc[RB][NB];
#pragma unroll
  for (int a = 0; a < RB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  float ss[RB] = {};
  load_cents(0, st[0]);
  load_cents(1, st[1]);
#pragma unroll
  for (int u = 0; u < P; ++u) load_points(u, xa[u]);
  store_cents(0, st[0]);
  __syncthreads();
  auto step = [&](int u, int32_t kc) {
    bf16x8 ah[RB], al[RB];
#pragma unroll
    for (int a = 0; a < RB; ++a) {
      float v[8] = {xa[u][a][0].x, xa[u][a][0].y, xa[u][a][0].z, xa[u][a][0].w,
                    xa[u][a][1].x, xa[u][a][1].y, xa[u][a][1].z, xa[u][a][1].w};
      if (MODE != 2) mask8(v, 32 * kc + 8 * s, d);
      split8(v, ah[a], al[a]);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss[a] += v[e] * v[e];
    }
    load_cents(kc + 2, st[u & 1]);
    load_points(kc + P, xa[u]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bf16x8 bh = sb[u & 1][b * 128 + lane], bl = sb[u & 1][b * 128 + 64 + lane];
#pragma unroll
      for (int a = 0; a < RB; ++a)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[a], bh, acc[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < RB; ++a)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[a], bl, acc[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < RB; ++a)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[a], bh, acc[a][b], 0, 0, 0);
    }
    store_cents((u + 1) & 1, st[(u + 1) & 1]);
    __syncthreads();
  };
  int32_t kc = 0;
  for (; kc + P <= nk; kc += P) {
#pragma unroll
    for (int u = 0; u < P; ++u) step(u, kc + u);
  }
#pragma unroll
  for (int u = 0; u + 1 < P; ++u)
    if (kc + u < nk) step(u, kc + u);
  float cn[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) cn[b] = cnorm[16 * b + i];
#pragma unroll
  for (int a = 0; a < RB; ++a) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      Best v{INFINITY, 0x7fffffff, INFINITY};
#pragma unroll
      for (int b = 0; b < NB; ++b) best_push(v, cn[b] - 2.f * acc[a][b][e], 16 * b + i);
      v = best_merge(v, best_ror<8>(v));
      v = best_merge(v, best_ror<4>(v));
      v = best_merge(v, best_ror<2>(v));
      v = best_merge(v, best_ror<1>(v));
      if (i == 0) {
        const int r = 16 * (RB * wave + a) + 4 * s + e;
        sbv[r] = v.bv;
        sbi[r] = v.bi;
        ssv[r] = v.sv;
      }
    }
    float q = ss[a];  // over the four dimension slots
    q += __shfl_xor(q, 16);
    q += __shfl_xor(q, 32);
    if (s == 0) sss[16 * (RB * wave + a) + i] = q;
  }
  __syncthreads();
  if (tid < ROWS && row0 + tid < n) {
    const Best v{sbv[tid], sbi[tid], ssv[tid]};
    if (!part)
      assign_decide(o, row0 + tid, v, sss[tid]);
    else
      part[row0 + tid] = float4{v.bv, __int_as_float(v.bi), v.sv, sss[tid]};
  }
}

// Most centroids of the narrow product.
constexpr int32_t kAsgNarrow = 128;

template <int MODE>
static void launch_narrow(const float* X, int64_t n, int32_t d, const bf16x8* cs, const float* cnorm,
                          const AssignOut& o, float4* part, hipStream_t st) {
  // 64 points per workgroup while 128 would leave CUs without one
  const bool few = n < 128 * 256;
  const dim3 grid(unsigned((n + (few ? 63 : 127)) / (few ? 64 : 128)));
#define LIDER_NARROW(NB)                                                                             \
  if (few)                                                                                           \
    hipLaunchKernelGGL((assign_narrow_kernel<MODE, NB, 1>), grid, dim3(256), 0, st, X, n, d, cs,     \
                       cnorm, o, part);                                                              \
  else                                                                                               \
    hipLaunchKernelGGL((assign_narrow_kernel<MODE, NB, 2>), grid, dim3(256), 0, st, X, n, d, cs,     \
                       cnorm, o, part);
  if (o.C <= 16) {
    LIDER_NARROW(1)
  } else if (o.C <= 32) {
    LIDER_NARROW(2)
  } else if (o.C <= 64) {
    LIDER_NARROW(4)
  } else {
    LIDER_NARROW(8)
  }
#undef LIDER_NARROW
}

// The groups' bests of each point merged and decided.
__global__ __launch_bounds__(256) void assign_merge_kernel(const float4* __restrict__ part,
                                                           int64_t n, int32_t G, AssignOut o) {
  const int64_t row = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (row >= n) return;
  Best v{INFINITY, 0x7fffffff, INFINITY};
  float ss = 0.f;
  for (int32_t g = 0; g < G; ++g) {
    const float4 p = part[int64_t(g) * n + row];
    v = best_merge(v, Best{p.x, __float_as_int(p.y), p.z});
    ss = p.w;
  }
  assign_decide(o, row, v, ss);
}

// Second decision of the queued points: the values g_j by FP64 MFMA
// (v_mfma_f64_16x16x4f64), whose bound is some 2^-28 of the split product's, so
// that only ties remain.  How many points the first bound leaves is the data's
// choice (120,000 x 768, 1,000 centroids: none of a mixture of separated blobs,
// tens of thousands of unit rows with a common mean); the sequential FP64 sums of all C
// distances would then cost many times the product itself, while this one is
// bounded by 2 C d FP64 operations a point at the MFMA rate (120,000 x 768,
// 1,000 centroids, whole call: isotropic rows 17.3 ms with the sequential sums
// alone, 1.14 ms now; unit rows with a common mean 51.7 and 1.82; d = 64: 0.29
// and 0.18, 0.48 and 0.19).
// A workgroup of 16 waves takes 32 points (16 while the queue fits the chip that
// way, for the shorter chain) and sweeps 512 centroids at a time, 32 per wave;
// operands straight from L2, one step of 16 dimensions ahead: 32 MFMAs of 64
// cycles hide them.  Lane (i, s) feeds dims [4 s, 4 s + 4) of a step to four
// MFMAs, as in the hash kernel.
// |g - (|mu|^2 - 2 x.mu)| <= (d + 2) 2^-53 (|x| + M)^2 (the fp32 x fp32 products
// are exact) and the definition's own sum is within (d + 3) 2^-53 (|x| + M)^2,
// so values further apart than 4 (d + 3) 2^-53 (|x| + M)^2 are in the
// definition's order; 16 (d + 8) is used.  The other term covers fp32 subnormals
// flushed on the way into FP64.  For the points that it leaves open (ties, as a
// rule of equal centroids) a second look lists the centroids within it, and those
// distances are summed sequentially; past the list's room, all of them.  All
// points tied (20,000 x 768, 1,000 centroids in 500 equal pairs): 30 ms by a
// workgroup per point over all distances, 1.8 now.
constexpr int kF64Waves = 16, kF64Grid = 512;

struct Best64 {
  double bv, sv;
  int32_t bi;
};

__device__ inline Best64 best_merge(const Best64& a, const Best64& b) {
  Best64 r;
  r.sv = fmin(fmin(a.sv, b.sv), fmax(a.bv, b.bv));
  r.bi = b.bv < a.bv ? b.bi : a.bi;
  r.bv = fmin(a.bv, b.bv);
  return r;
}

// The definition of one distance: a sequential sum without contraction.
template <bool VEC>
__device__ inline double distance_sequential(const float* __restrict__ x, const float* __restrict__ mu,
                                             int32_t d) {
#pragma clang fp contract(off)
  double acc = 0.0;
  if (VEC) {
#pragma unroll 4
    for (int32_t l = 0; l < d; l += 4) {
      const float4 a = *reinterpret_cast<const float4*>(x + l);
      const float4 b = *reinterpret_cast<const float4*>(mu + l);
      const double d0 = double(a.x) - double(b.x), d1 = double(a.y) - double(b.y);
      const double d2 = double(a.z) - double(b.z), d3 = double(a.w) - double(b.w);
      acc = acc + d0 * d0;
      acc = acc + d1 * d1;
      acc = acc + d2 * d2;
      acc = acc + d3 * d3;
    }
  } else {
#pragma unroll 4
    for (int32_t l = 0; l < d; ++l) {
      const double df = double(x[l]) - double(mu[l]);
      acc = acc + df * df;
    }
  }
  return acc;
}

__device__ inline void assign_write(const AssignOut& o, int64_t row, int32_t j) {
  o.assign[row] = j;
  if (o.prev && o.prev[row] != j) atomicAdd(o.changed, 1);
}

// The definition for the points open[0, no) over all centroids: a group of
// threads per point (as many points at a time as the workgroup holds such
// groups), ties to the smaller id.  The rows are each thread's own, so their
// loads bound it: 16 bytes at a time where they are aligned.
template <bool VEC, int NT>
__device__ void assign_sequential(const float* __restrict__ X, const int64_t* open, int32_t no,
                                  const float* __restrict__ cent, const AssignOut& o, double* sd,
                                  int32_t* sj) {
  const int tid = threadIdx.x;
  const int32_t d = o.d, C = o.C;
  int32_t tg = 32;  // threads per point
  while (tg < C && tg < NT) tg <<= 1;
  const int32_t me = tid / tg, lane = tid - me * tg;
  for (int32_t t0 = 0; t0 < no; t0 += NT / tg) {
    const bool in = t0 + me < no;
    double bd = INFINITY;
    int32_t bj = 0x7fffffff;
    if (in) {
      const float* x = X + open[t0 + me] * d;
      for (int32_t j = lane; j < C; j += tg) {
        const double v = distance_sequential<VEC>(x, cent + int64_t(j) * d, d);
        if (v < bd) {
          bd = v;
          bj = j;
        }
      }
    }
    sd[tid] = bd;
    sj[tid] = bj;
    __syncthreads();
#pragma unroll 1
    for (int32_t h = tg / 2; h > 0; h >>= 1) {
      if (lane < h) {
        const double od = sd[tid + h];
        const int32_t oj = sj[tid + h];
        if (od < sd[tid] || (od == sd[tid] && oj < sj[tid])) {
          sd[tid] = od;
          sj[tid] = oj;
        }
      }
      __syncthreads();
    }
    if (in && lane == 0) assign_write(o, open[t0 + me], sj[tid]);
    __syncthreads();
  }
}

template <bool VEC>
__global__ __launch_bounds__(64 * kF64Waves) void assign_f64_kernel(
    const float* __restrict__ X, const float* __restrict__ cent, const double* __restrict__ cn64,
    AssignOut o) {
  typedef double doublex4 __attribute__((ext_vector_type(4)));
  constexpr int NT = 64 * kF64Waves;
  __shared__ double sbv[kF64Waves][32], ssv[kF64Waves][32], sss[32];
  __shared__ int32_t sbi[kF64Waves][32];
  __shared__ double sd[NT];
  __shared__ int32_t sj[NT];
  // points that the bound leaves open, the largest value that can win (per point
  // of the workgroup) and the (point, centroid) pairs at or below it
  __shared__ int64_t open[32];
  __shared__ double sthr[32];
  __shared__ uint64_t smin[32];
  __shared__ int32_t smj[32];
  __shared__ int32_t cand_r[NT], cand_j[NT];
  __shared__ int32_t nopen, ncand;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, s = lane >> 4;
  const int32_t cnt = *o.amb_count, d = o.d, C = o.C;
  const bool two = cnt > 16 * kF64Grid;
  const int32_t per = two ? 32 : 16;
  const double M = double(__uint_as_float(*o.maxbits));
  // four values of a row of d from dim kk on, zeros past it, every load inside it
  auto load4 = [&](const float* row, int32_t kk) {
    float4 v;
    if (VEC) {  // d a multiple of 4: a float4 lies inside the row or past it
      v = *reinterpret_cast<const float4*>(row + min(kk, d - 4));
      if (kk >= d) v = float4{0.f, 0.f, 0.f, 0.f};
    } else {
      const float w[4] = {row[min(kk, d - 1)], row[min(kk + 1, d - 1)], row[min(kk + 2, d - 1)],
                          row[min(kk + 3, d - 1)]};
      v.x = kk < d ? w[0] : 0.f;
      v.y = kk + 1 < d ? w[1] : 0.f;
      v.z = kk + 2 < d ? w[2] : 0.f;
      v.w = kk + 3 < d ? w[3] : 0.f;
    }
    return v;
  };
  for (int64_t t0 = int64_t(blockIdx.x) * per; t0 < cnt; t0 += int64_t(kF64Grid) * per) {
    const float* xr[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
      xr[a] = X + o.amb[min(t0 + (two ? 16 * a : 0) + i, int64_t(cnt) - 1)] * d;
    // the products with this wave's columns, 32 at a time: done(c0, acc), element
    // acc[a][b][e] of lane (i, s) for point 16 a + s + 4 e, centroid c0 + 16 b + i
    auto sweep = [&](auto done) {
      for (int32_t c0 = 32 * wave; c0 < C; c0 += 32 * kF64Waves) {
        const float* cr[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) cr[b] = cent + int64_t(min(c0 + 16 * b + i, C - 1)) * d;
        doublex4 acc[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b) acc[a][b] = doublex4{0.0, 0.0, 0.0, 0.0};
        float4 nx[2], nc[2];
        auto fetch = [&](int32_t k0) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            nx[u] = load4(xr[u], k0 + 4 * s);
            nc[u] = load4(cr[u], k0 + 4 * s);
          }
        };
        if (VEC) fetch(0);
        for (int32_t k0 = 0; k0 < d; k0 += 16) {
          if (!VEC) fetch(k0);  // scalar loads a step ahead would spill
          const float x[2][4] = {{nx[0].x, nx[0].y, nx[0].z, nx[0].w}, {nx[1].x, nx[1].y, nx[1].z, nx[1].w}};
          const float y[2][4] = {{nc[0].x, nc[0].y, nc[0].z, nc[0].w}, {nc[1].x, nc[1].y, nc[1].z, nc[1].w}};
          if (VEC) fetch(k0 + 16);  // past the row: zeros
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const double x0 = double(x[0][e]), x1 = double(x[1][e]);
            const double y0 = double(y[0][e]), y1 = double(y[1][e]);
            acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y0, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y1, acc[0][1], 0, 0, 0);
            if (two) {
              acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y0, acc[1][0], 0, 0, 0);
              acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y1, acc[1][1], 0, 0, 0);
            }
          }
        }
        done(c0, acc, c0 + i < C ? cn64[c0 + i] : double(INFINITY),
             c0 + 16 + i < C ? cn64[c0 + 16 + i] : double(INFINITY));
      }
    };
    bool any = false;  // this wave has columns (wave-uniform)
    sweep([&](int32_t c0, const doublex4 (&acc)[2][2], double n0, double n1) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double inf = double(INFINITY);
          Best64 v = best_merge(Best64{n0 - 2.0 * acc[a][0][e], inf, c0 + i},
                                Best64{n1 - 2.0 * acc[a][1][e], inf, c0 + 16 + i});
#pragma unroll
          for (int x = 1; x < 16; x <<= 1)
            v = best_merge(v, Best64{__shfl_xor(v.bv, x), __shfl_xor(v.sv, x), __shfl_xor(v.bi, x)});
          const int r = 16 * a + s + 4 * e;
          if (i == 0) {  // this wave's own entries
            if (any) v = best_merge(Best64{sbv[wave][r], ssv[wave][r], sbi[wave][r]}, v);
            sbv[wave][r] = v.bv;
            ssv[wave][r] = v.sv;
            sbi[wave][r] = v.bi;
          }
        }
      any = true;
    });
    if (tid == 0) nopen = ncand = 0;
    {  // |x|^2: half a wave per point
      const int r = tid >> 5;
      const float* x = X + o.amb[min(t0 + r, int64_t(cnt) - 1)] * d;
      double q = 0.0;
#pragma unroll 4
      for (int32_t l = tid & 31; l < d; l += 32) q += double(x[l]) * double(x[l]);
      for (int h = 16; h > 0; h >>= 1) q += __shfl_xor(q, h);
      if ((tid & 31) == 0) sss[r] = q;
    }
    __syncthreads();
    if (tid < 32) {
      sthr[tid] = -INFINITY;
      smin[tid] = ~uint64_t(0);
      smj[tid] = -1;  // not open
    }
    if (tid < per && t0 + tid < cnt) {
      Best64 v{sbv[0][tid], ssv[0][tid], sbi[0][tid]};
      for (int w = 1; w < kF64Waves && 32 * w < C; ++w)
        v = best_merge(v, Best64{sbv[w][tid], ssv[w][tid], sbi[w][tid]});
      const int64_t row = o.amb[t0 + tid];
      const double r = sqrt(sss[tid]) * (1.0 + 9.5367431640625e-07) + M;
      const double E = 16.0 * double(d + 8) * 1.1102230246251565e-16 * r * r +
                       8.0 * sqrt(double(d)) * 1.1754943508222875e-38 * r;
      if (v.sv - v.bv > E) {  // false with a NaN or an infinite bound
        assign_write(o, row, v.bi);
      } else {
        sthr[tid] = v.bv + E;
        smj[tid] = 0x7fffffff;
        open[atomicAdd(&nopen, 1)] = row;
      }
    }
    __syncthreads();
    if (nopen > 0) {  // workgroup-uniform
      // the open points' centroids within the bound of the best, by a second look
      // (a value that is no number counts)
      sweep([&](int32_t c0, const doublex4 (&acc)[2][2], double n0, double n1) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = 16 * a + s + 4 * e;
            const double thr = sthr[r];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
              const int32_t j = c0 + 16 * b + i;
              if (j < C && !((b ? n1 : n0) - 2.0 * acc[a][b][e] > thr)) {
                const int32_t at = atomicAdd(&ncand, 1);
                if (at < NT) {
                  cand_r[at] = r;
                  cand_j[at] = j;
                }
              }
            }
          }
      });
      __syncthreads();
      const int32_t nc = ncand;
      if (nc <= NT) {  // a distance per thread, neighbours in the list on different waves
        const int32_t at = (tid & 63) * kF64Waves + wave;
        double v = 0.0;
        int32_t r = 0;
        if (at < nc) {
          r = cand_r[at];
          v = distance_sequential<VEC>(X + o.amb[t0 + r] * d, cent + int64_t(cand_j[at]) * d, d);
          // the smallest sum, then the smallest id among its equals (a NaN wins nothing)
          if (v < double(INFINITY))
            atomicMin(reinterpret_cast<unsigned long long*>(&smin[r]), (unsigned long long)__double_as_longlong(v));
        }
        __syncthreads();
        if (at < nc && uint64_t(__double_as_longlong(v)) == smin[r]) atomicMin(&smj[r], cand_j[at]);
        __syncthreads();
        if (tid < 32 && smj[tid] >= 0) assign_write(o, o.amb[t0 + tid], smj[tid]);
      } else {
        assign_sequential<VEC, NT>(X, open, nopen, cent, o, sd, sj);
      }
    }
    __syncthreads();
  }
}

// Groups of column tiles of the assignment: one while the point tiles alone
// fill the chip's 256 CUs (a workgroup per CU: 64 KB of LDS, two waves per
// SIMD), else as many as fill it (each group reads the points again, and the
// merge reads 16 B per point and group).
static int32_t asg_groups(int64_t n, int32_t C) {
  const int64_t pt = (n + kAsgTile - 1) / kAsgTile, ct = (int64_t(C) + kAsgTile - 1) / kAsgTile;
  return int32_t(std::min(ct, std::max<int64_t>(1, 256 / pt)));
}

// scratch: cnorm [256 tiles] f32 | cn64 [256 tiles] f64 | maxbits u32 |
// amb_count i32 | amb [n] i64 | split centroids [256 tiles x 32 steps] 2 bf16 |
// groups' bests [G x n] float4
static size_t asg_split_bytes(int32_t C, int32_t d) {
  return size_t((int64_t(C) + kAsgTile - 1) / kAsgTile) * kAsgTile * size_t(asg_steps(d)) * 32 * 4;
}

size_t kmeans_assign_scratch(int64_t n, int32_t d, int32_t C) {
  const int32_t G = asg_groups(n, C);
  return al256((size_t(C) + kAsgTile) * 4) + al256((size_t(C) + kAsgTile) * 8) + 256 +
         al256(size_t(n) * 8) + asg_split_bytes(C, d) + (G > 1 ? size_t(G) * n * sizeof(float4) : 0);
}

struct AsgScratch {
  float* cnorm;
  double* cn64;
  uint32_t* maxbits;
  int32_t* amb_count;
  int64_t* amb;
  bf16x8* cs;
  float4* part;
};

static AsgScratch asg_scratch(void* scratch, int64_t n, int32_t d, int32_t C) {
  AsgScratch a;
  char* p = static_cast<char*>(scratch);
  a.cnorm = reinterpret_cast<float*>(p);
  p += al256((size_t(C) + kAsgTile) * 4);
  a.cn64 = reinterpret_cast<double*>(p);
  p += al256((size_t(C) + kAsgTile) * 8);
  a.maxbits = reinterpret_cast<uint32_t*>(p);
  a.amb_count = reinterpret_cast<int32_t*>(p + 4);
  p += 256;
  a.amb = reinterpret_cast<int64_t*>(p);
  p += al256(size_t(n) * 8);
  a.cs = reinterpret_cast<bf16x8*>(p);
  p += asg_split_bytes(C, d);
  a.part = reinterpret_cast<float4*>(p);
  return a;
}

// The centroids split, then the product: decided through o, or (part) every
// group's best per point.
static void launch_product(const float* X, int64_t n, int32_t d, const float* cent, int32_t C,
                           const AsgScratch& a, int32_t G, const AssignOut& o, float4* part,
                           hipStream_t st) {
  const int32_t ntiles = int32_t((int64_t(C) + kAsgTile - 1) / kAsgTile);
  hipLaunchKernelGGL(zero_i32_kernel2, dim3(1), dim3(64), 0, st,
                     reinterpret_cast<int32_t*>(a.maxbits), int64_t(2));
  hipLaunchKernelGGL(cent_split_kernel, dim3(unsigned(ntiles) * (kAsgTile / 4)), dim3(256), 0, st,
                     cent, C, d, a.cs, a.cnorm, a.cn64, a.maxbits);
  const bool al = (reinterpret_cast<uintptr_t>(X) & 15) == 0;
  const dim3 grid(unsigned((n + kAsgTile - 1) / kAsgTile), unsigned(G));
  if (C <= kAsgNarrow) {
    if (al && d % 32 == 0)
      launch_narrow<2>(X, n, d, a.cs, a.cnorm, o, part, st);
    else if (al && d % 4 == 0)
      launch_narrow<1>(X, n, d, a.cs, a.cnorm, o, part, st);
    else
      launch_narrow<0>(X, n, d, a.cs, a.cnorm, o, part, st);
  } else if (al && d % 32 == 0)
    hipLaunchKernelGGL(assign_kernel<2>, grid, dim3(512), 0, st, X, n, d, a.cs, a.cnorm, ntiles, o, part);
  else if (al && d % 4 == 0)
    hipLaunchKernelGGL(assign_kernel<1>, grid, dim3(512), 0, st, X, n, d, a.cs, a.cnorm, ntiles, o, part);
  else
    hipLaunchKernelGGL(assign_kernel<0>, grid, dim3(512), 0, st, X, n, d, a.cs, a.cnorm, ntiles, o, part);
}

// The product alone: the groups' bests in part ([G x n]); returns G, and in
// maxbits where the largest |mu| is.
static int32_t launch_assign_product(const float* X, int64_t n, int32_t d, const float* cent,
                                     int32_t C, void* scratch, float4* part,
                                     const uint32_t** maxbits, hipStream_t st) {
  const AsgScratch a = asg_scratch(scratch, n, d, C);
  const int32_t G = asg_groups(n, C);
  launch_product(X, n, d, cent, C, a, G, AssignOut{d, C, a.maxbits, nullptr, nullptr, nullptr, nullptr, nullptr},
                 part, st);
  *maxbits = a.maxbits;
  return G;
}

int run_kmeans_assign(const float* X, int64_t n, int32_t d, const float* cent, int32_t C,
                      int32_t* assign, const int32_t* prev, int32_t* changed, void* scratch,
                      hipStream_t st) {
  const AsgScratch a = asg_scratch(scratch, n, d, C);
  const int32_t G = asg_groups(n, C);
  const AssignOut o{d, C, a.maxbits, assign, prev, changed, a.amb, a.amb_count};
  launch_product(X, n, d, cent, C, a, G, o, G > 1 ? a.part : nullptr, st);
  if (G > 1)
    hipLaunchKernelGGL(assign_merge_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st,
                       a.part, n, G, o);
  const bool vec = d % 4 == 0 && ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(cent)) & 15) == 0;
  if (vec)
    hipLaunchKernelGGL(assign_f64_kernel<true>, dim3(kF64Grid), dim3(64 * kF64Waves), 0, st, X, cent,
                       a.cn64, o);
  else
    hipLaunchKernelGGL(assign_f64_kernel<false>, dim3(kF64Grid), dim3(64 * kF64Waves), 0, st, X, cent,
                       a.cn64, o);
  return check_hip(hipGetLastError(), "k-means assignment kernels");
}

// ------------------------------------------------------------------ update
__global__ void iota_kernel(int32_t* p, int64_t n) {
  for (int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; t < n;
       t += int64_t(gridDim.x) * blockDim.x)
    p[t] = int32_t(t);
}

// off[j] = first position whose sorted key >= j  (j = 0..C)
__global__ void lower_bound_kernel(const uint32_t* __restrict__ sorted, int64_t n, int32_t C,
                                   int64_t* __restrict__ off) {
  const int32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j > C) return;
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    int64_t mid = (lo + hi) >> 1;
    if (sorted[mid] < uint32_t(j))
      lo = mid + 1;
    else
      hi = mid;
  }
  off[j] = lo;
}

// One thread per (cluster, dim): sequential FP64 sum over members (ascending
// id), mean rounded once to fp32.  The sums are a chain, the reads are not:
// sixteen members' loads are in flight at a time (200,000 x 768 in 200
// clusters: 835 us with one at a time, 124 us).
__global__ void mean_kernel(const float* __restrict__ X, int32_t d,
                            const int32_t* __restrict__ members, const int64_t* __restrict__ off,
                            int32_t C, float* __restrict__ cent) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= int64_t(C) * d) return;
  const int32_t j = int32_t(t / d);
  const int32_t l = int32_t(t - int64_t(j) * d);
  const int64_t a = off[j], e = off[j + 1];
  if (e == a) return;
  double s = 0.0;
  int64_t p = a;
  for (; p + 16 <= e; p += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = X[int64_t(members[p + u]) * d + l];
#pragma unroll
    for (int u = 0; u < 16; ++u) s = s + double(v[u]);
  }
  for (; p < e; ++p) s = s + double(X[int64_t(members[p]) * d + l]);
  cent[t] = float(s / double(e - a));
}

static int sort_bits(int32_t C) {
  int b = 1;
  while ((int64_t(1) << b) < int64_t(C) + 1) ++b;
  return b;
}

// scratch: keys_out [n] u32 | iota [n] i32 | members [n] i32 | off [C+1] i64 | sort temp
size_t centroid_means_scratch(int64_t n, int32_t C) {
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  return al(size_t(n) * 4) * 3 + al((size_t(C) + 1) * 8) + al(radix_sort_temp_bytes(n, 4));
}

int run_centroid_means(const float* X, int64_t n, int32_t d, const int32_t* assign, int32_t C,
                       float* cent, void* scratch, size_t scratch_bytes, hipStream_t st) {
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  char* p = static_cast<char*>(scratch);
  uint32_t* kout = reinterpret_cast<uint32_t*>(p);
  p += al(size_t(n) * 4);
  int32_t* io = reinterpret_cast<int32_t*>(p);
  p += al(size_t(n) * 4);
  int32_t* members = reinterpret_cast<int32_t*>(p);
  p += al(size_t(n) * 4);
  int64_t* off = reinterpret_cast<int64_t*>(p);
  p += al((size_t(C) + 1) * 8);
  size_t tmp = scratch_bytes - size_t(p - static_cast<char*>(scratch));
  hipLaunchKernelGGL(iota_kernel, dim3(1024), dim3(256), 0, st, io, n);
  const int rc = radix_sort_pairs<uint32_t>(reinterpret_cast<const uint32_t*>(assign), io, kout,
                                            members, n, sort_bits(C), p, tmp, st);
  if (rc != LIDER_OK) return rc;
  hipLaunchKernelGGL(lower_bound_kernel, dim3((C + 1 + 255) / 256), dim3(256), 0, st, kout, n, C,
                     off);
  const int64_t tot = int64_t(C) * d;
  hipLaunchKernelGGL(mean_kernel, dim3(unsigned((tot + 255) / 256)), dim3(256), 0, st, X, d,
                     members, off, C, cent);
  return check_hip(hipGetLastError(), "centroid mean kernels");
}

// ----------------------------------------------------- farthest-first seeding
// D_i = min_j |x_i - c_j|^2 over the chosen centroids in fp32 (relative error
// <= e); every row whose fp32 value is within the error band of the maximum is
// rescored exactly (FP64 minimum over all chosen centroids, sequential sums)
// and the FP64 argmax (ties to the smaller id) becomes the next centroid.
//
// Reading the whole corpus once per centroid bounds the plain form (200,000 x
// 768, 200 centroids: 207 us a round at 3 TB/s, and 89 us for the FP64
// rescoring).  D_i only falls as centroids are added, so the next centroids
// are found among few rows: a full pass brings an upper bound U_i of every D_i
// up to the centroids picked so far (the assignment product: one read of the
// corpus for all of them, plus its error bound), the rows with the largest U_i
// (at least tau, about 1% of the rows) become the short list, their D_i are
// formed as above, and rounds over the list alone pick centroids while the
// error band of the list's maximum stays at or above tau -- a row outside the
// list has D_i <= U_i < tau, so it cannot be a candidate.  The candidates of a
// round, and so the centroids, are those of the plain form.  Where the bounds
// are too wide for a single pick (values of D_i far below |x|^2), D_i itself is
// kept for every row from then on.  200,000 x 768, 200 centroids: 61 ms as a
// full pass and four launches per centroid, 4.5 ms as 6 lists (a full pass
// 0.15 ms, a list's values 0.1 ms, a round 7 us, 20-40 us where it has to
// decide among several candidates).
constexpr double kFFRel = 1.1920928955078125e-07;  // 2^-23 per dimension (fp32 + FP64 side)

struct FFState {
  int32_t t;          // centroids chosen
  int32_t status;     // kFFRun, kFFShort or kFFMany
  int32_t count;      // rows of the short list
  int32_t inc;        // centroids that the list's values include
  int32_t done;       // groups of the round's workgroups that are done
  uint32_t maxbits;   // largest value of the round (float bits)
  uint32_t fullmax;   // largest bound of the last full pass
  int32_t ncand;      // candidates (kFFMany)
  uint32_t taubits;   // smallest value of the list's rows
  int32_t all;        // every row is on the list
  // A round's workgroups count in 8 groups, each counter in a line of its own,
  // and leave their largest values in slots of their own: 256 workgroups with
  // one maximum and one counter, both at one address, spent most of a 37 us
  // round queueing there.
  int32_t gdone[8][32];
  uint32_t bmax[128];
};
// kFFShort: the list no longer holds every possible candidate; kFFMany: more
// candidates than the round's last workgroup rescores itself.
enum { kFFRun = 0, kFFShort = 1, kFFMany = 2 };
constexpr int kFFBins = 4096;       // bins of 2^11 ulp below the maximum
// candidates, and (candidate, centroid) sums, that a round decides itself
constexpr int kFFInline = 8, kFFPairs = 64;
constexpr int kFFChunk = 256;       // squares of such a sum formed at a time
constexpr int kFFRoundThreads = 1024, kFFRoundGrid = 128;
static_assert(kFFRoundGrid % 8 == 0, "eight groups of workgroups");

// Smallest fp32 value of a candidate when the largest is M.
__device__ inline double ff_threshold(double M, int32_t d) {
  const double e = double(d + 3) * kFFRel;
  return M * (1.0 - 2.0 * e) / (1.0 + 2.0 * e) - double(d) * 7.888609052210118e-31;
}

// |x - c|^2 of one row by a wave (every lane returns it).
template <bool VEC>
__device__ inline float ff_dist(const float* __restrict__ x, const float* __restrict__ c, int32_t d,
                                int lane) {
  float s = 0.f;
  if (VEC) {
#pragma unroll 4
    for (int32_t l = 4 * lane; l < d; l += 256) {
      const float4 a = *reinterpret_cast<const float4*>(x + l);
      const float4 b = *reinterpret_cast<const float4*>(c + l);
      const float p = a.x - b.x, q = a.y - b.y, r = a.z - b.z, w = a.w - b.w;
      s += p * p;
      s += q * q;
      s += r * r;
      s += w * w;
    }
  } else {
#pragma unroll 4
    for (int32_t l = lane; l < d; l += 64) {
      const float p = x[l] - c[l];
      s += p * p;
    }
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  return s;
}

// sd[k] <- min(sd[k], |x - c_j|^2) of row sid[k] (k if sid is null) over the
// centroids [c0, c1) of the launch's column (blockIdx.y, cper centroids each),
// as atomic minima of the float bits: all bits set is no value yet, and a NaN
// is above every value.  count null: n rows.  A wave takes 4 rows x 8
// centroids at a time, so a centroid value read serves 4 rows and a row value
// 8 centroids; the 32 sums of the 64 lanes are folded by exchanging halves
// (lane l ends with row l / 16, centroid (l / 2) % 8 of them).
template <bool VEC>
__global__ __launch_bounds__(256) void ff_values_kernel(const float* __restrict__ X, int64_t n,
                                                        int32_t d, const float* __restrict__ cent,
                                                        int32_t c0, int32_t c1, int32_t cper,
                                                        const int32_t* __restrict__ sid,
                                                        const int32_t* __restrict__ count,
                                                        uint32_t* __restrict__ sd) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int W = VEC ? 4 : 1;
  const int64_t rows = count ? int64_t(*count) : n;
  c0 += int32_t(blockIdx.y) * cper;
  c1 = min(c1, c0 + cper);
  for (int64_t r0 = (int64_t(blockIdx.x) * 4 + wave) * 4; r0 < rows; r0 += int64_t(gridDim.x) * 16) {
    const float* xr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t k = min(r0 + r, rows - 1);
      xr[r] = X + (sid ? int64_t(sid[k]) : k) * d;
    }
    float v = __builtin_nanf("");
    for (int32_t c = c0; c < c1; c += 8) {
      const float* cr[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) cr[j] = cent + int64_t(min(c + j, c1 - 1)) * d;
      float acc[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) acc[u] = 0.f;
      for (int32_t l = W * lane; l < d; l += 64 * W) {
        float x[4][W];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (VEC)
            *reinterpret_cast<float4*>(x[r]) = *reinterpret_cast<const float4*>(xr[r] + l);
          else
            x[r][0] = xr[r][l];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          float y[W];
          if (VEC)
            *reinterpret_cast<float4*>(y) = *reinterpret_cast<const float4*>(cr[j] + l);
          else
            y[0] = cr[j][l];
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < W; ++e) {
              const float p = x[r][e] - y[e];
              acc[8 * r + j] += p * p;
            }
        }
      }
#pragma unroll
      for (int h = 16; h > 0; h >>= 1) {  // 2 h sums -> h, lanes 2 h apart
        const bool up = lane & (2 * h);
#pragma unroll
        for (int u = 0; u < h; ++u) {
          const float keep = up ? acc[u + h] : acc[u], send = up ? acc[u] : acc[u + h];
          acc[u] = keep + __shfl_xor(send, 2 * h);
        }
      }
      float w = acc[0] + __shfl_xor(acc[0], 1);
      for (int o = 8; o > 1; o >>= 1) w = fminf(w, __shfl_xor(w, o));  // over the 8 centroids
      v = fminf(v, w);  // fminf drops the NaN start
    }
    const int64_t k = r0 + (lane >> 4);
    if ((lane & 15) == 0 && k < rows) atomicMin(&sd[k], __float_as_uint(v) & 0x7fffffffu);
  }
}

// U_i <- min(U_i, |x_i|^2 + g + E), rounded up, from the assignment product's
// best value g over the last centroids (the smallest over its groups), or +inf
// where a part of it overflowed: such a row goes on the list, and its distances
// decide; with no product, U already holds the values.  The largest U_i.
__global__ __launch_bounds__(256) void ff_bound_kernel(const float4* __restrict__ part, int64_t n,
                                                       int32_t d, int32_t G,
                                                       const uint32_t* __restrict__ maxbits,
                                                       int first, float* __restrict__ U,
                                                       FFState* __restrict__ fs) {
  __shared__ float wmax[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float mx = 0.f;
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
    float u = 0.f;
    if (part) {
      float g = INFINITY, ss = 0.f;
      for (int32_t y = 0; y < G; ++y) {
        const float4 p = part[int64_t(y) * n + i];
        g = fminf(g, p.x);
        ss = p.w;
      }
      const double xn = norm_above(ss, d);
      const double b = xn * xn + double(g) + assign_err(d, xn, double(__uint_as_float(*maxbits)));
      u = float(b);
      if (double(u) < b) u = nextafterf(u, INFINITY);
      if (u < 0.f) u = 0.f;
      // no bound where the square sum, the product or the largest |mu|
      // overflowed (g = -inf: the product did); |x|^2 is a NaN only with one in
      // the row, which is never a candidate
      if (!(b < double(INFINITY)) || !(g > -INFINITY)) u = ss == ss ? INFINITY : ss;
      if (!first) u = fminf(u, U[i]);
      U[i] = u;
    } else {
      u = U[i];
    }
    mx = fmaxf(mx, u);
  }
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if (lane == 0) wmax[wave] = mx;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(&fs->fullmax, __float_as_uint(fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]))));
}

// Counts of the values by their distance below the maximum in float bits.
__global__ __launch_bounds__(256) void ff_hist_kernel(const float* __restrict__ U, int64_t n,
                                                      const FFState* __restrict__ fs,
                                                      int32_t* __restrict__ hist) {
  __shared__ int32_t h[kFFBins];
  for (int b = threadIdx.x; b < kFFBins; b += 256) h[b] = 0;
  __syncthreads();
  const uint32_t M = fs->fullmax;
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) {
    const uint32_t v = __float_as_uint(U[i]);
    if (v <= M && ((M - v) >> 11) < kFFBins) atomicAdd(&h[(M - v) >> 11], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kFFBins; b += 256)
    if (h[b]) atomicAdd(&hist[b], h[b]);
}

// The list's smallest value: as many whole bins as hold at most `target` rows,
// and at least those that hold the candidates of the next round.  Without a
// positive threshold every row is a candidate and goes on the list.
__global__ __launch_bounds__(1024) void ff_tau_kernel(const int32_t* __restrict__ hist, int32_t d,
                                                      int32_t target, FFState* __restrict__ fs) {
  __shared__ int32_t part[1024];
  __shared__ int32_t best;
  const int tid = threadIdx.x;
  int32_t h[kFFBins / 1024], sum = 0;
#pragma unroll
  for (int u = 0; u < kFFBins / 1024; ++u) sum += h[u] = hist[tid * (kFFBins / 1024) + u];
  part[tid] = sum;
  if (tid == 0) best = 0;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int32_t y = tid >= o ? part[tid - o] : 0;
    __syncthreads();
    part[tid] += y;
    __syncthreads();
  }
  int32_t cum = part[tid] - sum;
#pragma unroll
  for (int u = 0; u < kFFBins / 1024; ++u) {
    cum += h[u];
    if (cum <= target) atomicMax(&best, tid * (kFFBins / 1024) + u);
  }
  __syncthreads();
  if (tid == 0) {
    const uint32_t M = fs->fullmax;
    const double T = ff_threshold(double(__uint_as_float(M)), d);
    fs->all = !(T > 0.0);
    uint32_t tau = M - min(M, (uint32_t(best + 1) << 11) - 1u);  // the last bin's smallest value
    if (T > 0.0) {
      float tf = float(T);  // rounded down, so that T >= tau as real numbers
      if (double(tf) > T) tf = nextafterf(tf, 0.f);
      tau = min(tau, __float_as_uint(tf));
    }
    fs->taubits = tau;
    fs->count = 0;
    fs->inc = fs->t;
    fs->done = 0;
    fs->status = kFFRun;
  }
}

// The short list: ids of the rows at or above tau, with their values, or none
// yet (all bits set) where U is only a bound.
__global__ __launch_bounds__(256) void ff_list_kernel(const float* __restrict__ U, int64_t n,
                                                      int bound, int32_t* __restrict__ sid,
                                                      uint32_t* __restrict__ sd,
                                                      FFState* __restrict__ fs) {
  const uint32_t tau = fs->taubits;
  const bool all = fs->all != 0;
  const int lane = threadIdx.x & 63;
  const int64_t stride = int64_t(gridDim.x) * 256;
  for (int64_t i0 = int64_t(blockIdx.x) * 256 + (threadIdx.x - lane); i0 < n; i0 += stride) {
    const int64_t i = i0 + lane;
    const uint32_t vb = i < n ? __float_as_uint(U[i]) : 0u;
    const bool in = i < n && (all || (vb >= tau && vb <= 0x7f800000u));  // no NaN
    const uint64_t m = __ballot(in);
    if (!m) continue;
    int32_t base = 0;
    if (lane == 0) base = atomicAdd(&fs->count, __popcll(m));
    base = __shfl(base, 0);
    if (in) {
      const int32_t at = base + __popcll(m & ((uint64_t(1) << lane) - 1));
      sid[at] = int32_t(i);
      sd[at] = bound ? 0xffffffffu : vb;
    }
  }
}

// Candidates of a round that its last workgroup left (kFFMany), for
// ff_exact_kernel.
__global__ void ff_candidates_kernel(const int32_t* __restrict__ sid, const float* __restrict__ sd,
                                     int32_t d, int64_t* __restrict__ cand,
                                     FFState* __restrict__ fs) {
  const double T = ff_threshold(double(__uint_as_float(fs->maxbits)), d);
  for (int32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < fs->count;
       k += int32_t(gridDim.x * blockDim.x))
    if (double(sd[k]) >= T) cand[atomicAdd(&fs->ncand, 1)] = sid[k];
}

// One round over the short list: a wave per row brings the row's value up to
// the last centroid; the workgroup that finishes last (an agent-scope counter;
// the values pass between workgroups as agent-scope atomics) finds the
// candidates, decides among them and writes the next centroid.  A single
// candidate needs no rescoring.  Up to kFFInline are rescored here: fp32
// distances to all centroids first, then the sequential FP64 sum of those that
// can be the nearest.  It does nothing once the list is used up, so the host
// enqueues many rounds and looks at the state once.
template <bool VEC>
__global__ __launch_bounds__(kFFRoundThreads) void ff_round_kernel(
    const float* __restrict__ X, int32_t d, float* cent, int32_t C, const int32_t* __restrict__ sid,
    float* sd, FFState* fs) {
#pragma clang fp contract(off)
  constexpr int NW = kFFRoundThreads / 64;
  __shared__ float wred[NW], cval[kFFInline];
  __shared__ int32_t s_last, s_n, s_np, cid[kFFInline];
  __shared__ int32_t pc[kFFPairs], pj[kFFPairs];
  __shared__ double pex[kFFPairs], sq[NW][kFFChunk];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t t = fs->t, count = fs->count;
  if (fs->status != kFFRun || t >= C) return;  // only a round's last workgroup changes these
  const bool update = fs->inc < t;
  const float* cl = cent + int64_t(t - 1) * d;
  float mx = 0.f;
  for (int32_t k = int32_t(blockIdx.x) * NW + wave; k < count; k += int32_t(gridDim.x) * NW) {
    float v = sd[k];
    if (update) {
      v = fminf(v, ff_dist<VEC>(X + int64_t(sid[k]) * d, cl, d, lane));
      if (lane == 0) __hip_atomic_store(&sd[k], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    mx = fmaxf(mx, v);
  }
  if (lane == 0) wred[wave] = mx;
  // this wave's stores have reached the agent's memory before the workgroup
  // counts as done (they are agent-scope atomics: waiting for them is enough,
  // a release fence would write back the whole L2 once per wave)
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < NW; ++w) mx = fmaxf(mx, wred[w]);
    __hip_atomic_store(&fs->bmax[blockIdx.x], __float_as_uint(mx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    const bool glast = __hip_atomic_fetch_add(&fs->gdone[blockIdx.x & 7][0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                       kFFRoundGrid / 8 - 1;
    s_last = glast && __hip_atomic_fetch_add(&fs->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 7;
    s_n = s_np = 0;
  }
  __syncthreads();
  if (!s_last) return;
  if (tid < kFFRoundGrid) {
    float v = __uint_as_float(__hip_atomic_load(&fs->bmax[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    if (lane == 0) wred[wave] = v;
  }
  if (tid < 8) fs->gdone[tid][0] = 0;
  __syncthreads();
  float M = wred[0];
  for (int w = 1; w < kFFRoundGrid / 64; ++w) M = fmaxf(M, wred[w]);
  __syncthreads();
  const double T = ff_threshold(double(M), d);
  const bool out = !fs->all && T < double(__uint_as_float(fs->taubits));
  if (out) {
    if (tid == 0) {
      fs->status = kFFShort;
      fs->done = 0;
    }
    return;
  }
  for (int32_t k = tid; k < count; k += kFFRoundThreads) {
    const float v = __hip_atomic_load(&sd[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (double(v) >= T) {
      const int slot = atomicAdd(&s_n, 1);
      if (slot < kFFInline) {
        cid[slot] = sid[k];
        cval[slot] = v;
      }
    }
  }
  __syncthreads();
  const int nc = s_n;
  int32_t np = 0;
  if (nc > 1 && nc <= kFFInline) {
    // the centroids that can be a candidate's nearest: fp32 distances against
    // the candidate's own minimum, sd
    const double e = double(d + 3) * kFFRel;
    for (int32_t u = wave; u < nc * t; u += NW) {
      const int32_t c = u / t, j = u - c * t;
      const double lim = double(cval[c]) * (1.0 + 2.0 * e) / (1.0 - 2.0 * e) + double(d) * 7.888609052210118e-31;
      const float f = ff_dist<VEC>(X + int64_t(cid[c]) * d, cent + int64_t(j) * d, d, lane);
      if (lane == 0 && !(double(f) > lim)) {
        const int slot = atomicAdd(&s_np, 1);
        if (slot < kFFPairs) {
          pc[slot] = c;
          pj[slot] = j;
        }
      }
    }
    __syncthreads();
    np = s_np;
  }
  if (nc > kFFInline || np > kFFPairs) {
    if (tid == 0) {
      fs->inc = t;
      fs->done = 0;
      fs->ncand = 0;
      fs->maxbits = __float_as_uint(M);
      fs->status = kFFMany;
    }
    return;
  }
  // the sequential FP64 sum of each (candidate, centroid): a wave forms the
  // squares 256 at a time in LDS, its lane 0 adds them in order
  for (int32_t u = wave; u < np; u += NW) {
    const float* xr = X + int64_t(cid[pc[u]]) * d;
    const float* mu = cent + int64_t(pj[u]) * d;
    double acc = 0.0;
    for (int32_t l0 = 0; l0 < d; l0 += kFFChunk) {
#pragma unroll
      for (int v = 0; v < kFFChunk; v += 64) {
        const int32_t l = l0 + v + lane;
        const double df = l < d ? double(xr[l]) - double(mu[l]) : 0.0;
        sq[wave][v + lane] = df * df;
      }
      __threadfence_block();
      __builtin_amdgcn_wave_barrier();
      if (lane == 0) {
        const int32_t m = min(d - l0, int32_t(kFFChunk));
#pragma unroll 8
        for (int32_t l = 0; l < m; ++l) acc = acc + sq[wave][l];
      }
      __threadfence_block();
      __builtin_amdgcn_wave_barrier();
    }
    if (lane == 0) pex[u] = acc;
  }
  __syncthreads();
  int32_t pick = nc > 0 ? cid[0] : 0;  // no candidate only with NaN input
  if (nc > 1) {
    double pv = -1.0;
    for (int c = 0; c < nc; ++c) {
      double v = INFINITY;  // the nearest centroid
      for (int u = 0; u < np; ++u)
        if (pc[u] == c) v = fmin(v, pex[u]);
      if (v > pv || (v == pv && cid[c] < pick)) {
        pv = v;
        pick = cid[c];
      }
    }
  }
  for (int l = tid; l < d; l += kFFRoundThreads) cent[int64_t(t) * d + l] = X[int64_t(pick) * d + l];
  if (tid == 0) {
    fs->inc = t;
    fs->t = t + 1;
    fs->done = 0;
  }
}

// Exact FP64 distance of each candidate to its nearest chosen centroid.
__global__ __launch_bounds__(256) void ff_exact_kernel(const float* __restrict__ X, int32_t d,
                                                       const float* __restrict__ cent, int32_t t,
                                                       const int64_t* __restrict__ cand,
                                                       const FFState* __restrict__ fs,
                                                       double* __restrict__ dex) {
#pragma clang fp contract(off)
  __shared__ double sd[256];
  const int32_t cnt = fs->ncand;
  for (int32_t k = blockIdx.x; k < cnt; k += gridDim.x) {
    const float* xr = X + cand[k] * d;
    double best = INFINITY;
    for (int32_t j = threadIdx.x; j < t; j += blockDim.x) {
      const float* mu = cent + int64_t(j) * d;
      double acc = 0.0;
      for (int l = 0; l < d; ++l) {
        double df = double(xr[l]) - double(mu[l]);
        acc = acc + df * df;
      }
      best = acc < best ? acc : best;
    }
    sd[threadIdx.x] = best;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (threadIdx.x < o) sd[threadIdx.x] = fmin(sd[threadIdx.x], sd[threadIdx.x + o]);
      __syncthreads();
    }
    if (threadIdx.x == 0) dex[k] = sd[0];
    __syncthreads();
  }
}

// FP64 argmax over the candidates (ties to the smaller row id); writes the
// new centroid row and lets the rounds go on.
__global__ __launch_bounds__(256) void ff_pick_kernel(const float* __restrict__ X, int32_t d,
                                                      float* __restrict__ cent, int32_t t,
                                                      const int64_t* __restrict__ cand,
                                                      const double* __restrict__ dex,
                                                      FFState* __restrict__ fs) {
  __shared__ double bv[256];
  __shared__ int64_t bi[256];
  const int32_t cnt = fs->ncand;
  double v = -1.0;
  int64_t id = INT64_MAX;
  for (int32_t k = threadIdx.x; k < cnt; k += blockDim.x) {
    const double dv = dex[k];
    const int64_t ci = cand[k];
    if (dv > v || (dv == v && ci < id)) {
      v = dv;
      id = ci;
    }
  }
  bv[threadIdx.x] = v;
  bi[threadIdx.x] = id;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      const double ov = bv[threadIdx.x + o];
      const int64_t oi = bi[threadIdx.x + o];
      if (ov > bv[threadIdx.x] || (ov == bv[threadIdx.x] && oi < bi[threadIdx.x])) {
        bv[threadIdx.x] = ov;
        bi[threadIdx.x] = oi;
      }
    }
    __syncthreads();
  }
  const int64_t pick = bi[0] == INT64_MAX ? 0 : bi[0];  // no candidate only with NaN input
  for (int l = threadIdx.x; l < d; l += blockDim.x) cent[int64_t(t) * d + l] = X[pick * d + l];
  __syncthreads();
  if (threadIdx.x == 0) {
    fs->t = t + 1;
    fs->status = kFFRun;
  }
}

__global__ void gather_rows_kernel(const float* __restrict__ X, int32_t d,
                                   const int64_t* __restrict__ ids, int32_t cnt,
                                   float* __restrict__ out) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= int64_t(cnt) * d) return;
  const int64_t j = t / d;
  out[t] = X[ids[j] * d + (t - j * d)];
}

// Farthest-first centroids 1 .. C - 1 into cent (centroid 0 is there).
// scratch: kmeans_assign_scratch(n, d, C) bytes.
static int run_farthest(const float* X, int64_t n, int32_t d, float* cent, int32_t C, void* scratch,
                        hipStream_t st) {
  float *U = nullptr, *sd = nullptr;
  int32_t *sid = nullptr, *hist = nullptr;
  int64_t* cand = nullptr;
  double* dex = nullptr;
  float4* part = nullptr;
  FFState* fs = nullptr;
  int rc = LIDER_OK;
  const int32_t gmax = asg_groups(n, C);  // of a product with at most C centroids
  if (hipMalloc(&U, size_t(n) * 4) != hipSuccess || hipMalloc(&sd, size_t(n) * 4) != hipSuccess ||
      hipMalloc(&sid, size_t(n) * 4) != hipSuccess ||
      hipMalloc(&hist, kFFBins * 4) != hipSuccess || hipMalloc(&fs, sizeof(FFState)) != hipSuccess ||
      hipMalloc(&part, size_t(gmax) * n * sizeof(float4)) != hipSuccess ||
      hipMalloc(&cand, size_t(n) * 8) != hipSuccess || hipMalloc(&dex, size_t(n) * 8) != hipSuccess)
    rc = set_error(LIDER_ENOMEM, "out of device memory: farthest-first buffers");
  // 16-byte loads: rows of both matrices start at multiples of 16 bytes
  const bool vec = d % 4 == 0 && ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(cent)) & 15) == 0;
  // About 1% of the rows, and at most 8,192 (24 MB of rows at d = 768: the
  // list stays in the Infinity Cache and a round is as short as its launch).
  const int32_t target = int32_t(std::min<int64_t>(8192, std::max<int64_t>(1024, n / 100)));
  const unsigned ngrid = unsigned(std::min<int64_t>((n + 255) / 256, 256));
  // |x - c|^2 of rows (list or all) over the centroids [c0, c1)
  auto values = [&](int64_t rows, const int32_t* ids, const int32_t* count, int32_t c0, int32_t c1,
                    float* out) {
    const int32_t cper = count ? 32 : c1 - c0;
    const dim3 grid(unsigned(std::min<int64_t>((rows + 15) / 16, 1 << 20)),
                    unsigned((c1 - c0 + cper - 1) / cper));
    if (vec)
      hipLaunchKernelGGL(ff_values_kernel<true>, grid, dim3(256), 0, st, X, n, d, cent, c0, c1, cper,
                         ids, count, reinterpret_cast<uint32_t*>(out));
    else
      hipLaunchKernelGGL(ff_values_kernel<false>, grid, dim3(256), 0, st, X, n, d, cent, c0, c1, cper,
                         ids, count, reinterpret_cast<uint32_t*>(out));
  };
  struct {
    int32_t t, status;
  } h{1, kFFRun};  // the state's first words
  static_assert(offsetof(FFState, t) == 0 && offsetof(FFState, status) == 4, "read back together");
  int32_t base = 0, guess = 32;
  bool direct = false;  // U holds D itself
  if (rc == LIDER_OK) {
    hipLaunchKernelGGL(zero_i32_kernel2, dim3(2), dim3(256), 0, st, reinterpret_cast<int32_t*>(fs),
                       int64_t(sizeof(FFState) / 4));
    rc = check_hip(hipMemcpyAsync(fs, &h, sizeof(h), hipMemcpyHostToDevice, st), "farthest-first state");
  }
  while (rc == LIDER_OK && h.t < C) {
    // every row up to the centroids [base, t), and the next list
    hipLaunchKernelGGL(zero_i32_kernel2, dim3(16), dim3(256), 0, st, hist, int64_t(kFFBins));
    hipLaunchKernelGGL(zero_i32_kernel2, dim3(1), dim3(64), 0, st,
                       reinterpret_cast<int32_t*>(&fs->fullmax), int64_t(1));
    if (direct) {
      if (base == 0)
        hipLaunchKernelGGL(fill_i32_kernel, dim3(ngrid), dim3(256), 0, st,
                           reinterpret_cast<int32_t*>(U), n, -1);
      values(n, nullptr, nullptr, base, h.t, U);
      hipLaunchKernelGGL(ff_bound_kernel, dim3(ngrid), dim3(256), 0, st, (const float4*)nullptr, n, d,
                         0, (const uint32_t*)nullptr, 0, U, fs);
    } else {
      const uint32_t* maxbits = nullptr;
      const int32_t G = launch_assign_product(X, n, d, cent + int64_t(base) * d, h.t - base, scratch,
                                              part, &maxbits, st);
      hipLaunchKernelGGL(ff_bound_kernel, dim3(ngrid), dim3(256), 0, st, part, n, d, G, maxbits,
                         base == 0 ? 1 : 0, U, fs);
    }
    hipLaunchKernelGGL(ff_hist_kernel, dim3(ngrid), dim3(256), 0, st, U, n, fs, hist);
    hipLaunchKernelGGL(ff_tau_kernel, dim3(1), dim3(1024), 0, st, hist, d, target, fs);
    hipLaunchKernelGGL(ff_list_kernel, dim3(ngrid), dim3(256), 0, st, U, n, direct ? 0 : 1, sid,
                       reinterpret_cast<uint32_t*>(sd), fs);
    if (!direct) values(target, sid, &fs->count, 0, h.t, sd);
    base = h.t;
    do {
      const int32_t rounds = std::min(guess, C - h.t);
      for (int32_t u = 0; u < rounds; ++u) {
        if (vec)
          hipLaunchKernelGGL(ff_round_kernel<true>, dim3(kFFRoundGrid), dim3(kFFRoundThreads), 0, st,
                             X, d, cent, C, sid, sd, fs);
        else
          hipLaunchKernelGGL(ff_round_kernel<false>, dim3(kFFRoundGrid), dim3(kFFRoundThreads), 0,
                             st, X, d, cent, C, sid, sd, fs);
      }
      rc = check_hip(hipGetLastError(), "farthest-first seeding");
      if (rc == LIDER_OK)
        rc = check_hip(hipMemcpyAsync(&h, fs, sizeof(h), hipMemcpyDeviceToHost, st), "farthest-first state");
      if (rc == LIDER_OK) rc = check_hip(hipStreamSynchronize(st), "farthest-first seeding");
      if (rc == LIDER_OK && h.status == kFFMany) {
        hipLaunchKernelGGL(ff_candidates_kernel, dim3(ngrid), dim3(256), 0, st, sid, sd, d, cand, fs);
        hipLaunchKernelGGL(ff_exact_kernel, dim3(256), dim3(256), 0, st, X, d, cent, h.t, cand, fs, dex);
        hipLaunchKernelGGL(ff_pick_kernel, dim3(1), dim3(256), 0, st, X, d, cent, h.t, cand, dex, fs);
        ++h.t;
        h.status = kFFRun;
      }
    } while (rc == LIDER_OK && h.status == kFFRun && h.t < C);
    // rounds past the list's end return at once, but are not free
    guess = std::min(64, std::max(8, h.t - base + (h.t - base) / 4));
    if (h.t == base && !direct) {  // not one pick: from now on the values themselves
      direct = true;
      base = 0;
    }
  }
  if (rc == LIDER_OK) rc = check_hip(hipStreamSynchronize(st), "farthest-first seeding");
  for (void* p : {(void*)U, (void*)sd, (void*)sid, (void*)hist, (void*)fs, (void*)cand, (void*)dex, (void*)part})
    if (p) (void)hipFree(p);
  return rc;
}

// Lloyd iterations into ix.cent / ix.assign.
int run_kmeans(Index& ix, const float* X, const int64_t* init_host, int32_t iters,
               int32_t seeding, hipStream_t st) {
  const int64_t n = ix.n;
  const int32_t C = ix.C, d = ix.d;
  int64_t* init_dev = nullptr;
  int32_t* bufs[2] = {nullptr, nullptr};
  int32_t* changed = nullptr;
  void* scr_a = nullptr;
  void* scr_m = nullptr;
  const size_t sa = kmeans_assign_scratch(n, d, C), sm = centroid_means_scratch(n, C);
  int rc = LIDER_OK;
  auto fail = [&](int code, const char* what) {
    rc = code == LIDER_ENOMEM ? set_error(LIDER_ENOMEM, std::string("out of device memory: ") + what)
                              : code;
  };
  if (hipMalloc(&init_dev, size_t(C) * 8) != hipSuccess ||
      hipMalloc(&bufs[0], size_t(n) * 4) != hipSuccess ||
      hipMalloc(&bufs[1], size_t(n) * 4) != hipSuccess || hipMalloc(&changed, 256) != hipSuccess ||
      hipMalloc(&scr_a, sa) != hipSuccess || hipMalloc(&scr_m, sm) != hipSuccess) {
    fail(LIDER_ENOMEM, "k-means buffers");
  }
  if (rc == LIDER_OK) {
    rc = check_hip(hipMemcpyAsync(init_dev, init_host, size_t(C) * 8, hipMemcpyHostToDevice, st),
                   "copy k-means initial ids");
  }
  if (rc == LIDER_OK) {
    const int64_t tot = int64_t(seeding ? 1 : C) * d;
    hipLaunchKernelGGL(gather_rows_kernel, dim3(unsigned((tot + 255) / 256)), dim3(256), 0, st,
                       X, d, init_dev, seeding ? 1 : C, ix.cent);
  }
  if (rc == LIDER_OK && seeding == 1 && C > 1) rc = run_farthest(X, n, d, ix.cent, C, scr_a, st);
  int cur = 0, fin = 0;
  int32_t it = 0;
  while (rc == LIDER_OK && it < iters) {
    hipLaunchKernelGGL(zero_i32_kernel2, dim3(1), dim3(64), 0, st, changed, int64_t(1));
    rc = run_kmeans_assign(X, n, d, ix.cent, C, bufs[cur], it > 0 ? bufs[cur ^ 1] : nullptr,
                           changed, scr_a, st);
    if (rc != LIDER_OK) break;
    if (it > 0) {
      int32_t h_changed = 0;
      rc = check_hip(hipMemcpyAsync(&h_changed, changed, 4, hipMemcpyDeviceToHost, st),
                     "read k-means change count");
      if (rc == LIDER_OK) rc = check_hip(hipStreamSynchronize(st), "k-means iteration");
      if (rc != LIDER_OK) break;
      if (h_changed == 0) {  // converged: centroids already are this assignment's means
        fin = cur;
        ++it;
        break;
      }
    }
    rc = run_centroid_means(X, n, d, bufs[cur], C, ix.cent, scr_m, sm, st);
    fin = cur;
    cur ^= 1;
    ++it;
  }
  ix.iters_run = it;
  if (rc == LIDER_OK)
    rc = check_hip(hipMemcpyAsync(ix.assign, bufs[fin], size_t(n) * 4, hipMemcpyDeviceToDevice, st),
                   "copy final assignment");
  if (rc == LIDER_OK) rc = check_hip(hipStreamSynchronize(st), "k-means");
  hipFree(init_dev);
  hipFree(changed);
  hipFree(scr_a);
  hipFree(scr_m);
  hipFree(bufs[0]);
  hipFree(bufs[1]);
  return rc;
}

}  // namespace lider
