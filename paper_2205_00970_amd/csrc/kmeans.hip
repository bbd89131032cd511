// k-means clustering of the corpus (Sections 3.2, 3.3.2): Lloyd iterations.
//
// Assignment = argmin_j |x - mu_j|^2 decided in FP64 with ties to the smaller
// j.  The distances come from a split bf16 MFMA product (g_j = |mu_j|^2 -
// 2 x.mu_j, the |x|^2 term is common to all j); when the best and second-best
// values are closer than a rigorous rounding-error bound allows, the point is
// queued and all its distances are recomputed sequentially in FP64 (sum over
// dimensions of (x_l - mu_l)^2, no contraction), which reproduces the FP64
// definition.
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

// The centroids split into h = bf16(mu) and l = bf16(mu - h) in the operand
// order of the assignment product: per 16-centroid block and 32-dim step the
// h part and the l part, 1 KB each, lane i + 16 s holding dims [8 s, 8 s + 8)
// of centroid i (zeros past d and past C).  One wave per centroid; it also
// writes |mu_j|^2 in fp32 (+inf for the centroids past C, which are never
// nearest) and an upper bound of max_j |mu_j| (as float bits, atomicMax).
__global__ __launch_bounds__(256) void cent_split_kernel(const float* __restrict__ cent, int32_t C,
                                                         int32_t d, bf16x8* __restrict__ out,
                                                         float* __restrict__ cnorm,
                                                         uint32_t* __restrict__ maxbits) {
  const int lane = threadIdx.x & 63;
  const int64_t j = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int32_t nk = asg_steps(d);
  const float* mu = cent + j * d;
  bf16x8* o = out + (j >> 4) * (int64_t(nk) * 128) + (j & 15);
  float s = 0.f;
  for (int32_t u = lane; u < 4 * nk; u += 64) {  // eight dims per lane
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = j < C && 8 * u + e < d ? mu[8 * u + e] : 0.f;
      s += v[e] * v[e];
    }
    bf16x8 h, l;
    split8(v, h, l);
    bf16x8* q = o + (u >> 2) * 128 + 16 * (u & 3);
    q[0] = h;
    q[64] = l;
  }
  for (int x = 32; x > 0; x >>= 1) s += __shfl_xor(s, x);
  if (lane == 0) {
    cnorm[j] = j < C ? s : INFINITY;
    if (j < C) {
      const double gam = double(d + 2) * 5.9604644775390625e-08;
      float ub = float(sqrt(double(s) * (1.0 + 2.0 * gam)) * (1.0 + 9.5367431640625e-07));
      atomicMax(maxbits, __float_as_uint(ub));
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

// Decides one point from its best and second-best value and |x|^2 (fp32), or
// queues it.  The split values x = h + l + r (|x - h| <= u |x|, |l| <= u (1 +
// u) |x|, |r| <= u^2 |x|, u = 2^-8) and the products h h + h l + l h leave x.mu
// within ((2 (1 + u)^2 + 1) u^2 + dot_err_coef(3 d) (1 + u)^2 (1 + 2 u)) |x|
// |mu|, plus absolute terms for parts below 2^-126; |mu|^2 in fp32 is within
// dot_err_coef(d) |mu|^2, and the fp32 combination adds 2^-22.
__device__ inline void assign_decide(const AssignOut& o, int64_t row, const Best& b, float ssr) {
  const double gam = double(o.d + 2) * 5.9604644775390625e-08;
  const double u = 0.00390625;
  const double dotc = ((2.0 * (1.0 + u) * (1.0 + u) + 1.0) * u * u +
                       dot_err_coef(3 * o.d) * (1.0 + u) * (1.0 + u) * (1.0 + 2.0 * u)) * 1.01;
  const double M = double(__uint_as_float(*o.maxbits));
  const double xn = sqrt(double(ssr) * (1.0 + 2.0 * gam)) * (1.0 + 9.5367431640625e-07);
  const double E = (dot_err_coef(o.d) + 2.384185791015625e-07) * M * M +
                   2.0 * (dotc + 2.384185791015625e-07) * xn * M +
                   6.0 * sqrt(double(o.d)) * 1.1754943508222875e-38 * (xn + M) +
                   double(o.d + 2) * 8.881784197001252e-16 * (xn + M) * (xn + M) +
                   6.0 * double(o.d) * 7.888609052210118e-31;
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
// product of 16 points per wave straight from L2, 740 us now (750 TFLOP/s of
// bf16 products, 77% of the rate of a plain 8192^3 library product once the
// last round of 469 workgroups on 256 CUs is allowed for).
// The values of a tile are reduced over the wave's columns (registers, then
// DPP rotations over the 16 lanes of a point) and merged into the point's
// best in LDS, so no value is stored.  One group: decided here, else the
// groups' bests are merged by assign_merge_kernel.
template <bool VEC>
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
        if (VEC) {  // d % 4 == 0: a whole float4 lies inside the point or past it
          xa[a][h] = kd < d ? *reinterpret_cast<const float4*>(xk + at) : float4{0.f, 0.f, 0.f, 0.f};
        } else {
          xa[a][h].x = kd < d ? xk[at] : 0.f;
          xa[a][h].y = kd + 1 < d ? xk[at + 1] : 0.f;
          xa[a][h].z = kd + 2 < d ? xk[at + 2] : 0.f;
          xa[a][h].w = kd + 3 < d ? xk[at + 3] : 0.f;
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
        const float v[8] = {xa[a][0].x, xa[a][0].y, xa[a][0].z, xa[a][0].w,
                            xa[a][1].x, xa[a][1].y, xa[a][1].z, xa[a][1].w};
        split8(v, ah[a], al[a]);
        if (t == t0) {
#pragma unroll
          for (int e = 0; e < 8; ++e) ss[a] += v[e] * v[e];
        }
      }
      const bool last = kc + 1 == nk;
      const bool more = !last || t + 1 < t1;
      if (more) {  // the next step's operands, in flight during this one
        load_cents(last ? t + 1 : t, last ? 0 : kc + 1);
        load_points(last ? 0 : kc + 1);
      }
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
      if (more) store_cents(slot ^ 1);
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
    if (G == 1)
      assign_decide(o, row0 + tid, v, sss[tid]);
    else
      part[int64_t(g) * n + row0 + tid] = float4{v.bv, __int_as_float(v.bi), v.sv, sss[tid]};
  }
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

// FP64 recompute for queued points: one block per point, threads over
// centroids, each distance a sequential sum without contraction.
__global__ __launch_bounds__(256) void assign_fixup_kernel(
    const float* __restrict__ X, int32_t d, const float* __restrict__ cent, int32_t C,
    int32_t* __restrict__ assign, const int32_t* __restrict__ prev, int32_t* __restrict__ changed,
    const int64_t* __restrict__ amb, const int32_t* __restrict__ amb_count) {
#pragma clang fp contract(off)
  __shared__ double sd[256];
  __shared__ int32_t sj[256];
  const int32_t cnt = *amb_count;
  for (int32_t t = blockIdx.x; t < cnt; t += gridDim.x) {
    const int64_t row = amb[t];
    const float* xr = X + row * d;
    double bd = INFINITY;
    int32_t bj = 0x7fffffff;
    for (int32_t j = threadIdx.x; j < C; j += blockDim.x) {
      const float* mu = cent + int64_t(j) * d;
      double acc = 0.0;
      for (int l = 0; l < d; ++l) {
        double df = double(xr[l]) - double(mu[l]);
        acc = acc + df * df;
      }
      if (acc < bd) {
        bd = acc;
        bj = j;
      }
    }
    sd[threadIdx.x] = bd;
    sj[threadIdx.x] = bj;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (threadIdx.x < o) {
        double od = sd[threadIdx.x + o];
        int32_t oj = sj[threadIdx.x + o];
        if (od < sd[threadIdx.x] || (od == sd[threadIdx.x] && oj < sj[threadIdx.x])) {
          sd[threadIdx.x] = od;
          sj[threadIdx.x] = oj;
        }
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      assign[row] = sj[0];
      if (prev && prev[row] != sj[0]) atomicAdd(changed, 1);
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

// scratch: cnorm [256 tiles] f32 | maxbits u32 | amb_count i32 | amb [n] i64 |
// split centroids [256 tiles x 32 steps] 2 bf16 | groups' bests [G x n] float4
static size_t asg_split_bytes(int32_t C, int32_t d) {
  return size_t((int64_t(C) + kAsgTile - 1) / kAsgTile) * kAsgTile * size_t(asg_steps(d)) * 32 * 4;
}

size_t kmeans_assign_scratch(int64_t n, int32_t d, int32_t C) {
  const int32_t G = asg_groups(n, C);
  return al256((size_t(C) + kAsgTile) * 4) + 256 + al256(size_t(n) * 8) + asg_split_bytes(C, d) +
         (G > 1 ? size_t(G) * n * sizeof(float4) : 0);
}

int run_kmeans_assign(const float* X, int64_t n, int32_t d, const float* cent, int32_t C,
                      int32_t* assign, const int32_t* prev, int32_t* changed, void* scratch,
                      hipStream_t st) {
  char* p = static_cast<char*>(scratch);
  float* cnorm = reinterpret_cast<float*>(p);
  p += al256((size_t(C) + kAsgTile) * 4);
  uint32_t* maxbits = reinterpret_cast<uint32_t*>(p);
  int32_t* amb_count = reinterpret_cast<int32_t*>(p + 4);
  p += 256;
  int64_t* amb = reinterpret_cast<int64_t*>(p);
  p += al256(size_t(n) * 8);
  bf16x8* cs = reinterpret_cast<bf16x8*>(p);
  p += asg_split_bytes(C, d);
  float4* part = reinterpret_cast<float4*>(p);
  const int32_t ntiles = int32_t((int64_t(C) + kAsgTile - 1) / kAsgTile);
  const int32_t G = asg_groups(n, C);
  const AssignOut o{d, C, maxbits, assign, prev, changed, amb, amb_count};
  hipLaunchKernelGGL(zero_i32_kernel2, dim3(1), dim3(64), 0, st,
                     reinterpret_cast<int32_t*>(maxbits), int64_t(2));
  hipLaunchKernelGGL(cent_split_kernel, dim3(unsigned(ntiles) * (kAsgTile / 4)), dim3(256), 0, st,
                     cent, C, d, cs, cnorm, maxbits);
  const bool vec = (d % 4 == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0);
  const dim3 grid(unsigned((n + kAsgTile - 1) / kAsgTile), unsigned(G));
  if (vec)
    hipLaunchKernelGGL(assign_kernel<true>, grid, dim3(512), 0, st, X, n, d, cs, cnorm, ntiles, o,
                       part);
  else
    hipLaunchKernelGGL(assign_kernel<false>, grid, dim3(512), 0, st, X, n, d, cs, cnorm, ntiles, o,
                       part);
  if (G > 1)
    hipLaunchKernelGGL(assign_merge_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st,
                       part, n, G, o);
  hipLaunchKernelGGL(assign_fixup_kernel, dim3(1024), dim3(256), 0, st, X, d, cent, C, assign,
                     prev, changed, amb, amb_count);
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
// id), mean rounded once to fp32.
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
  for (int64_t p = a; p < e; ++p) s = s + double(X[int64_t(members[p]) * d + l]);
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
// Round t: D_i <- min(D_i, |x_i - c_{t-1}|^2) in fp32 (relative error <= e),
// then every row whose fp32 value is within the error band of the maximum is
// rescored exactly (FP64 minimum over all chosen centroids, sequential sums)
// and the FP64 argmax (ties to the smaller id) becomes centroid t.
constexpr double kFFRel = 1.1920928955078125e-07;  // 2^-23 per dimension (fp32 + FP64 side)

__global__ __launch_bounds__(256) void ff_update_kernel(const float* __restrict__ X, int64_t n,
                                                        int32_t d, const float* __restrict__ c,
                                                        float* __restrict__ D,
                                                        uint32_t* __restrict__ maxbits, int first) {
  __shared__ float wmax[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float mx = 0.f;
  for (int64_t i = int64_t(blockIdx.x) * 4 + wave; i < n; i += int64_t(gridDim.x) * 4) {
    const float* xr = X + i * d;
    float s = 0.f;
    for (int l = lane; l < d; l += 64) {
      const float t = xr[l] - c[l];
      s += t * t;
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    float v = first ? s : fminf(D[i], s);
    if (lane == 0) D[i] = v;
    mx = fmaxf(mx, v);
  }
  if (lane == 0) wmax[wave] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    float m = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    atomicMax(maxbits, __float_as_uint(m));
  }
}

__global__ void ff_candidates_kernel(const float* __restrict__ D, int64_t n, int32_t d,
                                     const uint32_t* __restrict__ maxbits,
                                     int64_t* __restrict__ cand, int32_t* __restrict__ ncand) {
  const double e = double(d + 3) * kFFRel;
  const double M = double(__uint_as_float(*maxbits));
  const double T = M * (1.0 - 2.0 * e) / (1.0 + 2.0 * e) - double(d) * 7.888609052210118e-31;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x) {
    if (double(D[i]) >= T) cand[atomicAdd(ncand, 1)] = i;
  }
}

// Exact FP64 distance of each candidate to its nearest chosen centroid.
__global__ __launch_bounds__(256) void ff_exact_kernel(const float* __restrict__ X, int32_t d,
                                                       const float* __restrict__ cent, int32_t t,
                                                       const int64_t* __restrict__ cand,
                                                       const int32_t* __restrict__ ncand,
                                                       double* __restrict__ dex) {
#pragma clang fp contract(off)
  __shared__ double sd[256];
  const int32_t cnt = *ncand;
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
// new centroid row, resets the per-round counters.
__global__ __launch_bounds__(256) void ff_pick_kernel(const float* __restrict__ X, int32_t d,
                                                      float* __restrict__ cent, int32_t t,
                                                      int64_t* __restrict__ cand,
                                                      int32_t* __restrict__ ncand,
                                                      const double* __restrict__ dex,
                                                      uint32_t* __restrict__ maxbits) {
  __shared__ double bv[256];
  __shared__ int64_t bi[256];
  const int32_t cnt = *ncand;
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
    *ncand = 0;
    *maxbits = 0;
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
  if (rc == LIDER_OK && seeding == 1 && C > 1) {
    float* D = nullptr;
    int64_t* cand = nullptr;
    double* dex = nullptr;
    if (hipMalloc(&D, size_t(n) * 4) != hipSuccess || hipMalloc(&cand, size_t(n) * 8) != hipSuccess ||
        hipMalloc(&dex, size_t(n) * 8) != hipSuccess)
      fail(LIDER_ENOMEM, "farthest-first buffers");
    int32_t* ncand = changed;  // [0] candidate count, [1] max bits
    uint32_t* maxbits = reinterpret_cast<uint32_t*>(changed + 1);
    if (rc == LIDER_OK) {
      hipLaunchKernelGGL(zero_i32_kernel2, dim3(1), dim3(64), 0, st, changed, int64_t(2));
      const unsigned ub = unsigned(std::min<int64_t>((n + 3) / 4, 8192));
      const unsigned cb = unsigned(std::min<int64_t>((n + 255) / 256, 4096));
      for (int32_t t = 1; t < C; ++t) {
        hipLaunchKernelGGL(ff_update_kernel, dim3(ub), dim3(256), 0, st, X, n, d,
                           ix.cent + int64_t(t - 1) * d, D, maxbits, t == 1 ? 1 : 0);
        hipLaunchKernelGGL(ff_candidates_kernel, dim3(cb), dim3(256), 0, st, D, n, d, maxbits,
                           cand, ncand);
        hipLaunchKernelGGL(ff_exact_kernel, dim3(256), dim3(256), 0, st, X, d, ix.cent, t, cand,
                           ncand, dex);
        hipLaunchKernelGGL(ff_pick_kernel, dim3(1), dim3(256), 0, st, X, d, ix.cent, t, cand,
                           ncand, dex, maxbits);
      }
      rc = check_hip(hipGetLastError(), "farthest-first seeding");
      if (rc == LIDER_OK) rc = check_hip(hipStreamSynchronize(st), "farthest-first seeding");
    }
    if (D) hipFree(D);
    if (cand) hipFree(cand);
    if (dex) hipFree(dex);
  }
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
