// Batch normalisation (training mode) over an NHWC tensor viewed as [M][C]:
// statistics per channel over all M = N*H*W rows.
//
// Statistics are two-level and deterministic. Forward: the conv epilogue
// writes per-tile partial sums of (v - shift) and (v - shift)^2 with a sample
// of the channel as the shift (well conditioned when |mean| >> std), merged in
// fp64 by the pass that applies them (bn_coefs). Backward: each block reduces a
// contiguous range of rows to per-channel partial sums in fp32 (16-byte row
// chunks read coalesced, then a fixed-order LDS reduction), combined in fp64.
//
// The elementwise passes (apply + ReLU + residual, backward apply) are 16-byte
// HBM streams; a thread keeps its channels' coefficients in registers.
#include <hip/hip_ext.h>

#include <algorithm>

#include "kernels.h"
#include "pool.h"

namespace rn18 {

namespace {

constexpr int kMaxC = 512;

// Blocks of a grid-sweeping reduction over M rows, rows_per_iter rows per
// block step: every thread takes at least min_rows rows and at most cap
// blocks run, but while each thread would still take 8 rows there are at
// least floor_blocks. Measured on the BN backward reductions at bf16: up to
// two blocks per CU with 16 rows per thread beat more blocks with fewer rows
// (50176 x 256: 784 blocks 20.4 us, 392 blocks 15.7 us), and a grid smaller
// than the CU count is slower again.
int pick_blocks(long M, int rows_per_iter, int min_rows, int cap, int floor_blocks) {
  long b = M / ((long)rows_per_iter * min_rows);
  if (b > cap) b = cap;
  const long lo8 = M / ((long)rows_per_iter * 8), lo = lo8 < floor_blocks ? lo8 : floor_blocks;
  if (b < lo) b = lo;
  if (b < 1) b = 1;
  return (int)b;
}

__device__ inline double block_sum_d(double v, double* sh) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) sh[tid] += sh[tid + s];
    __syncthreads();
  }
  double r = sh[0];
  __syncthreads();
  return r;
}

// Batch statistics from the per-tile partials (rows n, shift x0, sum of
// v - x0, sum of (v - x0)^2) of the forward conv epilogue. Every tile's sums
// are re-referenced to one sample of the channel, K = tile 0's shift, in
// fp64 (d = x0 - K: S1 += s1 + n d, S2 += s2 + 2 d s1 + n d^2), so the
// tiles simply add; then mean = K + S1/M, biased variance S2/M - (S1/M)^2 for
// normalising, unbiased (M/(M-1)) for the running one.
//
// No kernel of its own finishes them: each block of the pass that applies the
// batch norm takes up to 64 channels (kCG) and adds up their partials itself
// in a fixed order (64 channels x 4 thread groups), so every block gets the
// same coefficients, and the first block of a channel group writes them for
// the backward pass. A layer with at most 64 tile partials needs no launch
// before it; above that bn_stats_tiles_reduce_kernel sums chunks of tiles
// first (at most 16, so that a block reads at most 24 KB). A launch of a few
// blocks costs 4-7 us beside its neighbours on MI355X: folding the finish took
// the batch-64 step at 128x128 from 1.63 to 1.50 ms.
__device__ inline void bn_tile_sum(const float4& p, double K, double& N, double& S1, double& S2) {
  const double n = p.x, d = (double)p.y - K, s1 = p.z;
  N += n;
  S1 += s1 + n * d;
  S2 += (double)p.w + 2.0 * d * s1 + n * d * d;
}

__global__ __launch_bounds__(256) void bn_stats_tiles_reduce_kernel(const float* __restrict__ st, int ntiles, int C,
                                                                    int per_chunk, double* __restrict__ red) {
  __shared__ double sh[3][4][64];
  const int cl = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + cl;
  const int z0 = blockIdx.y * per_chunk, z1 = min(ntiles, z0 + per_chunk);
  double N = 0.0, S1 = 0.0, S2 = 0.0;
  if (c < C) {
    const double K = (double)((const float4*)st)[c].y;
#pragma unroll 8
    for (int z = z0 + q; z < z1; z += 4) bn_tile_sum(((const float4*)st)[(long)z * C + c], K, N, S1, S2);
  }
  sh[0][q][cl] = N; sh[1][q][cl] = S1; sh[2][q][cl] = S2;
  __syncthreads();
  if (q == 0 && c < C) {
    double* out = red + ((long)blockIdx.y * C + c) * 3;
#pragma unroll
    for (int k = 0; k < 3; ++k) out[k] = ((sh[k][0][cl] + sh[k][1][cl]) + sh[k][2][cl]) + sh[k][3][cl];
  }
}

constexpr int kCG = 64;   // channels of a block of the applying passes

// Scale and shift of channels [c0, c0 + CG) into sc / sf (LDS), from the
// source b describes; a training pass's first block (write) stores them, the
// mean, rstd and the running statistics. All 256 threads; ends in a barrier.
__device__ inline void bn_coefs(const BnSrc& b, int C, int c0, int CG, bool write, double (&sh)[3][4][kCG], float* sc,
                                float* sf) {
  const int cl = threadIdx.x & 63, q = threadIdx.x >> 6, c = c0 + cl;
  if (b.kind == BnSrc::EVAL || b.kind == BnSrc::STORED) {
    if (q == 0 && cl < CG) {
      if (b.kind == BnSrc::STORED) {
        sc[cl] = b.scale[c];
        sf[cl] = b.shift[c];
      } else {
        const double rstd = 1.0 / sqrt((double)b.rv[c] + (double)b.eps);
        const double k = (double)b.gamma[c] * rstd;
        sc[cl] = (float)k;
        sf[cl] = (float)((double)b.beta[c] - (double)b.rm[c] * k);
        if (write) {
          b.scale[c] = sc[cl];
          b.shift[c] = sf[cl];
        }
      }
    }
    __syncthreads();
    return;
  }
  double N = 0.0, S1 = 0.0, S2 = 0.0, K = 0.0;
  float ga = 0.f, be = 0.f;
  if (cl < CG) {
    ga = b.gamma[c];
    be = b.beta[c];
    K = (double)((const float4*)b.st)[c].y;
    if (b.kind == BnSrc::TILES) {
#pragma unroll 8
      for (int z = q; z < b.n; z += 4) bn_tile_sum(((const float4*)b.st)[(long)z * C + c], K, N, S1, S2);
    } else {
#pragma unroll 4
      for (int z = q; z < b.n; z += 4) {
        const double* p = b.red + ((long)z * C + c) * 3;
        N += p[0];
        S1 += p[1];
        S2 += p[2];
      }
    }
  }
  sh[0][q][cl] = N; sh[1][q][cl] = S1; sh[2][q][cl] = S2;
  __syncthreads();
  if (q == 0 && cl < CG) {
    N = ((sh[0][0][cl] + sh[0][1][cl]) + sh[0][2][cl]) + sh[0][3][cl];
    S1 = ((sh[1][0][cl] + sh[1][1][cl]) + sh[1][2][cl]) + sh[1][3][cl];
    S2 = ((sh[2][0][cl] + sh[2][1][cl]) + sh[2][2][cl]) + sh[2][3][cl];
    const double m1 = S1 / N;
    double var = S2 / N - m1 * m1;
    if (var < 0.0) var = 0.0;
    const double mean = K + m1;
    const double rstd = 1.0 / sqrt(var + (double)b.eps);
    const double k = (double)ga * rstd;
    const float fs = (float)k, ff = (float)((double)be - mean * k);
    sc[cl] = fs;
    sf[cl] = ff;
    if (write) {
      b.mean[c] = (float)mean;
      b.rstd[c] = (float)rstd;
      b.scale[c] = fs;
      b.shift[c] = ff;
      if (b.rm) {
        b.rm[c] = (float)((1.0 - b.mom) * (double)b.rm[c] + b.mom * mean);
        b.rv[c] = (float)((1.0 - b.mom) * (double)b.rv[c] + b.mom * (N > 1.0 ? var * (N / (N - 1.0)) : 0.0));
      }
    }
  }
  __syncthreads();
}

// Block geometry of the applying passes: block b takes channel group b %
// groups and every (blocks / groups)-th step of rpi rows, four steps at a time;
// a thread keeps its channels, so their coefficients live in registers. The
// first loads are issued before the coefficients are known, so that the sums
// of the partials run while they arrive.
struct RowWalk {
  int CG, cpr, c0, cc, rr, rpi, rb, nrb;   // group channels, chunks per row, first channel, chunk, row, rows per step
  __device__ inline RowWalk(int C, int VW) {
    CG = min(kCG, C);
    const int groups = C / CG, cpg = CG / VW, g = blockIdx.x % groups;
    cpr = C / VW;
    c0 = g * CG;
    cc = g * cpg + (int)threadIdx.x % cpg;
    rr = threadIdx.x / cpg;
    rpi = 256 / cpg;
    rb = blockIdx.x / groups;
    nrb = gridDim.x / groups;
  }
};
constexpr int kRowsU = 4;   // rows per thread and step

// z = act(bn(y) [+ r] [+ bn2(r)]): RES 0, 1, 2. The pass is an HBM stream (2
// or 3 tensors).
template <typename T, int RES>
__global__ __launch_bounds__(256) void bn_apply_kernel(const T* __restrict__ y, BnSrc b1, int relu,
                                                       const T* __restrict__ r, BnSrc b2, T* __restrict__ z, long M,
                                                       int C, uint8_t* __restrict__ mbits) {
  constexpr int VW = TT<T>::VW, U = kRowsU;
  __shared__ double sh[3][4][kCG];
  __shared__ float lsc[kCG], lsf[kCG], lsc2[kCG], lsf2[kCG];
  const RowWalk w(C, VW);
  const long step = (long)w.nrb * w.rpi;
  struct Rows { uint4 y[U], r[RES ? U : 1]; };
  auto at = [&](long row) { return (uint32_t)(row * w.cpr + w.cc); };
  auto load = [&](long r0, Rows& d) {   // (rows past the end load the last row)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = at(min(r0 + u * step, M - 1));
      d.y[u] = ((const uint4*)y)[i];
      if constexpr (RES != 0) d.r[u] = ((const uint4*)r)[i];
    }
  };
  long r0 = (long)w.rb * w.rpi + w.rr;
  Rows d;
  load(r0, d);
  bn_coefs(b1, C, w.c0, w.CG, w.rb == 0, sh, lsc, lsf);
  if constexpr (RES == 2) bn_coefs(b2, C, w.c0, w.CG, w.rb == 0, sh, lsc2, lsf2);
  const int cl = w.cc * VW - w.c0;
  float sc[VW], sf[VW], sc2[VW], sf2[VW];
#pragma unroll
  for (int e = 0; e < VW; ++e) {
    sc[e] = lsc[cl + e];
    sf[e] = lsf[cl + e];
    sc2[e] = RES == 2 ? lsc2[cl + e] : 0.f;
    sf2[e] = RES == 2 ? lsf2[cl + e] : 0.f;
  }
  auto process = [&](long r0, const Rows& d) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r0 + u * step >= M) break;
      const uint32_t i = at(r0 + u * step);
      float v[VW];
      unpack<T>(d.y[u], v);
#pragma unroll
      for (int e = 0; e < VW; ++e) v[e] = bn_affine(v[e], sc[e], sf[e]);
      if constexpr (RES != 0) {
        float x[VW];
        unpack<T>(d.r[u], x);
#pragma unroll
        for (int e = 0; e < VW; ++e) v[e] += RES == 1 ? x[e] : x[e] * sc2[e] + sf2[e];
      }
      if (relu) {
#pragma unroll
        for (int e = 0; e < VW; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
      }
      const uint4 pk = pack<T>(v);
      ((uint4*)z)[i] = pk;
      if (mbits) {
        // bit e: element e of the chunk as stored is > 0 (its ReLU mask)
        float vr[VW];
        unpack<T>(pk, vr);
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < VW; ++e) bits |= (vr[e] > 0.f ? 1u : 0u) << e;
        mbits[i] = (uint8_t)bits;
      }
    }
  };
  while (r0 < M) {
    process(r0, d);
    r0 += U * step;
    if (r0 < M) load(r0, d);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void bn_bwd_partial_kernel(const T* __restrict__ dz, const uint8_t* __restrict__ mb,
                                                             const T* __restrict__ y, const float* __restrict__ mean,
                                                             const float* __restrict__ rstd,
                                                             const float* __restrict__ mscale,
                                                             const float* __restrict__ mshift, long M, int C,
                                                             float* __restrict__ part) {
  constexpr int VW = TT<T>::VW;
  __shared__ float red[2][256 * VW];
  const int tpc = C / VW, rpi = 256 / tpc;
  const int tid = threadIdx.x, cg = tid % tpc, rr = tid / tpc;
  // the grid sweeps the rows together: at each step block b takes rows
  // (step * G + b) * rpi .. + rpi - 1, so the whole grid reads one contiguous
  // stretch of each tensor at a time
  const long gstride = (long)gridDim.x * rpi;
  float mu[VW], rs[VW], s1[VW], s2[VW], msc[VW], msf[VW];
#pragma unroll
  for (int e = 0; e < VW; ++e) {
    mu[e] = mean[cg * VW + e];
    rs[e] = rstd[cg * VW + e];
    msc[e] = mscale ? mscale[cg * VW + e] : 0.f;
    msf[e] = mscale ? mshift[cg * VW + e] : 0.f;
    s1[e] = s2[e] = 0.f;
  }
  // four rows per step, all loads issued before any is used (rows past the
  // end load the thread's first row of the step and add nothing)
  constexpr int U = 4;
  for (long r0 = (long)blockIdx.x * rpi + rr; r0 < M; r0 += U * gstride) {
    uint4 qg[U], qy[U];
    uint32_t qm[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long r = r0 + u * gstride < M ? r0 + u * gstride : r0;
      const long o = r * C + cg * VW;
      qg[u] = *(const uint4*)(dz + o);
      qy[u] = *(const uint4*)(y + o);
      if (mb) qm[u] = mb[r * tpc + cg];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool live_row = r0 + u * gstride < M;
      float g[VW], yy[VW];
      unpack<T>(qg[u], g);
      unpack<T>(qy[u], yy);
      if (mb) {
#pragma unroll
        for (int e = 0; e < VW; ++e) g[e] = (qm[u] >> e) & 1u ? g[e] : 0.f;
      } else if (mscale) {
        // the ReLU mask of relu(bn(y)), from the stored value's arithmetic
#pragma unroll
        for (int e = 0; e < VW; ++e) g[e] = relu_stored<T>(yy[e], msc[e], msf[e]) > 0.f ? g[e] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        const float gv = live_row ? g[e] : 0.f;
        s1[e] += gv;
        s2[e] += gv * ((yy[e] - mu[e]) * rs[e]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < VW; ++e) {
    red[0][rr * C + cg * VW + e] = s1[e];
    red[1][rr * C + cg * VW + e] = s2[e];
  }
  __syncthreads();
  for (int c = tid; c < C; c += 256) {
    float a = 0.f, b = 0.f;
    for (int q = 0; q < rpi; ++q) {
      a += red[0][q * C + c];
      b += red[1][q * C + c];
    }
    part[((long)blockIdx.x * C + c) * 2 + 0] = a;
    part[((long)blockIdx.x * C + c) * 2 + 1] = b;
  }
}

__global__ __launch_bounds__(256) void bn_bwd_final_kernel(const float* __restrict__ part, int nblk, long M, int C,
                                                           const float* gamma, const float* rstd, float* dgamma,
                                                           float* dbeta, float* coef) {
  __shared__ double sh[256];
  const int c = blockIdx.x;
  double a = 0.0, b = 0.0;
  for (int q = threadIdx.x; q < nblk; q += 256) {
    a += part[((long)q * C + c) * 2 + 0];
    b += part[((long)q * C + c) * 2 + 1];
  }
  a = block_sum_d(a, sh);
  b = block_sum_d(b, sh);
  if (threadIdx.x == 0) {
    dbeta[c] = (float)a;
    dgamma[c] = (float)b;
    const double rs = (double)rstd[c];
    const double k1 = (double)gamma[c] * rs;
    coef[3 * c + 0] = (float)k1;
    coef[3 * c + 1] = (float)(-k1 * rs * b / (double)M);
    coef[3 * c + 2] = (float)(-k1 * a / (double)M);
  }
}

// Coefficients of the backward apply for channels [c0, c0 + CG) into k1, k2,
// k3 (LDS): from coef when the finish kernel ran, else from the partials, added
// up by every block (see bn_coefs); the first block of a channel group stores
// dgamma and dbeta. All 256 threads; ends in a barrier.
__device__ inline void bn_bwd_coefs(const BnBwdSrc& b, int C, int c0, int CG, bool write, double (&sh)[3][4][kCG],
                                    float* k1, float* k2, float* k3) {
  const int cl = threadIdx.x & 63, q = threadIdx.x >> 6, c = c0 + cl;
  if (b.coef) {
    if (q == 0 && cl < CG) {
      k1[cl] = b.coef[3 * c];
      k2[cl] = b.coef[3 * c + 1];
      k3[cl] = b.coef[3 * c + 2];
    }
    __syncthreads();
    return;
  }
  double s1 = 0.0, s2 = 0.0;
  float ga = 0.f, rs1 = 0.f;
  if (cl < CG) {
    ga = b.gamma[c];
    rs1 = b.rstd[c];
#pragma unroll 8
    for (int z = q; z < b.n; z += 4) {
      const float2 p = ((const float2*)b.part)[(long)z * C + c];
      s1 += p.x;
      s2 += p.y;
    }
  }
  sh[0][q][cl] = s1; sh[1][q][cl] = s2;
  __syncthreads();
  if (q == 0 && cl < CG) {
    s1 = ((sh[0][0][cl] + sh[0][1][cl]) + sh[0][2][cl]) + sh[0][3][cl];
    s2 = ((sh[1][0][cl] + sh[1][1][cl]) + sh[1][2][cl]) + sh[1][3][cl];
    const double rs = (double)rs1, kk = (double)ga * rs;
    k1[cl] = (float)kk;
    k2[cl] = (float)(-kk * rs * s2 / (double)b.M);
    k3[cl] = (float)(-kk * s1 / (double)b.M);
    if (write) {
      b.dbeta[c] = (float)s1;
      b.dgamma[c] = (float)s2;
    }
  }
  __syncthreads();
}

// dy = k1 g + k2 (y - mean) + k3, g = dz where the ReLU passed: MASK 0 none, 1
// mask bytes, 2 recomputed from y. An HBM stream (3 tensors).
template <typename T, int MASK>
__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(const T* __restrict__ dz, const uint8_t* __restrict__ mb,
                                                           const T* __restrict__ y, const float* __restrict__ mean,
                                                           BnBwdSrc b, const float* __restrict__ mscale,
                                                           const float* __restrict__ mshift, T* __restrict__ dy,
                                                           long M, int C) {
  constexpr int VW = TT<T>::VW, U = kRowsU;
  __shared__ double sh[3][4][kCG];
  __shared__ float l1[kCG], l2[kCG], l3[kCG];
  const RowWalk w(C, VW);
  const long step = (long)w.nrb * w.rpi;
  struct Rows { uint4 g[U], y[U]; uint32_t m[U]; };
  auto at = [&](long row) { return (uint32_t)(row * w.cpr + w.cc); };
  auto load = [&](long r0, Rows& d) {   // (rows past the end load the last row)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = at(min(r0 + u * step, M - 1));
      d.g[u] = ((const uint4*)dz)[i];
      d.y[u] = ((const uint4*)y)[i];
      d.m[u] = MASK == 1 ? mb[i] : 0u;
    }
  };
  long r0 = (long)w.rb * w.rpi + w.rr;
  Rows d;
  load(r0, d);
  bn_bwd_coefs(b, C, w.c0, w.CG, w.rb == 0, sh, l1, l2, l3);
  const int c0 = w.cc * VW, cl = c0 - w.c0;
  float k1[VW], k2[VW], k3[VW], mu[VW], msc[VW], msf[VW];
#pragma unroll
  for (int e = 0; e < VW; ++e) {
    k1[e] = l1[cl + e];
    k2[e] = l2[cl + e];
    k3[e] = l3[cl + e];
    mu[e] = mean[c0 + e];
    msc[e] = MASK == 2 ? mscale[c0 + e] : 0.f;
    msf[e] = MASK == 2 ? mshift[c0 + e] : 0.f;
  }
  auto process = [&](long r0, const Rows& d) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r0 + u * step >= M) break;
      float g[VW], yy[VW], o[VW];
      unpack<T>(d.g[u], g);
      unpack<T>(d.y[u], yy);
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        if constexpr (MASK == 1) g[e] = (d.m[u] >> e) & 1u ? g[e] : 0.f;
        if constexpr (MASK == 2) g[e] = relu_stored<T>(yy[e], msc[e], msf[e]) > 0.f ? g[e] : 0.f;
        o[e] = k1[e] * g[e] + k2[e] * (yy[e] - mu[e]) + k3[e];
      }
      ((uint4*)dy)[at(r0 + u * step)] = pack<T>(o);
    }
  };
  while (r0 < M) {
    process(r0, d);
    r0 += U * step;
    if (r0 < M) load(r0, d);
  }
}

// ---------------------------------------------------------------- stem + max pool
// The stem's BN-apply + ReLU feeds only the 3x3 stride-2 max pool, so the
// forward pass goes from the conv output y straight to the pooled tensor and
// its argmax; the ReLU output itself is never stored. The backward pass reads
// the pooled gradient and the argmax and gathers the gradient of each stem
// pixel on the fly (rounded to the storage type, as a stored tensor would be),
// with the ReLU mask recomputed from y by the same arithmetic.

template <typename T>
__global__ __launch_bounds__(256) void bn_apply_pool_kernel(const T* __restrict__ y, BnSrc b, T* __restrict__ pool,
                                                            uint8_t* __restrict__ arg, int N, int H, int W, int C,
                                                            int Ho, int Wo) {
  constexpr int VW = TT<T>::VW;
  __shared__ double sh[3][4][kCG];
  __shared__ float sc[kMaxC], sf[kMaxC];
  for (int c0 = 0; c0 < C; c0 += kCG) bn_coefs(b, C, c0, min(kCG, C - c0), blockIdx.x == 0, sh, sc + c0, sf + c0);
  const int cpr = C / VW;
  const int total = N * Ho * Wo * cpr;
  for (int q = blockIdx.x * 256 + threadIdx.x; q < total; q += gridDim.x * 256) {
    const int pix = q / cpr, cc = q - pix * cpr;
    const int t2 = pix / Wo, j = pix - t2 * Wo;
    const int n = t2 / Ho, i = t2 - n * Ho;
    const int c0 = cc * VW;
    auto act = [&](float* v) {
#pragma unroll
      for (int e = 0; e < VW; ++e) v[e] = relu_stored<T>(v[e], sc[c0 + e], sf[c0 + e]);
    };
    float best[VW];
    uint8_t bi[VW];
    pool_max_window<T>(y, n, i, j, cc, H, W, C, act, best, bi);
    ((uint4*)pool)[q] = pack<T>(best);
    ArgVec<VW>::store(arg + (long)q * VW, bi);
  }
}

// Masked stem gradients of the pixels of quad (n, qi, qj), chunk cg: g[p][]
// (0 for pixels past the edge) and y[p][], p = 2*py + px.
template <typename T>
__device__ inline void stem_grad_quad(const T* __restrict__ dpool, const uint8_t* __restrict__ arg,
                                      const T* __restrict__ y, const float* sc, const float* sf, int n, int qi, int qj,
                                      int cg, int cpr, int H, int W, int Ho, int Wo, float (*g)[TT<T>::VW],
                                      float (*yy)[TT<T>::VW]) {
  constexpr int VW = TT<T>::VW;
  pool_grad_quad<T>(dpool, arg, n, qi, qj, cg, cpr, Ho, Wo, g);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int h = 2 * qi + (p >> 1), w = 2 * qj + (p & 1);
    unpack<T>(((const uint4*)y)[((n * H + min(h, H - 1)) * W + min(w, W - 1)) * cpr + cg], yy[p]);
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int h = 2 * qi + (p >> 1), w = 2 * qj + (p & 1);
    const bool in = h < H && w < W;
#pragma unroll
    for (int e = 0; e < VW; ++e) {
      const float gr = TT<T>::to_f(TT<T>::from_f(g[p][e]));
      const bool live = in && relu_stored<T>(yy[p][e], sc[cg * VW + e], sf[cg * VW + e]) > 0.f;
      g[p][e] = live ? gr : 0.f;
      yy[p][e] = in ? yy[p][e] : 0.f;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void bn_bwd_partial_pool_kernel(const T* __restrict__ dpool,
                                                                  const uint8_t* __restrict__ arg,
                                                                  const T* __restrict__ y,
                                                                  const float* __restrict__ scale,
                                                                  const float* __restrict__ shift,
                                                                  const float* __restrict__ mean,
                                                                  const float* __restrict__ rstd, int N, int H, int W,
                                                                  int C, int Ho, int Wo, float* __restrict__ part) {
  constexpr int VW = TT<T>::VW;
  __shared__ float red[2][256 * VW];
  __shared__ float sc[kMaxC], sf[kMaxC];
  for (int c = threadIdx.x; c < C; c += 256) { sc[c] = scale[c]; sf[c] = shift[c]; }
  __syncthreads();
  const int Hq = (H + 1) / 2, Wq = (W + 1) / 2;
  const int Mq = N * Hq * Wq;
  const int tpc = C / VW, rpi = 256 / tpc;
  const int tid = threadIdx.x, cg = tid % tpc, rr = tid / tpc;
  const int per_blk = (Mq + gridDim.x - 1) / gridDim.x;
  const int q_begin = blockIdx.x * per_blk;
  const int q_end = min(Mq, q_begin + per_blk);
  float mu[VW], rs[VW], s1[VW], s2[VW];
#pragma unroll
  for (int e = 0; e < VW; ++e) {
    mu[e] = mean[cg * VW + e];
    rs[e] = rstd[cg * VW + e];
    s1[e] = s2[e] = 0.f;
  }
  for (int q = q_begin + rr; q < q_end; q += rpi) {
    const int t2 = q / Wq, qj = q - t2 * Wq;
    const int n = t2 / Hq, qi = t2 - n * Hq;
    float g[4][VW], yy[4][VW];
    stem_grad_quad<T>(dpool, arg, y, sc, sf, n, qi, qj, cg, tpc, H, W, Ho, Wo, g, yy);
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int e = 0; e < VW; ++e) {
        s1[e] += g[p][e];
        s2[e] += g[p][e] * ((yy[p][e] - mu[e]) * rs[e]);
      }
  }
#pragma unroll
  for (int e = 0; e < VW; ++e) {
    red[0][rr * C + cg * VW + e] = s1[e];
    red[1][rr * C + cg * VW + e] = s2[e];
  }
  __syncthreads();
  for (int c = tid; c < C; c += 256) {
    float a = 0.f, b = 0.f;
    for (int q = 0; q < rpi; ++q) {
      a += red[0][q * C + c];
      b += red[1][q * C + c];
    }
    part[((long)blockIdx.x * C + c) * 2 + 0] = a;
    part[((long)blockIdx.x * C + c) * 2 + 1] = b;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void bn_bwd_apply_pool_kernel(const T* __restrict__ dpool,
                                                                const uint8_t* __restrict__ arg,
                                                                const T* __restrict__ y,
                                                                const float* __restrict__ scale,
                                                                const float* __restrict__ shift,
                                                                const float* __restrict__ mean,
                                                                const float* __restrict__ coef, T* __restrict__ dy,
                                                                int N, int H, int W, int C, int Ho, int Wo) {
  constexpr int VW = TT<T>::VW;
  __shared__ float k1[kMaxC], k2[kMaxC], k3[kMaxC], mu[kMaxC], sc[kMaxC], sf[kMaxC];
  for (int c = threadIdx.x; c < C; c += 256) {
    k1[c] = coef[3 * c];
    k2[c] = coef[3 * c + 1];
    k3[c] = coef[3 * c + 2];
    mu[c] = mean[c];
    sc[c] = scale[c];
    sf[c] = shift[c];
  }
  __syncthreads();
  const int cpr = C / VW;
  const int Hq = (H + 1) / 2, Wq = (W + 1) / 2;
  const int nq = N * Hq * Wq * cpr;
  for (int q = blockIdx.x * 256 + threadIdx.x; q < nq; q += gridDim.x * 256) {
    const int quad = q / cpr, cg = q - quad * cpr;
    const int t2 = quad / Wq, qj = quad - t2 * Wq;
    const int n = t2 / Hq, qi = t2 - n * Hq;
    const int c0 = cg * VW;
    float g[4][VW], yy[4][VW];
    stem_grad_quad<T>(dpool, arg, y, sc, sf, n, qi, qj, cg, cpr, H, W, Ho, Wo, g, yy);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int h = 2 * qi + (p >> 1), w = 2 * qj + (p & 1);
      if (h >= H || w >= W) continue;
      float o[VW];
#pragma unroll
      for (int e = 0; e < VW; ++e) o[e] = k1[c0 + e] * g[p][e] + k2[c0 + e] * (yy[p][e] - mu[c0 + e]) + k3[c0 + e];
      ((uint4*)dy)[((n * H + h) * W + w) * cpr + cg] = pack<T>(o);
    }
  }
}

int stream_blocks(long nchunks) {
  long b = (nchunks + 255) / 256;
  if (b > 8192) b = 8192;
  if (b < 1) b = 1;
  return (int)b;
}

inline int ok() { return hipGetLastError() == hipSuccess ? 0 : -4; }

}  // namespace

namespace {
// Blocks of an applying pass: at most 8 per CU (each adds up its channels'
// partials first), four rows per thread and step. Alone, large tensors are
// slower than with one row per thread, 32 blocks per CU and coefficients that a
// launch of their own finished (802816 x 64 in bf16: 48 us against 42, with a
// residual 69 and 60, backward 68 and 60), but whole training steps are not:
// batch 256 at 224x224 5.93 ms both, fp16 batch 96 at 160x160 2.227 against 2.235.
int row_blocks(int prec, long M, int C) {
  const int CG = C < kCG ? C : kCG, groups = C / CG, rpi = 256 / (CG / prec_vw(prec)), cus = plan_cus();
  long b = (M + (long)rpi * kRowsU - 1) / ((long)rpi * kRowsU);
  if (b * groups < 2 * cus) {
    // small tensors: fewer rows per thread, up to two blocks per CU
    const long b1 = (M + rpi - 1) / rpi, lim = 2 * cus / groups;
    b = b1 < lim ? b1 : lim;
  }
  const long cap = 8 * cus / groups;
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return (int)b * groups;
}
bool row_shape_ok(int prec, long M, int C) {
  const int vw = prec_vw(prec), CG = C < kCG ? C : kCG;
  return C % vw == 0 && C % CG == 0 && 256 % (CG / vw) == 0 && M * (C / vw) < (1l << 31);
}
}  // namespace

int bn_apply_launch(int prec, const void* y, const BnSrc& b, int relu, int res_mode, const void* r, const BnSrc& b2,
                    void* z, long M, int C, hipStream_t s, uint8_t* mbits) {
  if (!row_shape_ok(prec, M, C)) return -1;
  const dim3 grid(row_blocks(prec, M, C)), block(256);
  return with_prec(prec, [&](auto tag) {
    using T = decltype(tag);
    if (res_mode == 0)
      hipLaunchKernelGGL((bn_apply_kernel<T, 0>), grid, block, 0, s, (const T*)y, b, relu, (const T*)r, b2, (T*)z, M, C,
                         mbits);
    else if (res_mode == 1)
      hipLaunchKernelGGL((bn_apply_kernel<T, 1>), grid, block, 0, s, (const T*)y, b, relu, (const T*)r, b2, (T*)z, M, C,
                         mbits);
    else
      hipLaunchKernelGGL((bn_apply_kernel<T, 2>), grid, block, 0, s, (const T*)y, b, relu, (const T*)r, b2, (T*)z, M, C,
                         mbits);
    return ok();
  });
}

int bn_bwd_partial_blocks(int prec, long M, int C) {
  return pick_blocks(M, 256 / (C / prec_vw(prec)), 16, 512, 256);
}

int bn_bwd_partial_pool_blocks(int prec, int N, int H, int W, int C) {
  const int rpi = 256 / (C / prec_vw(prec));
  return pick_blocks((long)N * ((H + 1) / 2) * ((W + 1) / 2), rpi, 8, 1024, 0);
}

int bn_bwd_partial_launch(int prec, const void* dz, const uint8_t* mb, const void* y, const float* mean,
                          const float* rstd, long M, int C, float* part, int* nblk, hipStream_t s,
                          const float* mscale, const float* mshift) {
  const int nb = bn_bwd_partial_blocks(prec, M, C);
  *nblk = nb;
  return with_prec(prec, [&](auto tag) {
    using T = decltype(tag);
    hipLaunchKernelGGL(bn_bwd_partial_kernel<T>, dim3(nb), dim3(256), 0, s, (const T*)dz, mb, (const T*)y, mean, rstd,
                       mscale, mshift, M, C, part);
    return ok();
  });
}

int bn_bwd_final_launch(const float* part, int nblk, long M, int C, const float* gamma, const float* rstd,
                        float* dgamma, float* dbeta, float* coef, hipStream_t s) {
  hipLaunchKernelGGL(bn_bwd_final_kernel, dim3(C), dim3(256), 0, s, part, nblk, M, C, gamma, rstd, dgamma, dbeta,
                     coef);
  return ok();
}

int bn_bwd_apply_launch(int prec, const void* dz, const uint8_t* mb, const void* y, const float* mean,
                        const BnBwdSrc& b, void* dy, long M, int C, hipStream_t s, const float* mscale,
                        const float* mshift, hipEvent_t done) {
  if (!row_shape_ok(prec, M, C)) return -1;
  const dim3 grid(row_blocks(prec, M, C)), block(256);
  return with_prec(prec, [&](auto tag) {
    using T = decltype(tag);
    auto launch = [&](auto kernel) {
      // (with done, the event completes with this kernel: no separate marker on the queue)
      if (done)
        hipExtLaunchKernelGGL(kernel, grid, block, 0, s, nullptr, done, 0, (const T*)dz, mb, (const T*)y, mean, b,
                              mscale, mshift, (T*)dy, M, C);
      else
        hipLaunchKernelGGL(kernel, grid, block, 0, s, (const T*)dz, mb, (const T*)y, mean, b, mscale, mshift, (T*)dy, M,
                           C);
    };
    if (mb) launch(bn_bwd_apply_kernel<T, 1>);
    else if (mscale) launch(bn_bwd_apply_kernel<T, 2>);
    else launch(bn_bwd_apply_kernel<T, 0>);
    return ok();
  });
}

int bn_apply_pool_launch(int prec, const void* y, const BnSrc& b, void* pool, uint8_t* arg, int N, int H, int W, int C,
                         int Ho, int Wo, hipStream_t s) {
  const int vw = prec_vw(prec);
  if (C > kMaxC || (long)N * H * W * (C / vw) >= (1l << 31)) return -1;  // 32-bit chunk indices
  const long total = (long)N * Ho * Wo * (C / vw);
  const int blocks = std::min(stream_blocks(total), 8 * plan_cus());   // (see row_blocks)
  return with_prec(prec, [&](auto tag) {
    using T = decltype(tag);
    hipLaunchKernelGGL(bn_apply_pool_kernel<T>, dim3(blocks), dim3(256), 0, s, (const T*)y, b, (T*)pool, arg, N, H, W,
                       C, Ho, Wo);
    return ok();
  });
}

int bn_bwd_partial_pool_launch(int prec, const void* dpool, const uint8_t* arg, const void* y, const float* scale,
                               const float* shift, const float* mean, const float* rstd, int N, int H, int W, int C,
                               int Ho, int Wo, float* part, int* nblk, hipStream_t s) {
  const int vw = prec_vw(prec);
  if (C > kMaxC || (long)N * H * W * (C / vw) >= (1l << 31)) return -1;  // 32-bit chunk indices
  const int nb = bn_bwd_partial_pool_blocks(prec, N, H, W, C);
  *nblk = nb;
  return with_prec(prec, [&](auto tag) {
    using T = decltype(tag);
    hipLaunchKernelGGL(bn_bwd_partial_pool_kernel<T>, dim3(nb), dim3(256), 0, s, (const T*)dpool, arg, (const T*)y,
                       scale, shift, mean, rstd, N, H, W, C, Ho, Wo, part);
    return ok();
  });
}

int bn_bwd_apply_pool_launch(int prec, const void* dpool, const uint8_t* arg, const void* y, const float* scale,
                             const float* shift, const float* mean, const float* coef, void* dy, int N, int H, int W,
                             int C, int Ho, int Wo, hipStream_t s) {
  const int vw = prec_vw(prec);
  if (C > kMaxC || (long)N * H * W * (C / vw) >= (1l << 31)) return -1;  // 32-bit chunk indices
  const long nchunks = (long)N * ((H + 1) / 2) * ((W + 1) / 2) * (C / vw);
  return with_prec(prec, [&](auto tag) {
    using T = decltype(tag);
    hipLaunchKernelGGL(bn_bwd_apply_pool_kernel<T>, dim3(stream_blocks(nchunks)), dim3(256), 0, s, (const T*)dpool,
                       arg, (const T*)y, scale, shift, mean, coef, (T*)dy, N, H, W, C, Ho, Wo);
    return ok();
  });
}

int bn_stats_tiles_chunks(int ntiles) {
  const int r = (ntiles + 63) / 64;
  return r < 1 ? 1 : r > 16 ? 16 : r;
}

int bn_stats_source(const float* tile_stats, int ntiles, int C, double* scratch, BnSrc* b, hipStream_t s) {
  const int chunks = bn_stats_tiles_chunks(ntiles);
  b->st = tile_stats;
  if (chunks == 1) {
    b->kind = BnSrc::TILES;
    b->n = ntiles;
    return 0;
  }
  b->kind = BnSrc::CHUNKS;
  b->red = scratch;
  b->n = chunks;
  hipLaunchKernelGGL(bn_stats_tiles_reduce_kernel, dim3((C + 63) / 64, chunks), dim3(256), 0, s, tile_stats, ntiles,
                     C, (ntiles + chunks - 1) / chunks, scratch);
  return ok();
}

}  // namespace rn18
