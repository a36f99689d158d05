// Colour likelihood of the t-links (Section 4: psi_1 = -log p(C | A) with p(C | A) a
// Gaussian mixture over RGB fitted by EM; Section 5: every pixel is a sample, weighted by
// the prior p(A = 1) for the object and by 1 - p for the background; Section 8.1: M = 3).
//
// Per label and iteration: one pass over tiles of io.tile pixels takes the E-step under
// the current mixtures (read as scalars) and accumulates, for every component, the
// responsibility-weighted count and the first and second moments about the component's
// mean (FP32 per thread, FP64 from the workgroup sum on, one partial per workgroup).  The
// partials are reduced in a fixed order and the new weights, means and covariances, their
// inverses and log-normalisers fitted in FP64, one thread per label and component: by every
// workgroup of the next pass for itself up to gmm_fuse tiles, by one workgroup in a launch
// between the passes above.  The start is the weighted mean and covariance of each label's samples with
// the means spread along the covariance's leading eigenvector.  A final pass adds psi_1 of
// both labels to the unary costs.
// The pixel passes read 7 bytes per pixel.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>

#include <algorithm>

#include "sp_internal.h"
#include "sp_kernels.h"
#include "sp_device.h"

namespace {

// Threads of a pixel pass: the first four wavefronts take the object's complement (label 0), the
// last four the object (label 1), each over all pixels of the tile: half the values and half the
// chain of one thread for both, and two wavefronts on a SIMD instead of one.
constexpr int GB = 2 * SP_BLOCK;
constexpr int GPX = SP_GMM_GPX;   // most pixels per thread of a tile
constexpr float kInv255 = 1.f / 255.f;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr double kLog2Pi = 1.8378770664093453;

__device__ __forceinline__ float ex(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }
__device__ __forceinline__ float lg(float x) { return __builtin_amdgcn_logf(x) * kLn2; }

// Products of a difference (xx, xy, xz, yy, yz, zz).
struct Prod {
  float v[6];
  __device__ __forceinline__ Prod(float dx, float dy, float dz)
      : v{dx * dx, dx * dy, dx * dz, dy * dy, dy * dz, dz * dz} {}
};

// Squared Mahalanobis distance d' P d with P stored as (xx, xy, xz, yy, yz, zz).
__device__ __forceinline__ float quad(const float* P, const Prod& d) {
  const float a = P[0] * d.v[0] + P[3] * d.v[3] + P[5] * d.v[5];
  const float b = P[1] * d.v[1] + P[2] * d.v[2] + P[4] * d.v[4];
  return fmaf(2.f, b, a);
}

// Moments of one sample with weight wr about the centre: count, first (3) and second (6).  Both orders
// take the rounded product of weight and difference: its rounding varies with the weight and averages
// out, where that of a product of differences is the same for all samples of one colour (a plain frame's
// covariance came out 1e-9 off).
__device__ __forceinline__ void add_moments(float* a, float wr, float dx, float dy, float dz) {
  const float ux = wr * dx, uy = wr * dy, uz = wr * dz;
  a[0] += wr;
  a[1] += ux;
  a[2] += uy;
  a[3] += uz;
  a[4] = fmaf(ux, dx, a[4]);
  a[5] = fmaf(ux, dy, a[5]);
  a[6] = fmaf(ux, dz, a[6]);
  a[7] = fmaf(uy, dy, a[7]);
  a[8] = fmaf(uy, dz, a[8]);
  a[9] = fmaf(uz, dz, a[9]);
}

// A label's mixture as the pixel loops use it, in scalar registers (read from LDS once).
__device__ __forceinline__ float uni(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }
template <int NC>
struct Mix {
  float mu[NC][3], P[NC][6], ln[NC];
  bool on[NC], lab;
  __device__ __forceinline__ void load(const GmmState& S, int L) {
    lab = __builtin_amdgcn_readfirstlane(S.label_on[L]) != 0;
#pragma unroll
    for (int m = 0; m < NC; ++m) {
      const GmmComp& g = S.comp[L][m];
      on[m] = __builtin_amdgcn_readfirstlane(g.on) != 0;
#pragma unroll
      for (int i = 0; i < 3; ++i) mu[m][i] = uni(g.mu[i]);
#pragma unroll
      for (int i = 0; i < 6; ++i) P[m][i] = uni(g.P[i]);
      ln[m] = uni(g.lnorm);
    }
  }
  // log(alpha_m N(c; mu_m, Sigma_m)) of component m, -inf for a dropped one
  __device__ __forceinline__ float logp(int m, const Prod& d) const {
    return on[m] ? ln[m] - 0.5f * quad(P[m], d) : -INFINITY;
  }
};

// The label of the wavefront and the thread's place among its four wavefronts.
__device__ __forceinline__ int label_of() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x / SP_BLOCK); }
__device__ __forceinline__ uint32_t slot_of() { return threadIdx.x % SP_BLOCK; }

// The workgroup's pixels in LDS: colour in [0, 1] and the prior, loaded once for both labels, all
// loads in flight together.  The pixel loops below are rolled: unrolled over a thread's pixels they
// take more registers and are no faster (9.0 against 8.2 us a pass at 640x480).
template <bool PRIOR>
struct Staged {
  uint32_t c[GPX / 2][3];
  float pi[GPX / 2];
  __device__ __forceinline__ void load(const GmmIO& io) {
    const gp<const uint8_t> rgb = G(io.rgb);
#pragma unroll
    for (int k = 0; k < GPX / 2; ++k) {
      if (k * GB >= io.tile) continue;   // uniform
      // past the end: not used
      const uint32_t i = min((uint32_t)(blockIdx.x * io.tile + k * GB) + threadIdx.x, (uint32_t)io.n - 1u);
      c[k][0] = rgb[3 * i];
      c[k][1] = rgb[3 * i + 1];
      c[k][2] = rgb[3 * i + 2];
      pi[k] = PRIOR ? G(io.prior)[i] : 0.f;
    }
  }
  __device__ __forceinline__ void put(const GmmIO& io, float4* px) const {
#pragma unroll
    for (int k = 0; k < GPX / 2; ++k)
      if (k * GB + (int)threadIdx.x < io.tile)
        px[k * GB + threadIdx.x] =
            make_float4((float)c[k][0] * kInv255, (float)c[k][1] * kInv255, (float)c[k][2] * kInv255, pi[k]);
  }
};

// LDS of a moment pass: the pixels, then the threads' sums.
constexpr int seg_of(int nv) { return GB / nv >= 8 ? 8 : (GB / nv >= 4 ? 4 : 2); }
template <int NC>
constexpr int LDS_N = 20 * NC * (SP_BLOCK + 2 * seg_of(20 * NC)) > 4 * GPX * SP_BLOCK ? 20 * NC * (SP_BLOCK + 2 * seg_of(20 * NC))
                                                                                     : 4 * GPX * SP_BLOCK;

// Moments of the tile into the partial slot of the workgroup.  EM = false: the start's
// moments of both labels about (0.5, 0.5, 0.5); EM = true: the E-step under the mixtures S
// and the moments of every component about its mean.  Each thread accumulates up to FP32_N of
// its pixels in FP32; the workgroup sum goes through LDS transposed: value v's thread sums are
// split into SEG interleaved segments, each summed in FP64 by one thread with four accumulators
// in a fixed order, and the segments are added in order.  A thread with more pixels has a second
// FP32 sum, which joins the first, and both the neighbouring thread's, in FP64, so half as many sums
// take the same LDS (640x480, three components, ten steps: 117 us with one FP32 sum of all pixels,
// 127 us so).
constexpr int FP32_N = 4;
static_assert(GPX <= 2 * FP32_N, "two FP32 sums per thread");
template <int M, bool EM>
__device__ __forceinline__ void tile_moments(const GmmIO& io, float* lds, const GmmState& S) {
  constexpr int NC = EM ? M : 1;
  constexpr int NV = 2 * NC * 10;
  constexpr int SEG = seg_of(NV);
  constexpr int TRW = SP_BLOCK + SEG;   // a wavefront reads 64 / SEG rows: no bank twice
  constexpr int TRD = SP_BLOCK / 2 + SEG;   // the same in doubles
  const float4* const px = reinterpret_cast<const float4*>(lds);
  float* const tr = lds;                // [NV][TRW], in the pixels' place
  __shared__ double segs[NV][SEG];
  const int L = label_of();
  float acc[NC][10];
  Mix<NC> X;
  if (EM) X.load(S, L);
  const int end = min(io.tile, io.n - (int)blockIdx.x * io.tile);
  const bool two = io.tile > FP32_N * SP_BLOCK;   // uniform over the launch
  // FP32 sums of the thread's pixels from tile position `from` on
  auto take = [&](int from, int to) {
#pragma unroll
    for (int m = 0; m < NC; ++m)
#pragma unroll
      for (int v = 0; v < 10; ++v) acc[m][v] = 0.f;
#pragma unroll 1
    for (int t = from + slot_of(); t < to; t += SP_BLOCK) {
      const float4 p = px[t];
      const float w = L ? p.w : 1.f - p.w;
      if constexpr (!EM) {
        const float dx = p.x - 0.5f, dy = p.y - 0.5f, dz = p.z - 0.5f;
        add_moments(acc[0], w, dx, dy, dz);
      } else {
        if (!X.lab) break;
        if constexpr (NC == 1) {   // its responsibility is 1: nothing to evaluate (1920x1080 212 -> 195 us)
          if (X.on[0]) {
            const float dx = p.x - X.mu[0][0], dy = p.y - X.mu[0][1], dz = p.z - X.mu[0][2];
            add_moments(acc[0], w, dx, dy, dz);
          }
          continue;
        }
        float lp[NC], mx = -INFINITY;
#pragma unroll
        for (int m = 0; m < NC; ++m) {
          lp[m] = X.logp(m, Prod(p.x - X.mu[m][0], p.y - X.mu[m][1], p.z - X.mu[m][2]));
          mx = fmaxf(mx, lp[m]);
        }
        float r[NC], sum = 0.f;
#pragma unroll
        for (int m = 0; m < NC; ++m) {
          r[m] = X.on[m] ? ex(lp[m] - mx) : 0.f;
          sum += r[m];
        }
        const float ws = w / sum;
#pragma unroll
        for (int m = 0; m < NC; ++m)
          if (X.on[m]) {
            const float dx = p.x - X.mu[m][0], dy = p.y - X.mu[m][1], dz = p.z - X.mu[m][2];
            add_moments(acc[m], ws * r[m], dx, dy, dz);
          }
      }
    }
  };
  take(0, min(end, FP32_N * SP_BLOCK));
  // the segment sums of rows of n thread sums, ld apart
  auto segments = [&](const auto* rows, int n, int ld) {
    if ((int)threadIdx.x < NV * SEG) {
      const int v = threadIdx.x / SEG, sg = threadIdx.x % SEG;
      const auto* row = rows + v * ld + sg;
      double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
      for (int j = 0; j < n / SEG; j += 4)
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] += (double)row[(j + i) * SEG];
      segs[v][sg] = (a[0] + a[1]) + (a[2] + a[3]);
    }
  };
  if (two) {
    float early[NC][10];
#pragma unroll
    for (int m = 0; m < NC; ++m)
#pragma unroll
      for (int v = 0; v < 10; ++v) early[m][v] = acc[m][v];
    take(FP32_N * SP_BLOCK, end);
    __syncthreads();
    double* const td = reinterpret_cast<double*>(lds);
    const int odd = slot_of() & 1u;
    double* const col = td + (L * NC * 10 + odd) * TRD + (slot_of() >> 1);
#pragma unroll
    for (int m = 0; m < NC; ++m)
#pragma unroll
      for (int v = 0; v < 10; v += 2) {   // the pair's even thread stores value v, the odd one v + 1
        double a = (double)early[m][v] + (double)acc[m][v], b = (double)early[m][v + 1] + (double)acc[m][v + 1];
        a += dpp_d<0xB1>(a);
        b += dpp_d<0xB1>(b);
        col[(m * 10 + v) * TRD] = odd ? b : a;
      }
    __syncthreads();
    segments(td, SP_BLOCK / 2, TRD);
  } else {
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NC; ++m)
#pragma unroll
      for (int v = 0; v < 10; ++v) tr[((L * NC + m) * 10 + v) * TRW + slot_of()] = acc[m][v];
    __syncthreads();
    segments(tr, SP_BLOCK, TRW);
  }
  __syncthreads();
  if ((int)threadIdx.x < NV) {
    double t = 0.0;
#pragma unroll
    for (int sg = 0; sg < SEG; ++sg) t += segs[threadIdx.x][sg];
    io.part_out[(size_t)blockIdx.x * NV + threadIdx.x] = t;
  }
}

// Symmetric 3x3 (xx, xy, xz, yy, yz, zz): determinant and inverse by cofactors.
__device__ __forceinline__ double sym_inverse(const double* A, double* I) {
  const double c00 = A[3] * A[5] - A[4] * A[4], c01 = A[2] * A[4] - A[1] * A[5], c02 = A[1] * A[4] - A[2] * A[3];
  const double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
  const double id = 1.0 / det;
  I[0] = c00 * id;
  I[1] = c01 * id;
  I[2] = c02 * id;
  I[3] = (A[0] * A[5] - A[2] * A[2]) * id;
  I[4] = (A[1] * A[2] - A[0] * A[4]) * id;
  I[5] = (A[0] * A[3] - A[1] * A[1]) * id;
  return det;
}

// Positive definite by its leading principal minors.
__device__ __forceinline__ bool sym_pd(const double* A) {
  const double m2 = A[0] * A[3] - A[1] * A[1];
  const double det = A[0] * (A[3] * A[5] - A[4] * A[4]) - A[1] * (A[1] * A[5] - A[4] * A[2]) +
                     A[2] * (A[1] * A[4] - A[3] * A[2]);
  return A[0] > 0.0 && m2 > 0.0 && det > 0.0 && isfinite(det);
}

// The E-step forms of the components flagged in live, from S.alpha, S.mu and S.cov, by threads
// q = L * M + m; the logarithms of the weights and of the determinants side by side.
template <int M>
__device__ __forceinline__ void set_comps(GmmState& S, bool live) {
  __shared__ double lg2[2][2 * M];
  const int q = threadIdx.x, L = q / M, m = q % M;
  if (q < 2 * M && live) {
    GmmComp& g = S.comp[L][m];
    double P[6];
    lg2[0][q] = S.alpha[L][m];
    lg2[1][q] = sym_inverse(S.cov[L][m], P);
    for (int i = 0; i < 3; ++i) g.mu[i] = (float)S.mu[L][m][i];
    for (int i = 0; i < 6; ++i) g.P[i] = (float)P[i];
  }
  __syncthreads();
  if (q < 4 * M) (&lg2[0][0])[q] = log((&lg2[0][0])[q]);   // unused values included
  __syncthreads();
  if (q < 2 * M && live) {
    S.comp[L][m].lnorm = (float)(lg2[0][q] - 0.5 * lg2[1][q] - 1.5 * kLog2Pi);
    S.comp[L][m].on = 1;
  }
  __syncthreads();
}

// The partial moments of every tile reduced in a fixed order.  A wavefront's load takes the values of
// TPL tiles, consecutive in memory, TB loads in flight: lane l of wavefront w sums value l % NV of
// every (8 TPL)-th tile from w TPL + l / NV on; then these sums are added in order.
template <int NV>
__device__ __forceinline__ void reduce_parts(const double* __restrict__ part, int ntiles, double* sums) {
  constexpr int NW = GB / 64, TB = 20, TPL = NV <= 64 ? 64 / NV : 1;
  __shared__ double ws[NW * TPL][NV];
  const int w = __builtin_amdgcn_readfirstlane(wave_id());
  const gp<const double> pp = G(part);
#pragma unroll 1
  for (int v0 = 0; v0 < NV; v0 += 64) {
    const int l = v0 + lane_id();
    double acc = 0.0;
#pragma unroll 1
    for (int t0 = w * TPL; t0 < ntiles; t0 += NW * TPL * TB) {
      double x[TB];
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        const int t = t0 + NW * TPL * u;
        if constexpr (TPL == 1)   // clamped and masked by scalars
          x[u] = *at_bytes(pp + (size_t)min(t, ntiles - 1) * NV, 8u * (uint32_t)min(l, NV - 1));
        else
          x[u] = *at_bytes(pp, 8u * (uint32_t)min(t * NV + l, ntiles * NV - 1));
      }
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        const int t = t0 + NW * TPL * u;
        acc += (TPL == 1 ? t < ntiles : t * NV + l < ntiles * NV) ? x[u] : 0.0;
      }
    }
    if (l < TPL * NV) (&ws[w * TPL][0])[l] = acc;
  }
  __syncthreads();
  if ((int)threadIdx.x < NV) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < NW * TPL; ++k) t += ws[k][threadIdx.x];
    sums[threadIdx.x] = t;
  }
}

// The start: the mixtures of both labels from the reduced moments, into S (LDS), by threads
// q = L * M + m: per label the weighted mean and covariance, the leading eigenvector by 64 power
// steps from (1, 1, 1) / sqrt 3, means spread along it.
template <int M>
__device__ __forceinline__ void fit_start(const double* sums, GmmState& S, float reg, int n) {
  __shared__ double ax[2][12];   // per label d (3), S (6), v (3) after the power steps
  __shared__ double lam_s[2];
  const int q = threadIdx.x;
  if (q < 2) {
    const int L = q;
    const double* a = sums + L * 10;
    const double W0 = a[0];
    S.label_on[L] = W0 > 1e-12 * (double)n ? 1 : 0;
    if (S.label_on[L]) {
      const double d[3] = {a[1] / W0, a[2] / W0, a[3] / W0};
      const double C[6] = {a[4] / W0 - d[0] * d[0], a[5] / W0 - d[0] * d[1], a[6] / W0 - d[0] * d[2],
                           a[7] / W0 - d[1] * d[1], a[8] / W0 - d[1] * d[2], a[9] / W0 - d[2] * d[2]};
      // 64 normalised power steps from v0 = (1, 1, 1) / sqrt 3 give C^64 v0 / |C^64 v0|: C^64
      // by six squarings (each scaled by its largest entry), then one product.  For a
      // symmetric C, C v0 = 0 is the only way the steps stop early, and then v stays v0.
      double A[6] = {C[0], C[1], C[2], C[3], C[4], C[5]};
      for (int it = 0; it < 6; ++it) {
        const double B[6] = {A[0] * A[0] + A[1] * A[1] + A[2] * A[2], A[0] * A[1] + A[1] * A[3] + A[2] * A[4],
                             A[0] * A[2] + A[1] * A[4] + A[2] * A[5], A[1] * A[1] + A[3] * A[3] + A[4] * A[4],
                             A[1] * A[2] + A[3] * A[4] + A[4] * A[5], A[2] * A[2] + A[4] * A[4] + A[5] * A[5]};
        double big = 0.0;
        for (int i = 0; i < 6; ++i) big = fmax(big, fabs(B[i]));
        const double sc = big > 0.0 ? 1.0 / big : 0.0;
        for (int i = 0; i < 6; ++i) A[i] = B[i] * sc;
      }
      double v[3] = {0.5773502691896258, 0.5773502691896258, 0.5773502691896258};
      {
        const double u0 = (A[0] * v[0] + A[1] * v[1] + A[2] * v[2]);
        const double u1 = (A[1] * v[0] + A[3] * v[1] + A[4] * v[2]);
        const double u2 = (A[2] * v[0] + A[4] * v[1] + A[5] * v[2]);
        const double nn = sqrt(u0 * u0 + u1 * u1 + u2 * u2);
        const bool moves = (C[0] * v[0] + C[1] * v[1] + C[2] * v[2]) != 0.0 || (C[1] * v[0] + C[3] * v[1] + C[4] * v[2]) != 0.0 ||
                           (C[2] * v[0] + C[4] * v[1] + C[5] * v[2]) != 0.0;
        if (moves && nn > 0.0) {
          v[0] = u0 / nn;
          v[1] = u1 / nn;
          v[2] = u2 / nn;
        }
      }
      int k = 0;
      for (int i = 1; i < 3; ++i)
        if (fabs(v[i]) > fabs(v[k])) k = i;
      if (v[k] < 0) v[0] = -v[0], v[1] = -v[1], v[2] = -v[2];
      const double Sv0 = C[0] * v[0] + C[1] * v[1] + C[2] * v[2];
      const double Sv1 = C[1] * v[0] + C[3] * v[1] + C[4] * v[2];
      const double Sv2 = C[2] * v[0] + C[4] * v[1] + C[5] * v[2];
      lam_s[L] = v[0] * Sv0 + v[1] * Sv1 + v[2] * Sv2;
      for (int i = 0; i < 3; ++i) ax[L][i] = d[i];
      for (int i = 0; i < 6; ++i) ax[L][3 + i] = C[i];
      for (int i = 0; i < 3; ++i) ax[L][9 + i] = v[i];
    }
  }
  __syncthreads();
  bool live = false;
  if (q < 2 * M) {
    const int L = q / M, m = q % M;
    S.alpha[L][m] = 0.0;
    S.comp[L][m].on = 0;
    if (S.label_on[L]) {
      const double sl = sqrt(fmax(lam_s[L], 0.0));
      const double z = M == 1 ? 0.0 : (m == M - 1 ? 1.0 : m * (2.0 / (M - 1)) - 1.0);
      for (int i = 0; i < 3; ++i) S.mu[L][m][i] = 0.5 + ax[L][i] + z * sl * ax[L][9 + i];
      for (int i = 0; i < 6; ++i) S.cov[L][m][i] = ax[L][3 + i] + ((i == 0 || i == 3 || i == 5) ? (double)reg : 0.0);
      live = sym_pd(S.cov[L][m]);
      S.alpha[L][m] = live ? 1.0 / M : 0.0;
    }
  }
  set_comps<M>(S, live);
}

// The M-step on S (LDS) in place, from the moments about its means: ten threads a component divide
// its moments by its count and form the covariance (one division's code for all), then one thread
// a component.  A component that drops out keeps its mean and covariance.
template <int M>
__device__ __forceinline__ void fit_step(const double* sums, GmmState& S, float reg) {
  __shared__ double dn[2 * M][10];   // count, first and second moments over the count
  __shared__ double cv[2 * M][6];
  __shared__ double nm[2][M];
  const int q = threadIdx.x, qc = q / 10, v = q - 10 * qc;
  if (q < 20 * M) dn[qc][v] = sums[q] / sums[10 * qc];
  __syncthreads();
  if (q < 20 * M && v >= 4) {
    const int i = v < 7 ? 1 : (v < 9 ? 2 : 3), j = v < 7 ? v - 3 : (v < 9 ? v - 5 : 3);
    const double c = dn[qc][v] - dn[qc][i] * dn[qc][j];
    cv[qc][v - 4] = i == j ? c + (double)reg : c;
  }
  __syncthreads();
  if (q < 2 * M) {
    const int L = q / M, m = q % M;
    nm[L][m] = 0.0;
    if (S.label_on[L]) {
      double W0 = 0.0;
      for (int k = 0; k < M; ++k) W0 += sums[(L * M + k) * 10];
      const double N = sums[q * 10];
      const GmmComp& g = S.comp[L][m];
      if (g.on && N > 1e-12 * W0 && sym_pd(cv[q])) {
        for (int i = 0; i < 3; ++i) S.mu[L][m][i] = (double)g.mu[i] + dn[q][1 + i];
        for (int i = 0; i < 6; ++i) S.cov[L][m][i] = cv[q][i];
        nm[L][m] = N;
      }
    }
  }
  __syncthreads();
  bool live = false;
  if (q < 2 * M) {
    const int L = q / M, m = q % M;
    if (S.label_on[L]) {
      double tot = 0.0;
      for (int k = 0; k < M; ++k) tot += nm[L][k];
      S.alpha[L][m] = tot > 0 ? nm[L][m] / tot : 0.0;
      live = S.alpha[L][m] > 0.0;
      if (!live) S.comp[L][m].on = 0;
    }
  }
  set_comps<M>(S, live);
}

// Workgroup 0 publishes the mixtures (the next launch's P, and the caller's copy).
template <int M>
__device__ __forceinline__ void publish(const GmmState& S, GmmState* out_st, float* out) {
  if (blockIdx.x != 0) return;
  const int* src = reinterpret_cast<const int*>(&S);
  int* dst = reinterpret_cast<int*>(out_st);
  for (int i = threadIdx.x; i < (int)(sizeof(GmmState) / sizeof(int)); i += GB) dst[i] = src[i];
  const int q = threadIdx.x;
  if (out && q < 2 * M) {
    const int L = q / M, m = q % M;
    float* o = out + ((size_t)L * M + m) * 10;
    const bool live = S.label_on[L] && S.alpha[L][m] > 0.0;
    o[0] = live ? (float)S.alpha[L][m] : 0.f;
    for (int i = 0; i < 3; ++i) o[1 + i] = live ? (float)S.mu[L][m][i] : 0.f;
    for (int i = 0; i < 6; ++i) o[4 + i] = live ? (float)S.cov[L][m][i] : 0.f;
  }
}

// A state copied into LDS (loads issued ahead of the reduction).
__device__ __forceinline__ void load_state(const GmmState* src, GmmState& P) {
  const gp<const int> s = G(reinterpret_cast<const int*>(src));
  int* d = reinterpret_cast<int*>(&P);
  for (int i = threadIdx.x; i < (int)(sizeof(GmmState) / sizeof(int)); i += GB) d[i] = s[i];
}

// The mixtures of a launch into S (LDS).  FIT = 0: those that the previous launch stored.
// FIT = 1, 2: the tiles' moments of the previous launch reduced in a fixed order, then the start
// or the M-step from its mixtures; workgroup 0 stores them for the next launch, which reads
// them and these moments while this one writes the other buffers.
// put() (the staged pixels) runs once the loads of the mixtures or the moments are in flight.
template <int M, int FIT, class Put>
__device__ __forceinline__ void mixtures(const GmmIO& io, GmmState& S, Put put) {
  if constexpr (FIT == 0) {
    load_state(io.st_prev, S);
    put();
    __syncthreads();
  } else {
    constexpr int NVI = 2 * (FIT == 1 ? 1 : M) * 10;
    __shared__ double sums[NVI];
    if (FIT == 2) load_state(io.st_prev, S);
    reduce_parts<NVI>(io.part_in, io.ntiles, sums);
    put();
    __syncthreads();
    if constexpr (FIT == 1)
      fit_start<M>(sums, S, io.reg, io.n);
    else
      fit_step<M>(sums, S, io.reg);
    publish<M>(S, io.st_next, io.out);
  }
}

// The moments of every tile: the start's (EM = false) or the E-step's under the launch's
// mixtures.  A pass bounded by its chain (pixels, mixtures, E-step, workgroup sum), not by its
// 7 bytes a pixel: at 640x480 with three components 9.2 us with both labels on
// a thread and four pixels unrolled on 300 workgroups, 6.6 us so with one FP32 sum per thread; with
// the fit in the same launch 10.4 us against 6.6 + 5.2 for the two, 11.4 us with two FP32 sums.
template <int M, bool EM, int FIT>
__global__ __launch_bounds__(GB) void k_gmm_acc(GmmIO io) {
  __shared__ __align__(16) float lds[LDS_N<EM ? M : 1>];
  __shared__ GmmState S;
  Staged<true> px;
  px.load(io);
  auto put = [&] { px.put(io, reinterpret_cast<float4*>(lds)); };
  if constexpr (EM) {
    mixtures<M, FIT>(io, S, put);
  } else {
    put();
    __syncthreads();
  }
  tile_moments<M, EM>(io, lds, S);
}

// One workgroup: the fit as a launch of its own.
template <int M, int FIT>
__global__ __launch_bounds__(GB) void k_gmm_fit(GmmIO io) {
  __shared__ GmmState S;
  mixtures<M, FIT>(io, S, [] {});
}

// psi_1 = -log sum_m alpha_m N(c; mu_m, Sigma_m) added to the unary cost of its label.
template <int M, int FIT>
__global__ __launch_bounds__(GB) void k_gmm_psi(GmmIO io) {
  __shared__ __align__(16) float lds[4 * GPX * SP_BLOCK];
  __shared__ float un_s[2][GPX * SP_BLOCK];
  __shared__ GmmState S;
  const int L = label_of(), first = blockIdx.x * io.tile, np = min(io.tile, io.n - first);
  const gp<float> un = G(io.unary) + (size_t)L * io.n + first;
  const int wf = wave_first() - L * SP_BLOCK;
  for (int t0 = 0; t0 + (int)slot_of() < np; t0 += SP_BLOCK)
    lds_load_u(&un_s[L][t0 + wf], (gp<const float>)un, 4u * (uint32_t)(t0 + slot_of()));
  Staged<false> px;
  px.load(io);
  mixtures<M, FIT>(io, S, [&] {
    px.put(io, reinterpret_cast<float4*>(lds));
    lds_wait();
  });
  Mix<M> X;
  X.load(S, L);
  if (!X.lab) return;
#pragma unroll 1
  for (int t = slot_of(); t < np; t += SP_BLOCK) {
    const float4 p = reinterpret_cast<const float4*>(lds)[t];
    float lp[M], mx = -INFINITY;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      lp[m] = X.logp(m, Prod(p.x - X.mu[m][0], p.y - X.mu[m][1], p.z - X.mu[m][2]));
      mx = fmaxf(mx, lp[m]);
    }
    if (!(mx > -INFINITY)) continue;
    float sum = 0.f;
#pragma unroll
    for (int m = 0; m < M; ++m) sum += X.on[m] ? ex(lp[m] - mx) : 0.f;
    un[t] = un_s[L][t] - (mx + lg(sum));
  }
}

// pass 0: the start's moments; 1: the E-step's; 2: psi.  fit 0: no fit in the launch; 1: the
// start; 2: the M-step.  pass -1: the fit alone, by one workgroup.
template <int M>
hipError_t launch_m(int pass, int fit, const GmmIO& io, hipStream_t st) {
  const dim3 grid(pass < 0 ? 1 : io.ntiles), block(GB);
  switch (4 * pass + fit) {
    case -3: hipLaunchKernelGGL((k_gmm_fit<M, 1>), grid, block, 0, st, io); break;
    case -2: hipLaunchKernelGGL((k_gmm_fit<M, 2>), grid, block, 0, st, io); break;
    case 0: hipLaunchKernelGGL((k_gmm_acc<M, false, 0>), grid, block, 0, st, io); break;
    case 4: hipLaunchKernelGGL((k_gmm_acc<M, true, 0>), grid, block, 0, st, io); break;
    case 5: hipLaunchKernelGGL((k_gmm_acc<M, true, 1>), grid, block, 0, st, io); break;
    case 6: hipLaunchKernelGGL((k_gmm_acc<M, true, 2>), grid, block, 0, st, io); break;
    case 8: hipLaunchKernelGGL((k_gmm_psi<M, 0>), grid, block, 0, st, io); break;
    case 9: hipLaunchKernelGGL((k_gmm_psi<M, 1>), grid, block, 0, st, io); break;
    case 10: hipLaunchKernelGGL((k_gmm_psi<M, 2>), grid, block, 0, st, io); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t sp_launch_gmm(int pass, int fit, int M, const GmmIO& io, hipStream_t st) {
  if (io.n <= 0) return hipSuccess;
  switch (M) {
    case 1: return launch_m<1>(pass, fit, io, st);
    case 2: return launch_m<2>(pass, fit, io, st);
    case 3: return launch_m<3>(pass, fit, io, st);
    case 4: return launch_m<4>(pass, fit, io, st);
    default: return hipErrorInvalidValue;
  }
}
