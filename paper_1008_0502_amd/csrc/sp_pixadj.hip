// Pixel-level adjoint of the saliency model (Section 3 / Section 7.2): dL/d frame_t from
// dL/dS_t, through the weighted sum, N(.), the across-scale sum, centre-surround, the Gabor
// maps, the pyramid and the level-0 features (the motion feature also reaches frame t-1).
// The forward maps of up to SP_PA_SLOTS frames are recomputed side by side by the forward
// kernels first (the across-scale sums come from the tape), and every pass here runs over all of
// them (blockIdx.z = frame slot): one 640x480 frame's passes were about 30 dependent launches
// of 2 to 37 us, 206 us a frame; eight frames at once take 31 us a frame.  Every pass
// here gathers: one thread per output element, each output a fixed-order sum over the
// inputs that depend on it, so results do not depend on scheduling.  Non-differentiable
// points follow one convention: the global minimum and maximum and each 8x8 block maximum
// of an N(.) input take the gradient at the first position in row-major order whose
// normalised value lies within 2^-20 of the extreme (maps with a vanishing difference
// over whole regions hold exact ties there, which rounding must not decide), a map at
// or below flat_tol passes none, |.| has sign(0) = 0, max(0, .) passes nothing at 0 and
// min(r', g') passes to r' on ties; the chromatic mask and colour maximum are constants.
// The branches of the features are decided from the frame's bytes, where they are exact
// (2R - G - B > 0 for the red opponent, and so on), not from the rounded ratios R / I.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>

#include <algorithm>

#include "sp_internal.h"
#include "sp_kernels.h"
#include "sp_device.h"

namespace {

constexpr int TILE = SP_PA_TILE;             // elements of a workgroup of the elementwise passes
constexpr int PER = TILE / SP_BLOCK;

typedef float Quad __attribute__((ext_vector_type(4)));   // a 16-byte access of global memory
typedef float Pair __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float kb(int i) {   // i in -2..2
  return i == 0 ? 0.375f : ((i == 1 || i == -1) ? 0.25f : 0.0625f);
}

// The workspace pointer of frame slot z.
template <class T>
__device__ __forceinline__ T* slot(T* p, const PaDesc& A, int z) {
  return reinterpret_cast<T*>(const_cast<char*>(reinterpret_cast<const char*>(p)) + (size_t)z * A.stride);
}

// dL/dS = gs / m - [x = x*] sum(gs S) / m^2 (zero when S was flat), in two launches.
__global__ __launch_bounds__(SP_BLOCK) void k_pa_gs(PaDesc A, const float* __restrict__ gs_, const float* __restrict__ S_,
                                                    const float* __restrict__ ms_, int n, float flat_tol) {
  // every workgroup: SP_BLOCK elements of gs / m and its FP64 partial of sum gs S; the
  // element at the argmax is left to k_pa_gs_fix
  __shared__ double sh[4];
  const int z = blockIdx.z;
  const float *gs = gs_ + (size_t)z * n, *S = S_ + (size_t)z * n, *ms = ms_ + 2 * z;
  const float m = ms[0];
  const int xs = __float_as_int(ms[1]);
  const bool flat = !(m > flat_tol);
  const int i = blockIdx.x * SP_BLOCK + threadIdx.x;
  const float g = i < n ? gs[i] : 0.f;
  const double dot = wave_sum_d(i < n ? (double)g * (double)S[i] : 0.0);
  if (i < n && i != xs) slot(A.gS, A, z)[i] = flat ? 0.f : g * (1.f / m);
  if (lane_id() == 0) sh[wave_id()] = dot;
  __syncthreads();
  if (threadIdx.x == 0) slot(A.gs_part, A, z)[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// The argmax element of gS: gs / m - (sum gs S) / m^2, the sum from the workgroups' partials
// in a fixed order.
__global__ __launch_bounds__(SP_BLOCK) void k_pa_gs_fix(PaDesc A, const float* __restrict__ gs_, const float* __restrict__ ms_,
                                                        int n, int nparts, float flat_tol) {
  __shared__ double sh[SP_BLOCK];
  const int z = blockIdx.z;
  const float *gs = gs_ + (size_t)z * n, *ms = ms_ + 2 * z;
  const double* part = slot(A.gs_part, A, z);
  double acc = 0.0;
  for (int k = threadIdx.x; k < nparts; k += SP_BLOCK) acc += part[k];
  const double dot = block_sum_d(acc, sh);
  const int xs = __float_as_int(ms[1]);
  if (threadIdx.x == 0 && xs >= 0 && xs < n) {   // an index outside the map was written by k_pa_gs
    const float m = ms[0];
    const float corr = (float)(dot / ((double)m * (double)m));
    slot(A.gS, A, z)[xs] = !(m > flat_tol) ? 0.f : gs[xs] * (1.f / m) - corr;
  }
}

// Tolerance (on the normalised map) within which values count as tied with an extreme.
constexpr float kTie = 0x1p-20f;

// Maps of the N(.) adjoint: m < 8 the across-scale sum of channel m (from the tape), then the
// eight centre-surround maps of each pair.  A pair's plane holds the signed difference D; the
// map is |D|.
struct MapView {
  gp<const float> X;   // the map, or D where abs is set
  gp<const float> g;   // dL/dN before the factor gs
  int h, w, m;
  float gs;
  bool abs;
  __device__ __forceinline__ float at(int i) const { return abs ? fabsf(X[i]) : X[i]; }
};
__device__ __forceinline__ MapView map_view(const PaDesc& A, const StreamDesc& sd, const float* fbar, int m, int z) {
  MapView M;
  const int k = m & (SP_NCH - 1);
  const size_t plc = (size_t)sd.Hl[sd.c_max] * sd.Wl[sd.c_max];
  M.m = m;
  if (m < SP_NCH) {
    M.X = G(fbar + ((size_t)z * SP_NCH + k) * plc);
    M.g = G((const float*)slot(A.gS, A, z));
    M.h = sd.Hl[sd.c_max];
    M.w = sd.Wl[sd.c_max];
    M.gs = sd.w[k];
    M.abs = false;
  } else {
    const int p = (m >> 3) - 1, c = sd.pc[p];
    M.h = sd.Hl[c];
    M.w = sd.Wl[c];
    const size_t n = (size_t)M.h * M.w;
    M.X = G((const float*)slot(A.D[p], A, z) + k * n);
    M.g = G((const float*)(c == sd.c_max ? slot(A.gfbar, A, z) : slot(A.gN[c], A, z)) + k * n);
    M.gs = 1.f;
    M.abs = true;
  }
  return M;
}

// Statistics of the N(.) adjoint: (1) the (min, max) of tiles of TILE pixels (the
// centre-surround pass takes its own); (2) per 8-row strip, with the map's range reduced from
// (1): each 8x8 block's maximum of Y = (X - mn) / range and its first position (row-major)
// within kTie of it, the strip's sums of the block maxima, g Y and g (FP64), and the first
// positions within kTie of the minimum and the maximum; (3) per map, the scalars below.

// The map's (min, max) and, for a pair, the scale max(|X(c)|, |X(s)|) from its tile partials
// (every thread gets them).
__device__ __forceinline__ void map_range(const PaDesc& A, const MapView& M, int z, float (*sh)[4], float& mn, float& mx,
                                          float& am) {
  const int nt = (M.h * M.w + TILE - 1) / TILE;
  const PaMM* mm = slot(A.mm, A, z) + (size_t)M.m * A.mm_n;
  float a = INFINITY, b = -INFINITY, c = 0.f;
  for (int k = threadIdx.x; k < nt; k += SP_BLOCK) {
    const PaMM v = mm[k];
    a = fminf(a, v.mn);
    b = fmaxf(b, v.mx);
    c = fmaxf(c, v.am);
  }
  a = wave_reduce<OpMin>(a);
  b = wave_reduce<OpMax>(b);
  c = wave_reduce<OpMax>(c);
  if (lane_id() == 0) {
    sh[0][wave_id()] = a;
    sh[1][wave_id()] = b;
    sh[2][wave_id()] = c;
  }
  __syncthreads();
  mn = fminf(fminf(sh[0][0], sh[0][1]), fminf(sh[0][2], sh[0][3]));
  mx = fmaxf(fmaxf(sh[1][0], sh[1][1]), fmaxf(sh[1][2], sh[1][3]));
  am = fmaxf(fmaxf(sh[2][0], sh[2][1]), fmaxf(sh[2][2], sh[2][3]));
}
// One tile's partial from the threads' values.
__device__ __forceinline__ void store_mm(float mn, float mx, float am, PaMM* out, float (*sh)[4]) {
  mn = wave_reduce<OpMin>(mn);
  mx = wave_reduce<OpMax>(mx);
  am = wave_reduce<OpMax>(am);
  if (lane_id() == 0) {
    sh[0][wave_id()] = mn;
    sh[1][wave_id()] = mx;
    sh[2][wave_id()] = am;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    *out = PaMM{fminf(fminf(sh[0][0], sh[0][1]), fminf(sh[0][2], sh[0][3])),
                fmaxf(fmaxf(sh[1][0], sh[1][1]), fmaxf(sh[1][2], sh[1][3])),
                fmaxf(fmaxf(sh[2][0], sh[2][1]), fmaxf(sh[2][2], sh[2][3])), 0.f};
}

__global__ __launch_bounds__(SP_BLOCK) void k_pa_nmm(PaDesc A, const StreamDesc* __restrict__ sds, const float* __restrict__ fbar) {
  __shared__ float sh[3][4];
  const int z = blockIdx.z;
  const MapView M = map_view(A, sds[z], fbar, blockIdx.y, z);
  const int n = M.h * M.w, base = blockIdx.x * TILE;
  if (base >= n) return;   // uniform
  float mn = INFINITY, mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = base + k * SP_BLOCK + threadIdx.x;
    const float v = M.at(min(i, n - 1));
    mn = i < n ? fminf(mn, v) : mn;
    mx = i < n ? fmaxf(mx, v) : mx;
  }
  store_mm(mn, mx, 0.f, slot(A.mm, A, z) + (size_t)M.m * A.mm_n + blockIdx.x, sh);
}

__global__ __launch_bounds__(SP_BLOCK) void k_pa_nstrip(PaDesc A, const StreamDesc* __restrict__ sds,
                                                        const float* __restrict__ fbar, int m0, float flat_tol) {
  __shared__ float sh[3][4];
  __shared__ double shd[3][4];
  __shared__ int shi[2][4];
  const int z = blockIdx.z;
  const MapView M = map_view(A, sds[z], fbar, m0 + blockIdx.y, z);
  if ((int)blockIdx.x >= (M.h + 7) >> 3) return;   // uniform
  float mn, mx, am;
  map_range(A, M, z, sh, mn, mx, am);
  const float rng = mx - mn;
  if (!(rng > flat_tol)) return;   // uniform: a flat map passes no gradient
  const float rr = 1.f / rng;
  const gp<int32_t> bpos = G(slot(A.bpos, A, z) + (size_t)M.m * A.nb_n);
  const int y0 = blockIdx.x * 8, nrow = min(8, M.h - y0), nbx = (M.w + 7) >> 3;
  double sb = 0.0, sgy = 0.0, sg = 0.0;
  int jn = 0x7fffffff, jx = 0x7fffffff;
  // a thread takes column x of the strip; the eight columns of a block are eight
  // consecutive lanes (the chunks of SP_BLOCK columns start at multiples of 8).  All sixteen
  // loads of a chunk are issued before any use.
  for (int x0 = 0; x0 < M.w; x0 += SP_BLOCK) {
    const int x = x0 + threadIdx.x;
    const bool cv = x < M.w;
    float Y[8], G8[8], cb = -INFINITY;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int i = (y0 + min(r, nrow - 1)) * M.w + min(x, M.w - 1);
      Y[r] = M.at(i);
      G8[r] = M.g[i];
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const bool ok = cv && r < nrow;
      const int i = (y0 + min(r, nrow - 1)) * M.w + min(x, M.w - 1);
      const float v = (Y[r] - mn) * rr;
      Y[r] = ok ? v : -INFINITY;
      cb = fmaxf(cb, Y[r]);
      if (ok) {
        const double g = (double)G8[r] * (double)M.gs;
        sgy += g * (double)v;
        sg += g;
        if (v <= kTie) jn = min(jn, i);
        if (v >= 1.f - kTie) jx = min(jx, i);
      }
    }
    // the block's maximum and its first position within kTie (row-major: smallest index)
    float best = cb;
    best = fmaxf(best, dpp_f<0xB1>(best));
    best = fmaxf(best, dpp_f<0x4E>(best));
    best = fmaxf(best, dpp_f<0x141>(best));
    int cand = 0x7fffffff;
#pragma unroll
    for (int r = 7; r >= 0; --r)
      if (Y[r] >= best - kTie) cand = (y0 + r) * M.w + x;
    cand = min(cand, dpp_i<0xB1>(cand));
    cand = min(cand, dpp_i<0x4E>(cand));
    cand = min(cand, dpp_i<0x141>(cand));
    if ((threadIdx.x & 7) == 0 && cv) {
      bpos[(y0 >> 3) * nbx + (x >> 3)] = cand;
      sb += (double)best;
    }
  }
  sb = wave_sum_d(sb);
  sgy = wave_sum_d(sgy);
  sg = wave_sum_d(sg);
  jn = wave_min_i(jn);
  jx = wave_min_i(jx);
  if (lane_id() == 0) {
    const int w = wave_id();
    shd[0][w] = sb;
    shd[1][w] = sgy;
    shd[2][w] = sg;
    shi[0][w] = jn;
    shi[1][w] = jx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    auto add = [&](int q) { return (shd[q][0] + shd[q][1]) + (shd[q][2] + shd[q][3]); };
    auto mini = [&](int q) { return min(min(shi[q][0], shi[q][1]), min(shi[q][2], shi[q][3])); };
    slot(A.strip, A, z)[(size_t)M.m * A.strip_n + blockIdx.x] = PaStrip{add(0), add(1), add(2), mini(0), mini(1)};
  }
}

__global__ __launch_bounds__(SP_BLOCK) void k_pa_nfin(PaDesc A, const StreamDesc* __restrict__ sds,
                                                      const float* __restrict__ fbar, int m0, float flat_tol) {
  __shared__ float sh[3][4];
  __shared__ int shi[2][4];
  __shared__ double shd[3][4];
  const int z = blockIdx.z;
  const MapView M = map_view(A, sds[z], fbar, m0 + blockIdx.y, z);
  float* sc = slot(A.sc, A, z) + (size_t)M.m * SP_PA_SC;
  const PaStrip* strip = slot(A.strip, A, z) + (size_t)M.m * A.strip_n;
  float mn, mx, am;
  map_range(A, M, z, sh, mn, mx, am);
  const float rng = mx - mn;
  if (!(rng > flat_tol)) {
    if (threadIdx.x == 0) {
      for (int k = 0; k < SP_PA_SC; ++k) sc[k] = 0.f;
      sc[6] = 1.f;
    }
    return;
  }
  const int ns = (M.h + 7) >> 3;
  double sb = 0.0, sgy = 0.0, sg = 0.0;
  int jn = 0x7fffffff, jx = 0x7fffffff;
  for (int k = threadIdx.x; k < ns; k += SP_BLOCK) {
    const PaStrip p = strip[k];
    sb += p.sb;
    sgy += p.sgy;
    sg += p.sg;
    jn = min(jn, p.jn);
    jx = min(jx, p.jx);
  }
  sb = wave_sum_d(sb);
  sgy = wave_sum_d(sgy);
  sg = wave_sum_d(sg);
  jn = wave_min_i(jn);
  jx = wave_min_i(jx);
  if (lane_id() == 0) {
    const int w = wave_id();
    shd[0][w] = sb;
    shd[1][w] = sgy;
    shd[2][w] = sg;
    shi[0][w] = jn;
    shi[1][w] = jx;
  }
  __syncthreads();
  const int nb = ((M.w + 7) >> 3) * ns;
  if (threadIdx.x == 0) {
    auto add = [&](int q) { return (shd[q][0] + shd[q][1]) + (shd[q][2] + shd[q][3]); };
    auto mini = [&](int q) { return min(min(shi[q][0], shi[q][1]), min(shi[q][2], shi[q][3])); };
    const double Sb = add(0), Sgy = add(1), Sg = add(2);
    const double mbar = nb > 1 ? (Sb - 1.0) / (nb - 1) : 0.0;
    const double a = (1.0 - mbar) * (1.0 - mbar);
    const double gb = nb > 1 ? -2.0 * (1.0 - mbar) * Sgy / (nb - 1) : 0.0;
    const double sgyy = a * Sgy + gb * Sb;   // sum gY Y
    const double sgyt = a * Sg + gb * nb;    // sum gY
    sc[0] = (float)(a / rng);
    sc[1] = (float)(gb / rng);
    sc[2] = (float)((sgyy - sgyt) / rng);
    sc[3] = (float)(-sgyy / rng);
    sc[4] = __int_as_float(mini(0));
    sc[5] = __int_as_float(mini(1));
    sc[6] = 0.f;
    sc[7] = am;
  }
}

// dL/dX of map M at element i (row y, column x):
// gN A / range + [block maximum] gb / range + [argmin] g(min) + [argmax] g(max).
__device__ __forceinline__ float napply_at(const MapView& M, const float* sc, gp<const int32_t> bpos, int nbx, int y, int x, int i) {
  if (sc[6] != 0.f) return 0.f;
  float v = M.g[i] * M.gs * sc[0];
  if (bpos[(y >> 3) * nbx + (x >> 3)] == i) v += sc[1];
  if (i == __float_as_int(sc[4])) v += sc[2];
  if (i == __float_as_int(sc[5])) v += sc[3];
  return v;
}

// The across-scale sums' adjoint gfbar (blockIdx.y = channel).
__global__ __launch_bounds__(SP_BLOCK) void k_pa_napply(PaDesc A, const StreamDesc* __restrict__ sds, const float* __restrict__ fbar) {
  const int z = blockIdx.z;
  const MapView M = map_view(A, sds[z], fbar, blockIdx.y, z);
  const float* sc = slot(A.sc, A, z) + (size_t)M.m * SP_PA_SC;
  const gp<const int32_t> bpos = G((const int32_t*)slot(A.bpos, A, z) + (size_t)M.m * A.nb_n);
  const int n = M.h * M.w, base = blockIdx.x * TILE, nbx = (M.w + 7) >> 3;
  const gp<float> out = G(slot(A.gfbar, A, z) + (size_t)blockIdx.y * n);
  Walk2 wk(base + threadIdx.x, M.w);
#pragma unroll
  for (int k = 0; k < PER; ++k, wk.next()) {
    const int i = base + k * SP_BLOCK + threadIdx.x;
    if (i < n) out[i] = napply_at(M, sc, bpos, nbx, wk.r, wk.c, i);
  }
}

// Weight of output position yo (of a clamped 5-tap blur over n positions) in the blur at yp.
__device__ __forceinline__ float blur_w(int yo, int yp, int n) {
  float a = 0.f;
#pragma unroll
  for (int i = -2; i <= 2; ++i) a += clampi(yp + i, 0, n - 1) == yo ? kb(i) : 0.f;
  return a;
}

// Transpose of one pyramid step at fine rows 2q, 2q+1 and columns 2r, 2r+1: coarse rows and
// columns q - 1 .. q + 1 reach them.  The nine coarse values of one channel serve the four
// outputs; the weights come from wy, wx [2][3] (zero outside the coarse level).  A wavefront
// wholly off the levels' borders has the same weights in every lane, constants then: the weights
// and the tests for zero were most of the instructions.
struct QuadT {
  float wy[2][3], wx[2][3];
  uint32_t o[3][3];   // clamped element offsets
  bool inner;         // uniform over the wavefront
  __device__ __forceinline__ QuadT(int q, int r, int h, int w, int hb, int wb) {
    inner = __all(q >= 2 && r >= 2 && q + 2 < hb && r + 2 < wb);
    if (!inner) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          const int y2 = q - 1 + b, x2 = r - 1 + b;
          wy[a][b] = (y2 >= 0 && y2 < hb) ? blur_w(2 * q + a, 2 * y2, h) : 0.f;
          wx[a][b] = (x2 >= 0 && x2 < wb) ? blur_w(2 * r + a, 2 * x2, w) : 0.f;
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b)
        o[a][b] = (uint32_t)clampi(q - 1 + a, 0, hb - 1) * (uint32_t)wb + (uint32_t)clampi(r - 1 + b, 0, wb - 1);
  }
  __device__ __forceinline__ void load(const gp<const float> src, float (&v)[3][3]) const {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) v[a][b] = src[o[a][b]];
  }
  // zero weights are skipped, not multiplied: they would turn an infinite gradient into NaN
  __device__ __forceinline__ void apply(const float (&v)[3][3], float (&out)[2][2]) const {
    if (inner) {
      // fine position 2q hears kb(2), kb(0), kb(2) of the three, 2q + 1 the last two's kb(1)
      float e[3], f[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        e[i] = kb(2) * v[i][0];
        e[i] += kb(0) * v[i][1];
        e[i] += kb(2) * v[i][2];
        f[i] = kb(1) * v[i][1];
        f[i] += kb(1) * v[i][2];
      }
      auto col = [](const float (&c)[3], float& top, float& bot) {
        top = kb(2) * c[0];
        top += kb(0) * c[1];
        top += kb(2) * c[2];
        bot = kb(1) * c[1];
        bot += kb(1) * c[2];
      };
      col(e, out[0][0], out[1][0]);
      col(f, out[0][1], out[1][1]);
      return;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          float r = 0.f;
#pragma unroll
          for (int j = 0; j < 3; ++j) r += wx[b][j] != 0.f ? v[i][j] * wx[b][j] : 0.f;
          acc += wy[a][i] != 0.f ? wy[a][i] * r : 0.f;
        }
        out[a][b] = acc;
      }
  }
};

// Transposed pyramid step from a level of hb x wb to the finer h x w, plane blockIdx.y (all
// eight channels, or I, RG, BY, M: planes 0, 1, 2, 7 when four); out is added to or written.
// A thread makes a 2x2 block from nine coarse values (one thread per output, with its up to
// nine values and weights, took 14.7 us for the last step of a 640x480 frame).
__global__ __launch_bounds__(SP_BLOCK) void k_pa_reduce_t(PaDesc A, const float* __restrict__ src_, float* __restrict__ out_,
                                                          int h, int w, int hb, int wb, int accumulate) {
  const int z = blockIdx.z;
  const int pl = gridDim.y == 4 && blockIdx.y == 3 ? 7 : blockIdx.y;
  const int i = blockIdx.x * SP_BLOCK + threadIdx.x;
  if (i >= hb * wb) return;
  const int q = i / wb, r = i - q * wb;
  const gp<const float> src = G((const float*)slot(src_, A, z) + (size_t)pl * hb * wb);
  const gp<float> out = G(slot(out_, A, z) + (size_t)pl * h * w);
  const QuadT T(q, r, h, w, hb, wb);
  float v[3][3], o[2][2];
  T.load(src, v);
  T.apply(v, o);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
      if (2 * q + a < h && 2 * r + b < w) {
        const uint32_t e = (uint32_t)(2 * q + a) * (uint32_t)w + (uint32_t)(2 * r + b);
        out[e] = accumulate ? out[e] + o[a][b] : o[a][b];
      }
}

// Bilinear sample-aligned tap of target position y at level offset d on n source samples.
__device__ __forceinline__ void tap(int y, int d, int n, int& i0, int& i1, float& w) {
  const float fy = fminf((float)y * __int_as_float((127 - d) << 23), (float)(n - 1));   // y * 2^-d, exact
  i0 = (int)fy;
  i1 = min(i0 + 1, n - 1);
  w = fy - (float)i0;
}

// D = X(c) - up X(s) of pair blockIdx.y / 8, channel blockIdx.y % 8 (kept for the adjoint), and
// the tile's partial: (min, max) of F = |D| and the largest |X(c)|, |X(s)|.
__global__ __launch_bounds__(SP_BLOCK) void k_pa_csmap(PaDesc A, const StreamDesc* __restrict__ sds) {
  __shared__ float sh[3][4];
  const int z = blockIdx.z, p = blockIdx.y >> 3, k = blockIdx.y & 7;
  const StreamDesc& sd = sds[z];
  const int c = sd.pc[p], s = sd.ps[p], d = s - c;
  const int h = sd.Hl[c], w = sd.Wl[c], hb = sd.Hl[s], wb = sd.Wl[s], n = h * w, base = blockIdx.x * TILE;
  if (base >= n) return;   // uniform
  const gp<const float> a = G(chan_ptr(sd, k, c)), b = G(chan_ptr(sd, k, s));
  const gp<float> out = G(slot(A.D[p], A, z) + (size_t)k * n);
  float mn = INFINITY, mx = -INFINITY, am = 0.f;
  // Four elements of a row a thread where rows are whole aligned quads and d >= 2, so that the four
  // share the rows and columns they sample: one load and store of the map for four, and four
  // surround values for sixteen (31 -> 23 us for eight 640x480 frames).
  const bool quad = (w & 3) == 0 && d >= 2 && ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
  if (quad) {
    static_assert(PER == 4, "a quad per thread");
    const int i = base + 4 * (int)threadIdx.x;
    if (i < n) {
      const int y = i / w, x = i - y * w;
      int y0, y1, x0[4], x1[4];
      float wy, wx[4];
      tap(y, d, hb, y0, y1, wy);
#pragma unroll
      for (int q = 0; q < 4; ++q) tap(x + q, d, wb, x0[q], x1[q], wx[q]);
      // the four positions lie between the same two samples
      const float b00 = b[y0 * wb + x0[0]], b01 = b[y0 * wb + x1[0]];
      const float b10 = b[y1 * wb + x0[0]], b11 = b[y1 * wb + x1[0]];
      const Quad X4 = *(gp<const Quad>)(a + i);
      const float X[4] = {X4.x, X4.y, X4.z, X4.w};
      float D[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float top = (1.f - wx[q]) * b00 + wx[q] * b01;
        const float bot = (1.f - wx[q]) * b10 + wx[q] * b11;
        D[q] = X[q] - ((1.f - wy) * top + wy * bot);
        mn = fminf(mn, fabsf(D[q]));
        mx = fmaxf(mx, fabsf(D[q]));
        am = fmaxf(am, fabsf(X[q]));
        if (i + q < hb * wb) am = fmaxf(am, fabsf(b[i + q]));
      }
      *(gp<Quad>)(out + i) = Quad{D[0], D[1], D[2], D[3]};
    }
    store_mm(mn, mx, am, slot(A.mm, A, z) + (size_t)(SP_NCH + blockIdx.y) * A.mm_n + blockIdx.x, sh);
    return;
  }
  Walk2 wk(base + threadIdx.x, w);
#pragma unroll
  for (int q = 0; q < PER; ++q, wk.next()) {
    const int i = base + q * SP_BLOCK + threadIdx.x;
    if (i < n) {
      int y0, y1, x0, x1;
      float wy, wx;
      tap(wk.r, d, hb, y0, y1, wy);
      tap(wk.c, d, wb, x0, x1, wx);
      const float top = (1.f - wx) * b[y0 * wb + x0] + wx * b[y0 * wb + x1];
      const float bot = (1.f - wx) * b[y1 * wb + x0] + wx * b[y1 * wb + x1];
      const float X = a[i], D = X - ((1.f - wy) * top + wy * bot);
      out[i] = D;
      mn = fminf(mn, fabsf(D));
      mx = fmaxf(mx, fabsf(D));
      am = fmaxf(am, fabsf(X));
      if (i < hb * wb) am = fmaxf(am, fabsf(b[i]));
    }
  }
  store_mm(mn, mx, am, slot(A.mm, A, z) + (size_t)(SP_NCH + blockIdx.y) * A.mm_n + blockIdx.x, sh);
}

// Derivative of |D| taken as 0 within this fraction of the pair's scale: there the sign of
// D is below what FP32 maps resolve (D vanishes identically on flat regions of both levels).
constexpr float kSignBand = 0x1p-16f;

// gD = sign(D) dL/dF outside the band (0 inside) in the place of D, for every pair of centre
// level A.cl[blockIdx.y / 8] in pair order, and their sum as that level's dL/dX.
__global__ __launch_bounds__(SP_BLOCK) void k_pa_csadj(PaDesc A, const StreamDesc* __restrict__ sds) {
  const int z = blockIdx.z, c = A.cl[blockIdx.y >> 3], k = blockIdx.y & 7;
  const StreamDesc& sd = sds[z];
  const int w = sd.Wl[c], n = sd.Hl[c] * w, base = blockIdx.x * TILE, nbx = (w + 7) >> 3;
  if (base >= n) return;   // uniform
  const gp<float> out = G(slot(A.gX[c], A, z) + (size_t)k * n);
  // Four elements of a row a thread where rows are whole aligned quads: they lie in one 8x8 block,
  // whose position is read once, and every other access is 16 bytes (50 -> 23 us for eight 640x480
  // frames; 170 MB, 33 us from memory, part of which stays on the chip).
  if ((w & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
    static_assert(PER == 4, "a quad per thread");
    const int i = base + 4 * (int)threadIdx.x;
    if (i >= n) return;
    const int y = i / w, x = i - y * w;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int p = 0; p < sd.n_pairs; ++p) {
      if (sd.pc[p] != c) continue;
      const MapView M = map_view(A, sd, nullptr, SP_NCH * (1 + p) + k, z);
      const float* sc = slot(A.sc, A, z) + (size_t)M.m * SP_PA_SC;
      const gp<float> D = G(slot(A.D[p], A, z) + (size_t)k * n);
      const int bp = G((const int32_t*)slot(A.bpos, A, z))[(size_t)M.m * A.nb_n + (uint32_t)((y >> 3) * nbx + (x >> 3))];
      const Quad g4 = *(gp<const Quad>)(M.g + i), d4 = *(gp<const Quad>)(D + i);
      const float g[4] = {g4.x, g4.y, g4.z, g4.w}, v[4] = {d4.x, d4.y, d4.z, d4.w};
      const float band = kSignBand * sc[7], s0 = sc[0], s1 = sc[1], s2 = sc[2], s3 = sc[3];
      const int jn = __float_as_int(sc[4]), jx = __float_as_int(sc[5]);
      const bool flat = sc[6] != 0.f;
      float gd[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float gf = g[q] * M.gs * s0;
        if (bp == i + q) gf += s1;
        if (jn == i + q) gf += s2;
        if (jx == i + q) gf += s3;
        gf = flat ? 0.f : gf;
        gd[q] = v[q] > band ? gf : (v[q] < -band ? -gf : 0.f);
        acc[q] += gd[q];
      }
      *(gp<Quad>)(D + i) = Quad{gd[0], gd[1], gd[2], gd[3]};
    }
    *(gp<Quad>)(out + i) = Quad{acc[0], acc[1], acc[2], acc[3]};
    return;
  }
  float acc[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) acc[q] = 0.f;
  for (int p = 0; p < sd.n_pairs; ++p) {
    if (sd.pc[p] != c) continue;
    const MapView M = map_view(A, sd, nullptr, SP_NCH * (1 + p) + k, z);
    const float* sc = slot(A.sc, A, z) + (size_t)M.m * SP_PA_SC;
    const gp<const int32_t> bpos = G((const int32_t*)slot(A.bpos, A, z) + (size_t)M.m * A.nb_n);
    const gp<float> D = G(slot(A.D[p], A, z) + (size_t)k * n);
    const float band = kSignBand * sc[7];
    Walk2 wk(base + threadIdx.x, w);
#pragma unroll
    for (int q = 0; q < PER; ++q, wk.next()) {
      const int i = base + q * SP_BLOCK + threadIdx.x;
      if (i < n) {
        const float gf = napply_at(M, sc, bpos, nbx, wk.r, wk.c, i), v = D[i];
        const float gd = v > band ? gf : (v < -band ? -gf : 0.f);
        D[i] = gd;
        acc[q] += gd;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int i = base + q * SP_BLOCK + threadIdx.x;
    if (i < n) out[i] = acc[q];
  }
}

// dL/dX(s) of surround level A.sl[blockIdx.y / 8]: up^T(-gD) of every pair with that
// surround, added to the level's centre part when it has one.  A level-s element gathers the
// level-c elements xs 2^d + k, |k| < 2^d, weight (2^d - |k|) / 2^d (1 beyond the last sample).
// Eight lanes per level-s element: lane j takes the window's rows j, j + 8, ..., each as the
// weighted sum of its columns (16 bytes a load where rows allow), and the lanes' sums are added in a
// fixed order.  A workgroup takes 128 elements: with sixteen elements and sixteen lanes each the
// launch of eight 640x480 frames was 57600 workgroups and 54 us, 41 us here.
static_assert(SP_BLOCK % 64 == 0, "whole wavefronts");
constexpr int UPT_L = 8;    // lanes per level-s element
constexpr int UPT_E = 128;  // level-s elements of a workgroup
__global__ __launch_bounds__(SP_BLOCK) void k_pa_up_t(PaDesc A, const StreamDesc* __restrict__ sds) {
  const int z = blockIdx.z, s = A.sl[blockIdx.y >> 3], ch = blockIdx.y & 7;
  const StreamDesc& sd = sds[z];
  const int hb = sd.Hl[s], wb = sd.Wl[s];
  const int e0 = blockIdx.x * UPT_E;
  if (e0 >= hb * wb) return;   // uniform
  // neighbouring lanes take neighbouring elements of the same window row, which lie in the same
  // cache lines; lanes 8 apart the rows
  const int j = lane_id() >> 3, own = wave_id() * (64 / UPT_L) + (lane_id() & 7);
  const gp<float> out = G(slot(A.gX[s], A, z) + (size_t)ch * hb * wb);
  const bool centre = (A.centres >> s) & 1u;
#pragma unroll 1
  for (int b = e0; b < min(e0 + UPT_E, hb * wb); b += SP_BLOCK / UPT_L) {
    const int e = b + own;
    const bool valid = e < hb * wb;   // every lane stays for the sum
    const int i = valid ? e : 0;
    const int ys = i / wb, xs = i - ys * wb;
    float tot = valid && j == 0 && centre ? out[e] : 0.f;
    for (int p = 0; p < sd.n_pairs; ++p) {
      if (sd.ps[p] != s) continue;
      const int c = sd.pc[p], d = s - c, st = 1 << d, ha = sd.Hl[c], wa = sd.Wl[c];
      const float inv = __int_as_float((127 - d) << 23);   // 2^-d
      const gp<const float> a = G((const float*)slot(A.D[p], A, z) + (size_t)ch * ha * wa);
      const bool quad = st >= 4 && (wa & 3) == 0 && (reinterpret_cast<uintptr_t>(a) & 15) == 0;   // uniform
      const int xc = xs * st, x_lo = max(0, xc - st + 1), x_hi = min(wa - 1, xc + st - 1);
      float acc = 0.f;
      if (valid)
        for (int ky = j - st + 1; ky < st; ky += UPT_L) {
          const int y = ys * st + ky;
          if (y < 0 || y >= ha) continue;
          const float ay = ys == hb - 1 && ky > 0 ? 1.f : (float)(st - abs(ky)) * inv;
          const gp<const float> row = a + (uint32_t)y * (uint32_t)wa;
          float r = 0.f;
          if (quad) {   // whole quads of columns from xc - st on; column xc - st itself is not in the window
#pragma unroll 4
            for (int x = xc - st; x < xc + st; x += 4) {
              if (x < 0 || x >= wa) continue;
              const Quad v4 = *(gp<const Quad>)(row + x);
              const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const int kx = x + q - xc;
                const float ax = xs == wb - 1 && kx > 0 ? 1.f : (float)(st - abs(kx)) * inv;
                if (q > 0 || kx > -st) r += ax * v[q];
              }
            }
          } else {
#pragma unroll 4
            for (int x = x_lo; x <= x_hi; ++x) {
              const int kx = x - xc;
              const float ax = xs == wb - 1 && kx > 0 ? 1.f : (float)(st - abs(kx)) * inv;
              r += ax * row[x];
            }
          }
          acc += ay * r;
        }
      // the eight lanes' sums: pairs, quads, halves (every lane ends with the total)
      acc += __shfl_xor(acc, 8);
      acc += __shfl_xor(acc, 16);
      acc += __shfl_xor(acc, 32);
      tot -= acc;
    }
    if (valid && j == 0) out[e] = tot;
  }
}

// dL/dI(l) += sum over the four orientations of the clamped Gabor correlation's transpose.
// With E(q) = sum_{v,u} h(v, u) gO(q - (v, u)) on the plane extended by the radius (gO zero
// outside the level), the transpose at p is the sum of E(q) over the q that clamp to p: q = p
// inside the level, the outside strip folded onto its border row or column.
// The kernels are sums of separable ones (h0 = gm(u) g(v), h90 = g(u) gm(v), h45 and h135 =
// gc gc -+ gs gs - c45 g g), so with P = gO45 + gO135 and Q = gO135 - gO45
//   E = H[gm] V[g] gO0 + H[g] (V[gm] gO90 - c45 V[g] P) + H[gc] V[gc] P + H[gs] V[gs] Q:
// 117 multiply-adds per position instead of the 676 of four 13x13 kernels, whose LDS reads
// (two 16-byte reads a tap) bound the launch: 37 us for one 640x480 frame, 33 us for eight of them here (38 with
// one output a thread and the staging loads waited for one at a time).
// One 16x16 tile of p per workgroup: gO0, gO90, P and Q of the tile plus twice the radius
// interleaved in LDS, the vertical pass over the rows of q the tile needs (its own, and the
// outside strips of a tile on the border), the horizontal pass, then the fold.
// RC: the radius when known at compile time (0: read from the stream description, with
// zero-padded taps).
constexpr int GT = 16;
template <int RC>
__global__ __launch_bounds__(SP_BLOCK) void k_pa_gabor_t(PaDesc A, const StreamDesc* __restrict__ sds) {
  constexpr int RM = RC ? RC : SP_PA_R, NS = GT + 4 * RM, NQ = GT + 2 * RM;
  // three rows and one value more than staged: read for outputs past the last, which are not stored
  __shared__ float4 st[(NS + 3) * NS];   // gO0, gO90, P, Q; then E [NQ][NQ]
  __shared__ float4 vp[NQ * NS + 1];     // V[g] gO0, V[gm] gO90 - c45 V[g] P, V[gc] P, V[gs] Q
  const int z = blockIdx.z, l = A.ul[blockIdx.y];
  const StreamDesc& sd = sds[z];
  const int h = sd.Hl[l], w = sd.Wl[l], R = RC ? RC : sd.gr;
  const uint32_t n = (uint32_t)h * (uint32_t)w;
  const int ntx = (w + GT - 1) / GT;
  if ((int)blockIdx.x >= ntx * ((h + GT - 1) / GT)) return;   // the level has fewer tiles
  const int ty0 = (blockIdx.x / ntx) * GT, tx0 = (blockIdx.x % ntx) * GT;
  const int E = GT + 4 * R, oy = ty0 - 2 * R, ox = tx0 - 2 * R;
  float* gI = slot(A.gX[l], A, z);
  const gp<const float> gO = G((const float*)gI + 3 * (size_t)n);
  const int py = ty0 + (int)(threadIdx.x >> 4), px = tx0 + (int)(threadIdx.x & 15);
  const float base = G((const float*)gI)[(uint32_t)min(py, h - 1) * (uint32_t)w + (uint32_t)min(px, w - 1)];   // added to last
  {
    // every load of the tile in flight at once: one at a time their latency was most of the launch
    constexpr int NI = (NS * NS + SP_BLOCK - 1) / SP_BLOCK;
    float v[NI][4];
    bool in[NI];
    Walk2 wk(threadIdx.x, E);
#pragma unroll
    for (int k = 0; k < NI; ++k, wk.next()) {
      const int y = oy + wk.r, x = ox + wk.c;
      in[k] = y >= 0 && y < h && x >= 0 && x < w;
      const uint32_t o = (uint32_t)clampi(y, 0, h - 1) * (uint32_t)w + (uint32_t)clampi(x, 0, w - 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[k][q] = gO[q * n + o];
    }
    Walk2 wl(threadIdx.x, E);
#pragma unroll
    for (int k = 0; k < NI; ++k, wl.next())
      if (k * SP_BLOCK + (int)threadIdx.x < E * E)
        st[wl.r * NS + wl.c] = in[k] ? make_float4(v[k][0], v[k][2], v[k][1] + v[k][3], v[k][3] - v[k][1])
                                     : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();
  // the q the tile needs: its own positions, and the outside strips on the level's borders
  const int th = min(GT, h - ty0), tw = min(GT, w - tx0);
  const int qy0 = ty0 == 0 ? -R : ty0, qy1 = ty0 + th - 1 + (ty0 + th == h ? R : 0);
  const int qx0 = tx0 == 0 ? -R : tx0, qx1 = tx0 + tw - 1 + (tx0 + tw == w ? R : 0);
  const int nqx = qx1 - qx0 + 1, nqy = qy1 - qy0 + 1;
  const int cx0 = qx0 - R, ncx = nqx + 2 * R;   // columns of the vertical pass
  // tap t of the 1-D factors g, gm, gc, gs: uniform scalars; position q reads q - (t - R).  For a
  // run-time radius the table is zero beyond 2 R + 1 and the position stays in the staged region.
  constexpr int NT = 2 * RM + 1;
  const float c45 = sd.c45;
  // vertical pass, VB consecutive rows of a column per thread: VB + 2 R reads for VB outputs
  constexpr int VB = 4, HB = 2;
  {
    const int ng = (nqy + VB - 1) / VB;
    Walk2 wk(threadIdx.x, ncx);
    for (int i = threadIdx.x; i < ng * ncx; i += SP_BLOCK, wk.next()) {
      const int q0 = wk.r * VB;
      // output row q0 + u, tap t reads column row q0 + u + R - t; m = u + 2 R - t runs over what they share
      const float4* col = st + (qy0 + q0 - R - oy) * NS + (cx0 + wk.c - ox);
      float a[VB], b[VB], gP[VB], c[VB], e[VB];
#pragma unroll
      for (int u = 0; u < VB; ++u) a[u] = b[u] = gP[u] = c[u] = e[u] = 0.f;
#pragma unroll
      for (int m = NT + VB - 2; m >= 0; --m) {   // taps in increasing order for every output
        if (RC == 0 && m > 2 * R + VB - 1) continue;
        const float4 v = col[m * NS];
#pragma unroll
        for (int u = 0; u < VB; ++u) {
          const int t = u + 2 * R - m;
          if (t < 0 || t > 2 * R) continue;
          a[u] = fmaf(sd.gf[0][t], v.x, a[u]);
          b[u] = fmaf(sd.gf[1][t], v.y, b[u]);
          gP[u] = fmaf(sd.gf[0][t], v.z, gP[u]);
          c[u] = fmaf(sd.gf[2][t], v.z, c[u]);
          e[u] = fmaf(sd.gf[3][t], v.w, e[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < VB; ++u)
        if (q0 + u < nqy) vp[(q0 + u) * NS + wk.c] = make_float4(a[u], b[u] - c45 * gP[u], c[u], e[u]);
    }
  }
  __syncthreads();
  float* eq = reinterpret_cast<float*>(st);   // the staged gradients are no longer read
  {
    const int ng = (nqx + HB - 1) / HB;
    Walk2 wk(threadIdx.x, ng);
    for (int i = threadIdx.x; i < nqy * ng; i += SP_BLOCK, wk.next()) {
      const int q0 = wk.c * HB;
      const float4* row = vp + wk.r * NS + q0;
      float e[HB];
#pragma unroll
      for (int u = 0; u < HB; ++u) e[u] = 0.f;
#pragma unroll
      for (int m = NT + HB - 2; m >= 0; --m) {
        if (RC == 0 && m > 2 * R + HB - 1) continue;
        const float4 v = row[m];
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          const int t = u + 2 * R - m;
          if (t < 0 || t > 2 * R) continue;
          e[u] = fmaf(sd.gf[1][t], v.x, fmaf(sd.gf[0][t], v.y, fmaf(sd.gf[2][t], v.z, fmaf(sd.gf[3][t], v.w, e[u]))));
        }
      }
#pragma unroll
      for (int u = 0; u < HB; ++u)
        if (q0 + u < nqx) eq[wk.r * NQ + q0 + u] = e[u];
    }
  }
  __syncthreads();
  if (py >= h || px >= w) return;
  const int fy0 = py == 0 ? -R : py, fy1 = py == h - 1 ? h - 1 + R : py;
  const int fx0 = px == 0 ? -R : px, fx1 = px == w - 1 ? w - 1 + R : px;
  float acc = 0.f;
  for (int qy = fy0; qy <= fy1; ++qy)
    for (int qx = fx0; qx <= fx1; ++qx) acc += eq[(qy - qy0) * NQ + (qx - qx0)];
  G(gI)[(uint32_t)py * (uint32_t)w + (uint32_t)px] = base + acc;
}

// Level 1 back to the frames: the last transposed pyramid step (2x2 pixels per thread from nine
// level-1 values a channel, never stored) and the level-0 features.  Frame t0 + z gets its own
// part and the motion part of frame t0 + z + 1 when that frame is in the launch; the first
// frame adds its motion part to frame t0 - 1, finished by the launch before.  Storing the four
// level-0 planes took two more passes over 16 bytes a pixel (14.7 + 4.8 us a 640x480 frame).
__global__ __launch_bounds__(SP_BLOCK) void k_pa_feat(PaDesc A, const StreamDesc* __restrict__ sds,
                                                      const uint8_t* __restrict__ frames, float* __restrict__ grad, int t0, int nz) {
  __shared__ float sh4[4];
  const int z = blockIdx.z, t = t0 + z;
  const StreamDesc& sd = sds[z];
  const int H = sd.H, W = sd.W, h1 = sd.Hl[1], w1 = sd.Wl[1];
  const size_t hw3 = 3 * (size_t)H * W;
  const int i = blockIdx.x * SP_BLOCK + threadIdx.x;
  const bool act = i < h1 * w1;
  const int q = min(i, h1 * w1 - 1) / w1, r = min(i, h1 * w1 - 1) - q * w1;
  const QuadT Q(q, r, H, W, h1, w1);
  const size_t n1 = (size_t)h1 * w1;
  const float* g1 = slot(A.gX[1], A, z);
  const bool next = z + 1 < nz;   // uniform
  // every gradient and byte is requested before the colour maximum is reduced; two pixels of a row
  // are six bytes, three 2-byte loads and three 8-byte stores where rows allow
  float v[5][3][3];
  Q.load(G(g1), v[0]);
  Q.load(G(g1 + n1), v[1]);
  Q.load(G(g1 + 2 * n1), v[2]);
  Q.load(G(g1 + 7 * n1), v[3]);
  if (next) Q.load(G((const float*)slot(A.gX[1], A, z + 1) + 7 * n1), v[4]);
  const bool pairs = (W & 1) == 0 && (reinterpret_cast<uintptr_t>(frames) & 1) == 0 && (reinterpret_cast<uintptr_t>(grad) & 7) == 0;
  const gp<const uint8_t> rgb = G(frames + (size_t)t * hw3);
  uint32_t c0[2][2][3], cp[2][2], cn[2][2];   // the frame's bytes, the sums of the previous and the next
  {
    auto two = [&](gp<const uint8_t> f, int y, uint32_t (&c)[2][3]) {
      const uint32_t o = 3u * ((uint32_t)min(y, H - 1) * (uint32_t)W + (uint32_t)(2 * r));
      if (pairs) {
        uint32_t u[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) u[k] = ((gp<const uint16_t>)(f + o))[k];
        c[0][0] = u[0] & 255u;
        c[0][1] = u[0] >> 8;
        c[0][2] = u[1] & 255u;
        c[1][0] = u[1] >> 8;
        c[1][1] = u[2] & 255u;
        c[1][2] = u[2] >> 8;
      } else {
        const uint32_t o1 = 2 * r + 1 < W ? o + 3u : o;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          c[0][k] = f[o + k];
          c[1][k] = f[o1 + k];
        }
      }
    };
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      two(rgb, 2 * q + a, c0[a]);
      uint32_t c[2][3];
      cp[a][0] = cp[a][1] = cn[a][0] = cn[a][1] = 0u;
      if (t > 0) {
        two(rgb - hw3, 2 * q + a, c);
        cp[a][0] = c[0][0] + c[0][1] + c[0][2];
        cp[a][1] = c[1][0] + c[1][1] + c[1][2];
      }
      if (next) {
        two(rgb + hw3, 2 * q + a, c);
        cn[a][0] = c[0][0] + c[0][1] + c[0][2];
        cn[a][1] = c[1][0] + c[1][1] + c[1][2];
      }
    }
  }
  // the frame's colour maximum from the partials (integers below 2^24: exact as floats)
  uint32_t m = 0;
  for (int k = threadIdx.x; k < sd.n_rgb; k += SP_BLOCK) m = max(m, G((const uint32_t*)sd.rgb_max_part)[k]);
  const uint32_t smax = (uint32_t)block_reduce<OpMax>((float)m, sh4);
  if (!act) return;
  float gI[2][2], gRG[2][2], gBY[2][2], gM[2][2], gN[2][2];
  Q.apply(v[0], gI);
  Q.apply(v[1], gRG);
  Q.apply(v[2], gBY);
  Q.apply(v[3], gM);
  if (next) Q.apply(v[4], gN);
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int y = 2 * q + a;
    if (y >= H) continue;
    float g6[2][3];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t R8 = c0[a][b][0], G8 = c0[a][b][1], B8 = c0[a][b][2];
      const int s8 = (int)(R8 + G8 + B8);
      const float rr = R8 * (1.f / 255.f), gg_ = G8 * (1.f / 255.f), bb = B8 * (1.f / 255.f);
      const float I = (rr + gg_ + bb) / 3.f;
      const bool chrom = 10u * (R8 + G8 + B8) > smax;
      float gIt = gI[a][b];
      if (t > 0) {
        // the sign of I_t - I_{t-1}, exact from the byte sums
        const int dm = s8 - (int)cp[a][b];
        const float sg = dm > 0 ? gM[a][b] : (dm < 0 ? -gM[a][b] : 0.f);
        gIt += sg;
        if (z == 0 && 2 * r + b < W) {
          const gp<float> gp_ = G(grad + (size_t)(t - 1) * hw3 + 3 * ((size_t)y * W + 2 * r + b));
          const float gpv = -sg / 3.f / 255.f;
          gp_[0] += gpv;
          gp_[1] += gpv;
          gp_[2] += gpv;
        }
      }
      float gr = 0.f, gg = 0.f, gb = 0.f;
      if (chrom) {
        const float ri = 1.f / I;
        // the branches of the opponent channels, exact from the bytes (r' = R / I with I > 0)
        const int r8 = (int)R8, g8 = (int)G8, b8 = (int)B8;
        const float vRG = gRG[a][b], vBY = gBY[a][b];
        const float guR = 2 * r8 - g8 - b8 > 0 ? vRG : 0.f, guG = 2 * g8 - r8 - b8 > 0 ? -vRG : 0.f;
        const float guB = 2 * b8 - r8 - g8 > 0 ? vBY : 0.f, guY = min(r8, g8) - b8 > 0 ? -vBY : 0.f;
        float grp = guR - 0.5f * guG - 0.5f * guB;
        float ggp = -0.5f * guR + guG - 0.5f * guB;
        const float gbp = -0.5f * guR - 0.5f * guG + guB - guY;
        if (r8 <= g8) grp += guY;
        else ggp += guY;
        gr = grp * ri;
        gg = ggp * ri;
        gb = gbp * ri;
        gIt -= (grp * rr + ggp * gg_ + gbp * bb) * ri * ri;
      }
      gr = (gr + gIt / 3.f) / 255.f;
      gg = (gg + gIt / 3.f) / 255.f;
      gb = (gb + gIt / 3.f) / 255.f;
      if (next) {
        const int dm = (int)cn[a][b] - s8;
        const float sg = dm > 0 ? gN[a][b] : (dm < 0 ? -gN[a][b] : 0.f);
        const float gpv = -sg / 3.f / 255.f;
        gr += gpv;
        gg += gpv;
        gb += gpv;
      }
      g6[b][0] = gr;
      g6[b][1] = gg;
      g6[b][2] = gb;
    }
    const gp<float> go = G(grad + (size_t)t * hw3 + 3 * ((size_t)y * W + 2 * r));
    if (pairs) {
      const gp<Pair> go2 = (gp<Pair>)go;
      go2[0] = Pair{g6[0][0], g6[0][1]};
      go2[1] = Pair{g6[0][2], g6[1][0]};
      go2[2] = Pair{g6[1][1], g6[1][2]};
    } else {
#pragma unroll
      for (int b = 0; b < 2; ++b)
        if (2 * r + b < W) {
          go[3 * b] = g6[b][0];
          go[3 * b + 1] = g6[b][1];
          go[3 * b + 2] = g6[b][2];
        }
    }
  }
}

// The io table of a clip's steps, for the frame slots here and in sp_run_clip (among the step kernels it
// moved those in their code object: 32 streams 272.3 us a step against 270.2).
// One thread a step: 1.4 us for 8 steps, 4.8 for 120.  A table copied from pinned memory made the call wait
// for the copy of the one before.
__global__ __launch_bounds__(SP_CLIP_IO) void k_clip_io(ClipIO a) {
  const int s = threadIdx.x;
  if (s >= a.n) return;
  auto at = [s](const ClipOut& o) { return o.p ? o.p + s * o.stride : nullptr; };
  StepIO io{};
  io.rgb_prev = a.rgb[s];
  io.rgb = a.rgb[s + 1];
  io.S_out = at(a.S_out);
  io.C_out = at(a.C_out);
  io.S_tape = at(a.S_tape);
  io.fbar = at(a.fbar);
  io.np_tape = at(a.np_tape);
  io.pairwise = at(a.pairwise);
  io.beta_out = at(a.beta_out);
  a.io[s] = io;
}

inline int blocks(long long n, int per = SP_BLOCK) { return (int)((n + per - 1) / per); }

}  // namespace

hipError_t sp_pixel_adjoint(const PaDesc& A, const StreamDesc* sds, const StreamDesc& g, int t0, int nz,
                            const uint8_t* frames, const float* gs, const float* S, const float* ms, const float* fbar,
                            float* grad, hipStream_t st) {
  if (nz <= 0) return hipSuccess;
  const dim3 b(SP_BLOCK);
  auto n_l = [&](int l) { return g.Hl[l] * g.Wl[l]; };
  auto grid = [&](int x, int y) { return dim3(x, y, nz); };
  const int cm = g.c_max, nc = n_l(cm), nF = SP_NCH * g.n_pairs;
  int maxc = 0, maxh = 0, maxs = 0, maxt = 0;
  for (int p = 0; p < g.n_pairs; ++p) {
    maxc = std::max(maxc, n_l(g.pc[p]));
    maxh = std::max(maxh, g.Hl[g.pc[p]]);
    maxs = std::max(maxs, n_l(g.ps[p]));
  }
  for (int q = 0; q < A.n_ul; ++q) maxt = std::max(maxt, blocks(g.Hl[A.ul[q]], GT) * blocks(g.Wl[A.ul[q]], GT));
  hipLaunchKernelGGL(k_pa_gs, grid(blocks(nc), 1), b, 0, st, A, gs, S, ms, nc, g.flat_tol);
  hipLaunchKernelGGL(k_pa_gs_fix, grid(1, 1), b, 0, st, A, gs, ms, nc, blocks(nc), g.flat_tol);
  hipLaunchKernelGGL(k_pa_nmm, grid(blocks(nc, TILE), SP_NCH), b, 0, st, A, sds, fbar);
  hipLaunchKernelGGL(k_pa_nstrip, grid(blocks(g.Hl[cm], 8), SP_NCH), b, 0, st, A, sds, fbar, 0, g.flat_tol);
  hipLaunchKernelGGL(k_pa_nfin, grid(1, SP_NCH), b, 0, st, A, sds, fbar, 0, g.flat_tol);
  hipLaunchKernelGGL(k_pa_napply, grid(blocks(nc, TILE), SP_NCH), b, 0, st, A, sds, fbar);
  for (int l = cm - 1; l >= g.c_min; --l)
    hipLaunchKernelGGL(k_pa_reduce_t, grid(blocks(n_l(l + 1)), SP_NCH), b, 0, st, A,
                       (const float*)(l + 1 == cm ? A.gfbar : A.gN[l + 1]), A.gN[l], g.Hl[l], g.Wl[l], g.Hl[l + 1],
                       g.Wl[l + 1], 0);
  hipLaunchKernelGGL(k_pa_csmap, grid(blocks(maxc, TILE), nF), b, 0, st, A, sds);
  hipLaunchKernelGGL(k_pa_nstrip, grid(blocks(maxh, 8), nF), b, 0, st, A, sds, fbar, SP_NCH, g.flat_tol);
  hipLaunchKernelGGL(k_pa_nfin, grid(1, nF), b, 0, st, A, sds, fbar, SP_NCH, g.flat_tol);
  hipLaunchKernelGGL(k_pa_csadj, grid(blocks(maxc, TILE), SP_NCH * A.n_cl), b, 0, st, A, sds);
  hipLaunchKernelGGL(k_pa_up_t, grid(blocks(maxs, UPT_E), SP_NCH * A.n_sl), b, 0, st, A, sds);
  if (g.gr == 6)
    hipLaunchKernelGGL(k_pa_gabor_t<6>, grid(maxt, A.n_ul), b, 0, st, A, sds);
  else
    hipLaunchKernelGGL(k_pa_gabor_t<0>, grid(maxt, A.n_ul), b, 0, st, A, sds);
  for (int l = g.top; l >= 2; --l)   // a level no pair uses starts from the level above
    hipLaunchKernelGGL(k_pa_reduce_t, grid(blocks(n_l(l)), 4), b, 0, st, A, (const float*)A.gX[l], A.gX[l - 1], g.Hl[l - 1],
                       g.Wl[l - 1], g.Hl[l], g.Wl[l], (int)((g.used >> (l - 1)) & 1u));
  hipLaunchKernelGGL(k_pa_feat, grid(blocks(n_l(1)), 1), b, 0, st, A, sds, frames, grad, t0, nz);
  return hipGetLastError();
}

hipError_t sp_launch_clip_io(const ClipIO& a, hipStream_t st) {
  hipLaunchKernelGGL(k_clip_io, dim3(1), dim3(SP_CLIP_IO), 0, st, a);
  return hipGetLastError();
}
