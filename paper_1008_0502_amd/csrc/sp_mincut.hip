// Minimum cut of the MRF (Section 4: the MAP labelling is the minimum s-t cut of the graph
// with one vertex per pixel, t-links c(s, v) and c(v, t) from the unary costs and a pair of
// equal directed n-links between 8-neighbours), on integer capacities q(c) =
// rint(c * scale) clamped to [0, 2^24], so the flow is exact.  The source side is the object:
// a pixel on the sink side pays U0, one on the source side U1.
//
// Push-relabel on the grid.  Each t-link pair is saturated up front (min(U0, U1) flows
// source -> pixel -> sink), leaving an excess U0 - min at the pixel and a residual U1 - min to
// the sink.  Then rounds of
//   * a global relabel: every height set to the exact distance to the sink in the residual
//     graph, by Bellman-Ford relaxation over 32x32 tiles in LDS (each pass relaxes its tile to
//     a fixed point against the neighbouring tiles' heights; passes repeat until none lowers a
//     height), and a count of the pixels with excess that can reach the sink;
//   * launches of push / relabel cycles over the tiles that hold such pixels: a pixel with
//     excess pushes to its lowest residual neighbour (or the sink) when it is higher, else lifts
//     itself above it.  A tile's excess, heights and residual capacities stay in registers and
//     LDS for all its cycles; a pixel only takes away what it holds itself, pushes across a
//     tile's border and the write-back add by device-scope atomics, so nothing is lost and
//     capacities never go negative whatever the interleaving; stale heights of neighbouring
//     tiles only delay work.
// The rounds end when no pixel with excess can reach the sink: the preflow is then maximum,
// and the pixels that can still reach the sink form the smallest sink side of all minimum
// cuts (the same for every maximum flow); the others are the object.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>

#include <algorithm>

#include "sp_internal.h"
#include "sp_kernels.h"
#include "sp_device.h"

namespace {

// Offsets of the n-link directions E, W, S, N, SE, NW, SW, NE.
__device__ __forceinline__ int DYf(int d) { return (d == 2 || d == 4 || d == 6) ? 1 : ((d == 3 || d == 5 || d == 7) ? -1 : 0); }
__device__ __forceinline__ int DXf(int d) { return (d == 0 || d == 4 || d == 7) ? 1 : ((d == 1 || d == 5 || d == 6) ? -1 : 0); }

__device__ __forceinline__ int32_t quant(float c, float scale) {
  float v = rintf(c * scale);
  if (!(v > 0.f)) return 0;   // negative and NaN
  return v >= (float)SP_CUT_CAPMAX ? SP_CUT_CAPMAX : (int32_t)v;
}

// Capacities and the saturated t-links.  The flow goes to one partial per workgroup (1200
// workgroups adding to one address took 20.6 us of a 640x480 cut, 7.7 us now); the counters start at
// zero.  The push tiles' flags hold anything until a cut's first relabel pass sets them all.
__global__ __launch_bounds__(SP_BLOCK) void k_cut_init(CutIO io) {
  __shared__ unsigned long long sh4[4];
  const int n = io.H * io.W;
  unsigned long long acc = 0;
  if (blockIdx.x == 0) {
    for (int k = threadIdx.x; k < SP_CUT_FLOW; k += SP_BLOCK) io.flow[k] = 0ull;
    for (int k = threadIdx.x; k < 2 * SP_CUT_CTL; k += SP_BLOCK) io.ctl[k] = 0;
  }
  for (int i = blockIdx.x * SP_BLOCK + threadIdx.x; i < n; i += gridDim.x * SP_BLOCK) {
    const int y = i / io.W, x = i - (i / io.W) * io.W;
    const int32_t cs = quant(io.unary[i], io.scale), ct = quant(io.unary[n + i], io.scale);
    const int32_t m = min(cs, ct);
    acc += (unsigned long long)m;
    io.e[i] = cs - m;
    io.rt[i] = ct - m;
    io.h[i] = ct - m > 0 ? 1 : 2;   // a lower bound of every distance to the sink
    // the capacity of a pair sits in the pairwise plane of its upper (or left) pixel
    const float* pw = io.pairwise;
    int32_t c[8];
    c[0] = x + 1 < io.W ? quant(pw[i], io.scale) : 0;                                       // E
    c[1] = x > 0 ? quant(pw[i - 1], io.scale) : 0;                                          // W
    c[2] = y + 1 < io.H ? quant(pw[n + i], io.scale) : 0;                                   // S
    c[3] = y > 0 ? quant(pw[n + i - io.W], io.scale) : 0;                                   // N
    c[4] = (y + 1 < io.H && x + 1 < io.W) ? quant(pw[2 * n + i], io.scale) : 0;             // SE
    c[5] = (y > 0 && x > 0) ? quant(pw[2 * n + i - io.W - 1], io.scale) : 0;                // NW
    c[6] = (y + 1 < io.H && x > 0) ? quant(pw[3 * n + i], io.scale) : 0;                    // SW
    c[7] = (y > 0 && x + 1 < io.W) ? quant(pw[3 * n + i - io.W + 1], io.scale) : 0;         // NE
#pragma unroll
    for (int d = 0; d < 8; ++d) io.r[(size_t)d * n + i] = c[d];
  }
  acc = block_sum_u64(acc, sh4);
  if (threadIdx.x == 0) io.flow_part[blockIdx.x] = acc;
}

// One tile of the global relabel.  Region: the tile and a one-pixel ring; the ring keeps
// the heights its owners had when read (an upper bound, which is all relaxation needs).  Pass
// io.pass counts the lowered heights and the active pixels in slot pass % SP_CUT_CTL; a pass
// after one that lowered nothing hands its count on and ends (the host enqueues passes without
// waiting for each).  A pixel at height 1 cannot be lowered, so only the others load their eight
// residuals: most pixels of a frame still have a way to the sink (11.7 us with every residual
// loaded, 7.7 us now at 640x480).
constexpr int RB = SP_CUT_T * SP_CUT_T;
__global__ __launch_bounds__(RB) void k_cut_relabel(CutIO io) {
  constexpr int RN = SP_CUT_T + 2, SUB = SP_CUT_T / SP_CUT_PT;   // push tiles per edge of a tile
  __shared__ int32_t hl[RN * RN];
  __shared__ int act_sh[SUB * SUB];
  int32_t* const changed = io.ctl;
  int32_t* const active = io.ctl + SP_CUT_CTL;
  const int slot = io.pass & (SP_CUT_CTL - 1), before = (io.pass - 1) & (SP_CUT_CTL - 1);
  if (blockIdx.x == 0 && threadIdx.x == 0) {   // a slot no queued pass uses, for later
    const int later = (io.pass + SP_CUT_CTL / 2) & (SP_CUT_CTL - 1);
    changed[later] = 0;
    active[later] = 0;
  }
  if (!io.first && changed[before] == 0) {   // uniform over the launch
    if (blockIdx.x == 0 && threadIdx.x == 0) active[slot] = active[before];
    return;
  }
  const int ntx = (io.W + SP_CUT_T - 1) / SP_CUT_T;
  const int ty0 = (blockIdx.x / ntx) * SP_CUT_T, tx0 = (blockIdx.x % ntx) * SP_CUT_T;
  const int n = io.H * io.W;
  for (int k = threadIdx.x; k < RN * RN; k += RB) {
    const int y = ty0 - 1 + k / RN, x = tx0 - 1 + k % RN;
    int32_t v = SP_CUT_INF;
    if (y >= 0 && y < io.H && x >= 0 && x < io.W) {
      const int i = y * io.W + x;
      v = io.reset ? (io.rt[i] > 0 ? 1 : SP_CUT_INF) : io.h[i];
    }
    hl[k] = v;
  }
  if (threadIdx.x < SUB * SUB) act_sh[threadIdx.x] = 0;
  const int ly = threadIdx.x / SP_CUT_T, lx = threadIdx.x % SP_CUT_T;
  const int y = ty0 + ly, x = tx0 + lx, i = y * io.W + x;
  const bool in = y < io.H && x < io.W;
  const int32_t e = in ? io.e[i] : 0;
  volatile int32_t* const c = hl + (ly + 1) * RN + lx + 1;
  __syncthreads();
  // the residual n-links of a pixel that may be lowered, as a bit mask (bit d: r(v, d) > 0)
  const int32_t h0 = c[0];
  uint32_t mask = 0;
  if (in && h0 > 1) {
    int32_t r[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) r[d] = io.r[(size_t)d * n + i];
#pragma unroll
    for (int d = 0; d < 8; ++d) mask |= r[d] > 0 ? 1u << d : 0u;
  }
  // four sweeps between two looks at whether any pixel was lowered (a pixel reads whatever
  // its neighbours hold at that time: heights only fall towards the fixed point)
  int32_t v = h0;
  for (int it = 0; it < RN * RN; it += 4) {
    const int32_t was = v;
    if (mask) {
#pragma unroll 1
      for (int sub = 0; sub < 4; ++sub) {
        int32_t best = v;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          const int32_t u = c[DYf(d) * RN + DXf(d)] + 1;
          best = min(best, (mask & (1u << d)) ? u : SP_CUT_INF);
        }
        if (best < v) {
          v = best;
          c[0] = v;
        }
      }
    }
    if (!__syncthreads_or(v != was)) break;
  }
  // write back the lowered heights (all of them in a reset pass); count the pixels with
  // excess that reach the sink, per push tile
  if (in && (io.reset || v != h0)) io.h[i] = v;
  const bool act = in && v < SP_CUT_INF && e > 0;
  // a wavefront covers whole rows of the tile, so lanes with the same column block count together
  static_assert(64 % SP_CUT_T == 0 && SP_CUT_PT % (64 / SP_CUT_T) == 0, "a wavefront stays in one row of push tiles");
  const unsigned long long votes = __ballot(act);
  if (lx % SP_CUT_PT == 0 && (lane_id() < SP_CUT_T)) {
    unsigned long long mine = 0;
#pragma unroll
    for (int q = 0; q < 64 / SP_CUT_T; ++q) mine |= ((1ull << SP_CUT_PT) - 1) << (q * SP_CUT_T + lx);
    const int cnt = __popcll(votes & mine);
    if (cnt) atomicAdd(&act_sh[(ly / SP_CUT_PT) * SUB + lx / SP_CUT_PT], cnt);
  }
  const bool any = __syncthreads_or(v != h0);
  if (threadIdx.x < SUB * SUB) {
    const int py = ty0 / SP_CUT_PT + threadIdx.x / SUB, px = tx0 / SP_CUT_PT + threadIdx.x % SUB;
    const int npx = (io.W + SP_CUT_PT - 1) / SP_CUT_PT, npy = (io.H + SP_CUT_PT - 1) / SP_CUT_PT;
    if (py < npy && px < npx) io.tile[py * npx + px] = act_sh[threadIdx.x];
  }
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int q = 0; q < SUB * SUB; ++q) tot += act_sh[q];
    if (tot) atomicAdd(&active[slot], tot);
    if (any) atomicOr(&changed[slot], 1);
  }
}

// Push / relabel cycles of one tile, one thread per pixel, until no pixel of the tile has excess
// to move or io.cycles have run.  A cycle: every active pixel pushes or lifts (a push inside the
// tile goes to the pusher's outbox word), then every pixel takes what its neighbours' outboxes
// hold for it.  Tiles whose flag is zero end at once (io.first: the flags are not set yet and a
// tile looks for active pixels itself); a push across the border sets the neighbour's flag for
// the next launch.  Bound by the instructions of the few CUs that hold active tiles: a cycle on
// global memory with an atomic per push took 0.73 us, one of a 32x32 tile in LDS 1.4 us (four
// wavefronts share each SIMD), one of a 16x16 tile 1.0 us.
constexpr int PT = SP_CUT_PT, PB = PT * PT;
__global__ __launch_bounds__(PB) void k_cut_push(CutIO io) {
  constexpr int RN = PT + 2;
  __shared__ uint32_t hl[RN * RN];    // heights, packed
  __shared__ uint32_t box[RN * RN];   // pushed amount << 4 | direction + 1 (amounts < 2^26)
  __shared__ int wpush[PB / 64 + 2];  // the wavefront (whole rows of the tile) pushed in this cycle
  __shared__ unsigned long long sunk_sh;
  __shared__ int go;
  if (threadIdx.x == 0) {
    go = io.first ? 1 : atomicExch(&io.tile[blockIdx.x], 0);
    sunk_sh = 0ull;
  }
  if (threadIdx.x < PB / 64 + 2) wpush[threadIdx.x] = 0;
  __syncthreads();
  if (go == 0) return;   // uniform
  constexpr uint32_t INF = SP_CUT_HINF;
  const int ntx = (io.W + PT - 1) / PT;
  const int tyi = blockIdx.x / ntx, txi = blockIdx.x % ntx;
  const int ty0 = tyi * PT, tx0 = txi * PT;
  const int n = io.H * io.W;
  const int ly = threadIdx.x / PT, lx = threadIdx.x % PT;
  const int y = ty0 + ly, x = tx0 + lx, li = (ly + 1) * RN + lx + 1;
  const bool in = y < io.H && x < io.W;
  const int i = in ? y * io.W + x : 0;
  int32_t e = in ? io.e[i] : 0, rt = in ? io.rt[i] : 0;
  if (io.first && !__syncthreads_or(e > 0)) return;   // uniform (the first heights are all finite)
  for (int k = threadIdx.x; k < RN * RN; k += PB) {
    const int yy = ty0 - 1 + k / RN, xx = tx0 - 1 + k % RN;
    const int32_t v = (yy >= 0 && yy < io.H && xx >= 0 && xx < io.W) ? io.h[yy * io.W + xx] : SP_CUT_INF;
    hl[k] = cut_pack(v);
    box[k] = 0u;
  }
  // key[d]: d where the residual in direction d is positive, else above every height
  int32_t r[8], r0[8];
  uint32_t key[8];
#pragma unroll
  for (int d = 0; d < 8; ++d) r[d] = r0[d] = in ? io.r[(size_t)d * n + i] : 0;
#pragma unroll
  for (int d = 0; d < 8; ++d) key[d] = r[d] > 0 ? d : INF;
  const int32_t e0 = e, rt0 = rt;
  const int w = wave_id();
  __syncthreads();
  uint32_t h = hl[li];
  const uint32_t h0 = h;
  unsigned long long sunk = 0;
  uint32_t out_tiles = 0;   // neighbouring tiles pushed to: bit (dy + 1) * 3 + dx + 1
  for (int cyc = 0; cyc < io.cycles; ++cyc) {
    uint32_t word = 0u;
    if (e > 0 && h < INF) {
      if (rt > 0) {   // the sink, at height 0
        const int32_t delta = min(e, rt);
        e -= delta;
        rt -= delta;
        sunk += (unsigned long long)delta;
      } else {
        uint32_t best = INF;
#pragma unroll
        for (int d = 0; d < 8; ++d) best = min(best, hl[li + DYf(d) * RN + DXf(d)] | key[d]);
        if (best >= INF) {
          h = INF;   // no residual path: it cannot reach the sink
          hl[li] = h;
        } else if (h > (best & ~7u)) {
          const int dm = best & 7u;
          int32_t cap = 0;
          int dy = 0, dx = 0;
#pragma unroll
          for (int d = 0; d < 8; ++d)
            if (d == dm) {
              cap = r[d];
              dy = DYf(d);
              dx = DXf(d);
            }
          const int32_t delta = min(e, cap);
          e -= delta;
#pragma unroll
          for (int d = 0; d < 8; ++d)
            if (d == dm) {
              r[d] -= delta;
              key[d] = r[d] > 0 ? d : INF;
            }
          if ((unsigned)(ly + dy) < (unsigned)PT && (unsigned)(lx + dx) < (unsigned)PT) {
            word = ((uint32_t)delta << 4) | (uint32_t)(dm + 1);
          } else {
            const int j = i + dy * io.W + dx;
            atomicAdd(io.r + (size_t)(dm ^ 1) * n + j, delta);
            atomicAdd(io.e + j, delta);
            const int by = ly + dy < 0 ? -1 : (ly + dy >= PT ? 1 : 0), bx = lx + dx < 0 ? -1 : (lx + dx >= PT ? 1 : 0);
            out_tiles |= 1u << ((by + 1) * 3 + bx + 1);
          }
        } else {
          h = (best & ~7u) + 8u;
          hl[li] = h;
        }
      }
    }
    box[li] = word;
    const bool wp = __any(word != 0u);
    if (lane_id() == 0) wpush[w + 1] = wp;
    __syncthreads();
    if (wpush[w] | wpush[w + 1] | wpush[w + 2]) {   // uniform over the wavefront
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        const uint32_t o = box[li + DYf(d) * RN + DXf(d)];   // the ring's words stay 0
        if ((o & 15u) == (uint32_t)((d ^ 1) + 1)) {
          r[d] += (int32_t)(o >> 4);
          key[d] = d;
          e += (int32_t)(o >> 4);
        }
      }
    }
    if ((cyc & 3) == 3) {
      if (!__syncthreads_or(e > 0 && h < INF)) break;
    } else {
      __syncthreads();
    }
  }
  // write back what changed, by addition where neighbouring tiles add too
  if (in) {
    if (e != e0) atomicAdd(io.e + i, e - e0);
#pragma unroll
    for (int d = 0; d < 8; ++d)
      if (r[d] != r0[d]) atomicAdd(io.r + (size_t)d * n + i, r[d] - r0[d]);
    if (rt != rt0) io.rt[i] = rt;
    if (h != h0) io.h[i] = cut_unpack(h);
  }
  if (sunk) atomicAdd(&sunk_sh, sunk);
  const bool more = __syncthreads_or(e > 0 && h < INF);
#pragma unroll
  for (int b = 0; b < 9; ++b)
    if ((out_tiles >> b) & 1u) atomicOr(&io.tile[(tyi + b / 3 - 1) * ntx + txi + b % 3 - 1], 1);
  if (threadIdx.x == 0) {
    if (more) atomicOr(&io.tile[blockIdx.x], 1);
    if (sunk_sh) atomicAdd(&io.flow[blockIdx.x & (SP_CUT_FLOW - 1)], sunk_sh);
  }
}

// The labels of the current heights and the flow so far, and the last pass's counters for the
// host (the result is final when both are zero).
__global__ __launch_bounds__(SP_BLOCK) void k_cut_labels(CutIO io, int nparts) {
  __shared__ unsigned long long sh4[4];
  const int n = io.H * io.W;
  for (int i = blockIdx.x * SP_BLOCK + threadIdx.x; i < n; i += gridDim.x * SP_BLOCK)
    io.labels[i] = io.h[i] >= SP_CUT_INF ? 1 : 0;
  if (blockIdx.x != 0) return;
  unsigned long long f = 0;
  for (int k = threadIdx.x; k < nparts; k += SP_BLOCK) f += io.flow_part[k];
  for (int k = threadIdx.x; k < SP_CUT_FLOW; k += SP_BLOCK) f += io.flow[k];
  f = block_sum_u64(f, sh4);
  if (threadIdx.x == 0) {
    if (io.flow_out) *io.flow_out = (int64_t)f;
    const int slot = io.pass & (SP_CUT_CTL - 1);
    io.status[0] = io.ctl[slot];
    io.status[1] = io.ctl[SP_CUT_CTL + slot];
  }
}

}  // namespace

hipError_t sp_launch_cut(int phase, const CutIO& io, hipStream_t st) {
  const int n = io.H * io.W;
  const int grid = (int)std::min(SP_CUT_PARTS, (n + SP_BLOCK - 1) / SP_BLOCK);
  const int tiles = ((io.H + SP_CUT_T - 1) / SP_CUT_T) * ((io.W + SP_CUT_T - 1) / SP_CUT_T);
  switch (phase) {
    case 0: hipLaunchKernelGGL(k_cut_init, dim3(grid), dim3(SP_BLOCK), 0, st, io); break;
    case 1: hipLaunchKernelGGL(k_cut_relabel, dim3(tiles), dim3(RB), 0, st, io); break;
    case 2: hipLaunchKernelGGL(k_cut_push, dim3(((io.H + PT - 1) / PT) * ((io.W + PT - 1) / PT)), dim3(PB), 0, st, io); break;
    case 3: hipLaunchKernelGGL(k_cut_labels, dim3(grid), dim3(SP_BLOCK), 0, st, io, grid); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
