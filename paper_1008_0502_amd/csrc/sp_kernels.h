// Launchers of the HIP kernels (implemented in sp_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include "sp_internal.h"

hipError_t sp_launch(int kind, const Job* jobs, int n, const StreamDesc* sds, const StepIO* ios,
                     const StepIO* io0, int flag, const float* aux, hipStream_t st, size_t lds = 0);
// Lets the across-scale kernel that sp_launch takes for this kind and flag use `bytes` of dynamic
// LDS.  Only that one: others hold more static LDS and would not fit a CU beside it.
hipError_t sp_across_reserve_lds(int kind, int flag, size_t bytes);
hipError_t sp_launch_clip_io(const ClipIO& a, hipStream_t st);
hipError_t sp_launch_bwd(int kind, int flag, const Job* jobs, int n, const StreamDesc* sds, const BwdIO* bios,
                         const BwdIO* b0, hipStream_t st);
// The recorded conspicuity maps of T steps dotted with each step's saliency adjoint (buffers
// of step t and stream i named by ios[t * n_streams + i]: fbar, np_tape, gs, dot, cx, ms_tape).
hipError_t sp_launch_consp_dot(const Job* jobs, int n, const StreamDesc* sds, const StepIO* ios, int n_streams, int T,
                               hipStream_t st);
// Adjoint reduction: one workgroup per stream of tab (or the single stream *one when tab
// is null), shared gains Kd and variances Pd of T steps.
hipError_t sp_launch_bwd_final(const BwdFin* tab, const BwdFin* one, int n_streams, int T, const double* Kd,
                               const double* Pd, double Q, double R, float flat_tol, hipStream_t st);
// Masked-MSE loss of n_streams clips (tab) or of the single clip *one, nblk partials each.
hipError_t sp_launch_loss(const LossIO* tab, const LossIO* one, int n_streams, int nblk, hipStream_t st);
// The colour-statistics launch of a batched step, which also starts the step (see
// BatchBegin).  RgbNodeArgs holds the argument values of that launch as a graph kernel
// node; sp_batch_rgb_node_params points p at them so the node can be re-pointed at the
// next step's frame table (the values must outlive the update call).
hipError_t sp_launch_batch_rgb(const Job* jobs, int n_jobs, const StreamDesc* sds, StepIO* ios, int want_d2,
                               const BatchBegin& bb, hipStream_t stream);
struct RgbNodeArgs {
  const Job* jobs;
  const StreamDesc* sds;
  const StepIO* ios;
  StepIO io0;
  int want_d2;
  BatchBegin bb;
  void* argv[6];
};
void sp_batch_rgb_node_params(RgbNodeArgs* a, int n_jobs, hipKernelNodeParams* p);
hipError_t sp_launch_batch_reset(int n, BatchState* st, hipStream_t stream);
// max_px: pixels of the largest stream.
hipError_t sp_launch_batch_copy_out(int n, size_t max_px, const BatchState* st, const StreamDesc* sds,
                                    float* const* out, hipStream_t stream);
// Counter calibration copy of n16 16-byte units (mode: 0 dword, 1 dwordx4, 2 global->LDS dword).
hipError_t sp_launch_calib(const float* src, float* dst, size_t n16, int mode, hipStream_t st);

// Device address of the allocation-free entry point's scratch array on the current device
// (SP_NOALLOC_BYTES bytes; looked up once per device, then remembered).
hipError_t sp_noalloc_scratch(void** ptr);
// Prior of the first frame from manual labels (n pixels).
hipError_t sp_launch_manual(const uint8_t* labels, float* pnext, float* pout, size_t n, float eps, hipStream_t st);
// Colour likelihood: pass 0 the start's moments, 1 the E-step's, 2 psi added to the unary costs, -1 no
// pixels (the fit alone); fit 0 the mixtures of io.st_prev, 1 the start and 2 the M-step from
// io.part_in, stored in io.st_next (M = components per label, 1..SP_GMM_MAXM).
hipError_t sp_launch_gmm(int pass, int fit, int M, const GmmIO& io, hipStream_t st);
// Minimum cut phases: 0 counters + capacities, 1 relabel pass, 2 push / relabel cycles,
// 3 labels, the flow value and the last pass's counters.
hipError_t sp_launch_cut(int phase, const CutIO& io, hipStream_t st);
// The pixel-level adjoint of frames t0 .. t0 + nz - 1 of a recorded clip (sp_pixadj.hip): their
// pyramid and Gabor maps are in the slots sds[0 .. nz - 1] (geometry g), gs, S, ms and fbar are
// frame t0's tape slots, grad [T][H][W][3] receives the gradients.
hipError_t sp_pixel_adjoint(const PaDesc& A, const StreamDesc* sds, const StreamDesc& g, int t0, int nz,
                            const uint8_t* frames, const float* gs, const float* S, const float* ms, const float* fbar,
                            float* grad, hipStream_t st);
