// Instantiations of the step kernels for one workgroup size (EMT_BS, set by
// the build: 64, 256 or 512) and one kind of kernel (EMT_PART_*: FWD with
// EMT_KIND, a StepKind; ADJ and PIPE with EMT_KIND, an AdjointKind), so that they
// compile in parallel.
#include <hip/hip_runtime.h>

#include "launch.h"
#include "step.h"

#ifndef EMT_BS
#error "EMT_BS must be defined"
#endif

namespace emt {

static_assert(STEP_LEVELS == 5 && ADJ_LEVELS == 2, "EMT_LEVELS below");

namespace {

#if defined(EMT_PART_FWD)
template <int BPT, int DT, bool SM>
hipError_t fwd(const DevCtx &c, const int32_t *order, int n_items, int64_t n0, int64_t ns, double *rec,
               size_t lds, hipStream_t st) {
  auto k = step::k_forward<EMT_BS, BPT, DT, SM, EMT_KIND>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(n_items), dim3(EMT_BS), lds, st, c, order, n0, ns, rec);
  return hipGetLastError();
}

#elif defined(EMT_PART_ADJ)
template <int BPT, int DT, bool SM>
hipError_t adj(const DevCtx &c, const int32_t *order, int n_items, const double *dJ, size_t lds,
               hipStream_t st) {
  auto k = step::k_adjoint<EMT_BS, BPT, DT, SM, EMT_KIND>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(n_items), dim3(EMT_BS), lds, st, c, order, dJ);
  return hipGetLastError();
}

#else
template <int BPT, int DT, bool SM>
hipError_t adj_pipe(const DevCtx &c, const int32_t *order, int n_items, const double *dJ, int32_t *pipe,
                    size_t lds, hipStream_t st) {
  auto k = step::k_adjoint_pipe<EMT_BS, BPT, DT, SM, EMT_KIND>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  DevCtx ca = c;
  const int32_t *oa = order;
  int na = n_items;
  const double *da = dJ;
  int32_t *pa = pipe;
  void *args[] = {&ca, &oa, &na, &da, &pa};
  return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(k), dim3(2 * n_items), dim3(EMT_BS), args,
                                    (unsigned)lds, st);
}

template <int BPT, int DT, bool SM>
hipError_t adj_pipe_occupancy(size_t lds, int *blocks) {
  auto k = step::k_adjoint_pipe<EMT_BS, BPT, DT, SM, EMT_KIND>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, reinterpret_cast<const void *>(k), EMT_BS, lds);
}
#endif

}  // namespace

// Branches per lane x dense-tail capacity (KernelShape::dt): LDS-staged
// variants for every count, global-memory fallbacks for the larger ones.
#define EMT_SHAPES_W(X, D) \
  X(1, D, true) X(2, D, true) X(4, D, true) X(6, D, true) X(8, D, true) X(12, D, true) X(16, D, true) \
  X(4, D, false) X(8, D, false) X(16, D, false)
// Tails of level passes are smaller than those of the closed form.
#if defined(EMT_PART_FWD)
#define EMT_LEVELS (EMT_KIND == 5)
#else
#define EMT_LEVELS (EMT_KIND == 2)
#endif
#if EMT_BS >= 512 && EMT_LEVELS
#define EMT_SHAPES(X) EMT_SHAPES_W(X, 64) EMT_SHAPES_W(X, 128)
#elif EMT_BS >= 512
#define EMT_SHAPES(X) EMT_SHAPES_W(X, 64) EMT_SHAPES_W(X, 128) EMT_SHAPES_W(X, 192)
#elif EMT_BS >= 256 && EMT_LEVELS
#define EMT_SHAPES(X) EMT_SHAPES_W(X, 64)
#elif EMT_BS >= 256
#define EMT_SHAPES(X) EMT_SHAPES_W(X, 64) EMT_SHAPES_W(X, 128)
#elif EMT_LEVELS
#define EMT_SHAPES(X) EMT_SHAPES_W(X, 32)
#else
#define EMT_SHAPES(X) EMT_SHAPES_W(X, 32) EMT_SHAPES_W(X, 64)
#endif

#ifdef EMT_PART_FWD
template <>
hipError_t launch_forward<EMT_BS, EMT_KIND>(const DevCtx &c, const KernelShape &ks, const int32_t *order, int n_items,
                                            int64_t n0, int64_t ns, double *rec, hipStream_t st) {
#define EMT_CASE(BPT, DT, SM)                      \
  if (ks.bpt == BPT && ks.dt == DT && ks.sm == SM) \
    return fwd<BPT, DT, SM>(c, order, n_items, n0, ns, rec, ks.lds_fwd, st);
  EMT_SHAPES(EMT_CASE)
#undef EMT_CASE
  return hipErrorInvalidValue;
}
#endif

#ifdef EMT_PART_ADJ
template <>
hipError_t launch_adjoint<EMT_BS, EMT_KIND>(const DevCtx &c, const KernelShape &ks, const int32_t *order,
                                              int n_items, const double *dJ, hipStream_t st) {
#define EMT_CASE(BPT, DT, SM) \
  if (ks.bpt == BPT && ks.dt == DT && ks.sm == SM) return adj<BPT, DT, SM>(c, order, n_items, dJ, ks.lds_adj, st);
  EMT_SHAPES(EMT_CASE)
#undef EMT_CASE
  return hipErrorInvalidValue;
}

#endif

#ifdef EMT_PART_PIPE
template <>
hipError_t launch_adjoint_pipe<EMT_BS, EMT_KIND>(const DevCtx &c, const KernelShape &ks, const int32_t *order,
                                                   int n_items, const double *dJ, int32_t *pipe, hipStream_t st) {
#define EMT_CASE(BPT, DT, SM) \
  if (ks.bpt == BPT && ks.dt == DT && ks.sm == SM) return adj_pipe<BPT, DT, SM>(c, order, n_items, dJ, pipe, ks.lds_adj, st);
  EMT_SHAPES(EMT_CASE)
#undef EMT_CASE
  return hipErrorInvalidValue;
}

template <>
hipError_t adjoint_pipe_blocks_per_cu<EMT_BS, EMT_KIND>(const KernelShape &ks, int *blocks) {
#define EMT_CASE(BPT, DT, SM) \
  if (ks.bpt == BPT && ks.dt == DT && ks.sm == SM) return adj_pipe_occupancy<BPT, DT, SM>(ks.lds_adj, blocks);
  EMT_SHAPES(EMT_CASE)
#undef EMT_CASE
  return hipErrorInvalidValue;
}
#endif

}  // namespace emt
