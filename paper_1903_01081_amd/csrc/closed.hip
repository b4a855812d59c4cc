// Numeric closed form of a component (closed.h): the clusters' inverses Q,
// N = -G_DS Q and the tail inverse W = (G_DD + N G_SD)^-1 of every (item,
// topology), FP64, gfx950.
//
// One workgroup per (item, topology). Q and N live in LDS; the tail is
// inverted in VGPRs in the step kernels' layout (step.h, Tail), one barrier
// per pivot: the pivot's row and column go through a double-buffered LDS
// line, every lane updates its share of the matrix. G is symmetric positive
// definite, so Gauss-Jordan needs no pivoting, and its pivots are those of
// LDL^T in the same order: a non-positive or non-finite one is counted in
// flags[0].
// This replaces, for components with a closed form, an LDL^T factorisation
// by one lane per row and a tail inverse by one lane per column over global
// memory (both chains of dependent memory reads).
#include <hip/hip_runtime.h>

#include "assemble.h"
#include "launch.h"
#include "step.h"

namespace emt {

namespace {

using step::emt_lds;
using step::lds_barrier;

__device__ __forceinline__ bool good_pivot(double p) { return p > 0.0 && p < INFINITY; }

// In-place Gauss-Jordan inverse of an s x s block in LDS by one wave: the
// entries off the pivot's row and column first, then these.
__device__ void invert_block(double *A, int s, int32_t *flags) {
  const int lane = (int)threadIdx.x & 63, li = lane >> 3, lj = lane & 7;
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  for (int p = 0; p < s; ++p) {
    const double piv = A[p * s + p];
    const bool ok = good_pivot(piv);
    if (!ok && lane == 0) atomicAdd(flags, 1);
    const double d = ok ? 1.0 / piv : 0.0;
    for (int i = li; i < s; i += 8) {
      const double ci = A[i * s + p];
      for (int j = lj; j < s; j += 8)
        if (i != p && j != p) A[i * s + j] = __builtin_fma(-ci, A[p * s + j] * d, A[i * s + j]);
    }
    wave_sync();
    for (int i = lane; i < s; i += 64) {
      if (i == p) {
        A[p * s + p] = d;
      } else {
        A[i * s + p] = -(A[i * s + p] * d);
        A[p * s + i] = A[p * s + i] * d;
      }
    }
    wave_sync();
  }
}

template <int BS, int DT>
__global__ __launch_bounds__(BS) void k_closed(DevCtx c, const int32_t *pairs, int values) {
  using T = step::Tail<BS, DT>;
  double *V = reinterpret_cast<double *>(emt_lds);
  // pivot rows and columns, two buffers each
  double *line = V + (values + 1) / 2 * 2;
  const int item = pairs[2 * blockIdx.x], t = pairs[2 * blockIdx.x + 1];
  const ItemDesc it = c.items[item];
  const SymDesc sd = c.syms[it.sym];
  const int n = it.n, d = sd.d, ns = sd.ns, tid = (int)threadIdx.x;
  double *Lr = c.lfull + it.fac + (int64_t)t * sd.nnz;
  double *D = c.dpiv + it.dfac + (int64_t)t * n;
  if (sd.closed == 2)
    assemble_g<BS, true>(c, it, sd, t, Lr, D);
  else
    assemble_g<BS>(c, it, sd, t, Lr, D);
  double *N = V + 2, *Q = N + sd.n_n;
  if (tid < 2) V[tid] = (double)tid;
  for (int q = tid; q < sd.n_q; q += BS) Q[q] = 0.0;
  double *W = c.wtail + it.w + (int64_t)t * d * d;
  for (int q = tid; q < d * d; q += BS) W[q] = 0.0;
  __syncthreads();
  const int32_t *I = c.symi;
  for (int i = tid; i < ns; i += BS) Q[I[sd.q_diag + i]] = D[i];
  for (int q = tid; q < sd.nq_off; q += BS) Q[I[sd.q_off + 2 * q + 1]] = Lr[I[sd.q_off + 2 * q]];
  for (int q = tid; q < sd.ns_off; q += BS) W[I[sd.s_off + 2 * q + 1]] = Lr[I[sd.s_off + 2 * q]];
  for (int a = tid; a < d; a += BS) W[a * (d + 1)] = D[ns + a];
  __syncthreads();
  // clusters, largest first: one node per lane, more nodes per wave
  {
    int ones = sd.ncl;
    for (int q = tid >> 6; q < sd.ncl; q += BS / 64) {
      const int s = I[sd.cluster + 2 * q];
      if (s == 1) break;
      invert_block(Q + I[sd.cluster + 2 * q + 1], s, c.flags);
    }
    // the first one-node cluster (they are sorted by size)
    int lo = 0;
    while (lo < ones) {
      const int mid = (lo + ones) / 2;
      if (I[sd.cluster + 2 * mid] > 1)
        lo = mid + 1;
      else
        ones = mid;
    }
    for (int q = lo + tid; q < sd.ncl; q += BS) {
      double *a = Q + I[sd.cluster + 2 * q + 1];
      const bool ok = good_pivot(*a);
      if (!ok) atomicAdd(c.flags, 1);
      *a = ok ? 1.0 / *a : 0.0;
    }
  }
  __syncthreads();
  for (int e = tid; e < sd.n_n; e += BS) {
    const int g = I[sd.n_grp + e], col = I[sd.n_col + e];
    double s = 0.0;
    for (int q = I[sd.n_ptr + g]; q < I[sd.n_ptr + g + 1]; ++q)
      s = __builtin_fma(Lr[I[sd.n_adj + 2 * q]], Q[I[sd.n_adj + 2 * q + 1] + col], s);
    N[e] = -s;
  }
  __syncthreads();
  for (int k = tid; k < sd.ns_key; k += BS) {
    const int key = I[sd.s_key + k];
    double s = W[key];
    for (int q = I[sd.s_ptr + k]; q < I[sd.s_ptr + k + 1]; ++q)
      s = __builtin_fma(N[I[sd.s_term + 2 * q]], Lr[I[sd.s_term + 2 * q + 1]], s);
    W[key] = s;
  }
  double *sv = c.svals + it.sv + (int64_t)t * sd.nsv;
  for (int q = tid; q < sd.nsv; q += BS) sv[q] = V[I[sd.vsrc + q]];
  if (d == 0) return;
  __syncthreads();
  T w;
  step::load_tail<BS, DT>(W, d, w);
  if (sd.closed == 2) {
    // with switches the step kernel inverts; here the matrix stays and its
    // pivots are checked with the switches' initial states
    __syncthreads();
    double *S = c.dyn + it.dyn + (int64_t)t * d * d;
    for (int q = tid; q < d * d; q += BS) S[q] = W[q];
    __syncthreads();
    const uint8_t *ins = c.cins + it.coef + (int64_t)t * it.n_br;
    for (int k = tid; k < it.n_swkey; k += BS) {
      const int key = I[it.swkey + k];
      double s = W[key];
      for (int q = I[it.swptr + k]; q < I[it.swptr + k + 1]; ++q) {
        const int term = I[it.swterm + q];
        const int br = c.sw_tab[it.swt + (term >> 1)].br;
        const double gs = ins[br] ? 1.0 / c.bR[it.br + br] : 0.0;
        s = (term & 1) ? s - gs : s + gs;
      }
      S[key] = s;
    }
    __syncthreads();
    step::load_tail<BS, DT>(S, d, w);
  }
  const int bad = step::invert_tail<BS, DT>(w, d, line);
  if (bad && tid == 0) atomicAdd(c.flags, bad);
  if (sd.closed == 2) return;
  const int g = tid >> 4, j = tid & 15;
#pragma unroll
  for (int k = 0; k < T::R; ++k) {
    const int row = g + k * T::G;
#pragma unroll
    for (int q = 0; q < T::Q; ++q) {
      const int col = 32 * q + 2 * j;
      if (row < d && col < d) W[row * d + col] = w.w[2 * (k * T::Q + q)];
      if (row < d && col + 1 < d) W[row * d + col + 1] = w.w[2 * (k * T::Q + q) + 1];
    }
  }
}

template <int BS, int DT>
hipError_t closed_launch(const DevCtx &c, const int32_t *pairs, int n_pairs, int values, hipStream_t st) {
  auto k = k_closed<BS, DT>;
  const size_t lds = ((size_t)(values + 1) / 2 * 2 + step::tail_lines(DT)) * sizeof(double);
  hipError_t e =
      hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(n_pairs), dim3(BS), lds, st, c, pairs, values);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_closed(const DevCtx &c, const int32_t *pairs, int n_pairs, int values, int max_tail,
                         hipStream_t st) {
  if (n_pairs == 0) return hipSuccess;
  if (max_tail <= 64) return closed_launch<256, 64>(c, pairs, n_pairs, values, st);
  if (max_tail <= 128) return closed_launch<512, 128>(c, pairs, n_pairs, values, st);
  if (max_tail <= 192) return closed_launch<512, 192>(c, pairs, n_pairs, values, st);
  return hipErrorInvalidValue;
}

}  // namespace emt
