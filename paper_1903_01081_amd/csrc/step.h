// Device code of the persistent step kernels (forward time loop and
// reverse-time adjoint), FP64, gfx950.
//
// One workgroup owns one work item (a connected component of one scenario)
// for many time steps; scenarios and components are more workgroups of the
// same launch. This is the paper's pair of parallel strategies (Sec. III-B):
// the processes of one layer run together and the layers are replayed in
// order every step; isomorphic scenarios run the same processes side by
// side. A step runs the four basic processes of an EMTP-type solver that the
// paper lists (Sec. III-A) as barrier-separated phases:
//   branch phase  (one branch per lane slot; coefficients and history in
//                 VGPRs): u = A^T v - e and i = g u + h of the previous step,
//                 the next history h = beta i + gamma u, the source EMF e and
//                 the branch injection J = g e - h into LDS;
//   gather        every node sums its incident branch ends' J in a fixed
//                 (CSR) order — a deterministic segmented sum, no atomics;
// and the solve, in closed form (closed.h) where that is planned,
//   forward       c = r_D + N r_S, the dense tail's right-hand side;
//   tail          x_D = W c, W held in VGPRs;
//   backward      x_S = Q r_S + N^T x_D,
// each a set of independent rows, or by level passes:
//   forward       L y = rhs over the leading part of the elimination order,
//                 one pass per level (level 0 needs none), then the tail's
//                 reduced right-hand side c = rhs_D - L_DS y_S;
//   tail          the same;
//   backward      x = D^{-1} y - L^T x, one pass per level.
// In a level pass each row is shared by 2^k <= 16 adjacent lanes (k per
// pass, so that a few long rows at the top of the tree use many lanes and
// many short rows one lane each); the lanes' partial sums meet in a fixed
// scan of DPP row shifts, so every run rounds identically.
// All factors of every topology are computed before the loop (k_factor and
// k_tail, or k_closed); a switching event swaps coefficients and factor
// pointers. Components with diodes or controlled switches factor the tail
// (closed form) or the whole component (level passes) anew inside the loop.
//
// Compiled with -ffp-contract=off so that identical formulas round
// identically in every code path (forward, checkpoint recompute, reload).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"
#include "trig.h"

namespace emt {
namespace step {

constexpr int64_t kNever = INT64_MAX;

// How the components of a kernel's batch are solved.
enum : int { CLOSED = 0, LEVELS = 1, BOTH = 2 };
constexpr int adjoint_solve(int gen) { return gen == ADJ_PLAIN ? CLOSED : (gen == ADJ_LEVELS ? LEVELS : BOTH); }

__device__ __forceinline__ double gamma_of(uint32_t pk, double g) {
  const uint32_t c = pk >> 30;
  return c == GAMMA_PLUS_G ? g : (c == GAMMA_MINUS_G ? -g : 0.0);
}

// gamma u from g u (gamma = g, -g or 0).
__device__ __forceinline__ double gamma_times(uint32_t pk, double gu) {
  const uint64_t b = __builtin_bit_cast(uint64_t, gu) ^ ((uint64_t)((pk << 1) & 0x80000000u) << 32);
  return (pk >> 31) ? 0.0 : __builtin_bit_cast(double, b);
}

__device__ __forceinline__ double source_emf(const DevCtx &c, int64_t gb, int64_t n) {
  const double t = (double)n * c.dt;
  return c.bE[gb] * emf_cos(c.bw[gb] * t + c.bph[gb]);
}

__device__ __forceinline__ int topo_of(const int64_t *topo, int ntopo, int64_t n) {
  int t = 0;
  while (t + 1 < ntopo && topo[t + 1] <= n) ++t;
  return t;
}

// The lane index, hidden from the optimiser at each use so that per-slot
// index and address arithmetic is recomputed inside the time loop (a few
// integer operations) instead of being hoisted out of it and held in VGPRs.
__device__ __forceinline__ int lane_id() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// The same for a packed branch descriptor, where registers are short.
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Workgroup barrier that orders LDS only. Lanes of a workgroup exchange
// data only through LDS here; global stores (recorded outputs, checkpoints,
// state) are read by later kernels or by the same lane, so a barrier need
// not wait for them to complete as __syncthreads() would.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Waits here for a value read from global memory. For the reads inside the
// time loop that only a switching step makes: left alone, the compiler waits
// for them at their first use in the loop, which every step passes, and as
// vector memory operations complete in order each step would wait there for
// the stores of the recorded voltages (about half of a 9-node component's
// step).
__device__ __forceinline__ void settle(double &x) { asm volatile("" : "+v"(x)); }

// The same for a workgroup of BS lanes. One wave's LDS accesses complete in
// the order they were issued, so a single-wave workgroup needs no wait at
// all, only that the compiler keeps the order.
template <int BS>
__device__ __forceinline__ void step_barrier() {
  if constexpr (BS == 64) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  } else {
    lds_barrier();
  }
}

// Dynamic LDS of the step kernels (addressed with 32-bit offsets so that
// every access compiles to a ds_* instruction).
extern __shared__ __align__(16) char emt_lds[];

// A read-only array either in LDS (32-bit byte offset) or in global memory.
template <class T, bool SM>
struct Ref;
template <class T>
struct Ref<T, true> {
  uint32_t off;
  __device__ __forceinline__ T operator[](int i) const { return reinterpret_cast<const T *>(emt_lds + off)[i]; }
};
template <class T>
struct Ref<T, false> {
  const T *p;
  __device__ __forceinline__ T operator[](int i) const { return p[i]; }
};

// A read-write LDS array.
template <class T>
struct Lds {
  uint32_t off;
  __device__ __forceinline__ T &operator[](int i) const { return reinterpret_cast<T *>(emt_lds + off)[i]; }
};

// LDS doubles of the tail inversion: two pivot rows and columns of up to dt
// (a multiple of 32) entries.
constexpr int tail_lines(int dt) { return 4 * ((dt + 31) / 32 * 32); }

// A row program (closed.h) as a wave runs it: its batches b0 .. b1 - 1, the
// first one's batch word, quad of codes and row id held in registers, the
// rest in LDS (SM) or global memory.
template <bool SM>
struct Rows {
  int b0, b1;
  uint32_t m0;
  uint64_t c0;
  int r0;
  Ref<int32_t, SM> word;
  Ref<uint64_t, SM> code;
  Ref<uint16_t, SM> row;
};

// Per-workgroup view of an item: sizes, LDS arrays, and the sweep data in
// LDS (SM = true) or global memory.
template <bool SM>
struct View {
  int n, d, ns, nbr, nreal, nsrc, nsv, nrec;  // nbr: padded to whole lane slots; nreal: not
  int closed, nfpass, nbpass, fvals;   // fvals: values of the forward program
  Rows<SM> gather, fwd, bwd;
  Ref<int32_t, SM> fpass, bpass;  // level passes: (first descriptor, log2 lanes) pairs
  Ref<uint64_t, SM> fdesc, bdesc;
  Ref<uint16_t, SM> fcol, brow, bpos, rnode, rcolumn;
  Lds<double> r, x, J, cD, sv_s, dinv_s, emf, vrow;  // x has n+1 entries, x[n] = 0; r: where the gather writes
  Lds<int32_t> flag;                           // adjoint: a word for broadcasts
  bool emf_direct;                             // no EMF table (not under SM)
  Ref<double, SM> sv, dinv;
  int lim;           // pairs of closed-form values staged in LDS (the rest: svg)
  const double *svg;  // the topology's closed-form values in global memory
  // items refactorised inside the loop, under SM: node CSR (where staged), the
  // factorisation's row pointers, level pointers (rows, entries), level rows
  Lds<int32_t> nptr;
  Lds<uint16_t> nent;
  Lds<int32_t> rf_rowptr, rf_flev, rf_fent_ptr;
  Lds<uint16_t> rf_rows;
  // closed form with switches: the tail inversion's lines, the switches'
  // conductances; and, also of items refactorised inside the loop, the last
  // step that changed a switch's state
  Lds<double> line, gsw;
  Lds<int32_t> swflag;
};

// 16-byte blocks into LDS, block i from at(i), U of a lane's loads in flight
// (loads past the end fetch the last block).
template <int BS, int U, class F>
__device__ __forceinline__ void copy_blocks(uint32_t off, int cnt, F &&at) {
  uint4 *dst = reinterpret_cast<uint4 *>(emt_lds + off);
  for (int q = (int)threadIdx.x; q < cnt; q += U * BS) {
    uint4 r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = *at(q + u * BS < cnt ? q + u * BS : cnt - 1);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (q + u * BS < cnt) dst[q + u * BS] = r[u];
  }
}

template <int BS, class T>
__device__ __forceinline__ void copy_to(uint32_t off, const T *src, int cnt) {
  T *dst = reinterpret_cast<T *>(emt_lds + off);
  for (int q = threadIdx.x; q < cnt; q += BS) dst[q] = src[q];
}

// Copy of int32 values below 65536 into uint16 LDS.
template <int BS>
__device__ __forceinline__ void copy_to_u16(uint32_t off, const int32_t *src, int cnt) {
  uint16_t *dst = reinterpret_cast<uint16_t *>(emt_lds + off);
  for (int q = threadIdx.x; q < cnt; q += BS) dst[q] = (uint16_t)src[q];
}

template <int BS, bool SM>
__device__ __forceinline__ void load_rows(const DevCtx &c, const RowProg &p, uint32_t ometa, uint32_t ocode,
                                          uint32_t orow, Rows<SM> &v) {
  const int32_t *meta = c.symi + p.meta;
  const uint64_t *code = reinterpret_cast<const uint64_t *>(c.symh + p.code);
  const uint16_t *row = c.symh + p.row;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  constexpr int W = BS / 64;
  v.b0 = v.b1 = 0;
  v.m0 = 0;
  v.c0 = 0;
  v.r0 = 0xFFFF;
  if (p.nb > 0) {
    v.b0 = __builtin_amdgcn_readfirstlane(meta[w]);
    v.b1 = __builtin_amdgcn_readfirstlane(meta[w + 1]);
    if (v.b0 < v.b1) {
      v.m0 = (uint32_t)__builtin_amdgcn_readfirstlane(meta[W + 1 + v.b0]);
      v.c0 = code[(int)(v.m0 & 0xFFFF) * 64 + lane];
      v.r0 = row[v.b0 * 64 + lane];
    }
  }
  if constexpr (SM) {
    v.word.off = ometa + 4 * (W + 1);
    v.code.off = ocode;
    v.row.off = orow;
    if (p.nb > 0) {
      copy_to<BS>(ometa, meta, W + 1 + p.nb);
      copy_to<BS>(ocode, code, p.nq * 64);
      copy_to<BS>(orow, row, p.nb * 64);
    }
  } else {
    v.word.p = meta + W + 1;
    v.code.p = code;
    v.row.p = row;
  }
}

// The LDS layout is step_lds() (device.h), which the host sizes launches by.
// LEV: how the batch's components are solved: CLOSED form, LEVEL passes or some
// each (the kernels of one kind carry no scalars of the other: those of both
// together spill, and level passes alone take a quarter of the registers less,
// which is twice the workgroups of a batch at once at 256 lanes).
// DT > 0: its items may have diodes or controlled switches in closed form.
template <int BS, bool SM, int LEV, int DT = 0>
__device__ __forceinline__ View<SM> make_view(const DevCtx &c, const ItemDesc &it, bool adjoint) {
  const SymDesc sd = c.syms[it.sym];
  View<SM> v;
  v.n = it.n;
  v.d = sd.d;
  v.ns = sd.ns;
  v.nbr = it.n_br;
  v.nreal = it.n_real;
  v.nsrc = it.n_src;
  v.nsv = sd.nsv;
  v.nrec = it.n_rec;
  v.closed = LEV == LEVELS ? 0 : (LEV == CLOSED ? 1 : sd.closed);
  v.nfpass = sd.nfpass;
  v.nbpass = sd.nbpass;
  v.fvals = sd.fwd.nq * 256;
  const int32_t *g_nptr = c.nptr + it.nptr;
  const bool dyn = LEV == BOTH && it.n_diodes > 0;
  const int nsw = DT > 0 ? it.n_diodes : 0;
  const int ne = SM && dyn && !c.csr_global ? g_nptr[v.n] : 0;
  const bool seeds = adjoint && (SM || !c.seeds_global);  // recorded columns' cotangents in LDS
  const RowProg gp = seeds ? it.ga : it.gf;
  // the closed form's values beyond what the LDS has room for stay in L2
  const int nstage = v.closed && sd.nsv > c.sv_cap ? c.sv_cap : sd.nsv;
  v.lim = SM ? nstage / 2 : 0;
  const StepShape sh{it.n,       sd.d,      sd.ns,     it.n_br,   it.n_src,  it.n_rec,  v.closed,
                     sd.nfpass,  sd.nbpass, nstage,    sd.nfdesc, sd.nbdesc, gp.nb,     gp.nq,
                     sd.fwd.nb,  sd.fwd.nq, sd.bwd.nb, sd.bwd.nq, dyn ? sd.nlev : 0, ne, nsw, nsw > 0 ? tail_lines(DT) : 0, BS,
                     SM ? 0 : c.row_global, SM ? 0 : c.seeds_global};
  const StepLds o = step_lds(sh, SM, adjoint);
  v.cD.off = o.cD;
  // closed form: the gather writes r (the tail's right-hand side where the
  // whole component is the tail), the solution goes to x; level passes work
  // in place on x
  v.x.off = o.xr + (v.closed ? (uint32_t)(v.n + 1) * 8u : 0u);
  v.r.off = v.closed && v.ns == 0 ? o.cD : o.xr;
  v.J.off = o.J;
  v.flag.off = o.flag;
  v.emf.off = o.emf;
  v.emf_direct = adjoint && !seeds;
  v.vrow.off = o.vrow;
  v.line.off = o.line;
  v.gsw.off = o.gsw;
  v.swflag.off = o.swflag;
  for (int q = threadIdx.x; q < (v.d + 31) / 32 * 32; q += BS) v.cD[q] = 0.0;
  if (threadIdx.x == 0) {
    v.x[v.n] = 0.0;  // the ground: every grounded terminal points here
    v.J[v.nbr] = 0.0;
    if (adjoint && (SM || !c.row_global)) v.vrow[v.n] = 0.0;
    reinterpret_cast<double *>(emt_lds + o.xr)[v.n] = 0.0;
  }
  load_rows<BS, SM>(c, gp, o.gmeta, o.gcode, o.grow, v.gather);
  if (v.closed) {
    load_rows<BS, SM>(c, sd.fwd, o.fmeta, o.fcode, o.frow, v.fwd);
    load_rows<BS, SM>(c, sd.bwd, o.bmeta, o.bcode, o.brw, v.bwd);
  } else if constexpr (SM) {
    const int nf = 2 * (v.nfpass + 1), nb = 2 * (v.nbpass + 1);
    v.fpass.off = o.pass;
    v.bpass.off = o.pass + 4 * nf;
    copy_to<BS>(o.pass, c.symi + sd.fpass, nf);
    copy_to<BS>(o.pass + 4 * nf, c.symi + sd.bpass, nb);
  } else {
    v.fpass.p = c.symi + sd.fpass;
    v.bpass.p = c.symi + sd.bpass;
  }
  if constexpr (SM) {
    v.sv_s.off = v.sv.off = o.sv;
    v.rnode.off = o.rnode;
    v.rcolumn.off = o.rcolumn;
    copy_to<BS>(o.rnode, c.rnode + it.rec, v.nrec);
    copy_to<BS>(o.rcolumn, c.rcolumn + it.rec, v.nrec);
    if (!v.closed) {
      v.dinv_s.off = v.dinv.off = o.dinv;
      v.fdesc.off = o.fdesc;
      v.bdesc.off = o.bdesc;
      v.fcol.off = o.fcol;
      v.brow.off = o.brow;
      v.bpos.off = o.bpos;
      copy_to<BS>(o.fdesc, c.symd + sd.fdesc, sd.nfdesc);
      copy_to<BS>(o.bdesc, c.symd + sd.bdesc, sd.nbdesc);
      copy_to<BS>(o.fcol, c.symh + sd.fcol, v.nsv);
      copy_to<BS>(o.brow, c.symh + sd.brow, v.nsv);
      copy_to<BS>(o.bpos, c.symh + sd.bpos, v.nsv);
    }
    if (dyn) {
      v.nptr.off = o.rf_nptr;
      v.nent.off = o.rf_nent;
      if (ne > 0) {
        copy_to<BS>(o.rf_nptr, g_nptr, v.n + 1);
        copy_to<BS>(o.rf_nent, c.nent + it.nent, ne);
      }
      v.rf_rowptr.off = o.rf_rowptr;
      v.rf_flev.off = o.rf_flev;
      v.rf_fent_ptr.off = o.rf_fent;
      v.rf_rows.off = o.rf_rows;
      copy_to<BS>(o.rf_rowptr, c.symi + sd.rowptr, v.n + 1);
      copy_to<BS>(o.rf_flev, c.symi + sd.flevptr, sd.nlev + 1);
      copy_to<BS>(o.rf_fent, c.symi + sd.fentptr, sd.nlev + 1);
      copy_to_u16<BS>(o.rf_rows, c.symi + sd.flevrows, v.n);
    }
  } else {
    v.fdesc.p = c.symd + sd.fdesc;
    v.bdesc.p = c.symd + sd.bdesc;
    v.fcol.p = c.symh + sd.fcol;
    v.brow.p = c.symh + sd.brow;
    v.bpos.p = c.symh + sd.bpos;
    v.rnode.p = c.rnode + it.rec;
    v.rcolumn.p = c.rcolumn + it.rec;
  }
  return v;
}

// The tail inverse W in VGPRs: a row of W is shared by the 16 lanes of a DPP
// row, lane j holding the column pairs 32 q + 2 j (so that one read of c is
// 256 contiguous bytes for the 16 lanes, without bank conflicts); each group
// of 16 lanes holds the rows g, g + BS/16, ... With one row per lane group
// and contiguous columns a step read c d/4 times as often: a wave's LDS
// reads return 64 x 16 B each even where the lanes read the same address, and
// those reads, not the multiply-adds, set the tail's time.
template <int BS, int DT>
struct Tail {
  static constexpr int G = BS / 16;          // groups of 16 lanes
  static constexpr int R = (DT + G - 1) / G;  // rows per group
  static constexpr int Q = (DT + 31) / 32;    // column pairs per lane
  double w[2 * R * Q];
};

// The lane's share of the d x d row-major W.
template <int BS, int DT>
__device__ __forceinline__ void load_tail(const double *W, int d, Tail<BS, DT> &T) {
  constexpr int G = Tail<BS, DT>::G, R = Tail<BS, DT>::R, Q = Tail<BS, DT>::Q;
  const int tid = lane_id();
  const int g = tid >> 4, j = tid & 15;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int row = g + k * G;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int col = 32 * q + 2 * j;
      T.w[2 * (k * Q + q)] = row < d && col < d ? W[row * d + col] : 0.0;
      T.w[2 * (k * Q + q) + 1] = row < d && col + 1 < d ? W[row * d + col + 1] : 0.0;
    }
  }
}

// In-place Gauss-Jordan inverse of the symmetric positive definite d x d
// matrix held in T's layout (zero past d): pivot p's row and column go
// through `line` (LDS, tail_lines(DT) doubles), one barrier per pivot. Returns
// the number of non-positive or non-finite pivots (the same in every lane).
// Entries of the pivot's row and column take the general update a - c r / p
// with (a, c) = (0, -1) and (a, r) = (0, 1).
template <int BS, int DT>
__device__ __forceinline__ int invert_tail(Tail<BS, DT> &T, int d, double *line) {
  constexpr int G = Tail<BS, DT>::G, R = Tail<BS, DT>::R, Q = Tail<BS, DT>::Q;
  static_assert(32 % G == 0, "a group's pivots share a column pair block");
  static_assert(2 * (Q * 32 + R * G) <= tail_lines(DT), "two pivot rows and columns");
  constexpr int kBuf = Q * 32 + R * G;
  const int tid = (int)threadIdx.x;
  const int g = tid >> 4, j = tid & 15;
  int bad = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    constexpr int kStep = 2;
    const int qk = k * G / 32;
    for (int r0 = 0; r0 < G && k * G + r0 < d; r0 += kStep) {
#pragma unroll
      for (int b = 0; b < kStep; ++b) {
        const int r = r0 + b, p = k * G + r;
        if (p >= d) break;
        double *prow = line + b * kBuf, *pcol = prow + Q * 32;
        const bool in_row = g == r, in_col = j == ((p & 31) >> 1);
        if (in_row) {
#pragma unroll
          for (int q = 0; q < Q; ++q)
            reinterpret_cast<double2 *>(prow)[16 * q + j] =
                make_double2(T.w[2 * (k * Q + q)], T.w[2 * (k * Q + q) + 1]);
        }
        if (in_col) {
#pragma unroll
          for (int i = 0; i < R; ++i) pcol[g + i * G] = T.w[2 * (i * Q + qk) + b];
        }
        step_barrier<BS>();
        const double piv = prow[p];
        const bool ok = piv > 0.0 && piv < INFINITY;
        bad += ok ? 0 : 1;
        const double inv = ok ? 1.0 / piv : 0.0;
        double rx[Q], ry[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const double2 rr = reinterpret_cast<const double2 *>(prow)[16 * q + j];
          rx[q] = rr.x * inv;
          ry[q] = rr.y * inv;
        }
        if (in_col) {
          if (b == 0)
            rx[qk] = inv;
          else
            ry[qk] = inv;
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
          double cc = pcol[g + i * G];
          const bool here = i == k && in_row;
          if (here) cc = -1.0;
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            double wx = T.w[2 * (i * Q + q)], wy = T.w[2 * (i * Q + q) + 1];
            if (here) wx = wy = 0.0;
            if (q == qk && in_col) {
              if (b == 0)
                wx = 0.0;
              else
                wy = 0.0;
            }
            T.w[2 * (i * Q + q)] = __builtin_fma(-cc, rx[q], wx);
            T.w[2 * (i * Q + q) + 1] = __builtin_fma(-cc, ry[q], wy);
          }
        }
      }
    }
  }
  return bad;
}

// In-place factor of such a matrix A = L D L^T for a solve in two triangular
// products: T ends as L^-1 on and below the diagonal and as its transpose
// above it, dv as 1/D of the rows whose sums the lane gets in tail_solve
// (A^-1 = L^-T D^-1 L^-1). For a component that a set of open switches leaves
// nearly floating, a product with the explicit inverse rounds each row of a
// large common potential by itself, and the differences between nodes are lost
// (6e-8 in a six-pulse bridge; 2e-10 if the rows of L^-1 are scaled by
// D^-1/2); here the common part is one number, injections into a floating
// part cancel exactly, and L^-1 of an M-matrix is formed without
// cancellation. Elimination below the pivot only, one barrier per pivot;
// `tmp` holds d * d doubles of global memory.
template <int BS, int DT>
__device__ __forceinline__ int factor_tail(Tail<BS, DT> &T, int d, double *line, double *tmp,
                                           double (&dv)[(Tail<BS, DT>::R + 3) / 4]) {
  constexpr int G = Tail<BS, DT>::G, R = Tail<BS, DT>::R, Q = Tail<BS, DT>::Q;
  static_assert(DT <= BS, "one lane per pivot's scale");
  constexpr int kBuf = Q * 32 + R * G;
  const int tid = (int)threadIdx.x;
  const int g = tid >> 4, j = tid & 15;
  int bad = 0;
  double scale = 0.0;  // 1/D of pivot tid
#pragma unroll
  for (int k = 0; k < R; ++k) {
    constexpr int kStep = 2;
    const int qk = k * G / 32;
    for (int r0 = 0; r0 < G && k * G + r0 < d; r0 += kStep) {
#pragma unroll
      for (int b = 0; b < kStep; ++b) {
        const int r = r0 + b, p = k * G + r;
        if (p >= d) break;
        double *prow = line + b * kBuf, *pcol = prow + Q * 32;
        const bool in_col = j == ((p & 31) >> 1);
        if (g == r) {
#pragma unroll
          for (int q = 0; q < Q; ++q)
            reinterpret_cast<double2 *>(prow)[16 * q + j] =
                make_double2(T.w[2 * (k * Q + q)], T.w[2 * (k * Q + q) + 1]);
        }
        if (in_col) {
#pragma unroll
          for (int i = k; i < R; ++i) pcol[g + i * G] = T.w[2 * (i * Q + qk) + b];
        }
        step_barrier<BS>();
        const double piv = prow[p];
        const bool ok = piv > 0.0 && piv < INFINITY;
        bad += ok ? 0 : 1;
        const double inv = ok ? 1.0 / piv : 0.0;
        if (tid == p) scale = inv;
        double rx[Q], ry[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const double2 rr = reinterpret_cast<const double2 *>(prow)[16 * q + j];
          rx[q] = rr.x;
          ry[q] = rr.y;
        }
        if (in_col) {
          if (b == 0)
            rx[qk] = 1.0;
          else
            ry[qk] = 1.0;
        }
#pragma unroll
        for (int i = k; i < R; ++i) {
          const bool below = i > k || g > r;
          const double a = below ? pcol[g + i * G] : 0.0;
          // a / piv to the last place: 1 where a floating part's row is the
          // pivot's negative
          double l = a * inv;
          l = __builtin_fma(__builtin_fma(-l, piv, a), inv, l);
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            double wx = T.w[2 * (i * Q + q)], wy = T.w[2 * (i * Q + q) + 1];
            if (q == qk && in_col && below) {
              if (b == 0)
                wx = 0.0;
              else
                wy = 0.0;
            }
            T.w[2 * (i * Q + q)] = __builtin_fma(-l, rx[q], wx);
            T.w[2 * (i * Q + q) + 1] = __builtin_fma(-l, ry[q], wy);
          }
        }
      }
    }
  }
  // the transpose through memory, 1/D through LDS
  __syncthreads();
  if (tid < DT) line[tid] = scale;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int row = g + k * G;
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int col = 32 * q + 2 * j + b;
        if (row >= d || col > row) continue;
        const double a = col == row ? 1.0 : T.w[2 * (k * Q + q) + b];
        tmp[row * d + col] = a;
        tmp[col * d + row] = a;
      }
  }
  __syncthreads();
  load_tail<BS, DT>(tmp, d, T);
#pragma unroll
  for (int k = 0; k < 2 * R * Q; ++k) settle(T.w[k]);
#pragma unroll
  for (int k = 0; k < R; k += 4) {
    const int row = g + (k + (j & 3)) * G;
    dv[k / 4] = row < d ? line[row] : 0.0;
  }
  __syncthreads();  // line and tmp are written again
  return bad;
}

// Factor values and the tail inverse of topology t (values and 1/D in LDS
// under SM, the lane's share of W in VGPRs). U: the closed form's values are
// staged U blocks of a lane at a time.
template <int BS, int DT, bool SM, int U = 1>
__device__ __forceinline__ void select_factor(const DevCtx &c, const ItemDesc &it, View<SM> &v, int t,
                                              Tail<BS, DT> &T) {
  const double *sv = c.svals + it.sv + (int64_t)t * v.nsv;
  const double *di = c.dinv + it.dfac + (int64_t)t * v.n;
  v.svg = sv;
  if constexpr (SM) {
    if constexpr (U > 1) {
      const uint4 *blocks = reinterpret_cast<const uint4 *>(sv);
      copy_blocks<BS, U>(v.sv_s.off, v.lim, [&](int i) { return blocks + i; });
    } else {
      copy_to<BS>(v.sv_s.off, sv, v.closed ? 2 * v.lim : v.nsv);
    }
    if (!v.closed) copy_to<BS>(v.dinv_s.off, di, v.ns);
  } else {
    v.sv.p = sv;
    v.dinv.p = di;
  }
  load_tail<BS, DT>(c.wtail + it.w + (int64_t)t * v.d * v.d, v.d, T);
#pragma unroll
  for (int k = 0; k < 2 * Tail<BS, DT>::R * Tail<BS, DT>::Q; ++k) settle(T.w[k]);
}

// DPP row_shr:K of a double: lane i receives lane i-K of its 16-lane row
// (0 where that lane is outside the row).
template <int K>
__device__ __forceinline__ double dpp_row_shr(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b & 0xffffffffu), 0x110 + K, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x110 + K, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// A double through a DPP control (quad_perm, row_ror) that reads within the
// lane's 16-lane row.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b & 0xffffffffu), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppRor4 = 0x124, kDppRor8 = 0x128;

// Sums of four values over the 16 lanes of a DPP row: on return a lane holds
// the sum of v[lane & 3]. Two halving exchanges leave one value per lane
// pair and quad, which two rotations complete: 33 instructions where four
// separate scans take 48, and the tail's sums are most of its instructions.
__device__ __forceinline__ double sum16x4(double v0, double v1, double v2, double v3, bool b0, bool b1) {
  const double k0 = b0 ? v1 : v0, s0 = b0 ? v0 : v1;  // even lanes keep rows 0 and 2, odd ones 1 and 3
  const double k1 = b0 ? v3 : v2, s1 = b0 ? v2 : v3;
  const double p0 = k0 + dpp_move<kDppXor1>(s0), p1 = k1 + dpp_move<kDppXor1>(s1);
  const double k = b1 ? p1 : p0, s = b1 ? p0 : p1;
  double a = k + dpp_move<kDppXor2>(s);
  a = a + dpp_move<kDppRor4>(a);
  return a + dpp_move<kDppRor8>(a);
}

// Sum over an aligned group of 2^lg <= 16 lanes by a scan of row shifts: the
// group's last lane ends with the sum, always added in the same order (the
// partial sums that reach it are its own group's; other lanes may pick up a
// neighbour group's, which nothing reads).
__device__ __forceinline__ double group_sum(double s, int lg) {
  if (lg >= 1) s = s + dpp_row_shr<1>(s);
  if (lg >= 2) s = s + dpp_row_shr<2>(s);
  if (lg >= 3) s = s + dpp_row_shr<4>(s);
  if (lg >= 4) s = s + dpp_row_shr<8>(s);
  return s;
}

// Runs a row program: per batch a lane adds up its quads' terms (quad(q,
// codes, acc) for the codes of quad q), the lanes of a row meet in the DPP
// scan, and the row's last lane hands the sum to out(row, sum). The rows of
// all batches are independent; the caller places the barriers.
// What bounds a step here is the chain of dependent LDS reads: code, operand,
// sum. The first quad's codes sit in registers, four operands are in flight
// at a time, and the batch word comes from a scalar register. (Row pointers,
// column and operand read one after another, with the level passes' table in
// global memory, took 2.3 us a step on 9-node components and 5.5 us on
// 100-node ones.)
template <bool SM, class F, class O>
__device__ __forceinline__ void run_rows(const Rows<SM> &p, F &&quad, O &&out) {
  if (p.b0 >= p.b1) return;
  const int lane = (int)threadIdx.x & 63;
  auto batch = [&](uint32_t m, uint64_t c, int row) {
    const int q0 = (int)(m & 0xFFFF), q1 = q0 + (int)((m >> 16) & 0xFF), lg = (int)(m >> 24);
    double acc = 0.0;
    quad(q0, c, acc);
    for (int q = q0 + 1; q < q1; ++q) quad(q, p.code[q * 64 + lane], acc);
    if (lg > 0) acc = group_sum(acc, lg);
    if (row != 0xFFFF) out(row, acc);
  };
  batch(p.m0, p.c0, p.r0);
  for (int b = p.b0 + 1; b < p.b1; ++b) {
    const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane(p.word[b]);
    batch(m, p.code[(int)(m & 0xFFFF) * 64 + lane], (int)p.row[b * 64 + lane]);
  }
}

// Gather: r_i = sum of the signed branch injections at node i (with the
// adjoint's program also the seeds of the node's recorded columns).
template <int BS, bool SM>
__device__ __forceinline__ void gather_all(const View<SM> &v) {
  const char *J = emt_lds + v.J.off;
  run_rows<SM>(
      v.gather,
      [&](int, uint64_t c, double &acc) {
        const uint32_t lo = (uint32_t)c, hi = (uint32_t)(c >> 32);
        const uint32_t e[4] = {lo & 0xFFFF, lo >> 16, hi & 0xFFFF, hi >> 16};
        double j[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) j[k] = *reinterpret_cast<const double *>(J + ((e[k] & 0xFFFE) << 2));
#pragma unroll
        for (int k = 0; k < 4; ++k)
          acc = acc + __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, j[k]) ^ ((uint64_t)(e[k] & 1) << 63));
      },
      [&](int row, double s) { v.r[row] = s; });
  step_barrier<BS>();
}

// Row sums of the closed form: sum of value * (right-hand side or solution).
template <bool SM, class O>
__device__ __forceinline__ void value_rows(const View<SM> &v, const Rows<SM> &p, int val0, O &&out) {
  const int lane = (int)threadIdx.x & 63;
  const char *xr = emt_lds + (v.x.off - (uint32_t)(v.n + 1) * 8u);
  run_rows<SM>(
      p,
      [&](int q, uint64_t c, double &acc) {
        const int i = (val0 >> 1) + q * 128 + lane;
        double2 a0, a1;
        if (SM && (val0 >> 1) + q * 128 < v.lim) {
          const double2 *a = reinterpret_cast<const double2 *>(emt_lds + v.sv_s.off);
          a0 = a[i];
          a1 = a[i + 64];
        } else {
          const double2 *a = reinterpret_cast<const double2 *>(v.svg);
          a0 = a[i];
          a1 = a[i + 64];
        }
        const uint32_t lo = (uint32_t)c, hi = (uint32_t)(c >> 32);
        const double x0 = *reinterpret_cast<const double *>(xr + ((lo & 0xFFFF) << 3));
        const double x1 = *reinterpret_cast<const double *>(xr + ((lo >> 16) << 3));
        const double x2 = *reinterpret_cast<const double *>(xr + ((hi & 0xFFFF) << 3));
        const double x3 = *reinterpret_cast<const double *>(xr + ((hi >> 16) << 3));
        acc = __builtin_fma(a0.x, x0, acc);
        acc = __builtin_fma(a0.y, x1, acc);
        acc = __builtin_fma(a1.x, x2, acc);
        acc = __builtin_fma(a1.y, x3, acc);
      },
      out);
}

// One forward pass: for each row descriptor (r, q0, cnt) the row's lanes
// sum sv[q] x[fcol[q]] over their strided entries; out[r - shift] =
// x[r] - sum (out = x for the leading levels, cD with shift ns for the tail
// rows).
template <int BS, bool SM>
__device__ __forceinline__ void forward_pass(const View<SM> &v, int p0, int p1, int lg, uint32_t out_off,
                                             int shift) {
  const int tid = lane_id();
  const int G = 1 << lg, sub = tid & (G - 1);
  for (int p = p0 + (tid >> lg); p < p1; p += (BS >> lg)) {
    const uint64_t dsc = v.fdesc[p];
    const int r = (int)(dsc & 0xFFFF), q0 = (int)((dsc >> 16) & 0xFFFF), cnt = (int)(dsc >> 32);
    const double xr = v.x[r];
    double s = 0.0;
    int q = q0 + sub;
    const int q1 = q0 + cnt;
    for (; q + G < q1; q += 2 * G) {
      const int c0 = v.fcol[q], c1 = v.fcol[q + G];
      const double a0 = v.sv[q], a1 = v.sv[q + G];
      const double x0 = v.x[c0], x1 = v.x[c1];
      s = s + a0 * x0;
      s = s + a1 * x1;
    }
    if (q < q1) s = s + v.sv[q] * v.x[v.fcol[q]];
    s = group_sum(s, lg);
    if (sub == G - 1) reinterpret_cast<double *>(emt_lds + out_off)[r - shift] = xr - s;
  }
  step_barrier<BS>();
}

// One backward pass: x_r = x_r / D_r - sum over the row's column entries of
// sv[bpos[q]] x[brow[q]].
template <int BS, bool SM>
__device__ __forceinline__ void backward_pass(const View<SM> &v, int p0, int p1, int lg) {
  const int tid = lane_id();
  const int G = 1 << lg, sub = tid & (G - 1);
  for (int p = p0 + (tid >> lg); p < p1; p += (BS >> lg)) {
    const uint64_t dsc = v.bdesc[p];
    const int r = (int)(dsc & 0xFFFF), q0 = (int)((dsc >> 16) & 0xFFFF), cnt = (int)(dsc >> 32);
    const double xr = v.x[r] * v.dinv[r];
    double s = 0.0;
    int q = q0 + sub;
    const int q1 = q0 + cnt;
    for (; q + G < q1; q += 2 * G) {
      const int i0 = v.bpos[q], i1 = v.bpos[q + G];
      const int r0 = v.brow[q], r1 = v.brow[q + G];
      const double a0 = v.sv[i0], a1 = v.sv[i1];
      const double x0 = v.x[r0], x1 = v.x[r1];
      s = s + a0 * x0;
      s = s + a1 * x1;
    }
    if (q < q1) s = s + v.sv[v.bpos[q]] * v.x[v.brow[q]];
    s = group_sum(s, lg);
    if (sub == G - 1) v.x[r] = xr - s;
  }
  step_barrier<BS>();
}

// x_D = W c (the layout is Tail's).
template <int BS, int DT, bool SM>
__device__ __forceinline__ void tail_solve(const View<SM> &v, const Tail<BS, DT> &T) {
  constexpr int G = Tail<BS, DT>::G, R = Tail<BS, DT>::R, Q = Tail<BS, DT>::Q;
  const int tid = lane_id();
  const int g = tid >> 4, j = tid & 15;
  const double2 *c = reinterpret_cast<const double2 *>(emt_lds + v.cD.off);
  const bool b0 = j & 1, b1 = j & 2;
  double2 cc[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) cc[q] = c[16 * q + j];
  // rows in fours
#pragma unroll
  for (int k0 = 0; k0 < R; k0 += 4) {
    if (k0 > 0 && k0 * G >= v.d) break;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (q > 0 && 32 * q >= v.d) break;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (k0 + k >= R) continue;
        acc[k] = __builtin_fma(T.w[2 * ((k0 + k) * Q + q)], cc[q].x, acc[k]);
        acc[k] = __builtin_fma(T.w[2 * ((k0 + k) * Q + q) + 1], cc[q].y, acc[k]);
      }
    }
    const double sum = sum16x4(acc[0], acc[1], acc[2], acc[3], b0, b1);
    const int row = g + (k0 + j) * G;
    if (j < 4 && row < v.d) v.x[v.ns + row] = sum;
  }
  step_barrier<BS>();
}

// x_D = L^-T (D^-1 (L^-1 c)) with factor_tail's layout: two triangular
// products, the vector between them in `line`. Blocks of a register row wholly on one side
// of the diagonal take part in one of them only.
template <int BS, int DT, bool SM>
__device__ __forceinline__ void tail_solve_factored(const View<SM> &v, const Tail<BS, DT> &T, const double *dv) {
  constexpr int G = Tail<BS, DT>::G, R = Tail<BS, DT>::R, Q = Tail<BS, DT>::Q;
  const int tid = lane_id();
  const int g = tid >> 4, j = tid & 15;
  const bool b0 = j & 1, b1 = j & 2;
  auto product = [&](int in, bool lower, auto out) {
    const double2 *c = reinterpret_cast<const double2 *>(emt_lds + in);
    double2 cc[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) cc[q] = c[16 * q + j];
#pragma unroll
    for (int k0 = 0; k0 < R; k0 += 4) {
      if (k0 > 0 && k0 * G >= v.d) break;
      double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (q > 0 && 32 * q >= v.d) break;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int first = (k0 + k) * G, last = first + G - 1;  // the register row's rows
          if (k0 + k >= R || (lower ? last < 32 * q : first > 32 * q + 31)) continue;
          double cx = cc[q].x, cy = cc[q].y;
          if (lower ? first < 32 * q + 31 : last > 32 * q) {
            const int row = g + first, col = 32 * q + 2 * j;
            if (lower ? col > row : col < row) cx = 0.0;
            if (lower ? col + 1 > row : col + 1 < row) cy = 0.0;
          }
          acc[k] = __builtin_fma(T.w[2 * ((k0 + k) * Q + q)], cx, acc[k]);
          acc[k] = __builtin_fma(T.w[2 * ((k0 + k) * Q + q) + 1], cy, acc[k]);
        }
      }
      const double sum = sum16x4(acc[0], acc[1], acc[2], acc[3], b0, b1);
      if (j < 4) out(g + (k0 + j) * G, k0 / 4, sum);
    }
    step_barrier<BS>();
  };
  product(v.cD.off, true, [&](int row, int k, double s) {
    if (row < Q * 32) v.line[row] = s * dv[k];  // zero past d
  });
  product(v.line.off, false, [&](int row, int, double s) {
    if (row < v.d) v.x[v.ns + row] = s;
  });
}

// The solve after the gather: closed form (c = r_D + N r_S, x_D = W c,
// x_S = Q r_S + N^T x_D; a component that is all tail gathers straight into
// c), or the level passes around the tail.
template <int BS, int DT, bool SM, int LEV, bool SW = false>
__device__ __forceinline__ void solve_after_gather(const View<SM> &v, const Tail<BS, DT> &T, const double *dv = nullptr,
                                                   bool factored = false) {
  if (LEV != LEVELS && (LEV == CLOSED || v.closed)) {
    if (v.d > 0) {
      if (v.ns > 0) {
        value_rows<SM>(v, v.fwd, 0, [&](int row, double s) { v.cD[row] = s; });
        step_barrier<BS>();
      }
      if (SW && factored)
        tail_solve_factored<BS, DT, SM>(v, T, dv);
      else
        tail_solve<BS, DT, SM>(v, T);
    }
    if (v.ns > 0) {
      value_rows<SM>(v, v.bwd, v.fvals, [&](int row, double s) { v.x[row] = s; });
      step_barrier<BS>();
    }
    return;
  }
  // from LDS the table's entries go to scalar registers; a uniform load from
  // memory the compiler moves there itself where it pays (1000 buses, solver
  // sparse: 269 us a step with every entry moved, 263 without, in a kernel that
  // carried the closed form's code as well; 244 in the present one)
  auto pass = [](const Ref<int32_t, SM> &p, int i) {
    if constexpr (SM)
      return __builtin_amdgcn_readfirstlane(p[i]);
    else
      return (int)p[i];
  };
  for (int k = 0; k < v.nfpass; ++k) {
    const int p0 = pass(v.fpass, 2 * k), lg = pass(v.fpass, 2 * k + 1), p1 = pass(v.fpass, 2 * k + 2);
    // the last forward pass of an item with a dense tail is the tail rows'
    const bool tail_rows = v.d > 0 && k == v.nfpass - 1;
    forward_pass<BS, SM>(v, p0, p1, lg, tail_rows ? v.cD.off : v.x.off, tail_rows ? v.ns : 0);
  }
  if (v.d > 0) tail_solve<BS, DT, SM>(v, T);
  for (int k = 0; k < v.nbpass; ++k) {
    const int p0 = pass(v.bpass, 2 * k), lg = pass(v.bpass, 2 * k + 1), p1 = pass(v.bpass, 2 * k + 2);
    backward_pass<BS, SM>(v, p0, p1, lg);
  }
}

// Lane state of the forward loop: coefficients of the current topology for
// each slot (branches padded to whole slots with inert ones, so every slot
// is valid) and the history current of slot 0. The history of the other
// slots lives in LDS as their injection: a slot j > 0 carries no source, so
// J = -h there exactly and h = -J is read back where it is needed.
template <int BPT>
struct Lane {
  double g[BPT], be[BPT], h0;
  uint32_t pk[BPT];
  // EMF of the current step of slot 0 (sources are numbered first and fit in
  // one slot; 0 elsewhere)
  double e0;
  // EMF table (View::emf): the EMFs of `eper` steps at a time, one per lane
  // (this lane's source, and step offset ek, -1: none).
  // A cosine is a chain of about 25 dependent FP64 operations; evaluated by
  // the source lanes each step it stood in the branch update's way.
  double sE, sw, sph;
  int ek, eper, enext;  // enext: the next step's place in the table
  double ed;            // without the table: the next step's EMF
};

template <int BS, int BPT>
__device__ __forceinline__ void load_lane(const DevCtx &c, const ItemDesc &it, Lane<BPT> &L) {
#pragma unroll
  for (int j = 0; j < BPT; ++j) L.pk[j] = c.bpack[it.br + threadIdx.x + j * BS];
  L.eper = it.n_src > 0 ? __builtin_amdgcn_readfirstlane(BS / it.n_src) : 0;
  const int k = it.n_src > 0 ? (int)threadIdx.x / it.n_src : 0;
  const bool src = it.n_src > 0 && k < L.eper;
  const int64_t b = it.br + (src ? (int)threadIdx.x - k * it.n_src : 0);
  L.ek = src ? k : -1;
  L.sE = src ? c.bE[b] : 0.0;
  L.sw = src ? c.bw[b] : 0.0;
  L.sph = src ? c.bph[b] : 0.0;
  L.e0 = 0.0;
  L.enext = 0;
}

// Moves the EMF table's place on to step n, filling the table from there
// when it is used up or `fresh` (a barrier must follow before it is read,
// and one lie between its last reader and this call).
template <int BPT, bool SM>
__device__ __forceinline__ void emf_advance(const DevCtx &c, const View<SM> &v, Lane<BPT> &L, int64_t n, bool fresh) {
  if constexpr (!SM) {
    if (v.emf_direct) {
      L.ed = (int)threadIdx.x < v.nsrc ? L.sE * emf_cos(L.sw * ((double)n * c.dt) + L.sph) : 0.0;
      return;
    }
  }
  if (L.eper == 0) return;
  if (!fresh && ++L.enext < L.eper) return;
  L.enext = 0;
  if (L.ek >= 0) v.emf[(int)threadIdx.x] = L.sE * emf_cos(L.sw * ((double)(n + L.ek) * c.dt) + L.sph);
}

template <int BS, int BPT>
__device__ __forceinline__ void load_coefs(const DevCtx &c, const ItemDesc &it, int t, double (&g)[BPT],
                                           double (&be)[BPT]) {
  const int64_t base = it.coef + (int64_t)t * it.n_br;
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    g[j] = c.cg[base + threadIdx.x + j * BS];
    be[j] = c.cb[base + threadIdx.x + j * BS];
  }
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    settle(g[j]);
    settle(be[j]);
  }
}

// History current h = beta*i + gamma*u from a stored state (i, u).
// History of the next step from a stored state (i, u): slot 0 into L.h0,
// the other slots straight into their injections J = -h.
template <int BS, int BPT, bool SM>
__device__ __forceinline__ void history_from_state(const double *si, const double *su, Lane<BPT> &L,
                                                   const View<SM> &v) {
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    const int b = threadIdx.x + j * BS;
    const double h = L.be[j] * si[b] + gamma_of(L.pk[j], L.g[j]) * su[b];
    if (j == 0)
      L.h0 = h;
    else
      v.J[b] = -h;
  }
}

// EMF at the table's place for the lane's slot-0 branch (0 if it is not a
// source).
template <int BPT, bool SM>
__device__ __forceinline__ double slot0_emf(const View<SM> &v, const Lane<BPT> &L, int tid) {
  if constexpr (!SM) {
    if (v.emf_direct) return L.ed;
  }
  return tid < v.nsrc ? v.emf[L.enext * v.nsrc + tid] : 0.0;
}

// Slot 0's injection of step n: J = g e - h (the other slots' injections
// were written with their history).
template <int BS, int BPT, bool SM>
__device__ __forceinline__ void inject(const DevCtx &c, const View<SM> &v, Lane<BPT> &L, int64_t n) {
  const int tid = lane_id();
  emf_advance<BPT, SM>(c, v, L, n, true);
  step_barrier<BS>();
  L.e0 = slot0_emf<BPT, SM>(v, L, tid);
  v.J[tid] = L.g[0] * L.e0 - L.h0;
}

// A trajectory row: the node voltages of the step just solved and the EMFs
// that entered it.
template <int BS, int BPT, bool SM>
__device__ __forceinline__ void store_row(const View<SM> &v, const Lane<BPT> &L, double *row) {
  const int tid = (int)threadIdx.x;
  for (int r = tid; r < v.n; r += BS) row[r] = v.x[r];
  if (tid < v.nsrc) row[v.n + tid] = L.e0;
}

// Branch phase of a step after which no coefficients change and which is
// not the launch's last: the same arithmetic as update_inject below without
// its cases (each a branch that every step would take). STORE: i of every
// slot goes to st_i. Slot pairs that are all padding are skipped (components
// of an uneven batch are padded to the largest one's slots).
template <int BS, int BPT, bool SM, bool STORE, bool PASS = false>
__device__ __forceinline__ void update_plain(const View<SM> &v, Lane<BPT> &L, double *st_i) {
  const int tid = lane_id();
  const double e_next = slot0_emf<BPT, SM>(v, L, tid);
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    if (j > 0 && (j & 1) == 0 && j * BS >= v.nreal) break;
    const int b = tid + j * BS;
    const uint32_t pk = L.pk[j];
    const double vk = v.x[pk & kTermGround], vm = v.x[(pk >> 15) & kTermGround];
    const bool pass = PASS && (pk >> 30) == GAMMA_PASS;
    const double h = (j == 0 && !pass) ? L.h0 : -v.J[b];
    const double u = j == 0 ? (vk - vm) - L.e0 : vk - vm;
    const double gu = L.g[j] * u;
    const double i = gu + h;
    if constexpr (STORE) st_i[b] = i;
    const double hn = L.be[j] * i + gamma_times(pk, gu);
    if (j == 0) {
      L.h0 = hn;
      if (!pass) v.J[b] = L.g[j] * e_next - hn;
    } else if (!pass) {
      v.J[b] = -hn;
    }
  }
  L.e0 = e_next;
}

// Branch phase after the solve of step n: u, i of step n with the current
// coefficients; optional stores of (i, u) to up to two places (null = none);
// if step n+1 starts a new topology its coefficients are loaded; the history
// of step n+1; and, when inj is set, the injections of step n+1.
template <int BS, int BPT, bool SM, bool PASS = false>
__device__ __forceinline__ void update_inject(const DevCtx &c, const View<SM> &v, Lane<BPT> &L, double *st_i,
                                              double *st_u, double *st2_i, double *st2_u, bool switch_next,
                                              int64_t next_coef, bool inj, int64_t n) {
  const int tid = lane_id();
  const double e_next = inj ? slot0_emf<BPT, SM>(v, L, tid) : 0.0;
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    const int b = tid + j * BS;
    const uint32_t pk = L.pk[j];
    // a line end's or a coupled member's history is its injection in every
    // slot (no source there), and a pass after this update, not the update,
    // writes its next injection and its stored state (PASS: the batch has
    // such branches; the kernels of other batches carry none of this)
    const bool line = PASS && (pk >> 30) == GAMMA_PASS;
    const double vk = v.x[pk & kTermGround], vm = v.x[(pk >> 15) & kTermGround];
    const double h = (j == 0 && !line) ? L.h0 : -v.J[b];
    double u = j == 0 ? (vk - vm) - L.e0 : vk - vm;
    // u of a branch out of service is 0; its coefficients are 0 too, so only
    // a stored state or a change of coefficients sees it
    if ((st_i || st2_i || switch_next) && L.g[j] == 0.0) u = 0.0;
    const double gu = L.g[j] * u;
    const double i = gu + h;
    if (st_i && !line) {
      st_i[b] = i;
      if (st_u) st_u[b] = u;
    }
    if (st2_i && !line) {
      st2_i[b] = i;
      st2_u[b] = u;
    }
    if (switch_next) {
      L.g[j] = c.cg[next_coef + b];
      L.be[j] = c.cb[next_coef + b];
      settle(L.g[j]);
      settle(L.be[j]);
    }
    const double gam = switch_next ? gamma_of(pk, L.g[j]) * u : gamma_times(pk, gu);
    const double hn = L.be[j] * i + gam;
    if (j == 0) {
      L.h0 = hn;
      if (inj && !line) v.J[b] = L.g[j] * e_next - hn;
    } else if (inj && !line) {
      v.J[b] = -hn;
    }
  }
  L.e0 = e_next;
}

// Distributed-parameter lines, one lane per line. Each end is a Norton
// equivalent to ground (1/Z) whose history current is the wave that left the
// other end tau = (D0 + f) dt earlier: h_k(n) = -[(1 - f) w_m(n - D0) +
// f w_m(n - D0 - 1)], w = g v + i, i = g v + h, w = 0 up to step 0 (the line
// starts at rest).
// The two ends' waves of a step are one 16-byte entry of the line's ring;
// the rings of all lines of one length are interleaved by step (device.h,
// LineDesc), so that neighbouring lanes, whose lines have neighbouring
// delays, read and write neighbouring entries. A lane keeps its first
// kLineRegs lines' descriptors in registers, carries the entry of step
// n - D0 over to the next step, where it is the one of n - D0 - 1, and reads
// the entry of n + 1 - D0 ahead of the solve (of D0 = 1 lines it is the one
// just formed). With a ring per end, descriptors read every step and four
// ring reads after the branch update, this pass was two dependent trips to
// L2 and 64 memory requests per wave and access: 3 of the 7.7 us of a step
// with 1350 lines.
constexpr int kLineRegs = 3, kGroupRegs = 2;

struct LineLane {
  uint32_t br, nd;  // local branches and nodes, k end | m end << 16
  int d0, mask, stride;
  double g, f;
  double2 *ring;  // the line's entry of slot 0
  double2 prev, ahead;
};

__device__ __forceinline__ double2 *ring_at(const LineLane &l, int64_t n) {
  return l.ring + (int64_t)((int)n & l.mask) * l.stride;
}
__device__ __forceinline__ double2 ring_read(const LineLane &l, int64_t n) {
  return n > 0 ? *ring_at(l, n) : make_double2(0.0, 0.0);
}

__device__ __forceinline__ void line_load(const DevCtx &c, const ItemDesc &it, int q, LineLane &l) {
  const LineDesc d = c.line_tab[it.lines + q];
  l.br = (uint32_t)d.bk | ((uint32_t)d.bm << 16);
  l.nd = (uint32_t)d.nk | ((uint32_t)d.nm << 16);
  l.d0 = d.d0;
  l.mask = d.mask;
  l.stride = d.stride;
  l.g = c.line_gf[2 * (it.lines + q)];
  l.f = c.line_gf[2 * (it.lines + q) + 1];
  l.ring = reinterpret_cast<double2 *>(c.ring + d.ring);
}

// The ends' injections of a step from the entries of n - D0 (now) and
// n - D0 - 1 (before).
template <bool SM>
__device__ __forceinline__ void line_inject(const View<SM> &v, const LineLane &l, double2 now, double2 before) {
  v.J[(int)(l.br & 0xFFFF)] = (1.0 - l.f) * now.y + l.f * before.y;
  v.J[(int)(l.br >> 16)] = (1.0 - l.f) * now.x + l.f * before.x;
}

// A line's injections of step n at the start of a launch.
template <bool SM>
__device__ __forceinline__ void line_start(const View<SM> &v, LineLane &l, int64_t n) {
  const double2 now = ring_read(l, n - l.d0);
  line_inject<SM>(v, l, now, ring_read(l, n - l.d0 - 1));
  l.prev = now;
}

// A line after the solve of step n: the waves of step n stored, the ends'
// state of step n (when st_i is set), the injections of step n + 1.
template <bool SM>
__device__ __forceinline__ void line_step(const View<SM> &v, LineLane &l, int64_t n, double *st_i, double *st_u) {
  const double vk = v.x[(int)(l.nd & 0xFFFF)], vm = v.x[(int)(l.nd >> 16)];
  const double ik = l.g * vk - v.J[(int)(l.br & 0xFFFF)], im = l.g * vm - v.J[(int)(l.br >> 16)];
  const double2 w = make_double2(l.g * vk + ik, l.g * vm + im);
  *ring_at(l, n) = w;
  if (st_i) {  // each end's current into the line and its voltage
    st_i[(int)(l.br & 0xFFFF)] = ik;
    st_u[(int)(l.br & 0xFFFF)] = vk;
    st_i[(int)(l.br >> 16)] = im;
    st_u[(int)(l.br >> 16)] = vm;
  }
  const double2 now = l.d0 == 1 ? w : l.ahead;
  line_inject<SM>(v, l, now, l.prev);
  l.prev = now;
}

// A lane's lines: the first NL in registers, any more through memory.
template <int NL>
struct Lines {
  LineLane l[NL > 0 ? NL : 1];
};

template <int BS, int NL, bool SM>
__device__ __forceinline__ void lines_start(const DevCtx &c, const ItemDesc &it, const View<SM> &v, Lines<NL> &R,
                                            int64_t n) {
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int q = (int)threadIdx.x + k * BS;
    if (q >= it.n_lines) break;
    line_load(c, it, q, R.l[k]);
    line_start<SM>(v, R.l[k], n);
  }
  for (int q = (int)threadIdx.x + NL * BS; q < it.n_lines; q += BS) {
    LineLane l;
    line_load(c, it, q, l);
    line_start<SM>(v, l, n);
  }
}

// Reads ahead of the solve of step n.
template <int BS, int NL>
__device__ __forceinline__ void lines_ahead(const ItemDesc &it, Lines<NL> &R, int64_t n) {
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    if ((int)threadIdx.x + k * BS >= it.n_lines) break;
    R.l[k].ahead = R.l[k].d0 > 1 ? ring_read(R.l[k], n + 1 - R.l[k].d0) : make_double2(0.0, 0.0);
  }
}

// Waits for these reads (before the step's own stores are queued behind
// them).
template <int BS, int NL>
__device__ __forceinline__ void lines_settle(const ItemDesc &it, Lines<NL> &R) {
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    if (k * BS >= it.n_lines) break;
    settle(R.l[k].ahead.x);
    settle(R.l[k].ahead.y);
  }
}

template <int BS, int NL, bool SM>
__device__ __forceinline__ void lines_step(const DevCtx &c, const ItemDesc &it, const View<SM> &v, Lines<NL> &R,
                                           int64_t n, double *st_i, double *st_u) {
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    if ((int)threadIdx.x + k * BS >= it.n_lines) break;
    line_step<SM>(v, R.l[k], n, st_i, st_u);
  }
  for (int q = (int)threadIdx.x + NL * BS; q < it.n_lines; q += BS) {
    LineLane l;
    line_load(c, it, q, l);
    l.prev = ring_read(l, n - l.d0);
    l.ahead = l.d0 > 1 ? ring_read(l, n + 1 - l.d0) : make_double2(0.0, 0.0);
    line_step<SM>(v, l, n, st_i, st_u);
  }
}

// Coupled three-phase groups, one lane per group. A member's current and
// history involve all three members through the circulant companion: with
// the group sums S_u, S_i,
//   i_p  = g u_p + g_o (S_u - u_p) + h_p,
//   h'_p = beta i_p + sgn g u_p + beta_o (S_i - i_p) + sgn g_o (S_u - u_p),
// sgn = +1 for R-L and -1 for C groups. Members carry no source (u = v_k -
// v_m); the branch update leaves their injections and stored state to this
// pass, which reads h_p = -J and writes J = -h'_p (when inj) and the state
// (when st_i is set). With init, (i, u) are the stored state instead (the
// start of a launch) and only the injections are written. The members take
// no events, so the coefficients of topology 0 hold in every topology. A
// lane's first kGroupRegs groups' descriptors and coefficients stay in
// registers.
struct GroupLane {
  uint32_t b01, b2, t[3];  // members' branches (b2's bit 16: a C group); terminals k | m << 16
  double g, go, be, bo;
  __device__ __forceinline__ int b(int p) const {
    return (int)(p == 0 ? b01 & 0xFFFF : (p == 1 ? b01 >> 16 : b2 & 0xFFFF));
  }
};

__device__ __forceinline__ void group_load(const DevCtx &c, const ItemDesc &it, int q, GroupLane &l) {
  const GroupDesc d = c.group_tab[it.groups + q];
  l.b01 = (uint32_t)d.b[0] | ((uint32_t)d.b[1] << 16);
  l.b2 = (uint32_t)d.b[2] | (d.sgn < 0 ? 0x10000u : 0u);
#pragma unroll
  for (int p = 0; p < 3; ++p) l.t[p] = (uint32_t)d.k[p] | ((uint32_t)d.m[p] << 16);
  const int64_t k0 = it.coef + d.b[0];
  l.g = c.cg[k0];
  l.go = c.cgo[k0];
  l.be = c.cb[k0];
  l.bo = c.cbo[k0];
}

template <bool SM>
__device__ __forceinline__ void group_step(const DevCtx &c, const ItemDesc &it, const View<SM> &v,
                                           const GroupLane &l, bool init, bool inj, double *st_i, double *st_u) {
  const double sg = (l.b2 >> 16) ? -1.0 : 1.0;
  double u[3], i[3];
  if (init) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      u[p] = c.su[it.br + l.b(p)];
      i[p] = c.si[it.br + l.b(p)];
    }
  } else {
#pragma unroll
    for (int p = 0; p < 3; ++p) u[p] = v.x[(int)(l.t[p] & 0xFFFF)] - v.x[(int)(l.t[p] >> 16)];
    const double su = u[0] + u[1] + u[2];
#pragma unroll
    for (int p = 0; p < 3; ++p) i[p] = (l.g * u[p] - v.J[l.b(p)]) + l.go * (su - u[p]);
    if (st_i) {
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        st_i[l.b(p)] = i[p];
        st_u[l.b(p)] = u[p];
      }
    }
  }
  if (init || inj) {
    const double su = u[0] + u[1] + u[2], si = i[0] + i[1] + i[2];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const double h = (l.be * i[p] + sg * l.g * u[p]) + (l.bo * (si - i[p]) + sg * l.go * (su - u[p]));
      v.J[l.b(p)] = -h;
    }
  }
}

template <int NG>
struct Groups {
  GroupLane l[NG > 0 ? NG : 1];
};

template <int BS, int NG>
__device__ __forceinline__ void groups_load(const DevCtx &c, const ItemDesc &it, Groups<NG> &R) {
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    const int q = (int)threadIdx.x + k * BS;
    if (q >= it.n_groups) break;
    group_load(c, it, q, R.l[k]);
    settle(R.l[k].g);
    settle(R.l[k].go);
    settle(R.l[k].be);
    settle(R.l[k].bo);
  }
}

template <int BS, int NG, bool SM>
__device__ __forceinline__ void groups_step(const DevCtx &c, const ItemDesc &it, const View<SM> &v, const Groups<NG> &R,
                                            bool init, bool inj, double *st_i, double *st_u) {
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    if ((int)threadIdx.x + k * BS >= it.n_groups) break;
    group_step<SM>(c, it, v, R.l[k], init, inj, st_i, st_u);
  }
  for (int q = (int)threadIdx.x + NG * BS; q < it.n_groups; q += BS) {
    GroupLane l;
    group_load(c, it, q, l);
    group_step<SM>(c, it, v, l, init, inj, st_i, st_u);
  }
}

// Ideal diodes (state-dependent switches). A diode is a resistive branch
// whose conductance is 1/R_on while it conducts and 0 while it blocks; its
// state lives in c.dstate and changes after a step (a conducting diode whose
// current g u went negative blocks, a blocking one whose voltage v_k - v_m
// went positive conducts), taking effect from the next step. dmask marks a
// lane's diode and controlled-switch slots, cmask the latter: a controlled
// switch's hysteresis comparator measures s = v_a - v_b of step n against
// its reference r = E cos(omega n dt + phase) + C and, with e = r - s,
// conducts from the next step if e > h, opens if e < -h, else keeps its
// state (h in the branch's L). Returns the slots that change; their new
// state is stored at once, their conductance only after the branch update
// of this step (which still uses the old one).
template <int BS, int BPT, bool SM>
__device__ __forceinline__ uint32_t diode_flips(const DevCtx &c, const ItemDesc &it, const View<SM> &v,
                                                const Lane<BPT> &L, uint32_t dmask, uint32_t cmask, int64_t n) {
  uint32_t fl = 0;
  const int tid = lane_id();
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    if (!((dmask >> j) & 1u)) continue;
    const bool on = L.g[j] != 0.0;
    bool next;
    if ((cmask >> j) & 1u) {
      const int64_t gb = it.br + tid + j * BS;
      const double s = v.x[c.bmeas[2 * gb]] - v.x[c.bmeas[2 * gb + 1]];
      const double r = c.bE[gb] * emf_cos(c.bw[gb] * ((double)n * c.dt) + c.bph[gb]) + c.bC[gb];
      const double e = r - s, h = c.bL[gb];
      next = e > h ? true : (e < -h ? false : on);
    } else {
      const uint32_t pk = L.pk[j];
      const double du = v.x[pk & kTermGround] - v.x[(pk >> 15) & kTermGround];
      next = on ? !(L.g[j] * du < 0.0) : (du > 0.0);
    }
    if (next != on) {
      fl |= 1u << j;
      c.dstate[it.br + tid + j * BS] = next ? 1 : 0;
    }
  }
  return fl;
}

// Diodes and controlled switches of a closed-form item (the rules are
// diode_flips'), one lane each, whose parameters and state stay in registers;
// any past BS lanes go through memory. A change is noted in the stored state,
// the conductance list and the flag; the tail's matrix and the branch slots
// follow at the start of the next step.
struct SwitchLane {
  SwitchDesc d;
  double E, w, ph, C, h, gon, ref;
  bool on;
};

__device__ __forceinline__ void switch_load(const DevCtx &c, const ItemDesc &it, int q, SwitchLane &s) {
  s.d = c.sw_tab[it.swt + q];
  const int64_t gb = it.br + s.d.br;
  s.E = c.bE[gb];
  s.w = c.bw[gb];
  s.ph = c.bph[gb];
  s.C = c.bC[gb];
  s.h = c.bL[gb];
  s.gon = 1.0 / c.bR[gb];
  s.on = c.dstate[gb] != 0;
}

// A controlled switch's reference at step n (ahead of the solve).
__device__ __forceinline__ void switch_reference(const DevCtx &c, SwitchLane &s, int64_t n) {
  if (!s.d.control) return;
  s.ref = s.C;
  if (s.E != 0.0) s.ref = s.E * emf_cos(s.w * ((double)n * c.dt) + s.ph) + s.C;
}

// The state from step n + 1 on.
template <bool SM>
__device__ __forceinline__ void switch_step(const DevCtx &c, const ItemDesc &it, const View<SM> &v, SwitchLane &s,
                                            int q, int64_t n) {
  bool next;
  if (s.d.control) {
    const double e = s.ref - (v.x[s.d.a] - v.x[s.d.b]);
    next = e > s.h ? true : (e < -s.h ? false : s.on);
  } else {
    const double du = v.x[s.d.k] - v.x[s.d.m];
    next = s.on ? !(s.gon * du < 0.0) : (du > 0.0);
  }
  if (next != s.on) {
    s.on = next;
    c.dstate[it.br + s.d.br] = next ? 1 : 0;
    v.gsw[q] = next ? s.gon : 0.0;
    v.swflag[0] = (int)n;
  }
}

// The tail's factor of a closed-form item with switches: their conductances
// stamped on the tail's matrix S (k_closed left a copy per topology in the
// item's scratch), factorised in the lanes' registers (factor_tail). The clusters' parts Q and N do not see
// them. One barrier per pivot of the tail, about 450 cycles each, against two
// barriers of about 2 us per level of the whole elimination tree (and no
// dense tail for the steps in between) when the component was factorised
// anew.
template <int BS, int DT, bool SM>
__device__ __forceinline__ void refactor_tail(const DevCtx &c, const ItemDesc &it, const View<SM> &v, int t,
                                              Tail<BS, DT> &w, double (&dv)[(Tail<BS, DT>::R + 3) / 4]) {
  const int d = v.d;
  const double *S0 = c.wtail + it.w + (int64_t)t * d * d;
  double *S = c.dyn + it.dyn + (int64_t)t * d * d;
  for (int k = (int)threadIdx.x; k < it.n_swkey; k += BS) {
    const int key = c.symi[it.swkey + k], e1 = c.symi[it.swptr + k + 1];
    double s = S0[key];
    for (int e = c.symi[it.swptr + k]; e < e1; ++e) {
      const int term = c.symi[it.swterm + e];
      const double g = v.gsw[term >> 1];
      s = (term & 1) ? s - g : s + g;
    }
    S[key] = s;
  }
  __syncthreads();
  load_tail<BS, DT>(S, d, w);
#pragma unroll
  for (int k = 0; k < 2 * Tail<BS, DT>::R * Tail<BS, DT>::Q; ++k) settle(w.w[k]);
  const int bad = factor_tail<BS, DT>(w, d, reinterpret_cast<double *>(emt_lds + v.line.off),
                                      c.dyn + it.dyn + (int64_t)it.n_topo * d * d, dv);
  if (bad && threadIdx.x == 0) atomicAdd(c.flags + 4, bad);
}

// The diode slots' conductances from their stored state.
template <int BS, int BPT>
__device__ __forceinline__ void diode_conductances(const DevCtx &c, const ItemDesc &it, Lane<BPT> &L,
                                                   uint32_t dmask) {
  const int tid = lane_id();
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    if (!((dmask >> j) & 1u)) continue;
    const int64_t gb = it.br + tid + j * BS;
    L.g[j] = c.dstate[gb] ? 1.0 / c.bR[gb] : 0.0;
    L.be[j] = 0.0;
  }
}

// A workgroup barrier for data in LDS (SM) or in global memory.
template <bool SM>
__device__ __forceinline__ void wg_sync() {
  if constexpr (SM)
    lds_barrier();
  else
    __syncthreads();
}

// log2 of the lanes that share one row or entry of a factorisation level
// with cnt of them: as many as fill the workgroup, at most 16 (one DPP row).
template <int BS>
__device__ __forceinline__ int team_log2(int cnt) {
  int lg = 0;
  while (lg < 4 && (cnt << (lg + 1)) <= BS) ++lg;
  return lg;
}

// A lane's first entry of a factorisation level: its CSR position and the
// range of its share of the entry's update pairs (start already offset by
// the lane's index in its team), fetched one level ahead, and its first
// PC pairs, fetched at the start of the level, so that neither global
// load waits inside the level. Pairs are read PC at a time.
template <int PC>
struct LevelEntry {
  int p, pos, r, r1, lg;
  uint32_t pr[PC];
};

template <int BS, int PC, class LV>
__device__ __forceinline__ LevelEntry<PC> first_entry(const LV &fent_ptr, int l, const int32_t *rent) {
  const int e0 = fent_ptr[l], e1 = fent_ptr[l + 1];
  LevelEntry<PC> f;
  f.lg = team_log2<BS>(e1 - e0);
  f.p = e0 + ((int)threadIdx.x >> f.lg);
  f.pos = 0;
  f.r = f.r1 = 0;
  if (f.p < e1) {
    f.pos = rent[2 * f.p];
    f.r = rent[2 * f.p + 1] + ((int)threadIdx.x & ((1 << f.lg) - 1));
    f.r1 = rent[2 * f.p + 3];
  }
  return f;
}

template <int PC>
__device__ __forceinline__ void load_pairs(uint32_t (&pr)[PC], const uint32_t *rpair, int r, int r1, int g) {
#pragma unroll
  for (int u = 0; u < PC; ++u) pr[u] = (r + u * g < r1) ? rpair[r + u * g] : 0u;
}

// LDL^T of the assembled G (D and Lr hold its diagonal and strictly lower
// entries on entry) by the factorisation's levels; the columns of one
// elimination-tree level depend only on lower levels:
//   D_j  = G_jj - sum_{k<j} L_jk^2 D_k
//   L_ij = (G_ij - sum_{k<j} L_ik D_k L_jk) / D_j
// Each row (first phase) and each entry (second phase) of a level is shared
// by a team of 2^lg adjacent lanes, lg from the level's width: the top of
// the elimination tree is a chain of one-row levels with long rows, which
// one lane per row would walk serially. An entry's terms come from its list
// of update pairs (the CSR positions of L_ik and L_jk for every common
// column k, precomputed on the host), so no lane searches the two rows; the
// team's partial sums meet in a fixed DPP scan. The structure comes through
// accessors (LDS copies or global arrays): row pointers and columns of L by
// rows, per level its rows and the range of its entries. Non-positive
// pivots are counted in *bad.
template <int BS, bool SM, int PC, class RP, class LV, class RW, class RC>
__device__ __forceinline__ void ldl_levels(int nlev, const RP &rowptr, const LV &flev, const RW &rows,
                                           const LV &fent_ptr, const RC &rowcol, const int32_t *rent,
                                           const uint32_t *rpair, double *Lr, double *D, int32_t *bad) {
  const int tid = (int)threadIdx.x;
  LevelEntry<PC> next = first_entry<BS, PC>(fent_ptr, 0, rent);
  for (int l = 0; l < nlev; ++l) {
    LevelEntry<PC> cur = next;
    load_pairs(cur.pr, rpair, cur.r, cur.r1, 1 << cur.lg);
    if (l + 1 < nlev) next = first_entry<BS, PC>(fent_ptr, l + 1, rent);
    {
      const int p0 = flev[l], p1 = flev[l + 1];
      const int lg = team_log2<BS>(p1 - p0), g = 1 << lg, sub = tid & (g - 1);
      for (int p = p0 + (tid >> lg); p < p1; p += BS >> lg) {
        const int j = rows[p];
        const int q1 = rowptr[j + 1];
        double acc = 0.0;
        for (int q = rowptr[j] + sub; q < q1; q += g) {
          const double ljk = Lr[q];
          acc = acc + ljk * ljk * D[rowcol[q]];
        }
        acc = group_sum(acc, lg);
        if (sub == g - 1) {
          const double d = D[j] - acc;
          D[j] = d;
          if (!(d > 0.0) || !isfinite(d)) atomicAdd(bad, 1);
        }
      }
    }
    wg_sync<SM>();
    {
      const int p1 = fent_ptr[l + 1];
      const int lg = team_log2<BS>(p1 - fent_ptr[l]), g = 1 << lg, sub = tid & (g - 1);
      for (int p = cur.p; p < p1; p += BS >> lg) {
        int pos = cur.pos, r = cur.r, r1 = cur.r1;
        uint32_t pr[PC];
#pragma unroll
        for (int u = 0; u < PC; ++u) pr[u] = cur.pr[u];
        if (p != cur.p) {
          pos = rent[2 * p];
          r = rent[2 * p + 1] + sub;
          r1 = rent[2 * p + 3];
          load_pairs(pr, rpair, r, r1, g);
        }
        double acc = 0.0;
        while (r < r1) {
#pragma unroll
          for (int u = 0; u < PC; ++u) {
            if (r + u * g < r1) {
              const int qi = (int)(pr[u] & 0xFFFFu), qj = (int)(pr[u] >> 16);
              acc = acc + Lr[qi] * D[rowcol[qj]] * Lr[qj];
            }
          }
          r += PC * g;
          if (r < r1) load_pairs(pr, rpair, r, r1, g);
        }
        acc = group_sum(acc, lg);
        if (sub == g - 1) Lr[pos] = (Lr[pos] - acc) / D[rowcol[pos]];
      }
    }
    wg_sync<SM>();
  }
}

// The factor of an item with diodes for its current conductances (the
// lanes' L.g), computed inside the time loop into the item's dynamic slot:
// G on the item's symbolic pattern (with any coupled groups' mutual
// stamps), LDL^T by the factorisation's levels (the same arithmetic as the
// factorisation before the loop), then the sweep values and 1/D, which the
// sweeps then read (staged into LDS under SM). Such items have no dense
// tail. Non-positive pivots are counted in c.flags[4].
template <int BS, int BPT, bool SM>
__device__ __forceinline__ void refactor_dynamic(const DevCtx &c, const ItemDesc &it, View<SM> &v, const Lane<BPT> &L) {
  const SymDesc sd = c.syms[it.sym];
  const int n = it.n;
  double *gcur = c.dyn + it.dyn;
  // Under SM the factorisation runs in LDS: without a dense tail the sweep
  // values are exactly L's nonzeros in row order (sv index = CSR position),
  // so L is built in place in the staged sweep values and D in the staged
  // 1/D, which is inverted at the end; the structure is read from LDS too
  // (the sweeps' column, row and position arrays are then L's by rows and
  // by columns). Otherwise in the dynamic slot in global memory.
  double *Lr, *D;
  if constexpr (SM) {
    Lr = reinterpret_cast<double *>(emt_lds + v.sv_s.off);
    D = reinterpret_cast<double *>(emt_lds + v.dinv_s.off);
  } else {
    Lr = gcur + it.n_br;
    D = Lr + sd.nnz;
  }
  double *sv = gcur + it.n_br + sd.nnz + n;
  double *di = sv + sd.nsv;
  const int32_t *g_rowptr = c.symi + sd.rowptr;
  const int32_t *g_nptr = c.nptr + it.nptr;
  const uint16_t *g_nent = c.nent + it.nent;
  const bool csr = SM && !c.csr_global;
  const int32_t *bk = c.bk + it.br, *bm = c.bm + it.br, *gpos = c.bgpos + it.br;
  const int tid = lane_id();
#pragma unroll
  for (int j = 0; j < BPT; ++j) gcur[tid + j * BS] = L.g[j];
  __syncthreads();
  for (int r = threadIdx.x; r < n; r += BS) {
    int q0, q1;
    if constexpr (SM) {
      q0 = v.rf_rowptr[r];
      q1 = v.rf_rowptr[r + 1];
    } else {
      q0 = g_rowptr[r];
      q1 = g_rowptr[r + 1];
    }
    for (int q = q0; q < q1; ++q) Lr[q] = 0.0;
    double d = 0.0;
    const int e1 = csr ? v.nptr[r + 1] : g_nptr[r + 1];
    for (int e = csr ? v.nptr[r] : g_nptr[r]; e < e1; ++e) {
      const int ent = csr ? v.nent[e] : g_nent[e];
      const int b = ent >> 1;
      const double gv = gcur[b];
      d = d + gv;
      const int other = (ent & 1) ? bk[b] : bm[b];
      if (other >= 0 && other < r) Lr[gpos[b]] = Lr[gpos[b]] - gv;
    }
    D[r] = d;
    if (it.n_groups > 0) {
      const int32_t *mp = c.mptr + it.mptr;
      const int32_t *me = c.ment + it.ment;
      const double *go = c.cgo + it.coef;
      for (int e = mp[r]; e < mp[r + 1]; ++e) {
        const int pos = me[2 * e], code = me[2 * e + 1];
        const double gv = go[code >> 1];
        Lr[pos] = (code & 1) ? Lr[pos] - gv : Lr[pos] + gv;
      }
    }
  }
  wg_sync<SM>();
  constexpr int kPC = 2;  // pairs per load round (more measured no faster)
  const int32_t *rent = c.symi + sd.rent;
  const uint32_t *rpair = reinterpret_cast<const uint32_t *>(c.symi + sd.rpair);
  if constexpr (SM) {
    ldl_levels<BS, SM, kPC>(sd.nlev, v.rf_rowptr, v.rf_flev, v.rf_rows, v.rf_fent_ptr, v.fcol, rent, rpair, Lr, D,
                       c.flags + 4);
    (void)sv;
    (void)di;
    for (int r = threadIdx.x; r < n; r += BS) D[r] = 1.0 / D[r];
    step_barrier<BS>();
  } else {
    const int32_t *rowcol = c.symi + sd.rowcol;
    const int32_t *flevptr = c.symi + sd.flevptr, *flevrows = c.symi + sd.flevrows;
    const int32_t *fentptr = c.symi + sd.fentptr;
    const int32_t *svmap = c.symi + sd.svmap;
    ldl_levels<BS, SM, kPC>(sd.nlev, g_rowptr, flevptr, flevrows, fentptr, rowcol, rent, rpair, Lr, D, c.flags + 4);
    for (int q = threadIdx.x; q < sd.nsv; q += BS) sv[q] = Lr[svmap[q]];
    for (int r = threadIdx.x; r < n; r += BS) di[r] = 1.0 / D[r];
    __syncthreads();
    v.sv.p = sv;
    v.dinv.p = di;
  }
}

// ---------------------------------------------------------------------------
// Forward loop: steps n0+1 .. n0+nsteps for every item.
// ---------------------------------------------------------------------------
// KIND (device.h, StepKind): what the batch's components need besides the
// closed-form solve; a variant carries only its own code and registers.
template <int BS, int BPT, int DT, bool SM, int KIND>
__global__ __launch_bounds__(BS) void k_forward(DevCtx c, const int32_t *order, int64_t n0, int64_t nsteps,
                                                double *rec) {
  constexpr int kSolve = KIND == STEP_FULL ? BOTH : (KIND == STEP_LEVELS ? LEVELS : CLOSED);
  // line ends or coupled members
  // A launch of a few steps is mostly staging. Where a lane carries several
  // branches the factor's values are many for the lanes that stage them, and
  // one load after another was a trip to memory each: one step a call on 40
  // buses (64 lanes) 15.5 -> 13.4 us, on 400 (512 lanes) 14.3 -> 13.4; long
  // launches of 20 to 1000 buses stay within 0.5 % or gain. With fewer branches a lane, or with
  // lines, groups or switches, the values are few or the longer code costs the
  // loop registers (lines at 64 lanes 3.03 -> 3.12 us a step).
  constexpr int kBlocks = KIND == STEP_PLAIN && BPT >= 4 ? 4 : 1;
  constexpr bool kPass = KIND == STEP_LINES || KIND == STEP_GROUPS || KIND == STEP_FULL;
  const ItemDesc it = c.items[order[blockIdx.x]];
  View<SM> v = make_view<BS, SM, kSolve, KIND == STEP_SWITCH ? DT : 0>(c, it, false);
  const int64_t *topo = c.topo + it.topo;
  int t = topo_of(topo, it.n_topo, n0 + 1);
  int64_t next = (t + 1 < it.n_topo) ? topo[t + 1] : kNever;
  Lane<BPT> L;
  Tail<BS, DT> w;
  load_lane<BS, BPT>(c, it, L);
  load_coefs<BS, BPT>(c, it, t, L.g, L.be);
  // diodes or controlled switches: refactorised by levels, or (switches) the
  // closed form's tail
  const bool diodes = KIND == STEP_FULL && it.n_diodes > 0;
  const bool switches = KIND == STEP_SWITCH && it.n_diodes > 0;
  uint32_t dmask = 0, cmask = 0;
  if (diodes || switches) {
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int kd = c.bkind[it.br + threadIdx.x + j * BS];
      if (kd == KIND_DIODE || kd == KIND_CSWITCH) dmask |= 1u << j;
      if (kd == KIND_CSWITCH) cmask |= 1u << j;
    }
    diode_conductances<BS, BPT>(c, it, L, dmask);
  }
  history_from_state<BS, BPT, SM>(c.si + it.br, c.su + it.br, L, v);
  if (diodes) {
    if (threadIdx.x == 0) v.swflag[0] = (int)n0 - 1;
    // no dense tail: w stays zero
#pragma unroll
    for (int k = 0; k < 2 * Tail<BS, DT>::R * Tail<BS, DT>::Q; ++k) w.w[k] = 0.0;
    refactor_dynamic<BS, BPT, SM>(c, it, v, L);
  } else {
    select_factor<BS, DT, SM, kBlocks>(c, it, v, t, w);
  }
  double dv[(Tail<BS, DT>::R + 3) / 4];
  SwitchLane sl;
  sl.on = false;
  sl.d.control = 0;
  if (switches) {
    const int nsw = it.n_diodes;
    for (int q = (int)threadIdx.x + BS; q < nsw; q += BS) {
      SwitchLane s;
      switch_load(c, it, q, s);
      v.gsw[q] = s.on ? s.gon : 0.0;
    }
    if ((int)threadIdx.x < nsw) {
      switch_load(c, it, (int)threadIdx.x, sl);
      v.gsw[(int)threadIdx.x] = sl.on ? sl.gon : 0.0;
    }
    if (threadIdx.x == 0) v.swflag[0] = (int)n0 - 1;
    __syncthreads();
    refactor_tail<BS, DT, SM>(c, it, v, t, w, dv);
  }
  inject<BS, BPT, SM>(c, v, L, n0 + 1);
  step_barrier<BS>();
  const bool lines = (KIND == STEP_LINES || KIND == STEP_FULL) && it.n_lines > 0;
  const bool groups = (KIND == STEP_GROUPS || KIND == STEP_FULL) && it.n_groups > 0;
  constexpr int NL = KIND == STEP_LINES ? kLineRegs : 0, NG = KIND == STEP_GROUPS ? kGroupRegs : 0;
  Lines<NL> ln;
  Groups<NG> gr;
  if (lines || groups) {
    if (lines) lines_start<BS, NL, SM>(c, it, v, ln, n0 + 1);
    if (groups) {
      groups_load<BS, NG>(c, it, gr);
      groups_step<BS, NG, SM>(c, it, v, gr, true, true, nullptr, nullptr);
    }
    step_barrier<BS>();
  }
  const int R = c.rec_stride;
  const int64_t n_end = n0 + nsteps;
  // the lane's first recorded node and its column
  const int tid0 = (int)threadIdx.x;
  const bool rec0 = rec && tid0 < v.nrec;
  const int rn0 = rec0 ? v.rnode[tid0] : 0;
  double *row = rec ? rec + (int64_t)it.scen * nsteps * R : nullptr;
  double *at0 = rec0 ? row + v.rcolumn[tid0] : nullptr;
  // steps with more to do than the plain ones: the next checkpoint (a
  // running step number: a 64-bit remainder each step costs more than the
  // whole branch update), the step before a topology change, the last one
  int64_t ck_step = c.K > 0 ? (n0 / c.K + 1) * c.K : kNever;
  auto special_step = [&]() {
    const int64_t m = next == kNever || next - 1 > n_end ? n_end : next - 1;
    return ck_step < m ? ck_step : m;
  };
  int64_t special = special_step();
  bool fresh = false;  // switches: the topology changed
  // the adjoint's trajectory rows (batches with checkpoints have no lines,
  // groups or diodes)
  double *rows = nullptr;
  if ((KIND == STEP_PLAIN || kSolve != CLOSED) && c.vt_full) rows = c.vt + it.vt + n0 * (int64_t)(v.n + v.nsrc);
  for (int64_t n = n0 + 1; n <= n_end; ++n) {
    emf_advance<BPT, SM>(c, v, L, n + 1, false);
    if (lines) lines_ahead<BS, NL>(it, ln, n);
    int changed = 0;
    if (switches) {
      changed = v.swflag[0];
      if ((int)threadIdx.x < it.n_diodes) switch_reference(c, sl, n);
    }
    gather_all<BS, SM>(v);
    if (switches) {
      // a switch changed state after the last step, or the topology changed
      if (fresh || __builtin_amdgcn_readfirstlane(changed) == (int)n - 1) {
        __syncthreads();  // the states stored by other lanes
        diode_conductances<BS, BPT>(c, it, L, dmask);
#pragma unroll
        for (int j = 0; j < BPT; ++j) settle(L.g[j]);
        refactor_tail<BS, DT, SM>(c, it, v, t, w, dv);
        fresh = false;
      }
    }
    solve_after_gather<BS, DT, SM, kSolve, KIND == STEP_SWITCH>(v, w, dv, switches);
    if (switches) {
      if ((int)threadIdx.x < it.n_diodes) switch_step<SM>(c, it, v, sl, (int)threadIdx.x, n);
      for (int q = (int)threadIdx.x + BS; q < it.n_diodes; q += BS) {
        SwitchLane s;
        switch_load(c, it, q, s);
        switch_reference(c, s, n);
        switch_step<SM>(c, it, v, s, q, n);
      }
    }
    if (lines) lines_settle<BS, NL>(it, ln);
    if (rows) {
      store_row<BS, BPT, SM>(v, L, rows);
      rows += v.n + v.nsrc;
    }
    // read here, stored after the update so that its own reads go ahead
    const double rv0 = rec0 ? v.x[rn0] : 0.0;
    if (v.nrec > BS && rec) {
      for (int q = tid0 + BS; q < v.nrec; q += BS) row[v.rcolumn[q]] = v.x[v.rnode[q]];
      row += R;
    }
    if (!kPass && n != special) {
      update_plain<BS, BPT, SM, false>(v, L, nullptr);
      if (rec0) {
        *at0 = rv0;
        at0 += R;
      }
      step_barrier<BS>();
      continue;
    }
    if (kPass && n != special && !diodes) {
      update_plain<BS, BPT, SM, false, true>(v, L, nullptr);
      if (lines || groups) {
        step_barrier<BS>();
        if (lines) lines_step<BS, NL, SM>(c, it, v, ln, n, nullptr, nullptr);
        if (groups) groups_step<BS, NG, SM>(c, it, v, gr, false, true, nullptr, nullptr);
      }
      if (rec0) {
        *at0 = rv0;
        at0 += R;
      }
      step_barrier<BS>();
      continue;
    }
    const bool sw = (n + 1 == next);
    const uint32_t fl = diodes ? diode_flips<BS, BPT, SM>(c, it, v, L, dmask, cmask, n) : 0u;
    double *ck_i = nullptr, *ck_u = nullptr, *st_i = nullptr, *st_u = nullptr;
    if (n == ck_step) {
      const int64_t o = it.ck + (n / c.K) * (int64_t)v.nbr;
      ck_i = c.ck_i + o;
      ck_u = c.ck_u + o;
      ck_step += c.K;
    }
    if (n == n_end) {
      st_i = c.si + it.br;
      st_u = c.su + it.br;
    }
    update_inject<BS, BPT, SM, kPass>(c, v, L, ck_i, ck_u, st_i, st_u, sw, it.coef + (int64_t)(t + 1) * v.nbr,
                               n < n_end, n);
    if (rec0) {
      *at0 = rv0;
      at0 += R;
    }
    if (lines || groups) {
      step_barrier<BS>();
      if (lines) lines_step<BS, NL, SM>(c, it, v, ln, n, st_i, st_u);
      if (groups) groups_step<BS, NG, SM>(c, it, v, gr, false, n < n_end, st_i, st_u);
    }
    if (diodes) {
      // a diode changed state or the topology switched: the conductances
      // of step n+1 and their factor, inside the loop (a word of the
      // kernel's own LDS: __syncthreads_or takes 256 bytes that the host's
      // layout does not know)
      if (fl != 0u) v.swflag[0] = (int)n;
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(v.swflag[0]) == (int)n || sw) {
        diode_conductances<BS, BPT>(c, it, L, dmask);
        refactor_dynamic<BS, BPT, SM>(c, it, v, L);
      }
    }
    if (sw) {
      ++t;
      next = (t + 1 < it.n_topo) ? topo[t + 1] : kNever;
      if (!diodes) select_factor<BS, DT, SM, kBlocks>(c, it, v, t, w);
      fresh = switches;
    }
    special = special_step();
    step_barrier<BS>();
  }
  for (int q = threadIdx.x; q < v.n; q += BS) c.sv_state[it.node + q] = v.x[q];
}

// ---------------------------------------------------------------------------
// Reverse-time adjoint over the whole horizon, one workgroup per item. For
// each checkpoint segment (last first): recompute its forward steps from the
// checkpoint into the segment buffer, then run the discrete adjoint of the
// step backwards:
//   ibar = beta_{n+1} hbar_{n+1};  q = gamma_{n+1} hbar_{n+1} + g_n ibar
//   vbar = dJ/dv_n + A q;          w = G_n^{-T} vbar (G symmetric: same solve)
//   hbar_n = ibar - A^T w
//   gbar += hbar_n u_n, betabar += hbar_n i_{n-1}, gammabar += hbar_n u_{n-1}
// ---------------------------------------------------------------------------
// Runs f(j, g_nx, be_nx) for every slot with the coefficients of step n+1:
// those of step n (in L) unless a switching event lies between the two
// steps (t_nx != t, uniform over the workgroup), then reloaded. Two fully
// unrolled loops, so every slot index is a constant.
template <int BS, int BPT, class F>
__device__ __forceinline__ void with_next_coefs(const DevCtx &c, const ItemDesc &it, const Lane<BPT> &L, int t,
                                                int t_nx, int nreal, F &&f) {
  if (t_nx == t) {
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      if (j > 0 && (j & 1) == 0 && j * BS >= nreal) break;  // padding
      f(j, L.g[j], L.be[j]);
    }
  } else {
    const int64_t o = it.coef + (int64_t)t_nx * it.n_br + lane_id();
#pragma unroll
    for (int j = 0; j < BPT; ++j) f(j, c.cg[o + j * BS], c.cb[o + j * BS]);
  }
}

template <int BS, int BPT, bool SM>
__device__ __forceinline__ void adjoint_seed(const DevCtx &c, const ItemDesc &it, const View<SM> &v,
                                             const Lane<BPT> &L, int t, int t_nx, const double (&hb_nx)[BPT],
                                             double seed0, const double *dJ, int64_t n) {
  const int tid = lane_id();
  with_next_coefs<BS, BPT>(c, it, L, t, t_nx, v.nreal, [&](int j, double g_nx, double be_nx) {
    const int b = tid + j * BS;
    const double ibar = be_nx * hb_nx[j];
    const double ga_nx = gamma_of(L.pk[j], g_nx);
    v.J[b] = (L.g[j] != 0.0) ? ga_nx * hb_nx[j] + L.g[j] * ibar : 0.0;
  });
  // the recorded columns' cotangents, which the gather adds at their nodes
  if (!SM && c.seeds_global) return;
  if (tid < v.nrec) v.J[v.nbr + 1 + tid] = seed0;
  if (v.nrec > BS) {
    const double *drow = dJ + ((int64_t)it.scen * c.T + (n - 1)) * c.rec_stride;
    for (int q = tid + BS; q < v.nrec; q += BS) v.J[v.nbr + 1 + q] = drow[v.rcolumn[q]];
  }
}

// The cotangents of step n from memory, where they are no part of the gather:
// a lane per node adds up its columns.
template <int BS, bool SM>
__device__ __forceinline__ void add_seeds(const DevCtx &c, const ItemDesc &it, const View<SM> &v, const double *dJ,
                                          int64_t n) {
  const int32_t *rp = c.rptr + it.nptr;
  const uint16_t *col = c.rcolumn + it.rec;
  const double *drow = dJ + ((int64_t)it.scen * c.T + (n - 1)) * c.rec_stride;
  for (int r = (int)threadIdx.x; r < v.n; r += BS) {
    const int q1 = rp[r + 1];
    double s = v.r[r];
    for (int q = rp[r]; q < q1; ++q) s = s + drow[col[q]];
    v.r[r] = s;
  }
  step_barrier<BS>();
}

// The cotangent of step n in the lane's first recorded column.
template <bool SM>
__device__ __forceinline__ double load_seed(const DevCtx &c, const ItemDesc &it, const View<SM> &v, const double *dJ,
                                            int64_t n) {
  const int tid = (int)threadIdx.x;
  return tid < v.nrec ? dJ[((int64_t)it.scen * c.T + (n - 1)) * c.rec_stride + v.rcolumn[tid]] : 0.0;
}

// The checkpoint segments. The reversal of a segment needs every step's
// branch currents and voltages. Where the forward run has kept the
// trajectory rows (all voltages and EMFs), a segment's currents follow from
// its checkpoint branch by branch, without a solve or a barrier
// (rebuild_segment); otherwise its steps are run again and leave rows of
// their own (recompute_segment). Either way the currents go to the segment
// buffer (row n - lo - 1 = step n) and the voltages are formed from the rows.
// A row is 8 (n + n_src) bytes a step, the branch state it stands for about
// 50 n; running the steps again took as long as the reversal itself.

// Runs steps lo+1..hi of segment s again from its checkpoint. Afterwards L's
// coefficients and the factors are those of step hi.
template <int BS, int BPT, int DT, bool SM, int LEV>
__device__ __forceinline__ void recompute_segment(const DevCtx &c, const ItemDesc &it, View<SM> &v, Lane<BPT> &L,
                                                  Tail<BS, DT> &w, int64_t s, double *seg_i, double *rows) {
  const int64_t *topo = c.topo + it.topo;
  const int nbr = v.nbr;
  const int64_t lo = s * c.K, hi = (lo + c.K < c.T) ? lo + c.K : c.T;
  const int64_t cko = it.ck + s * (int64_t)nbr;
  // the gather's seeds are zero in the forward steps
  if (SM || !c.seeds_global)
    for (int q = threadIdx.x; q < v.nrec; q += BS) v.J[v.nbr + 1 + q] = 0.0;
  int t = topo_of(topo, it.n_topo, lo + 1);
  int64_t next = (t + 1 < it.n_topo) ? topo[t + 1] : kNever;
  load_coefs<BS, BPT>(c, it, t, L.g, L.be);
  history_from_state<BS, BPT, SM>(c.ck_i + cko, c.ck_u + cko, L, v);
  select_factor<BS, DT, SM>(c, it, v, t, w);
  inject<BS, BPT, SM>(c, v, L, lo + 1);
  step_barrier<BS>();
  for (int64_t n = lo + 1; n <= hi; ++n) {
    emf_advance<BPT, SM>(c, v, L, n + 1, false);
    gather_all<BS, SM>(v);
    solve_after_gather<BS, DT, SM, LEV>(v, w);
    double *st_i = seg_i + (n - lo - 1) * (int64_t)nbr;
    store_row<BS, BPT, SM>(v, L, rows + (n - lo - 1) * (int64_t)(v.n + v.nsrc));
    if (n < hi && n + 1 != next) {
      update_plain<BS, BPT, SM, true>(v, L, st_i);
      step_barrier<BS>();
      continue;
    }
    const bool sw = (n + 1 == next) && n < hi;
    update_inject<BS, BPT, SM>(c, v, L, st_i, nullptr, nullptr, nullptr, sw, it.coef + (int64_t)(t + 1) * nbr, n < hi,
                               n);
    if (sw) {
      ++t;
      next = (t + 1 < it.n_topo) ? topo[t + 1] : kNever;
      select_factor<BS, DT, SM>(c, it, v, t, w);
    }
    step_barrier<BS>();
  }
}

// The branch currents of steps lo+1..hi of segment s from its checkpoint and
// its trajectory rows, every slot for itself. Rows come in blocks through the
// LDS of the right-hand side, solution and injections (idle here), the next
// block read into registers while this one's steps run: gathered from memory
// row by row a step was one trip to it. Afterwards L's coefficients are those
// of step hi.
template <int BS, int BPT, bool SM>
__device__ __forceinline__ void rebuild_segment(const DevCtx &c, const ItemDesc &it, const View<SM> &v, Lane<BPT> &L,
                                                int64_t s, double *seg_i, const double *rows) {
  constexpr int kRegs = 8;  // doubles per lane of a block
  const int64_t *topo = c.topo + it.topo;
  const int nbr = it.n_br, len = it.n + it.n_src;
  const int64_t lo = s * c.K, hi = (lo + c.K < c.T) ? lo + c.K : c.T;
  const int64_t cko = it.ck + s * (int64_t)nbr;
  double *buf = reinterpret_cast<double *>(emt_lds + (v.closed ? v.x.off - (uint32_t)(v.n + 1) * 8u : v.x.off));
  const int room = (int)(v.J.off - (uint32_t)((char *)buf - emt_lds)) / 8 + nbr;
  int per = (room < kRegs * BS ? room : kRegs * BS) / len;  // steps per block
  if (per < 1) per = 1;  // (a row of more than kRegs * BS entries: see below)
  int t = topo_of(topo, it.n_topo, lo + 1);
  int64_t next = (t + 1 < it.n_topo) ? topo[t + 1] : kNever;
  load_coefs<BS, BPT>(c, it, t, L.g, L.be);
  double h[BPT];
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    const int64_t b = cko + (int)threadIdx.x + j * BS;
    h[j] = L.be[j] * c.ck_i[b] + gamma_of(L.pk[j], L.g[j]) * c.ck_u[b];
  }
  double ahead[kRegs];
  auto read_block = [&](int64_t n, int cnt) {  // entries of steps n .. of a block
    const double *r = rows + (n - lo - 1) * (int64_t)len;
#pragma unroll
    for (int k = 0; k < kRegs; ++k) {
      const int q = lane_id() + k * BS;
      ahead[k] = q < cnt ? r[q] : 0.0;
    }
  };
  auto steps_from = [&](int64_t n) { return (int)(hi - n + 1 < per ? hi - n + 1 : per); };
  read_block(lo + 1, steps_from(lo + 1) * len);
  for (int64_t n0 = lo + 1; n0 <= hi; n0 += per) {
    const int m = steps_from(n0), cnt = m * len;
    __syncthreads();  // the block before has been read
#pragma unroll
    for (int k = 0; k < kRegs; ++k) {
      const int q = lane_id() + k * BS;
      if (q < cnt) buf[q] = ahead[k];
    }
    // what the registers do not hold of a very long row
    for (int q = (int)threadIdx.x + kRegs * BS; q < cnt; q += BS) buf[q] = rows[(n0 - lo - 1) * (int64_t)len + q];
    __syncthreads();
    if (n0 + m <= hi) read_block(n0 + m, steps_from(n0 + m) * len);
    for (int d = 0; d < m; ++d) {
      const int64_t n = n0 + d;
      const double *row = buf + d * len;
      const bool sw = n + 1 == next && n < hi;
      const int tid = lane_id();
#pragma unroll
      for (int j = 0; j < BPT; ++j) {
        if (j > 0 && (j & 1) == 0 && j * BS >= it.n_real) break;
        const uint32_t pk = opaque(L.pk[j]);
        const int k = (int)(pk & kTermGround), q = (int)((pk >> 15) & kTermGround);
        const double vk = k < it.n ? row[k] : 0.0, vm = q < it.n ? row[q] : 0.0;
        double u = vk - vm;
        if (j == 0) u = u - (tid < it.n_src ? row[it.n + tid] : 0.0);
        if (sw && L.g[j] == 0.0) u = 0.0;
        const double gu = L.g[j] * u;
        const double i = gu + h[j];
        seg_i[tid + j * BS] = i;
        double gam = gamma_times(pk, gu);
        if (sw) {
          const int64_t o = it.coef + (int64_t)(t + 1) * nbr + tid + j * BS;
          L.g[j] = c.cg[o];
          L.be[j] = c.cb[o];
          settle(L.g[j]);
          settle(L.be[j]);
          gam = gamma_of(pk, L.g[j]) * u;
        }
        h[j] = L.be[j] * i + gam;
      }
      seg_i += nbr;
      if (sw) {
        ++t;
        next = (t + 1 < it.n_topo) ? topo[t + 1] : kNever;
      }
    }
  }
  __syncthreads();
  // the zeros that the block overwrote
  if (threadIdx.x == 0) {
    v.x[v.n] = 0.0;
    v.J[nbr] = 0.0;
    *reinterpret_cast<double *>(emt_lds + (v.closed ? v.x.off - 8u : v.x.off + (uint32_t)v.n * 8u)) = 0.0;
  }
}

// Reverses steps hi..lo+1 of segment s from its currents and rows. On entry
// L's coefficients and the factors are those of step hi (topology t) and
// hb_nx holds hbar of step hi+1 (0 past the horizon); on exit hb_nx holds
// hbar of step lo+1, and the gradient accumulators have taken the segment's
// terms.
template <int BS, int BPT, int DT, bool SM, int GEN>
__device__ __forceinline__ void reverse_segment(const DevCtx &c, const ItemDesc &it, View<SM> &v, Lane<BPT> &L,
                                                Tail<BS, DT> &w, int64_t s, int t, const double *seg_i,
                                                const double *rows, double (&hb_nx)[BPT], double (&gb)[BPT],
                                                double (&bb)[BPT], double (&cb)[BPT], const double *dJ) {
  const int64_t *topo = c.topo + it.topo;
  const int nbr = v.nbr, len = v.n + v.nsrc, tid0 = (int)threadIdx.x;
  const int64_t T = c.T;
  const int64_t lo = s * c.K, hi = (lo + c.K < T) ? lo + c.K : T;
  const int64_t cko = it.ck + s * (int64_t)nbr;
  // the coefficients of step hi+1 are those of topology t_nx (unused at
  // hi = T, where hbar = 0)
  int t_nx = hi < T ? topo_of(topo, it.n_topo, hi + 1) : t;
  // the first step of topology t (every topology starts at a step of its
  // own); read from memory only when it changes
  auto first_step = [&](int tt) {
    int64_t f = tt > 0 ? topo[tt] : 0;
    asm volatile("" : "+v"(f));
    return f;
  };
  int64_t first = first_step(t);
  adjoint_seed<BS, BPT, SM>(c, it, v, L, t, t_nx, hb_nx, load_seed<SM>(c, it, v, dJ, hi), dJ, hi);
  // a row's entry q in v.vrow: past the voltages comes the ground's zero
  auto at = [&](int q) { return q < v.n ? q : q + 1; };
  // the row at hand: in LDS, or (a component whose arrays leave no room for
  // it) in memory, without the zero
  const bool row_lds = SM || !c.row_global;
  const double *at_row = rows + (hi - lo - 1) * (int64_t)len;
  auto row_at = [&](int q) {
    if (row_lds) return (double)v.vrow[q];
    return q == v.n ? 0.0 : at_row[q < v.n ? q : q - 1];
  };
  // the voltages of a row in the lane's slots, with the conductances that
  // tell a branch out of service
  auto row_u = [&](int j, double g) {
    const uint32_t pk = opaque(L.pk[j]);
    const double vk = row_at((int)(pk & kTermGround)), vm = row_at((int)((pk >> 15) & kTermGround));
    const double e = j == 0 && tid0 < v.nsrc ? row_at(v.n + 1 + tid0) : 0.0;
    const double u = j == 0 ? (vk - vm) - e : vk - vm;
    return g == 0.0 ? 0.0 : u;
  };
  if (row_lds) {
    const double *row = at_row;
    for (int q = tid0; q < len; q += BS) v.vrow[at(q)] = row[q];
  }
  step_barrier<BS>();
  // u of step n in the lane's slots, carried from one step (where it was the
  // earlier one) to the next
  double un[BPT];
#pragma unroll
  for (int j = 0; j < BPT; ++j) un[j] = row_u(j, L.g[j]);
  // the lane's entries of row m, read a step before they are needed
  double r0 = 0.0, r1 = 0.0;
  auto read_ahead = [&](int64_t m) {
    if (m <= lo || !row_lds) return;
    const double *row = rows + (m - lo - 1) * (int64_t)len;
    if (tid0 < len) r0 = row[tid0];
    if (tid0 + BS < len) r1 = row[tid0 + BS];
  };
  read_ahead(hi - 1);
  step_barrier<BS>();
  for (int64_t n = hi; n >= lo + 1; --n) {
    // global reads of this step's update (currents and row of step n - 1; at
    // the segment's first step the checkpoint) and the next step's seeds,
    // issued ahead of the solve
    const bool from_ck = n - 1 == lo;
    const double *i0 = from_ck ? c.ck_i + cko : seg_i + (n - lo - 2) * (int64_t)nbr;
    const double *row = rows + (n - lo - 2) * (int64_t)len;
    const int tid = lane_id();
    at_row = row;
    if (!from_ck && row_lds) {
      if (tid0 < len) v.vrow[at(tid0)] = r0;
      if (tid0 + BS < len) v.vrow[at(tid0 + BS)] = r1;
      for (int q = tid0 + 2 * BS; q < len; q += BS) v.vrow[at(q)] = row[q];
    }
    double ip[BPT];
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      ip[j] = 0.0;
      if (j > 0 && j * BS >= v.nreal) continue;
      ip[j] = i0[tid + j * BS];
    }
    read_ahead(n - 2);
    const double seed0 = from_ck ? 0.0 : load_seed<SM>(c, it, v, dJ, n - 1);
    gather_all<BS, SM>(v);
    if (!SM && c.seeds_global) add_seeds<BS, SM>(c, it, v, dJ, n);
    solve_after_gather<BS, DT, SM, adjoint_solve(GEN)>(v, w);
    if (!from_ck && n - 1 >= first && t_nx == t) {
      // no checkpoint and no topology change on either side: the update and
      // the next step's injections slot by slot (out of service: hbar = 0,
      // and u only ever meets that zero)
      const double e = tid < v.nsrc ? row_at(v.n + 1 + tid) : 0.0;
#pragma unroll
      for (int j = 0; j < BPT; ++j) {
        if (j > 0 && (j & 1) == 0 && j * BS >= v.nreal) break;
        const uint32_t pk = opaque(L.pk[j]);
        const int k = (int)(pk & kTermGround), m = (int)((pk >> 15) & kTermGround);
        const double wk = v.x[k], wm = v.x[m], vk = row_at(k), vm = row_at(m);
        const double up = j == 0 ? (vk - vm) - e : vk - vm;
        const double hb = L.g[j] != 0.0 ? L.be[j] * hb_nx[j] - (wk - wm) : 0.0;
        gb[j] = __builtin_fma(hb, un[j], gb[j]);
        bb[j] = __builtin_fma(hb, ip[j], bb[j]);
        cb[j] = __builtin_fma(hb, up, cb[j]);
        un[j] = up;
        hb_nx[j] = hb;
        v.J[tid + j * BS] = gamma_times(pk, L.g[j] * hb) + L.g[j] * (L.be[j] * hb);
      }
      if (SM || !c.seeds_global) {
        if (tid < v.nrec) v.J[v.nbr + 1 + tid] = seed0;
      }
      if (v.nrec > BS && (SM || !c.seeds_global)) {
        const double *drow = dJ + ((int64_t)it.scen * c.T + (n - 2)) * c.rec_stride;
        for (int q = tid + BS; q < v.nrec; q += BS) v.J[v.nbr + 1 + q] = drow[v.rcolumn[q]];
      }
      step_barrier<BS>();
      continue;
    }
    // a topology change between step n - 1 and step n: the earlier one's
    // conductances decide which of its branches were out of service
    const bool earlier = n - 1 < first && t > 0;
    with_next_coefs<BS, BPT>(c, it, L, t, t_nx, v.nreal, [&](int j, double g_nx, double be_nx) {
      (void)g_nx;
      const uint32_t pk = opaque(L.pk[j]);
      const double wk = v.x[pk & kTermGround], wm = v.x[(pk >> 15) & kTermGround];
      double up;
      if (from_ck)
        up = c.ck_u[cko + tid + j * BS];
      else
        up = row_u(j, earlier ? c.cg[it.coef + (int64_t)(t - 1) * nbr + tid + j * BS] : L.g[j]);
      const double ibar = be_nx * hb_nx[j];
      const double hb = (L.g[j] != 0.0) ? ibar - (wk - wm) : 0.0;
      gb[j] = __builtin_fma(hb, un[j], gb[j]);
      bb[j] = __builtin_fma(hb, ip[j], bb[j]);
      cb[j] = __builtin_fma(hb, up, cb[j]);
      un[j] = up;
      hb_nx[j] = hb;
    });
    // step n's coefficients become the next-step ones of step n-1
    t_nx = t;
    if (!from_ck) {
      if (n - 1 < first) {
        --t;
        first = first_step(t);
        load_coefs<BS, BPT>(c, it, t, L.g, L.be);
        select_factor<BS, DT, SM>(c, it, v, t, w);
      }
      adjoint_seed<BS, BPT, SM>(c, it, v, L, t, t_nx, hb_nx, seed0, dJ, n - 1);
    }
    step_barrier<BS>();
  }
}

template <int BS, int BPT>
__device__ __forceinline__ void store_branch_adjoints(const DevCtx &c, const ItemDesc &it, const double (&gb)[BPT],
                                                      const double (&bb)[BPT], const double (&cb)[BPT]) {
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    const int b = threadIdx.x + j * BS;
    c.gbar[it.br + b] = gb[j];
    c.bbar[it.br + b] = bb[j];
    c.cbar[it.br + b] = cb[j];
  }
}

// Serial adjoint: one workgroup per item rebuilds (or recomputes) and
// reverses each segment in turn, last segment first. The registers are those
// of one wave per SIMD (one workgroup of 256 lanes per compute unit): the
// reversal carries the voltages and three accumulators of every slot from step
// to step, 364 registers at 8 slots. Held to two waves it spills 168 of them
// (324 B a lane), and though a batch of more items than compute units then
// runs in fewer rounds it takes longer: 502 items 11.0 against 8.4 ms, 768
// items 19.6 against 10.2. Level passes alone (ADJ_LEVELS) need fewer and gain
// from two: 300 items of 150 nodes 34.2 against 58.3 us a step. GEN: an
// AdjointKind.
template <int BS, int BPT, int DT, bool SM, int GEN>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(BS == 256 && GEN == ADJ_LEVELS ? 2 : 1))) void k_adjoint(
    DevCtx c, const int32_t *order, const double *dJ) {
  const ItemDesc it = c.items[order[blockIdx.x]];
  View<SM> v = make_view<BS, SM, adjoint_solve(GEN)>(c, it, true);
  const int64_t nseg = (c.T + c.K - 1) / c.K;
  double *seg_i = c.seg_i + it.seg;
  Lane<BPT> L;
  Tail<BS, DT> w;
  load_lane<BS, BPT>(c, it, L);
  // per slot: hbar of step n+1 and the three gradient accumulators
  double hb_nx[BPT], gb[BPT], bb[BPT], cb[BPT];
#pragma unroll
  for (int j = 0; j < BPT; ++j) hb_nx[j] = gb[j] = bb[j] = cb[j] = 0.0;
  int t_w = -1;  // the topology whose factors are loaded
  for (int64_t s = nseg - 1; s >= 0; --s) {
    const int64_t hi = (s * c.K + c.K < c.T) ? s * c.K + c.K : c.T;
    const int t = topo_of(c.topo + it.topo, it.n_topo, hi);
    double *rows = c.vt + it.vt;
    if (GEN == ADJ_PLAIN || c.vt_full) {
      rows += s * c.K * (int64_t)(v.n + v.nsrc);
      rebuild_segment<BS, BPT, SM>(c, it, v, L, s, seg_i, rows);
      if (t != t_w) {
        select_factor<BS, DT, SM>(c, it, v, t, w);
        t_w = t;
      }
    } else {
      recompute_segment<BS, BPT, DT, SM, adjoint_solve(GEN)>(c, it, v, L, w, s, seg_i, rows);
    }
    __syncthreads();
    reverse_segment<BS, BPT, DT, SM, GEN>(c, it, v, L, w, s, t, seg_i, rows, hb_nx, gb, bb, cb, dJ);
    t_w = topo_of(c.topo + it.topo, it.n_topo, s * c.K + 1);
  }
  store_branch_adjoints<BS, BPT>(c, it, gb, bb, cb);
}

// Waits until *flag >= target: wave 0 polls (bounded), acquires at device
// scope, and the workgroup barrier releases the other waves. Returns false
// (and sets the error flag) if the wait gave up.
__device__ __forceinline__ bool wait_flag(const int32_t *flag, int32_t target, int32_t *err,
                                          Lds<int32_t> give_up) {
  if (threadIdx.x < 64) {
    int64_t spins = 0;
    bool quit = false;
    while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (++spins > (int64_t(1) << 24) || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        quit = true;
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
    if (threadIdx.x == 0) {
      give_up[0] = quit ? 1 : 0;
      if (quit) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
  return give_up[0] == 0;
}

// Publishes *flag = value after every wave's global stores: each wave
// waits for its own stores, the workgroup barrier joins them, lane 0
// releases at device scope and stores the flag.
__device__ __forceinline__ void publish_flag(int32_t *flag, int32_t value) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_store(flag, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Pipelined adjoint: two workgroups per item, resident together
// (cooperative launch). Workgroup n_items + i recomputes the segments of
// item order[i], last first, into two alternating segment buffers;
// workgroup i reverses each segment as soon as it is recomputed, so the
// recompute of segment s-1 overlaps the reversal of segment s. Per item,
// pipe[2q] counts recomputed segments and pipe[2q+1] reversed ones; the
// recompute of the k-th segment waits until the (k-2)-th is reversed.
template <int BS, int BPT, int DT, bool SM, int GEN>
__global__ __launch_bounds__(BS) void k_adjoint_pipe(DevCtx c, const int32_t *order, int n_items,
                                                     const double *dJ, int32_t *pipe) {
  const bool recompute = (int)blockIdx.x >= n_items;
  const int q = order[recompute ? blockIdx.x - n_items : blockIdx.x];
  const ItemDesc it = c.items[q];
  View<SM> v = make_view<BS, SM, adjoint_solve(GEN)>(c, it, true);
  const int64_t nseg = (c.T + c.K - 1) / c.K;
  const int64_t steps = c.K < c.T ? c.K : c.T;
  const int64_t seg_len = steps * (int64_t)v.nbr, row_len = v.n + v.nsrc;
  // the rows of the k-th segment handled
  auto rows_of = [&](int64_t k) {
    return c.vt + it.vt + (GEN == ADJ_PLAIN || c.vt_full ? (nseg - 1 - k) * c.K : (k & 1) * steps) * row_len;
  };
  int32_t *ready = pipe + 2 * q, *done = pipe + 2 * q + 1;
  Lane<BPT> L;
  Tail<BS, DT> w;
  load_lane<BS, BPT>(c, it, L);
  if (recompute) {
    for (int64_t k = 0; k < nseg; ++k) {
      if (k >= 2 && !wait_flag(done, (int32_t)(k - 1), c.flags + 2, v.flag)) return;
      const int64_t o = it.seg + (k & 1) * seg_len;
      if (GEN == ADJ_PLAIN || c.vt_full)
        rebuild_segment<BS, BPT, SM>(c, it, v, L, nseg - 1 - k, c.seg_i + o, rows_of(k));
      else
        recompute_segment<BS, BPT, DT, SM, adjoint_solve(GEN)>(c, it, v, L, w, nseg - 1 - k, c.seg_i + o, rows_of(k));
      publish_flag(ready, (int32_t)(k + 1));
    }
    return;
  }
  double hb_nx[BPT], gb[BPT], bb[BPT], cb[BPT];
#pragma unroll
  for (int j = 0; j < BPT; ++j) hb_nx[j] = gb[j] = bb[j] = cb[j] = 0.0;
  for (int64_t k = 0; k < nseg; ++k) {
    const int64_t s = nseg - 1 - k;
    if (!wait_flag(ready, (int32_t)(k + 1), c.flags + 2, v.flag)) return;
    const int64_t hi = (s * c.K + c.K < c.T) ? s * c.K + c.K : c.T;
    const int t = topo_of(c.topo + it.topo, it.n_topo, hi);
    load_coefs<BS, BPT>(c, it, t, L.g, L.be);
    select_factor<BS, DT, SM>(c, it, v, t, w);
    step_barrier<BS>();
    const int64_t o = it.seg + (k & 1) * seg_len;
    reverse_segment<BS, BPT, DT, SM, GEN>(c, it, v, L, w, s, t, c.seg_i + o, rows_of(k), hb_nx, gb, bb, cb, dJ);
    publish_flag(done, (int32_t)(k + 1));
  }
  store_branch_adjoints<BS, BPT>(c, it, gb, bb, cb);
}

}  // namespace step
}  // namespace emt
