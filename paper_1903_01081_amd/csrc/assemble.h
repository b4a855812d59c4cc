// Device code shared by the numeric kernels: assembly of a component's
// conductance matrix on its symbolic pattern.
#pragma once

#include <hip/hip_runtime.h>

#include "device.h"

namespace emt {

// G of one (item, topology), row by row from the node CSR in a fixed order:
// its strictly lower entries at L's row positions (Lr), its diagonal in D.
// STATIC leaves out diodes and controlled switches, whose conductances follow
// their state. The caller places the barrier.
template <int BS, bool STATIC = false>
__device__ __forceinline__ void assemble_g(const DevCtx &c, const ItemDesc &it, const SymDesc &sd, int t, double *Lr,
                                           double *D) {
  const int32_t *rowptr = c.symi + sd.rowptr;
  const int32_t *nptr = c.nptr + it.nptr;
  const uint16_t *nent = c.nent + it.nent;
  const double *g = c.cg + it.coef + (int64_t)t * it.n_br;
  const int32_t *bk = c.bk + it.br, *bm = c.bm + it.br, *gpos = c.bgpos + it.br;
  for (int r = threadIdx.x; r < it.n; r += BS) {
    for (int q = rowptr[r]; q < rowptr[r + 1]; ++q) Lr[q] = 0.0;
    double d = 0.0;
    for (int e = nptr[r]; e < nptr[r + 1]; ++e) {
      const int ent = nent[e];
      const int b = ent >> 1;
      double gv = g[b];
      if constexpr (STATIC) {
        const int kind = c.bkind[it.br + b];
        if (kind == KIND_DIODE || kind == KIND_CSWITCH) gv = 0.0;
      }
      d = d + gv;
      const int other = (ent & 1) ? bk[b] : bm[b];
      if (other >= 0 && other < r) Lr[gpos[b]] = Lr[gpos[b]] - gv;
    }
    D[r] = d;
    if (it.n_groups > 0) {
      // mutual conductances of coupled groups: +g_o between like terminals
      // of two members, -g_o between a k and an m terminal
      const int32_t *mp = c.mptr + it.mptr;
      const int32_t *me = c.ment + it.ment;
      const double *go = c.cgo + it.coef + (int64_t)t * it.n_br;
      for (int e = mp[r]; e < mp[r + 1]; ++e) {
        const int pos = me[2 * e], code = me[2 * e + 1];
        const double v = go[code >> 1];
        Lr[pos] = (code & 1) ? Lr[pos] - v : Lr[pos] + v;
      }
    }
  }
}

}  // namespace emt
