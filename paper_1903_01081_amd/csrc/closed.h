// Host-side plan of the closed-form solve of a component (no device code).
//
// The elimination order is cut at d nodes from its end: the trailing block D
// (the dense tail) separates the leading nodes S into small clusters, the
// connected pieces of the graph on S. With Q = G_SS^-1 (one small dense block
// per cluster), N = -G_DS Q and W = (G_DD + N G_SD)^-1, the solution of
// G x = r is
//   c = r_D + N r_S,   x_D = W c,   x_S = Q r_S + N^T x_D,
// three steps of independent rows in place of the level-scheduled sweeps
// (one per level of the elimination tree, up and down).
#pragma once

#include <cstdint>
#include <vector>

#include "analysis.h"

namespace emt {

// A set of row sums as the step kernels run it: rows are grouped into
// batches; one wave runs one batch at a time, 2^lg adjacent lanes (lg <= 4)
// sharing a row. A lane's share is a whole number of quads (four entries),
// padded with pad entries.
//   meta   [waves + 1] first batch of each wave, then per batch
//          first quad | quads << 16 | lg << 24
//   code   [quads][64][4]  what each entry multiplies or adds
//   row    [batches][64]   the row a lane writes (the last lane of each
//          group), 0xFFFF: none
//   src    [quads][2][64][2]  index of each entry's value (row sums with
//          values: the order the kernels read them in)
struct RowProgram {
  int batches = 0, quads = 0;
  std::vector<int32_t> meta, src;
  std::vector<uint16_t> code, row;
  std::vector<int> lg;  // log2 of the lanes that share each row given
};

struct RowSum {
  int row = 0;
  std::vector<std::pair<int, int>> e;  // (code, value index)
};

// Most entries of a row: a batch word counts a lane's quads in 8 bits and at
// most 16 lanes share a row. Wider counts cost every batch of every step their
// decoding (400-bus grid, 2000 steps: 5.40 -> 5.55 ms); a row is longer only
// where a node is recorded in more columns than that.
constexpr int kMaxRowEntries = 255 * 4 * 16;

// Throws Error (EMT_EINVAL) on a longer row. lg: the lanes of each row as in
// another program whose rows begin with the same entries, so that these meet
// in the same order and entries of value zero after them change no sum.
RowProgram schedule_rows(const std::vector<RowSum> &rows, int lanes, int pad_code, int pad_src,
                         const std::vector<int> *lg = nullptr);

// Sizes of the closed form at one cut.
struct ClosedSize {
  int64_t q = 0, nn = 0;  // entries of Q (all of each cluster's block) and of N
};

// Value indices of a plan: 0 is the constant 0, 1 the constant 1, then N,
// then Q.
struct ClosedPlan {
  int d = 0, ns = 0, n_n = 0, n_q = 0;
  int value_n(int e) const { return 2 + e; }
  int value_q(int e) const { return 2 + n_n + e; }
  // clusters: (nodes, first entry of Q), largest first
  std::vector<int32_t> cluster;
  // G_SS into Q: per leading node its diagonal entry; (L position, entry)
  // pairs, both triangles
  std::vector<int32_t> q_diag, q_off;
  // N, grouped by (row of D, cluster): per group the first of its (L
  // position, first entry of Q's row) pairs; per entry its group and column
  std::vector<int32_t> n_ptr, n_adj, n_grp, n_col;
  // the Schur complement's off-diagonal G_DD: (L position, a * d + b), both
  // triangles; and per entry N reaches: a * d + b, its first term; terms
  // (entry of N, L position)
  std::vector<int32_t> s_off, s_key, s_ptr, s_term;
  RowProgram fwd, bwd;
};

// Entries of the closed form for every cut d = 0 .. dmax.
std::vector<ClosedSize> closed_sizes(const Symbolic &S, int dmax);

// The plan at cut d for a workgroup of `lanes`; gpos: the positions in L's
// row structure that hold an entry of G. Codes index the right-hand side
// (node) and, past n + 1, the solution; n is the always-zero slot.
ClosedPlan plan_closed(const Symbolic &S, const std::vector<int> &gpos, int d, int lanes);

}  // namespace emt
