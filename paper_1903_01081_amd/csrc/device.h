// Device-side data layout shared by the kernels and the host code that
// uploads it. Everything is flattened into a few big arrays addressed by
// per-item offsets (structure of arrays; one work item = one connected
// component of one scenario).
#pragma once

#include <cstdint>

namespace emt {

enum : int {
  KIND_RL = 0, KIND_C = 1, KIND_R = 2, KIND_SWITCH = 3, KIND_SRC = 4, KIND_LINE = 5, KIND_DIODE = 6, KIND_CSWITCH = 7
};

// Packed branch descriptor for the step kernels: local terminals in 15 bits
// each (a grounded terminal holds the node count n: the step kernels keep a
// zero at x[n]) and the history-coefficient class in 2 bits: gamma = g (R-L
// and sources), -g (capacitors) or 0 (resistors, switches), or a branch
// whose history a pass after the branch update writes into its injection
// (a line end: the other end's travelling wave; a member of a coupled
// group: its circulant companion with the other members' currents and
// voltages).
constexpr uint32_t kTermGround = 0x7FFF;  // mask of one packed terminal
constexpr int kMaxItemNodes = 0x7FFF;
enum : uint32_t { GAMMA_PLUS_G = 0, GAMMA_MINUS_G = 1, GAMMA_ZERO = 2, GAMMA_PASS = 3 };

// A set of row sums as the step kernels run it (closed.h): offsets of its
// batch table in DevCtx::symi and of its codes and row ids in DevCtx::symh.
struct RowProg {
  int32_t nb, nq;           // batches, quads
  int64_t meta, code, row;  // int32 [waves + 1 + nb]; uint16 [nq][64][4]; uint16 [nb][64]
};

// Symbolic factor and sweep plan (shared by isomorphic items). Offsets index
// DevCtx::symi (int32) or DevCtx::symh (uint16).
struct SymDesc {
  int32_t n, d, ns, nnz;        // nodes, dense-tail size, leading size, nonzeros of L
  int32_t nsv, nfpass, nbpass, nlev;  // sweep entries, sweep passes, factor levels
  // row descriptors of the passes; backward levels; closed-form solve (0: level passes; 2: with diodes or controlled
  // switches, whose tail matrix, without them, is kept instead of its inverse)
  int32_t nfdesc, nbdesc, nlevb, closed;
  // int32 (symi): full factor structure for the numeric factorisation
  int64_t rowptr, rowcol, colptr, colrow, colpos, flevptr, flevrows, fentptr, fent;
  // int32 (symi): backward levels over all n rows (explicit inverse)
  int64_t blevptr, blevrows;
  // int32 (symi): sweep plan: sv entry -> L entry; per pass (first row
  // descriptor, log2 lanes per row) pairs, nfpass+1 / nbpass+1 of them
  int64_t svmap, fpass, bpass;
  // uint16 (symh): sweep plan
  int64_t fcol, brow, bpos;
  // uint64 (symd): row descriptors (row | first << 16 | count << 32)
  int64_t fdesc, bdesc;
  // int32 (symi), symbolics refactorised inside the time loop (else -1):
  // per level entry (in fent order) its CSR position and the start of its
  // update pairs, nnz+1 of them; the pairs (qi | qj << 16), the CSR
  // positions of L_ik and L_jk for every column k < j common to rows i and j
  int64_t rent, rpair;
  // closed-form solve (closed != 0; then nsv counts the values of the row
  // programs, 256 per quad, forward then backward): the programs, and for
  // the numeric kernel the plan's lists (closed.h) in symi
  RowProg fwd, bwd;
  int32_t ncl, n_n, n_q, nq_off, ns_off, ns_key;
  int64_t cluster, q_diag, q_off, n_ptr, n_adj, n_grp, n_col, s_off, s_key, s_ptr, s_term;
  int64_t vsrc;  // [nsv] value index of every program value
};

struct ItemDesc {
  int32_t scen, sym, n, n_br, n_src, n_topo, n_rec, n_lines;
  int64_t br;    // per-branch arrays
  int64_t coef;  // coefficient arrays [n_topo][n_br] (g, beta, in-service)
  int64_t nptr;  // node CSR pointers [n+1] (int32); also recorded-node pointers rptr
  int64_t nent;  // node CSR entries (uint16: local branch << 1 | end-is-m)
  RowProg gf, ga;  // injection sums per node, forward and adjoint (codes: J entry << 1 | negative)
  int64_t node;  // per-node state [n]
  int64_t fac;   // full L values [n_topo][nnz] (factorisation work)
  int64_t dfac;  // pivots D and 1/D [n_topo][n]
  int64_t sv;    // sweep values [n_topo][nsv]
  int64_t w;     // tail inverse [n_topo][d*d]
  int64_t rec;   // recorded pairs (uint16 local node, uint16 column) [n_rec]
  int64_t topo;  // scenario topology start steps [n_topo]
  int64_t ck;    // checkpoints (i, u) [n_ck][n_br]
  int64_t seg;   // adjoint segment buffer (i of each step) [K][n_br]
  int64_t vt;    // adjoint: trajectory rows (node voltages, then the sources' EMFs) [T or K][n + n_src]
  int64_t lines; // distributed-parameter lines: first entry of line_tab / line_gf
  int32_t n_groups, n_real;  // coupled three-phase groups; branches before the padding to whole slots
  int64_t groups;  // first entry of group_tab
  int64_t mptr;    // mutual stamps by row of L [n+1] (int32), into ment
  int64_t ment;    // mutual stamps: (L position, local branch << 1 | negative) pairs (int32)
  int32_t n_diodes, pad3;  // ideal diodes (state-dependent switches)
  // closed form with switches: their table, and the entries of the tail's
  // matrix they stamp: a * d + b, first term; terms (index << 1 | negative)
  int64_t swt, swkey, swptr, swterm;
  int32_t n_swkey, pad4;
  int64_t dyn;     // items with diodes: the factor refreshed inside the time loop, in DevCtx::dyn:
                   // current conductances [n_br], L [nnz], D [n], sweep values [nsv], 1/D [n]
};

// LDS of a step kernel's workgroup: byte offsets of its arrays (each 16-byte
// aligned) and their total, the same on the host and on the device.
struct StepShape {
  int n, d, ns, nbr, nsrc, nrec, closed, nfpass, nbpass, nsv, nfdesc, nbdesc;
  int gb, gq, fb, fq, bb, bq;  // batches and quads of the gather, forward and backward programs
  // factor levels and (where staged) node-CSR entries of an item refactorised inside the loop, else 0
  int nlev, nent;
  int nsw, line;               // closed form with switches: their number, doubles of the tail inversion's lines
  int bs;
  // adjoint: the earlier step's trajectory row is read from memory; the
  // recorded columns' cotangents are, and EMFs are evaluated step by step
  int row_global, seeds_global;
};
struct StepLds {
  uint32_t cD, xr, J, flag, emf, vrow, pass, sv, dinv, fdesc, bdesc, fcol, brow, bpos, gmeta, gcode, grow, fmeta, fcode,
      frow, bmeta, bcode, brw, rnode, rcolumn, rf_rowptr, rf_flev, rf_fent, rf_rows, rf_nptr, rf_nent, line, gsw, swflag, total;
};
inline
#ifdef __HIPCC__
    __host__ __device__
#endif
        StepLds step_lds(const StepShape &s, bool sm, bool adjoint) {
  StepLds o{};
  uint32_t at = 0;
  auto take = [&at](int cnt, int size) {
    const uint32_t r = at;
    at += ((uint32_t)cnt * (uint32_t)size + 15u) & ~15u;
    return r;
  };
  const int waves = s.bs / 64;
  o.cD = take((s.d + 31) / 32 * 32, 8);               // the tail's right-hand side, zero past d
  o.xr = take((s.closed ? 2 : 1) * (s.n + 1), 8);     // right-hand side (closed form), then the solution
  o.J = take(s.nbr + 1 + (adjoint && !s.seeds_global ? s.nrec : 0), 8);  // branch injections, a zero, the adjoint's seeds
  o.flag = take(adjoint ? 1 : 0, 4);
  o.emf = take(s.nsrc > 0 && !(adjoint && s.seeds_global) ? s.bs : 0, 8);
  o.line = take(s.line, 8);
  o.gsw = take(s.nsw, 8);
  o.swflag = take(s.nsw > 0 || s.nlev > 0 ? 1 : 0, 4);
  o.vrow = take(adjoint && !s.row_global ? s.n + 1 + s.nsrc : 0, 8);  // the earlier step's trajectory row, a zero between its parts
  if (sm) {
    o.gmeta = take(waves + 1 + s.gb, 4);
    o.gcode = take(s.gq * 256, 2);
    o.grow = take(s.gb * 64, 2);
    o.sv = take(s.nsv, 8);
    if (s.closed) {
      o.fmeta = take(waves + 1 + s.fb, 4);
      o.fcode = take(s.fq * 256, 2);
      o.frow = take(s.fb * 64, 2);
      o.bmeta = take(waves + 1 + s.bb, 4);
      o.bcode = take(s.bq * 256, 2);
      o.brw = take(s.bb * 64, 2);
    } else {
      o.pass = take(2 * (s.nfpass + s.nbpass + 2), 4);
      o.dinv = take(s.ns, 8);
      o.fdesc = take(s.nfdesc, 8);
      o.bdesc = take(s.nbdesc, 8);
      o.fcol = take(s.nsv, 2);
      o.brow = take(s.nsv, 2);
      o.bpos = take(s.nsv, 2);
    }
    o.rnode = take(s.nrec, 2);
    o.rcolumn = take(s.nrec, 2);
    if (s.nlev > 0) {
      o.rf_rowptr = take(s.n + 1, 4);
      o.rf_flev = take(s.nlev + 1, 4);
      o.rf_fent = take(s.nlev + 1, 4);
      o.rf_rows = take(s.n, 2);
      o.rf_nptr = take(s.nent > 0 ? s.n + 1 : 0, 4);
      o.rf_nent = take(s.nent, 2);
    }
  }
  o.total = at;
  return o;
}

// What the components of a batch need besides the closed-form solve: a
// forward kernel exists per kind.
enum StepKind : int {
  STEP_PLAIN = 0,   // nothing
  STEP_LINES = 1,   // distributed-parameter lines
  STEP_GROUPS = 2,  // coupled three-phase groups
  STEP_FULL = 3,    // several of these, or level passes with one (in-loop LDL^T of diodes and controlled switches)
  STEP_SWITCH = 4,  // diodes or controlled switches, closed form
  STEP_LEVELS = 5,  // level passes, every component
};
// The same of the adjoint's kernels (batches without lines, groups and
// switches).
enum AdjointKind : int {
  ADJ_PLAIN = 0,    // closed form, trajectory rows of the whole horizon kept
  ADJ_GENERAL = 1,  // any solve, segments run again where the rows are not kept
  ADJ_LEVELS = 2,   // level passes, every component; rows kept or not
};

// One diode or controlled switch of a closed-form item: its local branch, its
// terminals and a controlled switch's measured nodes (local; the ground is the
// item's zero node slot n).
struct SwitchDesc {
  int32_t br, k, m, a, b, control;
};

// One coupled three-phase group: its members' local branches and terminals
// (a grounded terminal is the item's zero node slot n) and the sign of its
// Gamma (+1: R-L, Gamma = G; -1: C, Gamma = -G).
struct GroupDesc {
  int32_t b[3], k[3], m[3], sgn;
};

// One distributed-parameter line: its two local branches (k end, m end),
// their local nodes, the integer part D0 of tau / dt and its ring of waves.
// A ring has mask + 1 slots, a power of two >= D0 + 2; the entry of step n
// (the waves leaving the k and the m end, 16 bytes) sits in slot n & mask.
// The rings of an item's lines of one length are interleaved: slot s of a
// line is at ring + 2 stride s doubles in DevCtx::ring, stride lines apart.
struct LineDesc {
  int32_t bk, bm, nk, nm, d0, mask, stride, pad;
  int64_t ring;
};

// Components too large for one workgroup's dense tail, solved with their
// whole inverse G^{-1} split by columns over P workgroups ("tiles"), each
// tile holding rt (16 or 32) columns in VGPRs. Per step a tile forms the
// right-hand side of its own nodes, multiplies it into a partial voltage
// vector for every node, writes that with a step tag, and sums the P
// partials of the nodes its branches touch once their tags are current.
constexpr int kSplitColsMax = 32;
constexpr int kSplitBS = 512;
// Most partials one lane sums for a node: a component has at most
// 2048 / rt tiles, and the lanes per node are raised until each lane's share
// fits (smaller for 32-column tiles, whose weight cache fills the registers).
constexpr int split_max_partials(int rt) { return rt >= 32 ? 8 : 16; }
// Exchange buffer layout: the partials of kSplitRowBlock consecutive nodes
// are interleaved per tile ([node / 4][tile][node % 4]), so one wave's
// stores of consecutive nodes land in 32-byte runs (a quarter of the
// memory transactions of one node per row) while a node's P partials still
// span few cache lines. Rows are padded to a multiple of kSplitRowBlock.
constexpr int kSplitRowBlock = 4;
constexpr int split_rows_padded(int n) { return (n + kSplitRowBlock - 1) / kSplitRowBlock * kSplitRowBlock; }

struct SplitItem {
  int32_t item, P, cb, rt;   // item, tiles, inverse columns per workgroup of k_inverse, columns per tile
  int32_t lq_lg;             // log2 of the lanes that sum one node's partials (same in every tile)
  int32_t t0;                // index of its first tile (its tiles are t0 .. t0 + P - 1)
  int64_t pos;               // SplitCtx::i32: [n] tile position of each column (tile * rt + k)
  int64_t gt;                // SplitCtx::gt: [n_topo][P][rt][n] inverse columns
  int64_t xbuf;              // SplitCtx::xbuf: [2][n4 / 4][Pp][4] tagged partial voltages (Pp = P rounded up
                             // to 8, n4 = n rounded up to 4)
};

struct SplitTile {
  int32_t sitem, p, cnt, nn;  // split item, tile index, owned columns, needed nodes (owned first)
  int32_t nsrc, nrec, ne, pad;  // sources (first tile slots), owned recorded nodes, owned-node CSR entries
  int64_t need;   // i32: [nn] item-local node of each slot
  int64_t br;     // i32: [kSplitBS * bpt] item-local branch | writer << 30 (-1 = padding)
  int64_t bpack;  // u32: [kSplitBS * bpt] slot terminals (ground = nn) | gamma class << 30
  int64_t nptr;   // i32: [cnt + 1] owned-node CSR of branch ends
  int64_t nent;   // u16: (tile slot << 1 | end is m)
  int64_t rec;    // u32: slot | output column << 16
};

struct SplitCtx {
  const SplitItem *items;
  const SplitTile *tiles;
  const int32_t *blk;  // [grid] tile of each workgroup, -1 = none (workgroup b runs on XCD b mod n_xcc)
  const int32_t *i32;
  const uint32_t *u32;
  const uint16_t *u16;
  double *gt, *xbuf;
  int32_t *err;  // set when a tile gives up waiting (the launch then ends early)
  int32_t *xcc;  // [n_tiles] XCD each tile ran on in the last launch (-1 before it starts)
  int32_t allow_local;  // 0: always exchange through device-coherent memory
};

// Everything a kernel needs, passed by value.
struct DevCtx {
  const ItemDesc *items;
  const SymDesc *syms;
  const int32_t *symi;
  const uint16_t *symh;
  const uint64_t *symd;
  // per item-branch arrays (ItemDesc::br + local branch)
  const uint32_t *bpack;
  const int32_t *bk, *bm, *bkind, *bline, *bgpos;
  const double *bE, *bw, *bph;
  double *bR, *bL, *bC;
  double *si, *su;             // branch state i, u
  double *gbar, *bbar, *cbar;  // adjoint accumulators
  // coefficients (ItemDesc::coef + t * n_br + b)
  double *cg, *cb;
  const uint8_t *cins;
  // node data
  const int32_t *nptr, *rptr;  // node CSR and recorded-column pointers (ItemDesc::nptr)
  const uint16_t *nent;        // (ItemDesc::nent)
  const uint16_t *rnode, *rcolumn;  // (ItemDesc::rec)
  double *sv_state;            // node voltages (ItemDesc::node)
  // numeric factors
  double *lfull, *dpiv, *dinv, *svals, *wtail;
  const int64_t *topo;
  double *ck_i, *ck_u, *seg_i;
  // trajectory rows: of every step, written by the forward run (vt_full), or
  // of one checkpoint segment, written by its recomputation; null without
  // checkpoints
  double *vt;
  int32_t vt_full;
  // 1: no room in the LDS for a trajectory row beside the largest component's
  // arrays (the adjoint's kernels without staged factors only)
  int32_t row_global;
  // 1: nor for the recorded columns' cotangents and the EMF table, or a node's
  // columns are too many for the adjoint's row sums; the cotangents are then
  // added from memory and EMFs evaluated every step (in the same kernels)
  int32_t seeds_global;
  int32_t *flags;  // [0] = bad pivots
  double dt;
  int64_t T;
  int32_t K;
  int32_t rec_stride;
  int32_t sv_cap;  // closed-form values per item staged in LDS at most (a multiple of 256)
  // 1: no room in the LDS for the node CSR of items refactorised inside the
  // loop beside their other staged arrays
  int32_t csr_global;
  // distributed-parameter lines (ItemDesc::lines + q): descriptor, (1/Z,
  // fractional delay f) pairs, and the wave rings
  const LineDesc *line_tab;
  const double *line_gf;
  double *ring;
  // coupled groups: descriptors, mutual stamps, per-branch mutual values and
  // member flags, and the mutual companion coefficients g_o, beta_o per
  // (topology, branch) beside cg, cb
  const GroupDesc *group_tab;
  const int32_t *mptr, *ment;
  const double *bRm, *bLm, *bCm;
  const int32_t *bgrp;
  double *cgo, *cbo;
  // ideal diodes and controlled switches: the dynamic factor slots and the
  // conducting state per branch (meaningful for those branches)
  double *dyn;
  int32_t *dstate;
  // controlled switches: per item-branch the measured node pair, item-local
  // (the ground is the item's zero node slot n); null when there is none
  const int32_t *bmeas;
  const SwitchDesc *sw_tab;  // ItemDesc::swt + q
};

}  // namespace emt
